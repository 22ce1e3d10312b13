"""GPU parity of prefill with heads of 64, whose workgroups share a CU in pairs when every CU of the share gets two
items and a load of at least 5/4 of the longest: against the fp64 oracle, and bit for bit across the shares on both sides of that line."""
import pytest

from _helpers import BF16_MAX_ABS, BF16_MEAN_ABS, errors, oracle_out

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2511_04791_amd as duet
    c = duet.Context(0)
    yield c
    c.close()


CASES = {
    # name: (heads, kv heads, head dim), requests.  On 32 CUs pairs run from 64 items on.
    "62 items": ((16, 2, 64), [(0, 512, 256), (0, 480, 256)]),
    "64 items": ((16, 2, 64), [(0, 512, 256), (0, 512, 256)]),
    "64 items, one as long as the mean load": ((16, 2, 64), [(0, 512, 0), (0, 512, 0)]),
    "every head alone, ragged rows": ((12, 4, 64), [(0, 1301, 3), (0, 63, 61)]),
    "heads in twos, units that merge themselves": ((4, 2, 64), [(0, 300, 2500), (0, 257, 2300), (0, 129, 1)]),
    "heads in fours, more than six pieces": ((8, 2, 64), [(0, 33, 12500), (0, 70, 12001), (0, 1, 7999)]),
    "page ids that leave no room for a pair": ((8, 1, 64), [(0, 40, 65530), (0, 5, 0)]),
    "beside streamed decodes": ((16, 2, 64), [(1, 1, 2999)] * 60 + [(0, 700, 1500)]),
}


@pytest.mark.parametrize("name", list(CASES))
def test_pairs(ctx, name):
    import paper_2511_04791_amd as duet
    from paper_2511_04791_amd import workloads as wl
    heads, reqs = CASES[name]
    b = wl.make_batch(wl.AttnShape(*heads, "bf16"), reqs, page_seed=640)
    q, kc, vc = (t.cuda() for t in wl.make_tensors(b, 6400, scale=1.0))
    pt = torch.as_tensor(b.page_table, device="cuda")
    out = ctx.attn_mixed_batch(q, kc, vc, pt, b.seq_meta, duet.CuSplit.split(32, 224), check_errors=True)
    for sp in (duet.CuSplit.split(96, 160), duet.CuSplit.split(224, 32), duet.CuSplit.agg()):
        other = ctx.attn_mixed_batch(q, kc, vc, pt, b.seq_meta, sp, check_errors=True)
        torch.cuda.synchronize()
        assert torch.equal(out, other), str(sp)
    mx, mean = errors(out, oracle_out(b, q, kc, vc))
    print(f"[parity] heads of 64, {name}: max_abs={mx:.3e} mean_abs={mean:.3e}", flush=True)
    assert mx <= BF16_MAX_ABS and mean <= BF16_MEAN_ABS
