"""GPU parity of prefill units cut into many pieces: up to six are merged by the last piece to finish, a
batch with more by a kernel of their own, both against the fp64 oracle and bit for bit across CU splits."""
import pytest

from _helpers import BF16_MAX_ABS, BF16_MEAN_ABS, errors, oracle_out, rows_of

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
    # name: (heads, kv heads, head dim), requests.  Pieces hold 8 tiles of 64 keys here.
    "6 and 7 pieces": ((8, 2, 128), [(0, 40, 3000), (0, 40, 3500)]),
    "7 pieces, every head alone": ((3, 3, 128), [(0, 257, 3300)]),
    "16 pieces, heads of 64": ((16, 2, 64), [(0, 70, 8000)]),
    "1, 2 and 7 pieces": ((8, 2, 128), [(0, 90, 0), (0, 64, 900), (0, 40, 3500)]),
    "2 to 6 pieces": ((12, 4, 128), [(0, 300, 700), (0, 40, 2900)]),
    "25 pieces, group of 2": ((4, 2, 64), [(0, 1, 12799), (0, 33, 12500)]),
    "rows of a wave before the last piece": ((8, 1, 128), [(0, 64, 4060)]),
    "beside decodes": ((8, 2, 128), [(1, 1, 700), (1, 1, 3), (0, 90, 6000)]),
    "beside streamed decodes": ((8, 2, 64), [(1, 1, 2999)] * 60 + [(0, 90, 6000)]),
}


@pytest.mark.parametrize("name", list(CASES))
def test_many_pieces(ctx, name):
    import paper_2511_04791_amd as duet
    from paper_2511_04791_amd import workloads as wl
    heads, reqs = CASES[name]
    b = wl.make_batch(wl.AttnShape(*heads, "bf16"), reqs, page_seed=700)
    q, kc, vc = (t.cuda() for t in wl.make_tensors(b, 7000, scale=1.0))
    pt = torch.as_tensor(b.page_table, device="cuda")
    out = ctx.attn_mixed_batch(q, kc, vc, pt, b.seq_meta, check_errors=True)
    for sp in (duet.CuSplit.split(96, 160), duet.CuSplit.split(224, 32), duet.CuSplit.agg()):
        other = ctx.attn_mixed_batch(q, kc, vc, pt, b.seq_meta, sp, check_errors=True)
        torch.cuda.synchronize()
        assert torch.equal(out, other), str(sp)
    mx, mean = errors(out, oracle_out(b, q, kc, vc))
    print(f"[parity] pieces, {name}: max_abs={mx:.3e} mean_abs={mean:.3e}", flush=True)
    assert mx <= BF16_MAX_ABS and mean <= BF16_MEAN_ABS


def test_many_pieces_beside_the_tail_split(ctx):
    """Units of eight pieces, merged by the kernel, beside 600 whole ones whose shortest 256 run as four
    pieces each and merge themselves."""
    import paper_2511_04791_amd as duet
    from paper_2511_04791_amd import workloads as wl
    b = wl.make_batch(wl.AttnShape(8, 2, 128, "bf16"), [(0, 1, 4200 + i % 9) for i in range(300)] + [(0, 16, 75000)],
                      page_seed=701)
    q, kc, vc = wl.make_tensors(b, 7001, scale=1.0, device="cuda")
    pt = torch.as_tensor(b.page_table, device="cuda")
    out = ctx.attn_mixed_batch(q, kc, vc, pt, b.seq_meta, check_errors=True)
    for _ in range(2):  # the arrival counters are ready for the next call
        other = ctx.attn_mixed_batch(q, kc, vc, pt, b.seq_meta, duet.CuSplit.split(96, 160), check_errors=True)
        torch.cuda.synchronize()
        assert torch.equal(out, other)
    some = [0, 7, 150, 299, 300]
    mx, mean = errors(out, oracle_out(b, q, kc, vc, some), rows_of(b, some))
    assert mx <= BF16_MAX_ABS and mean <= BF16_MEAN_ABS
