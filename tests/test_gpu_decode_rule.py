"""GPU parity of the bf16 decode kernels around the sizes where the decode rule changes the kernel.

The rule counts items of 32 pages (512 tokens): one workgroup per item (or per two or four short ones of a
long list) where no request has a second split or at most 96 items are there, streamed items of 16 pages up to 256 items, of 32 pages above.
Against the fp64 oracle with the bf16 bounds, and bit for bit across CU splits.
"""
import numpy as np
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


EDGES = [1, 15, 16, 17, 127, 128, 129, 255, 256, 257, 511, 512]  # tokens: waves, pages, a whole item
CASES = {
    # name: (heads, kv heads, head dim), contexts
    "one split": ((8, 2, 128), EDGES),
    "one split, d 64": ((16, 2, 64), EDGES),
    "one split, a head per group": ((4, 4, 128), EDGES),
    "one split, three heads": ((6, 2, 64), EDGES),
    "one split, sixteen heads": ((16, 1, 128), EDGES),
    "one split, many items": ((8, 2, 64), [200 + 7 * i % 311 for i in range(260)]),
    # short items that share a workgroup: 16 pages and fewer from 257 items on, 8 and fewer from 1024
    "256 short items": ((8, 8, 64), [1 + 9 * i % 300 for i in range(32)]),
    "pairs, an odd one": ((16, 1, 128), EDGES + [1 + 13 * i % 256 for i in range(245)]),
    "pairs only": ((8, 2, 128), [1 + 7 * i % 200 for i in range(130)]),
    "1023 items": ((6, 3, 64), [1 + 11 * i % 140 for i in range(341)]),
    "fours, one over": ((4, 4, 128), EDGES + [1 + 5 * i % 128 for i in range(245)]),
    "fours, two and three over": ((6, 2, 64), EDGES[3:] + [1 + 5 * i % 129 for i in range(508)]),
    "second split": ((8, 2, 128), EDGES + [513, 1024, 1025, 4000]),
    "96 items": ((8, 2, 128), [600] * 24),
    "97 items": ((8, 1, 128), [600] * 48 + [512]),
    "256 items, d 64": ((16, 2, 64), [513, 1000] * 32),
    "257 items": ((8, 1, 64), [513, 1023] * 64 + [77]),
    "one long request": ((16, 1, 128), [40000]),
}


@pytest.mark.parametrize("name", list(CASES))
def test_decode_rule_edges(ctx, name):
    import paper_2511_04791_amd as duet
    from paper_2511_04791_amd import workloads as wl
    heads, contexts = CASES[name]
    b = wl.make_batch(wl.AttnShape(*heads, "bf16"), [(1, 1, c - 1) for c in contexts], page_seed=300)
    q, kc, vc = (t.cuda() for t in wl.make_tensors(b, 5000, scale=1.0))  # scores of unit variance
    pt = torch.as_tensor(b.page_table, device="cuda")
    out = ctx.attn_mixed_batch(q, kc, vc, pt, b.seq_meta, check_errors=True)
    assert torch.isfinite(out).all()
    for sp in (duet.CuSplit.split(128, 128), duet.CuSplit.split(224, 32)):
        other = ctx.attn_mixed_batch(q, kc, vc, pt, b.seq_meta, sp, check_errors=True)
        torch.cuda.synchronize()
        assert torch.equal(out, other), str(sp)
    layers = ctx.attn_iteration([q, q], [kc, kc], [vc, vc], pt, b.seq_meta, check_errors=True)
    torch.cuda.synchronize()
    assert torch.equal(layers[0], out) and torch.equal(layers[1], out)
    mx, mean = errors(out, oracle_out(b, q, kc, vc))
    print(f"[parity] decode rule, {name}: max_abs={mx:.3e} mean_abs={mean:.3e}", flush=True)
    assert mx <= BF16_MAX_ABS and mean <= BF16_MEAN_ABS


def test_lookahead_steps_cross_the_rule(ctx):
    """Steps whose contexts grow from one split to two, and from 96 items to 97 and more: each step
    equals a call of its own over the same cache, bit for bit."""
    import paper_2511_04791_amd as duet
    from paper_2511_04791_amd import workloads as wl
    for heads, contexts in (((8, 2, 128), [509, 40, 511]), ((8, 2, 64), [1022] * 23 + [1023, 30])):
        k = 5
        b = wl.make_batch(wl.AttnShape(*heads, "bf16"), [(1, 1, c - 1) for c in contexts], page_seed=301,
                          reserve_tokens=k)
        q, kc, vc = (t.cuda() for t in wl.make_tensors(b, 5100, scale=1.0))
        qa, ka, va = wl.make_lookahead_tensors(b, k, 5101, device="cuda", scale=1.0)
        pt = torch.as_tensor(b.page_table, device="cuda")
        _, ahead = ctx.attn_lookahead([q], qa, ka, va, [kc], [vc], pt, b.seq_meta, duet.CuSplit.agg(k),
                                      check_errors=True)
        torch.cuda.synchronize()
        for s in range(1, k):
            meta = np.array(b.seq_meta)
            meta[:, 3] += s
            one = ctx.attn_mixed_batch(qa[s - 1], kc, vc, pt, meta, check_errors=True)
            torch.cuda.synchronize()
            assert torch.equal(one, ahead[s - 1]), f"step {s}"


def test_small_decode_bad_page_is_flagged(ctx):
    import paper_2511_04791_amd as duet
    from paper_2511_04791_amd import workloads as wl
    b = wl.make_batch(wl.AttnShape(8, 2, 128, "bf16"), [(1, 1, 300), (1, 1, 90)], page_seed=302)
    q, kc, vc = (t.cuda() for t in wl.make_tensors(b, 5200, scale=1.0))
    pt = torch.as_tensor(b.page_table, device="cuda")
    bad = pt.clone()
    bad[0, 9] = b.num_phys_pages
    with pytest.raises(duet.DuetError) as e:
        ctx.attn_mixed_batch(q, kc, vc, bad, b.seq_meta, check_errors=True)
    assert e.value.code == -6
    out = ctx.attn_mixed_batch(q, kc, vc, pt, b.seq_meta, check_errors=True)
    torch.cuda.synchronize()
    assert errors(out, oracle_out(b, q, kc, vc))[0] <= BF16_MAX_ABS


def test_short_items_beside_a_chunk(ctx):
    """Aggregated, items that share a workgroup run in one launch with the chunk: same bits as split."""
    import paper_2511_04791_amd as duet
    from paper_2511_04791_amd import workloads as wl
    for n in (130, 245):  # 260 and 490 items
        b = wl.make_batch(wl.AttnShape(8, 2, 128, "bf16"), [(1, 1, 3 * i % 300) for i in range(n)] + [(0, 300, 70)], page_seed=301)
        q, kc, vc = (t.cuda() for t in wl.make_tensors(b, 5001, scale=1.0))
        pt = torch.as_tensor(b.page_table, device="cuda")
        out = ctx.attn_mixed_batch(q, kc, vc, pt, b.seq_meta, check_errors=True)
        other = ctx.attn_mixed_batch(q, kc, vc, pt, b.seq_meta, duet.CuSplit.split(128, 128), check_errors=True)
        torch.cuda.synchronize()
        assert torch.equal(out, other)
        mx, mean = errors(out, oracle_out(b, q, kc, vc))
        assert mx <= BF16_MAX_ABS and mean <= BF16_MEAN_ABS
