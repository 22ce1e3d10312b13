"""GPU parity of the fp32 attention kernels at the edges of their tiles, against the fp64 oracle.

A prefill workgroup owns 16 queries of one head, its eight waves take every eighth page, and page
ids come 64 at a time (8192 tokens per round); a decode wave owns two pages, its 16 columns the
heads of a group.  Values are N(0, 1), so every output is a convex combination of values of at
most about 5, and fp32 sums of up to 16 products keep well inside the fp32 bound of 1e-5.
"""
import numpy as np
import pytest

from _helpers import F32_MAX_ABS, errors, oracle_out, to64

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


CASES = [
    # heads, kv heads, head dim; (kind, new tokens, cached tokens)
    ((4, 2, 64), [(0, 1, 0), (0, 15, 1), (0, 16, 0), (0, 17, 15), (1, 1, 0), (1, 1, 31), (1, 1, 32)]),
    ((4, 4, 128), [(0, 127, 3), (0, 128, 16), (0, 129, 0), (1, 1, 15), (1, 1, 16)]),     # a head per group
    ((6, 2, 64), [(0, 40, 500), (1, 1, 127), (1, 1, 600)]),                              # three heads
    ((16, 1, 128), [(0, 20, 111), (1, 1, 200)]),                                         # every column a head
    ((2, 1, 64), [(0, 3, 8190), (0, 18, 8300), (1, 1, 8191)]),                           # a second round of ids
]


@pytest.mark.parametrize("case", range(len(CASES)))
def test_f32_tile_edges(ctx, case):
    import paper_2511_04791_amd as duet
    from paper_2511_04791_amd import workloads as wl
    heads, reqs = CASES[case]
    b = wl.make_batch(wl.AttnShape(*heads, "f32"), reqs, page_seed=200 + case)
    q, kc, vc = (t.cuda() for t in wl.make_tensors(b, 4000 + case))
    pt = torch.as_tensor(b.page_table, device="cuda")
    out = ctx.attn_mixed_batch(q, kc, vc, pt, b.seq_meta, check_errors=True)
    other = ctx.attn_mixed_batch(q, kc, vc, pt, b.seq_meta, duet.CuSplit.split(64, 64), check_errors=True)
    torch.cuda.synchronize()
    assert torch.equal(out, other)
    mx, _ = errors(out, oracle_out(b, q, kc, vc))
    print(f"[parity] f32 edges {case}: max_abs={mx:.3e}", flush=True)
    assert mx <= F32_MAX_ABS


@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
def test_f32_later_values_do_not_reach_earlier_queries(ctx, bad):
    """A value that is not finite reaches the queries that attend its token and no others, also on
    the page that holds both."""
    from paper_2511_04791_amd import workloads as wl
    b = wl.make_batch(wl.AttnShape(4, 2, 64, "f32"), [(0, 40, 9)], page_seed=210)
    q, kc, vc = wl.make_tensors(b, 4100)
    token = 30                                                 # absolute position; query 21
    page, slot = int(b.page_table[0, token // 16]), token % 16
    pt = torch.as_tensor(b.page_table, device="cuda")
    want = ctx.attn_mixed_batch(q.cuda(), kc.cuda(), vc.cuda(), pt, b.seq_meta, check_errors=True)
    vc[page, 0, 5, slot] = bad
    out = ctx.attn_mixed_batch(q.cuda(), kc.cuda(), vc.cuda(), pt, b.seq_meta, check_errors=True)
    torch.cuda.synchronize()
    got, ref = to64(out), to64(want)
    assert np.abs(got[:21] - ref[:21]).max() <= F32_MAX_ABS    # queries before the token
    hit = got[21:, :2, 5]                                      # its dimension, the heads of its kv head
    assert not np.isfinite(hit).any()
    got[21:, :2, 5] = ref[21:, :2, 5]
    assert np.abs(got - ref).max() <= F32_MAX_ABS


def test_f32_bad_page_is_skipped_and_flagged(ctx):
    import paper_2511_04791_amd as duet
    from paper_2511_04791_amd import workloads as wl
    b = wl.make_batch(wl.AttnShape(4, 2, 64, "f32"), [(0, 40, 25), (1, 1, 90)], page_seed=211)
    q, kc, vc = (t.cuda() for t in wl.make_tensors(b, 4200))
    pt = torch.as_tensor(b.page_table, device="cuda")
    bad = pt.clone()
    bad[0, 1], bad[1, 2] = -5, b.num_phys_pages
    with pytest.raises(duet.DuetError) as e:
        ctx.attn_mixed_batch(q, kc, vc, bad, b.seq_meta, check_errors=True)
    assert e.value.code == -6
    out = ctx.attn_mixed_batch(q, kc, vc, pt, b.seq_meta, check_errors=True)  # the error word is cleared
    torch.cuda.synchronize()
    assert errors(out, oracle_out(b, q, kc, vc))[0] <= F32_MAX_ABS


def test_more_items_than_one_launch_holds(ctx):
    """More than 2^20 one-token requests: the grid of all of them would hold 2^32 threads.  A request
    without a prefix sees its own key only, so it returns that token's value."""
    import paper_2511_04791_amd as duet
    n, pages = (1 << 20) + 5, 1000
    g = torch.Generator(device="cuda").manual_seed(7)
    q = torch.randn(n, 1, 64, device="cuda", generator=g)
    kc, vc = torch.randn(pages, 1, 16, 64, device="cuda", generator=g), torch.randn(pages, 1, 64, 16, device="cuda", generator=g)
    pt = torch.randint(0, pages, (n, 1), device="cuda", generator=g, dtype=torch.int32)
    meta = np.zeros((n, 4), np.int32)
    meta[:, 1], meta[:, 2] = np.arange(n), 1
    c = duet.Context(0)  # its grown staging buffer goes with it
    try:
        out = c.attn_mixed_batch(q, kc, vc, pt, meta, check_errors=True)
        torch.cuda.synchronize()
    finally:
        c.close()
    assert torch.equal(out[:, 0], vc[pt[:, 0].long(), 0, :, 0])
