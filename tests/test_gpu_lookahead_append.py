"""Look-ahead decode with its cache writes ahead of the steps and its merges in the next layer's kernel, and
where neither may be: caches that layers share (a later layer writes over the rows an earlier one reads), and
key or value rows that an earlier step of the same call computes.  The reference runs the steps one at a time: the host writes the rows by index, then
duet_attn_iteration on the decode rows.  The same kernels on the same work lists, so every bit agrees.
"""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("alias", ["none", "caches", "rows"])
@pytest.mark.parametrize("kind", ["small", "streamed", "f32"])
@pytest.mark.parametrize("mode", ["agg", "split"])
def test_lookahead_rows_and_caches_in_use(mode, kind, alias):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2511_04791_amd as duet
    from paper_2511_04791_amd import workloads as wl
    shape, k, L = wl.TINY_F32 if kind == "f32" else wl.LLAMA3_8B, 4, 3
    # cached + 1 .. cached + 3 cross page boundaries (16 tokens) and, streamed, the ends of 256 and 512 token splits
    reqs = [(0, 33, 7), (1, 1, 14), (1, 1, 700), (1, 1, 31)]
    if kind == "streamed":  # more items than the small kernel takes
        reqs += [(1, 1, 254 + 128 * i % 1024) for i in range(12)]
    b = wl.make_batch(shape, reqs, page_seed=7101, reserve_tokens=k)
    n = (k - 1) * L
    qs, kcs, vcs, qa, ka, va = [], [], [], [None] * n, [None] * n, [None] * n
    for l in range(L):
        q, kc, vc = (t.cuda() for t in wl.make_tensors(b, 7200 + l, device="cpu"))
        qs.append(q), kcs.append(kc), vcs.append(vc)
        for dst, src in zip((qa, ka, va), wl.make_lookahead_tensors(b, k, 7300 + l, device="cpu")):
            for s in range(k - 1):
                dst[s * L + l] = src[s].cuda()
    if alias == "caches":
        kcs[2], vcs[2] = kcs[0], vcs[0]
    outs, outs_a = [torch.zeros_like(q) for q in qs], [torch.zeros_like(q) for q in qa]
    if alias == "rows":  # step s + 1 writes the first numbers that step s computed
        for x in range(L, len(ka)):
            ka[x] = outs_a[x - L].view(-1)[:ka[x].numel()].view_as(ka[x])
    seen = {}
    rk = [seen.setdefault(t.data_ptr(), t.clone()) for t in kcs]
    rv = [seen.setdefault(t.data_ptr(), t.clone()) for t in vcs]
    pt = torch.as_tensor(b.page_table, device="cuda")
    ctx = duet.Context(0)
    try:
        sp = duet.CuSplit.agg(k) if mode == "agg" else duet.CuSplit.split(96, 160, k)
        ctx.attn_lookahead(qs, qa, ka, va, kcs, vcs, pt, b.seq_meta, sp, outs=outs, outs_ahead=outs_a, check_errors=True)
        torch.cuda.synchronize()
        dec = [r for r in range(len(b.seq_meta)) if int(b.seq_meta[r][0]) == 1]
        dpt = pt[dec].contiguous()
        for s in range(k):
            meta = b.seq_meta[dec].copy()
            meta[:, 1], meta[:, 3] = range(len(dec)), meta[:, 3] + s
            for l in range(L):
                x = (s - 1) * L + l
                if s > 0:
                    for i, r in enumerate(dec):
                        pos = int(meta[i][3])
                        page = int(b.page_table[r][pos // 16])
                        rk[l][page, :, pos % 16, :] = ka[x][i]
                        rv[l][page, :, :, pos % 16] = va[x][i]
                rows = [int(b.seq_meta[r][1]) for r in dec]
                q = qs[l][rows].contiguous() if s == 0 else qa[x]
                want = ctx.attn_mixed_batch(q, rk[l], rv[l], dpt, meta, duet.CuSplit.agg())
                got = outs[l][rows] if s == 0 else outs_a[x]
                assert torch.equal(got, want), f"step {s} layer {l}"
        for got, want in zip(kcs + vcs, rk + rv):
            assert torch.equal(torch.nan_to_num(got.float()), torch.nan_to_num(want.float()))
    finally:
        ctx.close()


def test_merges_deferred_and_not():
    """17 requests of 32 heads: 544 pairs to merge are deferred into the next layer's kernel on 24 CUs and
    more, merged by a kernel of their own on 16 and 8.  Same bits."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2511_04791_amd as duet
    from paper_2511_04791_amd import workloads as wl
    k, L = 3, 3
    b = wl.make_batch(wl.LLAMA3_8B, [(1, 1, 500 + 90 * i) for i in range(17)], page_seed=7102, reserve_tokens=k)
    qs, kcs, vcs = zip(*[[t.cuda() for t in wl.make_tensors(b, 7400 + l, device="cpu")] for l in range(L)])
    ahead = [[t.cuda() for t in ts] for ts in wl.make_lookahead_tensors(b, k, 7500, device="cpu")]
    qa, ka, va = [[ts[s] for s in range(k - 1) for _ in range(L)] for ts in ahead]
    pt = torch.as_tensor(b.page_table, device="cuda")
    ctx = duet.Context(0)
    try:
        got = []
        for cus in (0, 128, 24, 16, 8):
            sp = duet.CuSplit.split(256 - cus, cus, k) if cus else duet.CuSplit.agg(k)
            outs, outs_a = ctx.attn_lookahead(list(qs), qa, ka, va, list(kcs), list(vcs), pt, b.seq_meta, sp, check_errors=True)
            torch.cuda.synchronize()
            got.append(torch.cat([t.flatten() for t in outs + outs_a]))
        assert torch.isfinite(got[0]).all()
        assert all(torch.equal(g, got[0]) for g in got[1:])
    finally:
        ctx.close()


def test_a_moved_chunk_replays_the_decode_graphs():
    """The decode launches of a call read nothing of its chunk: one token more of prefix (18 key tiles in
    place of 17, the same items) replays the graphs of the call before."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2511_04791_amd as duet
    from paper_2511_04791_amd import workloads as wl
    k = 3
    b = wl.make_batch(wl.LLAMA3_8B, [(0, 250, 1025), (1, 1, 700), (1, 1, 31)], page_seed=7103, reserve_tokens=k)
    q, kc, vc = (t.cuda() for t in wl.make_tensors(b, 7600, device="cpu"))
    qa, ka, va = ([t.cuda() for t in ts] for ts in wl.make_lookahead_tensors(b, k, 7601, device="cpu"))
    pt = torch.as_tensor(b.page_table, device="cuda")
    out, outs_a = torch.empty_like(q), [torch.empty_like(t) for t in qa]
    ctx = duet.Context(0)
    try:
        ws = torch.empty(2 * duet.lookahead_workspace_bytes(wl.LLAMA3_8B, b.seq_meta, k), dtype=torch.uint8, device="cuda")
        captured = []
        for prefix in (1024, 1025):
            meta = b.seq_meta.copy()
            meta[0, 3] = prefix
            ctx.attn_lookahead([q], qa, ka, va, [kc], [vc], pt, meta, duet.CuSplit.split(128, 128, k), outs=[out],
                               outs_ahead=outs_a, workspace=ws, check_errors=True)
            torch.cuda.synchronize()
            want = ctx.attn_mixed_batch(q, kc, vc, pt, meta)
            assert torch.equal(out, want)
            captured.append(ctx.decode_graph_stats()["captured"])
        assert captured[0] == captured[1] > 0
    finally:
        ctx.close()
