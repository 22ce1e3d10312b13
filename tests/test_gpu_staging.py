"""How a call's work lists reach the device: a call waits for the staging of its own upload only, a
workspace off a 16-byte boundary is served by a copy, a captured call carries its lists in the graph."""
import pytest

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


def _batch(seed, reqs=((1, 1, 300), (0, 77, 19), (1, 1, 1200))):
    from paper_2511_04791_amd import workloads as wl
    b = wl.make_batch(wl.LLAMA3_8B, list(reqs), page_seed=seed)
    q, kc, vc = wl.make_tensors(b, seed, device="cuda")
    return b, (q, kc, vc, torch.as_tensor(b.page_table, device="cuda"))


def test_a_call_far_ahead_waits_for_its_own_stream_only(ctx):
    """The fifth call behind a slow stream reuses the first one's staging buffer; it returns once that
    upload has run, however long another stream stays busy."""
    b, x = _batch(1)
    ctx.attn_mixed_batch(*x, b.seq_meta)
    t0, t1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    t0.record()
    torch.cuda._sleep(20_000_000)
    t1.record()
    torch.cuda.synchronize()
    cycles = int(20_000_000 * 400 / t0.elapsed_time(t1))  # of 0.4 s
    slow, other = torch.cuda.Stream(), torch.cuda.Stream()
    with torch.cuda.stream(other):
        for _ in range(20):  # 8 s
            torch.cuda._sleep(cycles)
        busy = torch.cuda.Event()
        busy.record()
    with torch.cuda.stream(slow):
        for _ in range(14):  # 5.6 s
            torch.cuda._sleep(cycles)
        outs = [ctx.attn_mixed_batch(*x, b.seq_meta) for _ in range(5)]
    assert not busy.query()
    torch.cuda.synchronize()
    assert all(torch.equal(o, outs[0]) for o in outs)


def test_workspace_off_a_16_byte_boundary(ctx):
    """Served by a copy command: same bits, also when more calls are queued than there are staging buffers."""
    import paper_2511_04791_amd as duet
    cases = [_batch(2), _batch(3, ((1, 1, 4000), (1, 1, 16), (0, 200, 0))), _batch(4, ((1, 1, 900),) * 5)]
    want = [ctx.attn_mixed_batch(*x, b.seq_meta) for b, x in cases]
    need = max(duet.workspace_bytes(duet.shape_of(x[0], x[1]), b.seq_meta) for b, x in cases)
    ws = torch.empty(need + 16, dtype=torch.uint8, device="cuda")[8:]
    assert ws.data_ptr() % 16 == 8
    got = [ctx.attn_mixed_batch(*x, b.seq_meta, workspace=ws) for _ in range(3) for b, x in cases]
    torch.cuda.synchronize()
    for i, g in enumerate(got):
        assert torch.equal(g, want[i % len(cases)]), i


@pytest.mark.parametrize("noalloc", [True, False])
def test_a_captured_call_replays_after_other_calls(ctx, noalloc):
    """Replays between eager calls of other batches, which reuse every staging buffer, give the captured
    batch's result for the queries of the moment.  Lists shorter and longer than one launch carries."""
    import paper_2511_04791_amd as duet
    for reqs in (((1, 1, 300), (0, 77, 19), (1, 1, 1200)), ((1, 1, 3000),) * 60 + ((0, 300, 100),)):
        b, (q, kc, vc, pt) = _batch(5, reqs)
        others = [_batch(6, ((1, 1, 4000), (0, 900, 40))), _batch(7, ((1, 1, 40),) * 9)]
        ws = torch.empty(duet.workspace_bytes(duet.shape_of(q, kc), b.seq_meta), dtype=torch.uint8, device="cuda")
        out = torch.empty_like(q)

        def call():
            if noalloc:
                return ctx.attn_mixed_batch_noalloc(q, kc, vc, pt, b.seq_meta, out=out)
            return ctx.attn_mixed_batch(q, kc, vc, pt, b.seq_meta, out=out, workspace=ws)

        call()
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            call()
        for seed in range(4):
            q.copy_(torch.randn(q.shape, generator=torch.Generator().manual_seed(seed)).to(q.dtype))
            want = ctx.attn_mixed_batch(q, kc, vc, pt, b.seq_meta)
            for ob, ox in others * 3:
                ctx.attn_mixed_batch(*ox, ob.seq_meta)
            out.fill_(float("nan"))
            graph.replay()
            torch.cuda.synchronize()
            assert torch.equal(out, want), (len(reqs), seed)
