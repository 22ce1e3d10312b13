"""Aggregated bf16 layers whose two halves run in one launch: bit for bit the outputs of the separate
kernels (per-kernel profiling keeps those), over every kind of decode work and head layout."""
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


def _dec(n, *lens):
    return [(1, 1, lens[i % len(lens)] - 1) for i in range(n)]


CASES = {
    # name: (heads, kv heads, head dim), requests; decode items of 32 pages in brackets
    "small, one split": ((8, 2, 128), _dec(5, 1, 17, 300, 512) + [(0, 70, 9)]),
    "small, many splits [84]": ((8, 2, 128), _dec(7, 2600) + [(0, 200, 100), (0, 3, 0)]),
    "small at the line [512]": ((8, 2, 64), _dec(256, 40, 500) + [(0, 65, 0)]),
    "small past the line [514]": ((8, 2, 64), _dec(257, 40, 500) + [(0, 65, 0)]),
    "short items [160]": ((8, 2, 128), _dec(20, 2000, 1800) + [(0, 300, 700)]),
    "streamed [600]": ((8, 2, 128), _dec(50, 3000, 2900) + [(0, 513, 0), (0, 64, 64)]),
    "streamed, a few tiles [1100]": ((16, 1, 64), _dec(275, 2000) + [(0, 1, 0)]),
    "chunk before decodes [300]": ((8, 2, 64), [(0, 260, 1000)] + _dec(30, 2500)),
    "group 1 [320]": ((4, 4, 128), _dec(10, 4000) + [(0, 280, 33)]),
    "group 2 [300]": ((4, 2, 128), _dec(25, 3000) + [(0, 150, 0)]),
    "group 3 [360]": ((12, 4, 64), _dec(15, 3000) + [(0, 90, 5)]),
    "split prefill units [300]": ((8, 2, 128), _dec(25, 3000) + [(0, 40, 9000)]),
    "too much prefill [2]": ((8, 2, 64), _dec(1, 9) + [(0, 1500, 3000)]),
}


@pytest.mark.parametrize("name", list(CASES))
def test_one_launch_equals_two(ctx, name):
    from paper_2511_04791_amd import workloads as wl
    heads, reqs = CASES[name]
    b = wl.make_batch(wl.AttnShape(*heads, "bf16"), reqs, page_seed=600)
    layers = [[t.cuda() for t in wl.make_tensors(b, 6000 + l, scale=1.0)] for l in range(3)]
    qs, kcs, vcs = ([x[i] for x in layers] for i in range(3))
    pt = torch.as_tensor(b.page_table, device="cuda")
    for _ in range(2):  # counters are left clear for the next call
        one = ctx.attn_iteration(qs, kcs, vcs, pt, b.seq_meta, check_errors=True)
    ctx.set_profiling(2)
    two = ctx.attn_iteration(qs, kcs, vcs, pt, b.seq_meta, check_errors=True)
    ctx.set_profiling(0)
    single = ctx.attn_mixed_batch(qs[2], kcs[2], vcs[2], pt, b.seq_meta, check_errors=True)
    torch.cuda.synchronize()
    for l in range(3):
        assert torch.equal(one[l], two[l]), f"layer {l}"
    assert torch.equal(single, one[2])
    if b.num_tokens < 600:
        mx, mean = errors(one[0], oracle_out(b, qs[0], kcs[0], vcs[0]))
        print(f"[parity] mixed, {name}: max_abs={mx:.3e} mean_abs={mean:.3e}", flush=True)
        assert mx <= BF16_MAX_ABS and mean <= BF16_MEAN_ABS


@pytest.mark.parametrize("reqs", [_dec(3, 300) + [(0, 50, 20)], _dec(40, 2000) + [(0, 50, 20)]])
def test_bad_pages_of_either_half_are_flagged(ctx, reqs):
    import paper_2511_04791_amd as duet
    from paper_2511_04791_amd import workloads as wl
    b = wl.make_batch(wl.AttnShape(8, 2, 128, "bf16"), reqs, page_seed=601)
    q, kc, vc = (t.cuda() for t in wl.make_tensors(b, 6100))
    pt = torch.as_tensor(b.page_table, device="cuda")
    for r in (1, b.num_reqs - 1):
        bad = pt.clone()
        bad[r, 2] = b.num_phys_pages + 5
        with pytest.raises(duet.DuetError) as e:
            ctx.attn_mixed_batch(q, kc, vc, bad, b.seq_meta, check_errors=True)
        assert e.value.code == -6
    out = ctx.attn_mixed_batch(q, kc, vc, pt, b.seq_meta, check_errors=True)
    torch.cuda.synchronize()
    assert not torch.isnan(out).any()


@pytest.mark.parametrize("chunk", [10, 1200])
def test_heads_of_64_beside_a_short_and_a_long_chunk(ctx, chunk):
    """2600 decode items of heads of 64: two launches beside ten tokens, one beside 1200.  Same bits as split."""
    import paper_2511_04791_amd as duet
    from paper_2511_04791_amd import workloads as wl
    b = wl.make_batch(wl.AttnShape(16, 2, 64, "bf16"), [(1, 1, 2000 + 17 * i % 1000) for i in range(260)] + [(0, chunk, 80)],
                      page_seed=880)
    q, kc, vc = wl.make_tensors(b, 8800, device="cuda")
    pt = torch.as_tensor(b.page_table, device="cuda")
    out = ctx.attn_mixed_batch(q, kc, vc, pt, b.seq_meta, check_errors=True)
    other = ctx.attn_mixed_batch(q, kc, vc, pt, b.seq_meta, duet.CuSplit.split(128, 128), check_errors=True)
    torch.cuda.synchronize()
    assert torch.isfinite(out).all() and torch.equal(out, other)
