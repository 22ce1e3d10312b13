"""GPU parity of the token-level operators at the edges of their chunks: RMSNorm and SwiGLU against their
fp64 definitions (one rounding to bf16), the QKV split bit for bit."""
import numpy as np
import pytest

from _helpers import to64

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

U = 2.0 ** -8  # bf16 unit roundoff


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2511_04791_amd as duet
    c = duet.Context(0)
    yield c
    c.close()


def _randn(seed, *shape, scale=1.0):
    gen = torch.Generator(device="cpu")
    gen.manual_seed(seed)
    return (torch.randn(*shape, generator=gen) * scale).to(torch.bfloat16)


@pytest.mark.parametrize("d", [8, 504, 2048, 2056, 4096, 4104, 8192, 8200, 20000])
def test_rmsnorm_widths(ctx, d):
    from oracle.block import rmsnorm
    x, w = _randn(5300 + d, 3, d), 1 + _randn(5301 + d, d, scale=0.1)
    ref = rmsnorm(to64(x), to64(w), 1e-5)
    err = np.abs(to64(ctx.rmsnorm(x.cuda(), w.cuda(), 1e-5)) - ref)
    # one rounding to bf16 of an fp32 value a few ulp off
    assert (err <= (U + 2.0 ** -16) * np.abs(ref) + 1e-30).all()


@pytest.mark.parametrize("m", [8, 2040, 2048, 2056, 4096, 4104, 14336])
def test_swiglu_widths(ctx, m):
    gu = _randn(5400 + m, 5, 2 * m, scale=2.0)
    g, u = to64(gu[:, :m]), to64(gu[:, m:])
    ref = g / (1 + np.exp(-g)) * u
    err = np.abs(to64(ctx.swiglu(gu.cuda())) - ref)
    # exp and the division in fp32 (a few ulp) before the one rounding
    assert (err <= (U + 2.0 ** -14) * np.abs(ref) + 1e-30).all()


def test_swiglu_of_more_blocks_than_one_launch_holds(ctx):
    """2^24 workgroups of 256 threads are one too many for a grid: the rows go in two launches."""
    rows, m = (1 << 24) + 3, 8
    gu = torch.randn(1 << 16, 2 * m, device="cuda").to(torch.bfloat16).repeat((rows >> 16) + 1, 1)[:rows].contiguous()
    out = torch.full((rows, m), float("nan"), dtype=torch.bfloat16, device="cuda")
    ctx.swiglu(gu, out=out)
    torch.cuda.synchronize()
    one = ctx.swiglu(gu[:1 << 16].contiguous())
    assert torch.equal(out[:1 << 16], one)
    assert torch.equal(out[1 << 16:rows - 3].view(-1, 1 << 16, m), one.expand((rows >> 16) - 1, -1, -1))
    assert torch.equal(out[rows - 3:], one[:3])



CASES = {
    # whole pages, pages covered in part at either end or both, one row, every start in a page
    "pages": ((4, 2, 128), [(0, 16, 0), (0, 48, 32), (0, 17, 15), (0, 31, 1), (0, 15, 0), (0, 2, 15), (1, 1, 16)]),
    "starts": ((2, 1, 64), [(0, 40 + s, s) for s in range(16)]),
    # more requests than one round of the search takes, and widths that end inside a workgroup
    "many": ((6, 3, 64), [(1, 1, 7 * i % 90) for i in range(150)] + [(0, 33, 20), (1, 1, 3), (0, 1, 0)]),
    "wide": ((20, 4, 128), [(0, 50, 5), (1, 1, 9)]),
}


@pytest.mark.parametrize("name", list(CASES))
def test_qkv_split_is_a_copy(ctx, name):
    from oracle.attention import append_token
    from paper_2511_04791_amd import workloads as wl
    (hq, hkv, d), reqs = CASES[name]
    sh = wl.AttnShape(hq, hkv, d, "bf16")
    b = wl.make_batch(sh, reqs, page_seed=5500)
    _, kc, vc = wl.make_tensors(b, 5501, device="cpu")
    T, nq, nk = b.num_tokens, hq * d, hkv * d
    qkv = _randn(5502, T, nq + 2 * nk)
    kcg, vcg = kc.cuda(), vc.cuda()
    q = ctx.qkv_split(qkv.cuda(), kcg, vcg, torch.as_tensor(b.page_table, device="cuda"), b.seq_meta, sh,
                      check_errors=True)
    torch.cuda.synchronize()
    as16 = lambda t: t.view(torch.int16).numpy()  # noqa: E731
    assert np.array_equal(as16(q.cpu()), as16(qkv[:, :nq].reshape(T, hq, d).contiguous()))
    kref, vref, q16 = as16(kc).copy(), as16(vc).copy(), as16(qkv)
    for r in range(b.num_reqs):
        _, q_start, q_len, cached = (int(x) for x in b.seq_meta[r])
        for t in range(q_len):
            row = q16[q_start + t]
            append_token(kref, vref, b.page_table[r], cached + t, row[nq:nq + nk].reshape(hkv, d),
                         row[nq + nk:].reshape(hkv, d), 16)
    assert np.array_equal(as16(kcg.cpu()), kref)
    assert np.array_equal(as16(vcg.cpu()), vref)
