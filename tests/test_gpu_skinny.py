"""GPU parity of blocks whose partitions hold few rows (the library's own projection kernels), against
the fp64 oracle with the block tests' bounds.

Edges: 16 rows per MFMA tile (and the last row count that takes the own kernels, 64), 128 columns
per workgroup (64 gate and 64 up ones), 32 rows of a weight per step, parts of d_in; an MLP width
need only be a multiple of 8.
"""
import numpy as np
import pytest

from test_gpu_block import _run_case, ctx  # noqa: F401 (ctx is the module's fixture)

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("rows", [1, 15, 16, 17, 32, 33, 48, 63, 64, 65])
def test_rows(ctx, rows):  # noqa: F811
    import paper_2511_04791_amd as duet
    _run_case(ctx, [(1, 1, 3 + 5 * i) for i in range(rows)], 512, 2, duet.CuSplit.agg(), 4300 + rows)


@pytest.mark.parametrize("ffn", [8, 40, 56, 72, 1000])
@pytest.mark.parametrize("heads", [(1, 1, 64), (3, 1, 64), (6, 2, 128)])
def test_widths(ctx, heads, ffn):  # noqa: F811
    import paper_2511_04791_amd as duet
    from paper_2511_04791_amd import workloads as wl
    reqs = [(1, 1, 20 + i) for i in range(5)] + [(0, 14, 30)]  # a short chunk beside the decodes
    _run_case(ctx, reqs, ffn, 3, duet.CuSplit.agg(), 4400 + ffn, wl.AttnShape(*heads, "bf16"))


@pytest.mark.parametrize("share", [32, 128])
def test_partitions(ctx, share):  # noqa: F811
    """Each partition takes its own route by its own rows: few on one side, many on the other."""
    import paper_2511_04791_amd as duet
    _run_case(ctx, [(1, 1, 100 + i) for i in range(20)] + [(0, 90, 5)], 520, 2,
              duet.CuSplit.split(256 - share, share), 4500)


@pytest.mark.parametrize("rows,cus", [(16, 256), (16, 128), (16, 64), (32, 96), (33, 96), (33, 256)])
def test_large_weights_on_both_sides_of_the_rule(ctx, rows, cus):  # noqa: F811
    """75 MB of weights a layer: own kernels aggregated and, up to 32 rows, on 96 CUs or more; the
    library's on the other shares."""
    import paper_2511_04791_amd as duet
    from paper_2511_04791_amd import workloads as wl
    split = duet.CuSplit.agg() if cus == 256 else duet.CuSplit.split(256 - cus, cus)
    _run_case(ctx, [(1, 1, 9 + 7 * i) for i in range(rows)], 4096, 1, split, 4650 + rows, wl.AttnShape(16, 8, 128, "bf16"))


def test_bad_page_is_flagged_and_not_written(ctx):  # noqa: F811
    import paper_2511_04791_amd as duet
    from paper_2511_04791_amd import workloads as wl
    b = wl.make_batch(wl.AttnShape(4, 2, 128, "bf16"), [(1, 1, 40), (1, 1, 50)], page_seed=4600)
    x, weights, caches = wl.make_block_tensors(b, 256, 1, 4600, device="cpu")
    bad = torch.as_tensor(b.page_table).clone()
    bad[1, 3] = b.num_phys_pages + 7  # holds the new token of the second request
    kc, vc = caches[0][0].cuda(), caches[0][1].cuda()
    with pytest.raises(duet.DuetError) as e:
        ctx.block_forward(x.cuda(), [{n: t.cuda() for n, t in weights[0].items()}], [kc], [vc], bad.cuda(), b.seq_meta,
                          256, check_errors=True)
    assert e.value.code == -6
    as16 = lambda t: t.cpu().view(torch.int16).numpy()  # noqa: E731
    changed = np.unique(np.nonzero(as16(kc) != as16(caches[0][0]))[0])
    assert list(changed) == [int(b.page_table[0, 2])]  # the first request's page only
