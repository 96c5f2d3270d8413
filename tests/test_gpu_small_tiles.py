"""Tensors of one launch, at the edges of their tiles (2048 quartic bytes) and
of the largest count of tiles that exchange their maxima (128), alone and in
batches with longer and shorter ones, at any alignment.  Bit-exact against the
oracle."""
import numpy as np
import pytest

import oracle
from paper_1802_07389_amd import workloads

pytestmark = pytest.mark.gpu

F32 = np.float32
TILE = 5 * 2048  # values of a tile
EDGE = 128 * TILE


@pytest.fixture(scope="module")
def ctx():
    from paper_1802_07389_amd import tlc
    c = tlc.Context(max_n=2 * EDGE + 200_000, max_tensors=16)
    yield c
    c.close()


def check(g, x, r, s, got, in_place=False):
    st, C, M, r_gpu = got
    r_ref = r.copy()
    st_ref, C_ref, M_ref = oracle.compress(x, r_ref, s, in_place=in_place)
    assert st == st_ref
    if st == 0:
        assert F32(M).tobytes() == F32(M_ref).tobytes()
        assert np.array_equal(C, C_ref)
    assert np.array_equal(g.bits(r_gpu), g.bits(r_ref))


@pytest.mark.parametrize("options", [0, 1], ids=["default", "in_place"])
@pytest.mark.parametrize("n", [1, 2, 3, 4, 6, 9, 39, 41, TILE - 6, TILE - 1, TILE, TILE + 1,
                               2 * TILE - 3, 2 * TILE + 1, 65 * TILE + 7, EDGE - 4, EDGE, EDGE + 1])
def test_tile_edges(ctx, options, n):
    import gpuutil as g
    ctx.set_options(options)
    try:
        for kind in range(3):
            x, r = workloads.normal([91, n, kind], n), workloads.normal([92, n, kind], n, 3e-3)
            if kind == 1:  # runs over tile edges, one value at either end
                x[:], r[:] = 0, 0
                x[0], x[-1] = 0.5, -0.5
            if kind == 2:  # refused
                x[n // 2] = np.nan
            for off, r_off in ((0, 0), (1, 3)):
                check(g, x, r, 1.5, g.gpu_compress(ctx, x, r, 1.5, offset=off, r_offset=r_off),
                      bool(options))
    finally:
        ctx.set_options(0)


@pytest.mark.parametrize("options", [0, 1], ids=["default", "in_place"])
def test_batch_of_all_kinds(ctx, options):
    """One batch with tensors of one tile, of a few, and of more than 128."""
    import torch

    import gpuutil as g
    from paper_1802_07389_amd import tlc
    sizes = [7, EDGE + 5, TILE + 1, 16, 5 * TILE, 64, 3 * TILE - 2, 2305]
    xs = [workloads.normal([93, t], n) for t, n in enumerate(sizes)]
    rs = [workloads.normal([94, t], n, 3e-3) for t, n in enumerate(sizes)]
    for bad in (None, 1, 4, 7):  # a refused tensor of each kind leaves the others alone
        xb = [x.copy() for x in xs]
        if bad is not None:
            xb[bad][-1] = np.inf
        xd = [g.to_dev(x, t % 3) for t, x in enumerate(xb)]
        rd = [g.to_dev(r, (t + 1) % 3) for t, r in enumerate(rs)]
        bufs = [torch.zeros(-(-n // 5), dtype=torch.uint8, device="cuda") for n in sizes]
        ctx.set_options(options)
        try:
            _, lens, scales, stat = tlc.tlc_compress_batch(
                ctx.handle, [x.data_ptr() for x in xd], [r.data_ptr() for r in rd], sizes,
                [1.75] * len(sizes), [b.data_ptr() for b in bufs], [b.numel() for b in bufs])
        finally:
            ctx.set_options(0)
        torch.cuda.synchronize()
        for t in range(len(sizes)):
            check(g, xb[t], rs[t], 1.75, (stat[t], bufs[t][:lens[t]].cpu().numpy(), scales[t],
                                          rd[t].cpu().numpy()), bool(options))


def test_decodes_right_after_a_refused_batch(ctx):
    """A refused tensor with a max pass: the descriptor slots that the decodes
    after it take over are no longer read by its blocks."""
    import torch

    import gpuutil as g
    from paper_1802_07389_amd import tlc
    n = EDGE + 50_001
    big, r = workloads.normal([96, n], n), np.zeros(n, F32)
    big[0] = np.inf
    x, small = workloads.normal([97, 0], 3000), np.zeros(3000, F32)
    r_ref = small.copy()
    _, C, M = oracle.compress(x, r_ref, 1.5)
    _, want = oracle.decompress(C, M, 3000, np.zeros(3000, F32))
    bd, rd, xd = g.to_dev(big), g.to_dev(r), g.to_dev(x)
    data = torch.from_numpy(C).cuda()
    outs = [[torch.zeros(3000, device="cuda") for _ in range(3)] for _ in range(6)]
    for _ in range(3):
        sd = g.to_dev(small)
        with pytest.raises(tlc.TLCError):
            ctx.compress_batch([bd, xd], [rd, sd], 1.5)
        for o in outs:
            ctx.decompress_batch([data] * 3, [M] * 3, o)
        ctx.sync()
        assert np.array_equal(g.bits(sd.cpu().numpy()), g.bits(r_ref))
        assert not rd.any()
        for o in outs:
            for t in o:
                assert np.array_equal(g.bits(t.cpu().numpy()), g.bits(want))
                t.zero_()
