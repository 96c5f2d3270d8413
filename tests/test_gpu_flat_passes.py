"""The flat passes of large tensors at the places where they can go wrong:
pointers at every dword alignment (the tensor's and the buffer's apart), m
off the float4 grid, lines and words of the buffer cut off by n, every value
quantizing to non-zero, none doing so.  Bit-exact against the oracle."""
import numpy as np
import pytest

import oracle
from paper_1802_07389_amd import workloads

pytestmark = pytest.mark.gpu

F32 = np.float32
# 65 tiles of 4096 quartic bytes and up take the three passes; in place, those of
# the default policy below 20,000,000 values, then their own
BASE = {0: 5 * 4096 * 512, 1: 5 * 4096 * 1000}
LINES = 4 * (20 * 4 * 256 * 256 - 3) + 1  # in place, see test_in_place_line_bounds


@pytest.fixture(scope="module")
def ctx():
    from paper_1802_07389_amd import tlc
    c = tlc.Context(max_n=max(BASE[1] + 256, LINES))
    yield c
    c.close()


def inputs(kind, n):
    if kind == "sparse":  # a few values reach half the scale, up to the last one
        x = workloads.normal([81, n], n)
        r = workloads.normal([82, n], n, 4e-3)
        x[[0, 31, 32, n // 2, n - 2, n - 1]] = 0.02
        return x, r
    if kind == "dense":  # every value is the largest or its negative
        x = np.where(np.arange(n) % 3 == 0, F32(-1.0), F32(1.0)).astype(F32)
        return x, np.zeros(n, F32)
    if kind == "spread":  # a few in every group of threads, more than a tile's list holds
        x = workloads.normal([87, n], n, 1e-5)
        x[::37] = np.where(np.arange(len(x[::37])) % 2 == 0, F32(0.5), F32(-0.5))
        return x, workloads.normal([88, n], n, 1e-5)
    return np.zeros(n, F32), np.full(n, -0.0, F32)  # "zero": M = 0, -0.0 kept


@pytest.mark.parametrize("options", [0, 1], ids=["default", "in_place"])
@pytest.mark.parametrize("kind", ["sparse", "dense", "zero", "spread"])
@pytest.mark.parametrize("extra,offset,r_offset", [(0, 0, 0), (1, 1, 0), (2, 0, 3), (3, 2, 2),
                                                   (29, 3, 1), (33, 0, 0), (127, 0, 1)])
def test_flat_passes(ctx, options, kind, extra, offset, r_offset):
    import gpuutil as g
    n = BASE[options] + extra  # m % 4 = 0 to 3
    x, r = inputs(kind, n)
    r_ref = r.copy()
    st_ref, C_ref, M_ref = oracle.compress(x, r_ref, 1.5)
    ctx.set_options(options)
    try:
        st, C, M, r_gpu = g.gpu_compress(ctx, x, r, 1.5, offset=offset, r_offset=r_offset)
    finally:
        ctx.set_options(0)
    assert st == st_ref == 0 and F32(M).tobytes() == F32(M_ref).tobytes()
    assert np.array_equal(C, C_ref)
    assert np.array_equal(g.bits(r_gpu), g.bits(r_ref))


@pytest.mark.parametrize("n", [4 * 1021 + 2, 4 * 524285 + 1, LINES])
@pytest.mark.parametrize("lane", range(8))
def test_in_place_line_bounds(ctx, n, lane):
    """One float4 of each 128-byte line reaches half the scale: its bound has to
    hold also where n cuts the unrolled loop of the max pass inside a line (n / 4
    three short of a multiple of its step, 4 * 256 float4s a block; only LINES is
    large enough for the in-place max pass)."""
    import gpuutil as g
    from paper_1802_07389_amd import tlc
    x = workloads.normal([85, n], n, 1e-5)
    x[4 * lane + 1::32] = F32(0.02)
    r = workloads.normal([86, n], n, 1e-5)
    for mode in (tlc.TLC_MODE_3LC, tlc.TLC_MODE_NO_ZRE):
        r_ref = r.copy()
        encode = oracle.compress if mode == tlc.TLC_MODE_3LC else oracle.compress_nozre
        st, C_ref, M_ref = encode(x, r_ref, 1.5)
        xd, rd = g.to_dev(x), g.to_dev(r)
        ctx.set_options(1)
        try:
            data, M = ctx.compress_mode(mode, xd, rd, 1.5)
        finally:
            ctx.set_options(0)
        assert st == 0 and F32(M).tobytes() == F32(M_ref).tobytes()
        assert np.array_equal(data.cpu().numpy(), C_ref)
        assert np.array_equal(g.bits(rd.cpu().numpy()), g.bits(r_ref))


@pytest.mark.parametrize("options", [0, 1], ids=["default", "in_place"])
@pytest.mark.parametrize("where", [0, -1])
def test_refused_tensor_off_the_grid(ctx, options, where):
    """Inf at either end: the buffer as it was, or (in place) the sums."""
    import gpuutil as g
    n = BASE[options] + 30
    x, r = inputs("sparse", n)
    x[where] = np.inf
    r_ref = r.copy()
    assert oracle.compress(x, r_ref, 1.5, in_place=bool(options))[0] == oracle.E_NONFINITE
    ctx.set_options(options)
    try:
        st, _, _, r_gpu = g.gpu_compress(ctx, x, r, 1.5, offset=1, r_offset=2)
    finally:
        ctx.set_options(0)
    assert st == oracle.E_NONFINITE
    assert np.array_equal(g.bits(r_gpu), g.bits(r_ref))


@pytest.mark.parametrize("n,offset", [(4, 1), (5, 2), (7, 3), (20479, 1), (20483, 2), (61447, 3)])
def test_comparison_packs_off_the_grid(ctx, n, offset):
    """No-ZRE and stochastic payloads, whose bytes come from trits: tiles cut
    off by m, and bytes stored at any address."""
    import torch

    import gpuutil as g
    from paper_1802_07389_amd import tlc
    x, r = workloads.normal([83, n], n), workloads.normal([84, n], n)
    m = -(-n // 5)
    for mode in (tlc.TLC_MODE_NO_ZRE, tlc.TLC_MODE_STOCHASTIC):
        r_ref = r.copy()
        if mode == tlc.TLC_MODE_NO_ZRE:
            st, Q, M = oracle.compress_nozre(x, r_ref, 1.25)
        else:
            st, Q, M = oracle.compress_stochastic(x, 1.25, 11, 5)
        xd, rd = g.to_dev(x, offset), g.to_dev(r, 4 - offset)
        buf = torch.full((m + 8,), 0xAB, dtype=torch.uint8, device="cuda")
        data, scale = ctx.compress_mode(mode, xd, rd, 1.25, seed=11, step=5,
                                        out=buf[offset:offset + m])
        assert st == 0 and F32(scale).tobytes() == F32(M).tobytes()
        assert np.array_equal(data.cpu().numpy(), Q)
        assert int((buf[:offset] != 0xAB).sum() + (buf[offset + m:] != 0xAB).sum()) == 0
        assert np.array_equal(g.bits(rd.cpu().numpy()), g.bits(r_ref))
