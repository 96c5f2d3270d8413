"""Batched encodes with tensors too large for the batch's one launch: those of
129 tiles of 2048 quartic bytes to 2048 of 4096 go through the three passes
together, larger ones one after the other, beside small ones.  Bit-exact
against the oracle, and no tensor is chained through the one launch (that took
up to 1.4 times as long)."""
import numpy as np
import pytest

import oracle
from paper_1802_07389_amd import workloads

pytestmark = pytest.mark.gpu

F32 = np.float32
EDGE = 128 * 5 * 2048       # the largest tensor of the one launch
WIDE = 32 * 5 * 2048        # beyond it, tensors join the passes of larger ones ...
CACHED = (256 << 20) // 8   # ... where they hold more values than this together
TILE = 5 * 4096             # values of a tile of the three passes
MIDDLE = 2048 * TILE       # the largest tensor whose passes are shared


@pytest.fixture(scope="module")
def ctx():
    from paper_1802_07389_amd import tlc
    c = tlc.Context(max_n=110_000_000, max_tensors=48)
    yield c
    c.close()


def tensor(kind, seed, n):
    if kind == "spikes":  # runs of zeros that cross tiles, a value at each edge
        x = np.zeros(n, F32)
        m = -(-n // 5)
        at = np.arange(4096, m, 4096 * 3)
        x[at], x[at - 1], x[0], x[-1] = 0.5, -0.5, 0.5, 0.5
        return x, np.zeros(n, F32)
    return workloads.normal([101, seed], n), workloads.normal([102, seed], n, 3e-3)


def encode_check(ctx, case, options, bad=None):
    """case: (n, kind, offset of the tensor, of the buffer) per tensor."""
    import torch

    import gpuutil as g
    from paper_1802_07389_amd import tlc
    xs, rs = zip(*[tensor(kind, t, n) for t, (n, kind, _, _) in enumerate(case)])
    if bad is not None:
        xs[bad][len(xs[bad]) * 2 // 3] = np.inf
    xd = [g.to_dev(x, c[2]) for x, c in zip(xs, case)]
    rd = [g.to_dev(r, c[3]) for r, c in zip(rs, case)]
    caps = [-(-c[0] // 5) for c in case]
    out = [torch.full((k,), 0xAB, dtype=torch.uint8, device="cuda") for k in caps]
    ctx.set_options(options)
    ctx.profile(True)
    ctx.profile_reset()
    try:
        st, lens, scales, stat = tlc.tlc_compress_batch(
            ctx.handle, [t.data_ptr() for t in xd], [t.data_ptr() for t in rd],
            [c[0] for c in case], [1.0 + t % 6 * 0.15 for t in range(len(case))],
            [o.data_ptr() for o in out], caps)
        torch.cuda.synchronize()
        launches = [ctx.profile_get(k)[1] for k in range(tlc.TLC_KERNEL_COUNT)]
    finally:
        ctx.profile(False)
        ctx.set_options(0)
    assert st == (tlc.TLC_OK if bad is None else tlc.TLC_E_NONFINITE)
    for t, (n, kind, _, _) in enumerate(case):
        r_ref = rs[t].copy()
        st_ref, C_ref, M_ref = oracle.compress(xs[t], r_ref, 1.0 + t % 6 * 0.15,
                                               in_place=bool(options))
        assert (stat[t] == 0) == (st_ref == 0) == (t != bad), t
        if st_ref == 0:
            assert F32(scales[t]).tobytes() == F32(M_ref).tobytes(), (t, n)
            assert np.array_equal(out[t][:lens[t]].cpu().numpy(), C_ref), (t, n)
        assert np.array_equal(g.bits(rd[t].cpu().numpy()), g.bits(r_ref)), (t, n)
    # one shared tile pass, and one for each large tensor
    edge = WIDE if sum(c[0] for c in case if WIDE < c[0] <= EDGE) > CACHED else EDGE
    large = sum(c[0] > MIDDLE for c in case)
    middle = any(edge < c[0] <= MIDDLE for c in case)
    assert launches[tlc.TLC_KERNEL_QUANT_ENCODE] == large + middle
    assert launches[tlc.TLC_KERNEL_QUANT_ENCODE_BATCH] == any(c[0] <= edge for c in case)
    g.log(f"{[c[0] for c in case]} options {options} bad {bad} ok")


@pytest.mark.parametrize("options", [0, 1], ids=["default", "in_place"])
def test_sizes_of_the_shared_passes(ctx, options):
    encode_check(ctx, [(EDGE + 1, "normal", 0, 0), (65 * TILE, "spikes", 1, 2),
                       (65 * TILE + 1, "spikes", 0, 0), (200 * TILE - 3, "normal", 3, 0),
                       (512 * TILE, "spikes", 0, 1), (257 * TILE + 4, "spikes", 0, 0)], options)
    encode_check(ctx, [(513 * TILE - 1, "spikes", 0, 0), (1500 * TILE + 3, "normal", 1, 0),
                       (MIDDLE, "spikes", 0, 0)], options)
    encode_check(ctx, [(200 * TILE + 2, "spikes", 2, 2)], options)  # alone, after the others


@pytest.mark.parametrize("options", [0, 1], ids=["default", "in_place"])
@pytest.mark.parametrize("bad", [None, 0, 1, 3, 4])
def test_all_kinds_together(ctx, options, bad):
    case = [(300, "normal", 0, 0), (2_600_003, "normal", 1, 0), (MIDDLE + 1, "spikes", 0, 0),
            (700_000, "normal", 0, 0), (MIDDLE + TILE + 7, "normal", 2, 1),
            (EDGE + 40, "spikes", 0, 3)]
    encode_check(ctx, case, options, bad)


@pytest.mark.parametrize("options", [0, 1], ids=["default", "in_place"])
@pytest.mark.parametrize("bad", [None, 0, 39, 40])
def test_many_wide_tensors(ctx, options, bad):
    """More values in tensors of 33 to 128 tiles than the cache holds: they join
    the shared passes, those of 32 tiles don't."""
    case = [(WIDE + 1 + 2731 * t * t % 971_000, "normal" if t % 8 else "spikes", t % 4, 0)
            for t in range(40)]
    case = [(max(c[0], 850_000) if t < 38 else c[0], *c[1:]) for t, c in enumerate(case)]
    encode_check(ctx, case + [(WIDE, "normal", 0, 1), (EDGE + 8, "spikes", 0, 0),
                              (77, "normal", 0, 0)], options, bad)
