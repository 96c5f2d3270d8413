"""Batched and summed decodes: what a call costs follows its own streams, not
the context's capacity, and streams decode the same whichever way their
descriptors reach the device.  Bit-exact against the oracle."""
import time

import numpy as np
import pytest

import oracle
from paper_1802_07389_amd import workloads

pytestmark = pytest.mark.gpu

F32 = np.float32


def stream(seed, n, s=1.0):
    x = workloads.normal([111, seed], n)
    st, C, M = oracle.compress(x, np.zeros(n, F32), s)
    assert st == 0
    return C, M


def dense_stream(seed, n):
    """About n / 5 bytes: half of the values quantize to non-zero."""
    x = np.random.default_rng([114, seed]).uniform(-1.0, 1.0, n).astype(F32)
    st, C, M = oracle.compress(x, np.zeros(n, F32), 1.0)
    assert st == 0 and C.size > n / 6
    return C, M


def test_capacity_costs_nothing():
    """A summed decode of 16 streams of several scan tiles on a context made for
    16 streams, and on one made for 65,536: it had copied a table of the whole
    capacity (4 MB) each time, for 2.5 times the time."""
    import torch

    from paper_1802_07389_amd import tlc
    n, P = 400_000, 16
    data = [stream(k, n) for k in range(P)]
    assert all(C.size > 8192 for C, _ in data)
    C = [torch.from_numpy(c).cuda() for c, _ in data]
    M = [m for _, m in data]
    out = torch.zeros(n, device="cuda")
    took = {}
    for cap in (P, 65536):
        with tlc.Context(max_n=n * P, max_tensors=cap) as ctx:
            best = []
            for _ in range(9):
                torch.cuda.synchronize()
                t0 = time.perf_counter()
                for _ in range(40):
                    ctx.decompress_sum(C, M, out)
                ctx.sync()
                best.append(time.perf_counter() - t0)
            took[cap] = min(best)
        ref = np.zeros(n, F32)
        for k, (c, m) in enumerate(data):
            _, ref = oracle.decompress(c, m, n, ref, k > 0)
        assert np.array_equal(out.cpu().numpy().view(np.uint32), ref.view(np.uint32))
    print(took, flush=True)
    assert took[65536] < 1.6 * took[P]


@pytest.mark.parametrize("count,base", [(1, 900_001), (2, 900_001), (9, 900_001), (11, 900_001),
                                        (3, 100_003), (6, 100_003), (7, 100_003),
                                        (12, 100_003), (40, 100_003)])
def test_few_streams_of_several_tiles(count, base):
    """Counts and lengths on both sides of the line between the two ways, calls of
    other counts between them on the same context."""
    import torch

    import gpuutil as g
    from paper_1802_07389_amd import tlc
    with tlc.Context(max_n=20_000_000, max_tensors=40) as ctx:
        for k in (count, 12, count, 1):
            ns = [300 if t == 1 else base + 1_009 * t for t in range(k)]
            data = [(stream if base > 500_000 else dense_stream)(20 + t, n)
                    for t, n in enumerate(ns)]
            assert data[0][0].size > 8192
            o0 = [workloads.normal([112, t], n) for t, n in enumerate(ns)]
            outs = [g.to_dev(o, t % 4) for t, o in enumerate(o0)]
            ctx.decompress_batch([torch.from_numpy(c).cuda() for c, _ in data],
                                 [m for _, m in data], outs, accumulate=True)
            ctx.sync()
            for (c, m), n, o, before in zip(data, ns, outs, o0):
                _, ref = oracle.decompress(c, m, n, before.copy(), True)
                assert np.array_equal(g.bits(o.cpu().numpy()), g.bits(ref))


@pytest.mark.parametrize("accumulate", [False, True])
@pytest.mark.parametrize("n,counts", [(100_003, (1, 2, 31, 32)), (2_003, (1, 31, 33)),
                                      (400_001, (33, 4, 32)), (3_000_002, (4, 1))])
def test_summed_streams(n, counts, accumulate):
    """Sums whose scan searches its stream and finds it in a table, of short and of
    long tiles, one after the other on a context."""
    import torch

    import gpuutil as g
    from paper_1802_07389_amd import tlc
    data = [dense_stream(60 + t, n) for t in range(max(counts))]
    dev = [torch.from_numpy(c).cuda() for c, _ in data]
    with tlc.Context(max_n=n * max(counts), max_tensors=max(counts)) as ctx:
        for k in counts:
            ref = workloads.normal([113, k], n)
            out = g.to_dev(ref, k % 4)
            ctx.decompress_sum(dev[:k], [m for _, m in data[:k]], out, accumulate=accumulate)
            ctx.sync()
            for t, (c, m) in enumerate(data[:k]):
                _, ref = oracle.decompress(c, m, n, ref, accumulate or t > 0)
            assert np.array_equal(g.bits(out.cpu().numpy()), g.bits(ref)), k
