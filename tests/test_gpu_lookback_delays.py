"""The look-back scans under scrambled publish order: the stress build of
the library (libtlc_delay.so, compiled with TLC_DELAY_INJECT) sleeps a
pseudo-random 0 to about 25 us before every status-word publish.  Each
user of the status words runs here once against the CPU oracle, bit for
bit: the tiles of small tensors, alone and in batches, which exchange maxima
and summaries; the no-allocation encode, whose tiles are chained by look-back
above that; and the decoder's index scan (single, batched and summed decodes;
the single decode's blocks also wait for their start entries and the stream's
verdict).  The three-pass encoders publish no status words; they run here
because a call mixes them with the others.  Every wait is bounded; a timeout
would surface as TLC_E_DEVICE, not a hang."""
import importlib.util
import os

import numpy as np
import pytest

import oracle
from paper_1802_07389_amd import workloads

pytestmark = pytest.mark.gpu

F32 = np.float32
ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_1802_07389_amd")


def bits(a):
    return np.ascontiguousarray(a, dtype=np.float32).view(np.uint32)


@pytest.fixture(scope="module")
def dt():
    """A second instance of the binding, bound to the stress build."""
    path = os.path.join(PKG, "libtlc_delay.so")
    assert os.path.exists(path), "libtlc_delay.so is not built: run __graft_entry__.build()"
    old = os.environ.get("TLC_LIBRARY")
    os.environ["TLC_LIBRARY"] = path
    try:
        spec = importlib.util.spec_from_file_location("tlc_delay", os.path.join(PKG, "tlc.py"))
        mod = importlib.util.module_from_spec(spec)
        spec.loader.exec_module(mod)
    finally:
        if old is None:
            del os.environ["TLC_LIBRARY"]
        else:
            os.environ["TLC_LIBRARY"] = old
    assert mod.LIB_PATH == path
    return mod


@pytest.fixture(scope="module")
def ctx(dt):
    c = dt.Context(max_n=2051 * 4096 * 5, max_tensors=400)
    yield c
    c.close()


def encode_check(ctx, x, r, s, tag):
    import torch
    xd = torch.from_numpy(x).cuda()
    rd = torch.from_numpy(r.copy()).cuda()
    C, M = ctx.compress(xd, rd, s)
    r_ref = r.copy()
    st, C_ref, M_ref = oracle.compress(x, r_ref, s)
    assert st == 0 and M == M_ref, tag
    assert np.array_equal(C.cpu().numpy(), C_ref), tag
    assert np.array_equal(bits(rd.cpu().numpy()), bits(r_ref)), tag
    print(f"{tag}: {C_ref.size} bytes ok", flush=True)
    return C_ref, M_ref


@pytest.fixture
def few_blocks(dt):
    """Sets how many blocks of a small tensor's encode are launched at a time
    (each launch ends before the next one starts), as if no more fitted."""
    yield dt.lib.tlc_stress_blocks
    dt.lib.tlc_stress_blocks(0)


@pytest.mark.parametrize("options", [0, 1], ids=["default", "in_place"])
@pytest.mark.parametrize("blocks", [0, 1, 2, 50])
def test_exchanging_tiles(dt, ctx, few_blocks, blocks, options):
    """Tensors of 2 to 128 tiles, whose tiles exchange maxima and summaries:
    with all blocks in one launch, and with so few at a time that the tiles a
    block waits for have not started (it then reads their values itself)."""
    import torch
    ctx.set_options(options)
    few_blocks(blocks)
    try:
        for k, n in enumerate([5 * 2048 * 128, 5 * 2048 * 128 - 3, 700_001, 5 * 2048 + 1]):
            # the largest value in the first tile, the last one and between
            x = workloads.normal([95, k], n, 1e-3)
            x[(n - 1) * k // 3] = F32(0.25)
            encode_check(ctx, x, workloads.normal([96, k], n, 1e-4), 1.25 + k / 8,
                         f"{n} values, {blocks} blocks at a time")
        x[n // 2] = np.nan  # refused by every tile
        r = workloads.normal([96, 9], n, 1e-4)
        rd = torch.from_numpy(r.copy()).cuda()
        with pytest.raises(dt.TLCError) as e:
            ctx.compress(torch.from_numpy(x).cuda(), rd, 1.5)
        assert e.value.code == dt.TLC_E_NONFINITE
        left = rd.cpu().numpy()
        want = r if not options else x + r
        ok = np.isfinite(want)
        assert np.array_equal(bits(left)[ok], bits(want)[ok])
    finally:
        ctx.set_options(0)


@pytest.mark.parametrize("n", [5 * 2048 * 128, 5 * 2048 * 128 + 1, 4_000_003, None])
def test_no_allocation_encode(dt, n):
    """128 exchanging tiles, then 65 to 410 of twice the size, chained by the
    block-wide look-back (lookback_block); None: the largest size."""
    import torch
    n = n or dt.TLC_NOALLOC_MAX_N
    x = workloads.normal([97, 0], n, 1e-3)
    x[n // 3:n // 2] = 0  # runs that cross tiles
    r = workloads.normal([97, 1], n, 1e-4)
    r[n // 3:n // 2] = 0
    m = dt.tlc_max_compressed_bytes(n)
    xd, rd = torch.from_numpy(x).cuda(), torch.from_numpy(r.copy()).cuda()
    buf = torch.zeros(m, dtype=torch.uint8, device="cuda")
    res = torch.zeros(4, dtype=torch.int32, device="cuda")
    st = dt.tlc_compress_noalloc(xd.data_ptr(), rd.data_ptr(), n, 1.5, buf.data_ptr(), m,
                                 res.data_ptr(), torch.cuda.current_stream().cuda_stream)
    assert st == dt.TLC_OK
    torch.cuda.synchronize()
    got = res.cpu().numpy()
    st, C_ref, M_ref = oracle.compress(x, r, 1.5)
    assert st == 0 and got[0] == dt.TLC_OK and got[1] == C_ref.size
    assert got[2:3].view(F32).tobytes() == F32(M_ref).tobytes()
    assert np.array_equal(buf[:C_ref.size].cpu().numpy(), C_ref)
    assert np.array_equal(bits(rd.cpu().numpy()), bits(r))
    print(f"no-allocation encode of {n} values ok", flush=True)


def test_three_pass_encoders(dt, ctx):
    # 400 tiles: the compaction combines the tiles' summaries itself
    n = 400 * 4096 * 5 - 3
    encode_check(ctx, workloads.normal([91, 0], n, 1e-3), workloads.normal([91, 1], n, 1e-4),
                 1.0, "three-pass, 400 tiles")
    # 2051 tiles: with the chunk pass (its last block scans the chunks)
    n = 2051 * 4096 * 5 - 7
    x = workloads.runs_tensor([91, 2], n)
    encode_check(ctx, x, np.zeros(n, F32), 1.5, "three-pass, 2051 tiles")
    n = 1 << 25
    encode_check(ctx, workloads.normal([91, 3], n, 1e-3), workloads.normal([91, 4], n, 1e-4),
                 1.0, "three-pass, m on the word grid")
    ctx.set_options(dt.TLC_OPT_IN_PLACE_FEEDBACK)  # bounds
    try:
        encode_check(ctx, workloads.normal([91, 5], n, 1e-3), workloads.normal([91, 6], n, 1e-4),
                     1.0, "three-pass in place")
    finally:
        ctx.set_options(0)


def test_batched_encoder(ctx):
    import torch
    sizes = workloads.c2_sizes()
    xs = [workloads.c2_gradient(0, t, n) for t, n in enumerate(sizes)]
    rs = [workloads.normal([92, t], n, 1e-5) for t, n in enumerate(sizes)]
    rd = [torch.from_numpy(r.copy()).cuda() for r in rs]
    pays = ctx.compress_batch([torch.from_numpy(x).cuda() for x in xs], rd, 1.75)
    for t, (x, r) in enumerate(zip(xs, rs)):
        st, C_ref, M_ref = oracle.compress(x, r, 1.75)
        assert st == 0 and pays[t][1] == M_ref, t
        assert np.array_equal(pays[t][0].cpu().numpy(), C_ref), t
        assert np.array_equal(bits(rd[t].cpu().numpy()), bits(r)), t
    print("batched encoder, 335 tensors ok", flush=True)


def test_batch_of_many_tiles(ctx):
    """Tensors of 128, 127, 2 and 33 exchanging tiles and of one, with one of
    400 larger tiles, which takes the three passes, in one call."""
    import torch
    T = 5 * 2048
    sizes = [128 * T, 500, 127 * T - 1, 800 * T - 3, T + 1, 33 * T, T]
    xs = [workloads.normal([98, t], n, 1e-3) for t, n in enumerate(sizes)]
    rs = [workloads.normal([99, t], n, 1e-4) for t, n in enumerate(sizes)]
    rd = [torch.from_numpy(r.copy()).cuda() for r in rs]
    pays = ctx.compress_batch([torch.from_numpy(x).cuda() for x in xs], rd, 1.25)
    for t, (x, r) in enumerate(zip(xs, rs)):
        st, C_ref, M_ref = oracle.compress(x, r, 1.25)
        assert st == 0 and pays[t][1] == M_ref, t
        assert np.array_equal(pays[t][0].cpu().numpy(), C_ref), t
        assert np.array_equal(bits(rd[t].cpu().numpy()), bits(r)), t
    print("batch of many tiles ok", flush=True)


def test_decoder_index_scans(ctx):
    """Streams of synthetic quartic bytes with half of them data bytes, so
    each stream spans about 160 index tiles; single, batched and summed
    decodes with accumulate.  The single decode's expanding blocks wait for
    start entries that are published late and out of order (the stress
    build delays them like status words)."""
    import torch
    n = (1 << 23) + 3
    m = oracle.quartic_len(n)
    streams = []
    for k in range(3):
        rng = np.random.default_rng([93, k])
        Q = np.full(m, 121, np.uint8)
        hit = rng.random(m) < 0.5
        Q[hit] = rng.integers(0, 243, int(hit.sum()), dtype=np.uint8)
        streams.append((oracle.zre_encode(Q), F32(1e-3 * (k + 1))))
    out0 = workloads.normal([94, 0], n, 1e-3)
    for C, M in streams:
        od = torch.from_numpy(out0.copy()).cuda()
        ctx.decompress(torch.from_numpy(C).cuda(), M, n, od, accumulate=True)
        ctx.sync()
        st, ref = oracle.decompress(C, M, n, out0.copy(), True)
        assert st == 0 and np.array_equal(bits(od.cpu().numpy()), bits(ref))
    print(f"single decodes ok ({streams[0][0].size} stream bytes each)", flush=True)
    outs = [torch.from_numpy(out0.copy()).cuda() for _ in streams]
    ctx.decompress_batch([torch.from_numpy(C).cuda() for C, _ in streams],
                         [M for _, M in streams], outs, accumulate=True)
    ctx.sync()
    for (C, M), o in zip(streams, outs):
        st, ref = oracle.decompress(C, M, n, out0.copy(), True)
        assert np.array_equal(bits(o.cpu().numpy()), bits(ref))
    total = torch.from_numpy(out0.copy()).cuda()
    ctx.decompress_sum([torch.from_numpy(C).cuda() for C, _ in streams],
                       [M for _, M in streams], total, accumulate=True)
    ctx.sync()
    ref = out0.copy()
    for C, M in streams:
        st, ref = oracle.decompress(C, M, n, ref, True)
    assert np.array_equal(bits(total.cpu().numpy()), bits(ref))
    print("batched and summed decodes ok", flush=True)
