"""bload_segment_scan on the GPU against the oracle's recurrence, element by element.

Bound used throughout (float32 arithmetic in time order, states handed across chunks of time as
decay^chunk * state + the chunk's own part, against the oracle's double): at the k-th slot of a
block (k counted from 1, an upper bound of the frame's place in its sequence)
|gpu - oracle| <= (3k + 4) * 2^-24 * S, S = the same recurrence on |x| with |decay|.
"""
import numpy as np
import pytest
import torch

import oracle
from paper_2310_10879_amd import workloads
from gpu_util import binding, gpu_plan, to_dev
from test_gpu_reduce import draw_source, random_flags

pytestmark = pytest.mark.gpu
EPS = 2.0 ** -24


def assert_scan_close(got, ref, scale, what):
    B, T, D = ref.shape
    k = np.arange(1, T + 1, dtype=np.float64)[None, :, None]
    bound = (3 * k + 4) * EPS * scale.astype(np.float64)
    err = np.abs(got.astype(np.float64) - ref.astype(np.float64))
    bad = err > bound
    if bad.any():
        at = tuple(np.argwhere(bad)[0])
        raise AssertionError(f"{what}: {int(bad.sum())} outside the bound, first at {at}: got {got[at]} "
                             f"want {ref[at]} bound {bound[at]}")


def gpu_scan(packed_np, reset, valid, D, dtype, decay):
    bl = binding()
    B, T = valid.shape
    out = torch.full((B, T, D), float("nan"), dtype=torch.float32, device="cuda")
    bl.bload_segment_scan(to_dev(packed_np.view(np.uint8).reshape(-1)), to_dev(reset), to_dev(valid), B, T, D,
                          dtype, decay, out=out)
    torch.cuda.synchronize()
    return out.cpu().numpy()


@pytest.mark.parametrize("dtype", ["u8", "f16", "f32"])
@pytest.mark.parametrize("B,T,D", [(1, 1, 1), (3, 10, 1), (700, 33, 1), (40, 5000, 1), (9, 4096, 2),
                                   (70, 130, 3), (300, 130, 16), (50, 700, 80), (60, 300, 100),
                                   (20, 3000, 256), (64, 32, 3072), (5, 257, 1040),
                                   # fewer than 8 slots in all, exactly 8, blocks shorter than 8 slots
                                   (2, 3, 5), (1, 7, 4), (1, 8, 4), (3, 5, 8), (11, 7, 16)])
def test_scan_follows_the_flags(B, T, D, dtype):
    rng = np.random.default_rng(B + T + D)
    for (p_valid, p_reset), decay in zip([(0.85, 0.02), (0.5, 0.3), (1.0, 0.0)], [0.9, -0.5, 1.0]):
        print(f"scan B={B} T={T} D={D} {dtype} valid {p_valid} reset {p_reset} decay {decay}", flush=True)
        valid, reset, _, _ = random_flags(rng, B, T, p_valid, p_reset)
        src = draw_source(rng, B * T, D, dtype)            # payload in every slot, padding included
        ref, scale = oracle.segment_scan_packed(src, reset, valid, D, dtype, decay)
        got = gpu_scan(src, reset, valid, D, dtype, decay)
        assert not got[valid == 0].any()                   # padding yields exact zeros
        assert_scan_close(got, ref, scale, f"{dtype} B={B} T={T} D={D}")


@pytest.mark.parametrize("wid", [1, 2, 3])
def test_scan_of_packed_workloads(wid):
    """Plan, pack and scan on the GPU; the oracle's recurrence on the ragged source, carried to the
    slots through the oracle's own pack tables, is the reference (sampled blocks at full size)."""
    bl = binding()
    w = workloads.WORKLOADS[wid]
    L = workloads.lengths(wid)
    so = workloads.src_offsets(L)
    src = workloads.source(wid, 0, int(so[-1]))
    D, T, F = w.frame_elems, w.t_blk, w.frame_bytes
    plan_dev = gpu_plan(L, T, 0)
    d_src = to_dev(src.view(np.uint8).reshape(-1))
    out = bl.bload_pack(d_src, to_dev(so), to_dev(L), plan_dev, F)
    decay = 0.97
    h = bl.bload_segment_scan(out.packed, out.reset, out.valid, plan_dev.num_blocks, T, D, w.dtype, decay)
    torch.cuda.synchronize()
    ref_plan = oracle.plan(L, T, oracle.order(w.n_seq, 0))
    rng = np.random.default_rng(wid)
    blocks = sorted(set([0, ref_plan.num_blocks - 1] +
                        rng.integers(0, ref_plan.num_blocks, size=6).tolist()))
    for b in blocks:
        print(f"scan workload {wid} block {b}", flush=True)
        packed, seq_id, frame_idx, reset, valid = oracle.pack_blocks(src, so, L, ref_plan, F, b, b + 1)
        seqs = ref_plan.order[ref_plan.block_first[b]:ref_plan.block_first[b + 1]]
        ref = np.zeros((1, T, D), np.float32)
        scale = np.zeros((1, T, D), np.float32)
        for i in seqs:                                      # the ragged definition, sequence by sequence
            hi, si = oracle.segment_scan(src[so[i]:so[i + 1]], np.array([0, L[i]]), L[i:i + 1], D, w.dtype, decay)
            o = ref_plan.offset_of_seq[i]
            ref[0, o:o + L[i]] = hi
            scale[0, o:o + L[i]] = si
        got = h[b:b + 1].cpu().numpy()
        assert not got[valid == 0].any()
        assert_scan_close(got, ref, scale, f"workload {wid} block {b}")


# Where the tiles of the two kernels end: frames of 63 / 64 / 65 elements (through LDS, whole quads, a
# last quad that lies over its neighbour), more than one slice of 64 quads, blocks of a tile's
# length and one slot more, enough blocks that every XCD takes whole ones, and single long blocks.
TILE_EDGES = [(3, 132, 63, "f16"), (3, 133, 63, "f32"), (2, 528, 64, "u8"), (2, 129, 64, "f32"), (5, 513, 65, "f16"),
              (300, 140, 66, "u8"), (1, 3000, 131, "f32"), (2, 300, 259, "u8"), (3, 130, 1031, "f16"),
              (1, 8448, 1, "f32"), (1, 20000, 1, "u8"), (2, 2305, 1, "f16"), (700, 2400, 1, "u8"), (290, 800, 7, "f32"),
              (257, 1100, 64, "u8"), (1, 2, 64, "u8"), (1, 15, 1, "f32"), (1, 17, 1, "f16")]


# Smaller frames go with 9, 17, 21, 25, 29 or 33 slots a lane: blocks that fill a tile of six or of four groups of
# lanes at each length and one slot more, one block a tile and several, and a tensor read with plain loads.
TILE_EDGES += [(900 if T < 100 else 600, T, 37, "f16") for T in (54, 55, 102, 103, 126, 127, 150, 151, 174, 175, 198, 199, 340)]
TILE_EDGES += [(7, 68, 63, "u8"), (800, 84, 63, "f32"), (3, 116, 57, "f32"), (2700, 100, 63, "f32")]


@pytest.mark.parametrize("B,T,D,dtype", TILE_EDGES)
def test_scan_tile_edges(B, T, D, dtype):
    """Flags with long runs that cross several tiles and flags without a start at all."""
    rng = np.random.default_rng(B + 3 * T + D)
    for p_valid, p_reset, decay in [(1.0, 0.0, 1.0), (0.999, 0.004, 0.9)]:
        print(f"scan edges B={B} T={T} D={D} {dtype} valid {p_valid} reset {p_reset}", flush=True)
        valid, reset, _, _ = random_flags(rng, B, T, p_valid, p_reset)
        src = draw_source(rng, B * T, D, dtype)
        ref, scale = oracle.segment_scan_packed(src, reset, valid, D, dtype, decay)
        got = gpu_scan(src, reset, valid, D, dtype, decay)
        assert not got[valid == 0].any()
        assert_scan_close(got, ref, scale, f"{dtype} B={B} T={T} D={D}")


@pytest.mark.parametrize("B,T,D,dtype", [(3, 700, 80, "f32"), (2, 600, 70, "u8"), (2, 9000, 1, "f16"), (5, 400, 33, "f32")])
def test_scan_without_a_word_from_the_tiles_in_front(B, T, D, dtype):
    """A library whose wait for other workgroups ends at once: every tile computes the ones in front
    of it itself, and gets the same bits."""
    import ctypes
    import os
    bl = binding()
    lib = ctypes.CDLL(os.path.join(os.path.dirname(bl.LIB_PATH), "libbload_scan_nowait.so"))
    fn = lib.bload_segment_scan
    fn.restype, fn.argtypes = ctypes.c_int, bl._lib.bload_segment_scan.argtypes
    rng = np.random.default_rng(B + T + D)
    for p_valid, p_reset in [(1.0, 0.0), (0.999, 0.004)]:
        valid, reset, _, _ = random_flags(rng, B, T, p_valid, p_reset)
        src = draw_source(rng, B * T, D, dtype)
        want = gpu_scan(src, reset, valid, D, dtype, 0.99)
        x, r, v = to_dev(src.view(np.uint8).reshape(-1)), to_dev(reset), to_dev(valid)
        out = torch.full((B, T, D), float("nan"), dtype=torch.float32, device="cuda")
        ws = torch.empty(max(16, bl.bload_segment_scan_workspace_bytes(B, T, D, dtype)), dtype=torch.uint8, device="cuda")
        assert fn(x.data_ptr(), r.data_ptr(), v.data_ptr(), B, T, D, bl.DTYPES[dtype], 0.99, out.data_ptr(),
                  ws.data_ptr(), ws.numel(), torch.cuda.current_stream().cuda_stream) == 0
        torch.cuda.synchronize()
        assert np.array_equal(out.cpu().numpy(), want)


def test_scan_state_beyond_float_powers():
    """decay^chunk overflows float32 while the state does not, underflows it under an infinite
    state, and a state of 0 meets an infinite power."""
    T = 20000
    valid, reset = np.ones((1, T), np.uint8), np.zeros((1, T), np.uint8)
    x = np.zeros((1, T, 1), np.float32)
    x[0, 1, 0] = np.float32(1e-30)
    got = gpu_scan(x, reset, valid, 1, "f32", 1.0125)
    ref, _ = oracle.segment_scan_packed(x.reshape(T, 1), reset, valid, 1, "f32", float(np.float32(1.0125)))
    k = np.arange(1, T + 1)
    fine = np.abs(ref[0, :, 0]) < 1e38
    assert np.all(np.abs(got[0, fine, 0].astype(np.float64) - ref[0, fine, 0]) <= (3 * k[fine] + 4) * EPS * np.abs(ref[0, fine, 0]))
    x[0, 1, 0] = np.inf
    got = gpu_scan(x, reset, valid, 1, "f32", 0.5)
    assert got[0, 0, 0] == 0 and np.isposinf(got[0, 1:, 0]).all()
    x[0, 1, 0] = 0
    assert not gpu_scan(x, reset, valid, 1, "f32", 1e9).any()


def serial_float32(x, decay):
    """The recurrence from end to end in float32, one rounding a step (the product and sum are exact in double)."""
    h = np.zeros_like(x)
    state = np.zeros((x.shape[0], x.shape[2]), np.float32)
    for t in range(x.shape[1]):
        state = (np.float64(decay) * state + x[:, t]).astype(np.float32)
        h[:, t] = state
    return h


@pytest.mark.parametrize("B,T,D,decay", [(60, 3000, 80, 0.9), (400, 3000, 9, 0.9), (90, 2000, 64, -0.97)])
def test_scan_hand_over_costs_no_accuracy(B, T, D, decay):
    """States cross the borders of stretches and tiles in 64 bits: against the double recurrence the result is as
    close as a float32 recurrence without any border (a million elements and more: the ratio of the root mean
    squares is good to 0.2 %; a hand-over in float32 costs 3 %)."""
    decay = float(np.float32(decay))
    x = np.random.default_rng(D).normal(size=(B, T, D)).astype(np.float32)
    valid, reset = np.ones((B, T), np.uint8), np.zeros((B, T), np.uint8)
    got, serial = gpu_scan(x, reset, valid, D, "f32", decay), serial_float32(x, decay)
    state, err, base = np.zeros((B, D)), 0.0, 0.0
    for t in range(T):
        state = decay * state + x[:, t]
        err += np.square(got[:, t] - state).sum()
        base += np.square(serial[:, t] - state).sum()
    print(f"B={B} T={T} D={D}: {np.sqrt(err / base):.4f}", flush=True)
    assert np.sqrt(err / base) <= 1.01


@pytest.mark.parametrize("T,D", [(20000, 1), (700, 7), (1200, 64)])
def test_scan_infinite_states(T, D):
    """A state that leaves the range of float32 stays infinite, wherever borders lie between; and under decay 0 an
    infinite value, in the last slot of a stretch as anywhere, makes NaN of the rest of its sequence."""
    at = [10, T // 4]
    x = np.zeros((1, T, D), np.float32)
    x[0, at] = 3e38
    valid, reset = np.ones((1, T), np.uint8), np.zeros((1, T), np.uint8)
    got = gpu_scan(x, reset, valid, D, "f32", 1.0)
    assert not got[0, :at[0]].any() and (got[0, at[0]:at[1]] == np.float32(3e38)).all() and np.isposinf(got[0, at[1]:]).all()
    for last in (8, 31, 32, 33, 65, 32 * 16 - 1, T // 2):
        x[:] = 1.0
        x[0, last] = np.inf
        got = gpu_scan(x, reset, valid, D, "f32", 0.0)
        assert (got[0, :last] == 1).all() and np.isposinf(got[0, last]).all() and np.isnan(got[0, last + 1:]).all()


# Less workspace than asked for, down to what is accepted (`room` bytes): a workgroup walks its block tile by tile.
# Frames under and from 64 elements on, one slice and several, blocks of two tiles and of many, the last one short.
@pytest.mark.parametrize("B,T,D,dtype,room", [(6144, 140, 63, "f32", 0), (12288, 270, 31, "u8", 0), (3072, 280, 130, "f32", 0),
                                              (700, 300, 63, "f32", 531312), (40, 1000, 4100, "f16", 1312080),
                                              (3, 4500, 1000, "f16", 744192), (6143, 140, 63, "f16", 1554192)])
def test_scan_with_less_workspace_than_asked_for(B, T, D, dtype, room):
    bl = binding()
    asked = bl.bload_segment_scan_workspace_bytes(B, T, D, dtype)
    assert room < asked
    rng = np.random.default_rng(B + T + D)
    for (p_valid, p_reset), decay in zip([(1.0, 0.0), (0.97, 0.01)], [0.999, -0.5]):
        valid, reset, _, _ = random_flags(rng, B, T, p_valid, p_reset)
        src = draw_source(rng, B * T, D, dtype)
        ref, scale = oracle.segment_scan_packed(src, reset, valid, D, dtype, decay)
        x, r, v = to_dev(src.view(np.uint8).reshape(-1)), to_dev(reset), to_dev(valid)
        print(f"room {room} of {asked}: B={B} T={T} D={D} {dtype}", flush=True)
        for take in (room, room - 1):
            out = torch.full((B, T, D), float("nan"), dtype=torch.float32, device="cuda")
            ws = torch.empty(max(room, 16), dtype=torch.uint8, device="cuda")
            st = bl._lib.bload_segment_scan(x.data_ptr(), r.data_ptr(), v.data_ptr(), B, T, D, bl.DTYPES[dtype], decay,
                                            out.data_ptr(), ws.data_ptr() if take > 0 else None, max(take, 0),
                                            torch.cuda.current_stream().cuda_stream)
            if take < room and room > 0:
                assert st == bl.EWORKSPACE
                continue
            assert st == bl.OK
            got = out.cpu().numpy()
            assert not got[valid == 0].any()
            assert_scan_close(got, ref, scale, f"{dtype} B={B} T={T} D={D}")
            if D >= 64:                                    # the same stretches: the same bits
                assert np.array_equal(got.view(np.int32), gpu_scan(src, reset, valid, D, dtype, decay).view(np.int32))


def test_scan_closed_forms_and_determinism():
    bl = binding()
    B, T, D = 7, 200, 64
    valid = np.ones((B, T), np.uint8)
    reset = np.zeros((B, T), np.uint8)
    reset[:, ::20] = 1
    x = np.full((B, T, D), 3.0, np.float32)
    t_in_seg = (np.arange(T) % 20)[None, :, None]
    for decay, want in ((0.0, x), (1.0, 3.0 * (t_in_seg + 1) + 0 * x), (0.5, 6.0 * (1 - 0.5 ** (t_in_seg + 1)) + 0 * x)):
        got = gpu_scan(x, reset, valid, D, "f32", decay)
        assert np.array_equal(got, want.astype(np.float32))       # all exact in float32
    rng = np.random.default_rng(1)
    x = rng.normal(size=(B, T, D)).astype(np.float32)
    a = gpu_scan(x, reset, valid, D, "f32", 0.8)
    b = gpu_scan(x, reset, valid, D, "f32", 0.8)
    assert np.array_equal(a, b)
    # a non-finite state does not leak across a start
    x[:, 19] = np.inf
    got = gpu_scan(x, reset, valid, D, "f32", 0.8)
    assert np.isfinite(got[:, 20:]).all() and np.isinf(got[:, 19]).all()


def test_scan_errors():
    bl = binding()
    z = torch.zeros(64, dtype=torch.uint8, device="cuda")
    with pytest.raises(bl.BloadError) as e:
        bl.bload_segment_scan(z, z, z, 1, 4, 4, "i32", 0.5)
    assert e.value.status == bl.EINVAL
    with pytest.raises(bl.BloadError) as e:
        bl.bload_segment_scan(z[1:], z, z, 1, 4, 4, "f32", 0.5)
    assert e.value.status == bl.EALIGN
    assert bl.bload_segment_scan(z, z, z, 0, 4, 4, "f32", 0.5).numel() == 0


# Frames of several slices whose output is whole cache lines: slices of 10 and 8, 16 and 14, 22, 22 and 22 groups of eight
# features, beside one feature more or less, whose tiles pass the cache by another way; then with the workspace that slices
# of equal width need (a state per feature, 8 bytes, behind each but the last of a block's tiles of 32 slots a lane), if it is less.
@pytest.mark.parametrize("dtype", ["u8", "f16", "f32"])
@pytest.mark.parametrize("B,T,D", [(400, 300, 288), (40, 700, 480), (40, 700, 479), (700, 129, 704), (300, 260, 270), (1200, 90, 100)])
def test_scan_slices_of_whole_lines(B, T, D, dtype):
    bl = binding()
    asked = bl.bload_segment_scan_workspace_bytes(B, T, D, dtype)
    units = -(-D // 4)
    groups = 256 // -(-units // -(-units // 64))
    tiles = -(-T // (32 * groups))
    tiles = -(-T // (32 * -(-(-(-T // tiles)) // 32)))
    equal = (B * (tiles - 1) * D * 8 + 15) // 16 * 16
    assert equal <= asked
    rng = np.random.default_rng(B + T + D)
    valid, reset, _, _ = random_flags(rng, B, T, 0.97, 0.01)
    src = draw_source(rng, B * T, D, dtype)
    ref, scale = oracle.segment_scan_packed(src, reset, valid, D, dtype, 0.95)
    x, r, v = to_dev(src.view(np.uint8).reshape(-1)), to_dev(reset), to_dev(valid)
    for room in sorted({asked, equal}):
        out = torch.full((B, T, D), float("nan"), dtype=torch.float32, device="cuda")
        ws = torch.empty(max(room, 16), dtype=torch.uint8, device="cuda")
        print(f"scan B={B} T={T} D={D} {dtype} workspace {room} of {asked}", flush=True)
        st = bl._lib.bload_segment_scan(x.data_ptr(), r.data_ptr(), v.data_ptr(), B, T, D, bl.DTYPES[dtype], 0.95, out.data_ptr(),
                                        ws.data_ptr(), room, torch.cuda.current_stream().cuda_stream)
        assert st == bl.OK
        got = out.cpu().numpy()
        assert not got[valid == 0].any()
        assert_scan_close(got, ref, scale, f"{dtype} B={B} T={T} D={D}")
