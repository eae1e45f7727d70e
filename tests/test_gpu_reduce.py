"""bload_segment_reduce on the GPU against the oracle's per-sequence sums / means
(computed in float64 from the ragged source, never from the packed tensor)."""
import numpy as np
import pytest
import torch

import oracle
from paper_2310_10879_amd import workloads
from gpu_util import binding, gpu_plan, to_dev

pytestmark = pytest.mark.gpu

NP_OF = {"u8": np.uint8, "f16": np.float16, "f32": np.float32, "i32": np.int32}
REL_TOL = 1e-5          # the bar for float32 reductions


def draw_source(rng, total, D, dtype):
    if dtype == "u8":
        return rng.integers(0, 256, size=(total, D), dtype=np.uint8)
    if dtype == "f16":
        return rng.standard_normal((total, D), dtype=np.float32).astype(np.float16)
    if dtype == "f32":
        return (rng.standard_normal((total, D), dtype=np.float32) * 2 - 4).astype(np.float32)
    return rng.integers(-2_000_000_000, 2_000_000_000, size=(total, D), dtype=np.int32)


def check_reduction(got, src, so, L, D, dtype, op):
    """|gpu - oracle| <= 1e-5 * max(|oracle|, A), A = mean|x| (mean) or sum|x| (sum) of the
    segment: the relative bar, with the scale of the summands as floor because a
    mean near zero has no relative accuracy in any finite-precision sum."""
    ref = oracle.segment_reduce(src, so, L, D, dtype, op)
    if dtype == "i32":
        assert got.dtype == np.int64
        assert np.array_equal(got, ref)
        return
    assert got.dtype == np.float32
    scale = np.add.reduceat(np.abs(src.astype(np.float64)), so[:-1], axis=0)
    if op == "mean":
        scale = scale / L[:, None]
    bound = REL_TOL * np.maximum(np.abs(ref.astype(np.float64)), scale)
    err = np.abs(got.astype(np.float64) - ref.astype(np.float64))
    worst = np.unravel_index(np.argmax(err - bound), err.shape)
    assert np.all(err <= bound), (f"worst at {worst}: got {got[worst]} want {ref[worst]} "
                                  f"err {err[worst]} bound {bound[worst]}")
    if dtype == "u8":
        if op == "sum":         # integer sums below 2^24 are exact in float32
            assert np.array_equal(got, ref)
        else:                   # one rounding of an exact quotient on either side
            assert np.all(err <= np.spacing(np.abs(ref)))


def reduce_case(n, T, D, dtype, op, kind, seed=0, poison=False):
    bl = binding()
    rng = np.random.default_rng(n * 13 + T * 5 + D)
    L = workloads.random_lengths(rng, n, T, kind)
    so = workloads.src_offsets(L)
    src = draw_source(rng, int(so[-1]), D, dtype)
    F = D * src.dtype.itemsize
    pl = oracle.plan(L, T, oracle.order(n, seed))
    packed, seq_id, frame_idx, reset, valid = oracle.pack(src, so, L, pl, F)
    if poison:      # garbage in the padding payload must not reach any sum
        packed = packed.copy()
        packed[valid == 0] = 0x7B
    out = bl.bload_segment_reduce(to_dev(packed), to_dev(seq_id), to_dev(reset), to_dev(valid),
                                  pl.num_blocks, T, D, dtype, op, n)
    torch.cuda.synchronize()
    check_reduction(out.cpu().numpy(), src, so, L, D, dtype, op)
    return out


CASES = [  # n, T, D: wide rows of every width, several time chunks, narrow tiles across blocks
    (1, 1, 1), (5, 7, 1), (300, 33, 1), (40, 5000, 1), (2000, 100, 1), (90, 4096, 1),
    (300, 33, 3), (60, 600, 5), (64, 32, 16), (64, 32, 17), (200, 130, 64), (100, 300, 80),
    (150, 64, 100), (80, 200, 192), (30, 3000, 256), (25, 700, 300), (12, 3000, 2048),
    (64, 32, 3072),
]


@pytest.mark.parametrize("dtype,op", [("u8", "mean"), ("u8", "sum"), ("f16", "mean"),
                                      ("f32", "mean"), ("f32", "sum"), ("i32", "sum")])
@pytest.mark.parametrize("n,T,D", CASES)
def test_reduce_matches_oracle(n, T, D, dtype, op):
    if n * T * D > 60_000_000:
        n = max(1, 60_000_000 // (T * D))
    for kind in ("uniform", "mixed"):
        print(f"reduce n={n} T={T} D={D} {dtype} {op} {kind}", flush=True)
        reduce_case(n, T, D, dtype, op, kind)


@pytest.mark.parametrize("n,T,D,dtype", [(200, 130, 64, "f32"), (300, 33, 1, "i32"),
                                         (30, 3000, 256, "u8"), (40, 5000, 2, "f16")])
def test_reduce_ignores_padding_payload(n, T, D, dtype):
    reduce_case(n, T, D, dtype, "sum", "uniform", poison=True)


def test_reduce_long_and_short_segments():
    for kind in ("short", "long"):
        reduce_case(3000, 4096, 1, "i32", "sum", kind)
        reduce_case(400, 512, 128, "f32", "mean", kind)


def test_reduce_closed_forms():
    # payload = sequence index: every mean gives the index back, so a frame taken
    # across a boundary (or a chunk stitched to the wrong sequence) shows
    bl = binding()
    for n, T, D, dtype in [(500, 700, 1, "f32"), (40, 3000, 256, "f32"), (700, 100, 2, "i32")]:
        rng = np.random.default_rng(n)
        L = workloads.random_lengths(rng, n, T, "mixed")
        so = workloads.src_offsets(L)
        src = np.repeat(np.arange(n), L)[:, None].repeat(D, axis=1).astype(NP_OF[dtype])
        pl = oracle.plan(L, T, oracle.order(n, 7))
        packed, seq_id, _, reset, valid = oracle.pack(src, so, L, pl, D * 4)
        op = "sum" if dtype == "i32" else "mean"
        out = bl.bload_segment_reduce(to_dev(packed), to_dev(seq_id), to_dev(reset),
                                      to_dev(valid), pl.num_blocks, T, D, dtype, op, n)
        got = out.cpu().numpy()
        want = np.arange(n)[:, None] * (L[:, None] if dtype == "i32" else 1)
        assert np.array_equal(got, np.broadcast_to(want, (n, D)).astype(got.dtype))


def test_reduce_is_deterministic_and_reports_errors():
    bl = binding()
    a = reduce_case(25, 700, 300, "f32", "mean", "uniform")
    b = reduce_case(25, 700, 300, "f32", "mean", "uniform")
    assert torch.equal(a, b)
    x = torch.zeros(16, dtype=torch.uint8, device="cuda:0")
    i = torch.zeros(4, dtype=torch.int32, device="cuda:0")
    with pytest.raises(bl.BloadError) as e:       # int32 mean is not defined
        bl.bload_segment_reduce(x, i, x[:4], x[:4], 1, 4, 1, "i32", "mean", 1)
    assert e.value.status == bl.EINVAL


@pytest.mark.parametrize("wid", [1, 2, 3, 5])
def test_reduce_workloads_full_size(wid):
    # plan + pack + reduce on the device at full size; the oracle sums the ragged source
    bl = binding()
    w = workloads.WORKLOADS[wid]
    L = workloads.lengths(wid)
    so = workloads.src_offsets(L)
    src = workloads.source(wid, 0, int(so[-1]))
    print(f"reduce workload {wid}", flush=True)
    plan_dev = gpu_plan(L, w.t_blk, 0)
    out = bl.bload_pack(to_dev(src.view(np.uint8).reshape(-1)), to_dev(so), to_dev(L), plan_dev,
                        w.frame_bytes)
    red = bl.bload_segment_reduce(out.packed, out.seq_id, out.reset, out.valid,
                                  plan_dev.num_blocks, w.t_blk, w.frame_elems, w.dtype, w.op,
                                  w.n_seq)
    torch.cuda.synchronize()
    check_reduction(red.cpu().numpy(), src, so, L, w.frame_elems, w.dtype, w.op)


# ---- float32 sums that are accurate by construction, not by the luck of random rounding

U = 2.0 ** -24          # unit roundoff of float32


def same_sign_source(rng, total, D):
    """Positive float32 values over six decades, every 97th frame a huge one in front of
    thousands of small ones: a single float32 accumulator per feature loses the small terms
    (error ~ n/2 units in the last place of the sum), which is what must not happen."""
    x = np.exp(rng.uniform(np.log(1e-3), np.log(1e3), size=(total, D))).astype(np.float32)
    x[::97] *= np.float32(4096.0)
    return x


def assert_sum_accuracy(got, src, so, L, D, op, ulps):
    """Against the float64 oracle: inside the 1e-5 bar, and inside `ulps` units of float32
    roundoff of sum |x| (what the summation scheme guarantees at any length)."""
    ref = oracle.segment_reduce(src, so, L, D, "f32", op).astype(np.float64)
    scale = np.add.reduceat(np.abs(src.astype(np.float64)), so[:-1], axis=0)
    if op == "mean":
        scale = scale / L[:, None]
    err = np.abs(got.astype(np.float64) - ref)
    assert np.all(err <= REL_TOL * np.maximum(np.abs(ref), scale)), f"max relative error {np.max(err / scale)}"
    assert np.all(err <= ulps * U * scale), f"{np.max(err / (U * scale)):.1f} units of roundoff, allowed {ulps}"


@pytest.mark.parametrize("n,T,D,ulps", [(48, 3000, 80, 12),      # lanes across features, many chunks + stitch
                                        (300, 3000, 80, 12),     # fewer chunks per block
                                        (6, 3000, 2048, 12),     # a wave per row
                                        (40, 30000, 1, 48),      # lanes across time, 8 tiles per sequence
                                        (64, 3000, 3, 48)])
@pytest.mark.parametrize("op", ["sum", "mean"])
def test_reduce_float32_sums_hold_at_any_length(n, T, D, ulps, op):
    bl = binding()
    rng = np.random.default_rng(T + D)
    L = np.full(n, T, dtype=np.int32)                 # every sequence fills a block
    so = workloads.src_offsets(L)
    src = same_sign_source(rng, int(so[-1]), D)
    pl = oracle.plan(L, T, oracle.order(n, 3))
    packed, seq_id, _, reset, valid = oracle.pack(src, so, L, pl, D * 4)
    out = bl.bload_segment_reduce(to_dev(packed), to_dev(seq_id), to_dev(reset), to_dev(valid),
                                  pl.num_blocks, T, D, "f32", op, n)
    assert_sum_accuracy(out.cpu().numpy(), src, so, L, D, op, ulps)


def test_reduce_float32_one_chunk_per_block_of_3000_frames():
    """8192 blocks of one 3000-frame sequence of 80 float32 features: enough blocks that every
    block is one chunk, so a sequence is summed by one row of lanes from end to end (the launch
    shape of the largest workload).  The payload is drawn on the device; the oracle sums sampled
    sequences copied back from it."""
    bl = binding()
    B, T, D = 8192, 3000, 80
    assert bl.bload_segment_reduce_workspace_bytes(B, T, D, "f32") == 0       # no chunk borders
    g = torch.Generator(device="cuda:0").manual_seed(5)
    x = torch.empty((B, T, D), dtype=torch.float32, device="cuda:0")
    x.uniform_(float(np.log(1e-3)), float(np.log(1e3)), generator=g).exp_()
    x[:, ::97] *= 4096.0
    seq_id = torch.arange(B, dtype=torch.int32, device="cuda:0")[:, None].expand(B, T).contiguous()
    valid = torch.ones((B, T), dtype=torch.uint8, device="cuda:0")
    reset = torch.zeros((B, T), dtype=torch.uint8, device="cuda:0")
    reset[:, 0] = 1
    out = bl.bload_segment_reduce(x, seq_id, reset, valid, B, T, D, "f32", "mean", B)
    pick = np.unique(np.concatenate([[0, B - 1], np.random.default_rng(1).integers(0, B, size=62)]))
    src = x[torch.from_numpy(pick).to("cuda:0")].cpu().numpy().reshape(-1, D)
    L = np.full(len(pick), T, dtype=np.int32)
    assert_sum_accuracy(out[torch.from_numpy(pick).to("cuda:0")].cpu().numpy(), src,
                        workloads.src_offsets(L), L, D, "mean", 12)


# ---- arbitrary flags: the consumer's rule, not only what a correct pack writes

def random_flags(rng, B, T, p_valid, p_reset):
    """valid / reset planes with runs of padding anywhere, start flags anywhere, and a seq_id
    plane that gives every segment of the consumer's rule its own row."""
    valid = (rng.random((B, T)) < p_valid).astype(np.uint8)
    # make padding come in runs so that long segments exist too
    keep = rng.random((B, T)) < 0.9
    for t in range(1, T):
        valid[:, t] = np.where(keep[:, t], valid[:, t - 1], valid[:, t])
    reset = ((rng.random((B, T)) < p_reset) & (valid == 1)).astype(np.uint8)
    prev_valid = np.concatenate([np.zeros((B, 1), np.uint8), valid[:, :-1]], axis=1)
    starts = (valid == 1) & ((reset == 1) | (prev_valid == 0))
    starts[:, 0] = valid[:, 0] == 1
    ids = np.cumsum(starts.reshape(-1)).reshape(B, T) - 1
    seq_id = np.where(valid == 1, ids, -1).astype(np.int32)
    return valid, reset, seq_id, int(starts.sum())


@pytest.mark.parametrize("dtype,op", [("f32", "mean"), ("i32", "sum"), ("u8", "sum"), ("f16", "mean")])
@pytest.mark.parametrize("B,T,D", [(3, 10, 1), (700, 33, 1), (40, 5000, 1), (9, 4096, 2),
                                   (300, 130, 16), (50, 700, 80), (20, 3000, 256), (64, 32, 3072)])
def test_reduce_follows_the_flags(B, T, D, dtype, op):
    bl = binding()
    rng = np.random.default_rng(B + T + D)
    for p_valid, p_reset in [(0.85, 0.02), (0.5, 0.3), (1.0, 0.0)]:
        valid, reset, seq_id, n_seg = random_flags(rng, B, T, p_valid, p_reset)
        src = draw_source(rng, B * T, D, dtype)          # payload in every slot, padding included
        packed = src.reshape(B, T, D)
        want, counted = oracle.segment_reduce_packed(packed, seq_id, reset, valid, D, dtype, op, n_seg)
        assert counted == n_seg
        print(f"flags B={B} T={T} D={D} {dtype} {op} valid~{p_valid} reset~{p_reset} segments={n_seg}",
              flush=True)
        if n_seg == 0:
            continue
        got = bl.bload_segment_reduce(to_dev(packed), to_dev(seq_id), to_dev(reset), to_dev(valid),
                                      B, T, D, dtype, op, n_seg).cpu().numpy()
        if dtype == "i32":
            assert np.array_equal(got, want)
            continue
        absval = np.abs(packed.astype(np.float64)).astype(np.float32)
        scale, _ = oracle.segment_reduce_packed(absval, seq_id, reset, valid, D, "f32", op, n_seg)
        bound = REL_TOL * np.maximum(np.abs(want.astype(np.float64)), scale.astype(np.float64)) + 1e-30
        err = np.abs(got.astype(np.float64) - want.astype(np.float64))
        assert np.all(err <= bound), f"max err {err.max()} at {np.unravel_index(np.argmax(err - bound), err.shape)}"


# Frames of 2 to 63 elements go through LDS in tiles of 256 / D groups of lanes: the widest and the
# narrowest of them, blocks of a tile's length and one slot more, many blocks per tile, planes of
# fewer than 16 slots, enough tiles for the longer lanes and too few for them.
@pytest.mark.parametrize("dtype,op", [("f32", "mean"), ("i32", "sum"), ("u8", "mean"), ("f16", "sum")])
@pytest.mark.parametrize("B,T,D", [(2, 4224, 2), (700, 4225, 2), (3, 1153, 2), (40, 132, 63), (600, 133, 63), (300, 36, 57),
                                   (5000, 37, 37), (900, 700, 7), (1, 2, 5), (1, 15, 3), (1, 17, 3), (4000, 19, 33),
                                   # rows of 16 bytes per lane whose last vector lies over its neighbour, in rows
                                   # of a few lanes, of a wave, and of several
                                   (3000, 140, 17), (800, 300, 65), (60, 300, 271), (30, 70, 1025), (20, 40, 2061)])
def test_reduce_staged_edges(B, T, D, dtype, op):
    test_reduce_follows_the_flags(B, T, D, dtype, op)


# A sequence over many chunks is put together from its pieces eight at a time behind the second: every number of
# pieces around those borders (chunks of 64 slots), the last chunk of a tensor among them, with shorter
# sequences in between; sums of whole numbers, so that every order and grouping must give the same bits.
@pytest.mark.parametrize("dtype", ["i32", "f32"])
@pytest.mark.parametrize("T", [64, 65, 128, 129, 192, 640, 641, 704, 1152, 1153, 1217, 4696])
def test_reduce_stitches_any_number_of_pieces(T, dtype):
    bl = binding()
    rng = np.random.default_rng(T)
    for L, D in [([T], 347), ([T, 1, T - 1, T // 2, T - T // 2, T], 64), ([T, T], 1)]:
        L = np.array(L, dtype=np.int32)
        so = workloads.src_offsets(L)
        src = rng.integers(-1000, 1000, size=(int(so[-1]), D)).astype(NP_OF[dtype])
        pl = oracle.plan(L, T, np.arange(len(L), dtype=np.int32))
        packed, seq_id, frame_idx, reset, valid = oracle.pack(src, so, L, pl, D * 4)
        print(f"stitch T={T} D={D} {dtype} n={len(L)}", flush=True)
        out = bl.bload_segment_reduce(to_dev(packed), to_dev(seq_id), to_dev(reset), to_dev(valid),
                                      pl.num_blocks, T, D, dtype, "sum", len(L)).cpu().numpy()
        want = np.add.reduceat(src.astype(np.int64), so[:-1], axis=0)
        assert np.array_equal(out.astype(np.int64), want)


# Frames that are no whole 16-byte vectors choose their lane width by bytes, idle lanes and slots per row of the
# result: each width on both sides of each line (rows of 16 lanes and of 17, a frame a vector over one and two
# waves, a third of the lanes idle and less, short and long pieces), with room asked for by the query.
@pytest.mark.parametrize("dtype,op", [("f32", "mean"), ("i32", "sum"), ("u8", "mean"), ("f16", "sum")])
@pytest.mark.parametrize("B,T,frame_bytes,n_rows", [(2100, 64, 252, 0), (2100, 64, 260, 0), (600, 130, 1028, 0),
                                                    (600, 130, 1364, 0), (600, 130, 1364, 10000), (600, 130, 1372, 0),
                                                    (500, 520, 66, 0), (500, 520, 66, 2), (300, 700, 126, 1)])
def test_reduce_lane_widths(B, T, frame_bytes, n_rows, dtype, op):
    """n_rows: more rows than segments, or so few that the pieces are taken for long ones."""
    bl = binding()
    D = frame_bytes // bl.ELEM_BYTES[dtype] + (1 if dtype == "u8" else 0)
    rng = np.random.default_rng(B + T + D)
    valid, reset, seq_id, n_seg = random_flags(rng, B, T, 0.97, 0.02 if n_rows not in (1, 2) else 0.0)
    src = draw_source(rng, B * T, D, dtype)
    want, _ = oracle.segment_reduce_packed(src.reshape(B, T, D), seq_id, reset, valid, D, dtype, op, n_seg)
    n = n_rows or n_seg
    print(f"widths B={B} T={T} D={D} {dtype} {op} rows {n} of {n_seg}", flush=True)
    got = bl.bload_segment_reduce(to_dev(src), to_dev(seq_id), to_dev(reset), to_dev(valid), B, T, D, dtype, op, n).cpu().numpy()
    m = min(n, n_seg)
    if dtype == "i32":
        assert np.array_equal(got[:m], want[:m])
        return
    absval = np.abs(src.astype(np.float64)).astype(np.float32).reshape(B, T, D)
    scale, _ = oracle.segment_reduce_packed(absval, seq_id, reset, valid, D, "f32", op, n_seg)
    bound = REL_TOL * np.maximum(np.abs(want.astype(np.float64)), scale.astype(np.float64)) + 1e-30
    assert np.all(np.abs(got[:m].astype(np.float64) - want[:m].astype(np.float64)) <= bound[:m])
    assert not got[m:].any()


# A 1 in front of frames of 2^-24, half a unit in its last place: added one by one to a float32 sum that holds the 1
# they all vanish, a unit of roundoff each.  Trees of eight lose at most three units, their sum in more than 32
# bits none and the result one, wherever in a lane the sequence lies.  (Blocks shorter than a tile: no
# partial sums.  Enough tiles for lanes of 17 slots, and few enough for 9.)
@pytest.mark.parametrize("n,T,D", [(30000, 33, 7), (2000, 33, 7), (16000, 60, 32), (900, 60, 32), (12000, 40, 3), (9000, 60, 47)])
def test_reduce_staged_lanes_lose_no_more_than_a_tree_of_eight(n, T, D):
    bl = binding()
    rng = np.random.default_rng(n + D)
    L = rng.integers(1, T, size=n, endpoint=True).astype(np.int32)
    so = workloads.src_offsets(L)
    src = np.full((int(so[-1]), D), 2.0 ** -24, np.float32)
    src[so[:-1]] = 1.0
    pl = oracle.plan(L, T, oracle.order(n, 1))
    packed, seq_id, _, reset, valid = oracle.pack(src, so, L, pl, D * 4)
    got = bl.bload_segment_reduce(to_dev(packed), to_dev(seq_id), to_dev(reset), to_dev(valid), pl.num_blocks, T, D,
                                  "f32", "sum", n).cpu().numpy().astype(np.float64)
    want = 1.0 + (L - 1)[:, None] * 2.0 ** -24
    lost = np.abs(got - want) / (U * want)
    print(f"n={n} T={T} D={D}: {lost.max():.1f} units of roundoff", flush=True)
    assert lost.max() <= 4


# Less room than the query answers, down to none where the leanest cut leaves no partial sums: blocks under 4096
# slots of frames under 64 elements (one workgroup goes through a block's tiles), longer blocks in chunks of
# 12288 slots, and wide frames that are no whole vectors in lanes of one element.  One byte less than the
# leanest cut needs is refused.
@pytest.mark.parametrize("dtype,op", [("f32", "mean"), ("i32", "sum"), ("u8", "mean"), ("f16", "sum")])
@pytest.mark.parametrize("B,T,D,chunks", [(67, 777, 37, 1), (68, 777, 37, 1), (5, 4095, 2, 1), (40, 133, 63, 1), (3, 2000, 9, 1),
                                          (2, 12288, 3, 1), (3, 12289, 5, 2), (300, 700, 65, 7), (90, 700, 201, 10)])
def test_reduce_with_less_workspace_than_asked_for(B, T, D, chunks, dtype, op):
    bl = binding()
    asked = bl.bload_segment_reduce_workspace_bytes(B, T, D, dtype)
    part = 8 if dtype == "i32" or (D < 64 and dtype in ("f16", "f32")) else 4
    n = B * chunks
    room = 0 if chunks == 1 else n * 16 + 2 * (-(-n * D * part // 16) * 16)
    assert room <= asked
    rng = np.random.default_rng(B + T + D)
    for p_valid, p_reset in [(1.0, 0.0), (0.97, 0.01)]:
        valid, reset, seq_id, n_seg = random_flags(rng, B, T, p_valid, p_reset)
        src = draw_source(rng, B * T, D, dtype)
        want, _ = oracle.segment_reduce_packed(src.reshape(B, T, D), seq_id, reset, valid, D, dtype, op, n_seg)
        absval = np.abs(src.astype(np.float64)).astype(np.float32).reshape(B, T, D)
        scale, _ = oracle.segment_reduce_packed(absval, seq_id, reset, valid, D, "f32", op, n_seg)
        x, ids, r, v = to_dev(src), to_dev(seq_id), to_dev(reset), to_dev(valid)
        print(f"room {room} of {asked}: B={B} T={T} D={D} {dtype} {op} segments={n_seg}", flush=True)
        for take in (room, room - 1):
            out = torch.zeros((n_seg, D), dtype=torch.int64 if dtype == "i32" else torch.float32, device="cuda")
            ws = torch.empty(max(room, 16), dtype=torch.uint8, device="cuda")
            st = bl._lib.bload_segment_reduce(x.data_ptr(), ids.data_ptr(), r.data_ptr(), v.data_ptr(), B, T, D,
                                              bl.DTYPES[dtype], bl.OPS[op], n_seg, out.data_ptr(),
                                              ws.data_ptr() if take > 0 else None, max(take, 0),
                                              torch.cuda.current_stream().cuda_stream)
            if take < room and room > 0:
                assert st == bl.EWORKSPACE
                continue
            assert st == bl.OK
            got = out.cpu().numpy()
            if dtype == "i32":
                assert np.array_equal(got, want)
            else:
                bound = REL_TOL * np.maximum(np.abs(want.astype(np.float64)), scale.astype(np.float64)) + 1e-30
                assert np.all(np.abs(got.astype(np.float64) - want.astype(np.float64)) <= bound)


# Staged blocks in two or three tiles that one workgroup takes one after another: segments that cross the borders,
# end at them and begin behind them, the carried sequence's id and count, in pieces long enough for that cut.
@pytest.mark.parametrize("dtype,op", [("f32", "mean"), ("i32", "sum"), ("u8", "mean"), ("f16", "sum")])
@pytest.mark.parametrize("B,T,D", [(9, 2177, 2), (30, 4352, 2), (20, 1446, 3), (11, 1734, 5), (700, 3300, 4), (650, 2312, 4)])
def test_reduce_runs_of_tiles(B, T, D, dtype, op):
    bl = binding()
    rng = np.random.default_rng(B + T + D)
    tile = 256 // D * 17
    valid, reset = np.ones((B, T), np.uint8), np.zeros((B, T), np.uint8)
    for b in range(B):
        for t in rng.choice([tile - 1, tile, tile + 1, 2 * tile - 1, 2 * tile, 2 * tile + 1, 1, T - 1, T // 2], size=rng.integers(0, 4)):
            if t < T:
                reset[b, t] = 1
        if b % 4 == 3:
            valid[b, min(T - 1, int(rng.choice([tile - 1, tile, tile + 1]))):][:int(rng.integers(1, 9))] = 0
    reset &= valid
    prev = np.concatenate([np.zeros((B, 1), np.uint8), valid[:, :-1]], axis=1)
    starts = (valid == 1) & ((reset == 1) | (prev == 0))
    seq_id = np.where(valid == 1, np.cumsum(starts.reshape(-1)).reshape(B, T) - 1, -1).astype(np.int32)
    n_seg = int(starts.sum())
    src = draw_source(rng, B * T, D, dtype)
    want, counted = oracle.segment_reduce_packed(src.reshape(B, T, D), seq_id, reset, valid, D, dtype, op, n_seg)
    assert counted == n_seg
    got = bl.bload_segment_reduce(to_dev(src), to_dev(seq_id), to_dev(reset), to_dev(valid), B, T, D, dtype, op, n_seg).cpu().numpy()
    if dtype == "i32":
        assert np.array_equal(got, want)
        return
    absval = np.abs(src.astype(np.float64)).astype(np.float32).reshape(B, T, D)
    scale, _ = oracle.segment_reduce_packed(absval, seq_id, reset, valid, D, "f32", op, n_seg)
    bound = REL_TOL * np.maximum(np.abs(want.astype(np.float64)), scale.astype(np.float64)) + 1e-30
    assert np.all(np.abs(got.astype(np.float64) - want.astype(np.float64)) <= bound)


# Rows of one wave and many short sequences: two waves share a chunk (64 slots; 67 and 66; 131 of 180 blocks of 3000; 65 and a
# last one of 3), part where a segment begins or ends next to its middle, and leave one whole that ends within 32 slots behind
# it.  Segments that begin and end at the chunks' borders and middles, as far behind the borders as they are followed, beside
# all of these and some slots off, some over several chunks, some from a middle to a border, padding there as well.
@pytest.mark.parametrize("B,T,dtype,op", [(12, 640, "f32", "mean"), (12, 640, "i32", "sum"), (12, 640, "u8", "mean"),
                                          (12, 640, "f16", "sum"), (7, 133, "f16", "mean"), (1, 128, "f16", "mean"),
                                          (180, 3000, "f16", "mean"), (3, 4033, "f32", "mean")])
def test_reduce_short_pieces_over_chunk_borders(B, T, dtype, op):
    bl = binding()
    rng = np.random.default_rng(B + T)
    D = 1024 // bl.ELEM_BYTES[dtype]
    chunk = -(-T // min(T // 64, -(-1024 * 4 // B)))
    chunks = B * -(-T // chunk)
    # (the query tells how many chunks there are)
    assert bl.bload_segment_reduce_workspace_bytes(B, T, D, dtype) == chunks * (16 + 2 * D * (8 if dtype == "i32" else 4))
    at = [t0 + m + k for t0 in range(0, T, chunk) for m in (0, (min(chunk, T - t0) + 1) // 2, 32)
          for k in (-9, -1, 0, 1, 5)]
    at = np.array([t for t in at if 0 < t < T])
    valid, reset = np.ones((B, T), np.uint8), np.zeros((B, T), np.uint8)
    for b in range(B):
        reset[b, rng.choice(at, size=int(rng.integers(0, len(at) // 2 + 1)), replace=False)] = 1
        if b % 3 == 2:
            for t in rng.choice(at, size=3):
                valid[b, t:t + int(rng.integers(1, 40))] = 0
    reset &= valid
    prev = np.concatenate([np.zeros((B, 1), np.uint8), valid[:, :-1]], axis=1)
    starts = (valid == 1) & ((reset == 1) | (prev == 0))
    seq_id = np.where(valid == 1, np.cumsum(starts.reshape(-1)).reshape(B, T) - 1, -1).astype(np.int32)
    n_seg = int(starts.sum())
    n = max(n_seg, B * T // 30)                             # rows enough to tell of short pieces
    src = draw_source(rng, B * T, D, dtype)
    want, _ = oracle.segment_reduce_packed(src.reshape(B, T, D), seq_id, reset, valid, D, dtype, op, n_seg)
    print(f"chunk borders B={B} T={T} {dtype} chunk {chunk} segments {n_seg}", flush=True)
    got = bl.bload_segment_reduce(to_dev(src), to_dev(seq_id), to_dev(reset), to_dev(valid), B, T, D, dtype, op, n).cpu().numpy()
    assert not got[n_seg:].any()
    if dtype == "i32":
        assert np.array_equal(got[:n_seg], want)
        return
    absval = np.abs(src.astype(np.float32)).reshape(B, T, D)
    scale, _ = oracle.segment_reduce_packed(absval, seq_id, reset, valid, D, "f32", op, n_seg)
    bound = REL_TOL * np.maximum(np.abs(want.astype(np.float64)), scale.astype(np.float64)) + 1e-30
    assert np.all(np.abs(got[:n_seg].astype(np.float64) - want.astype(np.float64)) <= bound)


# Frames whose whole multiples are at most 64 vectors, in long pieces: a wave takes a piece's bytes as one stream.  In every
# type several blocks to a workgroup (chunks < B), whole blocks and blocks cut into a few and into many shares (chunks >
# B), segments that begin and end around the quarters that the waves take, padding there as well, pieces of fewer frames
# than a step and of whole steps, several lanes to a feature and several features to a lane (from 33 on), the tensor's last
# bytes (also no whole vector), tensors beyond the memory-side cache.  The lanes' trees of four lose 2 units of roundoff of sum |x|,
# the result's rounding one, as does the oracle's.
@pytest.mark.parametrize("dtype,B,T,D,chunks", [
    ("u8", 2300, 400, 44, 1150), ("u8", 2300, 400, 128, 1150), ("f16", 3000, 600, 37, 1500), ("f16", 2300, 400, 62, 1150),
    ("f16", 2301, 401, 30, 1151), ("f32", 2100, 600, 11, 1050), ("i32", 2100, 600, 11, 1050),
    ("u8", 1100, 300, 48, 1100), ("u8", 1301, 777, 63, 1301), ("f16", 1100, 300, 24, 1100), ("f16", 1025, 777, 32, 1025),
    ("f32", 1100, 300, 12, 1100), ("f32", 1030, 160, 32, 1030), ("f32", 1400, 600, 64, 1400), ("i32", 1100, 300, 12, 1100),
    ("i32", 1400, 600, 64, 1400),
    ("u8", 160, 8001, 47, 1120), ("u8", 300, 7000, 8, 900), ("f16", 160, 8001, 22, 1120), ("f16", 300, 7000, 4, 900),
    ("f32", 160, 8001, 11, 1120), ("f32", 300, 7000, 2, 900), ("i32", 160, 8001, 11, 1120), ("i32", 300, 7000, 2, 900),
    ("u8", 3, 60000, 76, 834), ("f16", 15, 60000, 38, 1035), ("f32", 15, 60000, 19, 1035), ("i32", 15, 60000, 19, 1035),
    ("u8", 5500, 600, 86, 2750), ("f16", 5500, 600, 43, 2750), ("i32", 5500, 600, 23, 2750)])
def test_reduce_flat_streams(dtype, B, T, D, chunks):
    bl = binding()
    op = {"f32": "mean", "i32": "sum", "u8": "mean", "f16": "sum"}[dtype]
    rng = np.random.default_rng(B + T + D)
    valid, reset = np.ones((B, T), np.uint8), np.zeros((B, T), np.uint8)
    tile = T * -(-B // chunks) if chunks <= B else -(-T // (chunks // B))         # a workgroup's slots
    at = np.unique([(t0 + tile * w // 4 + k) % T for t0 in range(0, max(tile, T), tile) for w in range(5) for k in (-17, -1, 0, 1, 2, 16)])
    for b in range(B):
        if b % 3:
            reset[b, rng.choice(at, size=int(rng.integers(0, 4)))] = 1
        if b % 5 == 1:
            valid[b, int(rng.choice(at)):][:int(rng.integers(1, 12))] = 0
    reset &= valid
    prev = np.concatenate([np.zeros((B, 1), np.uint8), valid[:, :-1]], axis=1)
    starts = (valid == 1) & ((reset == 1) | (prev == 0))
    seq_id = np.where(valid == 1, np.cumsum(starts.reshape(-1)).reshape(B, T) - 1, -1).astype(np.int32)
    n_seg = int(starts.sum())
    src = draw_source(rng, B * T, D, dtype)
    want, _ = oracle.segment_reduce_packed(src.reshape(B, T, D), seq_id, reset, valid, D, dtype, op, n_seg)
    absval = np.abs(src.astype(np.float32)).reshape(B, T, D)
    scale, _ = oracle.segment_reduce_packed(absval, seq_id, reset, valid, D, "f32", op, n_seg)

    print(f"flat B={B} T={T} D={D} {dtype} segments {n_seg}", flush=True)
    assert bl.bload_segment_reduce_layout(B, T, D, dtype, n_seg) == ("flat", chunks)
    got = bl.bload_segment_reduce(to_dev(src), to_dev(seq_id), to_dev(reset), to_dev(valid), B, T, D, dtype, op, n_seg).cpu().numpy()
    if dtype == "i32":
        assert np.array_equal(got, want)
        return
    bound = 2.01 * U * scale.astype(np.float64) + 2 * U * np.abs(want.astype(np.float64))
    err = np.abs(got.astype(np.float64) - want.astype(np.float64))
    assert np.all(err <= bound), f"{np.max(err / (U * scale))} units"
