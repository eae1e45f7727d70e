"""bload_plan on the GPU against the oracle: bit-exact order, blocks, offsets."""
import numpy as np
import pytest
import torch

import oracle
from paper_2310_10879_amd import workloads
from gpu_util import assert_plan_equal, binding, gpu_plan, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["uniform", "short", "long", "mixed"])
@pytest.mark.parametrize("n,T", [(1, 1), (1, 9), (2, 2), (3, 5), (64, 32), (255, 7), (257, 600),
                                 (1000, 600), (2047, 33), (2048, 1), (2049, 4096), (5000, 3),
                                 (70001, 100),
                                 # around the tiles of the scans (2048), and up to and beyond the workgroup of 16 waves (12288)
                                 (4096, 17), (4097, 900), (8191, 2), (8192, 50), (8193, 7),
                                 (16384, 64), (16385, 300), (24577, 5)])
def test_plan_matches_oracle(kind, n, T):
    rng = np.random.default_rng(n * 7 + T)
    L = workloads.random_lengths(rng, n, T, kind)
    for seed in workloads.SHUFFLE_SEEDS:
        print(f"plan n={n} T={T} kind={kind} seed={seed}", flush=True)
        ref = oracle.plan(L, T, oracle.order(n, seed))
        assert_plan_equal(gpu_plan(L, T, seed), ref, n)


@pytest.mark.parametrize("case", range(16))
def test_plan_random_sizes_of_several_jump_tiles(case):
    # tiles of 2048 and 4096 positions, up to 79 of them, with groups from 40 on: every tile finds where the orbit of
    # position 0 enters it
    rng = np.random.default_rng(9000 + case)
    n = int(rng.integers(8193, 300000))
    T = int(rng.choice([1, 3, 64, 600, 4096, 100000]))
    kind = str(rng.choice(["uniform", "short", "long", "mixed"]))
    L = workloads.random_lengths(rng, n, T, kind)
    seed = int(rng.integers(0, 2 ** 63))
    print(f"plan n={n} T={T} kind={kind} seed={seed}", flush=True)
    assert_plan_equal(gpu_plan(L, T, seed), oracle.plan(L, T, oracle.order(n, seed)), n)


# From 40 jump tiles on a tile reaches its entry over the exits of groups of tiles (here 8 of 4096 positions, beyond 2^20
# of 8192): a last group of one position, blocks that pass over whole tiles and
# whole groups, blocks of one sequence, and both sides of 2^20, where the order kernel changes.
@pytest.mark.parametrize("n,T,kind", [(39 * 8192, 64, "mixed"), (39 * 8192 + 1, 64, "mixed"), (40 * 8192 + 1, 600, "short"),
                                      (48 * 8192 + 1, 20000, "short"), (600000, 200000, "short"), (600000, 70000, "short"),
                                      (400000, 1, "uniform"), (400001, 3, "long"), (1 << 20, 300, "uniform"),
                                      ((1 << 20) + 1, 300, "short"), (3000000, 4096, "mixed")])
def test_plan_entries_over_groups_of_tiles(n, T, kind):
    rng = np.random.default_rng(n + T)
    L = workloads.random_lengths(rng, n, T, kind)
    print(f"plan n={n} T={T} kind={kind}", flush=True)
    assert_plan_equal(gpu_plan(L, T, 5), oracle.plan(L, T, oracle.order(n, 5)), n)


def test_plan_refuses_bad_lengths_of_many_tiles():
    bl = binding()
    rng = np.random.default_rng(3)
    for bad in (0, -5, 301, 2 ** 31 - 1, -2 ** 31):
        L = workloads.random_lengths(rng, 400000, 300, "uniform")
        L[rng.integers(0, L.size, size=500)] = bad
        with pytest.raises(bl.BloadError) as e:
            gpu_plan(L, 300, 1)
        assert e.value.status == bl.ELENGTH


@pytest.mark.parametrize("wid", [1, 2, 3, 4, 5])
def test_plan_workloads_full_size(wid):
    w = workloads.WORKLOADS[wid]
    L = workloads.lengths(wid)
    for seed in workloads.SHUFFLE_SEEDS:
        print(f"plan workload {wid} seed={seed}", flush=True)
        ref = oracle.plan(L, w.t_blk, oracle.order(w.n_seq, seed))
        assert_plan_equal(gpu_plan(L, w.t_blk, seed), ref, w.n_seq)


@pytest.mark.parametrize("n", [4100, 8192, 20000])        # one workgroup of 16 waves, ten jump tiles
def test_plan_closed_forms(n):
    # every position a block head; one block head in 12; every position; every second one
    T = 12
    for L in (np.full(n, T), np.ones(n), np.full(n, T // 2 + 1), np.full(n, T // 2)):
        L = L.astype(np.int32)
        ref = oracle.plan(L, T, oracle.order(n, 5))
        assert_plan_equal(gpu_plan(L, T, 5), ref, n)


def test_plan_empty_and_errors():
    bl = binding()
    pl = gpu_plan(np.zeros(0, np.int32), 8, 0)
    assert pl.num_blocks == 0 and pl.total_frames == 0
    for bad in ([3, 0, 2], [3, 9, 2], [-1, 1, 1]):
        with pytest.raises(bl.BloadError) as e:
            gpu_plan(np.array(bad, dtype=np.int32), 8, 0)
        assert e.value.status == bl.ELENGTH
    with pytest.raises(bl.BloadError) as e:
        gpu_plan(np.array([1, 2], dtype=np.int32), 0, 0)
    assert e.value.status == bl.EINVAL
    # workspace too small
    L = to_dev(np.array([1, 2, 3], dtype=np.int32))
    with pytest.raises(bl.BloadError) as e:
        bl.bload_plan(L, 8, 0, workspace=torch.empty(16, dtype=torch.uint8, device=L.device))
    assert e.value.status == bl.EWORKSPACE
    # the library still works after the refused calls
    ref = oracle.plan(np.array([1, 2, 3], dtype=np.int32), 8, oracle.order(3, 0))
    assert_plan_equal(bl.bload_plan(L, 8, 0), ref, 3)


def test_plan_is_deterministic():
    L = workloads.lengths(3)
    a = gpu_plan(L, 3000, 11)
    b = gpu_plan(L, 3000, 11)
    assert torch.equal(a.order, b.order) and torch.equal(a.offset_of_seq, b.offset_of_seq)
    assert torch.equal(a.block_of_seq, b.block_of_seq)


# One workgroup of 16 waves, 1 to 13 positions per thread: both ends of each, both ends of its range, a last wave
# with one position, blocks of one sequence, of two, of nearly all, of all, and over several waves; and where prefix
# sums just fit 32 bits and just do not, which the other kernels then take.
@pytest.mark.parametrize("n", [256, 257, 1023, 1024, 1025, 2048, 3072, 3073, 5120, 5121, 7169, 9216, 9217, 11265, 12288, 12289])
def test_plan_one_workgroup_of_sixteen_waves(n):
    rng = np.random.default_rng(n)
    cases = [(np.ones(n), 1), (np.ones(n), 2), (np.full(n, 5), 14), (np.ones(n), n), (np.ones(n), n - 1), (np.ones(n), 700),
             (rng.integers(1, 4, size=n), 3000), (rng.integers(1, 3001, size=n), 3000),
             (np.clip(8 * (1 + rng.pareto(1.5, size=n)), 1, 3000), 3000), (np.where(rng.random(n) < 0.01, 900, 1), 900)]
    last = (2 ** 31 - 1) // (n + 1)
    cases += [(rng.integers(max(1, last // 3), last, size=n, endpoint=True), last), (np.full(n, last + 1), last + 1)]
    for k, (L, T) in enumerate(cases):
        L = np.asarray(L).astype(np.int32)
        print(f"plan n={n} T={T} case {k}", flush=True)
        assert_plan_equal(gpu_plan(L, T, 5 + k), oracle.plan(L, T, oracle.order(n, 5 + k)), n)
    bl = binding()
    for bad in (0, 301, -2 ** 31):
        L = rng.integers(1, 301, size=n).astype(np.int32)
        L[n // 2] = bad
        with pytest.raises(bl.BloadError) as e:
            gpu_plan(L, 300, 1)
        assert e.value.status == bl.ELENGTH


# A position to a lane: one wave (up to 64), up to 16 waves of one chunk of 64 positions (1024) or two (2048): both ends of each
# and of the permutation's domains, chunks of one position, blocks of one sequence, over a chunk's end and over all of them,
# and sums that leave 32 bits.
@pytest.mark.parametrize("n", [1, 2, 4, 5, 16, 17, 63, 64, 65, 127, 128, 129, 192, 255, 1023, 1024, 1025, 1088, 2047, 2048, 2049])
def test_plan_a_position_to_a_lane(n):
    rng = np.random.default_rng(100 + n)
    big = 2 ** 31 - 1
    cases = [(np.ones(n), 1), (np.ones(n), 3), (np.ones(n), 63), (np.ones(n), 64), (np.ones(n), 65), (np.ones(n), n),
             (np.full(n, 4), 7), (rng.integers(1, 33, size=n), 32), (rng.integers(1, 4, size=n), 300),
             (np.where(rng.random(n) < 0.03, 500, 1), 500), (np.full(n, big), big), (rng.integers(big // 9, big, size=n), big)]
    for k, (L, T) in enumerate(cases):
        L = np.asarray(L).astype(np.int32)
        print(f"plan n={n} T={T} case {k}", flush=True)
        assert_plan_equal(gpu_plan(L, T, 7 * n + k), oracle.plan(L, T, oracle.order(n, 7 * n + k)), n)
    bl = binding()
    for bad in (0, 301, -2 ** 31, big):
        L = np.full(n, 300, dtype=np.int32)
        L[rng.integers(0, n, size=1 + n // 3)] = bad
        with pytest.raises(bl.BloadError) as e:
            gpu_plan(L, 300, 1)
        assert e.value.status == bl.ELENGTH


# Jump tiles of 2048, 4096 and 8192 positions (up to 160000 sequences, 2^20, beyond): one position in the last tile, in the
# last group of 16 or 8 of them, both sides of the line from which on groups are used; the sequences fetch what
# they get from 2^19 on (unless the order's domain is much larger); blocks that pass over tiles and groups.
@pytest.mark.parametrize("n", [12289, 7 * 2048, 7 * 2048 + 1, 39 * 2048, 40 * 2048 - 1, 40 * 2048 + 1, 48 * 2048 + 1, 160000, 160001,
                               48 * 4096 + 1, (1 << 19) - 1, 1 << 19, 600001, (1 << 20) - 1, (1 << 20) + 1, 1200000])
@pytest.mark.parametrize("T,kind", [(1, "uniform"), (40, "short"), (3000, "uniform"), (4096, "heavy"), (100000, "short"), (300, "two")])
def test_plan_sizes_of_jump_tiles(n, T, kind):
    rng = np.random.default_rng(n + T)
    if kind == "heavy":
        L = np.clip(rng.zipf(1.2, size=n), 1, T).astype(np.int32)
    elif kind == "two":
        L = np.full(n, T // 2, dtype=np.int32)
    else:
        L = workloads.random_lengths(rng, n, T, kind)
    print(f"plan n={n} T={T} kind={kind}", flush=True)
    assert_plan_equal(gpu_plan(L, T, 7), oracle.plan(L, T, oracle.order(n, 7)), n)


# Sums that leave 32 bits keep up to 8192 sequences off the workgroup of 16 waves: they are one jump tile, entered at position 0;
# from 8193 on several.  Blocks of one sequence, of some, of nearly all and of all of them.
@pytest.mark.parametrize("n", [2049, 4097, 8191, 8192, 8193])
@pytest.mark.parametrize("T,lo,hi", [(1 << 24, 1, 1 << 24), (1 << 24, (1 << 23) + 1, 1 << 24), (1 << 24, 1, 1 << 14), (1 << 20, 100, 160),
                                     (2000000000, 1, 2000000000), (2000000000, 1, 3)])
def test_plan_one_jump_tile(n, T, lo, hi):
    rng = np.random.default_rng(n + hi)
    L = rng.integers(lo, hi, size=n, endpoint=True).astype(np.int32)
    print(f"plan n={n} T={T} lengths {lo} to {hi}", flush=True)
    assert_plan_equal(gpu_plan(L, T, 3), oracle.plan(L, T, oracle.order(n, 3)), n)


# Beyond 1024 jump tiles (of 8192) one thread finds where every tile is entered: both sides of that line, blocks of a few
# sequences, of one, and such that pass over whole tiles.
@pytest.mark.parametrize("n", [1024 * 8192, 1024 * 8192 + 1, 1027 * 8192 + 5000])
@pytest.mark.parametrize("T,kind", [(4096, "mixed"), (1, "uniform"), (100000, "short")])
def test_plan_entries_found_by_one_thread(n, T, kind):
    rng = np.random.default_rng(n + T)
    L = workloads.random_lengths(rng, n, T, kind)
    print(f"plan n={n} T={T} kind={kind}", flush=True)
    assert_plan_equal(gpu_plan(L, T, 9), oracle.plan(L, T, oracle.order(n, 9)), n)


# next[] is searched for in a window of 1024 positions (of t_blk, in shorter blocks) held in LDS, from blocks of 16 slots on, unless
# the first position's block passes over it: blocks of as many sequences as the window, one fewer and one more, of a few, of
# several windows; and blocks that differ so much that some positions of a workgroup find theirs in it and some behind it.
@pytest.mark.parametrize("n", [12289, 20000])
@pytest.mark.parametrize("T", [1, 2, 15, 16, 17, 1022, 1023, 1024, 1025, 1279, 1280, 1281, 5000])
def test_plan_window_of_next(n, T):
    rng = np.random.default_rng(n + T)
    rare = np.where(rng.random(n) < 0.002, T, 1)
    for k, L in enumerate((np.ones(n), np.minimum(rng.integers(1, 3, size=n), T), rare)):
        L = L.astype(np.int32)
        print(f"plan n={n} T={T} case {k}", flush=True)
        assert_plan_equal(gpu_plan(L, T, 5), oracle.plan(L, T, oracle.order(n, 5)), n)
