"""The row kernels' plan on the CPU: the library's own arithmetic (csrc/gt_plan.hpp,
compiled by tests/plan_probe.cpp) over random graphs' degree classes."""
import ctypes
import functools
import hashlib
import os
import shutil
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2605_31500_amd", "csrc")
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")

pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not installed")


class Tuning(ctypes.Structure):
    _fields_ = [(f, ctypes.c_int32) for f in ("light_max_deg", "heavy_min_deg", "chunk_edges", "grid_blocks",
                                              "dense_tiles", "bf16_weights")]


class RowCut(ctypes.Structure):
    _fields_ = [("N", ctypes.c_int64), ("E", ctypes.c_uint32), ("light_max", ctypes.c_int32),
                ("min_class", ctypes.c_int32), ("split_min", ctypes.c_uint32), ("chunk", ctypes.c_uint32),
                ("nq_floor", ctypes.c_uint32), ("nq_max", ctypes.c_uint32), ("group_len", ctypes.c_uint32),
                ("cap_slots", ctypes.c_uint32)]


class RowRule(ctypes.Structure):
    _fields_ = [("light_max", ctypes.c_int32), ("split_min", ctypes.c_uint32), ("chunk", ctypes.c_uint32),
                ("nq_floor", ctypes.c_uint32), ("nq_max", ctypes.c_uint32), ("group_len", ctypes.c_uint32),
                ("max_slots", ctypes.c_int64), ("likely_slots", ctypes.c_int64), ("forced", ctypes.c_bool)]


class SlotPlan(ctypes.Structure):
    _fields_ = [("cap", ctypes.c_uint32), ("slices", ctypes.c_int)]


class AttnShape(ctypes.Structure):
    _fields_ = [("N", ctypes.c_int64), ("E", ctypes.c_int64), ("H", ctypes.c_int32), ("D", ctypes.c_int32),
                ("elt_bytes", ctypes.c_int32), ("slice_heads", ctypes.c_int32), ("groups", ctypes.c_int32),
                ("gat", ctypes.c_bool), ("sorted", ctypes.c_bool)]


class AttnPlan(ctypes.Structure):
    _fields_ = [("need", ctypes.c_size_t), ("rule", RowRule), ("slots", SlotPlan), ("tiles", ctypes.c_bool),
                ("sorted", ctypes.c_bool), ("tile_min", ctypes.c_int), ("tile_max", ctypes.c_int32)] + [
                    (f, ctypes.c_size_t) for f in ("o_light", "o_deg", "o_win", "o_long", "o_ml", "o_acc", "bytes")]


@functools.lru_cache(maxsize=None)
def probe():
    srcs = [os.path.join(ROOT, "tests", "plan_probe.cpp"), os.path.join(CSRC, "gt_plan.hpp"),
            os.path.join(ROOT, "include", "gt_attn.h")]
    h = hashlib.sha256(b"".join(open(s, "rb").read() for s in srcs)).hexdigest()[:12]
    out = os.path.join(ROOT, "_build", "plan_probe-%s.so" % h)
    if not os.path.exists(out):
        os.makedirs(os.path.dirname(out), exist_ok=True)
        tmp = out + ".tmp%d" % os.getpid()
        r = subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-fPIC", "-shared", "-fsanitize=undefined",
                            "-fno-sanitize-recover=all", "-static-libubsan", "-D__HIP_PLATFORM_AMD__", "-D__host__=",
                            "-D__device__=", "-isystem", os.path.join(ROCM, "include"), "-I",
                            os.path.join(ROOT, "include"), "-I", CSRC, srcs[0], "-o", tmp],
                           capture_output=True, text=True)
        assert r.returncode == 0, r.stderr[-3000:]
        os.replace(tmp, out)
    L = ctypes.CDLL(out)
    L.probe_batches.restype = ctypes.c_int64
    return L


# Row kernels: bytes gathered per entry, `piece_bytes` of the rule, lane groups per wavefront.
KERNELS = [(512, 600, 4), (512, 600, 2), (256, 400, 8), (128, 300, 16), (64, 300, 16), (256, 600, 4), (1024, 2000, 1)]


def batches(cut, rows, P):
    rows = np.ascontiguousarray(rows, dtype=np.uint32)
    nq, total = np.zeros(32, np.uint32), np.zeros(8, np.uint64)
    p = lambda a: a.ctypes.data_as(ctypes.c_void_p)
    asked = ctypes.c_uint64()
    bound = probe().probe_batches(ctypes.byref(cut), p(rows), ctypes.c_uint32(P), p(nq), p(total), ctypes.byref(asked))
    assert bound >= 0 and asked.value < 1 << 32
    return bound, nq, total


def rule(N, E, slices, gather, piece, P, tuning=None):
    cut, r = RowCut(), RowRule()
    probe().probe_rule(ctypes.c_int64(N), ctypes.c_int64(E), slices, gather, piece, P,
                       ctypes.byref(tuning) if tuning else None, ctypes.byref(cut), ctypes.byref(r))
    return cut, r


def random_rows(rng, cut):
    """Rows per class of a graph with the cut's N and E."""
    rows, left_e, left_n = np.zeros(32, np.int64), int(cut.E), int(cut.N)
    for c in rng.permutation(np.arange(cut.min_class, 31)):
        most = min(left_e >> int(c), left_n)
        n = int(most * rng.choice([0, 0, 1e-3, 0.1, 0.5, 1.0]) * rng.random())
        if c == cut.min_class:  # (its shortest rows are longer than light_max)
            n = min(n, left_e // (cut.light_max + 1))
        rows[c], left_e, left_n = n, left_e - (n << int(c)), left_n - n
    return rows


@pytest.mark.parametrize("gather,piece,P", KERNELS)
def test_no_wave_with_batches_ends_early(gather, piece, P):
    """A wave ends where its number reaches the bound that the partition counts: every
    batch has to lie below it, also where classes lose pieces for want of partial states
    and what is left of them takes whole wavefronts."""
    rng = np.random.default_rng(gather + P)
    shrunk_and_spread = 0
    for _ in range(3000):
        N = int(np.exp(rng.uniform(np.log(100), np.log(1 << 24))))
        E = min(int(N * np.exp(rng.uniform(0, np.log(500)))), (1 << 31) - 1)
        tuning = None
        if rng.random() < 0.3:
            tuning = Tuning(light_max_deg=int(rng.choice([0, 1, 8, 100])), chunk_edges=int(rng.choice([0, 64, 200, 5000])),
                            heavy_min_deg=int(rng.choice([0, 64, 1000])))
        cut, r = rule(N, E, int(rng.choice([1, 2, 8])), gather, piece, P, tuning)
        cut.cap_slots = int(min(r.max_slots, 2**31) * rng.choice([1.0, 1.0, 0.3, 0.05, 0.001, 0.0]))
        rows = random_rows(rng, cut)
        bound, nq, total = batches(cut, rows, P)
        assert int(total.max()) <= bound, (N, E, cut.cap_slots, list(rows))
        for c in np.flatnonzero(rows):
            full = 1 if (1 << int(c)) < cut.split_min else min(max((2 << int(c)) // cut.chunk, cut.nq_floor), cut.nq_max)
            shrunk_and_spread += nq[c] < full and (2 << int(c)) // int(nq[c]) > cut.group_len
    assert shrunk_and_spread > 100


def test_halved_classes_take_whole_wavefronts():
    """Backward of fp32 8x64 features: 6200 rows of 600 entries among 600 K, with room for half of their pieces."""
    cut, _ = rule(600_000, 6200 * 600 + 3 * 600_000, 8, 512, 600, 4)
    cut.split_min, cut.chunk, cut.nq_floor, cut.group_len, cut.cap_slots = 64, 128, 8, 128, 6200 * 4
    rows = np.zeros(32)
    rows[9] = 6200
    bound, nq, total = batches(cut, rows, 4)
    assert nq[9] == 4 and total.max() == 6200 * 4 // 8 and total.max() <= bound


@pytest.mark.parametrize("P", [1, 4, 16])
@pytest.mark.parametrize("heavy_min_deg", [0, 1, 64])
@pytest.mark.parametrize("light_max_deg", [1, 2, 40, 0])
def test_largest_graphs_count_in_32_bits(P, light_max_deg, heavy_min_deg):
    """2^31 - 1 entries in rows of one class, as many as there can be: the lane groups that the partition counts do not
    wrap, and no wave with batches ends early."""
    cut, r = rule((1 << 31) - 1, (1 << 31) - 1, 1, 1024 // P, 300, P,
                  Tuning(light_max_deg=light_max_deg, heavy_min_deg=heavy_min_deg))
    for cap in (r.max_slots, 1 << 20, 1 << 10, 0):
        cut.cap_slots = cap
        for c in range(cut.min_class, 31):
            rows = np.zeros(32)
            rows[c] = (cut.E >> c) if c > cut.min_class else cut.E // (cut.light_max + 1)
            bound, _, total = batches(cut, rows, P)
            assert int(total.max()) <= bound


# ------------------------------------------------------------------------- the forward's plan

SCRATCH = 256 << 20
SHAPES = [(eb, H, D) for eb in (2, 4) for H in (1, 2, 4, 8) for D in (32, 64, 128, 256)] + [(2, H, 512) for H in (1, 2, 4)]


def shape(N, E, eb, H, D, gat=False):
    """The call's slices and row kernel: the heads of 256 bytes, or one; four lane groups or more per wavefront
    (two for GATv2) take light rows in step order."""
    heads = max(1, min(H, 256 // (D * eb)))
    groups = 64 // (heads * D * eb // 16)
    return AttnShape(N, E, H, D, eb, heads, groups, gat, groups >= (2 if gat else 4))


def attn_plan(a, tuning=None, noalloc=False):
    p = AttnPlan()
    probe().probe_attn(ctypes.byref(a), ctypes.byref(tuning) if tuning else None, int(noalloc), ctypes.byref(p))
    return p


def cut_of(p):
    """What decides the bits of a call's results."""
    return [getattr(p.rule, f) for f, _ in RowRule._fields_] + [p.slots.cap, p.slots.slices, p.tiles]


def in_order(p, a):
    """The workspace's regions follow one another without overlap."""
    rows = 9 if p.sorted else 0
    size = {"o_light": 8 * a.N if rows else 0, "o_deg": a.N if rows else 0, "o_win": (a.N + 63) // 64 if p.tiles else 0,
            "o_ml": p.slots.cap * p.slots.slices * a.slice_heads * 8,
            "o_acc": p.slots.cap * p.slots.slices * a.slice_heads * a.D * 4}
    lo = max(p.rule.light_max + 1, 1).bit_length() - 1
    size["o_long"] = 16 * sum(min(a.E >> c, a.N) for c in range(lo, 31))
    spans = sorted((getattr(p, k), getattr(p, k) + v) for k, v in size.items() if v) + [(p.bytes, p.bytes)]
    return spans[0][0] >= 512 and all(x[1] <= y[0] for x, y in zip(spans, spans[1:]))


@pytest.mark.parametrize("gat", [False, True])
def test_plans_of_large_graphs_end_and_fit(gat):
    """Up to 2^31 - 1 nodes and entries: the plan is found (the light bound that fits is), its regions are apart, the
    allocation-free entry point's workspace lies within its array, and both entry points cut rows alike wherever
    the former takes the call."""
    rng = np.random.default_rng(11 + gat)
    bounded = 0
    for _ in range(20000):
        eb, H, D = SHAPES[rng.integers(len(SHAPES))]
        N = int(np.exp(rng.uniform(np.log(1 << (10 if rng.random() < 0.3 else 23)), np.log((1 << 31) - 1))))
        if rng.random() < 0.4:
            N = int(rng.integers(25_000_000, 34_000_000))  # around where the light rows' order fills the array
        E = int(min(N * np.exp(rng.uniform(np.log(0.01), np.log(200))), (1 << 31) - 1))
        t = None
        if rng.random() < 0.3:
            t = Tuning(light_max_deg=int(rng.choice([0, 1, 300, 2**31 - 2**16])), dense_tiles=int(rng.choice([0, 1, -1])),
                       heavy_min_deg=int(rng.choice([0, 1, 5000])), chunk_edges=int(rng.choice([0, 64, 10**6])))
        a = shape(N, E, eb, H, D, gat)
        p = attn_plan(a, t)
        assert in_order(p, a), (N, E, eb, H, D)
        assert p.rule.light_max >= 1 and (not p.tiles or p.tile_max <= min(64, p.rule.light_max))
        states = p.slots.cap * p.slots.slices
        if p.need <= SCRATCH and not gat:
            # room for the longest rows' states, within the array
            assert states >= min(p.rule.max_slots, (23 << 20) // (a.slice_heads * (4 * D + 8)))
            q = attn_plan(a, t, noalloc=True)
            assert q.bytes <= SCRATCH and in_order(q, a), (N, E, eb, H, D)
            assert cut_of(p) == cut_of(q), (N, E, eb, H, D)
            bounded += 1
        else:
            assert states >= min(p.rule.max_slots, (128 << 20) // (a.slice_heads * (4 * D + 8)) - H)
    assert gat or bounded > 2000


@pytest.mark.parametrize("eb,H,D,N,E", [(2, 1, 32, 31_000_000, 31_000_000), (4, 4, 32, 31_000_000, 200_000_000)])
def test_plans_around_thirty_million_nodes_end(eb, H, D, N, E):
    a = shape(N, E, eb, H, D)
    p, q = attn_plan(a), attn_plan(a, noalloc=True)
    assert p.need <= SCRATCH and q.bytes <= SCRATCH and cut_of(p) == cut_of(q)
    assert p.sorted and not q.sorted


def test_rows_are_cut_however_large_the_lists_and_statistics_are():
    """The states of a call with a workspace of its own do not depend on what else is in it: backward of 8 heads of 64
    fp32 features on 4 M nodes (268 MB of statistics), and a reduction over 40 M nodes."""
    for N, E, slices, gather, piece, P, slot, other in [
            (4_000_000, 96_000_000, 8, 512, 2048, 4, 512, 4_000_000 * (8 * 8 + 9) + 96_000_000 // 4),
            (40_000_000, 1_500_000_000, 2, 256, 3264, 4, 1024, 40_000_000 * 9 + 1_500_000_000)]:
        _, r = rule(N, E, slices, gather, piece, P)
        s = SlotPlan()
        probe().probe_slots(ctypes.byref(r), slices, ctypes.c_int64(slot), ctypes.c_int64(other), 0, ctypes.byref(s))
        assert s.cap * s.slices * slot >= min(r.max_slots * slot, 127 << 20)


def test_tile_rows_stay_short_where_the_light_bound_is_raised():
    """700 M entries: the class lists fit the array from a light bound of 129 on; the tile path's rows hold 64."""
    p = attn_plan(shape(8_000_000, 700_000_000, 2, 4, 32))
    assert p.need <= SCRATCH and p.tiles and p.rule.light_max > 64 and p.tile_max == 64


def test_allocation_free_limit():
    """What the entry point counts against its array, to the byte (from the layout that its limit was first stated
    for): two counter sets, the row lists, the chunks and their states, the window flags, each in whole 256 bytes."""
    t, c = Tuning(light_max_deg=300), Tuning(chunk_edges=64, heavy_min_deg=100)
    for eb, H, D, N, E, tuning, need in [(2, 1, 32, 33_553_000, 1000, None, 268957696), (4, 4, 32, 1 << 21, 50_000_000, None, 16009728),
                                         (2, 2, 64, 1 << 20, 36_000_000, t, 16650496),
                                         (4, 4, 32, 100_000, 20_000_000, c, 365127680), (2, 4, 512, 1000, 900_000, None, 14598144)]:
        assert attn_plan(shape(N, E, eb, H, D), tuning).need == need
    # the least that is refused with 1x32 bf16 features and next to no entries
    assert attn_plan(shape(33_487_872, 1000, 2, 1, 32)).need <= SCRATCH < attn_plan(shape(33_487_873, 1000, 2, 1, 32)).need


# ------------------------------------------------------------------------- grids


class RowGrid(ctypes.Structure):
    _fields_ = [("blocks", ctypes.c_uint32), ("long_blocks", ctypes.c_uint32), ("light_first", ctypes.c_bool)]


def grid(N, E, groups, slices, tiles=False, resident=1024, tuning=None):
    g = RowGrid()
    probe().probe_grid(ctypes.c_int64(N), ctypes.c_int64(E), groups, slices, int(tiles), resident,
                       ctypes.byref(tuning) if tuning else None, ctypes.byref(g))
    return g.blocks, g.long_blocks


@pytest.mark.parametrize("tiles", [False, True])
@pytest.mark.parametrize("groups,slices", [(1, 4), (2, 2), (4, 1), (4, 8), (8, 1), (16, 1)])
def test_a_batch_per_wave_until_the_device_is_full(groups, slices, tiles):
    """Four waves per workgroup, whole eighths of a grid: a call whose light rows take up to four times the resident
    workgroups with one batch per wave gets that many; larger ones get two batches (four) per wave."""
    for N in (1, 63, 2000, 5003, 4 * 1024 * 4 * groups // slices - 4 * 8 * groups, 2_000_001):
        blocks, long_blocks = grid(N, 8 * N, groups, slices, tiles)
        batches = -(-N // groups)
        light = blocks - long_blocks
        assert blocks % 8 == 0 and long_blocks % 8 == 0 and long_blocks >= 8
        few = -(-batches // 4) * slices <= 4 * 1024 - 8 * slices
        per_wave = 1 if few else 4 if tiles else 2
        assert batches / per_wave <= 4 * light < batches / per_wave + 4 * 8 + 4


def test_long_rows_get_a_wave_per_128_entries():
    """12 K rows of 100 entries, a wavefront each: a wave per 128 entries, were three quarters of them in such rows."""
    for groups in (2, 4, 8, 16):
        _, long_blocks = grid(12_000, 1_200_000, groups, 2)
        assert abs(4 * long_blocks - 0.75 * 1_200_000 / 128) <= 4 * 8 + 4
    assert grid(1 << 20, 1 << 30, 4, 1)[1] == 8 * 1024  # at most eight times what the device holds
    assert grid(1 << 20, 1 << 30, 4, 1, tiles=True)[1] == 2 * 1024


def test_grids_of_the_largest_graphs_can_be_launched():
    """Fewer than 2^32 threads: 256 per workgroup."""
    for groups in (1, 2, 4, 8, 16):
        for N in (1 << 28, 540_000_000, (1 << 31) - 1):
            for resident in (512, 2048):
                blocks, long_blocks = grid(N, (1 << 31) - 1, groups, 1, resident=resident)
                assert blocks * 256 < 1 << 32 and blocks % 8 == 0 and long_blocks < blocks


def test_long_rows_workgroups_come_last_where_all_fit():
    """On graphs of 16 entries per row or more, and few workgroups; never on sparse or large ones."""
    def last(N, E, slices):
        g = RowGrid()
        probe().probe_grid(ctypes.c_int64(N), ctypes.c_int64(E), 4, slices, 0, 1024, None, ctypes.byref(g))
        return g.light_first
    assert last(3000, 300_000, 2) and last(16_000, 256_000, 2)
    assert not last(16_000, 120_000, 2) and not last(3000, 300_000, 8) and not last(1_000_000, 30_000_000, 1)


# ------------------------------------------------------------------------- the rule


@pytest.mark.parametrize("gather,piece,P", [k for k in KERNELS if k[2] >= 4])
@pytest.mark.parametrize("N", [2000, 12_000, 100_000, 2_000_000])
def test_usual_rows_are_light(gather, piece, P, N):
    """Graphs of one degree or about: up to 170 entries a row, no row up to a fifth longer is cut or takes a
    wavefront; and with long rows, eight pieces of each have room."""
    for mean in (1, 7, 32, 34, 50, 53, 60, 71, 99, 107, 150, 170):
        cut, r = rule(N, N * mean, 2, gather, piece, P)
        assert r.light_max >= min(1.2 * mean, 256) or 1.2 * mean <= 64
        assert r.split_min >= max(128, r.light_max + 1)
    for mean in (190, 290, 505):
        cut, r = rule(N, N * mean, 2, gather, piece, P)
        assert r.light_max == 64 and r.split_min in (128, 512)
        assert r.likely_slots >= min(8 * N, r.max_slots) or mean < r.split_min
        # an L2 holds the sources, and the rows fill the device
        assert (r.split_min == 512) == (N * gather <= 4 << 20 and 2 * N >= 4096)


def test_states_of_every_class_have_a_place():
    """max_slots is a bound: rows of one class alone, as many as there can be, in eight pieces each."""
    for gather, piece, P in KERNELS:
        for mean in (3, 24, 60, 200):
            cut, r = rule(100_000, 100_000 * mean, 2, gather, piece, P)
            for c in range(7, 31):
                if (1 << c) >= r.split_min:
                    n = (100_000 * mean) >> c
                    assert n * min(max((2 << c) // r.chunk, 8), 32) <= r.max_slots + 32


@pytest.mark.parametrize("heavy_min_deg", [1, 16, 17, 64, 100, 300, 5000, 2**31 - 2**16])
def test_heavy_min_deg_is_the_shortest_row_that_is_cut(heavy_min_deg):
    """Also below the default."""
    cut, r = rule(100_000, 700_000, 2, 512, 600, 4, Tuning(light_max_deg=4, heavy_min_deg=heavy_min_deg))
    assert r.split_min == max(16, heavy_min_deg)
    for c in range(cut.min_class, 31):
        rows = np.zeros(32)
        rows[c] = 1
        cut.cap_slots = 64
        _, nq, _ = batches(cut, rows, 4) if 700_000 >> c else (0, np.ones(32), 0)
        if 700_000 >> c:
            assert (nq[c] >= 8) == ((1 << c) >= max(16, heavy_min_deg))


def test_wide_slices_are_for_short_wide_rows_of_large_graphs():
    def wide(N, E, row):
        return bool(probe().probe_wide(ctypes.c_int64(N), ctypes.c_int64(E), ctypes.c_int64(row)))
    assert wide(60_000, 240_000, 4096) and wide(49152, 0, 4096) and wide(2**31 - 1, 2**31 - 1, 8192)
    assert not wide(60_000, 330_000, 4096) and not wide(49151, 0, 4096) and not wide(60_000, 240_000, 2048)


@pytest.mark.parametrize("case", ["fwd", "bwd"])
def test_a_graph_whose_classes_get_fewer_and_longer_pieces(case):
    """6200 rows of 600 entries among 60 K (the graph of a GPU test): the rule wants eight pieces each, the states of
    one launch hold four, and those are spread over wavefronts."""
    N, E = 60_000, 6200 * 600 + 53_800 * 3 // 2
    if case == "fwd":  # bf16 8x128
        p = attn_plan(shape(N, E, 2, 8, 128))
        r, cap, slices, P = p.rule, p.slots.cap, p.slots.slices, 4
        cut, _ = rule(N, E, 8, 512, 972, 4)
    else:  # fp32 8x64
        cut, r = rule(N, E, 8, 512, 2 * 512 + 1024, 4)
        s = SlotPlan()
        probe().probe_slots(ctypes.byref(r), 8, ctypes.c_int64(512), ctypes.c_int64(8 * 8 * N + 10 * N + E // 2), 0, ctypes.byref(s))
        cap, slices, P = s.cap, s.slices, 4
    assert slices == 8
    cut.cap_slots = cap
    rows = np.zeros(32)
    rows[9] = 6200
    bound, nq, total = batches(cut, rows, P)
    assert nq[9] == 4 and 1024 // 4 > cut.group_len and int(total.max()) <= bound
    # the waves of the long rows reach past what eight pieces by lane group would have asked for
    assert grid(N, E, P, slices)[1] // 8 * 4 > 6200 * 8 // (8 * P) + 32
