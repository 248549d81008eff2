"""The row partition's edges, on small graphs against the oracle: degrees around
the light bound and the degree octaves (rows whole, cut into pieces, spread over
a wavefront), more long rows than there are partial states for (classes get
fewer pieces), and rows in no order.  Every (lane group, heads per slice)
combination of the slices."""
import math

import numpy as np
import pytest

import oracle
import synth
from tests.helpers import TOL_BF16, TOL_F32, gate_error, run_gpu

pytestmark = pytest.mark.gpu

SHAPES = [("f32", 4, 32), ("f32", 8, 64), ("f32", 2, 128), ("f32", 1, 256), ("bf16", 1, 32), ("bf16", 4, 32),
          ("bf16", 2, 64), ("bf16", 8, 128), ("bf16", 2, 256), ("bf16", 1, 512)]
EDGES = [0, 1, 2, 3, 4, 5, 7, 8, 9, 15, 16, 17, 31, 32, 33, 63, 64, 65, 127, 128, 129, 255, 256, 257, 511, 512, 513,
         1023, 1024, 1025, 2047, 2048, 2600]


def graph(kind):
    """(rowptr, colidx) of N = 2700 nodes."""
    N = 2700
    rng = np.random.default_rng(5)
    if kind == "edges":
        deg = np.zeros(N, dtype=np.int64)
        deg[rng.permutation(N)[:4 * len(EDGES)]] = EDGES * 4
    elif kind == "many_short_pieces":  # rows just above the light bound: eight pieces each would not fit
        deg = np.full(N, 33, dtype=np.int64)
        deg[rng.permutation(N)[:40]] = 700
    else:
        deg = rng.integers(0, 90, N)
        deg[[0, 77, N - 1]] = (2500, 1300, 600)
    rowptr, colidx = synth.csr_from_degrees(9, N, deg, self_loops=False)
    if kind == "unsorted":
        for r in range(N):
            rng.shuffle(colidx[rowptr[r]:rowptr[r + 1]])
    return rowptr, colidx


@pytest.mark.parametrize("kind", ["edges", "many_short_pieces", "unsorted"])
@pytest.mark.parametrize("dtype,H,D", SHAPES)
def test_forward_at_partition_edges(dtype, H, D, kind):
    rowptr, colidx = graph(kind)
    Q, K, V = synth.features(H * D, rowptr.size - 1, H, D, dtype)
    scale = np.float32(1 / math.sqrt(D))
    got = run_gpu(rowptr, colidx, Q, K, V, scale)
    assert np.array_equal(got, run_gpu(rowptr, colidx, Q, K, V, scale))  # list orders differ from call to call
    ref, absagg, _ = oracle.gt_attn_fwd(rowptr, colidx, Q, K, V, scale, want_lse=False)
    assert gate_error(got, ref, absagg) <= (TOL_F32 if dtype == "f32" else TOL_BF16)


@pytest.mark.parametrize("kind", ["edges", "many_short_pieces", "unsorted"])
@pytest.mark.parametrize("dtype,F", [("f32", 16), ("f32", 64), ("f32", 512), ("bf16", 32), ("bf16", 256)])
def test_reduce_at_partition_edges(dtype, F, kind):
    """Values and sources, bit for bit."""
    from tests.test_gpu_reduce import check, features
    rowptr, colidx = graph(kind)
    check(rowptr, colidx, features(F, rowptr.size - 1, F, dtype), dtype, "max")


@pytest.mark.parametrize("kind", ["edges", "many_short_pieces", "unsorted"])
@pytest.mark.parametrize("dtype,H,D", [("f32", 4, 32), ("f32", 1, 128), ("bf16", 8, 64)])
def test_backward_at_partition_edges(dtype, H, D, kind):
    from tests.test_gpu_bwd import check_grads
    from tests.helpers import run_gpu_fwd_bwd
    rowptr, colidx = graph(kind)
    N, seed = rowptr.size - 1, 3 * H * D
    Q, K, V = synth.features(seed, N, H, D, dtype)
    dO, _, _ = synth.features(seed + 1, N, H, D, dtype)
    scale = np.float32(1 / math.sqrt(D))
    got = run_gpu_fwd_bwd(rowptr, colidx, Q, K, V, dO, scale)
    check_grads(rowptr, colidx, Q, K, V, dO, scale, got, dtype)


@pytest.mark.parametrize("op,dtype,width", [("reduce", "f32", 1024), ("reduce", "bf16", 2048), ("gatv2", "f32", 1024)])
def test_wide_slices_of_short_rows(op, dtype, width):
    """4 KB rows of four entries on average, worked on in slices of 1 KB (one lane group per wavefront), some of them
    long enough to be cut."""
    N = 48 * 1024 + 61
    rng = np.random.default_rng(17)
    deg = rng.integers(0, 8, N)
    longs = rng.permutation(N)[:30]
    deg[longs] = np.resize([255, 256, 257, 511, 513, 700, 1500, 4100], 30)
    rowptr, colidx = synth.csr_from_degrees(19, N, deg, self_loops=False)
    assert 2 * colidx.size < 11 * N
    rows = np.unique(np.concatenate([longs, rng.integers(0, N, 1500), [0, N - 1]]))
    if op == "reduce":
        from tests.test_gpu_reduce import check, features
        check(rowptr, colidx, features(5, N, width, dtype), dtype, "min", rows=rows)
    else:
        from tests.test_gpu_gatv2 import SLOPE, attention_vector, check
        L, R, _ = synth.features(6, N, 8, width // 8, dtype)
        check(rowptr, colidx, L, R, attention_vector(7, 8, width // 8), SLOPE, dtype, rows=rows)


@pytest.mark.parametrize("op,dtype,H,D", [("fwd", "bf16", 8, 128), ("bwd", "f32", 8, 64)])
def test_classes_short_of_partial_states(op, dtype, H, D):
    """6200 rows of 600 entries want eight pieces each, more partial states than the launch has: they get four, too long
    for one lane group, and every piece takes a wavefront (tests/test_plan.py shows that this graph does so)."""
    N, n_long = 60_000, 6200
    rng = np.random.default_rng(23)
    deg = rng.integers(0, 4, N)
    longs = np.sort(rng.permutation(N)[:n_long])
    deg[longs] = 600
    rowptr = np.zeros(N + 1, dtype=np.int64)
    rowptr[1:] = np.cumsum(deg)
    colidx = rng.integers(0, N, rowptr[-1]).astype(np.int32)
    for r in longs:
        colidx[rowptr[r]:rowptr[r + 1]].sort()
    Q, K, V = synth.features(31, N, H, D, dtype)
    scale = np.float32(1 / math.sqrt(D))
    rows = np.unique(np.concatenate([longs[::17], longs[-20:], rng.integers(0, N, 300)]))
    if op == "fwd":
        got = run_gpu(rowptr, colidx, Q, K, V, scale)[rows]
        ref, absagg, _ = oracle.gt_attn_fwd(rowptr, colidx, Q, K, V, scale, rows=rows, want_lse=False)
        assert np.all(np.isfinite(got)) and gate_error(got, ref, absagg) <= TOL_BF16
    else:
        from tests.helpers import run_gpu_fwd_bwd
        from tests.test_gpu_bwd import check_grads
        dO, _, _ = synth.features(32, N, H, D, dtype)
        got = run_gpu_fwd_bwd(rowptr, colidx, Q, K, V, dO, scale)
        check_grads(rowptr, colidx, Q, K, V, dO, scale, got, dtype, rows=rows, cols=rows[::9])
