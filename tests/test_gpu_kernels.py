"""Kernel-level GPU tests through the C ABI: sampler (bit-exact), grouped
GEMM (rigorous fp32 error bound), replica average (bit-exact tree, fp64
bound), fused update."""
import numpy as np
import pytest
import torch

import workloads as wk
from oracle import lsgd_oracle as O
from gpu_util import U32, gamma, device, to_dev

pytestmark = pytest.mark.gpu


def _lsgd():
    from paper_1808_07217_amd import lsgd as L
    return L


# ------------------------------------------------------------------ sampler
@pytest.mark.parametrize("K,N,B,seed", [
    (4, 4096, 32, 0x5EED0001), (16, 50000, 128, 0x5EED0002),
    (64, 50000, 64, 0x5EED0004), (3, 10, 5, 1), (1, 7, 9, 2**64 - 1),
    (5, 5, 4, 77), (2, 2**31 - 1, 13, 12345),
])
def test_sampler_bit_exact(K, N, B, seed):
    L = _lsgd()
    print(f"sampler K={K} N={N} B={B}", flush=True)
    cfg = L.make_config((1, 2), K, B, N, seed=seed)
    # the sampler reads neither X nor y: they only have to have N rows
    X = torch.empty((N, 1), device=device())
    y = torch.empty(N, dtype=torch.int32, device=device())
    w0 = torch.zeros(L.param_count(cfg), device=device())
    reps = L.Replicas(cfg, X, y, w0)
    for step in (0, 1, 7, 123456, 2**32 + 11):
        got = reps.sample_indices(step).cpu().numpy()
        want = np.stack([O.sample_indices(seed, step, k, K, N, B) for k in range(K)])
        np.testing.assert_array_equal(got, want)


@pytest.mark.parametrize("K,N,B,seed", [
    (4, 4096, 32, 0x5EED0001), (16, 50000, 128, 0x5EED0002),
    (64, 50000, 64, 0x5EED0004), (3, 10, 3, 1), (1, 7, 7, 2**64 - 1),
    (5, 1000, 4, 77), (2, 2**31 - 1, 13, 12345),
])
def test_epoch_sampler_bit_exact(K, N, B, seed):
    """The per-epoch reshuffled partition: every index of every worker at
    steps on both sides of epoch boundaries, against the oracle's Feistel
    permutation; within an epoch no row repeats."""
    L = _lsgd()
    print(f"epoch sampler K={K} N={N} B={B}", flush=True)
    cfg = L.make_config((1, 2), K, B, N, seed=seed, sampler="epoch")
    X = torch.empty((N, 1), device=device())
    y = torch.empty(N, dtype=torch.int32, device=device())
    w0 = torch.zeros(L.param_count(cfg), device=device())
    reps = L.Replicas(cfg, X, y, w0)
    S = O.steps_per_epoch(K, N, B)
    for step in sorted({0, 1, S - 1, S, S + 1, 5 * S + 2, 123456, 2**32 + 11}):
        got = reps.sample_indices(step).cpu().numpy()
        want = np.stack([O.sample_indices_epoch(seed, step, k, K, N, B) for k in range(K)])
        np.testing.assert_array_equal(got, want)
    if S <= 64:
        epoch = np.concatenate([reps.sample_indices(j).cpu().numpy().ravel()
                                for j in range(S)])
        assert np.unique(epoch).size == epoch.size


# ------------------------------------------------------------------ GEMM
GEMM_SHAPES = [(3, 70, 45, 37), (2, 64, 64, 16), (1, 1, 1, 1), (2, 33, 10, 130),
               (4, 128, 512, 512), (2, 128, 10, 512), (2, 512, 10, 128),
               (2, 3072, 512, 128), (1, 96, 200, 3072)]


@pytest.mark.parametrize("splits", [1, 3])
@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("ta,tb", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("shape", GEMM_SHAPES)
def test_grouped_gemm_error_bound(dtype, ta, tb, shape, splits):
    L = _lsgd()
    G, M, N, Kd = shape
    print(f"gemm {dtype} ta={ta} tb={tb} {shape} splits={splits}", flush=True)
    rng = np.random.default_rng(M * 7 + N * 3 + Kd + ta * 2 + tb)
    A = rng.standard_normal((G, Kd, M) if ta else (G, M, Kd)).astype(np.float32)
    B = rng.standard_normal((G, N, Kd) if tb else (G, Kd, N)).astype(np.float32)
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    Ad, Bd = to_dev(A).to(tdt), to_dev(B).to(tdt)
    C = L.grouped_gemm(Ad, Bd, bool(ta), bool(tb), splits=splits).cpu().numpy().astype(np.float64)
    A64 = Ad.to(torch.float64).cpu().numpy()   # the exact operand values used
    B64 = Bd.to(torch.float64).cpu().numpy()
    opA = A64.transpose(0, 2, 1) if ta else A64
    opB = B64.transpose(0, 2, 1) if tb else B64
    ref = opA @ opB
    bound = gamma(Kd + 1) * (np.abs(opA) @ np.abs(opB)) + 1e-30
    assert np.all(np.abs(C - ref) <= bound), np.max(np.abs(C - ref) / bound)


# whole-tile fp32 shapes, in one range of k and in splits: 64 x 64 tiles in slabs
# of 32 (192 = 6 of them), 128 x 128 ones in slabs of 16 where there are 256 of
# them or (with a split) the inner dimension reaches 2048
@pytest.mark.parametrize("tb", [0, 1])
@pytest.mark.parametrize("shape,splits", [((16, 128, 512, 512), 1), ((16, 128, 512, 512), 2),
                                          ((2, 64, 128, 192), 1), ((2, 256, 256, 3072), 1),
                                          ((2, 128, 256, 2048), 4)])
def test_grouped_gemm_whole_tiles(shape, splits, tb):
    L = _lsgd()
    G, M, N, Kd = shape
    print(f"gemm whole tiles {shape} splits={splits} tb={tb}", flush=True)
    rng = np.random.default_rng(G + M + N + Kd + splits + tb)
    A = rng.standard_normal((G, M, Kd)).astype(np.float32)
    B = rng.standard_normal((G, N, Kd) if tb else (G, Kd, N)).astype(np.float32)
    C = L.grouped_gemm(to_dev(A), to_dev(B), False, bool(tb), splits=splits)
    C = C.cpu().numpy().astype(np.float64)
    opB = B.astype(np.float64).transpose(0, 2, 1) if tb else B.astype(np.float64)
    ref = A.astype(np.float64) @ opB
    bound = gamma(Kd + 1) * (np.abs(A.astype(np.float64)) @ np.abs(opB)) + 1e-30
    assert np.all(np.abs(C - ref) <= bound), np.max(np.abs(C - ref) / bound)


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("ta,tb", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("shape,splits", [((2, 3, 2, 3), 1), ((2, 4, 5, 4), 1),      # quads and less
                                          ((2, 63, 65, 31), 1), ((1, 65, 66, 33), 1),  # 64 x 64 + 1
                                          ((1, 129, 127, 2049), 2),                    # deep, split
                                          ((1, 129, 127, 130), 8)])                    # empty splits
def test_grouped_gemm_ragged_edges(dtype, ta, tb, shape, splits):
    """Every remainder of a tile, a slab and a quad, and infinities among the
    operands: the same positions infinite or NaN as in fp64, the others within
    the fp32 bound."""
    L = _lsgd()
    G, M, N, Kd = shape
    print(f"gemm edges {dtype} ta={ta} tb={tb} {shape} splits={splits}", flush=True)
    rng = np.random.default_rng(M + 5 * N + 7 * Kd + ta * 2 + tb)
    A = rng.standard_normal((G, Kd, M) if ta else (G, M, Kd)).astype(np.float32)
    B = rng.standard_normal((G, N, Kd) if tb else (G, Kd, N)).astype(np.float32)
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    for special in (False, True):
        if special:
            A[0, -1, -1], A[0, 0, 0], B[0, -1, 0] = np.inf, -np.inf, np.inf
        Ad, Bd = to_dev(A).to(tdt), to_dev(B).to(tdt)
        C = L.grouped_gemm(Ad, Bd, bool(ta), bool(tb), splits=splits).cpu().numpy().astype(np.float64)
        A64 = Ad.to(torch.float64).cpu().numpy()
        B64 = Bd.to(torch.float64).cpu().numpy()
        opA = A64.transpose(0, 2, 1) if ta else A64
        opB = B64.transpose(0, 2, 1) if tb else B64
        with np.errstate(invalid="ignore"):
            ref = opA @ opB
            bound = gamma(Kd + 1) * (np.abs(opA) @ np.abs(opB)) + 1e-30
        fin = np.isfinite(ref)
        np.testing.assert_array_equal(C[~fin], ref[~fin])
        assert np.all(np.abs(C[fin] - ref[fin]) <= bound[fin])


@pytest.mark.parametrize("ta,tb", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("shape", [(2, 70, 65, 37), (1, 64, 64, 64), (2, 65, 3, 1), (2, 33, 70, 2),
                                   (1, 128, 256, 3)])
def test_grouped_gemm_over_the_range_of_fp32(shape, ta, tb):
    """Products of fp32 values from subnormal ones to the largest: the fp32 bound
    (and, where a result is subnormal, its spacing per addition) at every scale;
    an inner dimension of one gives the correctly rounded product."""
    L = _lsgd()
    G, M, N, Kd = shape
    rng = np.random.default_rng(M + 3 * N + 5 * Kd + 2 * ta + tb)
    A0 = rng.standard_normal((G, M, Kd)).astype(np.float32)
    B0 = rng.standard_normal((G, Kd, N)).astype(np.float32)
    # scales of A and B as powers of two; some leave products near 2^125, and
    # sums on both sides of 2^96 and operands of 2^112
    for ea, eb in ((-112, 0), (0, -120), (-133, 0), (-128, 30), (-60, -60), (122, 0), (70, 50),
                   (47, 47), (111, -20), (-90, 113)):
        print(f"gemm range {shape} ta={ta} tb={tb} 2^{ea} 2^{eb}", flush=True)
        A, B = np.ldexp(A0, ea), np.ldexp(B0, eb)
        At = A.transpose(0, 2, 1) if ta else A
        Bt = B.transpose(0, 2, 1) if tb else B
        C = L.grouped_gemm(to_dev(At), to_dev(Bt), bool(ta), bool(tb)).cpu().numpy().astype(np.float64)
        A64, B64 = A.astype(np.float64), B.astype(np.float64)
        ref = A64 @ B64
        bound = gamma(Kd + 1) * (np.abs(A64) @ np.abs(B64)) + (Kd + 1) * 2.0**-149
        assert np.all(np.isfinite(C)) and np.all(np.abs(C - ref) <= bound), \
            np.max(np.abs(C - ref) / bound)
        if Kd == 1:
            np.testing.assert_array_equal(C, ref.astype(np.float32))


def test_grouped_gemm_of_more_tiles_than_an_axis_of_the_grid():
    """65535 outer products of 1 x 16448, 257 tiles each: every result."""
    L = _lsgd()
    G, N = 65535, 16448
    A = torch.arange(1, G + 1, dtype=torch.float32, device=device()).view(G, 1, 1)
    B = torch.arange(1, N + 1, dtype=torch.float32, device=device()).expand(G, 1, N).contiguous()
    C = L.grouped_gemm(A, B, out=torch.full((G, 1, N), -1.0, device=device()))
    assert torch.equal(C, A * B)   # whole numbers: each product rounded once


def test_grouped_gemm_products_next_to_the_largest_number():
    """Finite operands whose leading bf16 pieces round up: to an infinity, or to
    a product beyond the largest fp32 number where x y itself is below it."""
    L = _lsgd()
    root = np.float32(2.0**64 * (1 - 2.0**-24))   # its square: 2^128 (1 - 2^-23)
    big = np.float32(np.finfo(np.float32).max)
    for x, y in ((root, root), (big, np.float32(0.5)), (big, np.float32(1)), (-big, np.float32(1))):
        A = np.zeros((1, 70, 40), np.float32)
        B = np.zeros((1, 40, 66), np.float32)
        A[0, :, 17], B[0, 17, :] = x, y
        C = L.grouped_gemm(to_dev(A), to_dev(B)).cpu().numpy()
        want = np.float32(np.float64(x) * np.float64(y))
        assert np.isfinite(want)
        np.testing.assert_array_equal(C, np.full_like(C, want))


# ------------------------------------------------------------------ average
def _tree_f32(rows):
    """The kernel's documented order in fp32: split at the largest power of
    two below n, left part first."""
    n = len(rows)
    if n == 1:
        return rows[0]
    h = 1
    while 2 * h < n:
        h *= 2
    return (_tree_f32(rows[:h]) + _tree_f32(rows[h:])).astype(np.float32)


def _tree_rows(W):
    """The same order on a device tensor's rows."""
    n = W.shape[0]
    if n == 1:
        return W[0]
    h = 1
    while 2 * h < n:
        h *= 2
    return _tree_rows(W[:h]) + _tree_rows(W[h:])


@pytest.mark.parametrize("K,P", [(1, 7), (3, 650), (4, 650), (16, 1841162 + 6),
                                 (64, 10001), (5, 4), (7, 1027)])
def test_replica_average(K, P):
    L = _lsgd()
    print(f"average K={K} P={P}", flush=True)
    rng = np.random.default_rng(K * 1000 + P)
    W = rng.standard_normal((K, P)).astype(np.float32)
    Wd = to_dev(W)
    L.replica_average(Wd)
    got = Wd.cpu().numpy()
    assert np.all(got == got[0:1])
    # bit-exact against the documented fp32 summation tree, then / K
    want = (_tree_f32([W[k] for k in range(K)]) / np.float32(K)).astype(np.float32)
    np.testing.assert_array_equal(got[0], want)
    # and within the pairwise-summation bound of the fp64 oracle mean
    ref = O.average(W.astype(np.float64))[0]
    depth = int(np.ceil(np.log2(K))) if K > 1 else 0
    bound = gamma(depth) * np.abs(W).astype(np.float64).sum(0) / K + U32 * np.abs(ref)
    assert np.all(np.abs(got[0] - ref) <= bound + 1e-45)


@pytest.mark.parametrize("K,P", [(6, 4099), (10, 1026), (12, 1025), (24, 1027),
                                 (5, (13 << 20) + 3)])  # 273 MB: streamed past the caches
def test_replica_average_rows_at_any_alignment(K, P):
    L = _lsgd()
    print(f"average K={K} P={P}", flush=True)
    W = np.random.default_rng(K + P).standard_normal((K, P), dtype=np.float32)
    Wd = to_dev(W)
    L.replica_average(Wd)
    got = Wd.cpu().numpy()
    want = (_tree_f32([W[k] for k in range(K)]) / np.float32(K)).astype(np.float32)
    for k in range(K):
        np.testing.assert_array_equal(got[k], want)


@pytest.mark.parametrize("K", [3, 5, 7, 9, 13, 15, 17, 20, 22, 31, 48, 63, 65, 100, 127, 128, 131, 300])
def test_averages_of_any_count(K):
    """Both averages in the documented order, bit for bit, for counts with an
    instance of their own, made of blocks of eight, and beyond 127; the rows'
    last elements no whole vector. (With m = 0, a step size of 1, w_s = 0 and
    u = 0 the global-momentum form leaves the mean.)"""
    L = _lsgd()
    for P in (1, 3, 1026, 2051):
        print(f"average K={K} P={P}", flush=True)
        W = np.random.default_rng(K + P).standard_normal((K, P), dtype=np.float32)
        want = (_tree_f32([W[k] for k in range(K)]) / np.float32(K)).astype(np.float32)
        Wd = to_dev(W)
        L.replica_average(Wd)
        np.testing.assert_array_equal(Wd.cpu().numpy(), np.broadcast_to(want, (K, P)))
        Wd, ws, u = to_dev(W), torch.zeros(P, device=device()), torch.zeros(P, device=device())
        L.replica_average_global_momentum(Wd, ws, u, 0.0, 1.0)
        np.testing.assert_array_equal(Wd.cpu().numpy(), np.broadcast_to(want, (K, P)))
        np.testing.assert_array_equal(u.cpu().numpy(), -want)


@pytest.mark.parametrize("K,P", [(5, (17 << 20) + 3), (20, (5 << 20) + 1)])  # 357 and 420 MB
def test_averages_streamed_past_the_caches(K, P):
    """Both averages, and the plain one within two blocks, on arrays that take
    the nontemporal form, bit for bit as in any other size."""
    L = _lsgd()
    print(f"streamed averages K={K} P={P}", flush=True)
    W = to_dev(np.random.default_rng(K).standard_normal((K, P), dtype=np.float32))

    def want(k0, k1):  # the documented order, on the device, in fp32
        t = _tree_rows(W[k0:k1]) / torch.full((), k1 - k0, dtype=torch.float32, device=device())
        return t.expand(k1 - k0, P)

    Wd = W.clone()
    L.replica_average(Wd)
    assert torch.equal(Wd, want(0, K))
    Wd, ws, u = W.clone(), torch.zeros(P, device=device()), torch.zeros(P, device=device())
    L.replica_average_global_momentum(Wd, ws, u, 0.0, 1.0)
    assert torch.equal(Wd, want(0, K))
    if K % 2 == 0:
        Wd = W.clone()
        L.replica_average_blocks(Wd, K // 2)
        assert torch.equal(Wd, torch.cat([want(0, K // 2), want(K // 2, K)]))


@pytest.mark.parametrize("K", [1, 2, 4, 16, 64])
def test_average_of_identical_replicas_is_identity(K):
    L = _lsgd()
    w = np.random.default_rng(K).standard_normal(4099).astype(np.float32)
    Wd = to_dev(np.repeat(w[None], K, axis=0))
    L.replica_average(Wd)
    np.testing.assert_array_equal(Wd.cpu().numpy(), np.repeat(w[None], K, axis=0))
    L.replica_average(Wd)  # averaging is idempotent, bit for bit
    np.testing.assert_array_equal(Wd.cpu().numpy()[0], w)


@pytest.mark.parametrize("K,Kb,P", [(16, 4, 1841162 + 6), (16, 2, 4099),
                                    (8, 8, 1027), (8, 1, 650), (6, 3, 7),
                                    (64, 16, 10001), (12, 4, 5), (10, 5, 4096)])
def test_replica_average_blocks(K, Kb, P):
    """Hierarchical block synchronisation: each block of Kb consecutive rows
    is replaced by its mean, bit-exact against the same fp32 tree within the
    block and within the pairwise bound of the oracle's block mean."""
    L = _lsgd()
    print(f"block average K={K} Kb={Kb} P={P}", flush=True)
    rng = np.random.default_rng(K * 100 + Kb * 10 + P)
    W = rng.standard_normal((K, P)).astype(np.float32)
    Wd = to_dev(W)
    L.replica_average_blocks(Wd, Kb)
    got = Wd.cpu().numpy()
    ref = O.average_blocks(W.astype(np.float64), Kb)
    depth = int(np.ceil(np.log2(Kb))) if Kb > 1 else 0
    for b in range(K // Kb):
        rows = W[b * Kb:(b + 1) * Kb]
        want = (_tree_f32(list(rows)) / np.float32(Kb)).astype(np.float32)
        for k in range(b * Kb, (b + 1) * Kb):
            np.testing.assert_array_equal(got[k], want)
        bound = (gamma(depth) * np.abs(rows).astype(np.float64).sum(0) / Kb
                 + U32 * np.abs(ref[b * Kb]))
        assert np.all(np.abs(got[b * Kb] - ref[b * Kb]) <= bound + 1e-45)
    if Kb == K:
        Wd2 = to_dev(W)
        L.replica_average(Wd2)
        np.testing.assert_array_equal(Wd2.cpu().numpy(), got)


def test_replica_average_blocks_rejects_a_block_size_not_dividing_k():
    L = _lsgd()
    Wd = to_dev(np.zeros((6, 8), np.float32))
    with pytest.raises(L.LsgdError):
        L.replica_average_blocks(Wd, 4)


@pytest.mark.parametrize("K,P,mg,lr", [(16, 1841162 + 6, 0.3, 0.001),
                                       (4, 650, 0.9, 0.1), (5, 1027, 0.5, 0.02),
                                       (1, 7, 0.0, 0.05), (64, 4100, 0.7, 0.01)])
def test_replica_average_global_momentum(K, P, mg, lr):
    """Global-momentum synchronisation against the oracle, elementwise within
    an fp32 bound: the mean by the K-way tree (gamma_depth of sum |w| / K),
    then a handful of roundings on the difference, the buffer and the step,
    each at most u times the magnitudes involved."""
    L = _lsgd()
    print(f"global momentum average K={K} P={P} mg={mg}", flush=True)
    rng = np.random.default_rng(K * 31 + P)
    ws = rng.standard_normal(P).astype(np.float32)
    W = (ws[None] + 0.01 * rng.standard_normal((K, P))).astype(np.float32)
    u = (rng.standard_normal(P) * 0.5).astype(np.float32)
    Wd, wsd, ud = to_dev(W), to_dev(ws), to_dev(u)
    L.replica_average_global_momentum(Wd, wsd, ud, mg, lr)
    W_got, ws_got, u_got = (t.cpu().numpy().astype(np.float64) for t in (Wd, wsd, ud))
    W_ref, ws_ref, u_ref = O.average_global_momentum(
        W.astype(np.float64), ws.astype(np.float64), u.astype(np.float64), mg, lr)
    assert np.all(W_got == W_got[0:1])
    np.testing.assert_array_equal(W_got[0], ws_got)
    depth = int(np.ceil(np.log2(K))) if K > 1 else 0
    a = np.abs
    e_mean = gamma(depth + 1) * a(W).astype(np.float64).sum(0) / K
    mean = W.astype(np.float64).mean(0)
    e_u = 2 * (e_mean / lr + 4 * U32 * (a(mg * u) + a(ws - mean) / lr + a(u_ref)
                                         + a(ws) / lr))
    e_w = 2 * (e_mean + 4 * U32 * (a(ws) + a(ws - mean) + a(ws_ref)
                                   + lr * a(mg * u) + lr * a(u_ref)))
    assert np.all(a(u_got - u_ref) <= e_u), np.max(a(u_got - u_ref) / e_u)
    assert np.all(a(ws_got - ws_ref) <= e_w), np.max(a(ws_got - ws_ref) / e_w)


def test_update_of_more_elements_than_an_axis_of_the_grid_holds_threads():
    """2^32 + 5 elements, one a thread (no whole vectors): every one updated."""
    L = _lsgd()
    n = 2**32 + 5
    W, U = torch.zeros(n, device=device()), torch.zeros(n, device=device())
    L.sgd_update(W, U, torch.ones(n, device=device()), 0.5, 0.0, 0.0)
    for t, v in ((W, -0.5), (U, 1.0)):
        assert all(bool((t[i:i + 2**28] == v).all()) for i in range(0, n, 2**28))


# ------------------------------------------------- sign-compressed sync
@pytest.mark.parametrize("K,P,ef", [(16, 1841168, False), (16, 1841168, True),
                                    (4, 8192 + 4, False), (3, 260, True),
                                    (1, 4, False), (64, 10004, True)])
def test_replica_sign_sync(K, P, ef):
    """Sign-compressed synchronisation (Algorithm 3; Algorithm 4 with the
    memories). Signs are decided in fp32 on the kernel's documented
    arithmetic ((w_s - w) + e), so the test takes them from the same fp32
    expression: a wrong or missed sign would move an element by at least
    p / K, far outside the rounding bound checked here. Against the fp64
    oracle, elements whose exact difference is within fp32 rounding of zero
    (possible only with memories) may carry either sign. Exact zeros
    (replica elements equal to w_s) must give sign 0."""
    L = _lsgd()
    print(f"sign sync K={K} P={P} ef={ef}", flush=True)
    rng = np.random.default_rng(K * 7 + P + ef)
    ws = rng.standard_normal(P).astype(np.float32)
    W = (ws[None] + 0.01 * rng.standard_normal((K, P))).astype(np.float32)
    W = np.where(rng.random((K, P)) < 0.05, ws[None], W).astype(np.float32)
    E = (0.003 * rng.standard_normal((K, P))).astype(np.float32) if ef else None
    Wd, wsd = to_dev(W), to_dev(ws)
    Ed = to_dev(E) if ef else None
    L.replica_sign_sync(Wd, wsd, Ed)
    got_w = wsd.cpu().numpy().astype(np.float64)
    assert np.all(Wd.cpu().numpy() == wsd.cpu().numpy()[None])

    d32 = (ws[None] - W) + E if ef else ws[None] - W          # fp32 decisions
    p64 = np.abs(d32).astype(np.float64).sum(axis=1) / P
    msgs = np.sign(d32).astype(np.float64) * p64[:, None]
    mine = ws.astype(np.float64) - msgs.sum(axis=0) / K
    bound = 4 * U32 * (np.abs(ws) + np.abs(msgs).sum(axis=0) / K) + 1e-30
    assert np.max(bound) < 0.5 * p64.min() / K       # one flipped sign shows
    assert np.all(np.abs(got_w - mine) <= bound), np.max(np.abs(got_w - mine) / bound)
    if ef:
        got_E = Ed.cpu().numpy().astype(np.float64)
        e_mine = d32.astype(np.float64) - msgs
        assert np.all(np.abs(got_E - e_mine) <= 4 * U32 * (np.abs(d32) + p64[:, None]))

    # the fp64 oracle
    W64, ws64 = W.astype(np.float64), ws.astype(np.float64)
    _, w_ref, E_ref = O.average_sign_compressed(W64, ws64, None if E is None
                                                else E.astype(np.float64))
    d64 = ws64[None] - W64 + (0 if E is None else E)
    amb = np.abs(d64) <= 4 * U32 * (np.abs(ws64[None] - W64) +
                                    (0 if E is None else np.abs(E)))
    if not ef:
        assert not amb[np.abs(d64) > 0].any()      # differences of fp32 values
    allow = bound + 4 * U32 * np.abs(w_ref) + (2 * p64[:, None] * amb).sum(axis=0) / K
    assert np.all(np.abs(got_w - w_ref) <= allow)
    assert np.array_equal(np.sign(d32) == 0, d64 == 0) or ef


# ------------------------------------------------------------------ update
@pytest.mark.parametrize("nesterov", [False, True])
def test_sgd_update_sign_step(nesterov):
    """The signSGD local step: every element moves by exactly lr * sign(d)
    (one fp32 rounding of w -+ lr), the buffer as in the plain step; where d
    is within fp32 rounding of zero either move (or none) is valid."""
    L = _lsgd()
    n = 1 << 16
    rng = np.random.default_rng(77 + nesterov)
    w, u, g = (rng.standard_normal(n).astype(np.float32) for _ in range(3))
    g[:64] = -1e-4 * w[:64] - 0.9 * u[:64]       # directions near zero
    Wd, Ud, Gd = to_dev(w), to_dev(u), to_dev(g)
    L.sgd_update(Wd, Ud, Gd, 0.01, 0.9, 1e-4, nesterov, sign_step=True)
    w2, u2 = O.sgd_update(w.astype(float), u.astype(float), g.astype(float),
                          0.01, 0.9, 1e-4, nesterov, sign_step=True)
    _, u_plain = O.sgd_update(w.astype(float), u.astype(float), g.astype(float),
                              0.01, 0.9, 1e-4, nesterov)
    gw = Wd.cpu().numpy().astype(np.float64)
    np.testing.assert_allclose(Ud.cpu().numpy(), u_plain, rtol=0,
                               atol=float(np.max(4 * U32 * (np.abs(u) + np.abs(g) + np.abs(w)))))
    gg = g + 1e-4 * w
    uu = 0.9 * u.astype(float) + gg
    d = gg + 0.9 * uu if nesterov else uu
    scale = np.abs(gg) + np.abs(uu) * (1.9 if nesterov else 1.0) + np.abs(w)
    clear = np.abs(d) > 8 * U32 * scale
    assert clear.sum() > n - 200
    np.testing.assert_allclose(gw[clear], w2[clear], rtol=0,
                               atol=float(np.max(U32 * np.abs(w2))) * 2)
    moved = np.abs(gw[~clear] - w[~clear])
    assert np.all((moved <= 2 * U32 * np.abs(w[~clear])) |
                  (np.abs(moved - 0.01) <= 4 * U32 * (np.abs(w[~clear]) + 0.01)))


@pytest.mark.parametrize("nesterov", [False, True])
@pytest.mark.parametrize("n", [1, 3, 4099, 1 << 20])
def test_sgd_update_matches_oracle(nesterov, n):
    L = _lsgd()
    rng = np.random.default_rng(n + nesterov)
    w, u, g = (rng.standard_normal(n).astype(np.float32) for _ in range(3))
    Wd, Ud, Gd = to_dev(w), to_dev(u), to_dev(g)
    L.sgd_update(Wd, Ud, Gd, 0.05, 0.9, 1e-4, nesterov)
    w2, u2 = O.sgd_update(w.astype(float), u.astype(float), g.astype(float),
                          0.05, 0.9, 1e-4, nesterov)
    scale_u = np.abs(u) + np.abs(g) + 1e-4 * np.abs(w)
    assert np.all(np.abs(Ud.cpu().numpy() - u2) <= 4 * U32 * scale_u)
    scale_w = np.abs(w) + 0.05 * 2 * scale_u
    assert np.all(np.abs(Wd.cpu().numpy() - w2) <= 8 * U32 * scale_w)
