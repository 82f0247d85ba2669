"""End-to-end parity of the HIP path with the CPU oracle, through the C ABI.

Tolerances (the floating-point bar of the build):
  * fp32 parameters: whole-vector normwise max |a - b| / max |b| <= 1e-5;
  * fp32 losses: relative error <= 1e-3 over the trajectory;
  * bf16 GEMM operands (fp32 master weights): losses <= 2e-2 relative;
  * sampled indices: bit-exact (checked in the kernel tests and here through
    the losses' data).
"""
import numpy as np
import pytest
import torch

import workloads as wk
from oracle import lsgd_oracle as O
from gpu_util import make_replicas, normwise, rel, device

pytestmark = pytest.mark.gpu

PARAM_TOL_FP32 = 1e-5
LOSS_TOL_FP32 = 1e-3
LOSS_TOL_BF16 = 2e-2
# bf16 operands: the GPU's errors against the bf16 oracle must stay below
# this fraction of the oracle's own distance to its run without roundings
NR_RATIO = 0.5


def _small(widths, dtype="fp32", nesterov=False, K=3, B=20, N=999, H=3,
           rounds=2, momentum=0.9, wd=1e-3, lr=0.02):
    return wk.Workload(name="small", model="mlp", widths=widths, dtype=dtype,
                       K=K, B_loc=B, H=H, rounds=rounds, lr=lr,
                       momentum=momentum, nesterov=nesterov, weight_decay=wd,
                       data="custom", N=N, sample_seed=0xABCDEF + K * 7 + B)


def _small_data(w, seed=5):
    rng = np.random.default_rng(seed)
    C = w.widths[-1]
    mu = rng.standard_normal((C, w.widths[0]))
    y = rng.integers(0, C, w.N).astype(np.int32)
    X = (mu[y] + rng.standard_normal((w.N, w.widths[0]))).astype(np.float32)
    w0 = np.concatenate([
        np.concatenate([(rng.standard_normal(a * b) * np.sqrt(2.0 / a)),
                        rng.standard_normal(b) * 0.1])
        for a, b in wk.layer_shapes(w.widths)]).astype(np.float32)
    return X, y, w0


def _compare_steps(w, X, y, w0, param_tol, loss_tol, rounds=None, nr_ratio=None):
    """Run both sides round by round; compare every replica after every
    local step and after every average.

    nr_ratio (bf16 operands): the oracle also runs the same schedule with
    every bf16 rounding removed, and the GPU's worst parameter and loss
    errors must stay below nr_ratio times that variant's largest distance
    from the bf16 oracle -- a path that skipped or misplaced the roundings
    lands at about that distance, so the bar tells the two apart."""
    reps = make_replicas(w, X, y, w0)
    st = O.State(w0, w.K)
    nr = O.State(w0, w.K) if nr_ratio else None
    w_nr = w.scaled(dtype="fp32")
    loss_d = torch.empty(w.K, device=device())
    worst = worst_loss = d_nr = dl_nr = 0.0
    for t, (H, lr) in enumerate(O.schedule(w)[:rounds]):
        for h in range(H):
            reps.local_step(lr, loss_d)
            want_loss = O.local_step(st, w, X, y, lr)
            got_loss = loss_d.cpu().numpy()
            assert np.all(rel(got_loss, want_loss) <= loss_tol), (t, h, got_loss, want_loss)
            worst_loss = max(worst_loss, float(np.max(rel(got_loss, want_loss))))
            if nr is not None:
                l_nr = O.local_step(nr, w_nr, X, y, lr)
                dl_nr = max(dl_nr, float(np.max(rel(l_nr, want_loss))))
            for k in range(w.K):
                e = normwise(reps.read_params(k).cpu().numpy(), st.W[k])
                worst = max(worst, e)
                assert e <= param_tol, (t, h, k, e)
                if nr is not None:
                    d_nr = max(d_nr, normwise(nr.W[k], st.W[k]))
        reps.average()
        st.W = O.average(st.W)
        if nr is not None:
            nr.W = O.average(nr.W)
        e = normwise(reps.read_params(-1).cpu().numpy(), st.W[0])
        assert e <= param_tol, (t, "avg", e)
        for k in (0, w.K - 1):
            np.testing.assert_array_equal(reps.read_params(k).cpu().numpy(),
                                          reps.read_params(0).cpu().numpy())
    if nr is not None:
        print(f"bf16: GPU params {worst:.3e}, losses {worst_loss:.3e}; oracle without "
              f"rounding: params {d_nr:.3e}, losses {dl_nr:.3e}", flush=True)
        assert worst <= nr_ratio * d_nr, (worst, d_nr)
        assert worst_loss <= nr_ratio * dl_nr, (worst_loss, dl_nr)
    return worst


@pytest.mark.parametrize("widths,nesterov,momentum", [
    ((70, 48, 36, 10), False, 0.9),
    ((70, 48, 36, 10), True, 0.9),
    ((64, 128, 64, 10), False, 0.0),
    ((37, 10), False, 0.5),
    ((130, 200, 66, 100, 7), True, 0.9),
    ((50, 24, 20), False, 0.9),        # 17..32 classes: the head of 32
    ((40, 33, 45), True, 0.9),         # > 32 classes: generic GEMM + loss path
    ((100, 256, 10), False, 0.9),      # register-resident head, 256 inputs
    ((48, 512, 512, 10), True, 0.9),   # register-resident head, 512 inputs
    ((64, 64, 13), True, 0.9),         # 13 classes: the head of 16
    ((128, 16), False, 0.9),           # the same, gathered rows, its own update
])
def test_small_mlp_every_step(widths, nesterov, momentum):
    w = _small(widths, nesterov=nesterov, momentum=momentum)
    print(f"small fp32 {widths} nesterov={nesterov}", flush=True)
    X, y, w0 = _small_data(w)
    _compare_steps(w, X, y, w0, PARAM_TOL_FP32, 1e-4)


@pytest.mark.parametrize("widths,K,B,dtype", [
    ((1025, 12), 3, 129, "fp32"),         # the head alone, gathered rows, a second pass of one row
    ((300, 17), 2, 7, "bf16"),
    ((31, 65, 32), 2, 127, "fp32"),       # 32 classes over 65 inputs, tiles of 64 + 1
    ((5, 3, 2), 2, 3, "fp32"),            # layers below a quad
    ((33, 130, 67, 11), 2, 33, "bf16"),   # bf16 rows at odd alignment, a batch of a slab + 1
    ((1000, 1040, 10), 32, 8, "fp32"),    # 268 MB of state: the update streamed past the caches
    ((1024, 1024, 10), 32, 80, "fp32"),   # and in whole tiles, five slabs
    ((1024, 1024, 10), 32, 64, "bf16"),
])
def test_update_and_head_at_tile_edges(widths, K, B, dtype):
    """Every layer's update, the losses and the next step's rows in one launch,
    and the head's kernels, at the edges of their tiles, quads and class
    counts; every replica after every step."""
    big = K > 3
    w = _small(widths, dtype=dtype, nesterov=True, K=K, B=B, lr=0.01, H=1 if big else 3,
               rounds=1 if big else 2)
    print(f"edges {widths} K={K} B={B} {dtype}", flush=True)
    X, y, w0 = _small_data(w)
    if dtype == "bf16":
        _compare_steps(w, X, y, w0, 2e-3, LOSS_TOL_BF16, nr_ratio=NR_RATIO)
    else:
        _compare_steps(w, X, y, w0, PARAM_TOL_FP32, 1e-4)


@pytest.mark.parametrize("widths,B", [((64, 64), 64),        # whole tiles
                                      ((64, 128, 10), 64),
                                      ((37, 45), 600)])      # ragged; rows past those kept in LDS
def test_a_value_beyond_the_split_products(widths, B):
    """One step with the largest fp32 number, which rounds to an infinity in
    bf16, in a dataset row that replica 0 draws: the wavefronts that meet it (as
    a gathered row of the forward product and of the update) form their tiles
    with the fp32 instruction. Every row of every layer, on its own scale."""
    w = _small(widths, B=B, N=4000, K=2, H=1, rounds=1, lr=0.01)
    X, y, w0 = _small_data(w)
    row = int(O.sample_indices(w.sample_seed, 0, 0, w.K, w.N, B)[B - 1])
    X[row, 5] = np.finfo(np.float32).max
    w0 *= np.float32(0.05)               # activations and logits below it
    y[row] = (y[row] + 1) % widths[-1]   # a class this row does not put first
    reps = make_replicas(w, X, y, w0)
    reps.local_step(w.lr)
    st = O.State(w0, w.K)
    O.local_step(st, w, X, y, w.lr)
    for k in range(w.K):
        got = O.unpack(reps.read_params(k).cpu().numpy().astype(np.float64), w.widths)
        for (gw, gb), (ow, ob) in zip(got, O.unpack(st.W[k], w.widths)):
            assert (np.abs(ow).max() > 1e28) == (k == 0)
            err = np.abs(gw - ow).max(axis=1) / np.abs(ow).max(axis=1)
            assert err.max() <= PARAM_TOL_FP32, (k, err.max())
            assert normwise(gb, ob) <= PARAM_TOL_FP32


def test_update_of_more_tiles_than_an_axis_of_the_grid():
    """33000 replicas of a 1-16384-2 network: 512 nearly empty tiles each, more
    workgroups together than an axis of a launch holds threads; replicas on both
    sides of every row of the grid, two steps (the second on rows that the first
    one drew)."""
    K, lr = 33000, 0.05
    w = _small((1, 16384, 2), K=K, B=1, N=K, H=2, rounds=1, lr=lr)
    X, y, w0 = _small_data(w)
    reps = make_replicas(w, X, y, w0)
    loss = torch.empty(2, K, device=device())
    for h in range(2):
        reps.local_step(lr, loss[h])
    loss = loss.cpu().numpy()
    # workgroups 2^23 and 2^24, behind 33136 of the losses and the sampler: tiles
    # of layer 1 of replica 32638 and of layer 2 of replica 32406
    for k in (0, 1, 32405, 32406, 32407, 32637, 32638, 32639, K - 1):
        m, u = w0.astype(np.float64), np.zeros(w0.size)
        for h in range(2):
            idx = O.sample_indices(w.sample_seed, h, k, K, w.N, 1)
            want, g = O.loss_and_grad(m, w.widths, X[idx], y[idx])
            m, u = O.sgd_update(m, u, g, lr, w.momentum, w.weight_decay, False)
            assert rel(loss[h, k], want) <= 1e-4, (k, h)
        assert normwise(reps.read_params(k).cpu().numpy(), m) <= PARAM_TOL_FP32, k
        assert normwise(reps.read_momentum(k).cpu().numpy(), u) <= 1e-4, k
    reps.close()


def test_batch_larger_than_the_gathered_row_cache():
    """A local batch of 600 rows (the weight-gradient kernel caches 512
    gathered row indices in LDS and reads the rest from memory)."""
    w = _small((70, 36, 10), B=600, N=5000, K=2, H=2, rounds=1, lr=0.01)
    X, y, w0 = _small_data(w)
    _compare_steps(w, X, y, w0, PARAM_TOL_FP32, 1e-4)


@pytest.mark.parametrize("widths,K,B,nesterov,seed", [
    ((256, 2048, 10), 32, 21, False, 5),       # gathered rows, slabs that end early
    ((384, 384, 384, 10), 115, 9, True, 6),    # 8970 tiles, no multiple of the 8 XCDs
    ((64, 1024, 1024, 10), 16, 20, False, 5),  # layers one tile high, activation rows
    ((512, 1024, 512, 10), 16, 128, True, 5),  # whole tiles and slabs below the head
])
def test_update_launch_shapes(widths, K, B, nesterov, seed):
    """The launch that updates every layer in 64 x 64 tiles, thousands of them
    (several a compute unit): every replica after every step.

    The data seeds keep every ReLU pre-activation of these runs clear of
    zero at fp32 resolution: perturbing the oracle's own initial weights by
    1e-7 (relative) moves every replica's parameters by at most ~3e-7. (With
    seed 5 the 115-replica case puts one hidden unit of replica 32 on the
    kink at the fourth step, where the same perturbation moves the fp64
    oracle by 2.45e-4 -- an fp32 result can legitimately differ there.)"""
    w = _small(widths, nesterov=nesterov, K=K, B=B, N=max(999, 4 * K), H=2,
               rounds=2, lr=0.01)
    print(f"update launch {widths} K={K} B={B}", flush=True)
    X, y, w0 = _small_data(w, seed=seed)
    _compare_steps(w, X, y, w0, PARAM_TOL_FP32, 1e-4)


@pytest.mark.parametrize("widths,K,B", [
    ((256, 2048, 10), 32, 21),        # gathered bf16 rows, a slab that ends early
    ((512, 1024, 512, 10), 16, 64),   # whole tiles and slabs of 64
])
def test_update_launch_bf16(widths, K, B):
    """The same launch on bf16 operands (fp32 master weights and momentum, the
    bf16 weight copy written by the update), every replica after every step."""
    w = _small(widths, dtype="bf16", K=K, B=B, N=max(999, 4 * K), H=2,
               rounds=2, lr=0.01)
    print(f"update launch bf16 {widths} K={K} B={B}", flush=True)
    X, y, w0 = _small_data(w)
    _compare_steps(w, X, y, w0, 2e-3, LOSS_TOL_BF16, nr_ratio=NR_RATIO)


@pytest.mark.parametrize("widths", [(70, 48, 36, 10), (64, 128, 64, 10),
                                    (72, 20), (40, 33, 45),
                                    # 10 classes over 512 / 1536 bf16 inputs:
                                    # the head forward with W_L in LDS
                                    (48, 512, 10), (40, 64, 1536, 10)])
def test_small_mlp_bf16_every_step(widths):
    w = _small(widths, dtype="bf16")
    print(f"small bf16 {widths}", flush=True)
    X, y, w0 = _small_data(w)
    # bf16 operands: an operand rounded on the other side of a tie moves by
    # 2^-8 relative; the parameter bound is the loss bound of the workload,
    # and both must sit well inside the distance to an unrounded run
    _compare_steps(w, X, y, w0, 2e-3, LOSS_TOL_BF16, nr_ratio=NR_RATIO)


def test_softmax_regression_full_run():
    """Workload 1 (softmax regression, K=4, H=4, 50 rounds): every step."""
    w = wk.get("softmax_d64")
    X, y = wk.dataset(w)
    _compare_steps(w, X, y, wk.initial_weights(w), PARAM_TOL_FP32, LOSS_TOL_FP32)


def test_softmax_regression_single_launch_rounds():
    """Workload 1 through lsgd_run_round, which runs each round of softmax
    regression as one launch (replicas and buffers in LDS): all 50 rounds'
    averaged models and every step's losses against the oracle."""
    w = wk.get("softmax_d64")
    X, y = wk.dataset(w)
    reps = make_replicas(w, X, y)
    reps.profile(True)
    st = O.State(wk.initial_weights(w), w.K)
    loss = torch.empty(w.H, w.K, device=device())
    worst = 0.0
    for t in range(w.rounds):
        reps.run_round([w.lr] * w.H, loss)
        want = O.run_round(st, w, X, y, w.H, w.lr)
        assert np.all(rel(loss.cpu().numpy(), want) <= LOSS_TOL_FP32), t
        e = normwise(reps.read_params(0).cpu().numpy(), st.W[0])
        worst = max(worst, e)
        assert e <= PARAM_TOL_FP32, (t, e)
    print(f"softmax single-launch rounds: worst params {worst:.3e}", flush=True)
    assert set(reps.profile_report()) == {"tiny_round_wide"}


@pytest.mark.parametrize("K,B,D,C,nesterov,momentum,sampler", [
    (5, 70, 24, 7, False, 0.9, "iid"), (3, 20, 24, 7, True, 0.9, "epoch"),
    (8, 8, 24, 7, False, 0.0, "iid"), (1, 33, 24, 7, True, 0.5, "epoch"),
    (2, 200, 24, 7, False, 0.9, "iid"), (4, 30, 23, 7, True, 0.9, "epoch"),
    (3, 20, 32, 7, True, 0.9, "iid"), (4, 16, 40, 20, False, 0.9, "iid"),
    (6, 12, 40, 20, True, 0.9, "epoch")])
def test_single_launch_round_variants(K, B, D, C, nesterov, momentum, sampler):
    """The single-launch round on ragged shapes: more replicas than waves
    (idle waves in the last slot), batches beyond one wave of rows, up to four
    replicas with a 256-thread group each (next step's rows prefetched, or
    staged between steps for a large batch or an input width not a multiple
    of 4; input widths with and without padding to the 16-deep MFMA steps;
    classes padded to 8 and to 32), both samplers, heavy ball / Nesterov /
    plain SGD, step sizes changing inside a round; every round against the
    oracle, and against the step-by-step multi-kernel path within fp32
    rounding."""
    w = _small((D, C), K=K, B=B, N=600, H=3, rounds=4, momentum=momentum,
               nesterov=nesterov, lr=0.05).scaled(sampler=sampler)
    X, y, w0 = _small_data(w, seed=K + B)
    lrs = [0.05, 0.03, 0.04]
    a, b = make_replicas(w, X, y, w0), make_replicas(w, X, y, w0)
    a.profile(True)          # to see which path ran the rounds
    st = O.State(w0, w.K)
    loss = torch.empty(3, w.K, device=device())
    for t in range(4):
        a.run_round(lrs, loss)
        for lr in lrs:
            b.local_step(lr)
        b.average()
        want = O.run_round(st, w, X, y, 3, lrs)
        assert np.all(rel(loss.cpu().numpy(), want) <= LOSS_TOL_FP32), t
        got = a.read_params(0).cpu().numpy()
        assert normwise(got, st.W[0]) <= PARAM_TOL_FP32, t
        assert normwise(got, b.read_params(0).cpu().numpy()) <= 1e-6, t
        for k in range(w.K):
            assert normwise(a.read_momentum(k).cpu().numpy(), st.U[k]) <= PARAM_TOL_FP32
    assert a.step == b.step == 12
    # K <= 4: the 256-thread-per-replica kernel; more: wave per replica
    assert set(a.profile_report()) == {"tiny_round_wide" if K <= 4 else "tiny_round"}


def test_single_launch_round_longest():
    """The longest round one launch takes (H = 64: every step's rows sampled
    up front, the largest LDS request of the softmax shape) against the
    oracle and the step-by-step path; H = 65 takes the multi-kernel path."""
    w = _small((64, 10), K=4, B=32, N=2000, H=64, rounds=1, momentum=0.9,
               nesterov=True, lr=0.02)
    X, y, w0 = _small_data(w, seed=64)
    for H, single in ((64, True), (65, False)):
        a, b = make_replicas(w, X, y, w0), make_replicas(w, X, y, w0)
        a.profile(True)
        st = O.State(w0, w.K)
        loss = torch.empty(H, w.K, device=device())
        a.run_round([w.lr] * H, loss)
        for _ in range(H):
            b.local_step(w.lr)
        b.average()
        want = O.run_round(st, w, X, y, H, w.lr)
        assert np.all(rel(loss.cpu().numpy(), want) <= LOSS_TOL_FP32), H
        got = a.read_params(0).cpu().numpy()
        assert normwise(got, st.W[0]) <= PARAM_TOL_FP32, H
        assert normwise(got, b.read_params(0).cpu().numpy()) <= 1e-6, H
        tags = set(a.profile_report())
        assert (tags == {"tiny_round_wide"}) == single, (H, tags)


@pytest.mark.parametrize("K,C", [(4, 10), (6, 20)])
def test_single_launch_rounds_are_bitwise_deterministic(K, C):
    """Two fresh runs of five single-launch rounds (the 256-thread kernel at
    K = 4, the wave-per-replica kernel at K = 6): bit-identical parameters,
    momentum buffers and losses."""
    w = _small((64, C), K=K, B=32, N=2000, H=4, rounds=5, momentum=0.9, lr=0.05)
    X, y, w0 = _small_data(w, seed=11)
    outs = []
    for _ in range(2):
        reps = make_replicas(w, X, y, w0)
        reps.profile(True)
        loss = torch.empty(5 * 4, w.K, device=device())
        for r in range(5):
            reps.run_round([w.lr] * 4, loss[4 * r:4 * r + 4])
        assert set(reps.profile_report()) == {"tiny_round_wide" if K <= 4 else "tiny_round"}
        outs.append((reps.read_params(0).cpu().numpy(),
                     np.stack([reps.read_momentum(k).cpu().numpy() for k in range(w.K)]),
                     loss.cpu().numpy()))
    for a, b in zip(outs[0], outs[1]):
        np.testing.assert_array_equal(a, b)


def test_h1_local_sgd_equals_minibatch_sgd_on_gpu():
    """H = 1 local SGD is mini-batch SGD with batch K * B_loc (the paper's
    special case below eq. 2): the GPU run against the oracle's separately
    written mini-batch SGD."""
    w = _small((70, 48, 36, 10), nesterov=True, H=1, rounds=6)
    X, y, w0 = _small_data(w, seed=9)
    reps = make_replicas(w, X, y, w0)
    for _ in range(6):
        reps.run_round([w.lr])
    ref = O.minibatch_sgd(w, X, y, w0, steps=6, lr=w.lr)
    assert normwise(reps.read_params(0).cpu().numpy(), ref) <= PARAM_TOL_FP32


def test_runs_are_bitwise_deterministic():
    w = _small((70, 48, 36, 10), nesterov=True, H=4, rounds=2)
    X, y, w0 = _small_data(w, seed=3)
    outs = []
    for _ in range(2):
        reps = make_replicas(w, X, y, w0)
        loss = torch.empty(8, w.K, device=device())
        reps.run_round([w.lr] * 4, loss[:4])
        reps.run_round([w.lr] * 4, loss[4:])
        outs.append((reps.read_params(-1).cpu().numpy(), loss.cpu().numpy()))
    np.testing.assert_array_equal(outs[0][0], outs[1][0])
    np.testing.assert_array_equal(outs[0][1], outs[1][1])


def test_run_round_equals_steps_then_average():
    w = _small((70, 48, 36, 10), H=3, rounds=1)
    X, y, w0 = _small_data(w, seed=4)
    a = make_replicas(w, X, y, w0)
    b = make_replicas(w, X, y, w0)
    a.run_round([0.02, 0.01, 0.03])
    for lr in (0.02, 0.01, 0.03):
        b.local_step(lr)
    b.average()
    np.testing.assert_array_equal(a.read_params(-1).cpu().numpy(),
                                  b.read_params(-1).cpu().numpy())
    for k in range(w.K):
        np.testing.assert_array_equal(a.read_momentum(k).cpu().numpy(),
                                      b.read_momentum(k).cpu().numpy())
    assert a.step == b.step == 3


def test_single_worker_rounds_are_plain_sgd():
    """K = 1: the average of one replica is that replica (bit for bit), so a
    round is H steps of mini-batch SGD with momentum on the one worker; against
    the oracle, and against the same steps taken one by one."""
    w = _small((70, 48, 36, 10), K=1, B=20, H=3, rounds=2, nesterov=True)
    X, y, w0 = _small_data(w, seed=81)
    a, b = make_replicas(w, X, y, w0), make_replicas(w, X, y, w0)
    st = O.State(w0, 1)
    loss = torch.empty(3, 1, device=device())
    for t in range(2):
        a.run_round([0.02, 0.01, 0.03], loss)
        for lr in (0.02, 0.01, 0.03):
            b.local_step(lr)
        want = O.run_round(st, w, X, y, 3, [0.02, 0.01, 0.03])
        assert np.all(rel(loss.cpu().numpy(), want) <= LOSS_TOL_FP32), t
        np.testing.assert_array_equal(a.read_params(0).cpu().numpy(),
                                      b.read_params(0).cpu().numpy())
        assert normwise(a.read_params(0).cpu().numpy(), st.W[0]) <= PARAM_TOL_FP32


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
def test_smallest_batch(dtype):
    """B_loc = 4, the smallest batch the boundary accepts (one row group per
    sampler call): every step against the oracle."""
    w = _small((36, 24, 10), K=3, B=4, H=2, rounds=2, dtype=dtype)
    X, y, w0 = _small_data(w, seed=83)
    tol = PARAM_TOL_FP32 if dtype == "fp32" else 2e-3
    _compare_steps(w, X, y, w0, tol, LOSS_TOL_FP32 if dtype == "fp32" else LOSS_TOL_BF16,
                   nr_ratio=None if dtype == "fp32" else NR_RATIO)


def test_momentum_buffers_are_not_averaged():
    w = _small((70, 48, 36, 10), H=2, rounds=1)
    X, y, w0 = _small_data(w, seed=6)
    reps = make_replicas(w, X, y, w0)
    st = O.State(w0, w.K)
    O.run_round(st, w, X, y, 2, w.lr)
    reps.run_round([w.lr] * 2)
    for k in range(w.K):
        assert normwise(reps.read_momentum(k).cpu().numpy(), st.U[k]) <= PARAM_TOL_FP32
    u0 = reps.read_momentum(0).cpu().numpy()
    assert not np.allclose(u0, reps.read_momentum(1).cpu().numpy())


def test_write_params_and_step_counter_resume_exactly():
    """Checkpoint/resume: state restored into a fresh context continues
    bit-identically (the sampler is stateless given the step counter)."""
    w = _small((70, 48, 36, 10), momentum=0.0, H=2, rounds=1)
    X, y, w0 = _small_data(w, seed=8)
    a = make_replicas(w, X, y, w0)
    a.run_round([0.02, 0.02])
    mid = a.read_params(-1)
    b = make_replicas(w, X, y, w0)
    b.write_params(mid)
    b.step = a.step
    a.run_round([0.02, 0.02])
    b.run_round([0.02, 0.02])
    np.testing.assert_array_equal(a.read_params(-1).cpu().numpy(),
                                  b.read_params(-1).cpu().numpy())


# ----------------------------------------------------- hierarchical local SGD
@pytest.mark.parametrize("K,Kb,nesterov", [(8, 4, False), (6, 3, True),
                                           (8, 2, False)])
def test_hierarchical_round_matches_oracle_step_by_step(K, Kb, nesterov):
    """Appendix D / Algorithm 5 on both sides: every replica after every local
    step and after every block average, then the global average; and the
    fused round entry point against the oracle's whole round."""
    w = _small((70, 48, 36, 10), K=K, B=12, nesterov=nesterov, rounds=1)
    X, y, w0 = _small_data(w, seed=9 + K)
    H, Hb = 2, 3
    print(f"hierarchical K={K} Kb={Kb} H={H} Hb={Hb}", flush=True)
    reps = make_replicas(w, X, y, w0)
    st = O.State(w0, w.K)
    loss_d = torch.empty(w.K, device=device())
    for b in range(Hb):
        for h in range(H):
            reps.local_step(w.lr, loss_d)
            want = O.local_step(st, w, X, y, w.lr)
            assert np.all(rel(loss_d.cpu().numpy(), want) <= LOSS_TOL_FP32), (b, h)
            for k in range(w.K):
                e = normwise(reps.read_params(k).cpu().numpy(), st.W[k])
                assert e <= PARAM_TOL_FP32, (b, h, k, e)
        reps.average_blocks(Kb)
        st.W = O.average_blocks(st.W, Kb)
        got = [reps.read_params(k).cpu().numpy() for k in range(w.K)]
        for k in range(w.K):
            e = normwise(got[k], st.W[k])
            assert e <= PARAM_TOL_FP32, (b, "block", k, e)
            np.testing.assert_array_equal(got[k], got[k - k % Kb])
        assert not np.array_equal(got[0], got[Kb])
    reps.average()
    st.W = O.average(st.W)
    e = normwise(reps.read_params(-1).cpu().numpy(), st.W[0])
    assert e <= PARAM_TOL_FP32, ("global", e)

    # the fused entry point over a whole round
    a = make_replicas(w, X, y, w0)
    st = O.State(w0, w.K)
    loss = torch.empty(H * Hb, w.K, device=device())
    a.run_hierarchical_round(H, Hb, Kb, [w.lr] * (H * Hb), loss)
    want = O.run_hierarchical_round(st, w, X, y, H, Hb, Kb, w.lr)
    assert np.all(rel(loss.cpu().numpy(), want) <= LOSS_TOL_FP32)
    for k in (0, w.K - 1):
        e = normwise(a.read_params(k).cpu().numpy(), st.W[k])
        assert e <= PARAM_TOL_FP32, ("fused", k, e)
    for k in range(w.K):
        e = normwise(a.read_momentum(k).cpu().numpy(), st.U[k])
        assert e <= PARAM_TOL_FP32, ("momentum", k, e)
    assert a.step == H * Hb


def test_hierarchical_round_reduces_to_local_sgd_bit_for_bit():
    """The limits of Appendix D on the GPU, launch for launch: H^b = 1 is one
    local SGD round; K' = K is H^b rounds of period H; K' = 1 is one round
    of H * H^b steps; and the fused round equals its steps with the block
    averages in between and the global average at the end."""
    w = _small((70, 48, 36, 10), K=8, B=12, rounds=1)
    X, y, w0 = _small_data(w, seed=31)
    lrs = [0.02, 0.01, 0.03, 0.02, 0.015, 0.025]

    def final(r):
        return (r.read_params(-1).cpu().numpy(),
                np.stack([r.read_momentum(k).cpu().numpy() for k in range(w.K)]))

    def same(a, b):
        for x, z in zip(final(a), final(b)):
            np.testing.assert_array_equal(x, z)

    a, b = make_replicas(w, X, y, w0), make_replicas(w, X, y, w0)
    a.run_hierarchical_round(6, 1, 4, lrs)
    b.run_round(lrs)
    same(a, b)

    a, b = make_replicas(w, X, y, w0), make_replicas(w, X, y, w0)
    a.run_hierarchical_round(2, 3, w.K, lrs)
    for i in range(3):
        b.run_round(lrs[2 * i:2 * i + 2])
    same(a, b)

    a, b = make_replicas(w, X, y, w0), make_replicas(w, X, y, w0)
    a.run_hierarchical_round(3, 2, 1, lrs)
    b.run_round(lrs)
    same(a, b)

    a, b = make_replicas(w, X, y, w0), make_replicas(w, X, y, w0)
    a.run_hierarchical_round(2, 3, 2, lrs)
    for i in range(3):
        b.local_step(lrs[2 * i])
        b.local_step(lrs[2 * i + 1])
        if i < 2:
            b.average_blocks(2)
    b.average()
    same(a, b)


def test_hierarchical_round_rejects_bad_blocks():
    from paper_1808_07217_amd import lsgd as L
    w = _small((70, 48, 36, 10), K=6, B=12, rounds=1)
    X, y, w0 = _small_data(w, seed=3)
    reps = make_replicas(w, X, y, w0)
    for Kb in (0, 4, 7):
        with pytest.raises(L.LsgdError):
            reps.average_blocks(Kb)
        with pytest.raises(L.LsgdError):
            reps.run_hierarchical_round(1, 2, Kb, [0.01, 0.01])
    with pytest.raises(L.LsgdError):
        reps.run_hierarchical_round(1, 0, 3, [])
    assert reps.step == 0


# -------------------------------------------------- global / hybrid momentum
def _sync_error(reps, st, w):
    """Model-space errors after a synchronisation: the replicas' model, and
    the global buffer's step lr * u (the buffer itself is a model change
    divided by the step size, so its own relative error carries the model's
    cancellation; in model space it is held to the parameter bar)."""
    got = reps.read_params(0).cpu().numpy()
    e_w = normwise(got, st.W[0])
    du = np.abs(reps.read_global_momentum().cpu().numpy().astype(np.float64)
                - st.u_global)
    e_u = float(np.max(du) * w.lr / np.max(np.abs(st.W[0])))
    return e_w, e_u


@pytest.mark.parametrize("mg,momentum,nesterov", [(0.5, 0.0, False),
                                                  (0.3, 0.9, False),
                                                  (0.9, 0.9, True)])
def test_global_momentum_rounds_match_oracle(mg, momentum, nesterov):
    """Local SGD with global momentum (local momentum 0) and the hybrid
    scheme (local heavy ball or Nesterov plus the global buffer): every
    replica and the global buffer after each of four rounds, the losses of
    every step."""
    w = _small((70, 48, 36, 10), K=4, B=12, H=3, rounds=4, momentum=momentum,
               nesterov=nesterov).scaled(global_momentum=mg)
    X, y, w0 = _small_data(w, seed=50)
    print(f"global momentum mg={mg} local m={momentum} nesterov={nesterov}", flush=True)
    reps = make_replicas(w, X, y, w0)
    st = O.State(w0, w.K)
    loss = torch.empty(w.H, w.K, device=device())
    for t in range(w.rounds):
        reps.run_round([w.lr] * w.H, loss)
        want = O.run_round(st, w, X, y, w.H, w.lr)
        assert np.all(rel(loss.cpu().numpy(), want) <= LOSS_TOL_FP32), t
        e_w, e_u = _sync_error(reps, st, w)
        assert e_w <= PARAM_TOL_FP32, (t, e_w)
        assert e_u <= PARAM_TOL_FP32, (t, e_u)
        for k in range(1, w.K):
            np.testing.assert_array_equal(reps.read_params(k).cpu().numpy(),
                                          reps.read_params(0).cpu().numpy())


def test_global_momentum_h1_is_minibatch_heavy_ball_on_the_gpu():
    """H = 1, no local momentum: the GPU run equals the oracle's mini-batch
    SGD with heavy-ball momentum m_g on the union batch."""
    w = _small((70, 48, 36, 10), K=4, B=12, H=1, rounds=6,
               momentum=0.0).scaled(global_momentum=0.8)
    X, y, w0 = _small_data(w, seed=51)
    reps = make_replicas(w, X, y, w0)
    for _ in range(6):
        reps.run_round([w.lr])
    ref = O.minibatch_sgd(w.scaled(momentum=0.8), X, y, w0, steps=6, lr=w.lr)
    assert normwise(reps.read_params(-1).cpu().numpy(), ref) <= PARAM_TOL_FP32


def test_global_momentum_entry_points_and_resume():
    """lsgd_average is refused once a global factor is set (the
    synchronisation needs the step size), synchronise() equals the end of
    run_round bit for bit, and a context restored from the synchronised
    model, the global buffer and the step counter continues bit-identically
    (no local momentum, so the local buffers carry nothing over)."""
    from paper_1808_07217_amd import lsgd as L
    w = _small((70, 48, 36, 10), K=4, B=12, H=2, rounds=1,
               momentum=0.0).scaled(global_momentum=0.6)
    X, y, w0 = _small_data(w, seed=52)
    a = make_replicas(w, X, y, w0)
    with pytest.raises(L.LsgdError):
        a.average()
    with pytest.raises(L.LsgdError):
        a.run_round([])
    b = make_replicas(w, X, y, w0)
    a.run_round([0.02, 0.03])
    b.local_step(0.02)
    b.local_step(0.03)
    b.synchronise(0.03)
    np.testing.assert_array_equal(a.read_params(-1).cpu().numpy(),
                                  b.read_params(-1).cpu().numpy())
    np.testing.assert_array_equal(a.read_global_momentum().cpu().numpy(),
                                  b.read_global_momentum().cpu().numpy())
    a.run_round([0.02, 0.02])          # a second round so that u != 0 matters
    c = make_replicas(w, X, y, w0)
    c.write_params(a.read_params(0))
    c.write_global_momentum(a.read_global_momentum())
    c.step = a.step
    a.run_round([0.02, 0.02])
    c.run_round([0.02, 0.02])
    np.testing.assert_array_equal(a.read_params(-1).cpu().numpy(),
                                  c.read_params(-1).cpu().numpy())


# ------------------------------------- sign-compressed synchronisation
def _sign_sync_allowance(st_W, w_sync, E, amb_abs):
    """Per element, the largest change that sign decisions on near-zero
    differences can make: 2 p^k / K summed over the workers whose corrected
    difference there is within ``amb_abs`` of zero (either sign, or none,
    is a valid decision there)."""
    K = st_W.shape[0]
    d = w_sync[None] - st_W + (0 if E is None else E)
    p = np.abs(d).sum(axis=1) / d.shape[1]
    amb = np.abs(d) <= amb_abs
    return (2 * p[:, None] * amb).sum(axis=0) / K, amb


@pytest.mark.parametrize("scheme,H,nesterov", [("ef_sign", 3, False),
                                               ("ef_sign", 1, True),
                                               ("sign", 1, True),
                                               ("sign", 1, False)])
def test_sign_schemes_rounds_match_oracle(scheme, H, nesterov):
    """Algorithms 3 (sign local steps, H' = 1) and 4 (EF-signSGD) over four
    rounds: the synchronised model, the error memories (in model space,
    against max |w|) and every loss."""
    w = _small((70, 48, 36, 10), K=4, B=12, H=H, rounds=4,
               nesterov=nesterov).scaled(scheme=scheme)
    X, y, w0 = _small_data(w, seed=70)
    print(f"{scheme} H={H} nesterov={nesterov}", flush=True)
    reps = make_replicas(w, X, y, w0)
    st = O.State(w0, w.K)
    loss = torch.empty(H, w.K, device=device())
    for t in range(4):
        reps.run_round([w.lr] * H, loss)
        want = O.run_round(st, w, X, y, H, w.lr)
        assert np.all(rel(loss.cpu().numpy(), want) <= LOSS_TOL_FP32), t
        e = normwise(reps.read_params(0).cpu().numpy(), st.W[0])
        assert e <= PARAM_TOL_FP32, (t, e)
        if scheme == "ef_sign":
            scale = np.max(np.abs(st.W[0]))
            for k in range(w.K):
                de = np.max(np.abs(reps.read_error_memory(k).cpu().numpy() - st.E[k]))
                assert de <= PARAM_TOL_FP32 * scale, (t, k, de / scale)


def test_signsgd_round_with_cancelling_steps():
    """Algorithm 3 with H' = 4: coordinates whose four sign steps cancel have
    an exactly zero model difference in exact arithmetic, but w - lr + lr
    leaves a rounding residue (in fp32 on the GPU, in fp64 in the oracle)
    whose sign is noise on both sides. Elsewhere the synchronised model
    matches the oracle elementwise; at cancelled coordinates it stays within
    the change such noise can make."""
    w = _small((70, 48, 36, 10), K=4, B=12, H=4, rounds=1,
               nesterov=True).scaled(scheme="sign")
    X, y, w0 = _small_data(w, seed=71)
    reps = make_replicas(w, X, y, w0)
    st = O.State(w0, w.K)
    loss = torch.empty(4, w.K, device=device())
    reps.run_round([w.lr] * 4, loss)
    want = [O.local_step(st, w, X, y, w.lr) for _ in range(4)]
    assert np.all(rel(loss.cpu().numpy(), np.stack(want)) <= LOSS_TOL_FP32)
    allow, amb = _sign_sync_allowance(st.W, st.w_sync, None, 0.5 * w.lr)
    print(f"cancelled coordinates: {amb.mean():.3%}", flush=True)
    assert amb.any()
    O.synchronise(st, w, w.lr)
    got = reps.read_params(0).cpu().numpy()
    err = np.abs(got - st.W[0])
    tol = PARAM_TOL_FP32 * np.max(np.abs(st.W[0]))
    assert np.all(err <= tol + allow)
    assert np.max(err[allow == 0]) <= tol


def test_sign_scheme_entry_points_and_resume():
    """Sign schemes synchronise through lsgd_synchronise (lsgd_average is
    refused); EF-signSGD resumes bit-identically from the synchronised model
    and the memories (no local momentum, so the buffers carry nothing)."""
    from paper_1808_07217_amd import lsgd as L
    w = _small((70, 48, 36, 10), K=4, B=12, H=2, rounds=1,
               momentum=0.0).scaled(scheme="ef_sign")
    X, y, w0 = _small_data(w, seed=72)
    a = make_replicas(w, X, y, w0)
    with pytest.raises(L.LsgdError):
        a.average()
    a.run_round([0.02, 0.02])
    a.run_round([0.02, 0.02])
    c = make_replicas(w, X, y, w0)
    c.write_params(a.read_params(0))
    for k in range(w.K):
        c.write_error_memory(k, a.read_error_memory(k))
    c.step = a.step
    a.run_round([0.02, 0.02])
    c.run_round([0.02, 0.02])
    np.testing.assert_array_equal(a.read_params(-1).cpu().numpy(),
                                  c.read_params(-1).cpu().numpy())
    for k in range(w.K):
        np.testing.assert_array_equal(a.read_error_memory(k).cpu().numpy(),
                                      c.read_error_memory(k).cpu().numpy())


@pytest.mark.parametrize("variant", ["hybrid", "ef_sign", "hier"])
def test_bf16_operands_with_the_newer_schemes(variant):
    """bf16 GEMM operands (fp32 masters) under hybrid momentum, EF-signSGD and
    hierarchical averaging: the bf16 operand copies are refreshed by every
    synchronisation kind, so the next round's GEMMs see the synchronised
    model -- two rounds against the oracle's bf16 emulation (one for
    EF-signSGD, see below)."""
    w = _small((64, 96, 64, 10), dtype="bf16", K=4, B=16, H=3, rounds=2)
    if variant == "hybrid":
        w = w.scaled(global_momentum=0.4)
    elif variant == "ef_sign":
        w = w.scaled(scheme="ef_sign")
    X, y, w0 = _small_data(w, seed=95)
    reps = make_replicas(w, X, y, w0)
    st = O.State(w0, w.K)
    loss = torch.empty(6, w.K, device=device())
    if variant == "ef_sign":
        # one round: the replicas after the local steps are held below half
        # of the no-rounding oracle's distance (as everywhere with bf16
        # operands). They then lie within rep * scale of the oracle's, so a
        # corrected difference further than twice that (plus fp32 rounding)
        # from zero has the oracle's sign; closer ones may take either sign,
        # and those elements are allowed the change a flipped sign makes.
        # Elsewhere the scale p^k moves by at most the replica distance. (A
        # second round would start from legitimately different memories.)
        nr, w_nr = O.State(w0, w.K), w.scaled(dtype="fp32")
        for h in range(3):
            reps.local_step(w.lr, loss[h])
            want = O.local_step(st, w, X, y, w.lr)
            O.local_step(nr, w_nr, X, y, w.lr)
            assert np.all(rel(loss.cpu().numpy()[h], want) <= LOSS_TOL_BF16)
        scale = np.max(np.abs(st.W))
        rep = max(normwise(reps.read_params(k).cpu().numpy(), st.W[k]) for k in range(w.K))
        d_nr = max(normwise(nr.W[k], st.W[k]) for k in range(w.K))
        assert rep <= NR_RATIO * d_nr, (rep, d_nr)
        bound = (2 * rep + 1e-6) * scale
        allow, amb = _sign_sync_allowance(st.W, st.w_sync, st.E, bound)
        reps.synchronise(w.lr)
        O.synchronise(st, w, w.lr)
        err = np.abs(reps.read_params(0).cpu().numpy() - st.W[0])
        print(f"bf16 ef_sign: replicas {rep:.3e} (oracle without rounding {d_nr:.3e}); "
              f"undetermined {amb.mean():.2%}", flush=True)
        assert np.all(err <= bound + allow)
        assert np.max(err[allow == 0]) <= bound
        return
    nr, w_nr = O.State(w0, w.K), w.scaled(dtype="fp32")   # no bf16 rounding
    worst = d_nr = 0.0
    for t in range(2):
        if variant == "hier":
            reps.run_hierarchical_round(3, 2, 2, [w.lr] * 6, loss)
            want = O.run_hierarchical_round(st, w, X, y, 3, 2, 2, w.lr)
            O.run_hierarchical_round(nr, w_nr, X, y, 3, 2, 2, w.lr)
        else:
            reps.run_round([w.lr] * 3, loss[:3])
            want = O.run_round(st, w, X, y, 3, w.lr)
            O.run_round(nr, w_nr, X, y, 3, w.lr)
        got_loss = loss.cpu().numpy()[:len(want)]
        assert np.all(rel(got_loss, want) <= LOSS_TOL_BF16), t
        e = normwise(reps.read_params(0).cpu().numpy(), st.W[0])
        assert e <= 2e-3, t
        worst, d_nr = max(worst, e), max(d_nr, normwise(nr.W[0], st.W[0]))
    print(f"bf16 {variant}: GPU {worst:.3e}, oracle without rounding {d_nr:.3e}", flush=True)
    assert worst <= NR_RATIO * d_nr


def test_full_state_checkpoint_resumes_bit_exactly():
    """Checkpoint and resume with every piece of state: the synchronised
    model, each replica's momentum buffer (Nesterov, heavy-ball buffers
    carry over rounds), and the step counter. A fresh context restored from
    them continues bit-identically, replicas and buffers alike."""
    w = _small((70, 48, 36, 10), K=4, B=12, H=3, rounds=1, nesterov=True)
    X, y, w0 = _small_data(w, seed=90)
    a = make_replicas(w, X, y, w0)
    a.run_round([0.02] * 3)
    a.run_round([0.01] * 3)
    c = make_replicas(w, X, y, w0)
    c.write_params(a.read_params(0))
    for k in range(w.K):
        c.write_momentum(k, a.read_momentum(k))
    c.step = a.step
    for r in (a, c):
        r.run_round([0.015, 0.02, 0.01])
    for k in range(w.K):
        np.testing.assert_array_equal(a.read_params(k).cpu().numpy(),
                                      c.read_params(k).cpu().numpy())
        np.testing.assert_array_equal(a.read_momentum(k).cpu().numpy(),
                                      c.read_momentum(k).cpu().numpy())


# ------------------------------------------------ training-procedure schedules
@pytest.mark.parametrize("post_local,kind", [(False, "exponential"), (True, None)])
def test_cifar_plan_with_the_epoch_sampler_matches_oracle(post_local, kind):
    """The CIFAR procedure on a small MLP: the per-epoch reshuffled
    partition, linear scaling with a gradual warm-up, the 50% / 75% decay,
    and rounds from post-local SGD's switch or an exponential local-step
    warm-up (rounds of 1, 2, 4, then 8 steps). Step sizes vary inside
    rounds. Every round's synchronised model and every loss against the
    oracle driven by its own schedule functions."""
    from paper_1808_07217_amd import schedules as S
    w = _small((70, 48, 36, 10), K=4, B=8, N=400, H=8, rounds=1,
               lr=0.01).scaled(sampler="epoch")
    X, y, w0 = _small_data(w, seed=80)
    K, B, N, epochs = w.K, w.B_loc, w.N, 6
    plan = S.cifar_plan(K=K, B=B, N=N, epochs=epochs, base_lr=w.lr, H=8, ref_batch=16,
                        lr_warmup_epochs=1, post_local=post_local, warmup=kind,
                        warmup_epochs=3)
    spe = O.steps_per_epoch(K, N, B)
    total = epochs * spe

    def f(s):
        return (O.goyal_lr(s, w.lr, K * B / 16, spe) *
                O.decay_factor(s, K * B, total * K * B))
    switch = (next(s for s in range(total) if O.decay_factor(s, K * B, total * K * B) < 1)
              if post_local else None)
    oracle_plan = O.schedule_rounds(total, spe, 8, f, h_kind=kind, h_warmup_epochs=3,
                                    switch_step=switch)
    assert [h for h, _ in plan] == [h for h, _ in oracle_plan]
    print(f"plan: {len(plan)} rounds, H {sorted(set(h for h, _ in plan))}", flush=True)
    reps = make_replicas(w, X, y, w0)
    st = O.State(w0, w.K)
    for t, ((h, lrs), (_, lrs_o)) in enumerate(zip(plan, oracle_plan)):
        loss = torch.empty(h, w.K, device=device())
        reps.run_round(lrs, loss)
        want = O.run_round(st, w, X, y, h, lrs_o)
        assert np.all(rel(loss.cpu().numpy(), want) <= LOSS_TOL_FP32), t
        e = normwise(reps.read_params(0).cpu().numpy(), st.W[0])
        assert e <= PARAM_TOL_FP32, (t, e)
    assert reps.step == total


# --------------------------------------------------------- full-size rounds
@pytest.fixture(scope="module")
def img_data():
    w = wk.get("mlp_512")
    return wk.dataset(w)


def test_mlp_512_first_round_full_size(img_data):
    """Workload 2 at its real shape (K=16, B_loc=128, H=16) against the oracle:
    every replica after the first local step, the losses of all 16 steps, and
    the averaged model after the round (the 1e-5 bar on parameters after one
    round). Before averaging, fp32 rounding differences are amplified by the
    training dynamics over the H steps (a plain fp32 CPU implementation of the
    same round already differs from fp64 by 6e-6 on one replica); each
    replica is held to 5e-5 there."""
    w = wk.get("mlp_512")
    X, y = img_data
    w0 = wk.initial_weights(w)
    print("mlp_512 round 1", flush=True)
    reps = make_replicas(w, X, y, w0)
    st = O.State(w0, w.K)
    loss = torch.empty(w.H, w.K, device=device())
    ref_loss = []
    for h in range(w.H):
        reps.local_step(w.lr, loss[h])
        ref_loss.append(O.local_step(st, w, X, y, w.lr))
        if h == 0:
            for k in range(w.K):
                e = normwise(reps.read_params(k).cpu().numpy(), st.W[k])
                assert e <= PARAM_TOL_FP32, ("after step 1", k, e)
    assert np.all(rel(loss.cpu().numpy(), np.stack(ref_loss)) <= LOSS_TOL_FP32)
    errs = [normwise(reps.read_params(k).cpu().numpy(), st.W[k]) for k in range(w.K)]
    print(f"mlp_512 per-replica errors before averaging: max {max(errs):.3e}",
          flush=True)
    assert max(errs) <= 5e-5, errs
    reps.average()
    st.W = O.average(st.W)
    e = normwise(reps.read_params(-1).cpu().numpy(), st.W[0])
    print(f"mlp_512 round-1 averaged params normwise error {e:.3e}", flush=True)
    assert e <= PARAM_TOL_FP32


def test_mlp_512_hierarchical_round_full_size(img_data):
    """Workload 2's shape (K=16, B_loc=128) as hierarchical local SGD with
    blocks of K'=4 replicas, H=4, H^b=2: the losses of all eight steps and
    the averaged model after the outer round against the oracle."""
    w = wk.get("mlp_512")
    X, y = img_data
    w0 = wk.initial_weights(w)
    H, Hb, Kb = 4, 2, 4
    print("mlp_512 hierarchical round", flush=True)
    reps = make_replicas(w, X, y, w0)
    st = O.State(w0, w.K)
    loss = torch.empty(H * Hb, w.K, device=device())
    reps.run_hierarchical_round(H, Hb, Kb, [w.lr] * (H * Hb), loss)
    want = O.run_hierarchical_round(st, w, X, y, H, Hb, Kb, w.lr)
    assert np.all(rel(loss.cpu().numpy(), want) <= LOSS_TOL_FP32)
    e = normwise(reps.read_params(-1).cpu().numpy(), st.W[0])
    print(f"mlp_512 hierarchical round params normwise error {e:.3e}", flush=True)
    assert e <= PARAM_TOL_FP32


def test_mlp_512_hybrid_momentum_two_rounds_full_size(img_data):
    """Workload 2's shape with hybrid momentum (local heavy ball 0.9, global
    0.3): two rounds of 16 steps, so the global buffer acts in the second."""
    w = wk.get("mlp_512").scaled(global_momentum=0.3)
    X, y = img_data
    w0 = wk.initial_weights(w)
    print("mlp_512 hybrid momentum, two rounds", flush=True)
    reps = make_replicas(w, X, y, w0)
    st = O.State(w0, w.K)
    loss = torch.empty(w.H, w.K, device=device())
    for t in range(2):
        reps.run_round([w.lr] * w.H, loss)
        want = O.run_round(st, w, X, y, w.H, w.lr)
        assert np.all(rel(loss.cpu().numpy(), want) <= LOSS_TOL_FP32), t
        e_w, e_u = _sync_error(reps, st, w)
        print(f"round {t + 1}: params {e_w:.3e}, lr * u {e_u:.3e}", flush=True)
        assert e_w <= PARAM_TOL_FP32 and e_u <= PARAM_TOL_FP32, (t, e_w, e_u)


def test_mlp_512_ef_signsgd_first_round_full_size(img_data):
    """Workload 2's shape under Algorithm 4, one round of 16 plain local
    steps. Before the synchronisation the replicas carry fp32 rounding
    amplified over 16 steps (held to 5e-5 of max |w| per replica in the
    plain run); where a worker's difference is that close to zero its sign
    is not determined, and the synchronised model may differ there by the
    change such signs can make. Elsewhere it matches the oracle
    elementwise."""
    w = wk.get("mlp_512").scaled(scheme="ef_sign")
    X, y = img_data
    w0 = wk.initial_weights(w)
    print("mlp_512 ef_sign round 1", flush=True)
    reps = make_replicas(w, X, y, w0)
    st = O.State(w0, w.K)
    loss = torch.empty(w.H, w.K, device=device())
    reps.run_round([w.lr] * w.H, loss)
    want = [O.local_step(st, w, X, y, w.lr) for _ in range(w.H)]
    assert np.all(rel(loss.cpu().numpy(), np.stack(want)) <= LOSS_TOL_FP32)
    near = 5e-5 * np.max(np.abs(st.W), axis=1, keepdims=True)
    allow, amb = _sign_sync_allowance(st.W, st.w_sync, None, near)
    O.synchronise(st, w, w.lr)
    got = reps.read_params(0).cpu().numpy()
    err = np.abs(got - st.W[0])
    tol = PARAM_TOL_FP32 * np.max(np.abs(st.W[0]))
    print(f"undetermined signs: {amb.mean():.3%}; max error off them "
          f"{np.max(err[allow == 0]) / np.max(np.abs(st.W[0])):.3e}", flush=True)
    assert np.all(err <= tol + allow)
    assert np.max(err[allow == 0]) <= tol


def test_mlp_512_signsgd_first_round_full_size(img_data):
    """Workload 2's shape under Algorithm 3 at H' = 1 (one sign step per
    worker, then the compressed synchronisation). The first step's
    direction is the gradient plus decay at w0 on both sides; where it is
    within 1e-5 of the largest direction entry of its replica, fp32 and fp64
    may take different signs (the GEMM's rounding is of that order), and the
    synchronised model may differ there by 2 p / K per such worker.
    Elsewhere it matches the oracle elementwise. (Over many sign steps such
    decisions compound, so longer runs are compared on small cases.)"""
    w = wk.get("mlp_512").scaled(scheme="sign", H=1)
    X, y = img_data
    w0 = wk.initial_weights(w)
    print("mlp_512 sign H'=1 round 1", flush=True)
    reps = make_replicas(w, X, y, w0)
    loss = torch.empty(1, w.K, device=device())
    reps.run_round([w.lr], loss)
    st = O.State(w0, w.K)
    want = O.local_step(st, w, X, y, w.lr)
    assert np.all(rel(loss.cpu().numpy()[0], want) <= LOSS_TOL_FP32)
    # the oracle's first directions d^k = grad + wd * w0 (u starts at 0)
    amb = np.zeros((w.K, st.W.shape[1]), bool)
    for k in range(w.K):
        idx = O.sample_indices(w.sample_seed, 0, k, w.K, w.N, w.B_loc)
        _, g = O.model_loss_and_grad(w, w0.astype(np.float64),
                                     np.asarray(X[idx], np.float64), y[idx])
        d = g + w.weight_decay * w0
        amb[k] = np.abs(d) <= 1e-5 * np.max(np.abs(d))
    p = np.abs(st.w_sync[None] - st.W).sum(axis=1) / st.W.shape[1]
    allow = (2 * p[:, None] * amb).sum(axis=0) / w.K
    O.synchronise(st, w, w.lr)
    got = reps.read_params(0).cpu().numpy()
    err = np.abs(got - st.W[0])
    tol = PARAM_TOL_FP32 * np.max(np.abs(st.W[0]))
    print(f"undetermined directions: {amb.mean():.4%}", flush=True)
    assert np.all(err <= tol + allow)
    assert np.max(err[allow == 0]) <= tol


def test_wide_bf16_first_round_two_replicas_full_size(img_data):
    """Workload 4 at its real shape (K=64, B_loc=64, H=8, bf16 operands):
    replicas 0 and 63 through the first round's local steps, then the
    synchronised model of all 64 replicas."""
    w = wk.get("wide_mlp_2048_bf16")
    X, y = img_data
    w0 = wk.initial_weights(w)
    print("wide bf16 round 1", flush=True)
    reps = make_replicas(w, X, y, w0)
    loss = torch.empty(w.H, w.K, device=device())
    for h in range(w.H):
        reps.local_step(w.lr, loss[h])
    st = O.State(w0, w.K)
    ref = np.stack([O.local_step(st, w, X, y, w.lr, replicas=[0, w.K - 1])
                    for _ in range(w.H)])
    got = loss.cpu().numpy()
    for k in (0, w.K - 1):
        assert np.all(rel(got[:, k], ref[:, k]) <= LOSS_TOL_BF16)
        e = normwise(reps.read_params(k).cpu().numpy(), st.W[k])
        print(f"wide bf16 replica {k} params normwise error {e:.3e}", flush=True)
        assert e <= 2e-3
    # the synchronised model (eq. 2) against the oracle's, at the seeded
    # sample positions tests/golden/make_round_models.py stored (oracle
    # only), with a bar below the distance of the oracle's run without any
    # bf16 rounding (same file): a path that skipped the roundings would fail
    import json
    import os
    here = os.path.join(os.path.dirname(os.path.abspath(__file__)), "golden")
    with open(os.path.join(here, "round1_wide_mlp_2048_bf16.json")) as f:
        gold = json.load(f)
    z = np.load(os.path.join(here, "round1_wide_mlp_2048_bf16.npz"))
    reps.average()
    wbar = reps.read_params(-1).cpu().numpy()
    err = float(np.max(np.abs(wbar[z["positions"]] - z["values"])) / gold["max_abs_model"])
    bar = NR_RATIO * gold["no_rounding_sampled_normwise"]
    lerr = float(np.max(rel(got.mean(axis=1), np.asarray(gold["round1_step_mean_loss"]))))
    lbar = NR_RATIO * gold["no_rounding_step_loss_rel"]
    print(f"wide bf16 averaged model {err:.3e} (bar {bar:.3e}; oracle without rounding "
          f"{gold['no_rounding_sampled_normwise']:.3e}), step losses {lerr:.3e} "
          f"(bar {lbar:.3e})", flush=True)
    assert err <= bar
    assert lerr <= lbar
