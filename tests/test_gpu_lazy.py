"""The lazy form of the plain average (lsgd_set_lazy_average): the mean is
written once and the next local step reads it for every replica. It must
give bit for bit the results of the default form, which writes the mean back
into every replica, whatever is called in between."""
import numpy as np
import pytest
import torch

import workloads as wk
from gpu_util import make_replicas, device

pytestmark = pytest.mark.gpu


def _small(widths, dtype="fp32", K=4, B=16, N=999, nesterov=False):
    return wk.Workload(name="small", model="mlp", widths=widths, dtype=dtype, K=K,
                       B_loc=B, H=3, rounds=3, lr=0.02, momentum=0.9,
                       nesterov=nesterov, weight_decay=1e-3, data="custom", N=N,
                       sample_seed=0x1A2B + K + B)


def _data(w, seed=3):
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


def _same(a, b, w):
    for k in range(w.K):
        np.testing.assert_array_equal(a.read_params(k).cpu().numpy(),
                                      b.read_params(k).cpu().numpy())
        np.testing.assert_array_equal(a.read_momentum(k).cpu().numpy(),
                                      b.read_momentum(k).cpu().numpy())


CASES = [
    ((70, 48, 36, 10), "fp32", 4, 16, False),     # fused head
    ((64, 128, 64, 10), "bf16", 4, 16, True),     # bf16 operand copies of the mean
    ((40, 33, 45), "fp32", 3, 20, True),          # > 32 classes: generic top layer
    ((256, 2048, 10), "fp32", 32, 21, False),     # thousands of update tiles
    ((512, 1024, 512, 10), "bf16", 16, 64, False),
]


@pytest.mark.parametrize("widths,dtype,K,B,nesterov", CASES)
def test_lazy_average_is_bit_identical(widths, dtype, K, B, nesterov):
    """Rounds through run_round, single local steps, lsgd_average, a block
    average, a one-replica write and the state blob: the lazy context and the
    default one agree bit for bit on losses, replicas, buffers and blobs."""
    w = _small(widths, dtype, K=K, B=B, N=max(999, 4 * K), nesterov=nesterov)
    X, y, w0 = _data(w)
    print(f"lazy average {widths} {dtype} K={K}", flush=True)
    a, b = make_replicas(w, X, y, w0), make_replicas(w, X, y, w0)
    b.set_lazy_average(True)
    la = torch.empty(3, w.K, device=device())
    lb = torch.empty(3, w.K, device=device())
    for t in range(3):
        lrs = [0.02, 0.01 * (t + 1), 0.015]
        a.run_round(lrs, la)
        b.run_round(lrs, lb)
        np.testing.assert_array_equal(la.cpu().numpy(), lb.cpu().numpy())
    # read while the mean is pending: every replica is the mean
    np.testing.assert_array_equal(a.read_params(-1).cpu().numpy(),
                                  b.read_params(-1).cpu().numpy())
    np.testing.assert_array_equal(a.read_params(w.K - 1).cpu().numpy(),
                                  b.read_params(1).cpu().numpy())
    for r in (a, b):
        r.local_step(0.02)
        r.average()
        r.local_step(0.01)
        r.average_blocks(2 if w.K % 2 == 0 else 1)
        r.run_round([0.01, 0.02])
    _same(a, b, w)
    # one replica overwritten while the mean is pending
    p = a.read_params(0) * 1.01
    for r in (a, b):
        r.write_params(p, replica=1)
        r.run_round([0.01])
    _same(a, b, w)
    sa, sb = a.read_state(), b.read_state()
    torch.cuda.synchronize()
    assert torch.equal(sa, sb)
    for r in (a, b):
        r.run_round([0.02, 0.02])
    b.set_lazy_average(False)            # writes the pending mean out
    _same(a, b, w)


@pytest.mark.parametrize("widths,dtype,K,B", [
    ((1024, 1024, 10), "fp32", 32, 32),    # 270 MB of state in whole tiles
    ((1000, 1040, 10), "fp32", 32, 8),     # and in ragged ones
    ((1024, 960, 10), "bf16", 32, 64),     # 317 MB with the bf16 copy
])
def test_lazy_average_of_a_state_streamed_past_the_caches(widths, dtype, K, B):
    """The update reads the shared mean through the caches and streams the rest:
    bit for bit the default form."""
    w = _small(widths, dtype, K=K, B=B, N=4 * K, nesterov=True)
    X, y, w0 = _data(w)
    print(f"lazy average, streamed state {widths} {dtype} K={K}", flush=True)
    a, b = make_replicas(w, X, y, w0), make_replicas(w, X, y, w0)
    b.set_lazy_average(True)
    for r in (a, b):
        r.run_round([0.02, 0.01])
        r.run_round([0.01])
    assert torch.equal(a.read_state(), b.read_state())


def test_lazy_average_with_the_single_launch_round():
    """Softmax regression: rounds run as one launch (which averages by
    itself), mixed with lazily averaged step-by-step rounds."""
    w = _small((64, 10), K=4, B=32, N=2000)
    X, y, w0 = _data(w, seed=9)
    a, b = make_replicas(w, X, y, w0), make_replicas(w, X, y, w0)
    b.set_lazy_average(True)
    for r in (a, b):
        r.local_step(0.02)
        r.average()
        r.run_round([0.02] * 3)      # one launch; the pending mean goes first
        r.local_step(0.01)
        r.average()
    _same(a, b, w)


@pytest.mark.parametrize("kind", ["resnet20", "ef_sign", "global_momentum"])
def test_lazy_average_refused_where_it_does_not_apply(kind):
    from paper_1808_07217_amd import lsgd as L
    if kind == "resnet20":
        base = wk.get("resnet20")
        w = base.scaled(K=2, N=4096, H=2)
        X, y = wk.dataset(base)
        X, y = np.ascontiguousarray(X[:4096]), np.ascontiguousarray(y[:4096])
        reps = make_replicas(w, X, y)
    else:
        w = _small((70, 48, 10))
        w = w.scaled(scheme="ef_sign") if kind == "ef_sign" else w.scaled(global_momentum=0.3)
        X, y, w0 = _data(w)
        reps = make_replicas(w, X, y, w0)
    with pytest.raises(L.LsgdError, match="unsupported"):
        reps.set_lazy_average(True)
