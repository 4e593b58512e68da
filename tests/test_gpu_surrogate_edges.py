"""The network's training and normalisation kernels at the sizes and
alignments where they can go wrong: one row, a ragged last 16-sample tile, one
workgroup and the most a launch takes, more tiles than waves, and arrays that
start 4 bytes off a 16-byte boundary (the scalar loads).

Bars: the BF16 gradient against the FP64 oracle as in test_gpu_surrogate.py
(3e-2 normwise: BF16 operands); the scalar and the vector loads of the same
rows bit for bit; means and standard deviations, FP64 sums rounded once to
FP32, within 2^-22 of numpy's; a training step against the same step computed
by Adam from the gradient that the library returns (1e-5 of the step's size
lr: FP32 sums of the same terms in the same order)."""
import numpy as np
import pytest

from oracle import surrogate as om
from paper_2111_00699_amd import scenes

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_cuda():
    import torch

    if not torch.cuda.is_available():
        pytest.fail("a GPU test ran without a visible GPU")
    return torch


def rows(count, seed):
    X = scenes.uniform(seed, 12 * count, 3, -2.0, 2.0).reshape(count, 12)
    T = scenes.uniform(seed, 12 * count, 4, -2.0, 2.0).reshape(count, 12)
    return X.astype(np.float32), T.astype(np.float32)


def shifted(torch, a):
    """The same values in device memory 4 bytes past a 16-byte boundary."""
    buf = torch.empty(a.size + 1, dtype=torch.float32, device="cuda")
    view = buf[1:].view(a.shape)
    view.copy_(torch.from_numpy(a))
    assert view.data_ptr() % 16 == 4
    return view


SIZES = [1, 15, 16, 63, 64, 65, 1000, 16384, 16385, 40003]


@pytest.mark.parametrize("count", SIZES)
def test_bf16_gradient_edges(torch_cuda, count):
    from paper_2111_00699_amd import mpm

    X, T = rows(count, 60)
    sur = mpm.Surrogate()
    theta = scenes.mlp_init(4)
    norm = np.concatenate([np.full(12, 0.1), np.full(12, 1.5), np.full(12, -0.1), np.full(12, 2.0)]).astype(np.float32)
    sur.set(theta, norm)
    loss, g = sur.loss_grad(X, T, precision=mpm.SUR_BF16)
    loss2, g2 = sur.loss_grad(shifted(torch_cuda, X), shifted(torch_cuda, T), precision=mpm.SUR_BF16)
    assert loss == loss2 and torch_cuda.equal(g, g2)
    mu, sd = norm[:12].astype(np.float64), norm[12:24].astype(np.float64)
    tmu, tsd = norm[24:36].astype(np.float64), norm[36:].astype(np.float64)
    Xn, Tn = (X - mu) / sd, (T - tmu) / tsd
    want, gref = om.loss(theta.astype(np.float64), Xn, Tn), om.grad(theta.astype(np.float64), Xn, Tn)
    g = g.cpu().numpy().astype(np.float64)
    assert abs(loss - want) <= 3e-2 * abs(want)
    assert np.abs(g - gref).max() <= 3e-2 * np.abs(gref).max()


@pytest.mark.parametrize("count", SIZES + [131072 * 16 + 5])
def test_bf16_forward_edges(torch_cuda, count):
    """BF16 forward pass at ragged sizes, up to more tiles than a launch has
    waves: each row alone gives what it gives among others, and 4 bytes off
    alignment, bit for bit; against the FP64 oracle within 1e-2 normwise."""
    from paper_2111_00699_amd import mpm

    X, _ = rows(count, 62)
    sur = mpm.Surrogate()
    theta = scenes.mlp_init(6)
    sur.set(theta)
    Y = sur.forward(X)
    off = sur.forward(shifted(torch_cuda, X))
    assert torch_cuda.equal(Y, off)
    some = np.unique(np.concatenate([np.arange(min(count, 40)), np.arange(max(0, count - 40), count)]))
    assert torch_cuda.equal(sur.forward(X[some]), Y[torch_cuda.from_numpy(some).cuda()])
    want = om.forward(theta.astype(np.float64), X[some])[0]
    assert np.abs(Y.cpu().numpy()[some] - want).max() <= 1e-2 * np.abs(want).max()


@pytest.mark.parametrize("batch", [16, 65, 4096, 16384, 20000])
def test_training_step_is_adam_on_the_drawn_rows(torch_cuda, batch):
    from paper_2111_00699_amd import mpm

    count, seed, lr = 5003, 12345, 1e-3
    X, T = rows(count, 61)
    sur = mpm.Surrogate()
    theta = scenes.mlp_init(5)
    sur.set(theta)
    with np.errstate(over="ignore"):
        z = np.uint64(seed) + np.arange(batch, dtype=np.uint64) * scenes.GOLDEN + scenes.GOLDEN
        z = (z ^ (z >> np.uint64(30))) * np.uint64(0xBF58476D1CE4E5B9)
        z = (z ^ (z >> np.uint64(27))) * np.uint64(0x94D049BB133111EB)
        z ^= z >> np.uint64(31)
    drawn = (z % np.uint64(count)).astype(np.int64)
    loss, g = sur.loss_grad(X[drawn], T[drawn], precision=mpm.SUR_BF16)
    losses = sur.train(X, T, steps=1, batch=batch, lr=lr, seed=seed)
    got = sur.get()[0].cpu().numpy().astype(np.float64)
    assert losses[0] == np.float32(loss)
    g = g.cpu().numpy().astype(np.float64)
    # the first step: m-hat = g, v-hat = g^2
    want = theta.astype(np.float64) - lr * g / (np.abs(g) + 1e-8)
    assert np.abs(got - want).max() <= 1e-5 * lr + 2.0 ** -23 * np.abs(theta).max()


@pytest.mark.parametrize("count", [1, 2, 255, 256, 257, 100003, 1200001])
def test_normalisation_edges(torch_cuda, count):
    from paper_2111_00699_amd import mpm

    X = (scenes.uniform(70, 12 * count, 0, -1.0, 3.0).reshape(count, 12) * np.arange(1, 13)).astype(np.float32)
    T = (scenes.uniform(71, 12 * count, 0, -5.0, 1.0).reshape(count, 12) + np.arange(12)).astype(np.float32)
    X[:, 11] = 1.0  # a constant column: its spread is the floor
    sur = mpm.Surrogate()
    sur.fit_norm(X, T)
    got = sur.get()[1].cpu().numpy()
    sur.fit_norm(shifted(torch_cuda, X), shifted(torch_cuda, T))
    off = sur.get()[1].cpu().numpy()
    want = []
    for A in (X.astype(np.float64), T.astype(np.float64)):
        want += [A.mean(0), np.maximum(A.std(0), 1e-6)]
    want = np.concatenate(want)
    # FP64 sums: E[x^2] - E[x]^2 leaves 2^-50 of E[x^2] in the variance
    tol = 2.0 ** -22 * np.abs(want) + 2.0 ** -24
    for a in (got, off):
        assert np.all(np.abs(a - want) <= tol)


@pytest.mark.parametrize("count", [4097, 16384, 16385])
def test_normalisation_in_one_launch_and_in_two(torch_cuda, count):
    """Up to 16,384 rows the columns are summed by the launch that stores the means."""
    test_normalisation_edges(torch_cuda, count)


def test_threads_share_a_surrogate(torch_cuda):
    """Gradients asked for by several threads at once from one network: each gets its own rows' (the calls
    enqueue on one stream, so nothing but their results can mix), bit for bit as when asked for alone."""
    import ctypes as ct
    import threading

    from paper_2111_00699_amd import mpm

    torch = torch_cuda
    threads, calls, count = 4, 500, 64
    sur = mpm.Surrogate()
    sur.set(scenes.mlp_init(4), np.concatenate([np.zeros(12), np.ones(12)] * 2).astype(np.float32))
    data = [[torch.from_numpy(a).cuda() for a in rows(count, 90 + k)] for k in range(threads)]
    alone = [sur.loss_grad(X, T, precision=mpm.SUR_BF16) for X, T in data]
    grad = torch.empty((threads, calls, mpm.SUR_PARAMS), dtype=torch.float32, device="cuda")
    loss = torch.empty((threads, calls), dtype=torch.float32, device="cuda")
    torch.cuda.synchronize()
    ptr = lambda t: ct.c_void_p(t.data_ptr())
    bad = []

    def work(k):
        X, T = data[k]
        args = [(sur.h, mpm.SUR_BF16, count, ptr(X), ptr(T), ptr(grad[k, i]), ptr(loss[k, i:])) for i in range(calls)]
        start.wait()
        for a in args:
            if sur.lib.mpm_surrogate_loss_grad(*a) != mpm.OK:
                bad.append(k)

    start = threading.Barrier(threads)
    pool = [threading.Thread(target=work, args=(k,)) for k in range(threads)]
    for t in pool:
        t.start()
    for t in pool:
        t.join()
    sur.synchronize()
    assert not bad
    for k in range(threads):
        wrong = (grad[k] != alone[k][1]).any(dim=1) | (loss[k] != alone[k][0])
        assert int(wrong.sum()) == 0, (k, int(wrong.sum()))
    sur.close()
