"""The closure kernels at the edges of their tiles and of the choice between
them: inference switches kernel at 4 096, 8 192 and 16 384 rows and takes 16,
32 or 64 rows per workgroup (32 per wavefront above), training 64.

A row's products and their order are the same in every inference kernel, so a
row gives the same bits in a batch of any size; the envelope flags are exact.
Gradients differ from the FP64 oracle (which rounds the same operands to
bfloat16) by binary32 accumulation and by the few bfloat16 roundings it turns
the other way: 1e-2 per tensor norm-wise, as in test_mlp_gpu.py.
"""
import numpy as np
import pytest

from oracle import mlp_oracle as M

pytestmark = pytest.mark.gpu


def problem(n, seed):
    params = M.init_params(seed)
    rng = np.random.default_rng(seed)
    for W, b in params:
        b[:] = rng.standard_normal(b.shape) * 0.05
    f32 = lambda a: np.asarray(a, dtype=np.float32).astype(np.float64)  # noqa: E731
    params = [[f32(W), f32(b)] for W, b in params]
    X = f32(rng.standard_normal((n, 40)))
    return params, X, f32(np.sin(X[:, 0]) + 0.3 * X[:, 1] * X[:, 2])


def test_inference_rows_do_not_depend_on_the_batch(gpu_lib):
    import torch
    N = 40001
    params, X, _ = problem(N, 5)
    mu, sd = np.linspace(-1, 1, 40), np.linspace(0.5, 2.0, 40)
    raw = (mu + sd * X).astype(np.float32)
    lo, hi = (mu - 2.5 * sd).astype(np.float32), (mu + 2.5 * sd).astype(np.float32)
    raw[7, 3], raw[N - 1, 39], raw[40, 0] = np.nan, np.inf, -np.inf
    m = gpu_lib.Mlp(max_batch=64)
    m.set_params(gpu_lib.mlp_pack(params))
    m.set_normaliser(mu, sd, lo, hi)
    with np.errstate(invalid="ignore"):
        out = ~((raw >= lo) & (raw <= hi)).all(axis=1)
    # inputs without a non-finite value, for the values
    good = np.isfinite(raw).all(axis=1)
    y_all, f_all = (t.cpu().numpy() for t in m.infer(raw))
    fw_all = m.forward(X).cpu().numpy()
    ref, _ = M.forward(params, ((raw - np.float32(mu)) / np.float32(sd)).astype(np.float64), bf16_ops=True)
    assert np.abs(y_all - ref)[good].max() / np.abs(ref[good]).max() < 2e-3
    assert np.array_equal(f_all.astype(bool), out)
    for n in (1, 15, 16, 17, 33, 65, 4096, 4097, 8191, 8192, 8193, 16383, 16384, 16385, 32769):
        print("inference of %d rows" % n, flush=True)
        y, f = (t.cpu().numpy() for t in m.infer(raw[:n]))
        fw = m.forward(X[:n]).cpu().numpy()
        assert np.array_equal(f, f_all[:n])
        assert np.array_equal(y[good[:n]], y_all[:n][good[:n]]) and np.isnan(y[~good[:n]]).all()
        assert np.array_equal(fw, fw_all[:n])
    torch.cuda.synchronize()


@pytest.mark.parametrize("n", [1, 63, 64, 65, 129, 4095])
def test_gradients_at_workgroup_edges(gpu_lib, n):
    params, X, y = problem(n, 30 + n)
    m = gpu_lib.Mlp(max_batch=n)
    m.set_params(gpu_lib.mlp_pack(params))
    g, loss = m.gradients(X, y)
    loss_ref, g_ref = M.loss_and_grads(params, X, y, bf16_ops=True)
    print("gradients of %d rows: loss %.8g, oracle %.8g" % (n, loss, loss_ref), flush=True)
    assert abs(loss - loss_ref) <= 1e-4 * abs(loss_ref) + 1e-7
    got = gpu_lib.mlp_unpack(g)
    for k in range(4):
        for j in range(2):
            a, b = np.asarray(got[k][j], dtype=np.float64), np.asarray(g_ref[k][j]).reshape(np.shape(got[k][j]))
            assert np.linalg.norm(a - b) <= 1e-2 * max(np.linalg.norm(b), 1e-30)
    # the same call twice gives the same bits, and a step equals Adam on that gradient
    g2, loss2 = m.gradients(X, y)
    assert np.array_equal(g, g2) and loss == loss2
    p0 = m.get_params().astype(np.float64)
    assert m.train_step(X, y, 1e-3) == loss
    g64 = g.astype(np.float64)
    step = 1e-3 * g64 / (np.abs(g64) + 1e-8)
    # the moments are divided by 1 - beta^1 in binary32: a few units of the last
    # place of the step and one of the parameter
    assert np.abs(m.get_params() - (p0 - step)).max() <= 1e-3 * 2e-5 + 2.0 ** -24 * np.abs(p0).max()
