"""Training kernels on a network of several output tiles and input chunks (32
species: 35 inputs, 33 outputs), against the numpy oracle."""
import numpy as np
import pytest

from oracle import mlp_oracle as mo

from gpu_common import to_gpu

pytestmark = pytest.mark.gpu
I, O = 35, 33


@pytest.fixture(scope="module")
def cg():
    from paper_2506_02602_amd import chemgpu
    return chemgpu


@pytest.fixture(scope="module")
def gm32(cg, mech32_path):
    return cg.chem_mech_load(mech32_path)


def _rel_fro(a, b):
    return float(np.linalg.norm(a - b) / np.linalg.norm(b))


@pytest.mark.parametrize("B", [1, 16, 17, 33, 500, 512])
def test_gradients_match_oracle(cg, gm32, B):
    """As for one output tile (the same tolerances): the zeroed columns past the
    outputs, three output tiles on three waves, two chunks of inputs and of
    outputs."""
    rng = np.random.Generator(np.random.PCG64(90 + B))
    Xn = rng.standard_normal((B, I)).astype(np.float32)
    Yn = rng.standard_normal((B, O)).astype(np.float32)
    s = cg.Surrogate(gm32, seed=5)
    theta, _ = s.get_params()
    grad, loss = cg.surrogate_grad(s, to_gpu(Xn), to_gpu(Yn))
    g_ref, loss_ref = mo.backward(theta.astype(np.float64), Xn.astype(np.float64),
                                  Yn.astype(np.float64), I, O)
    assert loss == pytest.approx(loss_ref, rel=1e-3)
    pg, pr = mo.unpack(grad.cpu().numpy().astype(np.float64), I, O), mo.unpack(g_ref, I, O)
    for name in pg:
        assert _rel_fro(pg[name], pr[name]) < 1e-2, name


def test_adam_steps_match_oracle(cg, gm32):
    """One batch of one repeated sample (the epoch's permutation then changes no
    sum): Adam on the kernel's own gradient, to the rounding of the FP32 update;
    and the packed weights that the step leaves give the gradient of the updated
    parameters."""
    rng = np.random.Generator(np.random.PCG64(95))
    B = 256
    X = np.repeat(rng.standard_normal((1, I)), B, axis=0).astype(np.float32)
    Y = np.repeat(rng.standard_normal((1, O)), B, axis=0).astype(np.float32)
    s = cg.Surrogate(gm32, seed=6)
    theta0, _ = s.get_params()
    ident = np.concatenate([np.zeros(I), np.ones(I), np.zeros(O), np.ones(O),
                            np.full(I, -10.0), np.full(I, 10.0)]).astype(np.float32)
    s.set_params(norm=ident)
    g0, _ = cg.surrogate_grad(s, to_gpu(X), to_gpu(Y))
    g0 = g0.cpu().numpy().astype(np.float64)
    cg.surrogate_train(s, to_gpu(X), to_gpu(Y), epochs=1, batch=B, lr=1e-3, seed=1)
    theta1, _ = s.get_params()
    ref, _, _ = mo.adam_step(theta0.astype(np.float64), g0, np.zeros_like(g0), np.zeros_like(g0), 1,
                             lr=1e-3, beta1=float(np.float32(0.9)), beta2=float(np.float32(0.999)))
    ulp = np.spacing(np.abs(ref).astype(np.float32)).astype(np.float64)
    assert (np.abs(theta1.astype(np.float64) - ref) <= ulp + 1e-9).all()
    # two epochs: the second step runs on the weights the first one packed
    t = cg.Surrogate(gm32, seed=6)
    t.set_params(theta=theta0, norm=ident)
    loss = cg.surrogate_train(t, to_gpu(X), to_gpu(Y), epochs=2, batch=B, lr=1e-3, seed=1)
    _, want = mo.backward(t_after_first(theta0, g0), X.astype(np.float64), Y.astype(np.float64), I, O)
    assert loss[1] == pytest.approx(want, rel=2e-3) and loss[1] < loss[0]


def t_after_first(theta0, g0):
    """theta after the first of two steps (the cosine schedule's full rate)."""
    ref, _, _ = mo.adam_step(theta0.astype(np.float64), g0, np.zeros_like(g0), np.zeros_like(g0), 1,
                             lr=1e-3)
    return ref
