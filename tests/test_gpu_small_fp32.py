"""The LDS-resident fp32 step and score at sizes where a tile can go wrong: widths, batches and held-out sets just below, at
and above multiples of 16, one layer to four, one input, and a network too large for the padded arrays (plain form)."""
import numpy as np
import pytest

from paper_1711_09846_amd import binding, workloads as W
from tests.harness import Pair

pytestmark = pytest.mark.gpu

SGD, ADAM, RMS = W.OPT_SGD_MOMENTUM, W.OPT_ADAM, W.OPT_RMSPROP
CONST = {SGD: dict(momentum=0.9), ADAM: dict(beta1=0.9, beta2=0.999, eps=1e-8), RMS: dict(rho=0.99, eps=1e-5)}
SHAPES = [
    # dims, batch, held-out rows, activation, optimiser
    ([1, 16, 2], 1, 1, W.ACT_RELU, SGD),
    ([11, 71, 20, 5], 17, 65, W.ACT_TANH, RMS),
    ([16, 32, 32], 16, 64, W.ACT_LEAKY_RELU, ADAM),
    ([17, 3], 33, 100, W.ACT_NONE, SGD),
    ([33, 15, 48, 9, 7], 63, 63, W.ACT_GELU, RMS),
    ([64, 96, 10], 31, 129, W.ACT_GELU, SGD),
    ([40, 50, 17], 128, 200, W.ACT_RELU, SGD),      # 157 KB unpadded, 174 KB padded
]


@pytest.mark.parametrize("dims,batch,n_eval,act,opt", SHAPES, ids=lambda v: str(v))
def test_step_and_score_against_the_oracle(dims, batch, n_eval, act, opt):
    """Three steps from the same start, then the score.  fp32 sums of at most 128 products of O(1) terms: 128 x 2^-24 = 8e-6
    at worst per sum, a few 1e-7 as a rule; 2e-5 leaves room for three chained layers and steps.  Adam and RMSProp divide by
    the root of near-zero mean squares in the first steps: 2e-4 there.  Losses near 1: same bound."""
    _step_and_score(dims, batch, n_eval, act, opt)


def _step_and_score(dims, batch, n_eval, act, opt):
    wl = W.MLP_SMALL.replace(P=3, dims=dims, batch=batch, n_eval=n_eval, n_train=500, n_trunc=1, act=act, optimizer=opt, n_classes=dims[-1],
                             opt_const=CONST[opt], priors=[("log", 1e-3, 1e-2)])
    pair = Pair(wl)
    pair.gpu.step(pair.d_train, 0)
    pair.gpu.step(pair.d_train, 1, n_steps=2)
    for s in range(3):
        loss = pair.step_ref(s)
    tol = 2e-5 if opt == SGD else 2e-4
    assert pair.scalar_errors(pair.gpu.get(binding.ARR_LOSS), loss, 1e-2) <= tol
    assert pair.tensor_errors(binding.ARR_W32, "theta") <= tol
    assert pair.tensor_errors(binding.ARR_OPT0, "s0") <= tol
    if opt == ADAM:
        assert pair.tensor_errors(binding.ARR_OPT1, "s1") <= tol
    assert np.all(pair.gpu.get(binding.ARR_T) == 3)
    pair.gpu.eval(pair.d_eval)
    assert pair.scalar_errors(pair.gpu.get(binding.ARR_SCORE), pair.eval_ref(), 1e-2) <= tol


def _padded(w):
    return -(-w // 16) * 16


def _step_fits_padded(dims, batch, opt):
    """Whether the step's arrays fit a compute unit's 160 KB when widths and rows are padded to 16 (and pitches by 4)."""
    pairs, rows = list(zip(dims[:-1], dims[1:])), _padded(batch)
    params = 0
    for fi, fo in pairs:
        params = -(-(params + fi * fo) // 64) * 64
        params = -(-(params + fo) // 64) * 64
    params = -(-params // 256) * 256
    floats = sum(_padded(fi) * (_padded(fo) + 4) + _padded(fo) for fi, fo in pairs) + params * (2 if opt == ADAM else 1)
    floats += rows * (2 * (_padded(dims[0]) + 4) + sum(_padded(w) + 4 for w in dims[1:-1]) + sum(_padded(w) + 4 for w in dims[1:])) + 3 * rows + 4
    return floats * 4 <= 160 * 1024


def _score_fits_padded(dims):
    """The same for the score: the parameters and two buffers of 64 rows of the widest layer, beside 1 KB."""
    floats = sum(_padded(fi) * (_padded(fo) + 4) + _padded(fo) for fi, fo in zip(dims[:-1], dims[1:])) + 2 * 64 * (_padded(max(dims)) + 4)
    return floats * 4 <= 159 * 1024


@pytest.mark.parametrize("dims,batch,n_eval,act,opt,plain", [
    ([40, 50, 17], 100, 200, W.ACT_GELU, ADAM, "step"),
    ([40, 50, 17], 128, 40, W.ACT_TANH, RMS, "step"),
    ([100, 66, 5], 33, 70, W.ACT_LEAKY_RELU, ADAM, "step"),
    ([8, 7, 6, 8, 5, 2], 3, 20, W.ACT_LEAKY_RELU, RMS, "chain"),
    ([32, 256, 4], 8, 150, W.ACT_RELU, SGD, "score"),
    ([16, 256, 10], 16, 17, W.ACT_GELU, RMS, "score"),
    ([320, 32, 10], 16, 33, W.ACT_TANH, SGD, "score"),
], ids=lambda v: str(v))
def test_plain_form_against_the_oracle(dims, batch, n_eval, act, opt, plain):
    """The form without padding: the step of networks whose padded arrays do not fit, the step of a chain of small layers, the score
    of networks whose 64 padded rows do not fit (their step does).  Bounds as above, for sums of up to 320 products."""
    if plain == "step":
        assert not _step_fits_padded(dims, batch, opt)
    elif plain == "chain":
        assert len(dims) > 4 and max(dims) <= 8 and batch <= 4
    else:
        assert _step_fits_padded(dims, batch, opt) and not _score_fits_padded(dims)
    _step_and_score(dims, batch, n_eval, act, opt)


@pytest.mark.parametrize("label", [0, 1])
@pytest.mark.parametrize("C", [2, 3, 4, 5, 7, 10])
def test_a_logit_that_is_nan_marks_its_member(C, label):
    """Member i's output i is NaN in every row (its bias is), the last member is sound.  The softmax of such a row is NaN throughout,
    also where no label names the class: the loss, every gradient and the score of the member are NaN, whichever class it is."""
    wl = W.MLP_SMALL.replace(P=C + 1, dims=[6, 20, C], batch=19, n_train=64, n_eval=70, n_trunc=0, n_classes=C)
    rng = np.random.default_rng(C)
    rows = lambda n: (rng.standard_normal((n, 6)).astype(np.float32), np.full(n, label, dtype=np.int32))  # noqa: E731
    pair = Pair(wl, data=(rows(wl.n_train), rows(wl.n_eval)))
    lay = pair.gpu.layout
    for i in range(C):
        theta = pair.gpu.get(binding.ARR_W32, i).reshape(-1)
        theta[lay.b_off[1] + i] = np.nan
        pair.gpu.set(binding.ARR_W32, theta, i)
    pair.gpu.eval(pair.d_eval)
    sc = pair.gpu.get(binding.ARR_SCORE)
    assert np.all(np.isnan(sc[:C])) and np.isfinite(sc[C]), sc
    pair.gpu.step(pair.d_train, 0)
    loss, grad = pair.gpu.get(binding.ARR_LOSS).reshape(-1), pair.gpu.get(binding.ARR_GRAD)
    assert np.all(np.isnan(loss[:C])) and np.isfinite(loss[C]), loss
    for l, (fi, fo) in enumerate(((6, 20), (20, C))):
        for off, n in ((lay.w_off[l], fi * fo), (lay.b_off[l], fo)):
            g = grad[:, off:off + n]
            if l == 1:
                assert np.all(np.isnan(g[:C])), (l, off)
            assert np.all(np.isfinite(g[C]))


def test_a_logit_that_is_infinite_marks_its_member():
    """Output i of member i is +infinity: exp(l - max) of that class is NaN, and with it its gradient (the labels name another)."""
    C = 5
    wl = W.MLP_SMALL.replace(P=C + 1, dims=[6, 20, C], batch=19, n_train=64, n_eval=70, n_trunc=0, n_classes=C)
    rng = np.random.default_rng(1)
    rows = lambda n: (rng.standard_normal((n, 6)).astype(np.float32), rng.integers(0, 1, n).astype(np.int32))  # noqa: E731
    pair = Pair(wl, data=(rows(wl.n_train), rows(wl.n_eval)))
    lay = pair.gpu.layout
    for i in range(1, C):
        theta = pair.gpu.get(binding.ARR_W32, i).reshape(-1)
        theta[lay.b_off[1] + i] = np.inf
        pair.gpu.set(binding.ARR_W32, theta, i)
    pair.gpu.step(pair.d_train, 0)
    loss, grad = pair.gpu.get(binding.ARR_LOSS).reshape(-1), pair.gpu.get(binding.ARR_GRAD)[:, lay.b_off[1]:lay.b_off[1] + C]
    assert np.all(np.isposinf(loss[1:C])) and np.isfinite(loss[0]) and np.isfinite(loss[C])
    for i in range(1, C):
        assert np.isnan(grad[i, i]) and np.isclose(grad[i, 0], -1.0) and np.all(np.delete(grad[i], [0, i]) == 0)


@pytest.mark.parametrize("opt", [SGD, ADAM, RMS])
@pytest.mark.parametrize("dims,batch", [([20, 40, 5], 19), ([11, 24, 17, 6], 33), ([13, 9, 10, 8, 7], 40), ([50, 5], 70),
                                        ([4, 8, 2], 16), ([32, 4], 32), ([32, 4], 33)], ids=lambda v: str(v))
def test_results_do_not_depend_on_the_size_of_the_population(dims, batch, opt):
    """More members than compute units take smaller workgroups (300: two to a compute unit, 1000: four).  A member's draws
    depend on its number alone, so the first eight are bit for bit those of a population of eight."""
    import torch
    rng = np.random.default_rng(2)
    x, y = rng.standard_normal((400, dims[0])).astype(np.float32), rng.integers(0, dims[-1], 400).astype(np.int32)
    arrays = [binding.ARR_W32, binding.ARR_OPT0, binding.ARR_GRAD, binding.ARR_LOSS, binding.ARR_T] + ([binding.ARR_OPT1] if opt == ADAM else [])
    got = {}
    for P in (8, 300, 1000):
        wl = W.MLP_SMALL.replace(P=P, dims=dims, batch=batch, n_eval=50, n_train=400, n_trunc=0, act=W.ACT_GELU, optimizer=opt, n_classes=dims[-1],
                                 opt_const=CONST[opt], priors=[("log", 1e-3, 1e-2)])
        pop = binding.Population(binding.make_config(wl, 7))
        pop.init_population(wl.priors)
        data = [torch.from_numpy(x).to(pop.device), torch.from_numpy(y).to(pop.device)]
        pop.step(data, 0, n_steps=3)
        pop.step(data, 3)
        got[P] = [pop.get(w) for w in arrays]
        assert np.all(np.isfinite(got[P][0])) and np.any(got[P][2][P - 1])
    for P in (300, 1000):
        for which, a, b in zip(arrays, got[8], got[P]):
            assert a.tobytes() == b[:8].tobytes(), (P, which)
