"""pbt_step_static (the step with the library's static working memory, for callers that cannot
allocate) against pbt_step: same kernels, so every array of the population store must come out
bit-identical, on two calls in a row that share the static array, the second with a smaller input."""
import numpy as np
import pytest

from paper_1711_09846_amd import binding, workloads
from tests.harness import Pair

pytestmark = pytest.mark.gpu

ARRAYS_BF16 = (binding.ARR_W32, binding.ARR_OPT0, binding.ARR_OPT1, binding.ARR_W16, binding.ARR_T, binding.ARR_LOSS)
ARRAYS_FP32 = (binding.ARR_W32, binding.ARR_OPT0, binding.ARR_T, binding.ARR_LOSS)


def _bigger():
    return workloads.MLP_WIDE.replace(P=6, dims=[72, 200, 136, 10], batch=40, n_train=4096, n_eval=300, n_trunc=1,
                                      priors=[("log", 1e-4, 3e-3), ("uniform", 0.8, 0.95), ("log", 1e-6, 1e-3)])


def _smaller():
    return workloads.MLP_WIDE.replace(P=3, dims=[40, 64, 10], batch=24, n_train=1024, n_eval=100, n_trunc=1,
                                      priors=[("log", 1e-4, 3e-3), ("uniform", 0.8, 0.95), ("log", 1e-6, 1e-3)])


def _same(a, b, arrays):
    for which in arrays:
        assert a.gpu.get(which).tobytes() == b.gpu.get(which).tobytes(), which


def test_static_step_equals_step_on_two_calls_the_second_smaller():
    # call 1: the bigger population fills the static array with its gradients and activations
    a, b = Pair(_bigger(), eval_chunk=128), Pair(_bigger(), eval_chunk=128)
    assert a.gpu.scratch.numel() <= binding.STATIC_SCRATCH_BYTES
    a.gpu.step(a.d_train, 0)
    b.gpu.step_static(b.d_train, 0)
    _same(a, b, ARRAYS_BF16)
    # call 2, straight after it: a smaller population, whose buffers now overlay what call 1 left behind
    c, d = Pair(_smaller()), Pair(_smaller())
    c.gpu.step(c.d_train, 0)
    d.gpu.step_static(d.d_train, 0)
    _same(c, d, ARRAYS_BF16)
    # and both keep agreeing over further alternating calls (padding of theta stays zero on both sides)
    for s in range(1, 4):
        a.gpu.step(a.d_train, s)
        b.gpu.step_static(b.d_train, s)
        c.gpu.step(c.d_train, s)
        d.gpu.step_static(d.d_train, s)
    _same(a, b, ARRAYS_BF16)
    _same(c, d, ARRAYS_BF16)
    lay = b.gpu.layout
    pad = np.ones(lay.stride, dtype=bool)
    for j in range(lay.n_seg):
        pad[lay.seg_off[j]:lay.seg_off[j] + lay.seg_len[j]] = False
    assert not np.any(b.gpu.get(binding.ARR_W32)[:, pad])
    # the scores that follow from those weights agree too
    a.gpu.eval(a.d_eval)
    b.gpu.eval(b.d_eval)
    assert a.gpu.get(binding.ARR_SCORE).tobytes() == b.gpu.get(binding.ARR_SCORE).tobytes()


def test_static_step_fp32_multi_step_launch():
    a, b = Pair(workloads.MLP_SMALL), Pair(workloads.MLP_SMALL)
    a.gpu.step(a.d_train, 0, n_steps=7)
    b.gpu.step_static(b.d_train, 0, n_steps=7)
    _same(a, b, ARRAYS_FP32)


def test_static_step_rejects_what_does_not_fit():
    """The full-size wide workload needs ~1 GB of working memory: refused with a clear error before any launch."""
    pop = binding.Population(binding.make_config(workloads.MLP_WIDE, 1))
    (tx, ty), _ = workloads.classifier_data(workloads.MLP_WIDE.replace(n_train=256, n_eval=16))
    import torch
    d = [torch.from_numpy(tx).to(pop.device), torch.from_numpy(ty).to(pop.device)]
    before = pop.get(binding.ARR_T).copy()
    with pytest.raises(binding.PbtError) as e:
        pop.step_static(d, 0)
    assert e.value.status == -2 and "static" in str(e.value)
    assert np.array_equal(pop.get(binding.ARR_T), before)


def _static_against_step(wl, inputs, steps=2, **kw):
    """Two populations of the same configuration, one stepped with each entry point: bit-identical stores.  Returns one of them."""
    a, b = (binding.Population(binding.make_config(wl, 1, **kw)) for _ in range(2))
    arrays = [binding.ARR_W32, binding.ARR_OPT0, binding.ARR_W16, binding.ARR_T, binding.ARR_LOSS]
    if wl.optimizer == workloads.OPT_ADAM:
        arrays.append(binding.ARR_OPT1)
    for pop in (a, b):
        pop.init_population(wl.priors)
    inputs = [x.to(a.device) for x in inputs]
    for s in range(steps):
        a.step(inputs, s)
        b.step_static(inputs, s)
    for which in arrays:
        assert a.get(which).tobytes() == b.get(which).tobytes(), which
    assert np.all(np.isfinite(b.get(binding.ARR_LOSS)))
    used = np.zeros(b.layout.stride, dtype=bool)
    for j in range(b.layout.n_seg):
        used[b.layout.seg_off[j]:b.layout.seg_off[j] + b.layout.seg_len[j]] = True
    assert not np.any(b.get(binding.ARR_W32)[:, ~used])
    return a


def test_static_step_does_not_count_the_held_out_pass():
    """A held-out set whose buffers alone are larger than the static array: a step does not touch them."""
    import torch
    wl = workloads.GAN_MLP.replace(P=2, dims=[16, 32, 40], dims2=[40, 32, 1], batch=8, n_train=300, n_eval=20000, n_trunc=0)
    assert binding.query_sizes(binding.make_config(wl, 1))[1] > binding.STATIC_SCRATCH_BYTES
    _static_against_step(wl, [torch.randn(300, 40)])


def _acting(P, dims, batch, unroll, latent):
    return workloads.A2C_MLP.replace(P=P, dims=dims, n_actions=dims[-1] - 1, batch=batch, unroll=unroll, latent=latent, n_trunc=0, on_policy=1)


@pytest.mark.parametrize("fused", [0, 1])
@pytest.mark.parametrize("wl,launches", [
    (_acting(6, [512, 256, 256, 19], 8, 5, 16), 0),    # packed weights and draws over the update's buffers
    (_acting(22, [320, 128, 256, 3], 2, 2, 15), 0),    # too large for those: the packed weights over the gradients
    (_acting(240, [8, 200, 3], 2, 1, 3), 2),           # larger than the gradients too: the kernels of one round each, two products per round
], ids=["over the update", "over the gradients", "in rounds"])
def test_static_step_of_acting_agents(wl, launches, fused):
    """Actor-critic populations whose packed weights, in memory of their own, are larger than what is left of the static array."""
    import torch
    noise = np.array([1.0, 0.1, 0.1])
    inputs = [torch.from_numpy(np.ascontiguousarray(x, dtype=np.float64)) for x in (*workloads.latent_system(wl), noise)]
    pop = _static_against_step(wl, inputs, steps=3, fuse_optimizer=fused)
    # which form of the unroll it was: the one-kernel form has no launches of the fetch class
    pop.timing_enable(binding.K_FETCH, 64)
    pop.step([x.to(pop.device) for x in inputs], 3)
    assert pop.timing_read()[1] == launches
    # gradients that no launch writes, and their padding, are zero
    grad, lay = pop.get(binding.ARR_GRAD), pop.layout
    written = np.zeros(lay.stride, dtype=bool)
    for j in range(lay.n_seg):
        if not fused or j % 2 or j == lay.n_seg - 2:
            written[lay.seg_off[j]:lay.seg_off[j] + lay.seg_len[j]] = True
    assert not np.any(grad[:, ~written]) and np.any(grad[:, written])


@pytest.mark.parametrize("P,vocab,d_model,heads,d_ff,blocks,seq,batch", [
    (2, 256, 128, 2, 512, 1, 32, 8),     # pieces of every weight gradient would not fit beside the rest
    (2, 512, 128, 2, 512, 1, 32, 8),
    (1, 96, 256, 4, 512, 1, 64, 4),
    (5, 120, 32, 1, 16, 4, 8, 45),       # short sequences: keep bits of the positions that exist
    (1, 40, 384, 6, 16, 1, 56, 6),
])
def test_static_step_of_small_transformers(P, vocab, d_model, heads, d_ff, blocks, seq, batch):
    import torch
    wl = workloads.TRANSFORMER.replace(P=P, vocab=vocab, d_model=d_model, heads=heads, d_ff=d_ff, n_blocks=blocks, seq=seq, batch=batch,
                                       n_train=60, n_eval=batch, n_trunc=0)
    tokens = torch.from_numpy(np.random.default_rng(3).integers(0, vocab, (60, seq + 1)).astype(np.int32))
    _static_against_step(wl, [tokens])
