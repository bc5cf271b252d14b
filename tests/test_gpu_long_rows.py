"""Matrices with rows of 2^24 elements, past what the products' buffer offsets span: every functor of the GEMM has to serve them.  The
networks are compared with narrow ones: whatever lies beyond the narrow width is switched off by its bias, which has to be added for that."""
import numpy as np
import pytest

from paper_1711_09846_amd import binding, workloads

pytestmark = pytest.mark.gpu

WIDE, NARROW = 1 << 24, 64
OFF = -1e4          # bias of what is switched off: exp(OFF) and relu(OFF + a) are zero
TOL_SUM = 1e-4      # fp32 sums of the same terms in another order (and zeros)
TOL_BF16 = 5e-2     # norm of a gradient: a stored bf16 value may round the other way after such a sum, one in a batch of 8 moves it by a few percent


def _population(wl, H):
    import torch
    pop = binding.Population(binding.make_config(wl, 5))
    pop.init_population(wl.priors)
    pop.device_view(binding.ARR_HYPER).copy_(torch.tensor([H]))
    return pop


def _segments(pop, which=binding.ARR_W32):
    lay, flat = pop.layout, pop.device_view(which)[0]
    return [flat[lay.seg_off[k]:lay.seg_off[k] + lay.seg_len[k]] for k in range(lay.n_seg)]


def _share(small, wide, cols=(), off=()):
    """The narrow population's weights into the wide one.  cols: arrays whose rows are wide; the others begin with the narrow array.  off: biases."""
    import torch
    for k, (a, b) in enumerate(zip(_segments(small), _segments(wide))):
        if k in cols:
            b.view(-1, WIDE)[:, :NARROW] = a.view(-1, NARROW)
        else:
            b[:a.numel()] = a
        if k in off:
            b[a.numel():] = OFF
    for pop in (small, wide):
        pop.device_view(binding.ARR_W16).view(torch.bfloat16).copy_(pop.device_view(binding.ARR_W32))


def _gradients_agree(small, wide, cols):
    for k, (a, b) in enumerate(zip(_segments(small, binding.ARR_GRAD), _segments(wide, binding.ARR_GRAD))):
        got = b.view(-1, WIDE)[:, :NARROW].reshape(-1) if k in cols else b[:a.numel()]
        scale = float(a.double().norm())
        assert float((got.double() - a.double()).norm()) <= TOL_BF16 * scale, k
        assert abs(float(b.double().norm()) - scale) <= TOL_BF16 * scale, k      # (nothing beyond the narrow part)


def _close(pop_a, pop_b, which):
    a, b = pop_a.get(which), pop_b.get(which)
    assert np.all(np.isfinite(a)) and np.max(np.abs(a - b) / np.abs(a)) <= TOL_SUM, (a, b)


def test_vocabulary():
    """Float logits, their gradient's products and the held-out statistics."""
    import torch
    pops = []
    for vocab in (NARROW, WIDE):
        wl = workloads.TRANSFORMER.replace(P=1, vocab=vocab, d_model=8, heads=1, d_ff=8, n_blocks=1, seq=8, batch=1, n_train=4, n_eval=2, n_trunc=0)
        pops.append(_population(wl, [1e-3, 0.1, 0.0]))
    n_seg = pops[0].layout.n_seg
    _segments(pops[0])[n_seg - 1].normal_(generator=torch.Generator("cuda").manual_seed(1))
    cols, off = {n_seg - 2}, {n_seg - 1}
    _share(*pops, cols=cols, off=off)
    tokens = torch.randint(NARROW, (4, 9), generator=torch.Generator("cuda").manual_seed(2), device="cuda").int()
    for pop in pops:
        pop.eval([tokens[:2].contiguous()])
        pop.step([tokens], 0)
    _close(*pops, binding.ARR_SCORE)
    _close(*pops, binding.ARR_LOSS)
    _gradients_agree(*pops, cols)


def test_hidden_layer():
    """Bias and activation, the derivative of the layer below, weight gradients on both sides of a wide hidden layer."""
    import torch
    pops = []
    for width in (NARROW, WIDE):
        wl = workloads.MLP_WIDE.replace(P=1, dims=[16, 8, width, 8, 4], act=workloads.ACT_RELU, batch=24, n_train=64, n_eval=16, n_classes=4, n_trunc=0)
        pops.append(_population(wl, [1e-3, 0.9, 1e-4]))
    _share(*pops, cols={2}, off={3})
    g = torch.Generator("cuda").manual_seed(3)
    x, y = torch.randn(64, 16, generator=g, device="cuda"), torch.randint(4, (64,), generator=g, device="cuda").int()
    for pop in pops:
        pop.eval([x[:16].contiguous(), y[:16].contiguous()])
        pop.step([x, y], 0)
    _close(*pops, binding.ARR_SCORE)
    _close(*pops, binding.ARR_LOSS)
    _gradients_agree(*pops, {2})


def test_held_out_rows():
    """The RBF sums of rows as wide: a generator whose last layer is its bias alone, so that its rows are known."""
    import torch
    E = 70      # more than a tile
    wl = workloads.GAN_MLP.replace(P=1, dims=[8, 8, WIDE], dims2=[WIDE, 8, 1], batch=1, n_train=1, n_eval=E, n_trunc=0)
    pop = _population(wl, [1e-4, 1e-4])
    seg = _segments(pop)
    seg[2].zero_()
    seg[3].normal_(generator=torch.Generator("cuda").manual_seed(4))
    pop.device_view(binding.ARR_W16).view(torch.bfloat16).copy_(pop.device_view(binding.ARR_W32))
    held = torch.randn(E, WIDE, generator=torch.Generator("cuda").manual_seed(5), device="cuda")
    pop.eval([held])
    x = torch.tanh(seg[3]).bfloat16()
    y = held.bfloat16()
    dot = torch.zeros(E, E, device="cuda", dtype=torch.float64)
    dxy = torch.zeros(E, device="cuda", dtype=torch.float64)
    for c in range(0, WIDE, 1 << 20):
        a, b = x[c:c + (1 << 20)].double(), y[:, c:c + (1 << 20)].double()
        dot += b @ b.T
        dxy += ((b - a) ** 2).sum(1)
    sq = dot.diagonal()
    kyy = torch.exp(-(sq[:, None] + sq[None, :] - 2 * dot) / (2 * WIDE))
    ref = -float(1 + kyy.mean() - 2 * torch.exp(-dxy / (2 * WIDE)).mean())
    got = float(pop.get(binding.ARR_SCORE)[0])
    # (a norm of 2^24 squares adds up in chains of 2^20 to 2^15 fp32 terms: a relative error of 2^-24 sqrt(2^20) = 6e-5 of an exponent of about 1)
    assert abs(got - ref) <= 1e-3, (got, ref)
