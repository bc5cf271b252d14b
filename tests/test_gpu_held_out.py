"""The held-out scores where their kernels' tiles and pieces have remainders, against the oracle."""
import numpy as np
import pytest

from paper_1711_09846_amd import binding, workloads
from tests import native
from tests.harness import GanPair, TransformerPair

pytestmark = pytest.mark.gpu

TOL_BF16 = 1e-2     # as in the free-running tests of the two workloads: bf16 activations on both sides
FLOOR = 1e-2


@pytest.mark.parametrize("n_eval", [1, 63, 129, 300])
def test_mmd_of_ragged_held_out_sets(n_eval):
    """Only the tiles at and right of the diagonal of the symmetric Gram matrices are computed: one row, one row less
    than a tile's 64 columns, one more than its 128 rows, several tiles with a remainder."""
    pair = GanPair(workloads.GAN_MLP.replace(P=3, dims=[16, 72, 40], dims2=[40, 136, 24, 1], batch=24, n_train=1024, n_eval=n_eval, n_trunc=1,
                                             priors=[("log", 1e-4, 2e-3), ("log", 1e-4, 2e-3)], n_modes=4, rank=8))
    for i in range(3):
        pair.sync_ref_from_gpu(i)
    pair.gpu.eval(pair.d_eval)
    sc, ref = pair.gpu.get(binding.ARR_SCORE), pair.eval_ref()
    assert np.max(np.abs(sc - ref) / np.maximum(np.abs(ref), FLOOR)) <= TOL_BF16, (sc, ref)


def test_mmd_on_persistent_tiles():
    """256 x 256 tiles, several to a workgroup, of symmetric matrices whose last row and column of tiles are ragged."""
    P, E, D = 18, 1701, 512
    assert native.tile(E, E, D, P, heavy=True, square=True, upper=True) == native.TILE_256 and 28 * P > 256
    pair = GanPair(workloads.GAN_MLP.replace(P=P, dims=[16, 24, D], dims2=[D, 24, 1], batch=24, n_train=1024, n_eval=E, n_trunc=0,
                                             priors=[("log", 1e-4, 2e-3), ("log", 1e-4, 2e-3)], n_modes=4, rank=8), ref_members=[0, P - 1])
    for i in pair.ref_ids:
        pair.sync_ref_from_gpu(i)
    pair.gpu.eval(pair.d_eval)
    sc, ref = pair.gpu.get(binding.ARR_SCORE)[pair.ref_ids], pair.eval_ref()
    assert np.max(np.abs(sc - ref) / np.maximum(np.abs(ref), FLOOR)) <= TOL_BF16, (sc, ref)


@pytest.mark.parametrize("vocab,seq,batch", [
    (8, 16, 3),          # one piece, narrower than a lane group's columns
    (104, 24, 5),        # narrow tile, three whole pieces of 32 and a remainder
    (1000, 32, 2),
    (8192, 128, 8),      # enough tiles for the wide one: pieces of 64
    (8200, 128, 8),      # and a remainder
])
def test_perplexity_from_pieces_of_rows(vocab, seq, batch):
    """The output layer hands over a maximum and a sum per piece of a row instead of logits."""
    wl = workloads.TRANSFORMER.replace(P=2, vocab=vocab, d_model=32, heads=2, d_ff=64, n_blocks=1, seq=seq, batch=batch, n_train=16,
                                       n_eval=2 * batch if vocab < 8000 else batch, n_trunc=1)
    pair = TransformerPair(wl)
    for i in range(2):
        pair.sync_ref_from_gpu(i)
    pair.gpu.eval(pair.d_eval)
    sc, ref = pair.gpu.get(binding.ARR_SCORE), pair.eval_ref()
    # the cross-entropy is compared (its exponential is the score): float sums over the vocabulary, bf16 activations before them
    assert np.max(np.abs(np.log(-sc) - np.log(-ref))) <= TOL_BF16, (sc, ref)


def test_perplexity_on_persistent_tiles():
    """The output layer on 256 x 256 tiles, several to a workgroup, ragged in rows and vocabulary."""
    P, V, d, seq, batch = 7, 8200, 512, 72, 7
    assert native.tile(seq * batch, V, d, P, heavy=True) == native.TILE_256 and 2 * 33 * P > 256
    wl = workloads.TRANSFORMER.replace(P=P, vocab=V, d_model=d, heads=8, d_ff=64, n_blocks=1, seq=seq, batch=batch, n_train=16, n_eval=batch, n_trunc=0)
    pair = TransformerPair(wl, ref_members=[0, P - 1])
    pair.gpu.eval(pair.d_eval)
    sc, ref = pair.gpu.get(binding.ARR_SCORE)[pair.ref_ids], pair.eval_ref()
    assert np.max(np.abs(np.log(-sc) - np.log(-ref))) <= TOL_BF16, (sc, ref)
