"""Loss head over large vocabularies (bf16): 128 statistics chunks of 2048 entries, the most that the
gradient kernel stages in LDS, 129, and 616 (above 614 chunks the stage would not fit the LDS and the call
failed). Against the oracle with test_gpu_loss's bf16 tolerance; the context stays usable.
"""
import numpy as np
import pytest

import oracle
from paper_2403_00835_amd import workload
from paper_2403_00835_amd.configs import ModelConfig
from tests.parity import log
from tests.test_gpu_loss import TOLS, _close_array, _close_rows, _grad_scales

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("vocab", [128 * 2048, 128 * 2048 + 1, 615 * 2048 + 70])
def test_loss_head_large_vocabulary(vocab):
    from paper_2403_00835_amd import binding
    cfg = ModelConfig(n_layers=1, d_model=64, n_heads=2, head_dim=32, ffn_dim=64, vocab=vocab)
    ws = workload.make_weights(cfg, seed=71)
    W = workload.as_f32(cfg, ws[-1]).astype(np.float64)
    m = binding.Model(cfg, max_ctx=64, max_block=8, max_new=8, weights=ws)
    tol = TOLS["bf16"]
    for P, A in ((2, 2), (1, 8)):  # rows of one and of two groups of eight
        log(f"[loss-vocab] {vocab} entries, P={P} A={A}")
        t, s, ar, tg = workload.make_head_rows(cfg, P, A, seed=72 + A)
        tg[-1] = vocab - 1
        g = m.loss_head(t, s, ar, tg, 0.7)
        o = oracle.loss_head(W, t, s, ar, tg, 0.7)
        _close_rows(g["kl"], o["kl"], tol, "kl")
        _close_rows(g["nll"], o["nll"], tol, "nll")
        sc_s, sc_a, _ = _grad_scales(W, t, s, ar, tg, 0.7)
        _close_array(g["d_student"], o["d_student"], sc_s, tol, "d_student")
        _close_array(g["d_ar"], o["d_ar"], sc_a, tol, "d_ar")
    m.close()
