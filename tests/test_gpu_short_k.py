"""Decode products of small models at the edges of their rules: K of 64 and of 65 k-steps (the down
product in one launch or over K ranges; a depth of four or two k-steps), 240 and 264 QKV tiles and
256 and 258 gate/up tile pairs (column tiles of one or several 16-column tiles), K shorter than the
eight waves' first k-steps, in bf16 and fp32. Blocks of 1 to 64 rows take every row-group variant.

Over three row tiles the one-launch down product has 144 or 264 workgroups of 16 columns (264: it takes
32-column ones).

The logits of each step are compared with the oracle's forward over prompt and block, and a
batched step (more than 64 rows: the multi-tile products) gives the bits of the single steps.
Tolerance: the suite's (1e-4 fp32, 2e-2 bf16) on every logit, and in the 2-norm about four times the
largest measured distance (fp32 2.5e-7; bf16 5.4e-5, from keys and values near a bf16 boundary). An
operand that lost its lo plane would be 2^-9 = 2e-3 off.
"""
import numpy as np
import pytest

import oracle
from paper_2403_00835_amd import workload
from paper_2403_00835_amd.configs import ModelConfig
from tests.parity import TOL, log, rel_err

pytestmark = pytest.mark.gpu

SHAPES = {
    # bf16: 32 values a k-step
    "bf16-k64": ModelConfig(n_layers=2, d_model=768, n_heads=12, head_dim=64, ffn_dim=2048, vocab=512),
    "bf16-k65": ModelConfig(n_layers=1, d_model=1280, n_heads=20, head_dim=64, ffn_dim=2080, vocab=500),
    "bf16-wide": ModelConfig(n_layers=1, d_model=1408, n_heads=22, head_dim=64, ffn_dim=4112, vocab=512),
    "bf16-two": ModelConfig(n_layers=1, d_model=1408, n_heads=22, head_dim=64, ffn_dim=1500, vocab=512),
    "bf16-k2": ModelConfig(n_layers=2, d_model=64, n_heads=2, head_dim=32, ffn_dim=70, vocab=100),
    # fp32: 16 values a k-step
    "f32-k64": ModelConfig(n_layers=1, d_model=128, n_heads=4, head_dim=32, ffn_dim=1024, vocab=300, dtype="f32"),
    "f32-k65": ModelConfig(n_layers=1, d_model=128, n_heads=4, head_dim=32, ffn_dim=1030, vocab=300, dtype="f32"),
    "f32-two": ModelConfig(n_layers=1, d_model=1408, n_heads=22, head_dim=64, ffn_dim=600, vocab=300, dtype="f32"),
}
BLOCKS = [1, 16, 17, 33, 64]
REL = {"f32": 1e-6, "bf16": 2.5e-4}


@pytest.mark.parametrize("shape", list(SHAPES))
def test_short_k_products(shape):
    from paper_2403_00835_amd import binding
    cfg = SHAPES[shape]
    ws = workload.make_weights(cfg, seed=41)
    prompt = workload.make_prompt(cfg, 21, seed=42)
    orc = oracle.Model(cfg, [workload.as_f32(cfg, t) for t in ws])
    rng = np.random.default_rng(43)
    single = binding.Model(cfg, max_ctx=256, max_block=64, max_new=8, weights=ws)
    batched = binding.Model(cfg, max_ctx=256, max_block=64, max_new=8, max_batch=len(BLOCKS), weights=ws)
    single.debug_logits(True)
    batched.debug_logits(True)
    blocks, rows = [], []
    for m in BLOCKS:
        log(f"[short-k] {shape}: block of {m}")
        y0 = single.prefill(prompt)
        block = np.concatenate([[y0], rng.integers(0, cfg.vocab, m - 1)]).astype(np.int32)
        single.jacobi_step(block)
        lg = single.last_logits(m)
        ref = orc.forward_full(np.concatenate([prompt, block]).astype(np.int32))[len(prompt):]
        e = float(np.abs(lg - ref).max())
        assert e <= TOL[cfg.dtype], f"block of {m}: max|dlogit| {e:.4g}"
        assert rel_err(lg, ref) <= REL[cfg.dtype], f"block of {m}: {rel_err(lg, ref):.3g} of the logits' norm"
        blocks.append(block)
        rows.append(lg)
    log(f"[short-k] {shape}: batched step of {sum(BLOCKS)} rows")
    for b in range(len(BLOCKS)):
        batched.prefill(prompt, seq=b)
    batched.jacobi_step_batch(list(range(len(BLOCKS))), blocks)
    assert np.array_equal(batched.last_logits(sum(BLOCKS)), np.concatenate(rows))
    single.close()
    batched.close()
