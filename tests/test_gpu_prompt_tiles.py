"""Prompt products at the edges of their tiles: prompts of 1 .. 513 rows whose row counts sit on both
sides of every tile choice (64- and 128-row tiles, one to four of them, several column widths) at
the LLaMA-2-7B width and at a narrow width whose column groups are ragged. The logits of each prompt's
last 64-row tile are compared with the oracle's forward over the longest prompt (a causal pass: the
rows of a prefix are the same), and a prefill in 64-row passes gives the same bits.

Tolerance: the bf16 one (2e-2) on every logit, and in the 2-norm about four times the largest measured
distance (2.9e-4 at the 7B width, 2.3e-5 at the narrow one: keys and values near a bf16 boundary). An
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
    "7b-width": ModelConfig(n_layers=1, d_model=4096, n_heads=32, head_dim=128, ffn_dim=11008, vocab=512),
    "d192": ModelConfig(n_layers=2, d_model=192, n_heads=3, head_dim=64, ffn_dim=500, vocab=1000),
}
REL = {"7b-width": 1.2e-3, "d192": 1e-4}
LENGTHS = [1, 16, 17, 64, 65, 128, 129, 192, 193, 256, 257, 385, 512, 513]


@pytest.mark.parametrize("shape", list(SHAPES))
def test_prompt_tiles_against_oracle(shape):
    from paper_2403_00835_amd import binding
    cfg = SHAPES[shape]
    ws = workload.make_weights(cfg, seed=31)
    prompt = workload.make_prompt(cfg, max(LENGTHS), seed=32)
    ref = oracle.Model(cfg, [workload.as_f32(cfg, t) for t in ws]).forward_full(prompt)
    got = {}
    for chunk in (0, 64):
        gpu = binding.Model(cfg, max_ctx=640, max_block=8, max_new=8, weights=ws, prefill_chunk=chunk)
        gpu.debug_logits(True)
        for n in LENGTHS:
            log(f"[prompt-tiles] {shape}: prefill of {n} rows, chunk {chunk}")
            gpu.prefill(prompt[:n])
            rows = (n - 1) % 64 + 1
            lg = gpu.last_logits(rows)
            if chunk == 0:
                e = float(np.abs(lg - ref[n - rows:n]).max())
                assert e <= TOL["bf16"], f"{n} rows: max|dlogit| {e:.4g}"
                r = rel_err(lg, ref[n - rows:n])
                assert r <= REL[shape], f"{n} rows: {r:.3g} of the logits' norm"
                got[n] = lg
            else:
                assert np.array_equal(lg, got[n]), f"{n} rows: 64-row passes differ"
        gpu.close()


@pytest.mark.parametrize("shape", list(SHAPES))
def test_prompt_passes_above_512_rows(shape):
    """Passes of up to 1100 rows (more than one round of the largest tile) give the bits of 64-row passes,
    which the oracle pins above."""
    from paper_2403_00835_amd import binding
    cfg = SHAPES[shape]
    ws = workload.make_weights(cfg, seed=31)
    prompt = workload.make_prompt(cfg, 1100, seed=33)
    block = workload.make_prompt(cfg, 8, seed=34)
    got = {}
    for chunk in (64, 2048):
        gpu = binding.Model(cfg, max_ctx=1200, max_block=8, max_new=8, weights=ws, prefill_chunk=chunk)
        gpu.debug_logits(True)
        for n in (513, 640, 897, 1024, 1025, 1100):
            log(f"[prompt-tiles] {shape}: prefill of {n} rows, chunk {chunk}")
            block[0] = gpu.prefill(prompt[:n])
            res = (gpu.last_logits((n - 1) % 64 + 1), gpu.hidden_rows(block))
            if chunk == 64:
                got[n] = res
            else:
                assert all(np.array_equal(a, b) for a, b in zip(res, got[n])), f"{n} rows: one pass differs"
        gpu.close()
