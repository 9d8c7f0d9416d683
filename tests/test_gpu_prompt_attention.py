"""Attention of prompt rows at the edges of its tiles: head widths 32, 64 and 128 (and 256, which
keeps the chunk-parallel pair), prompts of 1 to 257 rows on both sides of the 16-row groups, the
64-row workgroups and the pairs of 64-key chunks. The logits of the last 64-row tile are compared
with the oracle's forward, a prefill in 64-row passes (rows behind a committed context) gives the
same bits, and so does a pass shared by several prompts (compared through the logits of a step
over the caches it left).

Tolerance: the suite's bf16 one (2e-2); two layers stay an order of magnitude below.
"""
import numpy as np
import pytest

import oracle
from paper_2403_00835_amd import workload
from paper_2403_00835_amd.configs import ModelConfig
from tests.parity import TOL, log

pytestmark = pytest.mark.gpu

LENGTHS = [1, 15, 17, 63, 64, 65, 127, 128, 129, 191, 193, 257]


@pytest.mark.parametrize("hd", [32, 64, 128, 256])
def test_prompt_attention(hd):
    from paper_2403_00835_amd import binding
    cfg = ModelConfig(n_layers=2, d_model=256, n_heads=256 // hd, head_dim=hd, ffn_dim=320, vocab=500)
    ws = workload.make_weights(cfg, seed=61)
    prompt = workload.make_prompt(cfg, max(LENGTHS), seed=62)
    ref = oracle.Model(cfg, [workload.as_f32(cfg, t) for t in ws]).forward_full(prompt)
    block = workload.make_prompt(cfg, 8, seed=63)
    got, step = {}, {}
    for chunk in (0, 64):
        gpu = binding.Model(cfg, max_ctx=320, max_block=8, max_new=8, weights=ws, prefill_chunk=chunk)
        gpu.debug_logits(True)
        for n in LENGTHS:
            log(f"[prompt-attn] hd {hd}: prefill of {n} rows, chunk {chunk}")
            y0 = gpu.prefill(prompt[:n])
            rows = (n - 1) % 64 + 1
            lg = gpu.last_logits(rows)
            if chunk == 0:
                e = float(np.abs(lg - ref[n - rows:n]).max())
                assert e <= TOL["bf16"], f"{n} rows: max|dlogit| {e:.4g}"
                got[n] = lg
                block[0] = y0
                gpu.jacobi_step(block)
                step[n] = (block.copy(), gpu.last_logits(8))
            else:
                assert np.array_equal(lg, got[n]), f"{n} rows: 64-row passes differ"
        gpu.close()
    # one pass shared by ragged prompts, then a step on each slot
    lens = [1, 63, 65, 128, 193]
    bat = binding.Model(cfg, max_ctx=320, max_block=8, max_new=8, max_batch=len(lens), weights=ws)
    bat.debug_logits(True)
    bat.jacobi_decode_batch(list(range(len(lens))), [prompt[:n] for n in lens], 8, 1, None)
    for q, n in enumerate(lens):
        rows = bat.hidden_rows(step[n][0], seq=q)  # behind the decode's one committed token
        one = binding.Model(cfg, max_ctx=320, max_block=8, max_new=8, weights=ws)
        one.jacobi_decode(prompt[:n], 8, 1)
        assert np.array_equal(rows, one.hidden_rows(step[n][0])), f"{n} rows: the shared pass differs"
        one.close()
    bat.close()
