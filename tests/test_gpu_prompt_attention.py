"""Attention of prompt rows at the edges of its tiles: head widths 32, 64 and 128 (and 256, which
keeps the chunk-parallel pair), prompts of 1 to 257 rows on both sides of the 16-row groups, the
64-row workgroups and the pairs of 64-key chunks. The logits of the last 64-row tile are compared
with the oracle's forward; a prefill in 64-row passes (rows behind a committed context) gives the same
bits, there and in the logits of a step over the caches it left; and the caches of a pass shared by
several prompts give the rows of a block the same bits as a prefill of its own.

Tolerance: the suite's bf16 one (2e-2) on every logit, and in the 2-norm about four times the largest
measured distance (1.1e-4: keys and values near a bf16 boundary). Probabilities or queries that lost
their lo plane would be 2^-9 = 2e-3 off.
"""
import numpy as np
import pytest

import oracle
from paper_2403_00835_amd import workload
from paper_2403_00835_amd.configs import ModelConfig
from tests.parity import TOL, log, rel_err

pytestmark = pytest.mark.gpu

REL = 4.5e-4
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
            block[0] = y0
            gpu.jacobi_step(block)
            if chunk == 0:
                e = float(np.abs(lg - ref[n - rows:n]).max())
                assert e <= TOL["bf16"], f"{n} rows: max|dlogit| {e:.4g}"
                assert rel_err(lg, ref[n - rows:n]) <= REL, f"{n} rows: {rel_err(lg, ref[n - rows:n]):.3g}"
                got[n] = lg
                step[n] = gpu.last_logits(8)
            else:
                assert np.array_equal(lg, got[n]), f"{n} rows: 64-row passes differ"
                assert np.array_equal(gpu.last_logits(8), step[n]), f"{n} rows: the caches of 64-row passes differ"
        gpu.close()
    _check_shared_pass(cfg, ws, prompt, [1, 63, 65, 128, 193], block, 0)


def _check_shared_pass(cfg, ws, prompt, lens, block, chunk):
    """Ragged prompts through shared passes (a batched decode of one token), then the rows of a block
    on each slot: those of a prefill of its own, brought to the same committed length."""
    from paper_2403_00835_amd import binding
    opts = dict(max_ctx=max(lens) + 80, max_block=8, max_new=8, weights=ws, prefill_chunk=chunk)
    bat = binding.Model(cfg, max_batch=len(lens), **opts)
    bat.jacobi_decode_batch(list(range(len(lens))), [prompt[:n] for n in lens], 8, 1, None)
    one = binding.Model(cfg, **opts)
    for q, n in enumerate(lens):
        one.prefill(prompt[:n])
        L, pending = one.seq_state()
        assert L == n
        while L < bat.seq_state(q)[0]:
            one.jacobi_step(np.array([pending], np.int32))
            L, pending = one.seq_state()
        assert (L, pending) == bat.seq_state(q)
        block[0] = pending
        assert np.array_equal(bat.hidden_rows(block, seq=q), one.hidden_rows(block)), f"{n} rows: the shared pass differs"
    one.close()
    bat.close()


LONG = [768, 769, 1024, 1025, 1537, 2047, 2048, 2049, 2300]  # a split launch begins at 769 keys


@pytest.mark.parametrize("hd", [32, 64, 128])
def test_prompt_attention_long_contexts(hd):
    """Rows behind up to 2300 keys: one pass of the whole prompt (more than 32 tiles of 4 heads: one
    walk), 512-row passes and 64-row passes (split into pieces, from one row up). The logits of the last
    tile against the oracle, and the same bits whatever the passes."""
    from paper_2403_00835_amd import binding
    heads = 4
    cfg = ModelConfig(n_layers=2, d_model=heads * hd, n_heads=heads, head_dim=hd, ffn_dim=192, vocab=500)
    ws = workload.make_weights(cfg, seed=64)
    prompt = workload.make_prompt(cfg, max(LONG), seed=65)
    block = workload.make_prompt(cfg, 8, seed=66)
    ref = oracle.Model(cfg, [workload.as_f32(cfg, t) for t in ws]).forward_full(prompt)
    got, rows_got = {}, {}
    for chunk in (4096, 512, 64):
        gpu = binding.Model(cfg, max_ctx=2400, max_block=8, max_new=8, weights=ws, prefill_chunk=chunk)
        gpu.debug_logits(True)
        for n in LONG:
            log(f"[prompt-attn] hd {hd}: {n} keys, chunk {chunk}")
            block[0] = gpu.prefill(prompt[:n])
            rows = (n - 1) % 64 + 1
            lg = gpu.last_logits(rows)
            hr = gpu.hidden_rows(block)
            if chunk == 4096:
                e = float(np.abs(lg - ref[n - rows:n]).max())
                assert e <= TOL["bf16"], f"{n} keys: max|dlogit| {e:.4g}"
                assert rel_err(lg, ref[n - rows:n]) <= REL, f"{n} keys: {rel_err(lg, ref[n - rows:n]):.3g}"
                got[n], rows_got[n] = lg, hr
            else:
                assert np.array_equal(lg, got[n]), f"{n} keys: passes of {chunk} rows differ"
                assert np.array_equal(hr, rows_got[n]), f"{n} keys: the caches of passes of {chunk} rows differ"
        gpu.close()
    _check_shared_pass(cfg, ws, prompt, [1100, 3, 2100, 769, 130], block, 512)
