"""Loss-head products at the edges of their tiles: 16, 17, 64, 65, 96 and 97 GEMM rows (gemm_kernel,
tiles of 64, 96 and 128 rows; dH changes over at 32 and 33 rows), 1 to 64 loss rows around the 32-row padding of the packed gradients, a width that is no
multiple of the 128-column tiles (320) and a vocabulary one past a 2048-entry chunk. Against the
oracle, with test_gpu_loss's bf16 tolerance (relative to the sums of absolute terms).
"""
import numpy as np
import pytest

import oracle
from paper_2403_00835_amd import workload
from paper_2403_00835_amd.configs import ModelConfig
from tests.parity import log
from tests.test_gpu_loss import TOLS, _close_array, _close_rows, _grad_scales

pytestmark = pytest.mark.gpu

CFG = ModelConfig(n_layers=1, d_model=320, n_heads=5, head_dim=64, ffn_dim=64, vocab=2049)


@pytest.fixture(scope="module")
def head():
    from paper_2403_00835_amd import binding
    ws = workload.make_weights(CFG, seed=51)
    m = binding.Model(CFG, max_ctx=64, max_block=8, max_new=8, weights=ws)
    yield m, workload.as_f32(CFG, ws[-1]).astype(np.float64)
    m.close()


@pytest.mark.parametrize("P,A", [(32, 0), (32, 1), (1, 30), (1, 31), (1, 32), (31, 33), (1, 0), (8, 0), (0, 17), (48, 0), (48, 1)])
def test_loss_head_tiles(head, P, A):
    m, W = head
    tol = TOLS["bf16"]
    t, s, ar, tg = workload.make_head_rows(CFG, P, A, seed=52 + P + A)
    log(f"[loss-tiles] P={P} A={A}: {2 * P + A} GEMM rows, {P + A} loss rows")
    g = m.loss_head(t, s, ar, tg, 0.7, want_dw=True)
    o = oracle.loss_head(W, t, s, ar, tg, 0.7)
    _close_rows(g["kl"], o["kl"], tol, "kl")
    _close_rows(g["nll"], o["nll"], tol, "nll")
    sc_s, sc_a, sc_w = _grad_scales(W, t, s, ar, tg, 0.7)
    _close_array(g["d_student"], o["d_student"], sc_s, tol, "d_student")
    _close_array(g["d_ar"], o["d_ar"], sc_a, tol, "d_ar")
    _close_array(g["d_W"], o["d_W"], sc_w, tol, "d_W")


@pytest.mark.parametrize("off", [1, 2, 3])
def test_loss_head_device_unaligned_arrays(head, off):
    """Slices of a flat buffer at any float offset: the results of aligned arrays, nothing beside them."""
    import torch
    m, _ = head
    P, A, d, V = 5, 4, CFG.d_model, CFG.vocab
    t, s, ar, tg = workload.make_head_rows(CFG, P, A, seed=53)
    h = m.loss_head(t, s, ar, tg, 0.7, want_dw=True)

    def at(values):
        flat = torch.full((off + values.size + 4,), 7.0, device="cuda")
        flat[off:off + values.size] = torch.from_numpy(values.ravel()).cuda()
        return flat, flat[off:off + values.size].view(values.shape)

    ins = [at(x)[1] for x in (t, s, ar)]
    outs = [at(np.zeros(n, np.float32)) for n in ((P,), (A,), (P, d), (A, d), (V, d))]
    loss = torch.zeros(1, dtype=torch.float64, device="cuda")
    TG = torch.from_numpy(tg).cuda()
    torch.cuda.synchronize()
    log(f"[loss-tiles] arrays {off} floats past an aligned address")
    m.loss_head_device(P, A, 0.7, *ins, TG, *(o[1] for o in outs), loss)
    torch.cuda.synchronize()
    for (flat, view), key in zip(outs, ("kl", "nll", "d_student", "d_ar", "d_W")):
        assert np.array_equal(view.cpu().numpy(), h[key]), key
        assert bool((flat[:off] == 7.0).all()) and bool((flat[off + view.numel():] == 7.0).all()), key
    assert loss.item() == h["loss"]
