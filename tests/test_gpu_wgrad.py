"""Weight gradients at the grids and batches where the tiling of their kernels
can go wrong: the smallest grid (one row of tiles, halos that wrap onto
themselves), fewer tiles than workgroups, tile counts that do and do not split
over the XCDs, several samples, against the BF16-emulating oracle.

Bars: relative L2 norm per tensor 2e-3 and every entry within 2e-2 |ref| + 2e-3
max |ref|, the rounding of one BF16 value stored between the layers (2^-8 of
it), as for the whole network's gradients."""
import numpy as np
import pytest

from oracle import nn_oracle as NO

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny,batch", [(32, 16, 1), (32, 32, 3), (64, 16, 1), (32, 64, 2), (128, 32, 5)])
def test_gradients_vs_oracle(nx, ny, batch):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1804_02883_amd import Trainer
    print(f"[wgrad] {nx}x{ny} batch {batch}", flush=True)
    rng = np.random.default_rng(nx + 7 * ny + batch)
    params = [(rng.standard_normal((9, ci, co)) / np.sqrt(9 * ci), 0.1 * rng.standard_normal(co))
              for ci, co in ((5, 64), (64, 64), (64, 64), (64, 2))]
    flat = np.concatenate([np.concatenate([W.ravel(), b]) for W, b in params]).astype(np.float32)
    tr = Trainer(nx, ny, batch + 1, batch)
    tr.set_weights(flat)
    slots = np.arange(batch)[::-1] + 1  # not the order of the data
    rp = NO.round_params([(W.astype(np.float32).astype(float), b) for W, b in params], NO.bf16_round)
    ref = None
    for s in slots:
        w = 0.3 * rng.standard_normal((3, ny, nx))
        ph = 0.05 + 0.02 * rng.random((2, ny, nx))
        tr.set_pair(int(s), w, ph, 0.5, 32)
        o, cache = NO.forward(rp, NO.bf16_round(NO.make_input(w, 0.5, 32)), NO.bf16_round)
        _, go = NO.loss_and_grad_output(o, np.moveaxis(ph.astype(np.float32).astype(float), 0, -1), 0.1)
        g = NO.backward(rp, cache, go / batch, NO.bf16_round)
        ref = g if ref is None else [(a + c, b + d) for (a, b), (c, d) in zip(ref, g)]
    _, _, grad = tr.evaluate(slots, 0.1, grad=True)
    tr.close()
    off = 0
    for l, (W, b) in enumerate(ref):
        for r in (W.ravel(), b):
            d = grad[off:off + r.size].astype(float) - r
            off += r.size
            assert np.linalg.norm(d) <= 2e-3 * np.linalg.norm(r), (l, np.linalg.norm(d) / np.linalg.norm(r))
            assert np.all(np.abs(d) <= 2e-2 * np.abs(r) + 2e-3 * np.abs(r).max()), l
