"""The two-launch training kernels (blocks of 32 rows, hidden widths up to 256)
at the edges of their blocks, channel groups, wave shares and batch splits, and
the separate kernels that wider networks still take, against the FP64 network
under the elementwise bar of test_gpu_mlp.py."""
import numpy as np
import pytest

import paper_1810_06250_amd as rs
from gpu_util import dev32, host, note
from test_gpu_mlp import PHI_SCALE, _case, _check_blocks, _oracle_grad

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu_rows():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rs.load_library()


# Batch: one row, around a 32-row block, two shares of the weight gradients
# (from 4096 rows on); channels: around the 320 held at a time, 2 nchan not a
# multiple of 64; widths: fewer hidden units than waves; (64, 40, 320, 64),
# (64, 40, 64, 320) and 1040 channels (more LDS than a CU has) are the wide
# networks.
@pytest.mark.parametrize("B,nchan,h1,h2", [(1, 33, 64, 64), (31, 320, 256, 64), (32, 321, 64, 256), (33, 64, 192, 128),
                                          (97, 700, 256, 256), (5003, 20, 128, 192), (64, 40, 320, 64),
                                          (64, 40, 64, 320), (40, 1040, 256, 256)])
def test_gradient_edges(B, nchan, h1, h2):
    note(f"mlp rows B={B} nchan={nchan} h1={h1} h2={h2}")
    w, Q, U, phi, det, p32 = _case(3 * B + nchan, B, nchan, h1, h2)
    net = rs.Mlp(nchan, h1, h2, weights=w, phi_scale=PHI_SCALE, seed=1)
    net.set_params(p32)
    args = (dev32(Q), dev32(U), dev32(phi), dev32(det))
    g, loss = net.grad(*args)
    g, loss = host(g).astype(np.float64), float(host(loss)[0])
    (l_or, l_bar), grads, _, bars = _oracle_grad(p32, w, Q, U, phi, det, nchan, h1, h2)
    assert abs(loss - l_or) <= l_bar, (loss, l_or, l_bar)
    _check_blocks(g, grads, bars, nchan, h1, h2, "grad")
    again, _ = net.grad(*args)
    np.testing.assert_array_equal(host(again).astype(np.float64), g)
    # The first Adam step moves every parameter by -lr g / (|g| + eps'), a
    # number that depends on the gradient alone: the internal gradient of
    # train_step is the one returned above.
    lr = 1e-3
    net.train_step(*args, lr)
    moved = net.get_params().astype(np.float64) - p32
    want = -lr * g / (np.abs(g) + 1e-8)
    ulp = np.spacing(np.abs(p32).astype(np.float32)).astype(np.float64)
    assert np.all(np.abs(moved - want) <= ulp + 1e-4 * lr)
    net.close()
