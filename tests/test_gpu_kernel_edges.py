"""The kernels' own edges: sizes at which a dispatch rule changes sides or a tile is partly filled,
against the CPU oracle (codes, scales and integer sums bit for bit)."""
import numpy as np
import pytest
import torch

import oracle
from paper_2503_06545_amd import binding as qc
from test_gpu_parity import bits_equal, dev, random_x

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("M,K", [(1, 16), (9, 112), (8, 128), (7, 144), (9, 2032), (9, 2048), (9, 2064),
                                 (5, 6144), (5, 6160), (4609, 2048), (4610, 2048)])
def test_row_quantizers_at_the_edges_of_their_column_slices(M, K, dtype):
    """Eight lanes take 128 columns of a row per step, a wavefront one, three or nine steps: a last
    step that is partly or wholly past the row, and both sides of K = 2048, K = 6144 and
    M K = 8192 * 1152, where the number of steps changes."""
    rng = np.random.default_rng(M * 10007 + K)
    x = random_x(rng, M, K, dtype)
    q_ref, s_ref = oracle.quant_act(x)
    a_ref = oracle.quant_act_asym(x)
    qx, sx = qc.quant_act_t(dev(x))
    qa = qc.quant_act_asym_t(dev(x))
    torch.cuda.synchronize()
    assert bits_equal(sx.cpu().numpy(), s_ref) and np.array_equal(qx.cpu().numpy(), q_ref)
    assert np.array_equal(qa[0].cpu().numpy(), a_ref[0])
    assert bits_equal(qa[1].cpu().numpy(), a_ref[1]) and bits_equal(qa[2].cpu().numpy(), a_ref[2])
    if K % 16 == 0:
        r_ref = oracle.quant_act_rot(x, 16, 8)
        qr, sr = qc.quant_act_t(dev(x), 8, 16)
        assert bits_equal(sr.cpu().numpy(), r_ref[1]) and np.array_equal(qr.cpu().numpy(), r_ref[0])
