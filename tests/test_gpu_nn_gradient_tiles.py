"""The network's gradient on grids at the edges of the weight gradient's 16 x
4 x 4 voxel tiles (coarse levels of one to nine voxels a side, rows of 8 and
24 voxels, several samples, more tiles than workgroups), against the FP64
oracle with every ReLU open, where only BF16 rounding of the operands
differs.  Each sum over voxels carries a rounding of 2^-9 per operand of the
sum of its terms' magnitudes, which the random signs of dy cancel: the bound
is 2e-2 (3e-2 per convolution; as in the other gradient tests) of the gradient
for |dy|, whose terms do not cancel.  Two passes give the same bits."""
import numpy as np
import pytest

from oracle import nn
from paper_1606_00548_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _bf16(a):
    u = np.asarray(a, np.float32).view(np.uint32).astype(np.uint64)
    return ((((u + 0x7FFF + ((u >> 16) & 1)) >> 16) << 16).astype(np.uint32)).view(np.float32).astype(np.float64)


def _off(a, b, size):
    return np.linalg.norm(a - b) / np.linalg.norm(size)


@pytest.mark.parametrize("batch,shape", [(3, (8, 8, 8)), (1, (8, 40, 24)), (2, (24, 8, 72)), (1, (40, 64, 64))])
def test_gradient_matches_oracle(batch, shape):
    from paper_1606_00548_amd import cprmi
    convs, head = nn.unpack(synth.nn_initial_weights(3).astype(np.float64))
    theta = _bf16(nn.pack([(0.3 * W, np.full(b.shape, 3.0)) for W, b in convs], head))
    rng = np.random.default_rng(7)
    x = rng.standard_normal((batch,) + shape + (3,)).astype(np.float32)
    dy = rng.standard_normal((batch,) + shape).astype(np.float32)
    net = cprmi.Network(shape[2], shape[1], shape[0], max_batch=batch)
    net.set_params(theta.astype(np.float32))
    got = []
    for _ in range(2):
        xg = torch.from_numpy(x).cuda()
        net.forward(xg)
        xg.zero_()     # the gradient keeps its own copy of the input
        got.append(net.backward(torch.from_numpy(dy).cuda()).cpu().numpy().astype(np.float64))
    assert np.array_equal(got[0], got[1])
    _, cache = nn.forward(theta, x.astype(np.float64))
    want = nn.backward(theta, cache, dy.astype(np.float64))
    size = nn.backward(theta, cache, np.abs(dy).astype(np.float64))
    assert _off(got[0], want, size) <= 2e-2
    o = 0
    for ci, co in nn.CONVS:
        m = 27 * ci * co
        for part in (slice(o, o + m), slice(o + m, o + m + co)):
            assert _off(got[0][part], want[part], size[part]) <= 3e-2
        o += m + co
    assert _off(got[0][o:], want[o:], size[o:]) <= 2e-2
