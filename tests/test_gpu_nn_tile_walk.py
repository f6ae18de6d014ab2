"""Convolutions whose workgroups walk over several tiles, with shares that
differ by one tile and partial tiles at every edge (120x72x40, five samples:
7,200 full-resolution tiles over 1,024 workgroups, 900 half-resolution tiles
over 512 and 256).  Copies of one sample pass through different workgroups and
places in their walks and must come out bit for bit alike; a single sample,
whose half-resolution levels split the K-steps over waves instead, agrees to
3e-2 in the relative 2-norm, the tolerance of BF16 activations in the other
network tests, and so do a fifth of the batch's gradient and its own (every
ReLU open, dy positive: no mask flips, no cancellation).  The inference form,
whose head is fused and sums in another order, agrees to 1e-5 (16 products in
FP32, a condition of at most ten)."""
import numpy as np
import pytest

from oracle import nn
from paper_1606_00548_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

NX, NY, NZ, COPIES = 120, 72, 40, 5


def _rel(a, b):
    return float((a - b).norm() / b.norm())


def test_copies_of_a_sample_agree():
    from paper_1606_00548_amd import cprmi
    convs, head = nn.unpack(synth.nn_initial_weights(3).astype(np.float64))
    theta = nn.pack([(0.3 * W, np.full(b.shape, 3.0)) for W, b in convs], head)
    rng = np.random.default_rng(11)
    x = torch.from_numpy(rng.standard_normal((1, NZ, NY, NX, 3)).astype(np.float32)).cuda()
    dy = torch.from_numpy(np.abs(rng.standard_normal((1, NZ, NY, NX))).astype(np.float32)).cuda()
    net = cprmi.Network(NX, NY, NZ, max_batch=COPIES)
    net.set_params(theta.astype(np.float32))
    one = net.forward(x).clone()
    g_one = net.backward(dy).clone()
    assert _rel(net.infer(x), one) <= 1e-5
    many = net.forward(x.repeat(COPIES, 1, 1, 1, 1).contiguous()).clone()
    g_many = net.backward(dy.repeat(COPIES, 1, 1, 1).contiguous()).clone()
    for c in range(1, COPIES):
        assert torch.equal(many[c], many[0])
    assert _rel(many[0], one[0]) <= 3e-2
    assert _rel(g_many / COPIES, g_one) <= 3e-2
