"""Convolution layers of the proposal network at the edges of their tiles: every filter width, one
to 64 channels on either side (full, ragged and idle channel tiles), grids of one tile, the batches
at which a wave takes 1, 2 and 4 point tiles, and weight gradients over one and many parts, against
the FP64 oracle. The hidden biases keep every pre-activation away from zero, so that both sides
take the same ReLU decisions."""

import numpy as np
import pytest

from oracle import convnet
from synthetic import net_init
from tests._problems import rel, to_np
from tests.test_gpu_proposal import _flat, _states, _unflat

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,k,channels,width,batch,segments,cin", [
    (64, 1, 1, 1, 1, 1, 1), (64, 3, 16, 3, 2, 1, 2), (128, 16, 17, 5, 1, 4, 3),
    (64, 33, 33, 7, 3, 1, 16), (192, 64, 48, 9, 2, 16, 17), (64, 64, 64, 11, 1, 1, 64),
    (2048, 40, 64, 9, 8, 4, 6), (2048, 64, 64, 9, 16, 16, 1), (1024, 20, 32, 3, 16, 1, 5),
])
def test_layers_match_oracle(n, k, channels, width, batch, segments, cin):
    from paper_1906_01413_amd import ProposalNet
    import torch
    net = ProposalNet(n, k=k, channels=channels, layers=3, width=width, batch_max=batch,
                      segments=segments, in_channels=cin)
    params = []
    for W, b in net_init(n + k, net.layer_shapes()):
        params.append(((0.1 * W).astype(np.float32).astype(np.float64),
                       20.0 * (-1.0) ** np.arange(b.size) + 0.5))
    net.set_params(_flat(params))
    x = _states(batch, n, 3, cin)
    N = to_np(net.forward(x))
    gN = np.random.default_rng(5).standard_normal((batch, k, n)).astype(np.float32)
    got = _unflat(to_np(net.backward(torch.as_tensor(gN).cuda())), net.layer_shapes())
    ref = None
    for s in range(batch):
        Ns, acts = convnet.forward(params, x[s], segments)
        # FP32 chains of at most 64 * 11 + 1 terms, three layers: 3 sqrt(705) 2^-24 = 5e-6
        assert rel(N[s], Ns.T) < 5e-6
        gs = convnet.backward(params, acts, gN[s].astype(np.float64).T, segments)
        ref = gs if ref is None else [(a + c, b + d) for (a, b), (c, d) in zip(ref, gs)]
    for (gW, gb), (rW, rb) in zip(got, ref):
        assert rel(gW, rW) < 1e-5
        assert rel(gb, rb) < 1e-5
