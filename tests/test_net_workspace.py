"""The proposal network's workspace query for a very large batch (no GPU needed): answered at once."""

import ctypes
import time


def test_size_of_a_large_batch():
    from paper_1906_01413_amd.riot import _NetDesc, load_library
    lib = load_library()
    d = _NetDesc()
    d.n, d.layers, d.channels, d.k, d.width, d.segments, d.in_channels = 64, 8, 64, 64, 9, 1, 1

    def size(batch):
        d.batch_max = batch
        t0 = time.perf_counter()
        nb = lib.riot_net_workspace_bytes(ctypes.byref(d))
        return nb, time.perf_counter() - t0

    small, _ = size(1)
    large, seconds = size((1 << 31) - 1)
    # the activations of 8 layers of 64 channels, at least
    assert large > ((1 << 31) - 1) * 8 * 64 * 64 * 4 > small > 0
    assert seconds < 1.0
