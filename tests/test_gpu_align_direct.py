"""The direct alignment walk (at most 255 states) at the edges of its tiles,
state groups and byte words, bit for bit against the oracle; 256 states take
the class pipeline and are held to the same."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def _vocabulary(rng, V):
    """Lengths around the words of 8 bytes the walk reads, empty ones among them."""
    lens = rng.choice([0, 1, 2, 7, 8, 9, 15, 16, 17, 24, 40], size=V)
    lens[-1] = rng.choice([1, 7, 8, 9])     # the last token ends the byte array
    offsets = np.zeros(V + 1, np.int32)
    offsets[1:] = np.cumsum(lens)
    return offsets, rng.integers(0, 256, int(offsets[-1])).astype(np.uint8)


@pytest.mark.parametrize("S,V", [
    (1, 1), (1, 31), (2, 64), (7, 65), (8, 255), (9, 257), (16, 1000), (17, 4097),
    (255, 300), (254, 9000), (255, 33001), (256, 33001), (40, 66000), (3, 300001),
])
@pytest.mark.parametrize("dead", [0.02, 0.5])
def test_direct_walk(S, V, dead):
    import paper_2403_06988_amd as dv

    rng = np.random.default_rng(S * 7 + V)
    trans = rng.integers(0, S, (S, 256)).astype(np.int32)
    trans[rng.random((S, 256)) < dead] = -1
    trans[rng.random((S, 256)) < 0.01] = S          # outside the automaton: dead
    trans[rng.random((S, 256)) < 0.01] = 2**31 - 1
    offsets, data = _vocabulary(rng, V)
    accepting = (rng.random(S) < 0.5).astype(np.uint8)
    # tensors whose storage starts off every wider alignment
    shifted = torch.zeros(S * 256 + 1, dtype=torch.int32, device=DEV)[1:].view(S, 256)
    shifted.copy_(torch.from_numpy(trans))
    d_bytes = torch.zeros(len(data) + 3, dtype=torch.uint8, device=DEV)[3:]
    d_bytes.copy_(torch.from_numpy(data))
    d_off = torch.from_numpy(offsets).to(DEV)
    for eos in (None, 0, V - 1):
        kw = {} if eos is None else dict(accepting=torch.from_numpy(accepting).to(DEV), eos_token=eos)
        ns, al = dv.align(shifted, d_off, d_bytes, **kw)
        ns_o, al_o = (oracle.align(trans, offsets, data) if eos is None
                      else oracle.align_eos(trans, offsets, data, accepting, eos))
        assert np.array_equal(ns.cpu().numpy(), ns_o)
        assert np.array_equal(al.cpu().numpy().view(np.uint32), al_o)


@pytest.mark.parametrize("S", [1, 17, 255])
@pytest.mark.parametrize("last", [8, 9, 16, 17, 3001])
def test_direct_walk_long_tokens(S, last):
    """Tokens of many words of 8 bytes, which are read a word ahead of the walk,
    that live to their end; the last one ends the byte array."""
    import paper_2403_06988_amd as dv

    rng = np.random.default_rng(S + last)
    trans = rng.integers(0, S, (S, 256)).astype(np.int32)
    trans[rng.random((S, 256)) < 0.002] = -1
    lens = np.array([1, 3000, 0, 7, 64, 65, 63, 255, 256, 257, 1023, 8, 24, 40, 2, last])
    offsets = np.zeros(len(lens) + 1, np.int32)
    offsets[1:] = np.cumsum(lens)
    data = rng.integers(0, 256, int(offsets[-1])).astype(np.uint8)
    ns, al = dv.align(torch.from_numpy(trans).to(DEV), torch.from_numpy(offsets).to(DEV),
                      torch.from_numpy(data).to(DEV))
    ns_o, al_o = oracle.align(trans, offsets, data)
    assert np.array_equal(ns.cpu().numpy(), ns_o)
    assert np.array_equal(al.cpu().numpy().view(np.uint32), al_o)


def test_direct_walk_decreasing_offsets_read_as_empty():
    import paper_2403_06988_amd as dv

    rng = np.random.default_rng(5)
    S = 12
    trans = rng.integers(-1, S, (S, 256)).astype(np.int32)
    offsets = np.array([0, 9, 4, 12, 12, 20], np.int32)
    data = rng.integers(0, 256, 20).astype(np.uint8)
    ns, al = dv.align(torch.from_numpy(trans).to(DEV), torch.from_numpy(offsets).to(DEV),
                      torch.from_numpy(data).to(DEV), validate=False)
    ns_o, al_o = oracle.align(trans, offsets, data)
    assert np.array_equal(ns.cpu().numpy(), ns_o)
    assert np.array_equal(al.cpu().numpy().view(np.uint32), al_o)
