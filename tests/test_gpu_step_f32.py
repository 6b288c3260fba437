"""fp32 rows of the greedy step at the edges of their launch forms, bit for bit
against the oracle: one batch and less, chunks just under and over the length
from which lines without an allowed token are skipped, an odd last vector (its
mask bits share a byte with the tail's), several chunks a row, and rows whose
allowed tokens are all NaN, -inf or signed zeros."""
import numpy as np
import pytest
import torch

import oracle
from tests.gpu_common import to_oracle

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def _table(rng, S, V):
    """next_state and allow of S states: masks of every density, the last
    tokens (past the vectors' end) often the only ones allowed."""
    alive = rng.random((S, V)) < rng.choice([0.0005, 0.02, 0.3, 1.0], size=(S, 1))
    alive[0] = False
    alive[0, max(0, V - 5):] = True
    alive[1, : V - V // 3] = False
    ns = np.where(alive, rng.integers(0, S, (S, V)), -1).astype(np.int32)
    pad = np.zeros((S, (V + 31) // 32 * 32), bool)
    pad[:, :V] = alive
    return ns, np.packbits(pad, axis=1, bitorder="little").view("<u4").reshape(S, -1)


@pytest.mark.parametrize("B,V", [
    (1, 3), (2, 4), (3, 4095), (2, 4101), (5, 8197),
    (256, 32764), (257, 32768), (256, 32773),        # one chunk a row, at the skipping threshold
    (128, 65532), (130, 65541), (64, 131079),        # two, one and four chunks
    (9, 70007), (1, 262151),                         # many chunks
])
def test_f32_step_edges(B, V):
    import paper_2403_06988_amd as dv

    rng = np.random.default_rng(17 * B + V)
    S = 8
    ns, al = _table(rng, S, V)
    states = rng.integers(-1, S, B).astype(np.int32)
    x = rng.integers(-2, 3, (B, V)).astype(np.float32)  # many ties
    bits = x.view(np.uint32)
    special = np.array([0xFFFFFFFF, 0x7FC00001, 0xFF800000, 0x80000000, 0, 0x7F800000, 0xFF800001], np.uint32)
    at = rng.integers(0, x.size, 200)
    bits.reshape(-1)[at] = special[rng.integers(0, special.size, 200)]
    bits[0] = 0xFFFFFFFF                                  # a row of the lowest fast key only
    if B > 1:
        bits[1] = special[rng.integers(0, 3, V)]          # nothing above -inf
    if B > 2:
        bits[2] = special[rng.integers(0, 5, V)]          # signed zeros at the top
    xd = torch.from_numpy(x).to(DEV)
    args = [torch.from_numpy(a).to(DEV) for a in (ns, al.view(np.int32), states)]
    tok_o, new_o = oracle.masked_step(ns, al, states, to_oracle(xd))
    tok, new = dv.masked_step(*args, xd)
    np.testing.assert_array_equal(tok.cpu().numpy(), tok_o)
    np.testing.assert_array_equal(new.cpu().numpy(), new_o)
