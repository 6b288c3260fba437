"""Rows that start off a 16-byte boundary in every launch form of the greedy
step (streamed, chosen two batches ahead, mask bytes staged in LDS), bit for
bit against the oracle: the allow row's last byte full, so that a vector's two
mask bytes reach the row's end, and allowed tokens at the ends of chunks."""
import numpy as np
import pytest
import torch

import oracle
from tests.gpu_common import to_oracle

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("B,V,pad", [
    (4, 31, 2), (3, 32, 1), (5, 4096, 3), (2, 8224, 1),   # V a multiple of 32: no spare mask bits
    (3, 20001, 0), (100, 9999, 0),
    (260, 66016, 1), (257, 65535, 0),                      # long chunks
    (1040, 16416, 1), (2050, 4099, 0),                     # many blocks per compute unit
    (2060, 33001, 0),
])
def test_shifted_rows(dtype, B, V, pad):
    import paper_2403_06988_amd as dv

    rng = np.random.default_rng(B + 3 * V)
    S, ld = 7, V + pad
    alive = rng.random((S, V)) < rng.choice([0.0005, 0.01, 0.3, 1.0], size=(S, 1))
    alive[0] = False
    alive[0, -9:] = True                     # the last vectors and the tail only
    alive[1] = False
    alive[1, :9] = True                      # the head and the first vectors only
    alive[2, V // 8: V - V // 8] = False     # a long run of unread lines
    ns = np.where(alive, rng.integers(0, S, (S, V)), -1).astype(np.int32)
    bits = np.zeros((S, (V + 31) // 32 * 32), bool)
    bits[:, :V] = alive
    al = np.packbits(bits, axis=1, bitorder="little").view("<u4").reshape(S, -1)
    states = rng.integers(-1, S, B).astype(np.int32)
    g = torch.Generator(device=DEV).manual_seed(V)
    buf = torch.randint(-3, 4, (B * ld + 8,), generator=g, device=DEV).to(dtype)  # many ties
    at = torch.randint(0, buf.numel(), (300,), generator=g, device=DEV)
    special = torch.tensor([float("nan"), float("inf"), -float("inf"), -0.0], dtype=dtype, device=DEV)
    buf[at] = special[torch.arange(300, device=DEV) % 4]
    x = buf[1:1 + B * ld].view(B, ld)[:, :V]  # the first row one element past a boundary
    args = [torch.from_numpy(a).to(DEV) for a in (ns, al.view(np.int32), states)]
    tok_o, new_o = oracle.masked_step(ns, al, states, to_oracle(x.contiguous()))
    tok, new = dv.masked_step(*args, x)
    np.testing.assert_array_equal(tok.cpu().numpy(), tok_o)
    np.testing.assert_array_equal(new.cpu().numpy(), new_o)
