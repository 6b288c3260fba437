"""The sampled step where tokens are passed over by a bound of their key: dense
masks (groups of four tokens), rows at every alignment and length modulo four,
every launch form, and rows where no finite key can rule a token out, bit for
bit against the oracle."""
import numpy as np
import pytest
import torch

import oracle
from tests.gpu_common import to_oracle

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("B,V,pad", [
    (1, 1, 0), (2, 2, 1), (3, 3, 0), (5, 4, 1), (4, 5, 0), (3, 63, 0), (7, 66, 1),   # one group, the last group short
    (6, 4099, 0), (40, 16385, 2), (64, 9001, 0),      # half a mask word per lane
    (300, 16389, 1), (130, 40003, 0),                 # a whole word per lane
    (1030, 4102, 1), (1024, 33001, 0),                # a block per row
])
@pytest.mark.parametrize("inv_t", [1.0, 3.0e38, 1e-30])
def test_sample_bounds(dtype, B, V, pad, inv_t):
    import paper_2403_06988_amd as dv

    rng = np.random.default_rng(B + 5 * V)
    S, ld = 9, V + pad
    alive = rng.random((S, V)) < np.array([0, 0.01, 0.1, 0.3, 0.5, 0.8, 1, 1, 1])[:, None]
    alive[0, -3:] = True                              # the short last group only
    ns = np.where(alive, rng.integers(0, S, (S, V)), -1).astype(np.int32)
    bits = np.zeros((S, (V + 31) // 32 * 32), bool)
    bits[:, :V] = alive
    al = np.packbits(bits, axis=1, bitorder="little").view("<u4").reshape(S, -1)
    states = rng.integers(-1, S, B).astype(np.int32)
    g = torch.Generator().manual_seed(B + V)
    flat = torch.empty(B * ld + 1, dtype=dtype, device=DEV)[1:]      # off every wider alignment
    x = flat.view(B, ld)
    x.copy_(torch.randn(B, ld, generator=g) * 3)
    for r, values in enumerate([(-np.inf,), (np.nan,), (np.nan, -np.inf), (np.inf, 0.0), (-3e38,), (-0.0, 0.0)]):
        if r + 1 < B:                                                # rows without a key that rules tokens out
            pick = torch.randint(0, len(values), (ld,), generator=g)
            x[r + 1].copy_(torch.tensor(values, dtype=torch.float32)[pick])
            states[r + 1] = 5 + r % 4
    t_ns, t_al = torch.from_numpy(ns).to(DEV), torch.from_numpy(al.view(np.int32)).to(DEV)
    xs = to_oracle(x)
    for offset in (0, 2**33 + 7):
        tok_o, new_o = oracle.masked_sample(ns, al, states, xs, inv_t, 11, offset)
        tok, new = dv.masked_sample(t_ns, t_al, torch.from_numpy(states).to(DEV), x[:, :V], 11, offset, inv_t)
        np.testing.assert_array_equal(tok.cpu().numpy(), tok_o)
        np.testing.assert_array_equal(new.cpu().numpy(), new_o)
