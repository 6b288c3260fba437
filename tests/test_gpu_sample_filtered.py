"""The sampled step on rows that a filter has filled with one value so low that
it swallows the noise (-inf outside a top-k, or the type's lowest number): the
ties go to the lowest index, bit for bit against the oracle, and dense masks
of such rows cost about what other rows do."""
import numpy as np
import pytest
import torch

import oracle
from tests.gpu_common import to_oracle

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def _table(rng, S, V):
    alive = rng.random((S, V)) < np.array([0.02, 0.6, 0.95, 1.0])[np.arange(S) % 4][:, None]
    alive[3::4, : V // 2] = False                    # whole chunks and waves without a token
    ns = np.where(alive, rng.integers(0, S, (S, V)), -1).astype(np.int32)
    bits = np.zeros((S, (V + 31) // 32 * 32), bool)
    bits[:, :V] = alive
    return ns, np.packbits(bits, axis=1, bitorder="little").view("<u4").reshape(S, -1)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("B,V", [(24, 5), (24, 1003), (40, 20001), (300, 16389), (1030, 9002)])
@pytest.mark.parametrize("inv_t", [1.0, 1e-3])
def test_filled_rows(dtype, B, V, inv_t):
    import paper_2403_06988_amd as dv

    rng = np.random.default_rng(B + V)
    S = 8
    ns, al = _table(rng, S, V)
    states = (np.arange(B) % S).astype(np.int32)
    g = torch.Generator().manual_seed(V)
    low = torch.finfo(dtype).min
    # the last two at the line below which ties are passed over, and a bit above it
    fills = [(-float("inf"),), (low,), (low, -float("inf")), (-1e9,), (-1e9, -1.0625e9), (-4194304.0,), (-4000000.0,)]
    x = torch.empty((B, V), dtype=dtype)
    for b in range(B):
        fill = torch.tensor(fills[(b // S) % len(fills)], dtype=dtype)
        x[b] = fill[torch.randint(0, len(fill), (V,), generator=g)]
        if b % 3 == 0:
            x[b, torch.randint(0, V, (min(V, 50),), generator=g)] = 1.0
    args = [torch.from_numpy(a).to(DEV) for a in (ns, al.view(np.int32), states)]
    for seed in (1, 2):
        tok_o, new_o = oracle.masked_sample(ns, al, states, to_oracle(x), inv_t, seed, 3)
        tok, new = dv.masked_sample(*args, x.to(DEV), seed, 3, inv_t)
        np.testing.assert_array_equal(tok.cpu().numpy(), tok_o)
        np.testing.assert_array_equal(new.cpu().numpy(), new_o)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_filled_rows_cost_what_other_rows_do(dtype):
    """All but 50 logits of a row at -inf, against normal ones, 95 % of the
    tokens allowed.  On one card the two take 42 and 38 us at fp32, 40 and 34 at
    bf16; with every tie drawn the first took 62 and 60."""
    import paper_2403_06988_amd as dv

    rng = np.random.default_rng(1)
    S, B, V = 4, 256, 128256
    ns, al = _table(rng, S, V)
    ns[:], al[:] = ns[2], al[2]
    args = [torch.from_numpy(a).to(DEV) for a in (ns, al.view(np.int32), (np.arange(B) % S).astype(np.int32))]
    ws = dv.sample_workspace(B, V, DEV)
    out = [torch.empty(B, dtype=torch.int32, device=DEV) for _ in range(2)]
    normal = torch.randn((B, V), device=DEV).to(dtype)
    filled = torch.full((B, V), -float("inf"), dtype=dtype, device=DEV)
    filled.scatter_(1, torch.randint(0, V, (B, 50), device=DEV), normal[:, :50].contiguous())

    def us(x):
        best = 1e9
        for _ in range(5):
            t0, t1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            t0.record()
            for k in range(20):
                dv.masked_sample(*args, x, 7, k, token=out[0], new_state=out[1], workspace=ws)
            t1.record()
            t1.synchronize()
            best = min(best, t0.elapsed_time(t1) * 50)
        return best

    for x in (normal, filled):
        us(x)                                        # clocks and caches
    a, b = us(normal), us(filled)
    print(f"{dtype}: normal {a:.1f} us, filled {b:.1f} us", flush=True)
    assert b < 1.4 * a                               # 1.17 here, 1.65 and 1.81 with every tie drawn
