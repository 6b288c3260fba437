"""A workspace made for a batch serves every smaller one: the sizes that the
library asks for never fall as the batch grows, whatever number of blocks a
row is split over at each batch."""
import numpy as np
import pytest
import torch

import oracle
from tests.gpu_common import to_oracle

VOCABULARIES = [1, 1000, 8192, 16000, 24576, 24577, 32000, 32768, 33000, 50257, 70001, 128256, 256000, 258049, 600000,
                1100000, 2**24]


@pytest.mark.parametrize("V", VOCABULARIES)
@pytest.mark.parametrize("kind", ["step", "sample", "verify"])
def test_sizes_never_fall_with_the_batch(kind, V):
    import paper_2403_06988_amd as dv

    query = {"step": dv.masked_step_workspace_bytes, "sample": dv.masked_sample_workspace_bytes,
             "verify": lambda b, v: dv.spec_verify_workspace_bytes(b, 3, v)}[kind]
    sizes = [query(b, V) for b in range(0, 1101)]
    assert min(sizes) > 0
    falls = [b for b in range(1, 1101) if sizes[b] < sizes[b - 1]]
    assert not falls, falls


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("kind,made_for,batches", [("step", 80, (80, 64, 54, 1)), ("sample", 1100, (1000, 600, 512))])
def test_smaller_batches_in_a_larger_workspace(kind, made_for, batches, dtype):
    import paper_2403_06988_amd as dv

    dev = "cuda:0"
    rng = np.random.default_rng(made_for)
    S, V = 5, 128256 if kind == "step" else 32000
    alive = rng.random((S, V)) < 0.05
    ns = np.where(alive, rng.integers(0, S, (S, V)), -1).astype(np.int32)
    bits = np.zeros((S, (V + 31) // 32 * 32), bool)
    bits[:, :V] = alive
    al = np.packbits(bits, axis=1, bitorder="little").view("<u4").reshape(S, -1)
    t_ns, t_al = torch.from_numpy(ns).to(dev), torch.from_numpy(al.view(np.int32)).to(dev)
    ws = (dv.step_workspace if kind == "step" else dv.sample_workspace)(made_for, V, dev)
    for B in batches:
        states = rng.integers(0, S, B).astype(np.int32)
        x = torch.randn(B, V, generator=torch.Generator().manual_seed(B)).to(dtype)
        args = (t_ns, t_al, torch.from_numpy(states).to(dev), x.to(dev))
        if kind == "step":
            tok, new = dv.masked_step(*args, workspace=ws)
            tok_o, new_o = oracle.masked_step(ns, al, states, to_oracle(x))
        else:
            tok, new = dv.masked_sample(*args, 3, B, workspace=ws)
            tok_o, new_o = oracle.masked_sample(ns, al, states, to_oracle(x), 1.0, 3, B)
        np.testing.assert_array_equal(tok.cpu().numpy(), tok_o)
        np.testing.assert_array_equal(new.cpu().numpy(), new_o)
        assert int(ws.count_nonzero()) == 0
