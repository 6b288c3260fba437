"""The masked step's launch shapes, asked from the library's own rule, and the
greedy step at the shapes where a rule changes over."""
import ctypes
import os

import numpy as np
import pytest
import torch

import oracle
from tests.gpu_common import to_oracle

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
F32, BF16 = 0, 1
DEV = "cuda:0"


def step_shape(batch, num_tokens, dtype):
    """(vectors per chunk, chunks per row, lanes per block)"""
    lib = ctypes.CDLL(os.path.join(ROOT, "paper_2403_06988_amd", "libdv_probes.so"))
    out = [ctypes.c_int32() for _ in range(3)]
    assert lib.dvprobe_step_shape(batch, num_tokens, dtype, *[ctypes.byref(o) for o in out]) == 0
    return tuple(o.value for o in out)


@pytest.mark.parametrize("dtype", [F32, BF16])
def test_chunks_cover_every_row(dtype):
    per_vector = 4 if dtype == F32 else 8
    for V in (1, 7, 8, 1000, 4095, 4096, 4100, 8191, 24576, 24577, 32768, 33000, 50257, 128256, 258049, 1100000, 2**24):
        for B in [0, 1, 2, 3, 5, 8, 15, 16, 17, 63, 64, 65, 85, 86, 128, 129, 255, 256, 1023, 1024, 4096]:
            vectors, chunks, lanes = step_shape(B, V, dtype)
            whole = V // per_vector
            assert vectors % lanes == 0 and chunks >= 1, (B, V)
            assert vectors * chunks >= whole and vectors * (chunks - 1) < max(whole, 1), (B, V)
            assert vectors <= 32256 or dtype == F32, (B, V)     # the staged mask bytes
            if 16 <= B < 256 and V <= 258048:
                assert B * chunks <= 256, (B, V)


def test_short_fp32_rows_of_large_batches_take_few_lanes():
    for V in (1, 100, 1001, 4096):
        assert step_shape(257, V, F32)[1:] == (1, 256)
        assert step_shape(8192, V, F32)[1:] == (1, 256)
        assert step_shape(256, V, F32)[2] == 512
    assert step_shape(8192, 4100, F32)[2] == 512


@pytest.mark.gpu
@pytest.mark.parametrize("V", [1, 3, 255, 1024, 2049, 4093, 4096, 4099, 4100])
@pytest.mark.parametrize("pad", [0, 1])
def test_short_fp32_rows(V, pad):
    import paper_2403_06988_amd as dv

    rng = np.random.default_rng(V)
    B, S, ld = 1041, 6, V + pad
    alive = rng.random((S, V)) < np.array([0.0, 0.002, 0.05, 0.5, 1.0, 0.05])[:, None]
    alive[0, -1] = True
    ns = np.where(alive, rng.integers(0, S, (S, V)), -1).astype(np.int32)
    bits = np.zeros((S, (V + 31) // 32 * 32), bool)
    bits[:, :V] = alive
    al = np.packbits(bits, axis=1, bitorder="little").view("<u4").reshape(S, -1)
    states = rng.integers(-1, S, B).astype(np.int32)
    x = torch.from_numpy(rng.integers(-3, 4, (B, ld)).astype(np.float32))
    x.view(-1)[torch.from_numpy(rng.integers(0, B * ld, 300))] = float("nan")
    x[1], x[2] = -float("inf"), -0.0
    args = [torch.from_numpy(a).to(DEV) for a in (ns, al.view(np.int32), states)]
    tok_o, new_o = oracle.masked_step(ns, al, states, to_oracle(x[:, :V].contiguous()))
    tok, new = dv.masked_step(*args, x.to(DEV)[:, :V])
    np.testing.assert_array_equal(tok.cpu().numpy(), tok_o)
    np.testing.assert_array_equal(new.cpu().numpy(), new_o)
    # the same rows as the positions of sequences under verification
    if V > 3:
        b, s = 347, 2
        pos = x[: b * (s + 1), :V].reshape(b, s + 1, V).contiguous()
        props = rng.integers(0, V, (b, s)).astype(np.int32)
        got = dv.spec_verify(args[0], args[1], args[2][:b].contiguous(), torch.from_numpy(props).to(DEV), pos.to(DEV))
        want = oracle.spec_verify(ns, al, states[:b], props, to_oracle(pos))
        for g, w in zip(got, want):
            np.testing.assert_array_equal(g.cpu().numpy(), w)


@pytest.mark.parametrize("dtype,V", [(BF16, 24584), (BF16, 32000), (BF16, 32768), (F32, 12292), (F32, 16384)])
def test_rows_of_four_batches_take_two_chunks_at_most(dtype, V):
    for B in range(1, 256):
        assert step_shape(B, V, dtype)[1] == (2 if B <= 128 else 1), B


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("B,s,V", [(2, 8, 50257), (4, 3, 40000), (4, 4, 100000), (6, 8, 40001), (9, 6, 33000)])
def test_verification_of_a_few_positions(dtype, B, s, V):
    """16 to 63 positions, which are split further than a step's rows are, in a
    workspace of exactly the size asked for, left zero."""
    import paper_2403_06988_amd as dv

    rng = np.random.default_rng(B + s + V)
    S = 4
    alive = rng.random((S, V)) < np.array([0.5, 0.05, 1.0, 0.001])[:, None]
    ns = np.where(alive, rng.integers(0, S, (S, V)), -1).astype(np.int32)
    bits = np.zeros((S, (V + 31) // 32 * 32), bool)
    bits[:, :V] = alive
    al = np.packbits(bits, axis=1, bitorder="little").view("<u4").reshape(S, -1)
    states = rng.integers(0, S, B).astype(np.int32)
    x = (torch.randn(B, s + 1, V, generator=torch.Generator().manual_seed(V)) * 3).to(dtype)
    xo = to_oracle(x)
    props = np.zeros((B, s), np.int32)
    cur = states.copy()
    for j in range(s):                                        # the greedy choices, then some others
        props[:, j], cur = oracle.masked_step(ns, al, cur, np.ascontiguousarray(xo[:, j]))
    props[rng.random((B, s)) < 0.05] = 7
    t = [torch.from_numpy(a).to(DEV) for a in (ns, al.view(np.int32), states, props)]
    ws = dv.spec_workspace(B, s, V, DEV)
    want = oracle.spec_verify(ns, al, states, props, xo)
    for _ in range(2):
        got = dv.spec_verify(*t, x.to(DEV), workspace=ws)
        for g, w in zip(got, want):
            np.testing.assert_array_equal(g.cpu().numpy(), w)
        assert int(ws.count_nonzero()) == 0
