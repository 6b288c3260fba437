"""The class pipeline of the alignment at the smallest automata that take it
(256 states; fewer take the direct walk): every byte value, byte classes at
both ends of their range, whole tables in LDS with an end-of-sequence column,
empty tokens and tokens past their eighth byte, tables without a move."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def _csr(tokens):
    offsets = np.zeros(len(tokens) + 1, np.int32)
    offsets[1:] = np.cumsum([len(t) for t in tokens])
    return offsets, np.frombuffer(b"".join(tokens) or b"\0", np.uint8).copy()


def _check(trans, offsets, data, accepting=None, eos=None):
    import paper_2403_06988_amd as dv

    kw = {} if eos is None else dict(accepting=torch.from_numpy(accepting).to(DEV), eos_token=eos)
    ns, al = dv.align(torch.from_numpy(trans).to(DEV), torch.from_numpy(offsets).to(DEV),
                      torch.from_numpy(data).to(DEV), **kw)
    ns_o, al_o = (oracle.align(trans, offsets, data) if eos is None
                  else oracle.align_eos(trans, offsets, data, accepting, eos))
    np.testing.assert_array_equal(ns.cpu().numpy(), ns_o)
    np.testing.assert_array_equal(al.cpu().numpy().view(np.uint32), al_o)


@pytest.mark.parametrize("S", [256, 300, 600])
@pytest.mark.parametrize("dead_byte", [None, 0xFF, 0x00, 0x80])
def test_every_byte_value(S, dead_byte):
    """All 256 bytes live (no class left for dead bytes), or all but one (255
    classes, the dead byte's the last)."""
    rng = np.random.default_rng(5)
    trans = rng.integers(0, S, size=(S, 256)).astype(np.int32)
    if dead_byte is not None:
        trans[:, dead_byte] = -1
    toks = [bytes([b]) for b in range(256)] + [rng.integers(0, 256, 3).astype(np.uint8).tobytes() for _ in range(700)]
    toks += [bytes([0x41, b, 0x42]) for b in (0x00, 0x80, 0xFF)]
    _check(trans, *_csr(toks))


@pytest.mark.parametrize("S", [256, 300, 400])
@pytest.mark.parametrize("live", [1, 2, 20, 60, 90])
@pytest.mark.parametrize("V", [1, 31, 255, 257, 5000])
def test_few_live_columns(S, live, V):
    """Whole tables in LDS, and (from some 80 columns on) the prefix-table walk."""
    rng = np.random.default_rng(S + live + V)
    trans = np.full((S, 256), -1, np.int32)
    cols = rng.choice(256, live, replace=False)
    trans[:, cols] = np.where(rng.random((S, live)) < 0.9, rng.integers(0, S, (S, live)), -1)
    trans[rng.integers(0, S, 9), rng.integers(0, 256, 9)] = S          # out of range: dead
    lens = rng.choice([0, 1, 2, 7, 8, 9, 16, 17, 40], size=V)
    toks = [cols[rng.integers(0, live, n)].astype(np.uint8).tobytes() for n in lens]
    accepting = (rng.random(S) < 0.4).astype(np.uint8)
    offsets, data = _csr(toks)
    for eos in (None, 0, V - 1):
        _check(trans, offsets, data, accepting, eos)


def test_empty_tokens_and_dead_tables():
    rng = np.random.default_rng(1)
    S = 300
    _check(rng.integers(0, S, (S, 256)).astype(np.int32), np.zeros(70, np.int32), np.zeros(1, np.uint8))
    dead = np.full((S, 256), -1, np.int32)
    dead[2, 7] = 999                                                   # out of range: still dead
    _check(dead, *_csr([rng.integers(0, 256, n).astype(np.uint8).tobytes() for n in rng.integers(1, 12, 500)]))
