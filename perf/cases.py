"""The calls whose speed is measured: constrained decoding as a serving program
does it, over the sizes that this package is used at.

Four kinds of case:

  step    greedy masked decode steps, each on its own logits, the states fed
          from step to step.  With ``graph`` the steps are captured once into a
          HIP graph and replayed, as a decode loop is run (a Python call costs
          more than a small step); without, each is one eager call.
  sample  the same with sampled steps (Gumbel-max at temperature T).
  verify  greedy verification of s proposed tokens a row (speculation).
  align   the alignment table of a grammar's automaton and a vocabulary.

Sizes: batches of 1 to 1,024 sequences, vocabularies of 1,000 to 256,000
tokens (32,000, 50,257, 128,256 and 256,000 among them), automata of 16 to
8,192 states, bf16 and fp32 logits.  Everything is made from the seed:

  automata  "lexer": every state moves on a random set of 8 to 96 printable
            bytes to random states (few tokens allowed, scattered over the
            vocabulary); "union": the union of 40 such terminals behind one
            start state, accepting states chaining back (a grammar's scanner);
            "scanner": six states in ten read nearly any byte, as inside
            a string, comment or text (nearly all tokens allowed there), the
            others a few.
  tokens    the single bytes, then unique strings of printable bytes (a tenth
            of them not), 2 bytes and more with a geometric tail.
  logits    normal with deviation 3, fresh for each step.
"""
from __future__ import annotations

import ctypes
import math

import torch

import paper_2403_06988_amd as dv

DEV = "cuda"
MAX_LOGIT_BYTES = 540_000_000  # of a drawn case: no more than the largest listed step


def listed():
    return [
        # one sequence and a small model's vocabulary, one eager call: what an
        # interactive program pays for each token
        dict(name="step_1x32000_eager", kind="step", table="lexer", S=256, V=32000, B=1, dtype="bf16", steps=1, graph=False),
        # a few sequences, fp32 logits (models that return their logits widened)
        dict(name="step_8x32000_f32", kind="step", table="lexer", S=256, V=32000, B=8, dtype="f32", steps=32, graph=True),
        # a middling batch on a current tokenizer
        dict(name="step_64x128256", kind="step", table="lexer", S=1024, V=128256, B=64, dtype="bf16", steps=16, graph=True),
        # a server's batch on a union-of-terminals scanner: the benchmark's own step
        dict(name="step_256x128256", kind="step", table="union", S=8192, V=128256, B=256, dtype="bf16", steps=16, graph=True),
        # the largest step, one call
        dict(name="step_1024x256000", kind="step", table="lexer", S=4096, V=256000, B=1024, dtype="bf16", steps=1, graph=False),
        # an odd vocabulary (its rows start at every alignment), a batch that no power of two divides
        dict(name="step_100x50257", kind="step", table="scanner", S=92, V=50257, B=100, dtype="bf16", steps=16, graph=True),
        # fp32 logits at a server's sizes
        dict(name="step_128x128256_f32", kind="step", table="lexer", S=1024, V=128256, B=128, dtype="f32", steps=8, graph=True),
        # sampling where few tokens are allowed
        dict(name="sample_256x128256", kind="sample", table="union", S=8192, V=128256, B=256, dtype="bf16", steps=8, graph=True, inv_t=1.0),
        # sampling where most tokens are allowed (text inside a grammar's strings)
        dict(name="sample_64x32000_dense", kind="sample", table="scanner", S=92, V=32000, B=64, dtype="bf16", steps=16, graph=True, inv_t=1.25),
        # speculation: eight proposals a row
        dict(name="verify_256x9x128256", kind="verify", table="union", S=8192, V=128256, B=256, dtype="bf16", spec=8),
        # a user's new grammar met while serving: a small automaton, its table with the end-of-sequence column
        dict(name="align_92x32000_eos", kind="align", table="scanner", S=92, V=32000, eos=True),
        # a large grammar's table
        dict(name="align_8192x128256", kind="align", table="union", S=8192, V=128256, eos=False),
    ]


def _spread(rng, lo, hi):
    """A whole number between lo and hi, even over the logarithm."""
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choices(["step", "sample", "verify", "align"], [5, 2, 2, 2])[0]
    table = rng.choice(["lexer", "scanner", "union"])
    V = _spread(rng, 1000, 256000)
    if rng.random() < 0.3:
        V = (V + 7) // 8 * 8
    S = _spread(rng, 64 if table == "union" else 16, 512 if table == "scanner" else 4096)
    if kind == "align":
        return dict(kind=kind, table=table, S=S, V=V, eos=rng.random() < 0.5)
    dtype = rng.choice(["bf16", "bf16", "f32"])
    B = _spread(rng, 1, 1024)
    row = V * (2 if dtype == "bf16" else 4)
    if kind == "verify":
        spec = rng.randint(2, 10)
        B = max(1, min(B, 256, MAX_LOGIT_BYTES // (row * (spec + 1))))
        return dict(kind=kind, table=table, S=S, V=V, B=B, dtype=dtype, spec=spec)
    B = max(1, min(B, MAX_LOGIT_BYTES // row))
    steps = max(1, min(16, MAX_LOGIT_BYTES // 2 // (row * B)))
    case = dict(kind=kind, table=table, S=S, V=V, B=B, dtype=dtype, steps=steps, graph=steps > 1)
    if kind == "sample":
        case["inv_t"] = rng.choice([0.7, 1.0, 1.25])
    return case


# ------------------------------------------------------------------- inputs

def _generator(seed, stream):
    g = torch.Generator(device=DEV)
    g.manual_seed((int(seed) * 1_000_003 + stream * 7919 + 17) & (2**63 - 1))
    return g


def _lexer(g, S, lo, hi, target):
    """trans[S][256]: each state moves on a random set of printable bytes."""
    alphabet = torch.arange(0x20, 0x7F, device=DEV)
    n = alphabet.numel()
    size = torch.randint(lo, hi + 1, (S, 1), generator=g, device=DEV).clamp(max=n)
    rank = torch.rand((S, n), generator=g, device=DEV).argsort(1).argsort(1)
    trans = torch.full((S, 256), -1, dtype=torch.int64, device=DEV)
    trans[:, 0x20:0x7F] = torch.where(rank < size, target(g, (S, n)), -1)
    return trans


def _automaton(table, S, seed):
    """(trans[S][256] int32, accepting[S] uint8) of an automaton."""
    g = _generator(seed, 1)
    accepting = torch.rand(S, generator=g, device=DEV) < 0.25
    if table == "lexer":
        trans = _lexer(g, S, 8, 96, lambda g, shape: torch.randint(0, S, shape, generator=g, device=DEV))
    elif table == "union":
        # state 0 is the shared start; terminal k owns the states first[k] .. first[k + 1] - 1
        terms = min(40, max(1, (S - 1) // 8))
        first = 1 + torch.arange(terms + 1, device=DEV) * (S - 1) // terms
        which = torch.bucketize(torch.arange(1, S, device=DEV), first, right=True) - 1
        size, base = (first[1:] - first[:-1])[which], first[:-1][which]

        def inside(g, shape):
            u = torch.rand(shape, generator=g, device=DEV)
            return base[:, None] + torch.minimum((u * size[:, None]).long(), size[:, None] - 1)

        inner = _lexer(g, S - 1, 8, 64, inside)
        starts = inner[first[:-1] - 1]                      # [terms][256]
        has = starts >= 0
        pick = has.int().argmax(0)                          # the first terminal with a move on the byte
        start = torch.where(has.any(0), starts.gather(0, pick[None])[0], -1)
        back = accepting[1:, None] & (inner < 0)            # accepting states take the start's moves too
        trans = torch.cat([start[None], torch.where(back, start[None], inner)])
    else:  # scanner
        nd = max(1, S * 6 // 10)
        few = _lexer(g, S, 4, 40, lambda g, shape: torch.randint(0, S, shape, generator=g, device=DEV))
        dense = torch.randint(0, nd, (S, 256), generator=g, device=DEV)
        u = torch.rand((S, 256), generator=g, device=DEV)
        dense = torch.where(u < 0.7, torch.arange(S, device=DEV)[:, None], dense)  # most bytes stay in the state
        anywhere = torch.randint(0, S, (S, 256), generator=g, device=DEV)
        dense = torch.where(u > 0.99, anywhere, dense)
        dense[:, :0x20] = torch.where(u[:, :0x20] < 0.1, dense[:, :0x20], -1)      # few control bytes
        trans = torch.where((torch.arange(S, device=DEV) < nd)[:, None], dense, few)
    return trans.int().contiguous(), accepting.to(torch.uint8)


def _vocabulary(V, seed):
    """(offsets[V + 1] int32, bytes uint8): the single bytes, then unique longer strings."""
    g = _generator(seed, 2)
    singles = min(256, V // 4)
    cap = 16 if V <= 64000 else 32
    n = 2 * V + 4096
    length = 2 + (torch.log(torch.rand(n, generator=g, device=DEV).clamp_min(1e-7)) / math.log(1 - 0.22)).long()
    length = length.clamp(max=cap)
    text = torch.randint(0x20, 0x7F, (n, cap), generator=g, device=DEV)
    other = torch.randint(0, 256, (n, cap), generator=g, device=DEV)
    text = torch.where(torch.rand((n, cap), generator=g, device=DEV) < 0.9, text, other)
    inside = torch.arange(cap, device=DEV)[None] < length[:, None]
    text = torch.where(inside, text, 0)
    # one of each string: the first drawn, by a hash of its bytes and length
    mult = torch.randint(-2**62, 2**62, (cap,), generator=g, device=DEV) * 2 + 1
    key = (text * mult).sum(1) * 31 + length
    _, inverse = torch.unique(key, return_inverse=True)
    order = torch.arange(n, device=DEV)
    firsts = torch.full((n,), n, device=DEV).scatter_reduce(0, inverse, order, "amin")
    keep = (firsts[inverse] == order).nonzero()[: V - singles, 0]
    text, length = text[keep], length[keep]
    mat = torch.zeros((V, cap), dtype=torch.uint8, device=DEV)
    mat[:singles, 0] = torch.arange(singles, device=DEV)
    mat[singles:] = text
    lens = torch.ones(V, dtype=torch.int64, device=DEV)
    lens[singles:] = length
    offsets = torch.zeros(V + 1, dtype=torch.int32, device=DEV)
    offsets[1:] = lens.cumsum(0)
    return offsets, mat[torch.arange(cap, device=DEV)[None] < lens[:, None]].contiguous(), mat, lens


def _start_states(case, seed):
    return torch.randint(0, case["S"], (case["B"],), generator=_generator(seed, 3), device=DEV, dtype=torch.int32)


def _logits(case, seed, lead):
    """Normal logits [*lead][V], made one leading index at a time."""
    dtype = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
    out = torch.empty((*lead, case["V"]), dtype=dtype, device=DEV)
    g = _generator(seed, 4)
    flat = out.view(-1, case["V"])
    rows = max(1, 2**27 // case["V"])
    for r in range(0, flat.shape[0], rows):
        part = flat[r:r + rows]
        part.copy_(torch.randn(part.shape, generator=g, device=DEV).mul_(3.0))
    return out


# --------------------------------------------------------------- HIP graphs

class _Graph:
    """Launches captured by the HIP runtime's own stream capture, replayed on
    the current stream (torch's own graph capture slows the bandwidth-bound
    kernels that a process runs after it)."""

    lib = None

    @classmethod
    def runtime(cls):
        if cls.lib is None:
            vp = ctypes.c_void_p
            lib = ctypes.CDLL("libamdhip64.so")
            lib.hipStreamBeginCapture.argtypes = [vp, ctypes.c_int]
            lib.hipStreamEndCapture.argtypes = [vp, ctypes.POINTER(vp)]
            lib.hipGraphInstantiate.argtypes = [ctypes.POINTER(vp), vp, vp, ctypes.c_char_p, ctypes.c_size_t]
            lib.hipGraphLaunch.argtypes = [vp, vp]
            lib.hipGraphExecDestroy.argtypes = [vp]
            lib.hipGraphDestroy.argtypes = [vp]
            cls.lib = lib
        return cls.lib

    def __init__(self, launches):
        lib = self.runtime()
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):
            launches()  # what is set up on a first call is set up outside the capture
        torch.cuda.synchronize()
        self.graph, self.exec = ctypes.c_void_p(), ctypes.c_void_p()
        self.ok(lib.hipStreamBeginCapture(side.cuda_stream, 0))
        try:
            with torch.cuda.stream(side):
                launches()
        finally:
            rc = lib.hipStreamEndCapture(side.cuda_stream, ctypes.byref(self.graph))
        self.ok(rc)
        self.ok(lib.hipGraphInstantiate(ctypes.byref(self.exec), self.graph, None, None, 0))

    @staticmethod
    def ok(rc):
        if rc:
            raise RuntimeError("HIP graph call failed: %d" % rc)

    def replay(self):
        self.ok(self.lib.hipGraphLaunch(self.exec, torch.cuda.current_stream().cuda_stream))

    def __del__(self):
        if getattr(self, "exec", None):
            torch.cuda.synchronize()
            self.lib.hipGraphExecDestroy(self.exec)
            self.lib.hipGraphDestroy(self.graph)
            self.exec = None


# -------------------------------------------------------------------- a pass

def prepare(case, seed):
    trans, accepting = _automaton(case["table"], case["S"], seed)
    offsets, data, _, _ = _vocabulary(case["V"], seed)
    if case["kind"] == "align":
        S, V = case["S"], case["V"]
        st = dict(case=case, trans=trans, accepting=accepting, offsets=offsets, data=data)
        # tables and workspace are a program's own, kept from grammar to grammar
        st["next_state"] = torch.empty((S, V), dtype=torch.int32, device=DEV)
        st["allow"] = torch.empty((S, (V + 31) // 32), dtype=torch.int32, device=DEV)
        st["workspace"] = torch.empty(dv.align_workspace_bytes(S, V), dtype=torch.uint8, device=DEV)
        return st
    B, V, dev = case["B"], case["V"], torch.device(DEV, torch.cuda.current_device())
    next_state, allow = dv.align(trans, offsets, data)
    st = dict(case=case, next_state=next_state, allow=allow)
    if case["kind"] == "verify":
        s = case["spec"]
        logits = _logits(case, seed, (B, s + 1))
        st.update(states=_start_states(case, seed), logits=logits, proposals=_proposals(case, seed, next_state, allow, logits),
                  token=torch.empty((B, s + 1), dtype=torch.int32, device=DEV),
                  accepted=torch.empty(B, dtype=torch.int32, device=DEV),
                  new_state=torch.empty(B, dtype=torch.int32, device=DEV),
                  workspace=dv.spec_workspace(B, s, V, dev))
        return st
    steps = case["steps"]
    states = torch.empty((steps + 1, B), dtype=torch.int32, device=DEV)
    states[0] = _start_states(case, seed)
    st.update(states=states, logits=_logits(case, seed, (steps, B)), seed=int(seed),
              token=torch.empty((steps, B), dtype=torch.int32, device=DEV),
              workspace=(dv.sample_workspace if case["kind"] == "sample" else dv.step_workspace)(B, V, dev))
    st["rows"] = [(st["states"][k], st["logits"][k], st["token"][k], st["states"][k + 1]) for k in range(steps)]
    if case["graph"]:
        st["graph"] = _Graph(lambda: _steps(st))
    return st


def _proposals(case, seed, next_state, allow, logits):
    """A draft model's proposals: the greedy choice at nine positions in ten, else the next token id."""
    g = _generator(seed, 5)
    B, s, V = case["B"], case["spec"], case["V"]
    state = _start_states(case, seed)
    out = torch.empty((B, s), dtype=torch.int32, device=DEV)
    for j in range(s):
        token, state = dv.masked_step(next_state, allow, state, logits[:, j])
        wrong = torch.rand(B, generator=g, device=DEV) < 0.1
        out[:, j] = torch.where(wrong, (token + 1) % V, token)
    return out


def _steps(st):
    case = st["case"]
    for k, (state, logits, token, new_state) in enumerate(st["rows"]):
        if case["kind"] == "sample":
            dv.masked_sample(st["next_state"], st["allow"], state, logits, st["seed"], k, case["inv_t"],
                             token=token, new_state=new_state, workspace=st["workspace"])
        else:
            dv.masked_step(st["next_state"], st["allow"], state, logits, token=token, new_state=new_state,
                           workspace=st["workspace"])


def run(st):
    case = st["case"]
    if case["kind"] == "align":
        eos = dict(accepting=st["accepting"], eos_token=case["V"] - 1) if case["eos"] else {}
        return dv.align(st["trans"], st["offsets"], st["data"], next_state=st["next_state"], allow=st["allow"],
                        workspace=st["workspace"], **eos)
    if case["kind"] == "verify":
        return dv.spec_verify(st["next_state"], st["allow"], st["states"], st["proposals"], st["logits"],
                              token=st["token"], accepted=st["accepted"], new_state=st["new_state"],
                              workspace=st["workspace"])
    if case["graph"]:
        st["graph"].replay()
    else:
        _steps(st)
    return st["token"], st["states"]


def work(case):
    """Logits and mask rows read once, tokens and states written (whole rows:
    sparse masks leave some 128-byte lines of the logits unread); a table
    written once.  The choice itself is comparisons; sampling counts about 60
    operations for each allowed token's noise."""
    S, V = case["S"], case["V"]
    words = 4 * ((V + 31) // 32)
    if case["kind"] == "align":
        return {"bytes": S * (4 * V + words) + 1024 * S + 4 * V, "flops": 0}
    row = V * (2 if case["dtype"] == "bf16" else 4) + words + 16
    rows = case["B"] * (case["spec"] + 1 if case["kind"] == "verify" else case["steps"])
    share = 0.6 if case["table"] == "scanner" else 0.055
    return {"bytes": rows * row, "flops": 60 * share * rows * V if case["kind"] == "sample" else 0}


def tolerance(case):
    """Tokens, states and table entries are whole numbers and unique: the
    choice is made on exact values, ties go to the lowest index, and sampling
    noise is a fixed sequence of rounded operations."""
    return "exact"


# ----------------------------------------------------- the same, plainly, in 64 bits

def _walk(trans, mat, lens, rows):
    """Walks of every token from the states `rows`: [len(rows)][V], -1 where dead."""
    S = trans.shape[0]
    table = torch.cat([trans.long(), torch.full((1, 256), -1, device=DEV)])
    table = torch.where((table >= 0) & (table < S), table, S)  # row S: dead
    cur = rows.long()[:, None].expand(-1, mat.shape[0]).contiguous()
    for h in range(int(lens.max())):
        here = (lens > h).nonzero()[:, 0]
        cur[:, here] = table.view(-1)[cur[:, here] * 256 + mat[here, h].long()[None]]
    return torch.where(cur == S, -1, cur)


def _greedy(trans, mat, lens, states, logits):
    """(token, new state) of one greedy masked step."""
    uniq, at = torch.unique(states, return_inverse=True)
    nxt = _walk(trans, mat, lens, uniq.clamp_min(0))
    dead = (uniq < 0)[:, None]
    nxt = torch.where(dead, -1, nxt)
    token = torch.empty_like(states)
    new = torch.empty_like(states)
    for b in range(states.shape[0]):
        row = nxt[at[b]]
        x = torch.where(row >= 0, logits[b].double(), -math.inf)
        best = torch.where(row >= 0, x == x.max(), False).nonzero()[:, 0]
        token[b] = best[0] if best.numel() else -1
        new[b] = row[best[0]] if best.numel() else -1
    return token, new


def exact(case, seed):
    if case["kind"] == "sample":
        return None  # the draw is defined in binary32
    trans, accepting = _automaton(case["table"], case["S"], seed)
    _, _, mat, lens = _vocabulary(case["V"], seed)
    S, V = case["S"], case["V"]
    if case["kind"] == "align":
        next_state = torch.empty((S, V), dtype=torch.int32, device=DEV)
        for r in range(0, S, 256):
            rows = torch.arange(r, min(S, r + 256), device=DEV)
            next_state[rows] = _walk(trans, mat, lens, rows).int()
        if case["eos"]:
            next_state[:, V - 1] = torch.where(accepting != 0, torch.arange(S, device=DEV, dtype=torch.int32), -1)
        words = (V + 31) // 32
        bits = torch.zeros((S, words * 32), dtype=torch.bool, device=DEV)
        bits[:, :V] = next_state >= 0
        allow = torch.zeros((S, words), dtype=torch.int64, device=DEV)
        for j in range(32):
            allow |= bits[:, j::32].long() << j
        return next_state, torch.where(allow >= 2**31, allow - 2**32, allow).int()
    if case["kind"] == "verify":
        return None  # the same steps as below at each position
    if case["steps"] * case["B"] > 5000:
        return None  # too long, row by row
    logits = _logits(case, seed, (case["steps"], case["B"]))
    states, tokens = [_start_states(case, seed)], []
    for k in range(case["steps"]):
        token, new = _greedy(trans, mat, lens, states[-1], logits[k])
        tokens.append(token)
        states.append(new)
    return torch.stack(tokens), torch.stack(states)
