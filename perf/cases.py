"""The work a program on this library has it do, as cases that can be timed and compared.

A case is a plain dict: the model's shape, how the cache is laid out and what one pass asks for.  A pass is what a
serving or fine-tuning program does on a long-lived cache; its new messages are freed at the end, as a workflow's are
once it is over, which also makes a pass repeatable:

  decode   n_calls parallel generations: one append of their one-token tails, then `steps` times pc_decode_step (one
           token per tail and the attention of all calls)
  prefill  one append of the new messages, one pc_attend of their calls (and of `decodes` one-row calls beside them)
  rounds   every round each agent appends a message and attends to all of the earlier rounds, its own messages last
  train    a prefill that keeps the log-sum-exp, zeroed gradients, pc_attend_backward, pc_grad_keys_finalize

Layouts (message lengths, which call lists what and where) follow from the case; K, V, Q and the output gradients,
N(0,1) like in this repository's workloads, from the seed.
"""
import ctypes

import numpy as np
import torch

from paper_2512_23049_amd.binding import PC_BF16, PC_F32, Cache, pc_call, pc_sel

IDS = 1 << 18                          # a message id is never given out twice: room for the messages of many passes
DEV = "cuda:0"


# ------------------------------------------------------------------------------------------------------- the cases
def _b8(**kw):                         # 8B-shaped attention
    return dict(heads=32, kv_heads=8, dim=128, dtype="bf16", theta=500000.0, **kw)


def _b70(**kw):                        # 70B-shaped attention
    return dict(heads=64, kv_heads=8, dim=128, dtype="bf16", theta=500000.0, **kw)


def listed():
    return [
        # a few agents generate after a short common prompt: launches and host work count
        _b8(name="decode_few", kind="decode", layout=11, shared=300, pool=16, len_lo=40, len_hi=300, n_sel=3, n_calls=4, steps=16),
        # one generation over a long history: the whole chip serves one query token
        _b70(name="decode_one_long", kind="decode", layout=12, shared=0, pool=160, len_lo=64, len_hi=256, n_sel=150, n_calls=1, steps=8),
        # the parallel decode workload: a system message, 8 of 512 pool messages and a tail of its own per call
        _b8(name="decode_parallel", kind="decode", layout=13, shared=2048, pool=512, len_lo=128, len_hi=512, n_sel=8, n_calls=64, steps=8),
        # long-context generation: 32 calls over the same messages (about 64k tokens each) in orders of their own
        _b70(name="decode_long_shared", kind="decode", layout=14, shared=0, pool=512, len_lo=64, len_hi=256, n_sel=410, n_calls=32, steps=4),
        # a short ragged message after a few others: the small everyday prefill
        _b8(name="prefill_short", kind="prefill", layout=21, pool=12, len_lo=30, len_hi=400, n_sel=5, n_new=1, new_lo=77, new_hi=77, decodes=0),
        # the single-call prefill workload: 512 new tokens over about 8k listed ones
        _b8(name="prefill_single", kind="prefill", layout=22, pool=256, len_lo=64, len_hi=1024, n_sel=16, n_new=1, new_lo=512, new_hi=512, decodes=0),
        # the multi-agent workload: appends and prefills interleaved
        _b8(name="rounds", kind="rounds", layout=23, agents=8, rounds=6, msg_len=256),
        # the long-context workload: a 2048-row prefill and 32 one-row calls in one batch
        _b70(name="long_mixed", kind="prefill", layout=24, pool=512, len_lo=64, len_hi=256, n_sel=410, n_new=1, new_lo=2048, new_hi=2048, decodes=32),
        # reference precision: the tiny configuration, and a scaled single prefill with 8B-shaped heads
        dict(name="tiny_fp32", kind="prefill", heads=4, kv_heads=2, dim=64, dtype="f32", theta=10000.0, layout=31, pool=8, len_lo=16, len_hi=64,
             n_sel=4, n_new=1, new_lo=32, new_hi=32, decodes=0),
        dict(name="prefill_fp32", kind="prefill", heads=32, kv_heads=8, dim=128, dtype="f32", theta=500000.0, layout=32, pool=24, len_lo=40,
             len_hi=300, n_sel=6, n_new=1, new_lo=200, new_hi=200, decodes=0),
        # fine-tuning on a workflow trace, forward and backward: four new messages over shared cached ones
        _b8(name="train_bf16", kind="train", layout=41, pool=16, len_lo=64, len_hi=512, n_sel=7, n_new=4, new_lo=150, new_hi=320),
        # the same at reference precision and the size it is checked at
        dict(name="train_fp32", kind="train", heads=8, kv_heads=2, dim=64, dtype="f32", theta=10000.0, layout=42, pool=10, len_lo=20, len_hi=200,
             n_sel=5, n_new=2, new_lo=50, new_hi=110),
    ]


def draw(rng):
    def log(lo, hi):
        return int(round(lo * (hi / lo) ** rng.random()))
    layout = rng.randrange(1000, 1 << 30)
    lo = log(16, 200)
    lens = dict(layout=layout, len_lo=lo, len_hi=lo + log(8, 800))

    def history(most, pool_most=512):                    # how many messages a call lists for about that many tokens, of how many
        n_sel = max(1, min(pool_most // 2, 2 * log(min(50, most), most) // (lens["len_lo"] + lens["len_hi"])))
        return dict(n_sel=n_sel, pool=min(pool_most, n_sel + log(1, 3 * n_sel + 8)), **lens)
    shape = rng.choice((_b8, _b70))
    kind = rng.choice(("decode", "decode", "prefill", "prefill", "rounds", "train", "f32"))
    if kind == "decode":
        calls = log(1, 64)
        return shape(kind="decode", shared=rng.choice((0, log(64, 2048))), n_calls=calls, steps=log(2, 16), **history(min(65536, 600000 // calls)))
    if kind == "prefill":
        n_new = rng.choice((1, 1, 2, log(2, 8)))
        new = log(17, max(20, 2048 // n_new))
        return shape(kind="prefill", n_new=n_new, new_lo=max(17, new // 2), new_hi=new, decodes=rng.choice((0, 0, log(1, 32))), **history(40000))
    if kind == "rounds":
        return shape(kind="rounds", layout=layout, agents=rng.randint(2, 8), rounds=rng.randint(2, 6), msg_len=log(24, 300))
    if kind == "train" and rng.random() < 0.5:
        new = log(24, 320)
        return _b8(kind="train", n_new=rng.randint(1, 4), new_lo=max(10, new // 2), new_hi=new, **history(3000, 32))
    f32 = dict(dtype="f32", theta=10000.0, kv_heads=rng.choice((2, 4)), dim=rng.choice((64, 128)))
    new = log(8, 110 if kind == "train" else 300)
    if kind == "train":
        return dict(f32, kind="train", heads=8, n_new=rng.randint(1, 3), new_lo=max(4, new // 2), new_hi=new, **history(800, 32))
    return dict(f32, kind="prefill", heads=rng.choice((4, 8, 32)), n_new=rng.randint(1, 2), new_lo=max(4, new // 2), new_hi=new,
                decodes=rng.choice((0, 4)), **history(2000, 32))


# ------------------------------------------------------------------------------------------------------ the layout
def _layout(case):
    """(lengths of the cached messages, phases).  A phase: the lengths and reserves of the messages appended in it and
    its calls (sel, self, start, n_q); sel: [(kind, index, start)], kind 0 a cached message, 1 the index-th new message
    of the pass; self: index of the call's new message among those of the pass."""
    r = np.random.default_rng(case["layout"])
    kind = case["kind"]
    if kind == "rounds":
        A, L = case["agents"], case["msg_len"]
        phases = []
        for t in range(case["rounds"]):
            calls = []
            for a in range(A):
                others = [rr * A + aa for rr in range(t) for aa in range(A) if aa != a]
                order = [others[int(i)] for i in r.permutation(len(others))] + [rr * A + a for rr in range(t)]
                calls.append(([(1, m, i * L) for i, m in enumerate(order)], t * A + a, len(order) * L, L))
            phases.append(([L] * A, [L] * A, calls))
        return [], phases
    lens = [int(x) for x in r.integers(case["len_lo"], case["len_hi"] + 1, size=case["pool"])]
    first = 0
    if case.get("shared", 0) > 0:
        lens.insert(0, case["shared"])
        first = 1

    def one_list(overlap):
        sel, at = [], 0
        if first:
            sel.append((0, 0, 0))
            at = lens[0]
        for i in r.permutation(case["pool"])[:case["n_sel"]]:
            m = int(i) + first
            at += -int(r.integers(0, min(32, lens[m]) // 2 + 1)) if overlap else int(r.integers(0, 33))     # overlapping, or with gaps
            at = max(at, 0)
            sel.append((0, m, at))
            at += lens[m]
        return sel, at
    overlap = case["n_sel"] > 64
    if kind == "decode":
        n, steps = case["n_calls"], case["steps"]
        calls = []
        for c in range(n):
            sel, at = one_list(overlap)
            calls.append((sel, c, at, 1))
        return lens, [([1] * n, [1 + steps] * n, calls)]
    decodes = case.get("decodes", 0)
    new = [int(x) for x in r.integers(case["new_lo"], case["new_hi"] + 1, size=case["n_new"])]
    calls = []
    for c, L in enumerate([1] * decodes + new):
        sel, at = one_list(overlap)
        calls.append((sel, c, at, L))
    return lens, [([1] * decodes + new, [1] * decodes + new, calls)]


def _tokens(lens, new, call):
    return sum((lens if k == 0 else new)[m] for k, m, _ in call[0])


def work(case):
    lens, phases = _layout(case)
    es = 2 if case["dtype"] == "bf16" else 4
    kv = 2 * case["kv_heads"] * case["dim"] * es                                   # one token's K and V
    row = case["heads"] * case["dim"] * es                                         # one query or output row
    per_pair = 4 * case["dim"] * case["heads"]
    new = [L for ph in phases for L in ph[0]]
    steps = case["steps"] if case["kind"] == "decode" else 1
    by = fl = 0
    for ph_new, _, calls in phases:
        by += 2 * kv * sum(ph_new)                                                 # appended: read and written
        old = {(k, m) for c in calls for k, m, _ in c[0]}
        listed_once = sum((lens if k == 0 else new)[m] for k, m in old)
        for s in range(steps):
            grown = s + 1 if case["kind"] == "decode" else 0
            own = sum(new[c[1]] + grown for c in calls)
            by += kv * (listed_once + own) + 2 * row * sum(c[3] for c in calls) + (2 * kv * len(calls) if grown else 0)
            for c in calls:
                n = c[3]
                fl += per_pair * (n * (_tokens(lens, new, c) + new[c[1]] + grown) - n * (n - 1) // 2)
    if case["kind"] == "train":                                                    # S, dP, dQ, dK, dV besides the forward
        pairs = fl // per_pair
        fl += 10 * case["dim"] * case["heads"] * pairs
        rows = sum(c[3] for ph in phases for c in ph[2])
        grad = 2 * case["kv_heads"] * case["dim"] * 4 * (sum(lens) + sum(new))
        by += kv * (listed_once + own) + rows * (2 * row + 2 * case["heads"] * case["dim"] * 4) + grad
    return {"bytes": by, "flops": fl}


def tolerance(case):
    # bf16: stored keys, turned queries, probabilities and results are rounded to 8 bits each: two walks over the same call
    # (in place, over a packed copy, split elsewhere) differ by 4.4e-3, each from the exact result by 3e-3, the gradients
    # (through the forward's log-sum-exp) by 2e-3.  fp32: outputs and gradients are 3e-7 to 6e-7 from those in fp64, two
    # orders of the sums up to 8e-7 from each other.
    return {"rel": 1e-2} if case["dtype"] == "bf16" else {"rel": 4e-6}


# -------------------------------------------------------------------------------------------------------- one pass
class _State:
    pass


class _Batch:
    """The marshalled calls of one phase; ids of the pass's new messages are filled in per pass."""

    def __init__(self, calls):
        self.arr = (pc_call * len(calls))()
        n = sum(len(c[0]) for c in calls)
        self.sel = np.zeros((max(n, 1), 2), dtype=np.int32)                        # pc_sel rows: (message, start)
        self.new = np.zeros(max(n, 1), dtype=bool)
        self.own = [c[1] for c in calls]
        at = 0
        for i, (sel, _, start, n_q) in enumerate(calls):
            for j, (k, m, s) in enumerate(sel):
                self.sel[at + j] = (m, s)
                self.new[at + j] = k == 1
            self.arr[i].sel = ctypes.cast(self.sel.ctypes.data + at * ctypes.sizeof(pc_sel), ctypes.POINTER(pc_sel))
            self.arr[i].n_sel = len(sel)
            self.arr[i].self_start = start
            self.arr[i].n_q = n_q
            at += len(sel)
        self.rel = self.sel[:, 0].copy()
        self.any_new = bool(self.new.any())

    def bind(self, ids):
        if self.any_new:
            self.sel[:, 0] = np.where(self.new, np.asarray(ids, dtype=np.int32)[np.where(self.new, self.rel, 0)], self.rel)
        for i, m in enumerate(self.own):
            self.arr[i].self_msg = ids[m]
        return self.arr, self.sel


def prepare(case, seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    dt = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
    Hq, Hkv, D = case["heads"], case["kv_heads"], case["dim"]

    def normal(*shape):
        return torch.randn(shape, generator=g, device=DEV, dtype=torch.float32).to(dt)
    lens, phases = _layout(case)
    s = _State()
    s.case = case
    room = lambda n: (n + 31) // 32 * 32                                           # noqa: E731  (messages start on 32-token boundaries)
    cap = sum(room(L) for L in lens) + sum(room(L) for ph in phases for L in ph[1]) + 32
    s.cache = Cache(Hq, Hkv, D, PC_BF16 if dt == torch.bfloat16 else PC_F32, case["theta"], cap, IDS)
    for i in range(0, len(lens), 64):                                              # the cached messages
        part = lens[i:i + 64]
        k, v = [normal(L, Hkv, D) for L in part], [normal(L, Hkv, D) for L in part]
        s.cache.append_messages([t.data_ptr() for t in k], [t.data_ptr() for t in v], part)
        torch.cuda.synchronize()
    s.phases = []
    for new, reserves, calls in phases:
        p = _State()
        p.lens, p.reserves, p.calls = new, reserves, calls
        p.k, p.v = [normal(L, Hkv, D) for L in new], [normal(L, Hkv, D) for L in new]
        p.k_ptrs, p.v_ptrs = [t.data_ptr() for t in p.k], [t.data_ptr() for t in p.v]
        p.batch = _Batch(calls)
        rows = sum(c[3] for c in calls)
        steps = case["steps"] if case["kind"] == "decode" else 1
        p.q = normal(steps, rows, Hq, D)
        p.out = torch.empty_like(p.q)
        s.phases.append(p)
    if case["kind"] == "decode":
        s.tok_k, s.tok_v = normal(case["steps"], case["n_calls"], Hkv, D), normal(case["steps"], case["n_calls"], Hkv, D)
    if case["kind"] == "train":
        s.d_out = normal(rows, Hq, D)
        s.lse = torch.empty((rows, Hq), dtype=torch.float32, device=DEV)
        s.d_q = torch.empty((rows, Hq, D), dtype=torch.float32, device=DEV)
        slots = s.cache.cache_info()[2]
        s.d_k = torch.empty((slots, Hkv, D), dtype=torch.float32, device=DEV)
        s.d_v = torch.empty_like(s.d_k)
    torch.cuda.synchronize()
    return s


class _Calls:
    """What Cache.attend_backward marshals: one call's fields."""

    def __init__(self, sel, self_msg, self_start, n_q):
        self.sel, self.self_msg, self.self_start, self.n_q, self.q_pos = sel, self_msg, self_start, n_q, None


def run(s):
    c, kind = s.cache, s.case["kind"]
    ids, outs = [], []
    for p in s.phases:
        ids += c.append_messages(p.k_ptrs, p.v_ptrs, p.lens, p.reserves)
        bound = p.batch.bind(ids)
        if kind == "decode":
            for t in range(s.case["steps"]):
                c.decode_step(ids, s.tok_k[t].data_ptr(), s.tok_v[t].data_ptr(), p.calls, p.q[t].data_ptr(), p.out[t].data_ptr(), marshalled=bound)
        else:
            c.attend(p.calls, p.q.data_ptr(), p.out.data_ptr(), s.lse.data_ptr() if kind == "train" else 0, marshalled=bound)
        outs.append(p.out)
    if kind == "train":
        s.d_k.zero_()
        s.d_v.zero_()
        calls = [_Calls([(m, at) for _, m, at in sel], ids[own], start, n_q) for sel, own, start, n_q in p.calls]
        c.attend_backward(calls, p.q.data_ptr(), s.lse.data_ptr(), s.d_out.data_ptr(), s.d_q.data_ptr(), s.d_k.data_ptr(), s.d_v.data_ptr())
        c.grad_keys_finalize(s.d_k.data_ptr())
        outs += [s.lse, s.d_q, s.d_k, s.d_v]
    for m in ids:
        c.message_free(m)
    return outs
