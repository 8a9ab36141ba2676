"""The gradient of a bf16 batch at fp32 precision: pc_attend_backward against fp64 gradients of the same stored keys and
values (read back from the cache's memory, so that the keys' one bf16 rounding is not part of the difference) and the
fp64 log-sum-exp of those.

Bound: every product is exact or within 2^-24, what remains are the fp32 sums of the kernels, a sincos rounded to fp32
per rotation (two per side) and exp2's last bit: about ten roundings of 2^-24 per term in sequence, sums of up to a few
thousand terms whose errors add like their square roots.  2-norm of the difference over that of the gradient: 10 * 2^-24 =
6e-7 before cancellation (p (dp - Delta) loses up to another factor of a few); the bar is 3e-6, where arithmetic on
operands rounded to bf16 would be at 3e-3."""
import ctypes as C
import sys

import numpy as np
import pytest

pytestmark = pytest.mark.gpu
BAR = 3e-6


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


def rot(x, pos, theta):
    """x [T, ..., D] turned by pos [T] in fp64."""
    import torch
    half = x.shape[-1] // 2
    f = torch.tensor([float(np.float32(theta)) ** (-2.0 * i / x.shape[-1]) for i in range(half)], dtype=torch.float64, device=x.device)
    a = (pos.double()[:, None] * f).reshape([x.shape[0]] + [1] * (x.dim() - 2) + [half])
    c, s = a.cos(), a.sin()
    lo, hi = x[..., :half], x[..., half:]
    return torch.cat([lo * c - hi * s, lo * s + hi * c], -1)


def run_case(lens, calls, h_q, h_kv, dtype="bf16", D=128, theta=10000.0, bases=(), seed=5, capacity=None, bar=BAR, spoil=None):
    """lens: messages; calls: (sel, self, self_start, n_q); spoil(name, tensor): changes the k and v of a message, q and do."""
    spoil = spoil or (lambda name, t: None)
    import torch
    from paper_2512_23049_amd import binding
    from pc_inputs import Call
    td = torch.bfloat16 if dtype == "bf16" else torch.float32
    rng = torch.Generator(device="cuda:0")
    rng.manual_seed(seed)
    normal = lambda *s: torch.randn(s, generator=rng, device="cuda:0").to(td)      # noqa: E731
    cap = capacity or sum((L + 31) // 32 * 32 for L in lens) + 32
    cfg = binding.pc_config(h_q, h_kv, D, binding.PC_BF16 if dtype == "bf16" else binding.PC_F32, theta, 0.0, cap, len(lens) + 1, 1 << 20, 0, None, 0)
    nbytes = binding.lib().pc_cache_storage_bytes(C.byref(cfg))
    arena = torch.zeros(nbytes // td.itemsize, dtype=td, device="cuda:0")
    cache = binding.Cache(h_q, h_kv, D, cfg.dtype, theta, cap, len(lens) + 1, max_position=1 << 20, arena=arena.data_ptr(), arena_bytes=nbytes)
    for L in lens:
        k, v = normal(L, h_kv, D), normal(L, h_kv, D)
        spoil("k", k)
        spoil("v", v)
        cache.append_message(k.data_ptr(), v.data_ptr(), L)
        torch.cuda.synchronize()
    for m, b in bases:
        cache.reposition(m, b)
    torch.cuda.synchronize()
    slots = cache.cache_info()[2]
    n = h_kv * slots * D
    K = arena[:n].view(h_kv, slots, D).double()
    V = (arena[n:].view(h_kv, slots // 8, D, 8).transpose(2, 3).reshape(h_kv, slots, D) if dtype == "bf16" else arena[n:].view(h_kv, slots, D)).double()
    rows = sum(c[3] for c in calls)
    q, do = normal(rows, h_q, D), normal(rows, h_q, D)
    spoil("q", q)
    spoil("do", do)
    g, scale = h_q // h_kv, 1.0 / D ** 0.5
    want_q = torch.zeros(rows, h_q, D, dtype=torch.float64, device="cuda:0")
    want_k = torch.zeros(slots, h_kv, D, dtype=torch.float64, device="cuda:0")
    want_v = torch.zeros_like(want_k)
    lse = torch.zeros(rows, h_q, dtype=torch.float32, device="cuda:0")
    at = 0
    for sel, own, start, n_q in calls:
        segs = [(m, s) for m, s in sel] + ([(own, start)] if own >= 0 else [])
        slot = torch.cat([cache.message_info(m)[1] + torch.arange(lens[m]) for m, _ in segs]).cuda() if segs else torch.zeros(0, dtype=torch.long, device="cuda:0")
        shift = torch.cat([torch.full((lens[m],), s - cache.message_base(m)) for m, s in segs]).cuda() if segs else slot
        first = lens[own] - n_q if own >= 0 else 0
        qpos = start + first + torch.arange(n_q, device="cuda:0")
        qt = rot(q[at:at + n_q].double(), qpos, theta)
        kt = rot(K[:, slot].transpose(0, 1), shift, theta)                 # [T, h_kv, D] where the call puts them
        vt = V[:, slot].transpose(0, 1)
        seen = torch.ones(n_q, len(slot), dtype=torch.bool, device="cuda:0")
        if own >= 0:
            t = torch.arange(lens[own], device="cuda:0")
            seen[:, len(slot) - lens[own]:] = t[None, :] <= (first + torch.arange(n_q, device="cuda:0"))[:, None]
        for h in range(h_q):
            kh, vh = kt[:, h // g].contiguous(), vt[:, h // g].contiguous()
            s = (qt[:, h] @ kh.T.contiguous() * scale).masked_fill(~seen, -np.inf)
            l = torch.logsumexp(s, 1) if s.shape[1] else torch.full((n_q,), -np.inf, dtype=torch.float64, device="cuda:0")
            lse[at:at + n_q, h] = l.float()
            p = torch.exp(s - lse[at:at + n_q, h].double()[:, None]) if s.shape[1] else s
            gh = do[at:at + n_q, h].double()
            dp = gh @ vh.T.contiguous()
            ds = p * (dp - (p * dp).sum(1, keepdim=True)) * scale
            want_q[at:at + n_q, h] = rot((ds @ kh)[:, None], -qpos, theta)[:, 0]
            want_k[:, h // g].index_add_(0, slot, rot((ds.T.contiguous() @ qt[:, h].contiguous())[:, None], -shift, theta)[:, 0])
            want_v[:, h // g].index_add_(0, slot, p.T.contiguous() @ gh)
        at += n_q
    d_q = torch.full((rows, h_q, D), 7.0, dtype=torch.float32, device="cuda:0")
    d_k = torch.zeros(slots, h_kv, D, dtype=torch.float32, device="cuda:0")
    d_v = torch.zeros_like(d_k)
    cache.attend_backward([Call(list(s), o, st, nq, None) for s, o, st, nq in calls], q.data_ptr(), lse.data_ptr(), do.data_ptr(), d_q.data_ptr(),
                          d_k.data_ptr(), d_v.data_ptr())
    torch.cuda.synchronize()
    err = {}
    for name, got, want in (("dq", d_q, want_q), ("dk", d_k, want_k), ("dv", d_v, want_v)):
        assert torch.isfinite(got).all(), name
        err[name] = float((got.double() - want).norm() / want.norm().clamp_min(1e-300))
        assert not got[want == 0].any(), name + ": something where nothing belongs"
    say("  ", h_q, h_kv, "rows", rows, {k: "%.2e" % v for k, v in err.items()})
    cache.close()
    assert max(err.values()) <= bar, err


# (head shapes: every kind of sharing of a KV head, a group that does not divide a workgroup's 8 units;
#  rows: one, a block less and more than 32, several blocks; messages that end one before, at and one after a tile)
@pytest.mark.parametrize("h_q,h_kv", [(2, 2), (6, 2), (8, 2), (32, 2)])
@pytest.mark.parametrize("n_q", [1, 31, 33, 130])
def test_bf16_gradient_is_fp32(h_q, h_kv, n_q):
    lens = [31, 1, 64, 33, 100, max(n_q, 5) + 3]
    run_case(lens, [([(0, 0), (4, 40), (1, 7), (2, 300), (0, 500), (3, 140)], 5, 600, n_q)], h_q, h_kv)


def test_bf16_gradient_of_a_batch():
    """Calls that share messages, list nothing, have no new message, fewer rows than the new message; moved messages."""
    lens = [70, 128, 9, 40, 257, 96, 17]
    calls = [([(0, 0), (1, 70), (2, 210)], 3, 220, 40), ([], 4, 0, 257), ([(1, 5), (4, 900), (0, 100)], 5, 300, 61),
             ([(4, -20), (2, 400)], -1, 500, 34), ([], -1, 3, 2), ([(5, 0), (5, 30)], 6, 300, 1)]
    run_case(lens, calls, 8, 2, bases=[(0, 50), (4, -7)])


def test_bf16_gradient_over_many_splits():
    """One block of rows over a long history: the tiles are split over many workgroups."""
    lens = [int(x) for x in np.random.default_rng(3).integers(20, 300, size=40)] + [20]
    run_case(lens, [([(m, 300 * m) for m in range(40)], 40, 13000, 20)], 8, 2)


def test_bf16_gradient_of_a_batch_cut_into_several_runs():
    """More units (32-row blocks x heads) than one set of launches takes, the cut inside a call."""
    lens = [40] + [33] * 70 + [2100]
    calls = [([(0, 0)], 1 + i, 50, 33) for i in range(70)] + [([(0, 3)], 71, 60, 2100)]
    run_case(lens, calls, 128, 8)
