"""GPU test of what the append kernels leave in the cache (Sec. 2.4: new messages are appended to the
cache; here K turned to the in-message index, V key-transposed in groups of 8 slots).  The stores are read
back through a caller-owned arena: V is a pure data movement and must match bit for bit, K is the oracle's
rotation rounded once to bf16, rows and group remainders behind a message's last token stay zero.
Covers pc_append_message, pc_append_messages, pc_append_tokens and pc_append_tokens_batch."""
import ctypes as C
import sys

import numpy as np
import pytest

import pc_inputs as gen

pytestmark = pytest.mark.gpu


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


@pytest.mark.parametrize("h_kv", [2, 3])
def test_stored_form_after_every_kind_of_append(h_kv):
    import torch
    from oracle import choreo_oracle as orc
    from paper_2512_23049_amd import binding
    from paper_2512_23049_amd.harness import to_device
    assert torch.cuda.is_available(), "these tests need the MI355X"
    D, theta = 128, 10000.0
    rng = np.random.default_rng(31 + h_kv)

    def rnd(L):
        return gen.round_to_bf16(rng.standard_normal((L, h_kv, D)).astype(np.float32))
    cap = 2048
    cfg = binding.pc_config(2 * h_kv, h_kv, D, binding.PC_BF16, theta, 0.0, cap, 32, 1 << 20, 0, None, 0)
    nbytes = binding.lib().pc_cache_storage_bytes(C.byref(cfg))
    arena = torch.zeros(nbytes // 2, dtype=torch.bfloat16, device="cuda:0")
    cache = binding.Cache(2 * h_kv, h_kv, D, binding.PC_BF16, theta, cap, 32, max_position=1 << 20,
                          arena=arena.data_ptr(), arena_bytes=nbytes)
    slots = cap
    k_host, v_host, keep = {}, {}, []

    def dev(x):
        t = to_device(x, "bf16", "cuda:0")
        keep.append(t)
        return t
    # one at a time
    for L, res in [(1, 0), (7, 20), (8, 0), (33, 0)]:
        k, v = rnd(L), rnd(L)
        m = cache.append_message(dev(k).data_ptr(), dev(v).data_ptr(), L, res)
        k_host[m], v_host[m] = k, v
    # several in one launch
    lens, ress = [9, 100, 4, 64], [0, 0, 40, 70]
    kk, vv = [rnd(L) for L in lens], [rnd(L) for L in lens]
    ids = cache.append_messages([dev(x).data_ptr() for x in kk], [dev(x).data_ptr() for x in vv], lens, ress)
    for m, k, v in zip(ids, kk, vv):
        k_host[m], v_host[m] = k, v
    # five more tokens for message 1 (reserve 20), then one more each for messages 1, 6 and 7
    k5, v5 = rnd(5), rnd(5)
    cache.append_tokens(1, dev(k5).data_ptr(), dev(v5).data_ptr(), 5)
    k_host[1], v_host[1] = np.concatenate([k_host[1], k5]), np.concatenate([v_host[1], v5])
    k3, v3 = rnd(3), rnd(3)
    cache.append_tokens_batch([6, 1, 7], dev(k3).data_ptr(), dev(v3).data_ptr())
    for j, m in enumerate([6, 1, 7]):
        k_host[m], v_host[m] = np.concatenate([k_host[m], k3[j:j + 1]]), np.concatenate([v_host[m], v3[j:j + 1]])
    torch.cuda.synchronize()

    n = h_kv * slots * D
    k_store = arena[:n].view(h_kv, slots, D).float().cpu().numpy()
    v_bits = arena[n:2 * n].view(torch.int16).view(h_kv, slots // 8, D, 8).cpu().numpy()
    k_bits_zero = arena[:n].view(torch.int16).view(h_kv, slots, D).cpu().numpy()
    used = np.zeros(slots, dtype=bool)
    for m in sorted(k_host):
        ln, slot0, reserved = cache.message_info(m)
        assert ln == k_host[m].shape[0]
        say(f"  message {m}: len {ln} slots [{slot0}, {slot0 + reserved})")
        used[slot0:slot0 + ln] = True
        # V: bit for bit, key-transposed
        want_v = torch.from_numpy(v_host[m]).to(torch.bfloat16).view(torch.int16).numpy()      # [L, H, D]
        for t in range(ln):
            s = slot0 + t
            assert np.array_equal(v_bits[:, s // 8, :, s % 8], want_v[t]), (m, t)
        # K: the oracle's rotation to the in-message index, rounded once
        want = np.transpose(orc.rope(k_host[m].astype(np.float64), np.arange(ln), theta), (1, 0, 2))  # [H, L, D]
        got = k_store[:, slot0:slot0 + ln, :]
        bound = 2.0 ** -8 * (np.abs(want) + np.abs(np.roll(want, D // 2, axis=-1))) + 1e-6
        assert (np.abs(got - want) <= bound).all(), m
    # nothing was written anywhere else: K rows and V columns of unused slots are still zero
    free = ~used
    assert not k_bits_zero[:, free, :].any()
    v_by_slot = np.transpose(v_bits, (0, 1, 3, 2)).reshape(h_kv, slots, D)
    assert not v_by_slot[:, free, :].any()
    cache.close()


@pytest.mark.parametrize("batch", [False, True])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_reused_span_is_zero_behind_the_last_token(dtype, batch):
    """A span that held a message full of NaN is taken again by shorter ones: whatever of their reserves lies behind
    their last tokens reads as zeros, and the slots of the span that nobody took keep what they held."""
    import torch
    from paper_2512_23049_amd import binding
    h_kv, D = 3, 64 if dtype == "f32" else 128
    td = torch.float32 if dtype == "f32" else torch.bfloat16
    cfg = binding.pc_config(h_kv, h_kv, D, binding.PC_F32 if dtype == "f32" else binding.PC_BF16, 1e4, 0.0, 1024, 32, 1 << 20, 0, None, 0)
    nbytes = binding.lib().pc_cache_storage_bytes(C.byref(cfg))
    arena = torch.zeros(nbytes // td.itemsize, dtype=td, device="cuda:0")
    cache = binding.Cache(h_kv, h_kv, D, cfg.dtype, 1e4, 1024, 32, max_position=1 << 20, arena=arena.data_ptr(), arena_bytes=nbytes)
    bad = torch.full((700, h_kv, D), float("nan"), dtype=td, device="cuda:0")
    first = cache.append_message(bad.data_ptr(), bad.data_ptr(), 700)
    cache.message_free(first)
    # (len, reserve): one token, a whole tile, one past a tile, a group remainder, far beyond the message, past the freed span
    want = [(1, 0), (32, 0), (33, 0), (7, 8), (5, 200), (300, 600)]
    kv = [torch.ones((L, h_kv, D), dtype=td, device="cuda:0") for L, _ in want]
    if batch:
        ids = cache.append_messages([t.data_ptr() for t in kv], [t.data_ptr() for t in kv], [L for L, _ in want], [r for _, r in want])
    else:
        ids = [cache.append_message(t.data_ptr(), t.data_ptr(), L, r) for t, (L, r) in zip(kv, want)]
    torch.cuda.synchronize()
    n = h_kv * 1024 * D
    k = arena[:n].view(h_kv, 1024, D).float()
    v = arena[n:2 * n]
    v = (v.view(h_kv, 128, D, 8).transpose(2, 3).reshape(h_kv, 1024, D) if dtype == "bf16" else v.view(h_kv, 1024, D)).float()
    end = 0
    for m, (L, r) in zip(ids, want):
        _, s0, _ = cache.message_info(m)
        stop = s0 + (max(L, r) + 31) // 32 * 32
        end = max(end, stop)
        say(f"  message {m}: len {L} reserve {r} slots [{s0}, {stop})")
        assert torch.isfinite(k[:, s0:stop]).all() and torch.isfinite(v[:, s0:stop]).all()
        assert not k[:, s0 + L:stop].any() and not v[:, s0 + L:stop].any()
        assert (v[:, s0:s0 + L] == 1).all() and (k[:, s0, :] == 1).all()       # (token 0 sits at position 0: not turned)
    assert torch.isnan(k[:, end:704]).sum() == torch.isnan(k[:, end:700]).numel()
    cache.close()


def test_rotations_of_appended_tokens_are_the_nearest_fp32_numbers():
    """Tokens appended at positions that are their own angles (one frequency for all dimensions), stored in fp32: keys (1, 0) are left as
    the cosine and sine of their position, rounded from 64 bits.  With them the five whole numbers below 2^24 at which a cosine series
    without its term in x^14 rounds to another fp32 number, odd and even quarter turns, and the ends of the range."""
    import torch
    from paper_2512_23049_amd import binding
    D, h_kv = 64, 2
    pos = [180212, 1074636, 1981306, 3329500, 5866457, 1, 2, 3, 11, 1000, (1 << 24) - 1, -1, -180212, -(1 << 24) + 1]
    cap = 32 * len(pos)
    arena = torch.zeros((2, h_kv, cap, D), dtype=torch.float32, device="cuda:0")
    cache = binding.Cache(h_kv, h_kv, D, binding.PC_F32, 1.0, cap, len(pos), arena=arena.data_ptr(), arena_bytes=4 * arena.numel())
    k = torch.zeros((1, h_kv, D), device="cuda:0")
    k[..., :D // 2] = 1
    ids = [cache.append_message(k.data_ptr(), k.data_ptr(), 1, 3) for _ in pos]
    for m, p in zip(ids, pos):
        cache.reposition(m, p - 1)                       # the token at index 1 is turned to p
    for m in ids[:7]:
        cache.append_tokens(m, k.data_ptr(), k.data_ptr(), 1)
    both = k.repeat(len(ids) - 7, 1, 1)
    cache.append_tokens_batch(ids[7:], both.data_ptr(), both.data_ptr())
    torch.cuda.synchronize()
    keys = arena[0].cpu().numpy()
    for i, p in enumerate(pos):
        cos, sin = np.float32(np.cos(np.float64(p))), np.float32(np.sin(np.float64(p)))
        assert (keys[:, 32 * i + 1, :D // 2] == cos).all() and (keys[:, 32 * i + 1, D // 2:] == sin).all(), p
    cache.close()
