"""Decode batches that go to one launch, their lists in its arguments or, where those are too long, in pinned memory, at the sizes
where it can go wrong: a split of one tile, waves without a tile, calls with several rows, nothing to see, the same message twice,
two splits for as many (call, KV head) pairs as get any, as many messages in a split as a wave has lanes and one more (then the
plan builder's way).  Against the oracle to the bf16 bars of test_gpu_parity and the same calls the plan builder's way (which a
split size set by hand selects).  Decode steps: the stores hold, bit for bit, what pc_append_tokens_batch leaves there."""
import numpy as np
import pytest

import pc_inputs as gen
from pc_inputs import Call

pytestmark = pytest.mark.gpu
D, THETA = 128, 10000.0


def rnd(rng, *shape):
    return gen.round_to_bf16(rng.standard_normal(shape).astype(np.float32))


def fill(lens, h_q, h_kv, rng, reserves=None):
    import torch
    from paper_2512_23049_amd import binding, harness as hip
    ks, vs = [rnd(rng, L, h_kv, D) for L in lens], [rnd(rng, L, h_kv, D) for L in lens]
    cap = sum((max(L, r) + 31) // 32 * 32 for L, r in zip(lens, reserves or lens))
    arena = torch.zeros(2 * cap * h_kv * D, dtype=torch.bfloat16, device="cuda:0")
    cache = binding.Cache(h_q, h_kv, D, binding.PC_BF16, THETA, cap, len(lens), arena=arena.data_ptr(), arena_bytes=2 * arena.numel())
    for i, (k, v) in enumerate(zip(ks, vs)):
        kd, vd = hip.to_device(k, "bf16"), hip.to_device(v, "bf16")
        cache.append_message(kd.data_ptr(), vd.data_ptr(), len(k), (reserves or lens)[i])
        torch.cuda.synchronize()
    cache.set_decode_sharing(1)
    return ks, vs, cache, arena


def check(ks, vs, calls, q, got, lse):
    from oracle import choreo_oracle as orc
    at = 0
    for c in calls:
        o, l = orc.attend_call(ks, vs, c.sel, c.self_msg, c.self_start, c.n_q, c.q_pos, q[at:at + c.n_q], THETA, rows=list(range(c.n_q)))
        d = np.abs(got[at:at + c.n_q] - o)
        assert d.max() <= 2e-2 and d.mean() <= 1e-3 + np.abs(o).mean() / 512, (d.max(), d.mean())
        seen = np.isfinite(l)
        assert (np.isfinite(lse[at:at + c.n_q]) == seen).all() and (np.abs(lse[at:at + c.n_q][seen] - l[seen]) <= 2e-2).all()
        at += c.n_q


@pytest.mark.parametrize("h_q,h_kv,n_q", [(8, 2, 1), (8, 1, 2), (32, 2, 1), (2, 2, 13), (12, 4, 3), (32, 8, 1)])
@pytest.mark.parametrize("lens,n_calls", [([1], 1), ([31, 33, 32], 2), ([20] * 63, 3), ([20] * 64, 1), ([2100], 1), ([2100, 900, 5], 5), ([9] * 70, 1), ([70, 33], 60),
                                          ([2100, 900, 5], 14)])
def test_one_launch(h_q, h_kv, n_q, lens, n_calls):
    import torch
    from paper_2512_23049_amd import harness as hip
    rng = np.random.default_rng(len(lens) + n_q)
    own = [n_q + 40 * i for i in range(n_calls)]
    ks, vs, cache, arena = fill(lens + own, h_q, h_kv, rng)
    n = len(lens)
    calls = [Call([(int(m), int(rng.integers(-50, 3000))) for m in rng.permutation(n)], n + i, 2500, n_q, None) for i in range(n_calls)]
    calls.append(Call([(0, 5), (0, 900)], -1, 70, n_q, list(range(3, 3 + n_q))))       # a message twice, no message of its own
    calls.append(Call([], -1, 0, n_q, None))                                         # nothing to see
    rows = sum(c.n_q for c in calls)
    q = rnd(rng, rows, h_q, D)
    qd = hip.to_device(q, "bf16")
    outs = []
    for tiles_per_split in (0, 7):
        cache.set_tuning(tiles_per_split, 0)
        for _ in range(2):                                                           # (the second finds the counters as the first left them)
            out, lse = torch.full_like(qd, 7.0), torch.full((rows, h_q), 7.0, device="cuda:0")
            cache.attend(calls, qd.data_ptr(), out.data_ptr(), lse.data_ptr())
            torch.cuda.synchronize()
            outs.append((out.float().cpu().numpy(), lse.cpu().numpy()))
    cache.close()
    for out, lse in outs:
        check(ks, vs, calls, q, out, lse)
    assert (outs[0][0] == outs[1][0]).all() and (outs[0][1] == outs[1][1]).all()


@pytest.mark.parametrize("h_q,h_kv", [(8, 2), (64, 8), (4, 4)])
@pytest.mark.parametrize("first", [1, 30, 31, 32, 95])
def test_step_appends_its_tokens(h_q, h_kv, first):
    """Tails of `first` tokens and one more per step, over the edge of a tile; after three steps the stores are those of the
    two separate calls, bit for bit."""
    import torch
    from paper_2512_23049_amd import harness as hip
    lens, steps = [70, 300, first, first + 2, 40], 3
    stores, results = [], []
    for fused in (True, False):
        rng = np.random.default_rng(first)
        ks, vs, cache, arena = fill(lens, h_q, h_kv, rng, reserves=[70, 300, first + 8, first + 8, 40])
        cache.reposition(3, 11)
        ids, rows = [2, 3], 2
        for s in range(steps):
            tk, tv, q = rnd(rng, 2, h_kv, D), rnd(rng, 2, h_kv, D), rnd(rng, rows, h_q, D)
            for j, m in enumerate(ids):
                ks[m], vs[m] = np.concatenate([ks[m], tk[j:j + 1]]), np.concatenate([vs[m], tv[j:j + 1]])
            kd, vd, qd = (hip.to_device(x, "bf16") for x in (tk, tv, q))
            calls = [Call([(0, 3), (1, 80)], 3, 400, 1, None), Call([(4, 9)], 2, 60, 1, None)]
            out, lse = torch.full_like(qd, 7.0), torch.full((rows, h_q), 7.0, device="cuda:0")
            if fused:
                cache.decode_step(ids, kd.data_ptr(), vd.data_ptr(), calls, qd.data_ptr(), out.data_ptr(), lse.data_ptr())
            else:
                cache.set_tuning(7, 0)
                cache.append_tokens_batch(ids, kd.data_ptr(), vd.data_ptr())
                cache.attend(calls, qd.data_ptr(), out.data_ptr(), lse.data_ptr())
            torch.cuda.synchronize()
            check(ks, vs, calls, q, out.float().cpu().numpy(), lse.cpu().numpy())
            assert cache.message_info(3)[0] == first + 3 + s
        results.append((out, lse))
        # the grown message as another call's parent: its length in the device table
        calls = [Call([(3, 5)], -1, 600, 1, None)]
        out, lse = torch.full_like(qd[:1], 7.0), torch.full((1, h_q), 7.0, device="cuda:0")
        cache.attend(calls, qd.data_ptr(), out.data_ptr(), lse.data_ptr())
        torch.cuda.synchronize()
        check(ks, vs, calls, q[:1], out.float().cpu().numpy(), lse.cpu().numpy())
        stores.append(arena.view(torch.int16).cpu())
        cache.close()
    assert torch.equal(stores[0], stores[1])
    assert torch.allclose(results[0][0].float(), results[1][0].float(), atol=2e-2) and torch.allclose(results[0][1], results[1][1], atol=2e-2)


@pytest.mark.parametrize("n_listed", [63, 64])
def test_as_many_messages_as_lanes(n_listed):
    """33 unsplit calls of 8 KV heads over 63 messages and a tail of their own (64 entries, one a lane, the tail in the last one; lists in
    pinned memory) or 64 (the plan builder's way): decode steps, more of them than the staging ring has slots."""
    import torch
    from paper_2512_23049_amd import harness as hip
    h_q, h_kv, n_calls, steps = 16, 8, 33, 6
    lens = [1 + 13 * i % 45 for i in range(n_listed)] + [1 + 7 * i % 64 for i in range(n_calls)]
    tails = list(range(n_listed, n_listed + n_calls))
    stores, results = [], []
    for fused in (True, False):
        rng = np.random.default_rng(n_listed)
        ks, vs, cache, arena = fill(lens, h_q, h_kv, rng, reserves=lens[:n_listed] + [L + steps for L in lens[n_listed:]])
        order = [rng.permutation(n_listed) for _ in tails]
        calls = [Call([(int(m), 41 * j) for j, m in enumerate(o)], t, 3000 + t, 1, None) for o, t in zip(order, tails)]
        if not fused:
            cache.set_tuning(7, 0)
        outs = []
        for s in range(steps):
            tk, tv, q = rnd(rng, n_calls, h_kv, D), rnd(rng, n_calls, h_kv, D), rnd(rng, n_calls, h_q, D)
            for j, m in enumerate(tails):
                ks[m], vs[m] = np.concatenate([ks[m], tk[j:j + 1]]), np.concatenate([vs[m], tv[j:j + 1]])
            kd, vd, qd = (hip.to_device(x, "bf16") for x in (tk, tv, q))
            out, lse = torch.full_like(qd, 7.0), torch.full((n_calls, h_q), 7.0, device="cuda:0")
            if fused:
                cache.decode_step(tails, kd.data_ptr(), vd.data_ptr(), calls, qd.data_ptr(), out.data_ptr(), lse.data_ptr())
            else:
                cache.append_tokens_batch(tails, kd.data_ptr(), vd.data_ptr())
                cache.attend(calls, qd.data_ptr(), out.data_ptr(), lse.data_ptr())
            outs.append((out, lse, kd, vd, qd))          # (nothing waits between the steps: their inputs stay)
            if s in (0, steps - 1):
                torch.cuda.synchronize()
                check(ks, vs, calls, q, out.float().cpu().numpy(), lse.cpu().numpy())
        results.append(outs)
        stores.append(arena.view(torch.int16).cpu())
        cache.close()
    assert torch.equal(stores[0], stores[1])
    for one, two in zip(*results):
        assert torch.allclose(one[0].float(), two[0].float(), atol=2e-2) and torch.allclose(one[1], two[1], atol=2e-2)


@pytest.mark.parametrize("n_calls,tokens", [(1, 6000), (4, 700)])
def test_replays_of_a_captured_call(n_calls, tokens):
    """pc_attend_static in a HIP graph (lists in the arguments, splits that the launch merges itself): every replay, with eager calls
    on other queries in between, returns the eager result for the queries it finds."""
    import torch
    from paper_2512_23049_amd import harness as hip
    h_q, h_kv = 32, 8
    rng = np.random.default_rng(tokens)
    ks, vs, cache, arena = fill([tokens // 2, tokens // 2 + 5] + [3] * n_calls, h_q, h_kv, rng)
    calls = [Call([(0, 40 * i), (1, tokens)], 2 + i, 2 * tokens, 1, None) for i in range(n_calls)]
    queries = [hip.to_device(rnd(rng, n_calls, h_q, D), "bf16") for _ in range(4)]
    q, out, lse = torch.empty_like(queries[0]), torch.empty_like(queries[0]), torch.empty((n_calls, h_q), device="cuda:0")
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        cache.attend_static(calls, q.data_ptr(), out.data_ptr(), lse.data_ptr(), stream.cuda_stream)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        cache.attend_static(calls, q.data_ptr(), out.data_ptr(), lse.data_ptr(), stream.cuda_stream)
    for x in queries:
        want, want_lse = torch.empty_like(out), torch.empty_like(lse)
        cache.attend(calls, x.data_ptr(), want.data_ptr(), want_lse.data_ptr())
        torch.cuda.synchronize()
        q.copy_(x)
        out.fill_(7.0)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out.view(torch.int16), want.view(torch.int16)) and torch.equal(lse, want_lse)
    cache.close()


def test_the_host_runs_four_calls_ahead():
    """A split over more messages than a wave has lanes goes the plan builder's way, and takes one slot of the four of the staging
    ring a call like every other: four calls are enqueued while the stream is still busy with work in front of them."""
    import torch
    from paper_2512_23049_amd import binding, harness as hip
    h_q, h_kv, n_calls = 32, 8, 33                       # 264 (call, KV head) pairs: no call is split
    rng = np.random.default_rng(3)
    ks, vs, cache, arena = fill([5] * 70 + [2] * n_calls, h_q, h_kv, rng)
    calls = [Call([(int(m), 7 * j) for j, m in enumerate(rng.permutation(70))], 70 + i, 900, 1, None) for i in range(n_calls)]
    lists = binding.marshal_calls(calls)
    q = hip.to_device(rnd(rng, n_calls, h_q, D), "bf16")
    out = torch.empty_like(q)
    cache.attend(calls, q.data_ptr(), out.data_ptr(), marshalled=lists)
    x = torch.ones(8192, 8192, dtype=torch.bfloat16, device="cuda:0")
    y = torch.empty_like(x)
    torch.mm(x, x, out=y)
    torch.cuda.synchronize()
    for _ in range(200):                                 # at least 0.1 s
        torch.mm(x, x, out=y)
    in_front = torch.cuda.Event()
    in_front.record()
    for _ in range(4):
        cache.attend(calls, q.data_ptr(), out.data_ptr(), marshalled=lists)
    assert not in_front.query()
    torch.cuda.synchronize()
    cache.close()


def test_outputs_at_any_element():
    """Outputs that start at an odd element: unsplit calls and calls whose splits the launch merges."""
    import torch
    from paper_2512_23049_amd import harness as hip
    h_q, h_kv, n_calls = 32, 8, 4
    rng = np.random.default_rng(1)
    ks, vs, cache, arena = fill([90, 2100] + [3] * n_calls, h_q, h_kv, rng)
    q = hip.to_device(rnd(rng, n_calls, h_q, D), "bf16")
    for parent in (0, 1):
        calls = [Call([(parent, 5 * i)], 2 + i, 3000, 1, None) for i in range(n_calls)]
        want, buf = torch.empty_like(q), torch.full((q.numel() + 2,), 7.0, dtype=torch.bfloat16, device="cuda:0")
        cache.attend(calls, q.data_ptr(), want.data_ptr())
        cache.attend(calls, q.data_ptr(), buf[1:].data_ptr())
        torch.cuda.synchronize()
        assert torch.equal(buf[1:-1].view(torch.int16), want.view(torch.int16).flatten()) and (buf[[0, -1]] == 7.0).all()
    cache.close()


@pytest.mark.parametrize("seed", range(12))
def test_forms_of_calls(seed):
    """Random batches over every form a decode call takes (any order, repeats, messages that are nobody's, freed and re-used spans, stored
    bases, further extents, positions up to the limit, rows' positions given, one frequency for all dimensions, 1 to 16
    columns a KV head): one launch against the plan builder's way, attended at once and after a step's tokens."""
    import torch
    from paper_2512_23049_amd import binding
    r = np.random.default_rng(seed)
    h_kv, g, grow = int(r.choice([1, 2, 8])), int(r.choice([1, 3, 4, 8, 16])), seed % 3 == 0
    h_q, n_q = h_kv * g, 1 if grow else int(r.integers(1, max(2, 16 // g + 1)))
    lens, n_calls = [int(x) for x in r.integers(1, int(r.choice([20, 200, 1500])), int(r.integers(5, 100)))], int(r.choice([1, 3, 7, 40]))
    max_position = (0, (1 << 28) - 1)[seed % 2]
    far = (4000, (max_position or 1 << 24) - 5000)[seed % 4 // 2]
    cap = sum(L + 31 for L in lens) + 256 * n_calls + 8192
    cache = binding.Cache(h_q, h_kv, D, binding.PC_BF16, (1.0, 10000.0)[seed % 5 > 0], cap, len(lens) + 2 * n_calls + 50, max_position,
                          flags=binding.PC_FLAG_GROW_EXTENTS if grow else 0)
    gen_dev = torch.Generator(device="cuda:0").manual_seed(seed)
    kept = []

    def normal(*shape):
        kept.append(torch.randn(shape, generator=gen_dev, device="cuda:0").to(torch.bfloat16))
        return kept[-1]

    def append(n, reserve=0):
        return cache.append_message(normal(n, h_kv, D).data_ptr(), normal(n, h_kv, D).data_ptr(), n, reserve)
    ids = [append(n) for n in lens]
    for m in ids[1::3]:
        cache.message_free(m)
    ids = [m for i, m in enumerate(ids) if i % 3 != 1] + [append(int(n)) for n in r.integers(1, 40, 3)]
    for m in ids[:4]:
        cache.reposition(m, int(r.integers(-far, far)))
    own = [append(n, n if grow else n + 8) for n in (int(x) for x in r.integers(n_q, n_q + 70, n_calls))]
    cache.set_decode_sharing(1)
    for step in range(3):
        calls = []
        for m in own:
            n = int(r.integers(0, min(len(ids), 100) + 1))
            pick = r.permutation(len(ids))[:n] if r.random() < 0.8 else r.integers(0, len(ids), n)
            calls.append(Call([(ids[int(p)], int(r.integers(-far, far))) for p in pick], m if r.random() < 0.9 else -1, int(r.integers(-far, far)),
                              n_q, [int(x) for x in r.integers(-far, far, n_q)] if r.random() < 0.3 else None))
        q = normal(n_calls * n_q, h_q, D)
        got = [(torch.full_like(q, 7.0), torch.full((n_calls * n_q, h_q), 7.0, device="cuda:0")) for _ in range(2)]
        if step:
            tk, tv = normal(n_calls, h_kv, D), normal(n_calls, h_kv, D)
            cache.decode_step(own, tk.data_ptr(), tv.data_ptr(), calls, q.data_ptr(), got[0][0].data_ptr(), got[0][1].data_ptr())
        else:
            cache.attend(calls, q.data_ptr(), got[0][0].data_ptr(), got[0][1].data_ptr())
        cache.set_tuning(5, 0)
        cache.attend(calls, q.data_ptr(), got[1][0].data_ptr(), got[1][1].data_ptr())
        cache.set_tuning(0, 0)
        torch.cuda.synchronize()
        (one, one_lse), (two, two_lse) = got
        seen = torch.isfinite(two_lse)
        assert torch.equal(torch.isfinite(one_lse), seen) and (one_lse[seen] - two_lse[seen]).abs().max().item() <= 2e-2
        # (each side rounds probabilities and an output below 4 to bf16: half of 2^-6 either side)
        assert (one.float() - two.float()).abs().max().item() <= 2e-2
    cache.close()
