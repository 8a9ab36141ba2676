"""pc_attend_static recorded into a HIP graph with lists longer than a kernel's arguments: every replay returns what pc_attend returns
for the queries it finds, bit for bit, though calls with other lists went through the pinned staging ring and the fixed workspace
in between.  Decode in one launch, a split over more messages than that takes, prefill beside decode, shared decode, and lists
that the copy engine brings to an ordinary call.  And replays beside pc_attend calls on another stream: the two entry points share
neither workspace nor counters."""
import numpy as np
import pytest

from pc_inputs import Call
from tests.test_gpu_one_launch import fill, rnd

pytestmark = pytest.mark.gpu
H_Q, H_KV, D = 32, 8, 128


def batches(kind, rng):
    """(message lengths, calls to capture, calls in between, decode sharing)"""
    if kind == "decode":                                 # about 4.5 KB
        lens = [70, 33] + [1 + i for i in range(60)]
        calls = [[Call([(int(m), 60 * j) for j, m in enumerate(rng.permutation(2))], 2 + i, 400 + s, 1, None) for i in range(60)] for s in (0, 9)]
        return lens, calls[0], calls[1][::-1], 1
    if kind == "many_messages":
        lens = [3 + i % 9 for i in range(80)] + [2] * 33
        calls = [[Call([(int(m), 12 * j + s) for j, m in enumerate(rng.permutation(80)[:70])], 80 + i, 2000, 1, None) for i in range(33)] for s in (0, 9)]
        return lens, calls[0], calls[1][5:], 1
    if kind == "mixed":
        lens = [4 + i % 60 for i in range(500)] + [45, 1, 1, 1]
        calls = [[Call([(int(m), 50 * j + s) for j, m in enumerate(rng.permutation(500))], 500, 30000, 45, None)] +
                 [Call([(int(m), 50 * j) for j, m in enumerate(rng.permutation(500)[:30])], 501 + i, 30000, 1, None) for i in range(3)] for s in (0, 9)]
        return lens, calls[0], calls[1][1:] + calls[1][:1], 0
    if kind == "shared":
        lens = [20 + i for i in range(60)] + [1] * 16
        calls = [[Call([(int(m), 90 * j + s) for j, m in enumerate(rng.permutation(60))], 60 + i, 7000, 1, None) for i in range(16)] for s in (0, 9)]
        return lens, calls[0], calls[1][3:], 2
    assert kind == "copied"                              # 320 KB
    lens = [2 + i for i in range(20)] + [1] * 20
    calls = [[Call([(int(m), 30 * j + s) for j, m in enumerate(rng.integers(0, 20, 2000))], 20 + i, 70000, 1, None) for i in range(20)] for s in (0, 9)]
    return lens, calls[0], calls[1][1:], 1


@pytest.mark.parametrize("kind", ["decode", "many_messages", "mixed", "shared", "copied"])
def test_replays_with_other_calls_in_between(kind):
    import torch
    from paper_2512_23049_amd import harness as hip
    rng = np.random.default_rng(5)
    lens, calls, between, sharing = batches(kind, rng)
    ks, vs, cache, arena = fill(lens, H_Q, H_KV, rng)
    cache.set_decode_sharing(sharing)
    cache.set_key_gather(1)                              # (pc_attend_static never gathers)
    rows = sum(c.n_q for c in calls)
    queries = [hip.to_device(rnd(rng, rows, H_Q, D), "bf16") for _ in range(4)]
    q, out, lse = torch.empty_like(queries[0]), torch.empty_like(queries[0]), torch.empty((rows, H_Q), device="cuda:0")
    scratch = torch.empty_like(out)
    wants = []
    for x in queries:
        want, want_lse = torch.empty_like(out), torch.empty_like(lse)
        cache.attend(calls, x.data_ptr(), want.data_ptr(), want_lse.data_ptr())
        torch.cuda.synchronize()
        wants.append((want, want_lse))
    stream = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        cache.attend_static(calls, q.data_ptr(), out.data_ptr(), lse.data_ptr(), stream.cuda_stream)
    for x, (want, want_lse) in zip(queries, wants):
        for _ in range(3):                               # (more staged calls than the ring has slots)
            cache.attend(between, queries[0].data_ptr(), scratch.data_ptr())
            cache.attend_static(between, queries[0].data_ptr(), scratch.data_ptr())
        q.copy_(x)
        out.fill_(7.0)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out.view(torch.int16), want.view(torch.int16)) and torch.equal(lse, want_lse)
    cache.close()


def test_replays_beside_pc_attend():
    import torch
    from paper_2512_23049_amd import harness as hip
    rng = np.random.default_rng(8)
    n = 4                                                # calls over 60 tiles, each in several splits that the last one merges
    ks, vs, cache, arena = fill([900, 1000] + [3] * n, H_Q, H_KV, rng)
    calls = [Call([(0, 40 * i), (1, 1500)], 2 + i, 4000, 1, None) for i in range(n)]
    others = [Call([(1, 7 * i), (0, 1500), (1, 2600)], 2 + i, 4000, 1, None) for i in range(n)]      # another number of splits
    q = [hip.to_device(rnd(rng, n, H_Q, D), "bf16") for _ in range(2)]
    wants = [torch.empty_like(q[0]) for _ in range(2)]
    for want, x, which in zip(wants, q, (calls, others)):
        cache.attend(which, x.data_ptr(), want.data_ptr())
    rounds = 300
    out, outs = torch.empty_like(q[0]), torch.empty((rounds, *q[0].shape), dtype=torch.bfloat16, device="cuda:0")
    graph = torch.cuda.CUDAGraph()
    replays, eager = torch.cuda.Stream(), torch.cuda.Stream()
    with torch.cuda.graph(graph, stream=replays):
        cache.attend_static(calls, q[0].data_ptr(), out.data_ptr(), 0, replays.cuda_stream)
    torch.cuda.synchronize()
    for i in range(rounds):
        with torch.cuda.stream(replays):
            graph.replay()
        cache.attend(others, q[1].data_ptr(), outs[i].data_ptr(), 0, eager.cuda_stream)
    torch.cuda.synchronize()
    assert torch.equal(out.view(torch.int16), wants[0].view(torch.int16))
    assert (outs.view(torch.int16) == wants[1].view(torch.int16)).all()
    out.fill_(7.0)
    torch.cuda.synchronize()
    graph.replay()
    torch.cuda.synchronize()
    assert torch.equal(out.view(torch.int16), wants[0].view(torch.int16))
    cache.close()
