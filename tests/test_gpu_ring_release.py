"""GPU test of how a slot of the pinned ring that a call's lists lie in becomes free: the call's merge says so, where it has one.
Calls with other lists each, enqueued behind a long kernel faster than the GPU takes them, so that every slot is waited for several
times, give the bits of the same calls made one at a time."""
import numpy as np
import pytest

from pc_inputs import Call

pytestmark = pytest.mark.gpu

HQ, HKV, D, LEN, N = 32, 8, 128, 64, 160


@pytest.mark.parametrize("rows, sharing", [(512, 0), (1, 0), (1, 2)], ids=["prefill", "decode", "shared walk"])
def test_calls_ahead_of_the_gpu(rows, sharing):
    import torch
    from paper_2512_23049_amd.binding import PC_BF16, Cache
    assert torch.cuda.is_available(), "these tests need the MI355X"
    g = torch.Generator(device="cuda:0")
    g.manual_seed(rows + sharing)
    k, v = (torch.randn((N * LEN + 512, HKV, D), generator=g, device="cuda:0").to(torch.bfloat16) for _ in range(2))
    cache = Cache(HQ, HKV, D, PC_BF16, 10000.0, N * LEN + 512, N + 1)
    at = [2 * D * HKV * LEN * i for i in range(N)]
    cache.append_messages([k.data_ptr() + a for a in at], [v.data_ptr() + a for a in at], [LEN] * N)
    tail = cache.append_message(k.data_ptr() + 2 * D * HKV * LEN * N, v.data_ptr() + 2 * D * HKV * LEN * N, 512, 0)
    cache.set_decode_sharing(sharing)

    def lists(i):                                        # 24 rotating messages a call; a prefill call, or 40 one-row calls
        if rows > 1:
            return [Call([((7 * i + j) % N, 70 * j) for j in range(24)], tail, 70 * 24, rows, None)]
        return [Call([((7 * i + 3 * c + j) % N, 70 * j + c) for j in range(24)], -1, 0, 1, np.asarray([1800 + i], dtype=np.int32)) for c in range(40)]
    n_q = rows if rows > 1 else 40
    q = torch.randn((n_q, HQ, D), generator=g, device="cuda:0").to(torch.bfloat16)
    outs = [[torch.empty_like(q) for _ in range(14)] for _ in range(2)]
    for i, out in enumerate(outs[0]):
        cache.attend(lists(i), q.data_ptr(), out.data_ptr())
        torch.cuda.synchronize()
    calls = [lists(i) for i in range(len(outs[1]))]
    a = torch.randn((8192, 8192), generator=g, device="cuda:0")
    for _ in range(2):
        a @ a                                            # some milliseconds, in which the host gets ahead
        for c, out in zip(calls, outs[1]):
            cache.attend(c, q.data_ptr(), out.data_ptr())
    torch.cuda.synchronize()
    for x, y in zip(*outs):
        assert torch.equal(x, y)
    assert not torch.equal(outs[0][0], outs[0][1])
    cache.close()


def test_calls_far_ahead_of_the_gpu():
    """The host waits for a slot for so long that it asks how the stream stands, which is busy."""
    import time
    import torch
    from paper_2512_23049_amd.binding import PC_BF16, Cache
    g = torch.Generator(device="cuda:0")
    g.manual_seed(3)
    k, v = (torch.randn((512, HKV, D), generator=g, device="cuda:0").to(torch.bfloat16) for _ in range(2))
    cache = Cache(HQ, HKV, D, PC_BF16, 10000.0, 2048, 4)
    for i in range(4):
        cache.append_message(k.data_ptr() + 2 * D * HKV * i, v.data_ptr() + 2 * D * HKV * i, 500)
    q = torch.randn((40, HQ, D), generator=g, device="cuda:0").to(torch.bfloat16)
    cache.set_decode_sharing(2)
    calls = [[Call([(m, 600 * i + c) for m in range(4)], -1, 0, 1, np.asarray([9000], dtype=np.int32)) for c in range(40)] for i in range(6)]
    outs = [[torch.empty_like(q) for _ in calls] for _ in range(2)]
    for c, out in zip(calls, outs[0]):
        cache.attend(c, q.data_ptr(), out.data_ptr())
        torch.cuda.synchronize()
    a = torch.randn((8192, 8192), generator=g, device="cuda:0", dtype=torch.float64)
    a @ a
    stream = torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(stream):
        start = time.perf_counter()
        for _ in range(6):
            a @ a                                        # more than 100 ms
        for c, out in zip(calls, outs[1]):
            cache.attend(c, q.data_ptr(), out.data_ptr(), 0, stream.cuda_stream)
        waited = time.perf_counter() - start
    torch.cuda.synchronize()
    assert waited > 0.04, waited
    for x, y in zip(*outs):
        assert torch.equal(x, y)
    cache.close()
