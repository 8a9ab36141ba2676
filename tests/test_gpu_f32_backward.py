"""The gradient of an fp32 batch against fp64 gradients of the same stored keys and values, at the edges of its tiles: 32
(row, head) columns, 32-key tiles shared out over eight waves (rows; four at D = 128) or one a wave (keys), column blocks split over
workgroups.  Bound as in test_gpu_backward_precision: fp32 sums, 5e-7 measured, the bar is 3e-6."""
import numpy as np
import pytest

from tests.test_gpu_backward_precision import run_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("h_q,h_kv,D", [(2, 2, 64), (6, 2, 64), (32, 2, 64), (4, 4, 128), (3, 1, 128), (40, 2, 128)])
@pytest.mark.parametrize("n_q", [1, 31, 33, 70])
def test_columns_and_tiles(h_q, h_kv, D, n_q):
    lens = [31, 1, 64, 33, 100, max(n_q, 5) + 3]
    run_case(lens, [([(0, 0), (4, 40), (1, 7), (2, 300), (0, 500), (3, 140)], 5, 600, n_q)], h_q, h_kv, dtype="f32", D=D)


@pytest.mark.parametrize("D", [64, 128])
def test_batch(D):
    """Calls that share messages, list nothing, have no new message, fewer rows than the new message; moved messages."""
    lens = [70, 128, 9, 40, 257, 96, 17]
    calls = [([(0, 0), (1, 70), (2, 210)], 3, 220, 40), ([], 4, 0, 257), ([(1, 5), (4, 900), (0, 100)], 5, 300, 61),
             ([(4, -20), (2, 400)], -1, 500, 34), ([], -1, 3, 2), ([(5, 0), (5, 30)], 6, 300, 1)]
    run_case(lens, calls, 8, 2, dtype="f32", D=D, bases=[(0, 50), (4, -7)])


def test_many_blocks_over_a_long_history():
    lens = [int(x) for x in np.random.default_rng(3).integers(20, 300, size=30)] + [300]
    run_case(lens, [([(m, 300 * m) for m in range(30)], 30, 13000, 300)], 8, 2, dtype="f32", D=64)


# Values v0 + N(0,1) and keys k0 + N(0,1): dO . v is rounded at sqrt(1 + v0^2) times the size of its spread, which is all that ds = p (dp - Delta)
# keeps of it, and times keys sqrt(1 + k0^2) times as large as their own spread: the ten roundings of 2^-24 times both factors.  (Sums of
# p dp K and p K whose difference is taken at their end are at twice to three times that: 4.9e-6 for the last shape at 3, 1.)
@pytest.mark.parametrize("off", [(1.0, 1.0), (3.0, 0.0), (3.0, 1.0), (10.0, 0.0), (0.0, 3.0)])
@pytest.mark.parametrize("D", [64, 128])
def test_values_and_keys_with_a_common_part(D, off):
    import torch
    bar = 10 * 2.0 ** -24 * ((1 + off[0] ** 2) * (1 + off[1] ** 2)) ** 0.5

    def spoil(name, t):
        if name == "v":
            t += off[0]
        if name == "k":
            t += off[1] * torch.tensor([1.0, -1.0, -1.0, 1.0], device="cuda:0").repeat(D // 4)
    run_case([500, 90], [([(0, 0)], 1, 500, 90)], 4, 2, dtype="f32", D=D, spoil=spoil, bar=bar)
    run_case([300, 1000, 40], [([(0, 3), (1, 300)], 2, 1400, 40)], 8, 2, dtype="f32", D=D, spoil=spoil, bar=bar)


@pytest.mark.parametrize("D", [64, 128])
def test_long_walk(D):
    # the ten roundings a term, and the sum's own: one per 16 keys, of which a wave has 100 thousand in 8 (4) parts: sqrt(1563) * 2^-25 = 1.2e-6
    run_case([100000, 9], [([(0, -500)], 1, 300000, 9)], 4, 2, dtype="f32", D=D, bar=10 * 2.0 ** -24 + 1563 ** 0.5 * 2.0 ** -25)


@pytest.mark.parametrize("dtype,D", [("f32", 64), ("f32", 128), ("bf16", 128)])
def test_later_tokens_that_are_not_finite(dtype, D):
    """What stands behind a row's own token does not reach its gradient."""
    import torch
    from paper_2512_23049_amd import binding
    from pc_inputs import Call
    h_q, h_kv, n, at = 4, 2, 64, 37
    rng = torch.Generator(device="cuda:0")
    rng.manual_seed(2)
    td = torch.float32 if dtype == "f32" else torch.bfloat16
    k, v, q, g = (torch.randn((n, h, D), generator=rng, device="cuda:0").to(td) for h in (h_kv, h_kv, h_q, h_q))
    grads, lse = [], torch.empty((n, h_q), device="cuda:0")
    for bad in (False, True):
        if bad:
            k[at, :, 3] = float("inf")
            v[at, :, 5] = float("nan")
        cache = binding.Cache(h_q, h_kv, D, binding.PC_F32 if dtype == "f32" else binding.PC_BF16, 10000.0, 128, 2)
        m = cache.append_message(k.data_ptr(), v.data_ptr(), n)
        call = [Call([], m, 0, n, None)]
        if not bad or dtype == "f32":                    # (the bf16 forward asks for finite values in a whole tile)
            out = torch.empty((n, h_q, D), dtype=td, device="cuda:0")
            cache.attend(call, q.data_ptr(), out.data_ptr(), lse.data_ptr())
        d_q = torch.empty((n, h_q, D), device="cuda:0")
        d_k, d_v = (torch.zeros((128, h_kv, D), device="cuda:0") for _ in range(2))
        cache.attend_backward(call, q.data_ptr(), lse.data_ptr(), g.data_ptr(), d_q.data_ptr(), d_k.data_ptr(), d_v.data_ptr())
        torch.cuda.synchronize()
        cache.close()
        grads.append(d_q[:at].clone())
    assert torch.isfinite(grads[1]).all()
    assert float((grads[1] - grads[0]).norm() / grads[0].norm()) <= 3e-6


@pytest.mark.parametrize("dtype,D", [("f32", 64), ("f32", 128), ("bf16", 128)])
def test_rows_that_saw_nothing(dtype, D):
    """A log-sum-exp of -inf: no gradient, whatever the row's query and output gradient hold."""
    import torch
    from paper_2512_23049_amd import binding
    from pc_inputs import Call
    h_q, h_kv, n = 4, 2, 70
    rng = torch.Generator(device="cuda:0")
    rng.manual_seed(3)
    td = torch.float32 if dtype == "f32" else torch.bfloat16
    k, v, q, g = (torch.randn((n, h, D), generator=rng, device="cuda:0").to(td) for h in (h_kv, h_kv, h_q, h_q))
    cache = binding.Cache(h_q, h_kv, D, binding.PC_F32 if dtype == "f32" else binding.PC_BF16, 10000.0, 128, 2)
    m = cache.append_message(k.data_ptr(), v.data_ptr(), n)
    call = [Call([], m, 0, n, None)]
    out, lse = torch.empty((n, h_q, D), dtype=td, device="cuda:0"), torch.empty((n, h_q), device="cuda:0")
    cache.attend(call, q.data_ptr(), out.data_ptr(), lse.data_ptr())
    dead = [5, 33, 69]
    lse[dead] = -float("inf")
    res = []
    for bad in (False, True):
        if bad:
            q[dead], g[dead] = float("nan"), float("inf")
        d_q = torch.full((n, h_q, D), 7.0, device="cuda:0")
        d_k, d_v = (torch.zeros((128, h_kv, D), device="cuda:0") for _ in range(2))
        cache.attend_backward(call, q.data_ptr(), lse.data_ptr(), g.data_ptr(), d_q.data_ptr(), d_k.data_ptr(), d_v.data_ptr())
        torch.cuda.synchronize()
        res.append((d_q, d_k, d_v))
    cache.close()
    assert (res[1][0][dead] == 0).all()
    for a, b in zip(*res):
        assert torch.isfinite(b).all() and float((a - b).norm()) <= 1e-6 * float(a.norm())


def test_message_of_more_than_a_million_tokens():
    # dq: a wave adds the terms of an eighth of the keys in one chain, 131 thousand fp32 roundings: sqrt(131e3) * 2^-24 = 2.2e-5
    run_case([1048600, 3], [([(0, -500000)], 1, 600000, 3)], 1, 1, dtype="f32", D=64, bar=2.2e-5)
