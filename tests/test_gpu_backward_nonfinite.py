"""Infinite and NaN keys and values in the gradient, both cache types.  A row whose log-sum-exp is finite gives a key with a score
of -inf a probability of exactly zero, so the key leaves no trace in the gradients of anything else; a row that saw nothing (or a score that is no
number) leaves no trace at all, whatever the values hold that it would have met."""
import pytest

pytestmark = pytest.mark.gpu
KINDS = [("f32", 64), ("f32", 128), ("bf16", 128)]


def tensors(dtype, D, sizes, seed):
    import torch
    rng = torch.Generator(device="cuda:0")
    rng.manual_seed(seed)
    td = torch.float32 if dtype == "f32" else torch.bfloat16
    return [torch.randn((n, h, D), generator=rng, device="cuda:0").to(td) for n, h in sizes]


def gradients(dtype, D, h_q, h_kv, messages, call, q, g, lse=None):
    """(lse, d_q, [d_k of each message], [d_v of each message]); lse: taken instead of the forward's."""
    import torch
    from paper_2512_23049_amd import binding
    cache = binding.Cache(h_q, h_kv, D, binding.PC_F32 if dtype == "f32" else binding.PC_BF16, 10000.0, 512, len(messages))
    for k, v in messages:
        cache.append_message(k.data_ptr(), v.data_ptr(), len(k))
    if lse is None:
        out, lse = torch.empty_like(q), torch.empty(q.shape[:2], device="cuda:0")
        cache.attend([call], q.data_ptr(), out.data_ptr(), lse.data_ptr())
    d_q = torch.full(q.shape, 7.0, device="cuda:0")
    d_k, d_v = (torch.zeros((512, h_kv, D), device="cuda:0") for _ in range(2))
    cache.attend_backward([call], q.data_ptr(), lse.data_ptr(), g.data_ptr(), d_q.data_ptr(), d_k.data_ptr(), d_v.data_ptr())
    torch.cuda.synchronize()
    spans = [slice(cache.message_info(m)[1], cache.message_info(m)[1] + len(k)) for m, (k, _) in enumerate(messages)]
    cache.close()
    return lse, d_q, [d_k[s] for s in spans], [d_v[s] for s in spans]


def same(a, b):
    import torch
    # the same sums in fp32; atomics add a few parts in no fixed order
    return torch.isfinite(b).all() and float((a - b).norm()) <= 3e-6 * float(a.norm())


@pytest.mark.parametrize("dtype,D", KINDS)
def test_infinite_key_with_a_score_of_minus_infinity(dtype, D):
    import torch
    from pc_inputs import Call
    h_q, h_kv, half = 4, 2, D // 2
    k0, v0, k1, v1, q, g = tensors(dtype, D, [(90, h_kv), (90, h_kv), (75, h_kv), (75, h_kv), (40, h_q), (40, h_q)], 5)
    # the slowest pair turns by 1e-4 a position: both components of the stored key are +inf, both of every turned query negative
    q[..., half - 1], q[..., D - 1] = -3.0, -3.0
    call = Call([(0, 0)], 1, 100, 40, None)
    res, lse = [], None
    for big in (1e4, float("inf")):                      # 1e4: a score of about -2000, a probability of zero as well
        k0[37, :, half - 1] = k1[33, :, half - 1] = big   # (every row of the call sees both)
        lse, *r = gradients(dtype, D, h_q, h_kv, [(k0, v0), (k1, v1)], call, q, g, lse)
        res.append(r)
    (q_a, k_a, v_a), (q_b, k_b, v_b) = res
    dims = [d for d in range(D) if d % half != half - 1]  # (that pair of dq is zero times infinity)
    assert same(q_a[..., dims], q_b[..., dims])
    for a, b in zip(k_a + v_a, k_b + v_b):
        assert same(a, b)
    assert not k_b[0][37].any() and not v_b[1][33].any()


@pytest.mark.parametrize("dtype,D", KINDS)
@pytest.mark.parametrize("n_dead", [1, 33])
def test_dead_rows_leave_no_trace_of_values_that_are_not_finite(dtype, D, n_dead):
    import torch
    from pc_inputs import Call
    h_q, h_kv, n = 4, 2, 33
    k, v, q, g = tensors(dtype, D, [(n, h_kv), (n, h_kv), (n, h_q), (n, h_q)], 6)
    call = Call([], 0, 0, n, None)
    lse = gradients(dtype, D, h_q, h_kv, [(k, v)], call, q, g)[0]
    lse[n - n_dead:] = -float("inf")
    res = []
    for bad in (False, True):
        if bad:
            k[n - n_dead:, :, 3], v[n - n_dead:, 1, 7], v[n - n_dead:, 0, 7] = float("nan"), float("nan"), float("inf")
        res.append(gradients(dtype, D, h_q, h_kv, [(k, v)], call, q, g, lse)[1:])
    (q_a, k_a, v_a), (q_b, k_b, v_b) = res
    assert not q_b[n - n_dead:].any() and not k_b[0][n - n_dead:].any() and not v_b[0][n - n_dead:].any()
    for a, b in ((q_a, q_b), (k_a[0], k_b[0]), (v_a[0], v_b[0])):
        assert same(a, b)


def test_values_that_are_not_finite_reach_their_own_gradient():
    """A row with a gradient that sees such a value has none that is a number, and neither has the value's key."""
    import torch
    from pc_inputs import Call
    D, h_q, h_kv = 128, 4, 2
    k, v, q, g = tensors("bf16", D, [(70, h_kv), (70, h_kv), (70, h_q), (70, h_q)], 7)
    call = Call([], 0, 0, 70, None)
    lse, q_a, k_a, v_a = gradients("bf16", D, h_q, h_kv, [(k, v)], call, q, g)
    v[40, 0, 5], v[40, 1, 6] = float("nan"), float("inf")
    _, q_b, k_b, v_b = gradients("bf16", D, h_q, h_kv, [(k, v)], call, q, g, lse)
    assert same(q_a[:40], q_b[:40]) and same(v_a[0], v_b[0])
    assert torch.isnan(k_b[0][40]).all() and not torch.isfinite(q_b[40:]).any()
