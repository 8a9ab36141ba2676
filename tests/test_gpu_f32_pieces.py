"""fp32 caches: numbers cut into three bf16 pieces.  Magnitudes far from one up to the ends of fp32's range, where the pieces of the number
itself no longer hold it (bar as in test_gpu_f32_attend; finite inputs), and infinities, which have no pieces: a key whose score is -inf leaves no trace, one whose score is +inf
makes the row a NaN, an infinite value reaches the rows that see it and no others."""
import numpy as np
import pytest

from tests.test_gpu_f32_attend import BAR, check, run_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("size", [1e-30, 1e-3, 1e30])
def test_magnitudes(D, size):
    pairs = [d for d in range(D) if d % (D // 2) % 3 == 0]

    def spoil(ks, vs):                                   # (the values' size is the result's; keys: small in a third of the pairs, where
        for k in ks:                                     # queries are as much larger, so that those make as much of the scores)
            k[..., pairs] *= 1e-6
        for v in vs:
            v *= np.float32(size)

    def spoil_q(q):
        q[..., pairs] *= 1e6
    for got, got_lse, want, want_lse in run_case([200, 33, 90], [([(0, 5), (1, 300)], 2, 400, 90)], 8, 2, D, spoil, spoil_q=spoil_q):
        want = want * np.float64(np.float32(size))
        assert np.linalg.norm(got - want) <= BAR * np.linalg.norm(want)
        assert np.abs(got_lse - want_lse).max() <= 1e-5


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("n_tok", [50, 700])
@pytest.mark.parametrize("where", ["query", "key"])
def test_largest_numbers(D, n_tok, where):
    """3.4e38 is finite but rounds to infinity in bf16.  In the slowest pair, where the other side holds numbers of 3e-38: scores of order one."""
    big, half = np.float32(3.4e38), D // 2

    def spoil(ks, vs):
        if where == "key":
            ks[0][7, :, half - 1], ks[0][7, :, D - 1] = big, 0
        else:
            for k in ks:
                k[..., half - 1::half] *= np.float32(3e-38)

    def spoil_q(q):
        if where == "query":
            q[5, 0, half - 1], q[5, 0, D - 1], q[33, 3, half - 1], q[33, 3, D - 1] = big, 0, -big, 0
        else:
            q[..., half - 1::half] *= np.float32(3e-38)
    check(run_case([n_tok, 64], [([(0, 0)], 1, n_tok, 64)], 4, 2, D, spoil, spoil_q=spoil_q))


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("size", [1e-32, 1e-34, 1e-36])
@pytest.mark.parametrize("where", ["values", "queries", "keys"])
def test_smallest_numbers(D, size, where):
    """Below 2^-110 (8e-34) a number has bits below bf16's least.  Values: the result's size.  Queries and keys: in a third of the pairs, with
    the other side as much larger."""
    c = np.float32(size)
    pairs = [d for d in range(D) if d % (D // 2) % 3 == 0]

    def spoil(ks, vs):
        for k in ks:
            if where != "values":
                k[..., pairs] *= c if where == "keys" else 1 / c
        for v in vs:
            if where == "values":
                v *= c

    def spoil_q(q):
        if where != "values":
            q[..., pairs] *= c if where == "queries" else 1 / c
    for n_tok in (40, 700):
        for got, got_lse, want, want_lse in run_case([n_tok, 33, 90], [([(0, 5), (1, 300)], 2, n_tok + 300, 90)], 8, 2, D, spoil, spoil_q=spoil_q):
            want = want * (np.float64(c) if where == "values" else 1.0)
            assert np.linalg.norm(got - want) <= BAR * np.linalg.norm(want)
            assert np.abs(got_lse - want_lse).max() <= 1e-5


@pytest.mark.parametrize("D", [64, 128])
def test_a_key_with_a_score_of_minus_1e30(D):
    """The only one a row sees: a probability of one."""
    def spoil(ks, vs):
        ks[0][..., D // 2 - 1], ks[0][..., D - 1] = 1e10, 0

    def spoil_q(q):
        q[..., D // 2 - 1], q[..., D - 1] = -1e20, 0
    (got, got_lse, want, want_lse), = run_case([1], [([], 0, 0, 1)], 4, 2, D, spoil, spoil_q=spoil_q)
    assert np.linalg.norm(got - want) <= BAR * np.linalg.norm(want)
    assert (np.abs(got_lse - want_lse) <= 1e-6 * np.abs(want_lse)).all() and (want_lse < -1e28).all()


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("n_tok", [40, 700])
def test_infinite_key(D, n_tok):
    from oracle import choreo_oracle as orc
    at, dim, theta = 17, 5, 10000.0

    def spoil(ks, vs):
        ks[0][at, :, dim] = np.inf
    with np.errstate(invalid="ignore"):
        (got, got_lse, _, _), = run_case([n_tok, 40], [([(0, 0)], 1, n_tok, 40)], 2, 1, D, spoil)
    rng = np.random.default_rng(7)                       # run_case's data again: keys, values, queries
    k0, k1, v0, v1 = [rng.standard_normal((L, 1, D)).astype(np.float32) for L in (n_tok, 40, n_tok, 40)]
    q = rng.standard_normal((40, 2, D)).astype(np.float32)
    want, want_lse = orc.attend_call([k0[:at], k0[at + 1:], k1], [v0[:at], v0[at + 1:], v1], [(0, 0), (1, at + 1)], 2, n_tok, 40, None, q, theta)
    # the stored key is infinite in that dim and its partner; its score is -inf where both meet a query dim of the other sign
    f = theta ** (-2.0 * dim / D)
    a, t = ((n_tok + np.arange(40)) * f)[:, None], at * f
    x, y = q[:, :, dim].astype(np.float64), q[:, :, dim + D // 2].astype(np.float64)
    low = ((x * np.cos(a) - y * np.sin(a)) * np.cos(t) < 0) & ((x * np.sin(a) + y * np.cos(a)) * np.sin(t) < 0)
    assert low.any() and not low.all()
    assert (got[~low] == 0).all() and (got_lse[~low] == -np.inf).all()     # a score that is not a number, as ever
    assert np.linalg.norm(got[low] - want[low]) <= BAR * np.linalg.norm(want[low])
    assert np.abs(got_lse[low] - want_lse[low]).max() <= 1e-5


@pytest.mark.parametrize("D", [64, 128])
def test_infinite_value(D):
    def spoil(ks, vs):
        vs[0][3, :, 7] = np.inf
    (got, got_lse, want, want_lse), = run_case([50, 64], [([(0, 0)], 1, 60, 64)], 4, 2, D, spoil)
    assert (got[:, :, 7] == np.inf).all()
    got[:, :, 7] = want[:, :, 7]
    check([(got, got_lse, want, want_lse)])


@pytest.mark.parametrize("D", [64, 128])
def test_infinite_output_gradient(D):
    """It reaches its row's dq, the keys' gradients through that row, and of dV only its own dim, with its sign."""
    import torch
    from paper_2512_23049_amd import binding
    from pc_inputs import Call
    h_q, h_kv, n, at, dim = 4, 2, 100, 41, 5
    rng = torch.Generator(device="cuda:0")
    rng.manual_seed(4)
    k, v, q, g = (torch.randn((n, h, D), generator=rng, device="cuda:0") for h in (h_kv, h_kv, h_q, h_q))
    cache = binding.Cache(h_q, h_kv, D, binding.PC_F32, 10000.0, 128, 2)
    m = cache.append_message(k.data_ptr(), v.data_ptr(), n)
    call = [Call([], m, 0, n, None)]
    out, lse = torch.empty((n, h_q, D), device="cuda:0"), torch.empty((n, h_q), device="cuda:0")
    cache.attend(call, q.data_ptr(), out.data_ptr(), lse.data_ptr())
    res = []
    for bad in (False, True):
        if bad:
            g[at, 0, dim] = float("inf")
        d_q = torch.empty((n, h_q, D), device="cuda:0")
        d_k, d_v = (torch.zeros((128, h_kv, D), device="cuda:0") for _ in range(2))
        cache.attend_backward(call, q.data_ptr(), lse.data_ptr(), g.data_ptr(), d_q.data_ptr(), d_k.data_ptr(), d_v.data_ptr())
        torch.cuda.synchronize()
        res.append((d_q, d_k[:n], d_v[:n]))
    cache.close()
    (q0, k0, v0), (q1, k1, v1) = res
    assert not torch.isfinite(q1[at, 0]).any() and not torch.isfinite(k1[:at + 1, 0]).any()
    assert (v1[:at + 1, 0, dim] == float("inf")).all()
    q1[at, 0], k1[:at + 1, 0], v1[:, 0, dim] = q0[at, 0], k0[:at + 1, 0], v0[:, 0, dim]    # (later keys: that row's zero times it)
    for a, b in ((q0, q1), (k0, k1), (v0, v1)):
        assert float((a - b).norm()) <= 3e-6 * float(a.norm())


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("where", ["q", "do", "k", "v"])
def test_gradient_of_the_largest_numbers(D, where):
    """As above: one number near the largest in the slowest pair of a row or key, what meets it there of 3e-38.  (Its own gradient's bound
    is that of every other: a tensor's distance is that of its largest part, where it has one.)"""
    from tests import test_gpu_backward_precision as precision
    half, other = D // 2, {"q": "k", "k": "q", "do": "v", "v": "do"}[where]
    done = []

    def spoil(name, t):
        if name == other:
            t[..., half - 1::half] *= 3e-38
        elif name == where and not done and len(t) > 60:
            t[7, 0, half - 1], t[7, 0, D - 1] = 3.4e38, 0
            done.append(1)
    precision.run_case([90, 64], [([(0, 0)], 1, 100, 64)], 4, 2, dtype="f32", D=D, spoil=spoil, bar=precision.BAR)


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("size", [1e-30, 1e-34, 1e-36, 1e15])
@pytest.mark.parametrize("where", ["q", "do", "k", "v"])
def test_gradient_at_magnitudes_far_from_one(D, size, where):
    """Values or output gradients all of that size, and with them products and gradients; queries or keys in a third of the pairs, with the
    other side as much larger."""
    from tests import test_gpu_backward_precision as precision
    pairs = [d for d in range(D) if d % (D // 2) % 3 == 0]

    def spoil(name, t):
        if where in "qk" and name in "qk":
            t[..., pairs] *= size if name == where else 1 / size
        elif name == where:
            t *= size
    precision.run_case([90, 33, 64], [([(0, 0), (1, 95)], 2, 130, 64)], 4, 2, dtype="f32", D=D, spoil=spoil, bar=precision.BAR)
