"""The attention of fp32 caches against the oracle (numpy, fp64) at the edges of its tiles: columns are (row, head) pairs in
blocks of 32, keys come in tiles of 32 of which eight waves take an eighth each, few columns split the tiles further.

Bound: products are fp32 and sums of D = 128 terms, a few thousand keys follow each other, the keys are turned twice (as they are
stored, and to the call's positions) and the queries once by rotations rounded to fp32: about ten roundings of 2^-24 a term, 6e-7 in the
2-norm (4e-7 measured); the bar is 3e-6."""
import sys

import numpy as np
import pytest

pytestmark = pytest.mark.gpu
BAR = 3e-6


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


def run_case(lens, calls, h_q, h_kv, D, spoil=None, seed=7, static=False, spoil_q=None):
    """lens: messages; calls: (sel, self, self_start, n_q); spoil(ks, vs), spoil_q(q): put values into the caller's data."""
    import torch
    from oracle import choreo_oracle as orc
    from paper_2512_23049_amd import binding
    from pc_inputs import Call
    rng = np.random.default_rng(seed)
    ks = [rng.standard_normal((L, h_kv, D)).astype(np.float32) for L in lens]
    vs = [rng.standard_normal((L, h_kv, D)).astype(np.float32) for L in lens]
    clean_v = [v.copy() for v in vs]
    if spoil:
        spoil(ks, vs)
    cache = binding.Cache(h_q, h_kv, D, binding.PC_F32, 10000.0, sum((L + 31) // 32 * 32 for L in lens) + 32, len(lens) + 1)
    for k, v in zip(ks, vs):
        tk, tv = torch.from_numpy(k).cuda(), torch.from_numpy(v).cuda()
        cache.append_message(tk.data_ptr(), tv.data_ptr(), len(k))
        torch.cuda.synchronize()
    rows = sum(c[3] for c in calls)
    q = rng.standard_normal((rows, h_q, D)).astype(np.float32)
    if spoil_q:
        spoil_q(q)
    tq = torch.from_numpy(q).cuda()
    out = torch.full((rows, h_q, D), 7.0, device="cuda:0")
    lse = torch.full((rows, h_q), 7.0, device="cuda:0")
    say("  ", h_q, h_kv, D, [c[3] for c in calls])
    cs = [Call(list(s), o, st, n, None) for s, o, st, n in calls]
    (cache.attend_static if static else cache.attend)(cs, tq.data_ptr(), out.data_ptr(), lse.data_ptr())
    torch.cuda.synchronize()
    got, got_lse = out.cpu().numpy().astype(np.float64), lse.cpu().numpy().astype(np.float64)
    cache.close()
    at = 0
    for sel, own, start, n_q in calls:
        want, want_lse = orc.attend_call(ks, clean_v, sel, own, start, n_q, None, q[at:at + n_q], 10000.0, rows=list(range(n_q)))
        yield got[at:at + n_q], got_lse[at:at + n_q], want, want_lse
        at += n_q


def check(cases):
    for got, got_lse, want, want_lse in cases:
        assert np.isfinite(got).all()
        err = np.linalg.norm(got - want) / max(np.linalg.norm(want), 1e-30)
        seen = np.isfinite(want_lse)
        assert (got_lse[~seen] == -np.inf).all() and (got[~seen] == 0).all()
        assert np.abs(got_lse[seen] - want_lse[seen]).max(initial=0) <= 1e-5
        assert err <= BAR, err


@pytest.mark.parametrize("h_q,h_kv,D", [(2, 2, 64), (6, 2, 64), (32, 2, 64), (4, 4, 128), (3, 1, 128), (40, 2, 128)])
@pytest.mark.parametrize("n_q", [1, 31, 33, 70])
def test_columns_and_tiles(h_q, h_kv, D, n_q):
    lens = [31, 1, 64, 33, 100, max(n_q, 5) + 3]
    check(run_case(lens, [([(0, 0), (4, 40), (1, 7), (2, 300), (0, 500), (3, 140)], 5, 600, n_q)], h_q, h_kv, D))


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("static", [False, True])
def test_batch_and_splits(D, static):
    """Few columns over a long history (split), a call that sees nothing, one without a new message, own rows only."""
    lens = [int(x) for x in np.random.default_rng(3).integers(20, 300, size=12)] + [20, 70, 1]
    long = [(m, 300 * m) for m in range(12)]
    check(run_case(lens, [(long, 12, 4000, 20), ([], -1, 3, 2), (long[:3], -1, 900, 5), ([], 13, 0, 70), (long[::-1], 14, 5000, 1)], 4, 2, D, static=static))


def test_many_columns():
    """More blocks of columns than compute units: no split."""
    lens = [200, 64, 300]
    check(run_case(lens, [([(1, 5), (0, 100)], 2, 400, 300)], 32, 2, 64))


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("bad", [np.nan, np.inf])
def test_later_tokens_that_are_not_finite(D, bad):
    """A row does not see the tokens behind its own: what they hold must not reach it."""
    at = 37

    def spoil(ks, vs):
        vs[1][at, :, 5] = bad
    (got, got_lse, want, want_lse), = run_case([50, 64], [([(0, 0)], 1, 60, 64)], 4, 2, D, spoil)
    assert np.isfinite(got[:at]).all() and not np.isfinite(got[at:, :, 5]).any()
    got[at:, :, 5] = want[at:, :, 5]
    check([(got, got_lse, want, want_lse)])
