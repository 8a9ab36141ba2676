"""fp32 batches whose attention launch plans for itself (short lists, at most 64 entries a call) and the ones beside them that the plan builder
serves, against the oracle: as many entries as a wave has lanes and one more, splits that start inside a message, rows that share a block of
32 columns with another head's, 1 to 8 heads a KV head, calls that list nothing, positions far out, repositioned messages.  The bar is that
of test_gpu_f32_attend."""
import numpy as np
import pytest

from pc_inputs import Call
from tests.test_gpu_f32_attend import BAR, check, run_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("h_q,h_kv,D", [(8, 8, 64), (4, 2, 64), (8, 1, 128), (8, 4, 128)])
@pytest.mark.parametrize("lens,rows", [([1], 1), ([5] * 62, 3), ([5] * 63, 3), ([5] * 64, 3), ([900, 33, 1, 64], 2), ([40, 70], 45), ([31, 32, 33, 400], 17)])
def test_entries_and_splits(h_q, h_kv, D, lens, rows):
    r = np.random.default_rng(len(lens) + rows)
    n = len(lens)
    calls = [([(int(m), int(r.integers(-50, 3000))) for m in r.permutation(n)], n, 2000, rows), ([], n + 1, 7, 1), ([(0, 3), (0, 90)], -1, 400, 2)]
    check(run_case(lens + [rows + 4, 1], calls, h_q, h_kv, D))
    check(run_case(lens + [rows + 4, 1], calls, h_q, h_kv, D, static=True))


@pytest.mark.parametrize("D", [64, 128])
def test_bases_positions_and_reused_spans(D):
    import torch
    from oracle import choreo_oracle as orc
    from paper_2512_23049_amd import binding
    r = np.random.default_rng(D)
    h_q, h_kv, lens = 8, 2, [20, 50, 90, 33]
    cache = binding.Cache(h_q, h_kv, D, binding.PC_F32, 10000.0, 4096, 64, (1 << 28) - 1)
    dev = lambda x: torch.from_numpy(x).cuda()           # noqa: E731
    rnd = lambda *s: r.standard_normal(s).astype(np.float32)      # noqa: E731
    ks, vs = {}, {}

    def append(n):
        k, v = rnd(n, h_kv, D), rnd(n, h_kv, D)
        kd, vd = dev(k), dev(v)
        m = cache.append_message(kd.data_ptr(), vd.data_ptr(), n)
        torch.cuda.synchronize()
        ks[m], vs[m] = k, v
        return m
    ids = [append(n) for n in lens]
    cache.message_free(ids[1])
    ids[1] = append(41)
    cache.reposition(ids[2], -700)
    own = append(12)
    calls = [Call([(ids[2], 100), (ids[1], 300), (ids[3], 5)], own, 600, 7, [600 + 3 * i for i in range(7)]), Call([(ids[0], 0)], own, 250000, 1, None)]
    q = rnd(8, h_q, D)
    qd, out, lse = dev(q), torch.full((8, h_q, D), 7.0, device="cuda:0"), torch.full((8, h_q), 7.0, device="cuda:0")
    cache.attend(calls, qd.data_ptr(), out.data_ptr(), lse.data_ptr())
    torch.cuda.synchronize()
    cache.close()
    n = max(ks) + 1
    kl, vl = [ks.get(i, np.zeros((1, h_kv, D), np.float32)) for i in range(n)], [vs.get(i, np.zeros((1, h_kv, D), np.float32)) for i in range(n)]
    at = 0
    for c in calls:
        want, want_lse = orc.attend_call(kl, vl, c.sel, c.self_msg, c.self_start, c.n_q, c.q_pos, q[at:at + c.n_q], 10000.0, rows=list(range(c.n_q)))
        got = out[at:at + c.n_q].double().cpu().numpy()
        # (the moved keys are rounded once more; an angle of 250000 radians is known to 2^-53 of itself)
        assert np.linalg.norm(got - want) <= 2 * BAR * np.linalg.norm(want) and np.abs(lse[at:at + c.n_q].cpu().numpy() - want_lse).max() <= 1e-5
        at += c.n_q
