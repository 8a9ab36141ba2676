"""Calls around the sizes at which their tiles are split over workgroups (bf16 caches): below 16 tiles not at all, from 16 on in
runs of 4 with fp32 partial results, from 32 on with fp16 ones; decode calls (one row) and prefill calls, against the oracle
to the bf16 bars of test_gpu_parity, and pc_attend_static against pc_attend bit for bit."""
import numpy as np
import pytest

import pc_inputs as gen
from pc_inputs import Call

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tiles", [3, 7, 15, 16, 17, 31, 32, 33])
@pytest.mark.parametrize("n_q,n_calls,h_q,h_kv", [(1, 1, 8, 2), (1, 5, 32, 2), (40, 1, 8, 2), (33, 3, 16, 2)])
def test_splits(tiles, n_q, n_calls, h_q, h_kv):
    import torch
    from oracle import choreo_oracle as orc
    from paper_2512_23049_amd import binding, harness as hip
    D, theta = 128, 10000.0
    rng = np.random.default_rng(tiles)
    own = (n_q + 31) // 32
    lens = [32 * (tiles - own) - 5] + [n_q] * n_calls

    def rnd(*shape):
        return gen.round_to_bf16(rng.standard_normal(shape).astype(np.float32))
    ks, vs = [rnd(L, h_kv, D) for L in lens], [rnd(L, h_kv, D) for L in lens]
    cache = binding.Cache(h_q, h_kv, D, binding.PC_BF16, theta, sum((L + 31) // 32 * 32 for L in lens), len(lens))
    for k, v in zip(ks, vs):
        kd, vd = hip.to_device(k, "bf16"), hip.to_device(v, "bf16")
        cache.append_message(kd.data_ptr(), vd.data_ptr(), len(k))
        torch.cuda.synchronize()
    cache.set_decode_sharing(1)
    calls = [Call([(0, 7 * i)], 1 + i, 32 * tiles + 9, n_q, None) for i in range(n_calls)]
    rows = n_q * n_calls
    q = rnd(rows, h_q, D)
    qd = hip.to_device(q, "bf16")
    out, out2 = torch.full_like(qd, 7.0), torch.full_like(qd, 9.0)
    lse, lse2 = (torch.full((rows, h_q), x, device="cuda:0") for x in (7.0, 9.0))
    cache.attend(calls, qd.data_ptr(), out.data_ptr(), lse.data_ptr())
    torch.cuda.synchronize()
    cache.attend_static(calls, qd.data_ptr(), out2.data_ptr(), lse2.data_ptr())
    torch.cuda.synchronize()
    cache.close()
    assert torch.equal(out.view(torch.int16), out2.view(torch.int16)) and torch.equal(lse, lse2)
    got, got_lse = out.float().cpu().numpy(), lse.cpu().numpy()
    for i, c in enumerate(calls):
        o, l = orc.attend_call(ks, vs, c.sel, c.self_msg, c.self_start, n_q, None, q[n_q * i:n_q * (i + 1)], theta, rows=list(range(n_q)))
        d = np.abs(got[n_q * i:n_q * (i + 1)] - o)
        assert d.max() <= 2e-2 and d.mean() <= 1e-3, (d.max(), d.mean())
        assert np.abs(got_lse[n_q * i:n_q * (i + 1)] - l).max() <= 2e-2
