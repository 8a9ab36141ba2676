"""Prefill batches of more workgroups than one round of compute units takes: the items of the last round are split, alone, and
their rows merged (bf16 caches, both walks, every grouping of heads, an item with few rows, the last item of a call), against the
oracle to the bf16 bars of test_gpu_parity and, tighter, against the unsplit walk (which a tuning of one split gives): fp32
partial results leave the two a rounding of the bf16 output apart."""
import numpy as np
import pytest

import pc_inputs as gen
from pc_inputs import Call

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("gather", [1, 2])
@pytest.mark.parametrize("h_q,h_kv,n_calls,n_q", [(64, 64, 5, 40), (128, 64, 3, 150), (64, 8, 35, 20), (64, 32, 9, 97)])
def test_last_round(h_q, h_kv, n_calls, n_q, gather):
    import torch
    from oracle import choreo_oracle as orc
    from paper_2512_23049_amd import binding, harness as hip
    D, theta = 128, 10000.0
    rng = np.random.default_rng(n_calls)
    lens = [200, 77, 300] + [n_q + 3 * (i % 2) for i in range(n_calls)]

    def rnd(*shape):
        return gen.round_to_bf16(rng.standard_normal(shape, dtype=np.float32))
    ks, vs = [rnd(L, h_kv, D) for L in lens], [rnd(L, h_kv, D) for L in lens]
    cache = binding.Cache(h_q, h_kv, D, binding.PC_BF16, theta, sum((L + 31) // 32 * 32 for L in lens), len(lens))
    for k, v in zip(ks, vs):
        kd, vd = hip.to_device(k, "bf16"), hip.to_device(v, "bf16")
        cache.append_message(kd.data_ptr(), vd.data_ptr(), len(k))
        torch.cuda.synchronize()
    cache.set_key_gather(gather)
    calls = [Call([(2, 5 * i), (0, 340), (1, 560 - i)], 3 + i, 700, n_q, None) for i in range(n_calls)]
    rows = n_q * n_calls
    q = rnd(rows, h_q, D)
    qd = hip.to_device(q, "bf16")
    res = []
    for tuning in (0, 10000):
        cache.set_tuning(0, tuning)
        out, lse = torch.full_like(qd, 7.0), torch.full((rows, h_q), 7.0, device="cuda:0")
        cache.attend(calls, qd.data_ptr(), out.data_ptr(), lse.data_ptr())
        torch.cuda.synchronize()
        res.append((out.float(), lse))
    cache.close()
    # two sums of the same products: their fp32 difference moves a bf16 rounding here and there (2^-8 of the value)
    assert float((res[0][0] - res[1][0]).norm() / res[1][0].norm()) <= 2e-3
    assert float((res[0][1] - res[1][1]).abs().max()) <= 1e-2
    got = res[0][0].cpu().numpy()
    for i in (0, n_calls - 2, n_calls - 1):
        c = calls[i]
        some = sorted({0, 1, n_q // 2, n_q - 2, n_q - 1})
        o, _ = orc.attend_call(ks, vs, c.sel, c.self_msg, c.self_start, n_q, None, q[n_q * i:n_q * (i + 1)], theta, rows=some)
        d = np.abs(got[[n_q * i + r for r in some]] - o)
        assert d.max() <= 2e-2 and d.mean() <= 1e-3, (i, d.max(), d.mean())
