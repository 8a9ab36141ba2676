"""Call lists of every size class: passed in the plan builder's arguments (up to 3.5 KB), read by it from pinned memory (up to
256 KB), copied in front of it; bf16 and fp32, against the oracle, several different batches in a row through the same ring."""
import numpy as np
import pytest

import pc_inputs as gen
from pc_inputs import Call

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,h_q,h_kv,D", [("bf16", 8, 2, 128), ("f32", 4, 2, 64)])
@pytest.mark.parametrize("shape", [[(1, 2, 1)] * 6, [(4, 90, 1), (4, 96, 1), (5, 100, 1), (1, 380, 1), (1, 420, 3)], [(8, 300, 1), (3, 10, 200), (70, 480, 1), (2, 4, 40)]])
def test_list_sizes(dtype, h_q, h_kv, D, shape):
    """shape: batches of (calls, listed messages, query rows)."""
    import torch
    from oracle import choreo_oracle as orc
    from paper_2512_23049_amd import binding, harness as hip
    rng = np.random.default_rng(len(shape))
    rows_most = max(n for _, _, n in shape)
    lens = [1, 2, 3, 1, 40, 1, 2] + [rows_most + 1]

    def rnd(*s):
        x = rng.standard_normal(s).astype(np.float32)
        return gen.round_to_bf16(x) if dtype == "bf16" else x
    ks, vs = [rnd(L, h_kv, D) for L in lens], [rnd(L, h_kv, D) for L in lens]
    cache = binding.Cache(h_q, h_kv, D, binding.PC_BF16 if dtype == "bf16" else binding.PC_F32, 10000.0, 1024, len(lens))
    for k, v in zip(ks, vs):
        kd, vd = hip.to_device(k, dtype), hip.to_device(v, dtype)
        cache.append_message(kd.data_ptr(), vd.data_ptr(), len(k))
        torch.cuda.synchronize()
    cache.set_decode_sharing(1)
    runs = []
    for n_calls, n_sel, n_q in shape:                    # all enqueued before the first is looked at
        calls = [Call([(int(m), int(p)) for m, p in zip(rng.integers(0, 7, n_sel), rng.integers(0, 3000, n_sel))], 7, 3000, n_q,
                      rng.integers(2990, 3400, n_q).astype(np.int32) if i % 2 else None) for i in range(n_calls)]
        q = rnd(n_calls * n_q, h_q, D)
        qd = hip.to_device(q, dtype)
        out = torch.full_like(qd, 7.0)
        torch.cuda.synchronize()
        cache.attend(calls, qd.data_ptr(), out.data_ptr())
        runs.append((calls, q, qd, out, n_q))
    torch.cuda.synchronize()
    cache.close()
    for calls, q, _, out, n_q in runs:
        got = out.float().cpu().numpy()
        for i in {0, 1 % len(calls), len(calls) // 2, len(calls) - 1}:
            c = calls[i]
            o, _ = orc.attend_call(ks, vs, c.sel, c.self_msg, c.self_start, n_q, c.q_pos, q[n_q * i:n_q * (i + 1)], 10000.0, rows=list(range(n_q)))
            d = np.abs(got[n_q * i:n_q * (i + 1)] - o)
            assert d.max() <= (2e-2 if dtype == "bf16" else 1e-4) and d.mean() <= (1e-3 if dtype == "bf16" else 1e-5), (len(calls), len(c.sel), d.max(), d.mean())
