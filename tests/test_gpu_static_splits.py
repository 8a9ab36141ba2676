"""pc_attend_static returns pc_attend's bits also where the split parts of the batch would fill its fixed workspace: prefill batches
of a few more workgroups than compute units, whose last round pc_attend splits.  Against pc_attend bit for bit and the oracle to the
bf16 bars of test_gpu_parity."""
import numpy as np
import pytest

import pc_inputs as gen
from pc_inputs import Call

pytestmark = pytest.mark.gpu


# 384 groups, 280 groups (parts of 24 of them), 512 whole-round groups, 288 groups of long walks
@pytest.mark.parametrize("n_calls,n_q,parent", [(6, 256, 1660), (5, 200, 600), (8, 256, 300), (9, 128, 3000)])
def test_bits_of_pc_attend(n_calls, n_q, parent):
    import torch
    from oracle import choreo_oracle as orc
    from paper_2512_23049_amd import binding, harness as hip
    h_q, h_kv, D, theta = 64, 8, 128, 10000.0
    rng = np.random.default_rng(n_calls)
    lens = [parent] + [n_q] * n_calls

    def rnd(*shape):
        return gen.round_to_bf16(rng.standard_normal(shape, dtype=np.float32))
    ks, vs = [rnd(L, h_kv, D) for L in lens], [rnd(L, h_kv, D) for L in lens]
    cache = binding.Cache(h_q, h_kv, D, binding.PC_BF16, theta, sum((L + 31) // 32 * 32 for L in lens), len(lens))
    for k, v in zip(ks, vs):
        kd, vd = hip.to_device(k, "bf16"), hip.to_device(v, "bf16")
        cache.append_message(kd.data_ptr(), vd.data_ptr(), len(k))
        torch.cuda.synchronize()
    calls = [Call([(0, 3 * i)], 1 + i, parent + 40, n_q, None) for i in range(n_calls)]
    rows = n_q * n_calls
    q = rnd(rows, h_q, D)
    qd = hip.to_device(q, "bf16")
    res = []
    for entry in (cache.attend, cache.attend_static):
        out, lse = torch.full_like(qd, 7.0), torch.full((rows, h_q), 7.0, device="cuda:0")
        entry(calls, qd.data_ptr(), out.data_ptr(), lse.data_ptr())
        torch.cuda.synchronize()
        res.append((out, lse))
    cache.close()
    assert torch.equal(res[0][0].view(torch.int16), res[1][0].view(torch.int16)) and torch.equal(res[0][1], res[1][1])
    got = res[0][0].float().cpu().numpy()
    for i in (0, n_calls - 1):
        c, some = calls[i], [0, n_q // 2, n_q - 1]
        o, _ = orc.attend_call(ks, vs, c.sel, c.self_msg, c.self_start, n_q, None, q[n_q * i:n_q * (i + 1)], theta, rows=some)
        d = np.abs(got[[n_q * i + r for r in some]] - o)
        assert d.max() <= 2e-2 and d.mean() <= 1e-3, (i, d.max(), d.mean())


# (heads, calls, messages, listed by each; the shared walk): one group, and two of 30 calls, whose tables pass the workspace; one that fits
@pytest.mark.parametrize("h_q,n_calls,pool,n_sel,shared", [(32, 32, 2200, 240, False), (32, 16, 4400, 900, False), (64, 60, 1500, 200, False), (32, 32, 1500, 300, True)])
def test_tables_beyond_the_workspace(h_q, n_calls, pool, n_sel, shared):
    """Decode batches that the shared walk would serve at the least price, with a rotation for every row and message of the union, of which
    each row lists few: where those pass the fixed workspace, both entry points take the calls' own walks."""
    import torch
    from paper_2512_23049_amd import binding
    h_kv, D, L = 8, 128, 20
    r, g = np.random.default_rng(n_calls), torch.Generator(device="cuda:0").manual_seed(pool)
    k, v = (torch.randn((pool * L, h_kv, D), generator=g, device="cuda:0").to(torch.bfloat16) for _ in range(2))
    cache = binding.Cache(h_q, h_kv, D, binding.PC_BF16, 10000.0, pool * 32, pool)
    at = [2 * D * h_kv * L * i for i in range(pool)]
    for i in range(0, pool, 100):
        cache.append_messages([k.data_ptr() + a for a in at[i:i + 100]], [v.data_ptr() + a for a in at[i:i + 100]], [L] * 100)
    calls = [Call([(int(m), int(r.integers(0, 9000))) for m in r.permutation(pool)[:n_sel]], -1, 9000 + i, 1, None) for i in range(n_calls)]
    q = torch.randn((n_calls, h_q, D), generator=g, device="cuda:0").to(torch.bfloat16)

    def run(entry, sharing=0):
        out, lse = torch.full_like(q, 7.0), torch.full((n_calls, h_q), 7.0, device="cuda:0")
        cache.set_decode_sharing(sharing)
        entry(calls, q.data_ptr(), out.data_ptr(), lse.data_ptr())
        torch.cuda.synchronize()
        return out.view(torch.int16), lse
    got, static, own = run(cache.attend), run(cache.attend_static), run(cache.attend, 1)
    assert torch.equal(got[0], static[0]) and torch.equal(got[1], static[1])
    assert torch.equal(got[0], own[0]) != shared
    assert (got[0].view(torch.bfloat16).float() - own[0].view(torch.bfloat16).float()).norm() <= 1e-2 * own[0].view(torch.bfloat16).float().norm()
    cache.close()
