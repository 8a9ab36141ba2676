"""Device memory that pc_attend_backward of a bf16 cache takes: the queries and partial sums of a run of row blocks, a bounded size
however long the batch, given in pc.h."""
import pytest

from pc_inputs import Call

pytestmark = pytest.mark.gpu


def test_workspace_of_a_long_batch():
    import torch
    from paper_2512_23049_amd import binding
    D, h_q, h_kv, n = 128, 128, 8, 4096                 # 128 row blocks of 128 heads: 16384 units
    k, v = (torch.randn((n, h_kv, D), device="cuda:0").to(torch.bfloat16) for _ in range(2))
    q, g = (torch.randn((n, h_q, D), device="cuda:0").to(torch.bfloat16) for _ in range(2))
    lse = torch.full((n, h_q), 5.0, device="cuda:0")
    d_q = torch.empty((n, h_q, D), device="cuda:0")
    d_k, d_v = (torch.zeros((n, h_kv, D), device="cuda:0") for _ in range(2))
    cache = binding.Cache(h_q, h_kv, D, binding.PC_BF16, 10000.0, n, 1)
    cache.append_message(k.data_ptr(), v.data_ptr(), n)
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    cache.attend_backward([Call([], 0, 0, n, None)], q.data_ptr(), lse.data_ptr(), g.data_ptr(), d_q.data_ptr(), d_k.data_ptr(), d_v.data_ptr())
    torch.cuda.synchronize()
    took = free - torch.cuda.mem_get_info()[0]
    cache.close()
    print("took", took >> 20, "MiB", flush=True)
    # 256 MB and a quarter of it in reserve; the batch's tables are 6 MB, the kernels' own code and scratch memory comes on top
    assert took <= 512 << 20
