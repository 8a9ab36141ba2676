"""Prefill calls over a packed copy of many short messages: the copy has no padding between messages, so the walk has far fewer
tiles than the messages fill, and it is the walk's tiles that decide how the call is split and in which type the parts are kept."""
import numpy as np
import pytest

from pc_inputs import Call

pytestmark = pytest.mark.gpu
MERGE = "merge"


def walk(h_q, h_kv, lens, n_q, gather, tunings, seed=1):
    """out, lse and the launches of the split merge, for each tuning of the tiles per split (0: the library's own)."""
    import torch
    from paper_2512_23049_amd import binding
    D = 128
    rng = torch.Generator(device="cuda:0")
    rng.manual_seed(seed)
    normal = lambda *s: torch.randn(s, generator=rng, device="cuda:0").to(torch.bfloat16)      # noqa: E731
    lens = list(lens) + [n_q]
    cache = binding.Cache(h_q, h_kv, D, binding.PC_BF16, 10000.0, sum((L + 31) // 32 * 32 for L in lens), len(lens))
    for L in lens:
        k, v = normal(L, h_kv, D), normal(L, h_kv, D)
        cache.append_message(k.data_ptr(), v.data_ptr(), L)
        torch.cuda.synchronize()
    cache.set_key_gather(gather)
    q = normal(n_q, h_q, D)
    at = np.concatenate([[0], np.cumsum(lens[:-1])])
    calls = [Call([(m, int(at[m])) for m in range(len(lens) - 1)], len(lens) - 1, int(at[-1]), n_q, None)]
    res = []
    for t in tunings:
        cache.set_tuning(0, t)
        out, lse = torch.full_like(q, 7.0), torch.full((n_q, h_q), 7.0, device="cuda:0")
        cache.profile_enable(True)
        cache.profile_read(reset=True)
        cache.attend(calls, q.data_ptr(), out.data_ptr(), lse.data_ptr())
        n = cache.profile_read(reset=True)[MERGE][1]
        cache.profile_enable(False)
        res.append((out, lse, n))
    cache.close()
    return res


# Fewer than 32 tiles in the copy, more in the messages: the plain rule (16 tiles a split) leaves such a call whole.  A value whose
# parts move it by a share d of itself before it is rounded to bf16 (steps of 2^-8 to 2^-7 of it, s = 5.5e-3 in the mean) falls on
# another step with probability d / s, so the 2-norm of the difference is sqrt(d s) of the value's.  fp32 parts: the loops of the
# walk sum their probabilities before or after these are rounded (2^-9 / sqrt 3 each), and a split moves tiles from one kind of loop
# to another: d <= 1.1e-3 * 1.65 / sqrt(500 keys) = 8e-5 if every tile changes its kind, 6.6e-4.  fp16 parts: d = 2^-11 / sqrt 12 on
# top, which gives 9.4e-4.
@pytest.mark.parametrize("h_q,h_kv,n_q,n_msgs,msg_len,gather", [(64, 8, 512, 24, 20, 0), (64, 8, 512, 30, 10, 0), (8, 2, 40, 60, 10, 2), (32, 8, 70, 70, 9, 2)])
def test_parts_of_a_short_walk_are_fp32(h_q, h_kv, n_q, n_msgs, msg_len, gather):
    (a, lse_a, _), (b, lse_b, _) = walk(h_q, h_kv, [msg_len] * n_msgs, n_q, gather, (0, 10000))
    a, b = a.float(), b.float()
    rel = float((a - b).norm() / b.norm())
    print("split against whole:", rel, float((lse_a - lse_b).abs().max()), flush=True)
    assert rel <= 6.6e-4


# 512 rows x 64 heads over 480 (300) tokens in 31 (26) tiles: whole, one round of workgroups and no merge, costs less than two parts
@pytest.mark.parametrize("n_msgs,msg_len", [(24, 20), (30, 10)])
def test_split_follows_the_tiles_that_are_walked(n_msgs, msg_len):
    (_, _, many), = walk(64, 8, [msg_len] * n_msgs, 512, 0, (0,))
    (_, _, one), = walk(64, 8, [msg_len * n_msgs], 512, 0, (0,))
    assert many == one == 0
