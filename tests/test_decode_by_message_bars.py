"""What the bars of test_gpu_decode_by_message.py can see: over its shapes, one message of a row that is turned to another position, or left out, moves
some head's output by more than the bar, whichever message it is."""
import numpy as np
import pytest

from tests.test_gpu_decode_by_message import D, OUT_BAR, SHAPES, lengths, value_scale


@pytest.mark.parametrize("h_q,h_kv,n_calls,n_sel,pool", SHAPES)
def test_one_wrong_message_exceeds_the_bar(h_q, h_kv, n_calls, n_sel, pool):
    # N(0,1) queries and keys of 128 dimensions give scores of about N(0,1), and other ones at another position
    r = np.random.default_rng(n_calls)
    lens = lengths(r, pool)
    lens = [lens[0]] + lens[1:n_sel + 1] + lens[-3:]
    total, moved = np.zeros((2, h_q, len(lens))), np.zeros((2, h_q, len(lens), D))      # sums of exp(score), and of values times that; at two positions
    for i, n in enumerate(lens):
        v = value_scale(n) * r.standard_normal((n, D))
        for at in range(2):
            p = np.exp(r.standard_normal((h_q, n)))
            total[at, :, i], moved[at, :, i] = p.sum(1), p @ v
    p, o = total[0].sum(1)[:, None], moved[0].sum(1)[:, None]
    for what, (dp, do) in {"turned": (total[1] - total[0], moved[1] - moved[0]), "left out": (-total[0], -moved[0])}.items():
        far = np.linalg.norm((o + do) / (p + dp)[..., None] - o / p[..., None], axis=-1) / np.linalg.norm(o / p[..., None], axis=-1)
        least = far.max(0).min()                         # of the heads the one that shows most, of the messages the one that shows least
        assert least > 2 * OUT_BAR, (what, least, lens[int(far.max(0).argmin())])
