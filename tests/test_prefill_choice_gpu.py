"""Which prompt kernel serves batches of whole prompts, on both sides of the lines that the lengths and the heads draw, and
every sampled row of such a batch against the oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_2311_18677_amd import binding as sw
from helpers import assert_parity
from test_prefill_halves_gpu import random_call, serving_kernel

pytestmark = pytest.mark.gpu


def check(n_qh, n_kvh, lens, kernel, spare=0):
    """`spare`: positions that the caches have beyond the longest prompt."""
    n, max_len = len(lens), max(lens) + spare
    call, out = random_call(n_qh, n_kvh, lens, lens, max_len, False)
    assert serving_kernel(call, out) == kernel
    # first and last rows of every request from the oracle, over the caches random_call made
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(sum(lens) + n_qh)
    lay = sw.sw_kv_layout(n, n_kvh, 128, max_len)
    k, v = (torch.randn(lay.total_elems, generator=gen, dtype=torch.float16, device="cuda:0") for _ in range(2))
    q = torch.randn(sum(lens), n_qh, 128, generator=gen, dtype=torch.float16, device="cuda:0")
    k_host, v_host, q_host = (x.cpu().numpy().view(np.uint16) for x in (k, v, q))
    got = out.cpu().numpy()
    for t in (0, 31, 32, -1):
        rows = [sum(lens[:r]) + t % L for r, L in enumerate(lens)]
        ref = oracle.decode_attn(np.ascontiguousarray(q_host[rows]), k_host, v_host, np.array([t % L + 1 for L in lens], np.int32),
                                 n, n_qh, n_kvh, 128, max_len, lay.stride_req, lay.stride_kvh, lay.stride_tok)
        assert_parity(got[rows], ref, "token %d" % t)


@pytest.mark.parametrize("n_qh,n_kvh,lens,kernel", [
    (40, 8, [63] * 13, 1), (10, 1, [110] * 28, 1), (15, 1, [36] * 60, 1), (6, 2, [147] * 42, 1),
    (40, 8, [63] * 12, 2),                                  # 184 workgroups
])
def test_short_prompts_whose_heads_do_not_fill_the_waves(n_qh, n_kvh, lens, kernel):
    """Counted as they are launched, not as if all their waves computed."""
    check(n_qh, n_kvh, lens, kernel)


@pytest.mark.parametrize("n_qh,n_kvh,lens,spare,kernel", [
    (8, 1, [2996] + [214] * 12, 0, 2), (5, 5, [4638] + [117] * 37, 0, 2), (2, 1, [16012] + [254] * 61, 0, 2),
    (64, 8, [800, 40, 30], 0, 2), (8, 1, [4962] + [619] * 6, 0, 2), (8, 8, [4000, 2700, 1000, 1000], 0, 2),
    (8, 1, [371] * 14, 0, 1), (8, 1, [371] * 14, 4096, 2),      # ... as far as the caches' positions tell
    (8, 1, [343] * 14, 0, 1), (8, 1, [342] * 14, 0, 2),         # 150 full workgroups and 149, tokens of all alike
    (8, 1, [500] + [360] * 14, 0, 1), (8, 1, [530] + [358] * 14, 0, 2),         # 152 and 148 against the longest
    (64, 8, [94] * 8, 50, 1), (14, 14, [206] * 17, 60, 1),      # short chains
    (16, 1, [960] * 3, 0, 1), (16, 1, [950] * 3, 0, 2),         # 180 and 178
    (5, 5, [1370] * 9, 0, 1), (5, 5, [1360] * 9, 0, 2),         # 240 and 238
    (5, 5, [1600] + [1480] * 8, 0, 1), (5, 5, [1800] + [1455] * 8, 0, 2),     # 250 and 228 against the longest
    (3, 3, [3125] * 8, 0, 1), (3, 3, [3250] + [3108] * 7, 0, 2),              # 292 and 282
])
def test_lengths_apart(n_qh, n_kvh, lens, spare, kernel):
    """A batch moves to the shared-tile kernel where its longest prompt can be no longer than its mean allows."""
    check(n_qh, n_kvh, lens, kernel, spare)


@pytest.mark.parametrize("n_qh,n_kvh,lens,kernel", [
    (5, 1, [5000, 5000], 3), (5, 1, [4799, 4800], 2),           # 312 workgroups of five waves, 299
    (7, 1, [3200, 3200, 3200], 3), (7, 1, [3505, 3505, 3505], 3), (7, 1, [7000, 1760, 1790], 3),
    (7, 1, [3680, 3680, 3679], 3), (7, 1, [3680, 3680, 3680], 1),               # 344 of seven and 345, below 5000 tokens
    (7, 1, [6400, 6399], 3), (7, 1, [6400, 6400], 1),           # 399 and 400
    (3, 1, [8000, 6500], 2),                                    # 226 of six; threes have no part in this
])
def test_whole_prompts_of_groups_of_five_and_seven(n_qh, n_kvh, lens, kernel):
    check(n_qh, n_kvh, lens, kernel)


@pytest.mark.parametrize("n_qh,n_kvh,lens,spare,kernel", [
    (2, 1, [13035] + [1302] * 8, 0, 2), (1, 1, [25148] + [1478] * 15, 0, 2), (8, 1, [5400, 500, 1], 0, 2),
    (8, 1, [4600, 2300], 0, 2), (8, 1, [4800, 2400], 0, 3),     # 432 and 450: as before, whatever the lengths
    (8, 1, [7000, 200, 200], 0, 3), (6, 2, [9300, 200], 0, 2),  # ... but with eight waves filled
    (8, 1, [1840] * 3, 0, 3), (8, 1, [1830] * 3, 0, 2),         # 345 and 344 of 1400 tokens and more
    (8, 1, [1399] * 4, 0, 2), (8, 1, [1400] * 4, 0, 3),
    (8, 1, [2270, 1900, 1350], 500, 3), (8, 1, [2270, 1900, 1350], 520, 2),     # 250 and 249 against the longest
    (8, 1, [1100] * 6, 0, 3), (8, 1, [1099] * 6, 0, 2),         # 413
    (6, 2, [1000] * 10, 0, 3), (6, 2, [999] * 10, 0, 1),        # 470: tokens, of groups of three
    (12, 4, [2490, 2500], 0, 3), (8, 1, [2500, 2480, 2520, 1170], 0, 2),        # two of them; 542 of 2167
    (4, 2, [2500] * 7, 0, 3), (4, 2, [2499] * 7, 0, 1),         # 547: tokens
    (8, 1, [3090] * 3, 0, 3), (8, 1, [3110] * 3, 0, 1),         # 580 and 584, below 4500 tokens
    (8, 1, [4700, 4620], 0, 3), (8, 1, [4480, 4830], 0, 3),     # 583, not below
    (4, 2, [5440] * 4, 0, 3), (4, 2, [5450] * 4, 0, 1),         # 680 and 682
])
def test_lines_of_the_halves_kernel(n_qh, n_kvh, lens, spare, kernel):
    check(n_qh, n_kvh, lens, kernel, spare)
