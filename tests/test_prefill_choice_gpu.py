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
