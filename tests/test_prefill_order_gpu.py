"""Items of a batch found by a scan of the lengths, numbered by work (shared-tile kernel) or request by
request: every query block of every request is served once, whatever the lengths.  Rows are those of the request in a call
of its own, bit for bit (one request is numbered as it comes); 65 requests take the other numbering.
And the kernel that serves prompts of one or two rounds of the halves kernel's workgroups."""
import numpy as np
import pytest
import torch

import oracle
from paper_2311_18677_amd import binding as sw
from helpers import assert_parity, launches
from test_prefill_halves_gpu import random_call, serving_kernel

pytestmark = pytest.mark.gpu


def i32(a):
    return torch.tensor(a, dtype=torch.int32, device="cuda:0")


@pytest.mark.parametrize("kernel", [1, 2])
@pytest.mark.parametrize("n_qh,n_kvh,reqs", [
    (8, 1, [(600, 600), (500, 500), (400, 400)]),                       # similar lengths: the scan or not
    (6, 2, [(640, 640), (320, 320)]), (2, 2, [(1000, 1000), (3, 3), (990, 990), (1000, 1000)]),
    (8, 1, [(700, 700), (90, 90)]),
    (8, 1, [(1600, 1600), (900, 900)]), (4, 1, [(1100, 1100), (900, 900), (700, 700), (600, 600)]),      # a sixth of a full grid
    (8, 1, [(33, 33), (0, 0), (1, 1), (1500, 1500), (64, 64), (32, 32)]),
    (8, 2, [(2047, 2047), (60, 60), (5, 5)]),                            # 64 levels of 64 tokens or fewer: bands of one
    (8, 1, [(2049, 2049), (31, 31), (40, 40)]),                         # 65 levels: bands of two
    (8, 1, [(9000, 130), (8, 8), (4097, 97), (300, 300), (2600, 65)]),  # pieces behind earlier tokens
    (2, 2, [(1100, 1100), (257, 257), (256, 256), (3, 3)]),             # blocks of 256 queries
    (8, 1, [(20 + 37 * (i % 11) * (i % 3), 20 + 37 * (i % 11) * (i % 3)) for i in range(64)]),
    (8, 1, [(20 + 37 * (i % 11) * (i % 3), 20 + 37 * (i % 11) * (i % 3)) for i in range(65)]),
])
def test_rows_are_those_of_the_request_alone(n_qh, n_kvh, reqs, kernel):
    n, max_len, max_q = len(reqs), max(L for L, _ in reqs), max(q for _, q in reqs)
    tot = sum(q for _, q in reqs)
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(tot)
    lay = sw.sw_kv_layout(n, n_kvh, 128, max_len)
    k, v = (torch.randn(lay.total_elems, generator=gen, dtype=torch.float16, device="cuda:0") for _ in range(2))
    q = torch.randn(tot, n_qh, 128, generator=gen, dtype=torch.float16, device="cuda:0")
    starts = [sum(c for _, c in reqs[:r]) for r in range(n)]
    got, alone = (torch.full_like(q, float("nan")) for _ in range(2))
    sw.sw_set_param(sw.SW_PARAM_PREFILL_KERNEL, kernel)
    try:
        # (q_starts counts rows; single query tokens go through the token phase in either call)
        sw.sw_mixed_attn(q, k, v, i32([L for L, _ in reqs]), i32(starts), i32([c for _, c in reqs]), got, tot, n, n_qh, n_kvh,
                         128, max_len, max_q)
        one = lay.stride_req
        for r, (L, c) in enumerate(reqs):
            if c > 0:
                rows = slice(starts[r], starts[r] + c)
                sw.sw_mixed_attn(q[rows], k[r * one:(r + 1) * one], v[r * one:(r + 1) * one], i32([L]), i32([0]), i32([c]),
                                 alone[rows], c, 1, n_qh, n_kvh, 128, max_len, max_q)
        torch.cuda.synchronize()
    finally:
        sw.sw_set_param(sw.SW_PARAM_PREFILL_KERNEL, 0)
    assert not torch.isnan(got).any()
    assert torch.equal(got.view(torch.int16), alone.view(torch.int16))


@pytest.mark.parametrize("n_qh,n_kvh,lens,kernel", [
    (8, 1, [5344], 2), (8, 1, [5376], 3),                  # 334 and 336 of its workgroups
    (8, 1, [3500, 3600], 2), (8, 1, [3600, 3560], 3),      # 444 and 448
    (32, 8, [999, 1000], 2), (32, 8, [1000, 1010], 3),     # tokens of a request
    (16, 1, [2050, 1030, 1000], 3), (16, 1, [2080, 1030, 1000], 2),      # 512 and 516
    (28, 4, [1499], 2), (28, 4, [1500], 3),                # blocks of 128 positions: tokens
    (8, 8, [1499, 1498, 1499, 1500, 1499], 2), (8, 8, [1500] * 5, 3),
])
def test_the_kernel_that_serves_whole_prompts(n_qh, n_kvh, lens, kernel):
    call, out = random_call(n_qh, n_kvh, lens, lens, max(lens), False)
    assert serving_kernel(call, out) == kernel
    call()
    torch.cuda.synchronize()
    # first and last rows of every request from the oracle, over the caches random_call made
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(sum(lens) + n_qh)
    n, max_len = len(lens), max(lens)
    lay = sw.sw_kv_layout(n, n_kvh, 128, max_len)
    k, v = (torch.randn(lay.total_elems, generator=gen, dtype=torch.float16, device="cuda:0") for _ in range(2))
    q = torch.randn(sum(lens), n_qh, 128, generator=gen, dtype=torch.float16, device="cuda:0")
    k_host, v_host, q_host = (x.cpu().numpy().view(np.uint16) for x in (k, v, q))
    got = out.cpu().numpy()
    for t in (0, 31, 32, 700, -33, -1):
        rows = [sum(lens[:r]) + t % L for r, L in enumerate(lens)]
        ref = oracle.decode_attn(np.ascontiguousarray(q_host[rows]), k_host, v_host, np.array([t % L + 1 for L in lens], np.int32),
                                 n, n_qh, n_kvh, 128, max_len, lay.stride_req, lay.stride_kvh, lay.stride_tok)
        assert_parity(got[rows], ref, "token %d" % t)


def grid_of(n_qh, n_kvh, lens, kernel):
    """Workgroups that the prompt kernel (SW_PARAM_PREFILL_KERNEL) is launched with."""
    n, tot, max_len = len(lens), sum(lens), max(lens)
    k, v = (torch.zeros(sw.sw_kv_layout(n, n_kvh, 128, max_len).total_elems, dtype=torch.float16, device="cuda:0") for _ in range(2))
    q = torch.zeros(tot, n_qh, 128, dtype=torch.float16, device="cuda:0")
    out, seq, first = torch.empty_like(q), i32(lens), i32([sum(lens[:r]) for r in range(n)])
    torch.cuda.synchronize()
    sw.sw_set_param(sw.SW_PARAM_PREFILL_KERNEL, kernel)
    try:
        (grid, _), = launches(lambda s: sw.sw_prefill_attn(q, k, v, seq, first, out, tot, n, n_qh, n_kvh, 128, max_len, stream=s))
    finally:
        sw.sw_set_param(sw.SW_PARAM_PREFILL_KERNEL, 0)
    return grid


@pytest.mark.parametrize("n_qh,n_kvh,lens,items", [
    # blocks of 32 query tokens by shape (requests x blocks of the longest), or by rows where the lengths are scanned
    (1, 1, [960 + r for r in range(17)] + [900], 18 * 31),        # 545 by rows: late blocks of all requests first
    (2, 2, [915, 1044, 986, 956, 963, 1042], 6 * 33),             # 196
    (8, 1, [1600, 1000], 2 * 50),                                 # 85: less than 15 % of the grid
    (8, 1, [1600, 900], 78 + 4),                                  # 82 of 100
    (2, 1, [1600, 900], 2 * 50),                                  # ... of a grid that the chip holds at once
    (8, 8, [1600, 900], 2 * 50),                                  # ... where a request's pairs reach all XCDs
    (8, 1, [700, 90], 24 + 4),                                    # of 44: a good part
])
def test_which_batches_the_key_split_kernel_scans(n_qh, n_kvh, lens, items):
    # (pairs of a block and a key/value head come in eights)
    assert grid_of(n_qh, n_kvh, lens, 2) == (items * n_kvh + 7) // 8 * 8 * (n_qh // n_kvh)


@pytest.mark.parametrize("n_qh,n_kvh,lens,items", [
    (32, 8, [2133, 1066], 49 + 4),                         # blocks of 64: of 68, long chains
    (32, 8, [2133, 1900], 2 * 34),                         # 66: less than a tenth
    (40, 8, [227] * 38 + [297], 39 * 10),                  # blocks of 32: 356, many rounds of short chains
    (64, 16, [501] + [250] * 23, 24 * 8),                  # 145 of 192, the same
    (64, 16, [501] + [200] * 23, 79 + 48),                 # of 192: a good part anyway
])
def test_which_batches_the_shared_tile_kernel_scans(n_qh, n_kvh, lens, items):
    assert grid_of(n_qh, n_kvh, lens, 1) == items * n_kvh             # (all heads of a group in one workgroup)
