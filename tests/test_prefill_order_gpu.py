"""Items of a batch found by a scan of the lengths, numbered by work (shared-tile and halves kernels) or request by
request: every query block of every request is served once, whatever the lengths.  Rows are those of the request in a call
of its own, bit for bit (one request is numbered as it comes); 65 requests take the other numbering.
And the kernel that serves prompts of one or two rounds of the halves kernel's workgroups, and which batches are
scanned."""
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


@pytest.mark.parametrize("n_qh,n_kvh,lens,items,parts", [
    (14, 2, [1944] + [1300] * 9, 53 + 20, 7),              # items of 256, of 80; as blocks of 32 446 of 610
    (14, 2, [1944] + [1800] * 9, 80, 7),                   # 590 of 610
    (6, 2, [1500] + [1100] * 6, 31 + 14, 3),               # items of 256, of 42; as blocks of 64 140 of 168
    (6, 2, [1300] + [1200] * 6, 42, 3),                    # 146 of 147
])
def test_which_batches_of_flat_columns_the_shared_tile_kernel_scans(n_qh, n_kvh, lens, items, parts):
    """By how much of the grid of whole heads a scan removes, whose blocks are finer than a flat item."""
    assert grid_of(n_qh, n_kvh, lens, 1) == items * n_kvh * parts


def exact_rows(q, k, v, lay, r, L, first, n_qh, n_kvh):
    """Request r's rows from position `first` on, in 64 bits: q its query rows [L - first, n_qh, 128]."""
    rows = [x.as_strided((n_kvh, L, 128), (lay.stride_kvh, lay.stride_tok, 1), r * lay.stride_req).double() for x in (k, v)]
    ref = torch.empty(L - first, n_qh, 128, dtype=torch.float64, device=q.device)
    for h in range(n_qh):
        kt, vg = rows[0][h // (n_qh // n_kvh)].t().contiguous(), rows[1][h // (n_qh // n_kvh)].contiguous()
        for a in range(0, L - first, 1024):
            b = min(a + 1024, L - first)
            later = torch.arange(L, device=q.device)[None, :] > (first + torch.arange(a, b, device=q.device))[:, None]
            ref[a:b, h] = torch.softmax((q[a:b, h].double().contiguous() @ kt / 128 ** 0.5).masked_fill_(later, -float("inf")), dim=-1) @ vg
    return ref


# cut: query rows that the first and the last request lack
@pytest.mark.parametrize("n_qh,n_kvh,lens,cut", [
    (16, 1, [3400, 133, 500], (0, 0)), (16, 1, [3400, 133, 500], (100, 70)),        # one column of waves a head: blocks of 32
    (32, 8, [1910, 136], (0, 0)), (32, 8, [1910, 136], (34, 10)),
    (8, 1, [5000, 1, 33, 700, 1500, 64, 400], (0, 0)), (8, 1, [5000, 1, 33, 700, 1500, 64, 400], (99, 71)),
    (4, 2, [9000, 6000, 65, 1, 300], (0, 0)), (4, 2, [9000, 6000, 65, 1, 300], (200, 64)),         # two: of 64
    (8, 8, [4000, 130, 2700, 1000], (0, 0)), (8, 8, [4000, 130, 2700, 1000], (300, 128)),          # four: of 128
    (6, 2, [4500, 4200, 700, 33], (0, 0)), (6, 2, [4500, 4200, 800, 33], (99, 20)),                # columns dealt flat: of 128
    (12, 4, [2500, 1500, 1000], (0, 0)), (12, 4, [2600, 1500, 1100], (129, 64)), (6, 1, [4000, 3990, 1200, 40], (65, 1)),    # and of 64
])
def test_every_row_of_an_uneven_batch_in_the_halves_kernel(n_qh, n_kvh, lens, cut):
    """Blocks of several requests numbered by work: every row is written and within the parity bound of 64 bits, rows
    outside [0, n_tokens) are left out, and block tables give the same bits."""
    n, max_len, bs = len(lens), max(lens), 16
    tot = sum(lens) - sum(cut)
    starts = [sum(lens[:r]) - cut[0] for r in range(n)]
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(tot)

    def rand(*shape):
        return torch.randn(*shape, generator=gen, dtype=torch.float16, device="cuda:0")
    lay = sw.sw_kv_layout(n, n_kvh, 128, max_len)
    k, v, q = rand(lay.total_elems), rand(lay.total_elems), rand(tot, n_qh, 128)
    out, paged = torch.zeros_like(q), torch.full_like(q, float("nan"))
    seq, first = i32(lens), i32(starts)

    def call():
        sw.sw_prefill_attn(q, k, v, seq, first, out, tot, n, n_qh, n_kvh, 128, max_len)
    assert serving_kernel(call, out) == 3
    out.fill_(float("nan"))
    call()
    for r, L in enumerate(lens):
        lo, hi = max(0, -starts[r]), min(L, tot - starts[r])
        if hi > lo:
            # (the rows that are missing at the end attend to nothing that the others see)
            ref = exact_rows(q[starts[r] + lo:starts[r] + hi], k, v, lay, r, hi, lo, n_qh, n_kvh)
            assert_parity(out[starts[r] + lo:starts[r] + hi].cpu().numpy(), ref.cpu().numpy(), "request %d" % r)
    mb = -(-max_len // bs)
    lay_p = sw.sw_kv_paged_layout(n * mb, n_kvh, 128, bs)
    table = torch.randperm(n * mb, generator=gen, device="cuda:0").to(torch.int32).view(n, mb).contiguous()
    kp, vp = rand(lay_p.total_elems), rand(lay_p.total_elems)
    sw.sw_kv_unpack(k, v, table, seq, kp, vp, n, n_kvh, 128, max_len, bs, mb, n * mb)
    sw.sw_prefill_attn_paged(q, kp, vp, table, seq, first, paged, tot, n, n_qh, n_kvh, 128, bs, mb, n * mb)
    torch.cuda.synchronize()
    assert torch.equal(paged.view(torch.int16), out.view(torch.int16))
