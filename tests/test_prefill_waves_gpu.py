"""Waves per workgroup of the key-split prompt kernel, chosen by the call's size: on both sides of
every line of the rule the result is that of the named number of waves, dense and over blocks, and
within the library's parity bound against the oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_2311_18677_amd import binding as sw
from helpers import MAX_ABS, MAX_REL_L2, assert_parity, parity_errors

pytestmark = pytest.mark.gpu


def i32(a):
    return torch.tensor(a, dtype=torch.int32, device="cuda:0")


@pytest.mark.parametrize("n_qh,n_kvh,lens,waves", [
    (2, 1, [899], 4), (2, 1, [900], 8),                     # tokens of a request
    (3, 1, [900, 899], 4), (3, 1, [999, 825], 8),           # their mean
    (8, 2, [1154], 4), (8, 2, [1150], 8),                   # 296 and 288 workgroups of short chains
    (6, 6, [1859], 4), (5, 5, [1859], 8),                   # 354 and 295 of long ones
    (4, 2, [4097], 4), (4, 2, [4096], 8),                   # 516 and 512
])
def test_waves_by_size(n_qh, n_kvh, lens, waves):
    bs, n, tot, max_len = 16, len(lens), sum(lens), max(lens) + 3
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(tot)

    def rand(*shape):
        return torch.randn(*shape, generator=gen, dtype=torch.float16, device="cuda:0")
    lay = sw.sw_kv_layout(n, n_kvh, 128, max_len)
    k, v, q = rand(lay.total_elems), rand(lay.total_elems), rand(tot, n_qh, 128)
    starts = [sum(lens[:r]) for r in range(n)]
    out, paged = torch.zeros_like(q), torch.zeros_like(q)
    seq, first = i32(lens), i32(starts)
    # the same rows in blocks
    mb = -(-max_len // bs)
    lay_p = sw.sw_kv_paged_layout(n * mb, n_kvh, 128, bs)
    table = torch.randperm(n * mb, generator=gen, device="cuda:0").to(torch.int32).view(n, mb).contiguous()
    kp, vp = rand(lay_p.total_elems), rand(lay_p.total_elems)
    sw.sw_kv_unpack(k, v, table, seq, kp, vp, n, n_kvh, 128, max_len, bs, mb, n * mb)

    def call(o):
        sw.sw_prefill_attn(q, k, v, seq, first, o, tot, n, n_qh, n_kvh, 128, max_len)
    bits = []
    try:
        for kernel, w in ((0, 0), (2, 0), (2, 4), (2, 8)):
            sw.sw_set_param(sw.SW_PARAM_PREFILL_KERNEL, kernel)
            sw.sw_set_param(sw.SW_PARAM_PREFILL_WAVES, w)
            out.zero_()
            call(out)
            bits.append(out.view(torch.int16).clone())
    finally:
        sw.sw_set_param(sw.SW_PARAM_PREFILL_KERNEL, 0)
        sw.sw_set_param(sw.SW_PARAM_PREFILL_WAVES, 0)
    sw.sw_prefill_attn_paged(q, kp, vp, table, seq, first, paged, tot, n, n_qh, n_kvh, 128, bs, mb, n * mb)
    torch.cuda.synchronize()
    want, other = (bits[3], bits[2]) if waves == 8 else (bits[2], bits[3])
    assert torch.equal(bits[0], want) and torch.equal(bits[1], want) and not torch.equal(want, other)
    assert torch.equal(paged.view(torch.int16), want)
    # a sample of the rows from the oracle: around every ninth edge of a query block, and the last
    got = bits[0].cpu().numpy().view(np.float16).reshape(tot, n_qh, 128)
    k_host, v_host, q_host = (x.cpu().numpy().view(np.uint16) for x in (k, v, q))
    for r, L in enumerate(lens):
        for t in sorted({min(L - 1, 288 * b + o) for b in range(L // 288 + 1) for o in (0, 31)} | {L - 1}):
            at, row = np.array([0] * r + [t + 1] + [0] * (n - r - 1), np.int32), starts[r] + t
            qs = np.zeros((n, n_qh, 128), np.uint16)
            qs[r] = q_host[row]
            ref = oracle.decode_attn(qs, k_host, v_host, at, n, n_qh, n_kvh, 128, max_len, lay.stride_req, lay.stride_kvh,
                                     lay.stride_tok)
            assert_parity(got[row:row + 1], ref[r:r + 1], "request %d token %d" % (r, t))


@pytest.mark.parametrize("n_qh,n_kvh,L,others", [
    (2, 1, 1000, [1000] * 11),                              # 64 workgroups alone, 750 in the batch
    (2, 1, 4000, [4000, 3990, 17]),
    (8, 2, 1150, [64, 1]),                                  # the batch's mean is below the rule's line
    (1, 1, 9000, [8990, 9000]),
])
def test_a_prompt_alone_and_in_a_batch_on_the_other_side_of_the_rule(n_qh, n_kvh, L, others):
    """With kernel and waves named, the prompt's rows have the same bits; by default, where the two calls take eight
    and four waves, they are the named ones' of those numbers, within the parity bounds."""
    lens = [L] + others
    n, tot, max_len = len(lens), sum(lens), max(lens)
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(tot)
    lay = sw.sw_kv_layout(n, n_kvh, 128, max_len)
    k, v = (torch.randn(lay.total_elems, generator=gen, dtype=torch.float16, device="cuda:0") for _ in range(2))
    q = torch.randn(tot, n_qh, 128, generator=gen, dtype=torch.float16, device="cuda:0")
    starts = [sum(lens[:r]) for r in range(n)]

    def rows(kernel, waves):
        batch, alone = torch.full_like(q, float("nan")), torch.full_like(q[:L], float("nan"))
        sw.sw_set_param(sw.SW_PARAM_PREFILL_KERNEL, kernel)
        sw.sw_set_param(sw.SW_PARAM_PREFILL_WAVES, waves)
        try:
            sw.sw_prefill_attn(q, k, v, i32(lens), i32(starts), batch, tot, n, n_qh, n_kvh, 128, max_len)
            sw.sw_prefill_attn(q[:L], k, v, i32([L]), i32([0]), alone, L, 1, n_qh, n_kvh, 128, max_len)
            torch.cuda.synchronize()
        finally:
            sw.sw_set_param(sw.SW_PARAM_PREFILL_KERNEL, 0)
            sw.sw_set_param(sw.SW_PARAM_PREFILL_WAVES, 0)
        assert not torch.isnan(batch).any()
        return batch[:L].view(torch.int16), alone.view(torch.int16)
    named = {}
    for waves in (4, 8):
        batch, alone = rows(2, waves)
        assert torch.equal(batch, alone)
        named[waves] = alone
    assert not torch.equal(named[4], named[8])
    batch, alone = rows(1, 0)
    assert torch.equal(batch, alone)
    for kernel in (0, 2):
        batch, alone = rows(kernel, 0)
        assert torch.equal(alone, named[8]) and torch.equal(batch, named[4])
    # either is within the bound of the exact rows, so the two are within twice the bound of each other
    four, eight = (named[w].view(torch.float16).cpu().numpy() for w in (4, 8))
    max_abs, rel, _ = parity_errors(four, eight.astype(np.float64))
    assert max_abs <= 2 * MAX_ABS and rel <= 2 * MAX_REL_L2
