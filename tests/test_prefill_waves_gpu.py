"""Waves per workgroup of the key-split prompt kernel, chosen by the call's size: on both sides of
every line of the rule the result is that of the named number of waves, dense and over blocks, and
within the library's parity bound against the oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_2311_18677_amd import binding as sw
from helpers import assert_parity

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
