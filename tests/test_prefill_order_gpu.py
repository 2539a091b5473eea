"""Items of a batch numbered by work (shared-tile kernel, 2 to 64 requests): every query block of every
request is served once, whatever the lengths.  Rows are those of the request in a call of its own, bit
for bit (one request is numbered as it comes); 65 requests take the other numbering."""
import pytest
import torch

from paper_2311_18677_amd import binding as sw

pytestmark = pytest.mark.gpu


def i32(a):
    return torch.tensor(a, dtype=torch.int32, device="cuda:0")


@pytest.mark.parametrize("n_qh,n_kvh,reqs", [
    (8, 1, [(700, 700), (90, 90)]),
    (8, 1, [(33, 33), (0, 0), (1, 1), (1500, 1500), (64, 64), (32, 32)]),
    (8, 2, [(2047, 2047), (60, 60), (5, 5)]),                            # 64 levels of 64 tokens or fewer: bands of one
    (8, 1, [(2049, 2049), (31, 31), (40, 40)]),                         # 65 levels: bands of two
    (8, 1, [(9000, 130), (8, 8), (4097, 97), (300, 300), (2600, 65)]),  # pieces behind earlier tokens
    (2, 2, [(1100, 1100), (257, 257), (256, 256), (3, 3)]),             # blocks of 256 queries
    (8, 1, [(20 + 37 * (i % 11) * (i % 3), 20 + 37 * (i % 11) * (i % 3)) for i in range(64)]),
    (8, 1, [(20 + 37 * (i % 11) * (i % 3), 20 + 37 * (i % 11) * (i % 3)) for i in range(65)]),
])
def test_rows_are_those_of_the_request_alone(n_qh, n_kvh, reqs):
    n, max_len, max_q = len(reqs), max(L for L, _ in reqs), max(q for _, q in reqs)
    tot = sum(q for _, q in reqs)
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(tot)
    lay = sw.sw_kv_layout(n, n_kvh, 128, max_len)
    k, v = (torch.randn(lay.total_elems, generator=gen, dtype=torch.float16, device="cuda:0") for _ in range(2))
    q = torch.randn(tot, n_qh, 128, generator=gen, dtype=torch.float16, device="cuda:0")
    starts = [sum(c for _, c in reqs[:r]) for r in range(n)]
    got, alone = (torch.full_like(q, float("nan")) for _ in range(2))
    sw.sw_set_param(sw.SW_PARAM_PREFILL_KERNEL, 1)
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
