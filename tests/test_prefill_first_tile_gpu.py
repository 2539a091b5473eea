"""The first tiles of the prompt kernels, whose weights' rest goes into the second product as well: the shared-tile
kernel's rows are no further from 64 bits than the key-split kernel's wherever they lie in a prompt, a row's bits do not
depend on where its block of queries begins, infinities in those tiles' V rows arrive as they are, and a query that is not
finite costs its neighbours nothing."""
import pytest
import torch

from paper_2311_18677_amd import binding as sw
from test_prefill_order_gpu import exact_rows, i32

pytestmark = pytest.mark.gpu

EDGES = (0, 128, 256, 512, 1024, 2048)


def rand(gen, *shape):
    return torch.randn(*shape, generator=gen, dtype=torch.float16, device="cuda:0")


@pytest.mark.parametrize("n_qh,n_kvh,lens", [
    (8, 1, [371] * 14), (12, 4, [1001, 900, 1100, 77]), (5, 5, [1488] * 4), (7, 1, [2300, 1400]), (1, 1, [128] * 40),
    (8, 1, [1840] * 3), (7, 1, [3505] * 3),             # by default in the halves kernel
])
def test_no_further_from_64_bits_than_the_key_split_kernel_in_any_range(n_qh, n_kvh, lens):
    """A row has one maximum in the shared-tile kernel, two in the halves kernel, whose own keys' weights are exact, against
    four in the key-split kernel; by default (0) a call has one of these three.  An error's norm
    over n values whose roundings are independent is good to one part in sqrt(2 n); four of that are let pass."""
    n, max_len, tot = len(lens), max(lens), sum(lens)
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(tot + n_qh)
    lay = sw.sw_kv_layout(n, n_kvh, 128, max_len)
    k, v, q = rand(gen, lay.total_elems), rand(gen, lay.total_elems), rand(gen, tot, n_qh, 128)
    starts = [sum(lens[:r]) for r in range(n)]
    got = {}
    try:
        for kernel in (0, 1, 2):
            sw.sw_set_param(sw.SW_PARAM_PREFILL_KERNEL, kernel)
            got[kernel] = torch.zeros_like(q)
            sw.sw_prefill_attn(q, k, v, i32(lens), i32(starts), got[kernel], tot, n, n_qh, n_kvh, 128, max_len)
            torch.cuda.synchronize()
    finally:
        sw.sw_set_param(sw.SW_PARAM_PREFILL_KERNEL, 0)
    err = {kernel: [0.0] * len(EDGES) for kernel in got}
    values = [0] * len(EDGES)
    for r, L in enumerate(lens):
        ref = exact_rows(q[starts[r]:starts[r] + L], k, v, lay, r, L, 0, n_qh, n_kvh)
        for j, lo in enumerate(EDGES):
            rows = slice(lo, min(L, EDGES[j + 1] if j + 1 < len(EDGES) else L))
            if rows.stop <= lo:
                continue
            values[j] += ref[rows].numel()
            for kernel in got:
                err[kernel][j] += float((got[kernel][starts[r]:starts[r] + L][rows].double() - ref[rows]).square().sum())
    for kernel in (0, 1):
        ratio = [(err[kernel][j] / err[2][j]) ** 0.5 for j in range(len(EDGES)) if values[j]]
        print("kernel %d, error over the key-split kernel's, by position from %s on: %s" % (kernel, EDGES, ["%.4f" % x for x in ratio]))
        for x, count in zip(ratio, values):
            assert x <= 1 + 4 / (2 * count) ** 0.5


@pytest.mark.parametrize("n_qh,n_kvh", [(8, 1), (3, 1), (1, 1)])
@pytest.mark.parametrize("first", [5, 100, 127, 150])
def test_a_prompt_in_pieces_has_the_bits_of_the_whole(n_qh, n_kvh, first):
    """Pieces whose first query is no multiple of 32: rows of a wave lie on both sides of any position."""
    L = 1300 if n_qh == 3 else 300
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(L + first + n_qh)
    lay = sw.sw_kv_layout(1, n_kvh, 128, L)
    k, v, q = rand(gen, lay.total_elems), rand(gen, lay.total_elems), rand(gen, L, n_qh, 128)
    whole, pieces = (torch.full_like(q, float("nan")) for _ in range(2))
    sw.sw_set_param(sw.SW_PARAM_PREFILL_KERNEL, 1)
    try:
        sw.sw_prefill_attn(q, k, v, i32([L]), i32([0]), whole, L, 1, n_qh, n_kvh, 128, L)
        for lo, hi in ((0, first), (first, L)):
            sw.sw_mixed_attn(q[lo:hi], k, v, i32([hi]), i32([0]), i32([hi - lo]), pieces[lo:hi], hi - lo, 1, n_qh, n_kvh, 128, L, hi - lo)
        torch.cuda.synchronize()
    finally:
        sw.sw_set_param(sw.SW_PARAM_PREFILL_KERNEL, 0)
    assert not torch.isnan(whole).any()
    assert torch.equal(pieces.view(torch.int16), whole.view(torch.int16))


@pytest.mark.parametrize("kernel", [0, 1, 2])
@pytest.mark.parametrize("n_qh,n_kvh,L,row", [(8, 1, 200, 0), (8, 1, 200, 63), (12, 4, 1200, 17), (64, 8, 870, 45)])
def test_infinities_in_v_keep_their_sign(n_qh, n_kvh, L, row, kernel):
    """Row `row` of V, of the first two tiles, is infinite in two dims: the queries behind it see
    its sign there, and the other dims as without it.  (By default one prompt of 870 tokens takes the halves kernel.)"""
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(L + row)
    lay = sw.sw_kv_layout(1, n_kvh, 128, L)
    k, v, q = rand(gen, lay.total_elems), rand(gen, lay.total_elems), rand(gen, L, n_qh, 128)
    heads = v.as_strided((n_kvh, L, 128), (lay.stride_kvh, lay.stride_tok, 1))
    outs = []
    sw.sw_set_param(sw.SW_PARAM_PREFILL_KERNEL, kernel)
    try:
        for spoil in (False, True):
            if spoil:
                heads[:, row, 3], heads[:, row, 64] = float("inf"), float("-inf")
            outs.append(torch.zeros_like(q))
            sw.sw_prefill_attn(q, k, v, i32([L]), i32([0]), outs[-1], L, 1, n_qh, n_kvh, 128, L)
            torch.cuda.synchronize()
    finally:
        sw.sw_set_param(sw.SW_PARAM_PREFILL_KERNEL, 0)
    plain, spoiled = outs[0][row:], outs[1][row:]
    assert (spoiled[:, :, 3] == float("inf")).all() and (spoiled[:, :, 64] == float("-inf")).all()
    others = [d for d in range(128) if d not in (3, 64)]
    # (without the rest of the first tile's weights: either is within the parity bound of 64 bits)
    assert (spoiled[:, :, others].float() - plain[:, :, others].float()).abs().max().item() <= 4e-3


@pytest.mark.parametrize("kernel", [0, 1])
@pytest.mark.parametrize("n_qh,n_kvh,L", [(8, 1, 200), (12, 4, 1200), (64, 8, 870)])
def test_a_query_that_is_not_finite_changes_no_other_row(n_qh, n_kvh, L, kernel):
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(L)
    lay = sw.sw_kv_layout(1, n_kvh, 128, L)
    k, v, q = rand(gen, lay.total_elems), rand(gen, lay.total_elems), rand(gen, L, n_qh, 128)
    outs, bad = [], [0, 45, 100, L - 1]
    sw.sw_set_param(sw.SW_PARAM_PREFILL_KERNEL, kernel)
    try:
        for spoil in (False, True):
            if spoil:
                q[bad] = float("nan")
            outs.append(torch.zeros_like(q))
            sw.sw_prefill_attn(q, k, v, i32([L]), i32([0]), outs[-1], L, 1, n_qh, n_kvh, 128, L)
            torch.cuda.synchronize()
    finally:
        sw.sw_set_param(sw.SW_PARAM_PREFILL_KERNEL, 0)
    others = [i for i in range(L) if i not in bad]
    assert torch.isnan(outs[1][bad]).all()
    assert torch.equal(outs[1][others].view(torch.int16), outs[0][others].view(torch.int16))
