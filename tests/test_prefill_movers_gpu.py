"""The shared-tile prompt kernel's moving waves: prompts that end at, before and behind a tile's edge, from one
tile to one round and a half of the three staging buffers, in workgroups of every number of computing waves; over block
tables of every addressing kind the same bits as dense.  Tolerance: the library's parity bound against the oracle.
And columns dealt flat to workgroups: the same bits as with whole heads in each, every row written and within the bound of
64 bits, behind earlier context, over block tables and where rows are missing."""
import numpy as np
import pytest

from paper_2311_18677_amd import binding as sw
from paper_2311_18677_amd import workloads as wl
from helpers import MAX_ABS, MAX_REL_L2, assert_parity
from test_prefill_gpu import run_prefill, to_dev
from test_prefill_order_gpu import exact_rows, i32

pytestmark = pytest.mark.gpu

LENS = [1, 31, 32, 33, 64, 65, 95, 96, 97, 128, 129, 160, 0]


# heads and waves: SW_PARAM_PREFILL_HEADS and _WAVES, whose product is the number of computing waves (0: 8, 7, 6 or 5)
@pytest.mark.parametrize("n_qh,n_kvh,heads,waves", [
    (8, 1, 0, 0), (7, 1, 0, 0), (6, 2, 0, 0), (5, 1, 0, 0), (1, 1, 0, 0), (4, 1, 4, 1), (3, 1, 3, 1), (4, 2, 2, 1), (2, 1, 1, 1),
])
def test_tile_edges(n_qh, n_kvh, heads, waves):
    import torch
    cfg = wl.custom_config("mv%d_%d_%d" % (n_qh, n_kvh, heads), len(LENS), n_qh, n_kvh, 128, 160)
    batch = wl.make_batch(cfg, seed=8100 + n_qh, seq_lens=LENS)
    qt, starts = wl.make_prefill_queries(batch)
    starts_d = torch.from_numpy(np.ascontiguousarray(starts, dtype=np.int32)).to("cuda:0")
    sw.sw_set_param(sw.SW_PARAM_PREFILL_KERNEL, 1)
    sw.sw_set_param(sw.SW_PARAM_PREFILL_HEADS, heads)
    sw.sw_set_param(sw.SW_PARAM_PREFILL_WAVES, waves)
    try:
        dense, ref = run_prefill(batch, qt, starts, tag="movers")
        assert_parity(dense, ref, cfg.name)
        for bs in (4, 8, 16, 32, 128):
            pb = sw.upload_paged_batch(batch, bs, pad_bits=0x7E00)
            out = torch.full(qt.shape, float("nan"), dtype=torch.float16, device="cuda:0")
            print("movers", cfg.name, "block", bs, flush=True)
            sw.sw_prefill_attn_paged(to_dev(qt), pb["k_pool"], pb["v_pool"], pb["block_table"], pb["seq_lens"], starts_d,
                                     out, qt.shape[0], len(LENS), n_qh, n_kvh, 128, bs, pb["max_blocks"], pb["n_blocks"])
            torch.cuda.synchronize()
            assert np.array_equal(out.cpu().numpy().view(np.uint16), dense.view(np.uint16)), bs
    finally:
        sw.sw_set_param(sw.SW_PARAM_PREFILL_KERNEL, 0)
        sw.sw_set_param(sw.SW_PARAM_PREFILL_HEADS, 0)
        sw.sw_set_param(sw.SW_PARAM_PREFILL_WAVES, 0)


@pytest.mark.parametrize("n_qh,n_kvh,lens", [
    (3, 1, [1000, 1025, 1279, 1281, 1536]), (6, 2, [1024, 1057]), (6, 1, [1087, 1100]), (5, 1, [1023, 1153, 1200]),
    (7, 1, [1500, 1504, 993]), (12, 4, [2300]), (12, 1, [1700, 900]),
])
def test_flat_columns(n_qh, n_kvh, lens):
    import torch
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(sum(lens))
    n, max_len, tot = len(lens), max(lens), sum(lens)
    lay = sw.sw_kv_layout(n, n_kvh, 128, max_len)
    k, v = (torch.randn(lay.total_elems, generator=gen, dtype=torch.float16, device="cuda:0") for _ in range(2))
    q = torch.randn(tot, n_qh, 128, generator=gen, dtype=torch.float16, device="cuda:0")
    seq = torch.tensor(lens, dtype=torch.int32, device="cuda:0")
    first = torch.tensor([sum(lens[:r]) for r in range(n)], dtype=torch.int32, device="cuda:0")
    outs = []
    sw.sw_set_param(sw.SW_PARAM_PREFILL_KERNEL, 1)
    try:
        for heads in (0, 1, n_qh // n_kvh):            # flat, one head a workgroup, a group
            sw.sw_set_param(sw.SW_PARAM_PREFILL_HEADS, heads if heads <= 8 else 6)
            outs.append(torch.full_like(q, float("nan")))
            print("flat", n_qh, n_kvh, lens, "heads", heads, flush=True)
            sw.sw_prefill_attn(q, k, v, seq, first, outs[-1], tot, n, n_qh, n_kvh, 128, max_len)
            torch.cuda.synchronize()
    finally:
        sw.sw_set_param(sw.SW_PARAM_PREFILL_KERNEL, 0)
        sw.sw_set_param(sw.SW_PARAM_PREFILL_HEADS, 0)
    assert not torch.isnan(outs[0]).any()
    for other in outs[1:]:
        assert torch.equal(outs[0].view(torch.int16), other.view(torch.int16))


@pytest.mark.parametrize("n_qh,n_kvh,n", [(12, 4, 3700), (6, 1, 7201), (24, 8, 1889)])
def test_flat_columns_in_the_halves_kernel(n_qh, n_kvh, n):
    """Whole prompts whose heads come in threes and sixes: within twice the parity bounds of the other kernels, the
    largest difference's and a row's 2-norm's (each is within them of 64 bits), every row written."""
    import torch
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(n)
    lay = sw.sw_kv_layout(1, n_kvh, 128, n)
    k, v = (torch.randn(lay.total_elems, generator=gen, dtype=torch.float16, device="cuda:0") for _ in range(2))
    q = torch.randn(n, n_qh, 128, generator=gen, dtype=torch.float16, device="cuda:0")
    seq = torch.tensor([n], dtype=torch.int32, device="cuda:0")
    first = torch.zeros(1, dtype=torch.int32, device="cuda:0")
    outs = []
    try:
        for kernel in (0, 1, 2):
            sw.sw_set_param(sw.SW_PARAM_PREFILL_KERNEL, kernel)
            outs.append(torch.full_like(q, float("nan")))
            sw.sw_prefill_attn(q, k, v, seq, first, outs[-1], n, 1, n_qh, n_kvh, 128, n)
            torch.cuda.synchronize()
    finally:
        sw.sw_set_param(sw.SW_PARAM_PREFILL_KERNEL, 0)
    assert not torch.isnan(outs[0]).any()
    for other in outs[1:]:
        assert not torch.equal(outs[0].view(torch.int16), other.view(torch.int16))
        apart = outs[0].float() - other.float()
        assert apart.abs().max().item() <= 2 * MAX_ABS
        assert (apart.norm(dim=-1) / other.float().norm(dim=-1)).max().item() <= 2 * MAX_REL_L2


# (positions, of which queries) of every request; cut: query rows that the first and the last request lack
@pytest.mark.parametrize("n_qh,n_kvh,reqs,cut", [
    (3, 1, [(1100, 1100), (1537, 1003), (1000, 1000)], (0, 0)), (3, 1, [(1300, 1300), (1537, 1003), (1090, 1090)], (130, 95)),
    (6, 2, [(3000, 3000), (1000, 1000), (33, 33), (400, 400)], (0, 0)),            # lengths apart: numbered by work
    (6, 1, [(2609, 1100), (1045, 1045)], (0, 0)), (6, 1, [(2609, 1100), (1045, 1045)], (31, 33)),
    (5, 1, [(1777, 1250), (1009, 1009)], (0, 0)), (5, 1, [(1200, 1200), (4000, 1030)], (129, 1)),
    (7, 1, [(1031, 1001), (1017, 1017)], (0, 0)), (7, 1, [(3100, 3100), (64, 64), (300, 300)], (257, 70)),
    (12, 1, [(1500, 1190), (1003, 1003)], (7, 2)),
])
def test_every_row_of_flat_columns(n_qh, n_kvh, reqs, cut):
    import torch
    n, max_len, max_q, bs = len(reqs), max(L for L, _ in reqs), max(c for _, c in reqs), 16
    tot = sum(c for _, c in reqs) - sum(cut)
    assert tot // n >= 1000                              # flat, not whole heads
    starts = [sum(c for _, c in reqs[:r]) - cut[0] for r in range(n)]
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(tot + n_qh)

    def rand(*shape):
        return torch.randn(*shape, generator=gen, dtype=torch.float16, device="cuda:0")
    lay = sw.sw_kv_layout(n, n_kvh, 128, max_len)
    k, v, q = rand(lay.total_elems), rand(lay.total_elems), rand(tot, n_qh, 128)
    out, paged = (torch.full_like(q, float("nan")) for _ in range(2))
    seq, first, nq = i32([L for L, _ in reqs]), i32(starts), i32([c for _, c in reqs])
    mb = -(-max_len // bs)
    lay_p = sw.sw_kv_paged_layout(n * mb, n_kvh, 128, bs)
    table = torch.randperm(n * mb, generator=gen, device="cuda:0").to(torch.int32).view(n, mb).contiguous()
    kp, vp = rand(lay_p.total_elems), rand(lay_p.total_elems)
    sw.sw_kv_unpack(k, v, table, seq, kp, vp, n, n_kvh, 128, max_len, bs, mb, n * mb)
    sw.sw_set_param(sw.SW_PARAM_PREFILL_KERNEL, 1)
    try:
        print("flat", n_qh, n_kvh, reqs, cut, flush=True)
        sw.sw_mixed_attn(q, k, v, seq, first, nq, out, tot, n, n_qh, n_kvh, 128, max_len, max_q)
        sw.sw_mixed_attn_paged(q, kp, vp, table, seq, first, nq, paged, tot, n, n_qh, n_kvh, 128, bs, mb, n * mb, max_q)
        torch.cuda.synchronize()
    finally:
        sw.sw_set_param(sw.SW_PARAM_PREFILL_KERNEL, 0)
    assert not torch.isnan(out).any()
    assert torch.equal(paged.view(torch.int16), out.view(torch.int16))
    for r, (L, c) in enumerate(reqs):
        lo, hi = max(0, -starts[r]), min(c, tot - starts[r])
        rows = slice(starts[r] + lo, starts[r] + hi)
        # (the rows that are missing at the end attend to nothing that the others see)
        ref = exact_rows(q[rows], k, v, lay, r, L - c + hi, L - c + lo, n_qh, n_kvh)
        assert_parity(out[rows].cpu().numpy(), ref.cpu().numpy(), "request %d" % r)
