"""The shared-tile prompt kernel's moving waves: prompts that end at, before and behind a tile's edge, from one
tile to one round and a half of the three staging buffers, in workgroups of every number of waves; over block
tables of every addressing kind the same bits as dense.  Tolerance: the library's parity bound against the oracle.
And columns dealt flat to workgroups: the same bits as with whole heads in each, every row written."""
import numpy as np
import pytest

from paper_2311_18677_amd import binding as sw
from paper_2311_18677_amd import workloads as wl
from helpers import assert_parity
from test_prefill_gpu import run_prefill, to_dev

pytestmark = pytest.mark.gpu

LENS = [1, 31, 32, 33, 64, 65, 95, 96, 97, 128, 129, 160, 0]


@pytest.mark.parametrize("n_qh,n_kvh", [(8, 1), (7, 1), (6, 2), (5, 1), (1, 1)])
def test_tile_edges(n_qh, n_kvh):
    import torch
    cfg = wl.custom_config("mv%d_%d" % (n_qh, n_kvh), len(LENS), n_qh, n_kvh, 128, 160)
    batch = wl.make_batch(cfg, seed=8100 + n_qh, seq_lens=LENS)
    qt, starts = wl.make_prefill_queries(batch)
    starts_d = torch.from_numpy(np.ascontiguousarray(starts, dtype=np.int32)).to("cuda:0")
    sw.sw_set_param(sw.SW_PARAM_PREFILL_KERNEL, 1)
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
    """Whole prompts whose heads come in threes and sixes: within twice the parity bound of the shared-tile kernel
    (each is within it of 64 bits), every row written."""
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
        assert (outs[0].float() - other.float()).abs().max().item() <= 4e-3
