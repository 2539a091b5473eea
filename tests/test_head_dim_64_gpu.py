"""head_dim 64 on the matrix-core token-phase kernel: a load instruction brings eight rows, a
staged K row covers half of the banks and V rows change places in pairs, so the lengths, the
position of an appended row and the block size are taken around multiples of 4, 8 and 32.
Tolerance: the library's parity bound for binary16 results (helpers.assert_parity)."""
import numpy as np
import pytest

import oracle
from paper_2311_18677_amd import binding as sw
from paper_2311_18677_amd import workloads as wl
from helpers import assert_parity

pytestmark = pytest.mark.gpu

D = 64
EDGES = [0, 1, 3, 4, 5, 7, 8, 9, 15, 16, 17, 31, 32, 33, 40, 63, 64, 65, 127, 128, 129, 255, 256, 257, 300, 511, 513, 700]


def dev(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a).view(np.int16).reshape(-1)).to("cuda:0").view(torch.float16)


@pytest.mark.parametrize("combine", [1, 2])
@pytest.mark.parametrize("n_qh,n_kvh", [(1, 1), (6, 2), (16, 1), (17, 1), (128, 2)])
def test_lengths_around_tile_edges(n_qh, n_kvh, combine):
    import torch
    cfg = wl.custom_config("d64", len(EDGES), n_qh, n_kvh, D, 700)
    batch = wl.make_batch(cfg, seed=6400 + n_qh, seq_lens=EDGES)
    bufs = sw.upload_batch(batch, pad_bits=0x7E00)
    lay = bufs["layout"]
    ref = oracle.decode_attn(batch.q, bufs["k_host"], bufs["v_host"], batch.seq_lens, cfg.n_req, n_qh, n_kvh, D,
                             cfg.max_len, lay.stride_req, lay.stride_kvh, lay.stride_tok)
    sw.sw_set_param(sw.SW_PARAM_COMBINE, combine)
    try:
        sw.run_batch(bufs, cfg)
        torch.cuda.synchronize()
        dense = bufs["out"].cpu().numpy()
        assert_parity(dense, ref, "dense")
        for bs in (4, 8, 16, 64):
            pb = sw.upload_paged_batch(batch, bs, pad_bits=0x7E00, seed=bs)
            sw.run_paged_batch(pb, cfg)
            torch.cuda.synchronize()
            # the same tiles in the same order: the same bits
            assert np.array_equal(pb["out"].cpu().numpy().view(np.uint16), dense.view(np.uint16)), bs
    finally:
        sw.sw_set_param(sw.SW_PARAM_COMBINE, 0)


@pytest.mark.parametrize("bs", [0, 4, 8])
def test_appended_row_at_every_place_of_a_load(bs):
    import torch
    lens = list(range(0, 36)) + [255, 256, 319, 320]            # 320 = full: nothing is stored
    n_qh, n_kvh = 6, 2
    cfg = wl.custom_config("d64a", len(lens), n_qh, n_kvh, D, 320)
    batch = wl.make_batch(cfg, seed=6500, seq_lens=lens)
    k_new, v_new = wl.make_new_rows(cfg, 6500)
    bufs = sw.upload_batch(batch, pad_bits=0x7E00)
    lay = bufs["layout"]
    k_ref, v_ref = bufs["k_host"].copy(), bufs["v_host"].copy()
    lens1 = oracle.kv_append(k_new, v_new, k_ref, v_ref, batch.seq_lens, cfg.n_req, n_kvh, D, cfg.max_len,
                             lay.stride_req, lay.stride_kvh, lay.stride_tok)
    ref = oracle.decode_attn(batch.q, k_ref, v_ref, lens1, cfg.n_req, n_qh, n_kvh, D, cfg.max_len,
                             lay.stride_req, lay.stride_kvh, lay.stride_tok)
    if bs == 0:
        sw.sw_decode_attn_append(bufs["q"], dev(k_new), dev(v_new), bufs["k_cache"], bufs["v_cache"], bufs["seq_lens"],
                                 bufs["out"], cfg.n_req, n_qh, n_kvh, D, cfg.max_len)
        torch.cuda.synchronize()
        assert_parity(bufs["out"].cpu().numpy(), ref, "append")
        assert np.array_equal(bufs["k_cache"].cpu().numpy().view(np.uint16), k_ref)
        assert np.array_equal(bufs["v_cache"].cpu().numpy().view(np.uint16), v_ref)
        return
    pb = sw.upload_paged_batch(batch, bs, pad_bits=0x7E00, seed=bs, room=1)
    sw.sw_decode_attn_paged_append(pb["q"], dev(k_new), dev(v_new), pb["k_pool"], pb["v_pool"], pb["block_table"],
                                   pb["seq_lens"], pb["out"], cfg.n_req, n_qh, n_kvh, D, bs, pb["max_blocks"],
                                   pb["n_blocks"])
    torch.cuda.synchronize()
    assert_parity(pb["out"].cpu().numpy(), ref, "paged append %d" % bs)


def test_the_caller_cannot_force_the_kernel_at_this_head_size():
    cfg = wl.custom_config("d64f", 2, 2, 1, D, 64)
    bufs = sw.upload_batch(wl.make_batch(cfg, seed=1, seq_lens=[3, 64]))
    sw.sw_set_param(sw.SW_PARAM_KERNEL, 2)
    try:
        with pytest.raises(sw.SwError) as e:
            sw.run_batch(bufs, cfg)
        assert e.value.code == sw.SW_ERR_UNSUPPORTED
    finally:
        sw.sw_set_param(sw.SW_PARAM_KERNEL, 0)
