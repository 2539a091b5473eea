"""head_dim 64 on the matrix-core token-phase kernel: a load instruction brings eight rows, a
staged K row covers half of the banks and V rows change places in pairs, so the lengths, the
position of an appended row and the block size are taken around multiples of 4, 8 and 32.
Tolerance: the library's parity bound for binary16 results (helpers.assert_parity)."""
import numpy as np
import pytest

import oracle
from paper_2311_18677_amd import binding as sw
from paper_2311_18677_amd import workloads as wl
from helpers import MAX_ABS, assert_parity

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


def spoiled_batch(n_qh, n_kvh):
    """Infinities and NaN in V (first, middle and last positions, one beside a weight of about 2^-40),
    in K and in Q; every case in a request of its own, the last request is clean."""
    inf = np.float16("inf")
    lens = [1, 33, 300, 257, 200, 129, 90, 70, 64, 300]
    cfg = wl.custom_config("d64nf", len(lens), n_qh, n_kvh, D, 304)
    batch = wl.make_batch(cfg, seed=6600 + n_qh, seq_lens=lens)
    k, v, q = batch.k_rows, batch.v_rows, batch.q
    v[0][0, 0, 3] = inf
    v[1][0, 32, 0], v[1][0, 0, 63], v[1][0, 7, 63] = -inf, inf, -inf        # dim 63: NaN
    v[2][0, 100, 5], v[2][0, 299, 6], v[2][0, 299, 7] = inf, -inf, np.nan
    v[3][:, 40:60, 8] = inf
    v[3][:, 256, 9] = -inf
    # position 17's score lies about 28 (40 bits) below position 0's, and its row is infinite
    q[4], k[4][:, :, 0] = 0, 0
    q[4, :, 0], k[4][:, 0, 0], k[4][:, 17, 0] = 8, 14, -14
    v[4][:, 17, 1] = -inf
    k[5][0, 60, 2] = inf                                                    # scores of +inf or -inf by head
    k[6][0, 89, 2] = np.nan
    q[7, 0, 11] = inf
    return cfg, batch


def assert_same_kind(out, ref, what):
    """NaN and infinities where the reference has them, the other values within the parity bound."""
    out = out.astype(np.float64)
    assert np.array_equal(np.isnan(out), np.isnan(ref)), what
    big = np.isinf(ref)
    assert np.array_equal(out[big], ref[big]) and not np.isinf(out[~big]).any(), what
    fine = np.isfinite(ref)
    assert np.abs(out[fine] - ref[fine]).max() <= MAX_ABS, what


@pytest.mark.parametrize("n_qh,n_kvh", [(1, 1), (8, 2), (17, 1)])
@pytest.mark.parametrize("chunk,combine,waves", [(0, 0, 0), (64, 1, 0), (64, 2, 0), (128, 1, 0), (256, 2, 8)])
def test_infinite_rows_weigh_in_as_infinities(n_qh, n_kvh, chunk, combine, waves):
    import torch
    cfg, batch = spoiled_batch(n_qh, n_kvh)
    bufs = sw.upload_batch(batch, pad_bits=0x7E00)
    lay = bufs["layout"]
    with np.errstate(invalid="ignore"):
        ref = oracle.decode_attn(batch.q, bufs["k_host"], bufs["v_host"], batch.seq_lens, cfg.n_req, n_qh, n_kvh, D,
                                 cfg.max_len, lay.stride_req, lay.stride_kvh, lay.stride_tok)
    for key, value in ((sw.SW_PARAM_CHUNK, chunk), (sw.SW_PARAM_COMBINE, combine), (sw.SW_PARAM_WAVES, waves)):
        sw.sw_set_param(key, value)
    try:
        for kernel in (1, 0):
            sw.sw_set_param(sw.SW_PARAM_KERNEL, kernel)
            sw.run_batch(bufs, cfg)
            torch.cuda.synchronize()
            assert_same_kind(bufs["out"].cpu().numpy(), ref, "kernel %d" % kernel)
        for bs in (4, 16, 64):
            pb = sw.upload_paged_batch(batch, bs, pad_bits=0x7E00, seed=bs)
            sw.run_paged_batch(pb, cfg)
            torch.cuda.synchronize()
            assert_same_kind(pb["out"].cpu().numpy(), ref, "blocks of %d" % bs)
    finally:
        for key in (sw.SW_PARAM_CHUNK, sw.SW_PARAM_COMBINE, sw.SW_PARAM_WAVES, sw.SW_PARAM_KERNEL):
            sw.sw_set_param(key, 0)


@pytest.mark.parametrize("bs", [0, 4, 16])
def test_an_appended_infinite_row(bs):
    import torch
    n_qh, n_kvh = 6, 2
    lens = [0, 5, 31, 32, 40, 300]
    cfg = wl.custom_config("d64anf", len(lens), n_qh, n_kvh, D, 304)
    batch = wl.make_batch(cfg, seed=6700, seq_lens=lens)
    k_new, v_new = wl.make_new_rows(cfg, 6700)
    v_new = v_new.copy()
    v_new[:, 0, 4] = np.float16("-inf")
    v_new[2:, 1, 9] = np.float16("nan")
    batch.v_rows[4][0, 3, 20] = np.float16("inf")
    bufs = sw.upload_batch(batch, pad_bits=0x7E00)
    lay = bufs["layout"]
    k_ref, v_ref = bufs["k_host"].copy(), bufs["v_host"].copy()
    lens1 = oracle.kv_append(k_new, v_new, k_ref, v_ref, batch.seq_lens, cfg.n_req, n_kvh, D, cfg.max_len,
                             lay.stride_req, lay.stride_kvh, lay.stride_tok)
    ref = oracle.decode_attn(batch.q, k_ref, v_ref, lens1, cfg.n_req, n_qh, n_kvh, D, cfg.max_len,
                             lay.stride_req, lay.stride_kvh, lay.stride_tok)
    if bs:
        pb = sw.upload_paged_batch(batch, bs, pad_bits=0x7E00, seed=bs, room=1)
        sw.sw_decode_attn_paged_append(pb["q"], dev(k_new), dev(v_new), pb["k_pool"], pb["v_pool"], pb["block_table"],
                                       pb["seq_lens"], pb["out"], cfg.n_req, n_qh, n_kvh, D, bs, pb["max_blocks"],
                                       pb["n_blocks"])
        torch.cuda.synchronize()
        assert_same_kind(pb["out"].cpu().numpy(), ref, "paged append")
        return
    sw.sw_decode_attn_append(bufs["q"], dev(k_new), dev(v_new), bufs["k_cache"], bufs["v_cache"], bufs["seq_lens"],
                             bufs["out"], cfg.n_req, n_qh, n_kvh, D, cfg.max_len)
    torch.cuda.synchronize()
    assert_same_kind(bufs["out"].cpu().numpy(), ref, "append")
    assert np.array_equal(bufs["k_cache"].cpu().numpy().view(np.uint16), k_ref)
    assert np.array_equal(bufs["v_cache"].cpu().numpy().view(np.uint16), v_ref)


@pytest.mark.parametrize("waves", [4, 8])
@pytest.mark.parametrize("combine", [1, 2])
@pytest.mark.parametrize("n_req,n_qh,n_kvh", [(64, 4, 2), (65, 4, 2), (256, 3, 1), (257, 3, 1), (1024, 2, 1), (1025, 2, 1)])
def test_every_size_class_of_the_batch(n_req, n_qh, n_kvh, combine, waves):
    """The lengths are scanned in a form per size class (64, 256 and 1024 requests); four and eight waves
    walk the tiles of a chunk."""
    import torch
    lens = [(37 * r + 11 * (r // 7)) % 301 for r in range(n_req)]          # zeros among them, up to five chunks of 64
    cfg = wl.custom_config("d64s", n_req, n_qh, n_kvh, D, 300)
    batch = wl.make_batch(cfg, seed=6800 + n_req, seq_lens=lens)
    bufs = sw.upload_batch(batch, pad_bits=0x7E00)
    lay = bufs["layout"]
    ref = oracle.decode_attn(batch.q, bufs["k_host"], bufs["v_host"], batch.seq_lens, n_req, n_qh, n_kvh, D,
                             cfg.max_len, lay.stride_req, lay.stride_kvh, lay.stride_tok)
    sw.sw_set_param(sw.SW_PARAM_COMBINE, combine)
    sw.sw_set_param(sw.SW_PARAM_WAVES, waves)
    try:
        for chunk in (64, 256):                       # a chunk of 64 runs four waves whatever is asked for
            sw.sw_set_param(sw.SW_PARAM_CHUNK, chunk)
            bufs["out"].fill_(float("nan"))
            sw.run_batch(bufs, cfg)
            torch.cuda.synchronize()
            dense = bufs["out"].cpu().numpy()
            assert_parity(dense, ref, "chunk %d" % chunk)
            pb = sw.upload_paged_batch(batch, 8, pad_bits=0x7E00, seed=n_req)
            sw.run_paged_batch(pb, cfg)
            torch.cuda.synchronize()
            assert np.array_equal(pb["out"].cpu().numpy().view(np.uint16), dense.view(np.uint16)), chunk
    finally:
        for key in (sw.SW_PARAM_COMBINE, sw.SW_PARAM_WAVES, sw.SW_PARAM_CHUNK):
            sw.sw_set_param(key, 0)


def test_the_default_takes_the_matrix_core_kernel():
    """No parameter forces it at this head size; the two kernels round differently."""
    import torch
    cfg = wl.custom_config("d64k", 8, 8, 2, D, 600)
    bufs = sw.upload_batch(wl.make_batch(cfg, seed=6900, seq_lens=[600, 599, 512, 300, 257, 100, 33, 5]))
    bits = []
    try:
        for kernel in (1, 0):
            sw.sw_set_param(sw.SW_PARAM_KERNEL, kernel)
            sw.run_batch(bufs, cfg)
            torch.cuda.synchronize()
            bits.append(bufs["out"].cpu().numpy().view(np.uint16).copy())
    finally:
        sw.sw_set_param(sw.SW_PARAM_KERNEL, 0)
    assert not np.array_equal(bits[0], bits[1])
