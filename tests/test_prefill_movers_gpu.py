"""The shared-tile prompt kernel's moving waves: prompts that end at, before and behind a tile's edge, from one
tile to one round and a half of the three staging buffers, in workgroups of every number of waves; over block
tables of every addressing kind the same bits as dense.  Tolerance: the library's parity bound against the oracle."""
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
