"""A mixed batch's two phases in one launch (the library's choice beside the four-wave key-split
prompt kernel, once the token phase has more than four chunks) against the same phases in
launches of their own: the same bits, on dense caches and block pools, for one query head, a group
of eight, two head tiles, and every size class of the batch; and where the library keeps the launches
apart.  Which form ran is read off the recorded launches.
Tolerance against the oracle: the library's parity bound."""
import numpy as np
import pytest

from paper_2311_18677_amd import binding as sw
from paper_2311_18677_amd import workloads as wl
from helpers import assert_parity, launches
from test_mixed_gpu import run_mixed, NAN_BITS
from test_mixed_paged_gpu import run_paged

pytestmark = pytest.mark.gpu


@pytest.fixture
def merge():
    def set_merge(value):
        sw.sw_set_param(sw.SW_PARAM_MIXED_MERGE, value)
    sw.sw_set_param(sw.SW_PARAM_PREFILL_KERNEL, 2)
    sw.sw_set_param(sw.SW_PARAM_CHUNK, 64)           # eleven chunks: the two-kernel form of the token phase
    yield set_merge
    sw.sw_set_param(sw.SW_PARAM_MIXED_MERGE, 0)
    sw.sw_set_param(sw.SW_PARAM_CHUNK, 0)
    sw.sw_set_param(sw.SW_PARAM_PREFILL_KERNEL, 0)


LENS = [700, 64, 65, 1, 0, 129, 699, 33, 512, 640, 300]
QLENS = [1, 64, 1, 1, 1, 100, 1, 33, 0, 2, 1]


def batch_of(n_req, n_qh, n_kvh, more_queries=()):
    lens = [LENS[i % len(LENS)] for i in range(n_req)]
    qls = [QLENS[i] if i < len(QLENS) else (1 if lens[i] else 0) for i in range(n_req)]
    for i, n in more_queries:
        qls[i] = n
    cfg = wl.custom_config("mx1_%d_%d_%d" % (n_req, n_qh, n_kvh), n_req, n_qh, n_kvh, 128, 700)
    batch = wl.make_batch(cfg, seed=6100 + n_req + n_qh, seq_lens=lens)
    qt, starts, _ = wl.make_mixed_queries(batch, qls)
    return batch, qt, starts, qls


def same_bits(got, want):
    assert np.array_equal(got.view(np.uint16), want.view(np.uint16))


def form(batch, bufs, qt, starts, qls):
    """"one" launch for both phases and the combine kernel, or "two": the token phase in a launch of its own, then
    the prompt kernel with the merge; "three": the token phase, the combine kernel, the prompt kernel."""
    import torch
    cfg = batch.cfg
    i32 = lambda a: torch.from_numpy(np.ascontiguousarray(a, dtype=np.int32)).to("cuda:0")
    q = torch.zeros(qt.shape[0], cfg.n_qh, 128, dtype=torch.float16, device="cuda:0")
    out, qs, ql = torch.zeros_like(q), i32(starts), i32(qls)
    torch.cuda.synchronize()
    got = launches(lambda stream: sw.sw_mixed_attn(
        q, bufs["k_cache"], bufs["v_cache"], bufs["seq_lens"], qs, ql, out, qt.shape[0], cfg.n_req, cfg.n_qh,
        cfg.n_kvh, 128, cfg.max_len, 700, stream))
    n_ht = (cfg.n_qh // cfg.n_kvh + 15) // 16                # head tiles; with several, the items come in eights
    token = cfg.n_req * cfg.n_kvh * -(-cfg.max_len // 64)
    token = token if n_ht == 1 else -(-token // 8) * 8 * n_ht
    if len(got) == 3:
        assert got[0] == (token, 256)
        return "three"
    assert len(got) == 2 and got[0][1] == 256 and got[0][0] >= token
    return "one" if got[0][0] > token else "two"


@pytest.mark.parametrize("n_req,n_qh,n_kvh,more,default", [
    (11, 8, 1, (), "one"), (11, 3, 3, (), "one"), (11, 17, 1, (), "one"), (2, 8, 1, (), "one"), (65, 6, 2, (), "one"),
    (257, 2, 1, (), "one"),
    (11, 8, 2, [(0, 700), (6, 699)], "one"),        # 392 prompt workgroups
    (11, 10, 2, [(0, 700), (6, 699)], "two"),       # 490: more than the line
    (65, 12, 12, (), "one"),                        # 60 prompt workgroups beside 780 (request, key/value head) pairs
    (65, 14, 14, (), "two"),                        # 70 beside 910
])
def test_one_launch_gives_the_bits_of_two(n_req, n_qh, n_kvh, more, default, merge):
    batch, qt, starts, qls = batch_of(n_req, n_qh, n_kvh, more)
    outs, bufs = [], None
    for m in (0, 1, 0):
        merge(m)
        out, ref, bufs = run_mixed(batch, qt, starts, qls, 700, bufs=bufs, tag="merge %d" % m)
        assert_parity(out, ref, batch.cfg.name)
        outs.append(out.copy())
    same_bits(outs[0], outs[1])
    same_bits(outs[2], outs[1])
    for m, want in ((0, default), (1, "three"), (2, "two")):
        merge(m)
        assert form(batch, bufs, qt, starts, qls) == want


@pytest.mark.parametrize("block_size", [4, 16, 64])
def test_one_launch_over_block_pools(block_size, merge):
    batch, qt, starts, qls = batch_of(11, 8, 1)
    pb = sw.upload_paged_batch(batch, block_size, pad_bits=NAN_BITS)
    outs = []
    for m in (0, 1):
        merge(m)
        out, ref = run_paged(batch, pb, qt, starts, qls, 700, "merge %d" % m)
        assert_parity(out, ref, batch.cfg.name)
        outs.append(out.copy())
    same_bits(outs[0], outs[1])


def test_timing_records_one_pair_of_launches_per_call(merge):
    batch, qt, starts, qls = batch_of(11, 8, 1)
    counts = []
    for m in (0, 1):
        merge(m)
        sw.sw_prof_start(8)
        run_mixed(batch, qt, starts, qls, 700, tag="timed, merge %d" % m)
        counts.append(sw.sw_prof_stop()[2])
    assert counts == [2, 2]
