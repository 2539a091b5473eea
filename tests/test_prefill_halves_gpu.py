"""The prompt kernel that takes a long prompt's keys in two halves (the default for one request of
432 to 512 of its workgroups, somewhat beyond for long ones, a whole prompt from 336 on, and batches of whole prompts
of 345 to 680, for which see test_prefill_order_gpu.py and test_prefill_choice_gpu.py): where it serves and where not, one query head per workgroup column, two, four, ragged last
tiles and query blocks, prompts with earlier context, block tables of every addressing kind, and
keys scaled by 8 (maxima raised late, rows of a single key).
Tolerance: the library's parity bound against the oracle; over block tables the same bits as dense."""
import numpy as np
import pytest

import oracle
from paper_2311_18677_amd import binding as sw
from paper_2311_18677_amd import workloads as wl
from helpers import assert_parity

pytestmark = pytest.mark.gpu


def dev(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a).view(np.int16).reshape(-1)).to("cuda:0").view(torch.float16)


def i32(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.int32)).to("cuda:0")


# (query heads, key/value heads, cached positions, of which queries, key scale)
CASES = [(64, 64, 1000, 1000, 1.0), (64, 64, 929, 929, 8.0), (64, 32, 901, 901, 1.0), (64, 8, 863, 863, 1.0),
         (64, 8, 1441, 865, 1.0), (40, 8, 1500, 1500, 1.0)]


def serving_kernel(call, out):
    """Which kernel serves a call: 1 or 2 where its bits are those of SW_PARAM_PREFILL_KERNEL 1 or 2, 3 where
    they are neither's (the kernels round differently, and no parameter forces the third).
    `out` holds the call's own result afterwards."""
    import torch
    bits = []
    try:
        for kernel in (1, 2, 0):
            sw.sw_set_param(sw.SW_PARAM_PREFILL_KERNEL, kernel)
            out.zero_()
            call()
            torch.cuda.synchronize()
            bits.append(out.view(torch.int16).clone())
    finally:
        sw.sw_set_param(sw.SW_PARAM_PREFILL_KERNEL, 0)
    assert not torch.equal(bits[0], bits[1])
    return 1 if torch.equal(bits[2], bits[0]) else 2 if torch.equal(bits[2], bits[1]) else 3


def random_call(n_qh, n_kvh, lens, nqs, max_len, mixed):
    """(call, out) over seeded caches: sw_mixed_attn, or sw_prefill_attn where not mixed."""
    import torch
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(sum(lens) + n_qh)
    lay = sw.sw_kv_layout(len(lens), n_kvh, 128, max_len)
    k, v = (torch.randn(lay.total_elems, generator=gen, dtype=torch.float16, device="cuda:0") for _ in range(2))
    q = torch.randn(sum(nqs), n_qh, 128, generator=gen, dtype=torch.float16, device="cuda:0")
    out = torch.zeros_like(q)
    args = (q, k, v, i32(lens), i32([sum(nqs[:r]) for r in range(len(nqs))]))
    tail = (out, sum(nqs), len(lens), n_qh, n_kvh, 128, max_len)
    if mixed:
        nq = i32(nqs)
        return lambda: sw.sw_mixed_attn(*args, nq, *tail, max(nqs)), out
    return lambda: sw.sw_prefill_attn(*args, *tail), out


@pytest.mark.parametrize("n_qh,n_kvh,lens,nqs,max_len,mixed,kernel", [
    (8, 1, [6880], [6880], 6900, True, 2),             # 430 workgroups
    (8, 1, [6913], [6913], 6940, True, 3),             # 434
    (8, 1, [8192], [8192], 8192, False, 3),            # 512: two rounds
    (8, 1, [8193], [8193], 8200, True, 3),             # beyond, long and from the start
    (8, 1, [8193], [8193], 30000, True, 2),            # ... or behind earlier context, as far as the host knows
    (8, 1, [9600], [9600], 9600, False, 3),            # 600; the shared-tile kernel's otherwise
    (8, 1, [19400], [9700], 19400, True, 1),
    (8, 1, [12000], [12000], 12000, False, 1),         # 750
    (64, 8, [863], [863], 900, True, 3),
    (64, 8, [1040], [1040], 1040, True, 2),            # short prompts beyond two rounds
    (64, 8, [1560], [1560], 1560, True, 1),
    (64, 64, [1000], [1000], 1000, True, 3),
    (64, 64, [1030], [1030], 1030, True, 2),
    (5, 1, [6800], [6800], 6800, True, 2),
    (5, 1, [11500], [11500], 11500, True, 3),
    (3, 1, [20000], [20000], 20000, True, 1),          # thirds of the columns: never behind earlier context, as far as the call tells
    (8, 1, [6400, 3400], [6400, 3400], 6400, True, 1),         # several requests: not at eight waves
    (8, 8, [3300, 3300, 3300], [3300, 3300, 3300], 3300, False, 1),
    (7, 1, [3200, 3200, 3200], [3200, 3200, 3200], 3200, False, 3),
])
def test_the_kernel_that_serves_a_call(n_qh, n_kvh, lens, nqs, max_len, mixed, kernel):
    assert serving_kernel(*random_call(n_qh, n_kvh, lens, nqs, max_len, mixed)) == kernel


@pytest.mark.parametrize("n_qh,n_kvh,L,nq,scale", CASES)
def test_one_long_prompt_against_the_oracle(n_qh, n_kvh, L, nq, scale):
    import torch
    d, max_len = 128, L + 3
    cfg = wl.Config("halves", 1, n_qh, n_kvh, d, max_len, ("fixed", (0,)),
                    k_row_scale=(0.1, scale) if scale != 1.0 else ())
    batch = wl.make_batch(cfg, seed=9000 + L, seq_lens=[L])
    qt, starts, nqs = wl.make_mixed_queries(batch, [nq])
    bufs = sw.upload_batch(batch, pad_bits=0x7E00)
    lay = bufs["layout"]
    out = torch.full((nq, n_qh, d), float("nan"), dtype=torch.float16, device="cuda:0")
    q = dev(qt)
    args = (bufs["seq_lens"], i32(starts), i32(nqs))
    assert serving_kernel(lambda: sw.sw_mixed_attn(q, bufs["k_cache"], bufs["v_cache"], *args, out, nq, 1, n_qh, n_kvh, d,
                                                   max_len, nq), out) == 3
    dense = out.cpu().numpy()
    # the same rows from the oracle, a sample of them: the first and last of every 32-query block and
    # of its neighbours, and a stride through the rest
    rows = sorted({min(nq - 1, 32 * b + o) for b in range(0, nq // 32 + 1, 5) for o in (0, 15, 16, 31)} | set(range(0, nq, 61)) | {nq - 1})
    for i in rows:
        ref = oracle.decode_attn(qt[i:i + 1], bufs["k_host"], bufs["v_host"], np.array([L - nq + i + 1], dtype=np.int32),
                                 1, n_qh, n_kvh, d, max_len, lay.stride_req, lay.stride_kvh, lay.stride_tok)
        assert_parity(dense[i:i + 1], ref, "row %d" % i)
    for bs in (4, 16, 64):
        pb = sw.upload_paged_batch(batch, bs, pad_bits=0x7E00, seed=bs)
        out2 = torch.full_like(out, float("nan"))
        sw.sw_mixed_attn_paged(q, pb["k_pool"], pb["v_pool"], pb["block_table"], *args, out2, nq, 1, n_qh, n_kvh, d, bs,
                               pb["max_blocks"], pb["n_blocks"], nq)
        torch.cuda.synchronize()
        assert np.array_equal(out2.cpu().numpy().view(np.uint16), dense.view(np.uint16)), bs


@pytest.mark.parametrize("n_qh,n_kvh,n,key,value,kernel", [
    (8, 1, 8192, sw.SW_PARAM_PREFILL_WAVES, 8, 2), (8, 1, 8192, sw.SW_PARAM_PREFILL_HEADS, 8, 2),
    (64, 32, 901, sw.SW_PARAM_PREFILL_WAVES, 2, 2), (8, 1, 9700, sw.SW_PARAM_PREFILL_HEADS, 2, 1),
    (8, 1, 9700, sw.SW_PARAM_PREFILL_WAVES, 1, 1),
])
def test_chosen_heads_and_waves_count(n_qh, n_kvh, n, key, value, kernel):
    """A call that this kernel would serve, with the caller's heads or waves: the kernel whose shape
    they are, with them."""
    import torch
    call, out = random_call(n_qh, n_kvh, [n], [n], n, False)
    assert serving_kernel(call, out) == 3
    try:
        sw.sw_set_param(key, value)
        assert serving_kernel(call, out) == kernel
        if kernel == 2 and key == sw.SW_PARAM_PREFILL_WAVES:       # other waves, other sums
            chosen = out.clone()
            sw.sw_set_param(key, 4)
            call()
            torch.cuda.synchronize()
            assert not torch.equal(chosen.view(torch.int16), out.view(torch.int16))
    finally:
        sw.sw_set_param(key, 0)


def test_several_long_prompts_one_of_them_alone_in_its_last_steps():
    """Lengths far apart: waves of finished query blocks keep arriving at the barrier."""
    import torch
    n_qh, n_kvh, d = 5, 1, 128
    lens = [6400, 1, 3700]                        # 3367 tokens on average, 315 workgroups of the shared-tile kernel
    cfg = wl.custom_config("halves3", 3, n_qh, n_kvh, d, max(lens))
    batch = wl.make_batch(cfg, seed=77, seq_lens=lens)
    qt, starts = wl.make_prefill_queries(batch)
    bufs = sw.upload_batch(batch)
    lay = bufs["layout"]
    n_tokens = sum(lens)
    out = torch.zeros(n_tokens, n_qh, d, dtype=torch.float16, device="cuda:0")
    args = (dev(qt), bufs["k_cache"], bufs["v_cache"], bufs["seq_lens"], i32(starts))
    assert serving_kernel(lambda: sw.sw_prefill_attn(*args, out, n_tokens, 3, n_qh, n_kvh, d, cfg.max_len), out) == 3
    got = out.cpu().numpy()
    for r, i in ((0, 0), (0, 6399), (0, 4777), (1, 0), (2, 3699), (2, 31), (2, 2600)):
        one = np.zeros(3, dtype=np.int32)
        one[r] = i + 1
        q3 = np.zeros((3, n_qh, d), dtype=np.float16)
        q3[r] = qt[starts[r] + i]
        ref = oracle.decode_attn(q3, bufs["k_host"], bufs["v_host"], one, 3, n_qh, n_kvh, d, cfg.max_len,
                                 lay.stride_req, lay.stride_kvh, lay.stride_tok)
        assert_parity(got[starts[r] + i][None], ref[r:r + 1], "request %d row %d" % (r, i))


@pytest.mark.parametrize("n_qh,n_kvh,L,nq", [(64, 32, 901, 901), (64, 8, 863, 863), (16, 1, 3500, 3500), (64, 8, 3500, 865)])
def test_no_further_from_64_bits_than_the_key_split_kernel(n_qh, n_kvh, L, nq):
    """A row's weights are rounded to binary16 relative to a maximum of each wave's, whose own key's
    weight is exact: four maxima in the key-split kernel, two here, which takes its waves' first
    tiles with the rounding's rest.  Both norms are over n = nq * n_qh * d values whose roundings are
    independent: each is good to one part in sqrt(2 n), and four of that are let pass."""
    import torch
    d, max_len = 128, L
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(L + nq)
    lay = sw.sw_kv_layout(1, n_kvh, d, max_len)
    k, v = (torch.randn(lay.total_elems, generator=gen, dtype=torch.float16, device="cuda:0") for _ in range(2))
    q = torch.randn(nq, n_qh, d, generator=gen, dtype=torch.float16, device="cuda:0")
    later = torch.arange(L, device="cuda:0")[None, :] > (L - nq + torch.arange(nq, device="cuda:0"))[:, None]
    ref = torch.empty(nq, n_qh, d, dtype=torch.float64, device="cuda:0")
    rows = [x.as_strided((n_kvh, L, d), (lay.stride_kvh, lay.stride_tok, 1)).double() for x in (k, v)]
    for h in range(n_qh):
        g = h // (n_qh // n_kvh)
        scores = (q[:, h].double() @ rows[0][g].t().contiguous()) / d ** 0.5
        ref[:, h] = torch.softmax(scores.masked_fill_(later, -float("inf")), dim=-1) @ rows[1][g]
    err = {}
    try:
        for kernel in (0, 2):
            sw.sw_set_param(sw.SW_PARAM_PREFILL_KERNEL, kernel)
            out = torch.zeros_like(q)
            sw.sw_mixed_attn(q, k, v, i32([L]), i32([0]), i32([nq]), out, nq, 1, n_qh, n_kvh, d, max_len, nq)
            torch.cuda.synchronize()
            err[kernel] = float((out.double() - ref).norm() / ref.norm())
    finally:
        sw.sw_set_param(sw.SW_PARAM_PREFILL_KERNEL, 0)
    assert 0 < err[0] <= err[2] * (1 + 4 / (2 * nq * n_qh * d) ** 0.5), err
