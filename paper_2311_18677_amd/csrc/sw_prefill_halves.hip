// Prompt-phase (causal) attention, shared tiles with the key range in two halves (gfx950,
// wave64), head_dim 128: the form for a few long prompts.
//
// The shared-tile kernel (sw_prefill_mfma.hip) stages every K/V tile once for the eight waves of
// a workgroup, which is what keeps the L2 traffic low, but with few workgroups its time is the
// chain of tiles of the longest prompt's last block: 0.75 us for every 32 positions, on a partly
// idle chip.  The key-split kernel (sw_prefill_split.hip) has short chains but streams the key
// range through L2 once per 32 queries and head.  Here four of the waves take the even tiles and four
// the odd ones, for half as many (query head, 32 positions) columns: half the chain, twice the
// workgroups -- late (long) blocks first, so that the short ones fill up behind them -- and a
// tile still serves four waves.  The two groups' (maximum, sum, accumulator) triples are merged
// through LDS at the end.
//
// A step of a wave is one tile: first product, softmax, second product, one after the other; the two
// waves of a SIMD fill each other's gaps.  (With the first product of the next tile beside the softmax
// of this one a step took 1.06 us instead of 0.95: that form has all eight waves wait for the same
// LDS reads behind the barrier, before their first matrix instruction.)  K operands are read two
// 32-dim steps, V operands three 16-dim blocks ahead of their products, and no further, which would
// take registers.
// Four further waves request the tiles (TileMover in sw_prefill_common.h), 32 requests a step; dealt to the waves
// that compute they held up all of these behind every barrier.  With two moving waves prompts over block
// tables take up to 7 % longer, dense ones the same.
//
// Rounding.  Weights are binary16, relative to a maximum that a wave takes from its first tile, so
// the largest weight of that tile is exact.  The key-split kernel has four such maxima for a row, here
// there are two, which costs 1.5 % of the error against 64 bits (2.57e-4 -> 2.61e-4 of the 2-norm
// for a prompt of 8192 tokens, nearly all of it in rows of few positions).  The waves therefore
// multiply their first tile by the rest of its weights as well: 2.47e-4, rows behind 2600
// and more positions are as far off as the key-split kernel's.  The first tile is a step of its own, in front
// of the loop (one prompt of 8192 tokens with its cache store 141 -> 136 us against the rest taken inside it).
//
// Measured (8 heads on one key/value head, attention alone): one prompt of 8192 tokens 144 us with the requests dealt to the
// computing waves, 140 to 141 without, over blocks of 16 positions 163 -> 140, of 4 positions 180 -> 145; key-split 181.  With
// the first tile in front of the loop 134.
// What bounds it: the chain of a wave's own instructions, with two such waves to a SIMD (see sw_prefill_mfma.hip),
// and power: 127 us with all inputs zero.  (A third of the keys for each of twelve computing waves: 145.)
#include "sw_prefill_common.h"

#include <type_traits>

namespace {

using namespace sw_prefill;

constexpr int kMovers = 4;        // waves that only request tiles
constexpr int kBufs = 3;          // steps' worth of K and of V tiles in the staging rings

// Eight waves = 2 * (query heads per workgroup) * (waves per head): wave w works on tile
// 2 * i + w / 4 of step i.
// PAGED: K and V are block pools addressed through the request's row of the block table
// (position t = row t % block_size of pool block table[t / block_size]).
template <bool PAGED>
__global__ __launch_bounds__(512 + 64 * kMovers, 1)
void sw_prefill_halves_kernel(SwPrefillArgs a)
{
    constexpr int NW = 8;                             // waves
    constexpr int KS = 2;                             // key tiles staged per step
    constexpr int NC = NW / KS;                       // (query head, 32 positions) columns
    constexpr int kStepBytes = KS * kTileBytes;       // the K (or V) tiles of one step
    constexpr int kVBase = kBufs * kStepBytes;        // K ring, then V ring
    __shared__ __attribute__((aligned(16))) unsigned char lds[2 * kBufs * kStepBytes];

    // blockIdx -> (item = (request, query block), key/value head, part of the item's columns, later
    // positions first)
    const int q_block = kQPerWave * a.qw;        // query tokens of an item
    const unsigned n_parts = (unsigned)(a.group * a.qw) / NC;
    const Columns mine(a, (int)(n_parts - 1 - blockIdx.x % n_parts), NC);
    const unsigned rest = blockIdx.x / n_parts;
    const int g = (int)(rest % (unsigned)a.n_kvh);
    const QItem it = find_item<true>(a, rest / (unsigned)a.n_kvh, q_block);
    if (!it.valid) return;
    const int r = it.r, qb = it.qb, L = it.L, NQ = it.NQ;   // NQ: the request's last NQ tokens are its queries
    const long long q_first = it.q_first;
    const int P0 = L - NQ;                       // position of query index 0
    const int Q0 = qb * q_block;                 // first query index of the item
    if (Q0 + kQPerWave * mine.block(0) >= NQ) return;

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n16  = lane & 15;
    const int gq   = lane >> 4;
    // dense: the (request, head) slab; block table: the head's rows inside pool block 0
    const long long slab = PAGED ? (long long)g * a.stride_kvh : (long long)r * a.stride_req + (long long)g * a.stride_kvh;
    const char *kslab = reinterpret_cast<const char *>(a.k) + 2 * slab;
    const char *vslab = reinterpret_cast<const char *>(a.v) + 2 * slab;
    settled(kslab);
    settled(vslab);
    const_table_t table = PAGED ? (const_table_t)(a.block_table + (long long)r * a.max_blocks) : nullptr;

    // tiles the workgroup walks: up to the position of its last query
    const int last_pos = P0 + min(Q0 + kQPerWave * (mine.block(NC - 1) + 1), NQ) - 1;
    const int n_steps = last_pos / (kTile * KS) + 1;

    using I0 = std::integral_constant<int, 0>;
    using I1 = std::integral_constant<int, 1>;
    using I2 = std::integral_constant<int, 2>;

    if (wave >= NW) {
        const unsigned at = lds_offset(lds);
        TileMover<PAGED, kMovers, KS>(a, kslab, vslab, table, L, wave - NW, lane).walk(n_steps, at, at + kVBase, kStepBytes);
        __syncthreads();                         // the two of the merge
        __syncthreads();
        return;
    }

    const int kg   = wave / NC;                  // which of a step's KS tiles
    const int col  = wave % NC;
    const int hh   = mine.head(col);               // query head within the group
    const int sb   = mine.block(col);              // which 32 query positions of the item
    const int qw0  = Q0 + kQPerWave * sb;        // first query index of the wave ...
    const int aw0  = P0 + qw0;                   // ... and its position
    const int h    = g * a.group + hh;
    // steps this wave computes in: up to the position of its own last query
    const int my_tiles = qw0 < NQ ? min(aw0 + kQPerWave - 1, L - 1) / kTile + 1 : 0;
    const int my_steps = my_tiles > kg ? (my_tiles - kg + KS - 1) / KS : 0;

    unsigned vt_off[8];
    vt_offsets(n16, gq, vt_off);
    float m[2] = {kNegBig, kNegBig};
    float l[2] = {0.f, 0.f};                               // this lane's share of the weights' sums
    const float lazy_raw = kLazyBits / a.scale_log2e;      // the threshold in raw score units
    float4_t o[2][8];
#pragma unroll
    for (int nb = 0; nb < 2; ++nb)
#pragma unroll
        for (int e = 0; e < 8; ++e) o[nb][e] = float4_t{0.f, 0.f, 0.f, 0.f};

    // ---- Q^T operands
    Frag qreg[2][4];
    load_q(a, q_first, qw0, NQ, h, n16, gq, qreg);
#pragma unroll
    for (int nb = 0; nb < 2; ++nb)
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) asm volatile("" : "+v"(qreg[nb][kk].u));
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(0) & 0xc07f);

    const unsigned char *kmine = lds + kg * kTileBytes;
    const unsigned char *vmine = lds + kVBase + kg * kTileBytes;
    const int t_mine = kg * kTile;

    // Step i, staged in ring slot B (= i % kBufs, as a compile-time constant).
    auto step = [&](int i, auto buf_c, auto first_c) __attribute__((always_inline)) {
        constexpr int B = decltype(buf_c)::value;
        constexpr bool FIRST = decltype(first_c)::value;
        // the step's tiles have landed, and this wave is done with the step before
        __builtin_amdgcn_s_waitcnt(0xc07f);
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        if (i >= my_steps) return;
        const unsigned char *kb = kmine + B * kStepBytes;
        const unsigned char *vb = vmine + B * kStepBytes;

        // ---- S^T = K Q^T
        float4_t s[2][2];
#pragma unroll
        for (int nb = 0; nb < 2; ++nb) s[nb][0] = s[nb][1] = float4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) {
            const int off = n16 * kRowBytes + (((4 * kk + gq) ^ n16) << 4);   // row n16, piece 4kk+gq
            Frag k0, k1;
            k0.u = *reinterpret_cast<const uint4_t *>(kb + off);
            k1.u = *reinterpret_cast<const uint4_t *>(kb + 16 * kRowBytes + off);
#pragma unroll
            for (int nb = 0; nb < 2; ++nb) {
                s[nb][0] = __builtin_amdgcn_mfma_f32_16x16x32_f16(k0.h, qreg[nb][kk].h, s[nb][0], 0, 0, 0);
                s[nb][1] = __builtin_amdgcn_mfma_f32_16x16x32_f16(k1.h, qreg[nb][kk].h, s[nb][1], 0, 0, 0);
            }
        }
        __builtin_amdgcn_sched_group_barrier(0x100, 4, 0);          // LDS reads of two 32-dim steps ...
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            __builtin_amdgcn_sched_group_barrier(0x008, 4, 0);      // ... products of one ...
            __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);      // ... reads of the one after next
        }
        __builtin_amdgcn_sched_group_barrier(0x008, 8, 0);
        const int t0 = i * (KS * kTile) + t_mine;
        if (t0 + kTile > aw0) mask_tile(s, aw0, t0, n16, gq);

        Frag p[2];
        Rest left[2];
        float psum[2];
        if constexpr (FIRST) {
            first_weights(s, a.scale_log2e, lazy_raw, m, p, psum, left);
        } else {
            // Optimistic pass: weights against the running maximum as it stands; the exact pass where
            // some lane's weights sum to more than kSumBound (rare).
#pragma unroll
            for (int nb = 0; nb < 2; ++nb) weights_block(s[nb], a.scale_log2e, -m[nb] * a.scale_log2e, p[nb], psum[nb]);
            if (__builtin_amdgcn_ballot_w64(!(psum[0] <= kSumBound && psum[1] <= kSumBound)) != 0) {
#pragma unroll
                for (int nb = 0; nb < 2; ++nb)
                    raise_block(s[nb], a.scale_log2e, lazy_raw, m[nb], l[nb], o[nb], p[nb], psum[nb]);
            }
        }
        l[0] += psum[0];
        l[1] += psum[1];

        // ---- O^T += V^T P^T
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const Frag v = v_operand(vb, vt_off, e);
#pragma unroll
            for (int nb = 0; nb < 2; ++nb) o[nb][e] = __builtin_amdgcn_mfma_f32_16x16x32_f16(v.h, p[nb].h, o[nb][e], 0, 0, 0);
        }
        __builtin_amdgcn_sched_group_barrier(0x100, 6, 0);          // LDS reads of three 16-dim blocks ahead
#pragma unroll
        for (int j = 0; j < 5; ++j) {
            __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);
            __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
        }
        __builtin_amdgcn_sched_group_barrier(0x008, 6, 0);
        if constexpr (FIRST) add_rest(vb, vt_off, left, l, o);
    };
    using First = std::true_type;
    using Later = std::false_type;
    step(0, I0{}, First{});
    static_assert(kBufs == 3, "the loop below is unrolled by the number of buffers");
    for (int i = 1; i < n_steps; i += kBufs) {
        step(i, I1{}, Later{});
        if (i + 1 < n_steps) step(i + 1, I2{}, Later{});
        if (i + 2 < n_steps) step(i + 2, I0{}, Later{});
    }
    l[0] = quad_rows_sum(l[0]);
    l[1] = quad_rows_sum(l[1]);

    // ---- this lane's query rows: dims 16e + 4gq .. +3 of query 16nb + n16
    auto store_dims = [&](int nb, int e, float inv) __attribute__((always_inline)) {
        const int qpos = qw0 + 16 * nb + n16;        // query index
        const long long row = q_first + qpos;
        if (qpos >= NQ || row < 0 || row >= a.n_tokens) return;
        const half2_t lo = __builtin_convertvector((float2_t){o[nb][e][0] * inv, o[nb][e][1] * inv}, half2_t);
        const half2_t hi = __builtin_convertvector((float2_t){o[nb][e][2] * inv, o[nb][e][3] * inv}, half2_t);
        union { half2_t h[2]; unsigned long long u; } pk;
        pk.h[0] = lo;
        pk.h[1] = hi;
        *reinterpret_cast<unsigned long long *>(reinterpret_cast<_Float16 *>(a.out) + (row * a.n_qh + h) * kD + 16 * e + 4 * gq) = pk.u;
    };
    // The two waves of a column hold the same queries and dims in the same lanes: each hands the
    // accumulators of one query block to the other through LDS ([column][block][e][lane]) and
    // finishes the other block.
    static_assert(NC * 2 * 8 * 1024 + NC * 2 * 512 <= 2 * kBufs * kStepBytes, "the merge must fit in the staging area");
    __syncthreads();                             // every wave is past its last tile
    float4_t *mo = reinterpret_cast<float4_t *>(lds);
    float2_t *mml = reinterpret_cast<float2_t *>(lds + NC * 2 * 8 * 1024);
    auto send = [&](int nb) __attribute__((always_inline)) {
#pragma unroll
        for (int e = 0; e < 8; ++e) mo[((col * 2 + nb) * 8 + e) * 64 + lane] = o[nb][e];
        mml[(col * 2 + nb) * 64 + lane] = float2_t{m[nb], l[nb]};
    };
    auto finish = [&](int nb) __attribute__((always_inline)) {
        const float2_t other = mml[(col * 2 + nb) * 64 + lane];
        const float mx = fmaxf(m[nb], other[0]);
        const float f_own = __builtin_amdgcn_exp2f((m[nb] - mx) * a.scale_log2e);
        const float f_other = __builtin_amdgcn_exp2f((other[0] - mx) * a.scale_log2e);
        const float inv = 1.0f / fmaf(f_other, other[1], l[nb] * f_own);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const float4_t y = mo[((col * 2 + nb) * 8 + e) * 64 + lane];
#pragma unroll
            for (int t = 0; t < 4; ++t) o[nb][e][t] = fmaf(f_other, y[t], o[nb][e][t] * f_own);
            store_dims(nb, e, inv);
        }
    };
    if (kg == 0) send(1);
    else         send(0);
    __syncthreads();
    if (kg == 0) finish(0);
    else         finish(1);
}

}  // namespace

hipError_t sw_launch_prefill_halves(const SwPrefillArgs &a_in, hipStream_t stream, const SwLaunchEvents *ev)
{
    SwPrefillArgs a = a_in;
    if (a.head_dim != kD || a.hp != 0 || a.qw < 1 || a.group * a.qw % 4 != 0) return hipErrorInvalidValue;
    int compact;
    const long long blocks = sw_prefill_blocks_by_work(a, 4, &compact);
    a.compact = compact;
    if (blocks <= 0 || blocks > 0x7fffffffLL) return hipErrorInvalidValue;
    const dim3 grid((unsigned)blocks);
    return a.block_table ? sw_launch(sw_prefill_halves_kernel<true>, grid, dim3(512 + 64 * kMovers), 0, stream, ev, a)
                         : sw_launch(sw_prefill_halves_kernel<false>, grid, dim3(512 + 64 * kMovers), 0, stream, ev, a);
}
