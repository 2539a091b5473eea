// Prompt-phase (causal) attention on the matrix cores (gfx950, wave64),
// head_dim 128, any number of query heads per key/value head (up to 8 of them share a workgroup).
//
// The prompt phase processes all tokens of a prompt in one pass (paper section
// 2.2) and is compute bound (section 3.5, Insight V): prompt token i attends to
// cached positions 0..i.  One workgroup takes one (request, key/value head) and a
// block of query positions; every wave owns 32 query positions of one query
// head, so no result is ever merged across waves.  K and V tiles of 32 positions
// travel global->LDS once per workgroup (three buffers, two tiles in flight) and
// are shared by all waves; the contractions are the ones of the token-phase
// kernel with the query position, not the head, on the 16-wide N axis:
//
//   S^T = K Q^T   A = K rows from LDS (swizzled), B = Q^T kept in registers
//   O^T += V^T P^T   A = V^T built in registers from V rows, B = P^T (binary16)
//
// Each lane therefore owns one query position: its running maximum, its sum and
// its causal bound are per-lane scalars, and its output row is stored straight
// from the accumulators.
//
// Two further waves request the tiles (TileMover in sw_prefill_common.h); the others only read LDS, multiply
// and weigh.  What bounds a computing wave is its own chain: 32 matrix instructions of 16 cycles, about
// 95 vector instructions of about 8 (a wave alone cannot issue them faster) and the LDS reads between
// them, with two such waves to a SIMD that a barrier keeps in step.  Behind it, on long calls, power: with all
// inputs zero one prompt of 32768 tokens takes 1.54 ms.
// Measured (8 heads on one, attention alone) against requests dealt to the computing waves: one prompt of 32768 tokens
// 1920 -> 1800 to 1900 us, of 16384 500 -> 468, 12 of 618 to 8039 560 -> 527; 8 heads on 8, 8 of 1024
// 36.1 -> 32.7; over blocks of 16 positions one of 16384 559 -> 459, 16 of 1024 57.4 -> 48.7.  One moving wave
// or four: dense within 1 % of two; over blocks of 4 positions one takes 8 % longer (its table reads).
// Tried: both products' operands read before the first product, the same; each product of one query block beside the other's weights 13 % slower; the first product at a raised
// wave priority 4 % slower; the key range in thirds for twelve waves, three to a SIMD, 6 % slower.
#include "sw_prefill_common.h"

#include <type_traits>

namespace {

using namespace sw_prefill;

constexpr int kBufBytes = 2 * kTileBytes;          // K tile, then V tile
constexpr int kBufs     = 3;
constexpr int kMovers   = 2;                       // waves that only request tiles
// A prompt's first tiles whose weights' rest is taken into the second product as well.  A row has one maximum here,
// whose own key's weight is exact, against the key-split kernel's four, and with weights of binary16 alone is up to 9 %
// further off 64 bits.  Error over the key-split kernel's, rows before position 128, from there to 256, to 512 and
// behind: one tile 0.92, 1.05, 1.03, 1.02; two 0.87, 0.99, 1.00, 1.00 (8 heads on one, 14 prompts of 371 tokens; 12 on
// 4, 900 to 1100).
constexpr int kRestTiles = 2;

// NW = computing waves per workgroup = (query heads per workgroup) * (waves per head); kMovers more
// request the tiles.
// PAGED: K and V are block pools addressed through the request's row of the block table
// (position t = row t % block_size of pool block table[t / block_size]).
template <int NW, bool PAGED>
__global__ __launch_bounds__(64 * (NW + kMovers), 1)
void sw_prefill_mfma_kernel(SwPrefillArgs a)
{
    __shared__ __attribute__((aligned(16))) unsigned char lds[kBufs * kBufBytes];

    // blockIdx -> (item = (request, query block), key/value head, part of the item's columns, later
    // positions first)
    const int q_block = kQPerWave * a.qw;        // query tokens of an item
    const unsigned n_parts = a.hp ? (unsigned)(a.group / a.hp) : (unsigned)(a.group * a.qw) / NW;
    const Columns mine(a, (int)(n_parts - 1 - blockIdx.x % n_parts), NW);
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
    const int last_pos = P0 + min(Q0 + kQPerWave * (mine.block(NW - 1) + 1), NQ) - 1;
    const int n_tiles = last_pos / kTile + 1;

    if (wave >= NW) {
        const unsigned at = lds_offset(lds);
        TileMover<PAGED, kMovers, 1>(a, kslab, vslab, table, L, wave - NW, lane).walk(n_tiles, at, at + kTileBytes, kBufBytes);
        return;
    }

    const int hh   = mine.head(wave);               // query head within the group
    const int sb   = mine.block(wave);              // which 32 query positions of the item
    const int qw0  = Q0 + kQPerWave * sb;        // first query index of the wave ...
    const int aw0  = P0 + qw0;                   // ... and its position
    const int h    = g * a.group + hh;

    // tiles this wave computes on: up to the position of its own last query
    const int my_tiles = qw0 < NQ ? min(aw0 + kQPerWave - 1, L - 1) / kTile + 1 : 0;

    if (my_tiles == 0) {                         // no query of its own: only the barriers
        for (int ti = 0; ti < n_tiles; ++ti) __builtin_amdgcn_s_barrier();
        return;
    }

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

    // One tile, staged in buffer B (= ti % kBufs, as a compile-time constant).  REST: the tile is
    // one of the first kRestTiles.
    auto step = [&](int ti, auto buf_c, auto rest_c) __attribute__((always_inline)) {
        constexpr int B = decltype(buf_c)::value;
        constexpr bool REST = decltype(rest_c)::value;
        // the tile has landed, and this wave is done with the one before
        __builtin_amdgcn_s_waitcnt(0xc07f);
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        if (ti >= my_tiles) return;

        const unsigned char *kb = lds + B * kBufBytes;
        const unsigned char *vb = kb + kTileBytes;
        const int t0 = ti * kTile;

        // K operands are read two 32-dim steps, V operands three 16-dim blocks ahead of their
        // products, and no further, which would take registers.
        float4_t sacc[2][2];
        qk_tile(kb, qreg, n16, gq, sacc);
        __builtin_amdgcn_sched_group_barrier(0x100, 4, 0);          // LDS reads of two 32-dim steps ...
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            __builtin_amdgcn_sched_group_barrier(0x008, 4, 0);      // ... products of one ...
            __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);      // ... reads of the one after next
        }
        __builtin_amdgcn_sched_group_barrier(0x008, 8, 0);
        if (t0 + kTile > aw0) mask_tile(sacc, aw0, t0, n16, gq);
        Frag p[2];
        Rest left[2];
        float psum[2];
        if constexpr (REST && B == 0) {
            first_weights(sacc, a.scale_log2e, lazy_raw, m, p, psum, left);
        } else {
            // Optimistic pass: weights against the running maximum as it stands; the exact pass where
            // some lane's weights sum to more than kSumBound (rare).
            auto weigh = [&](int nb) __attribute__((always_inline)) {
                if constexpr (REST) weights_rest_block(sacc[nb], a.scale_log2e, -m[nb] * a.scale_log2e, p[nb], psum[nb], left[nb]);
                else                weights_block(sacc[nb], a.scale_log2e, -m[nb] * a.scale_log2e, p[nb], psum[nb]);
            };
            weigh(0);
            weigh(1);
            if (__builtin_amdgcn_ballot_w64(!(psum[0] <= kSumBound && psum[1] <= kSumBound)) != 0) {
#pragma unroll
                for (int nb = 0; nb < 2; ++nb) {
                    raise_max(sacc[nb], a.scale_log2e, lazy_raw, m[nb], l[nb], o[nb]);
                    weigh(nb);
                }
            }
        }
        l[0] += psum[0];
        l[1] += psum[1];
        Frag va[8];
        load_vt(vb, vt_off, va);
#pragma unroll
        for (int e = 0; e < 8; ++e)
#pragma unroll
            for (int nb = 0; nb < 2; ++nb)
                o[nb][e] = __builtin_amdgcn_mfma_f32_16x16x32_f16(va[e].h, p[nb].h, o[nb][e], 0, 0, 0);
        __builtin_amdgcn_sched_group_barrier(0x100, 6, 0);          // LDS reads of three 16-dim blocks ahead
#pragma unroll
        for (int k = 0; k < 5; ++k) {
            __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);
            __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
        }
        __builtin_amdgcn_sched_group_barrier(0x008, 6, 0);
        if constexpr (REST) add_rest(vb, vt_off, left, l, o);
    };
    using I0 = std::integral_constant<int, 0>;
    using I1 = std::integral_constant<int, 1>;
    using I2 = std::integral_constant<int, 2>;
    using Rested = std::true_type;
    using Later = std::false_type;
    static_assert(kBufs == 3 && kRestTiles == 2, "tiles by number and by buffer");
    step(0, I0{}, Rested{});
    if (n_tiles > 1) step(1, I1{}, Rested{});
    for (int ti = 2; ti < n_tiles; ti += kBufs) {
        step(ti, I2{}, Later{});
        if (ti + 1 < n_tiles) step(ti + 1, I0{}, Later{});
        if (ti + 2 < n_tiles) step(ti + 2, I1{}, Later{});
    }

    // ---- this lane's query rows: dims 16e + 4gq + i
#pragma unroll
    for (int nb = 0; nb < 2; ++nb) {
        const float ls = quad_rows_sum(l[nb]);
        const int qpos = qw0 + 16 * nb + n16;        // query index
        const long long row = q_first + qpos;
        if (qpos < NQ && row >= 0 && row < a.n_tokens) {
            const float inv = 1.0f / ls;
            _Float16 *dst = reinterpret_cast<_Float16 *>(a.out) + (row * a.n_qh + h) * kD + 4 * gq;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const half2_t lo = __builtin_convertvector((float2_t){o[nb][e][0] * inv, o[nb][e][1] * inv}, half2_t);
                const half2_t hi = __builtin_convertvector((float2_t){o[nb][e][2] * inv, o[nb][e][3] * inv}, half2_t);
                union { half2_t h[2]; unsigned long long u; } pk;
                pk.h[0] = lo;
                pk.h[1] = hi;
                *reinterpret_cast<unsigned long long *>(dst + 16 * e) = pk.u;
            }
        }
    }
}

}  // namespace

bool sw_prefill_mfma_supported(const SwPrefillArgs &a)
{
    return a.head_dim == kD && a.group >= 1 && a.qw >= 1 && (a.hp == 0 ? a.group * a.qw % 8 == 0 : a.hp >= 1 && a.hp <= 8 && a.group % a.hp == 0);
}

// How a workgroup with whole heads is shaped: hp query heads of one group, the largest divisor of the group size
// up to eight, and qw waves (32 query positions each) per head, as many of the eight as that leaves.  (Cutting
// small problems into smaller workgroups was tried and measured slower: half the waves per staged tile, same
// chain of dependent tiles.)
void sw_prefill_shape(int group, int *hp, int *qw)
{
    int h = group < 8 ? group : 8;
    while (h > 1 && group % h != 0) --h;
    *hp = h;
    *qw = 8 / h;
}

hipError_t sw_launch_prefill_mfma(const SwPrefillArgs &a_in, hipStream_t stream, const SwLaunchEvents *ev)
{
    SwPrefillArgs a = a_in;
    if (!sw_prefill_mfma_supported(a)) return hipErrorNotSupported;
    int compact;
    const long long blocks = sw_prefill_blocks_by_work(a, 8, &compact);
    a.compact = compact;
    if (blocks <= 0 || blocks > 0x7fffffffLL) return hipErrorInvalidValue;
    const dim3 grid((unsigned)blocks);
    const int nw = a.hp ? a.hp * a.qw : 8;
#define SW_PREFILL_CASE(W) \
    if (nw == W) return a.block_table ? sw_launch(sw_prefill_mfma_kernel<W, true>, grid, dim3(64 * (W + kMovers)), 0, stream, ev, a) \
                                      : sw_launch(sw_prefill_mfma_kernel<W, false>, grid, dim3(64 * (W + kMovers)), 0, stream, ev, a);
    SW_PREFILL_CASE(8) SW_PREFILL_CASE(7) SW_PREFILL_CASE(6) SW_PREFILL_CASE(5)
    SW_PREFILL_CASE(4) SW_PREFILL_CASE(3) SW_PREFILL_CASE(2) SW_PREFILL_CASE(1)
#undef SW_PREFILL_CASE
    return hipErrorInvalidValue;
}
