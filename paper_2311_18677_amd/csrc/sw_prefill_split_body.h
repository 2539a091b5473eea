// The key-split prompt kernel's workgroup (see sw_prefill_split.hip), as a device function: the
// prompt kernel of its own runs it, and so does the mixed-batch kernel, beside the token-phase
// workgroups.
#pragma once
#include "sw_prefill_common.h"

#include <type_traits>

namespace sw_split {

using namespace sw_prefill;

constexpr int kWaveLds = 2 * kTileBytes;     // K tile + V tile; reused for the merge (32 rows x 128 floats)

// LDS of a workgroup of WAVES waves.
template <int WAVES>
struct SplitLds {
    __attribute__((aligned(16))) unsigned char tiles[WAVES * kWaveLds];
    __attribute__((aligned(16))) unsigned char q[kQPerWave * kRowBytes];     // the block's 32 query rows
    float m[WAVES][kQPerWave];
    float l[WAVES][kQPerWave];
};

// Block-table variant: byte offset of the pool block behind each of a tile's 8 load instructions.
struct TileBlocks { long long off[8]; };

// PAGED: K and V are block pools addressed through the request's row of the block table
// (position t = row t % block_size of pool block table[t / block_size]).  `block` is the
// workgroup's number among the prompt workgroups.
template <int WAVES, bool PAGED>
__device__ __forceinline__ void prompt_workgroup(const SwPrefillArgs &a, unsigned block, SplitLds<WAVES> &sm)
{
    unsigned char *lds = sm.tiles, *sm_q = sm.q;
    float (&sm_m)[WAVES][kQPerWave] = sm.m;
    float (&sm_l)[WAVES][kQPerWave] = sm.l;

    // block -> (item = (request, query block), key/value head, query head of the group).
    // The heads of a group walk the same K/V tiles; consecutive workgroup numbers go to
    // different XCDs (eight L2s), so the heads of one (item, key/value head) are numbered
    // eight apart and meet behind the same L2.  With x = id % 8, y = id / 8: head y % group
    // of pair (y / group) * 8 + x (the host rounds the pairs up to a multiple of eight;
    // numbers past the last pair find no item).
    const unsigned x8 = block & 7u, y8 = block >> 3;
    const unsigned hh = y8 % (unsigned)a.group;
    const unsigned rest = (y8 / (unsigned)a.group) * 8u + x8;
    const int g = (int)(rest % (unsigned)a.n_kvh);
    const QItem it = find_item(a, rest / (unsigned)a.n_kvh, kQPerWave);
    if (!it.valid) return;
    const int r = it.r, qb = it.qb, L = it.L, NQ = it.NQ;   // NQ: the request's last NQ tokens are its queries
    const long long q_first = it.q_first;
    const int Q0 = qb * kQPerWave;               // first query index of the block ...
    if (Q0 >= NQ) return;
    const int A0 = L - NQ + Q0;                  // ... and its position

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n16  = lane & 15;
    const int gq   = lane >> 4;
    const int h    = g * a.group + (int)hh;
    unsigned char *wlds = lds + wave * kWaveLds;
    unsigned char *vlds = wlds + kTileBytes;
    const unsigned k_at = lds_offset(lds) + wave * kWaveLds;
    const unsigned v_at = k_at + kTileBytes;

    // ---- the block's query rows go global->LDS (pieces XOR-swizzled by row like K's), each
    // wave fetching its share; every load of the kernel is then of one kind and the waits
    // below count exactly.  Rows past the prompt repeat its last row (never stored).
    const unsigned q_at = lds_offset(sm_q);
#pragma unroll
    for (int c = 0; c < 8 / WAVES; ++c) {
        const int j = wave + WAVES * c;                   // rows 4j .. 4j+3
        const int qi = 4 * j + gq;
        const int qpos = min(Q0 + qi, NQ - 1);
        long long row = q_first + qpos;
        row = row < 0 ? 0 : (row >= a.n_tokens ? a.n_tokens - 1 : row);
        const uint16_t *src = a.q + (row * a.n_qh + h) * kD + 8 * (n16 ^ (qi & 15));
        request_1k_at(src, q_at + j * 1024);
    }

    // dense: the (request, head) slab; block table: the head's rows inside pool block 0
    const long long slab = PAGED ? (long long)g * a.stride_kvh : (long long)r * a.stride_req + (long long)g * a.stride_kvh;
    const char *kslab = reinterpret_cast<const char *>(a.k) + 2 * slab;
    const char *vslab = reinterpret_cast<const char *>(a.v) + 2 * slab;
    settled(kslab);
    settled(vslab);
    const_table_t table = PAGED ? (const_table_t)(a.block_table + (long long)r * a.max_blocks) : nullptr;
    const int in_block = PAGED ? (1 << a.block_shift) - 1 : ~0;

    // the tiles that hold every position the block's queries may see (all start inside the context)
    const int n_tiles = min(A0 + kQPerWave - 1, L - 1) / kTile + 1;

    // Per-lane byte offsets of a tile's load instructions relative to the tile's first row,
    // computed once: instruction n brings rows 4n .. 4n+3 (lane group gq row 4n+gq, lane n16
    // one 16-byte piece; K pieces XOR-swizzled by row).  A tile that lies wholly inside a
    // dense context then needs one 32-bit add per instruction in the vector unit: a
    // wave-uniform slab base plus (tile offset + these offsets).  Only a tile that reaches
    // past the context's end (the last one) takes the slow path that clamps every row.
    // (Keeping the whole uniform part in scalar registers was tried: the compiler then
    // builds 64-bit per-lane pointers and the loads lose their scalar-base form; no gain.)
    unsigned koff[4];
#pragma unroll
    for (int n = 0; n < 4; ++n) {
        const int rho = 4 * n + gq;
        koff[n] = (unsigned)(rho * kRowBytes + ((n16 ^ (rho & 15)) << 4));     // rows 16..31: + 4096
    }
    // V pieces are swizzled too (v_swizzle); rows 4n+gq and 4(n+2)+gq share a swizzle
    unsigned voff[2];
#pragma unroll
    for (int n = 0; n < 2; ++n) {
        const int rho = 4 * n + gq;
        voff[n] = (unsigned)(rho * kRowBytes + ((n16 ^ v_swizzle(rho)) << 4));   // rows +8, +16, +24: + 2048 each
    }
    // Block table: the same per-lane offsets inside a pool block, for tiles that lie wholly
    // inside the context (no row to clamp).  Row 4n + gq of a tile is row
    // (t0 + 4n + gq) % block_size of its block; tiles start at multiples of 32 and blocks hold
    // a power of two of positions, so that is (t0 % block_size) + ((4n + gq) % block_size)
    // with a wave-uniform first term, which goes into the scalar base of the load.
    unsigned pk_off[8], pv_off[8];
    if (PAGED) {
#pragma unroll
        for (int n = 0; n < 8; ++n) {
            const int rho = 4 * n + gq;
            const unsigned row = ((unsigned)rho & (unsigned)in_block) << 8;
            pk_off[n] = row | (unsigned)((n16 ^ (rho & 15)) << 4);
            pv_off[n] = row | (unsigned)((n16 ^ v_swizzle(rho)) << 4);
        }
    }
    unsigned vt_off[8];
    vt_offsets(n16, gq, vt_off);

    // Block table: byte offset of the pool block that holds row 4n of tile t0 (clamped like
    // the rows themselves).  The four rows of one load instruction always share a block:
    // blocks hold a multiple of four positions and tiles start at multiples of 32.  One
    // wave-uniform table read per instruction; ids are clamped into the pool.
    auto find_blocks = [&](int t0) __attribute__((always_inline)) {
        TileBlocks tb;
        if (PAGED && a.block_shift >= 5) {
            // blocks of 32 positions or more hold the whole tile: one table read
            int id = table[min(t0, L - 1) >> a.block_shift];
            id = id < 0 ? 0 : (id >= a.n_blocks ? a.n_blocks - 1 : id);
            const long long off = 2 * (long long)id * a.stride_block;
#pragma unroll
            for (int n = 0; n < 8; ++n) tb.off[n] = off;
            return tb;
        }
        if (PAGED && a.block_shift == 4) {
            // blocks of 16 positions: one read per half tile
            int id0 = table[min(t0, L - 1) >> 4];
            int id1 = table[min(t0 + 16, L - 1) >> 4];
            id0 = id0 < 0 ? 0 : (id0 >= a.n_blocks ? a.n_blocks - 1 : id0);
            id1 = id1 < 0 ? 0 : (id1 >= a.n_blocks ? a.n_blocks - 1 : id1);
            const long long off0 = 2 * (long long)id0 * a.stride_block;
            const long long off1 = 2 * (long long)id1 * a.stride_block;
#pragma unroll
            for (int n = 0; n < 8; ++n) tb.off[n] = n < 4 ? off0 : off1;
            return tb;
        }
        // (all eight table reads first, then the arithmetic: one wait instead of eight)
        int id[8];
#pragma unroll
        for (int n = 0; n < 8; ++n) id[n] = PAGED ? table[min(t0 + 4 * n, L - 1) >> a.block_shift] : 0;   // wave-uniform
#pragma unroll
        for (int n = 0; n < 8; ++n) {
            const int c = id[n] < 0 ? 0 : (id[n] >= a.n_blocks ? a.n_blocks - 1 : id[n]);
            tb.off[n] = PAGED ? 2 * (long long)c * a.stride_block : 0;
        }
        return tb;
    };

    auto issue_k = [&](int t0, const TileBlocks &tb) __attribute__((always_inline)) {
        if (!PAGED && t0 + kTile <= L) {
            // slab base (scalar) + one 32-bit add per instruction (a slab is below 4 GiB)
            const unsigned tile = (unsigned)t0 << 8;
#pragma unroll
            for (int n = 0; n < 8; ++n)
                request_1k<true>(kslab, tile + (n >> 2) * 4096 + koff[n & 3], k_at + n * 1024);
        } else if (PAGED && t0 + kTile <= L) {
            const long long in_blk = (long long)(((unsigned)t0 & (unsigned)in_block) << 8);
#pragma unroll
            for (int n = 0; n < 8; ++n)
                request_1k<false>(kslab + (tb.off[n] + in_blk), pk_off[n], k_at + n * 1024);
        } else {
#pragma unroll
            for (int n = 0; n < 8; ++n) {
                const int rho = 4 * n + gq;
                const int t = min(t0 + rho, L - 1);      // rows past the context repeat its last row (masked)
                request_1k<false>(kslab + tb.off[n], (((unsigned)t & (unsigned)in_block) << 8) | (unsigned)((n16 ^ (rho & 15)) << 4),
                           k_at + n * 1024);
            }
        }
    };
    auto issue_v = [&](int t0, const TileBlocks &tb) __attribute__((always_inline)) {
        if (!PAGED && t0 + kTile <= L) {
            const unsigned tile = (unsigned)t0 << 8;
#pragma unroll
            for (int n = 0; n < 8; ++n)
                request_1k<true>(vslab, tile + (n >> 1) * 2048 + voff[n & 1], v_at + n * 1024);
        } else if (PAGED && t0 + kTile <= L) {
            const long long in_blk = (long long)(((unsigned)t0 & (unsigned)in_block) << 8);
#pragma unroll
            for (int n = 0; n < 8; ++n)
                request_1k<false>(vslab + (tb.off[n] + in_blk), pv_off[n], v_at + n * 1024);
        } else {
#pragma unroll
            for (int n = 0; n < 8; ++n) {
                const int rho = 4 * n + gq;
                const int t = min(t0 + rho, L - 1);
                request_1k<false>(vslab + tb.off[n], (((unsigned)t & (unsigned)in_block) << 8) | (unsigned)((n16 ^ v_swizzle(rho)) << 4),
                           v_at + n * 1024);
            }
        }
    };

    Frag qreg[2][4];
    float m[2] = {kNegBig, kNegBig};
    float l[2] = {0.f, 0.f};                               // this lane's share of the weights' sums
    const float lazy_raw = kLazyBits / a.scale_log2e;
    float4_t o[2][8];
#pragma unroll
    for (int nb = 0; nb < 2; ++nb)
#pragma unroll
        for (int e = 0; e < 8; ++e) o[nb][e] = float4_t{0.f, 0.f, 0.f, 0.f};

    // One tile (scores s): its V is in flight or there on entry, and so is the next tile's K.
    // MORE: the wave has a next tile; ahead (wave-uniform): and one after that.
    // The first product of the next tile runs beside this tile's softmax: the matrix cores
    // work while the wave's vector unit does the exponentials.
    auto process_tile = [&](int t0, auto more_c, bool ahead, bool first, TileBlocks &vb, float4_t (&s)[2][2],
                            float4_t (&s_next)[2][2]) __attribute__((always_inline)) {
        constexpr bool MORE = decltype(more_c)::value;
        const int t1 = t0 + WAVES * kTile;
        TileBlocks nb2;
        Frag kop[2][4];
        if (MORE) {
            // block ids of the tile after next: requested first, needed once K(next) has been read
            nb2 = ahead ? find_blocks(t1 + WAVES * kTile) : vb;
            // outstanding, oldest first: K(next) x8, V(this) x8 -- on the first tile the other way round
            if (first) __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
            else       __builtin_amdgcn_s_waitcnt(vmcnt_imm(8));
            asm volatile("" ::: "memory");
            load_k_ops(wlds, n16, gq, kop);
            // every read of the K tile has returned before its area is refilled
            __builtin_amdgcn_s_waitcnt(0xc07f);
            if (ahead) issue_k(t1 + WAVES * kTile, nb2);
            qk_block(0, kop, qreg, s_next);
            qk_block(1, kop, qreg, s_next);
        }
        // Optimistic pass: weights against the running maximum as it stands; the exact pass where
        // some lane's weights sum to more than kSumBound (rare after the first tiles).
        Frag p[2];
        float psum[2];
#pragma unroll
        for (int nb = 0; nb < 2; ++nb) weights_block<true>(s[nb], a.scale_log2e, -m[nb] * a.scale_log2e, p[nb], psum[nb]);
        if (MORE) {
#pragma unroll
            for (int k = 0; k < 16; ++k) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);      // one matrix instruction ...
                __builtin_amdgcn_sched_group_barrier(0x002, 4, 0);      // ... four vector instructions
            }
        }
        if (__builtin_amdgcn_ballot_w64(!(psum[0] <= kSumBound && psum[1] <= kSumBound)) != 0) {
#pragma unroll
            for (int nb = 0; nb < 2; ++nb)
                raise_block<true>(s[nb], a.scale_log2e, lazy_raw, m[nb], l[nb], o[nb], p[nb], psum[nb]);
        }
        l[0] += psum[0];
        l[1] += psum[1];
        // outstanding, oldest first: V(this) x8, then K(after next) x8 if it exists
        if (MORE && ahead) __builtin_amdgcn_s_waitcnt(vmcnt_imm(8));
        else               __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
        asm volatile("" ::: "memory");
        Frag va[8];
        load_vt(vlds, vt_off, va);
        if (MORE) {
            __builtin_amdgcn_s_waitcnt(0xc07f);
            issue_v(t1, vb);
            vb = nb2;
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            o[0][e] = __builtin_amdgcn_mfma_f32_16x16x32_f16(va[e].h, p[0].h, o[0][e], 0, 0, 0);
            o[1][e] = __builtin_amdgcn_mfma_f32_16x16x32_f16(va[e].h, p[1].h, o[1][e], 0, 0, 0);
        }
        if (MORE && t1 + kTile > A0) mask_tile(s_next, A0, t1, n16, gq);
    };

    int ti = wave;
    TileBlocks vb = find_blocks(0);                     // blocks of the next tile whose V is to be requested
    if (ti < n_tiles) {
        const TileBlocks tb = find_blocks(ti * kTile);
        issue_k(ti * kTile, tb);
        issue_v(ti * kTile, tb);
        vb = find_blocks((ti + WAVES) * kTile);         // (clamped to the context)
        __builtin_amdgcn_s_waitcnt(vmcnt_imm(16));      // this wave's query rows have landed
    } else {
        __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
    }
    __builtin_amdgcn_s_barrier();                       // ... and so have the other waves'
    asm volatile("" ::: "memory");

    if (ti < n_tiles) {
        // Q^T operands: lane (n16, gq) holds dims 32kk + 8gq .. +7 of query 16nb + n16
#pragma unroll
        for (int nb = 0; nb < 2; ++nb)
#pragma unroll
            for (int kk = 0; kk < 4; ++kk)
                qreg[nb][kk].u = *reinterpret_cast<const uint4_t *>(
                    sm_q + (16 * nb + n16) * kRowBytes + (((4 * kk + gq) ^ n16) << 4));
        float4_t s0[2][2], s1[2][2];
        {
            Frag kop[2][4];
            __builtin_amdgcn_s_waitcnt(vmcnt_imm(8));   // K(first) has landed
            asm volatile("" ::: "memory");
            load_k_ops(wlds, n16, gq, kop);
            __builtin_amdgcn_s_waitcnt(0xc07f);
            if (ti + WAVES < n_tiles) issue_k((ti + WAVES) * kTile, vb);
            qk_block(0, kop, qreg, s0);
            qk_block(1, kop, qreg, s0);
            if ((ti + 1) * kTile > A0) mask_tile(s0, A0, ti * kTile, n16, gq);
        }
        bool first = true;
        for (;;) {
            if (ti + WAVES >= n_tiles) break;
            process_tile(ti * kTile, std::true_type{}, ti + 2 * WAVES < n_tiles, first, vb, s0, s1);
            ti += WAVES;
            first = false;
            if (ti + WAVES >= n_tiles) { copy_scores(s1, s0); break; }
            process_tile(ti * kTile, std::true_type{}, ti + 2 * WAVES < n_tiles, false, vb, s1, s0);
            ti += WAVES;
        }
        process_tile(ti * kTile, std::false_type{}, false, false, vb, s0, s1);
    }
    l[0] = quad_rows_sum(l[0]);
    l[1] = quad_rows_sum(l[1]);

    // ---- merge the waves through LDS.  Each wave writes its accumulators over its own
    // staging area as [query 0..31][dim 0..127] floats (16-byte pieces XOR-swizzled by
    // query); this lane owns query 16nb + n16, dims 16e + 4gq + i.
    float *mo = reinterpret_cast<float *>(wlds);
#pragma unroll
    for (int nb = 0; nb < 2; ++nb) {
        const int qi = 16 * nb + n16;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int piece = 4 * e + gq;                                 // dims 4*piece .. 4*piece+3
            *reinterpret_cast<float4_t *>(mo + qi * kD + 4 * (piece ^ qi)) = o[nb][e];
        }
        if (gq == 0) {
            sm_m[wave][qi] = m[nb];
            sm_l[wave][qi] = l[nb];
        }
    }
    __syncthreads();
    for (int idx = threadIdx.x; idx < kQPerWave * (kD / 4); idx += 64 * WAVES) {
        const int qi = idx >> 5;
        const int piece = idx & 31;
        const int qpos = Q0 + qi;                   // query index
        const long long row = q_first + qpos;
        if (qpos >= NQ || row < 0 || row >= a.n_tokens) continue;
        float mx = sm_m[0][qi];
#pragma unroll
        for (int w = 1; w < WAVES; ++w) mx = fmaxf(mx, sm_m[w][qi]);
        float4_t num = float4_t{0.f, 0.f, 0.f, 0.f};
        float den = 0.f;
#pragma unroll
        for (int w = 0; w < WAVES; ++w) {
            const float f = __builtin_amdgcn_exp2f((sm_m[w][qi] - mx) * a.scale_log2e);
            const float4_t x = *reinterpret_cast<const float4_t *>(
                reinterpret_cast<const float *>(lds + w * kWaveLds) + qi * kD + 4 * (piece ^ qi));
#pragma unroll
            for (int t = 0; t < 4; ++t) num[t] = fmaf(f, x[t], num[t]);
            den = fmaf(f, sm_l[w][qi], den);
        }
        const float inv = 1.0f / den;
        const half2_t lo = __builtin_convertvector((float2_t){num[0] * inv, num[1] * inv}, half2_t);
        const half2_t hi = __builtin_convertvector((float2_t){num[2] * inv, num[3] * inv}, half2_t);
        union { half2_t h[2]; unsigned long long u; } pk;
        pk.h[0] = lo;
        pk.h[1] = hi;
        *reinterpret_cast<unsigned long long *>(reinterpret_cast<_Float16 *>(a.out) + (row * a.n_qh + h) * kD + 4 * piece) = pk.u;
    }
}

}  // namespace sw_split
