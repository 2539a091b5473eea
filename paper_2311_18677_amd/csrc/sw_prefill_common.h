// Pieces shared by the three prompt-phase (causal attention) kernels: operand
// types, the per-query online softmax and the second matrix product, both for a
// wave that owns 32 query positions (two 16-wide MFMA column blocks) of one head
// and works on tiles of 32 cached positions.  Lane (n16 = lane % 16, gq = lane / 16)
// owns query 16*nb + n16 of block nb and, of a tile's scores, positions
// 16*tb + 4*gq + i.
#pragma once
#include "sw_internal.h"
#include "sw_lane_ops.h"
#include "sw_worklist.h"

namespace sw_prefill {

typedef _Float16 half8_t __attribute__((ext_vector_type(8)));
typedef float float4_t __attribute__((ext_vector_type(4)));
typedef unsigned int uint4_t __attribute__((ext_vector_type(4)));
typedef float float2_t __attribute__((ext_vector_type(2)));
typedef _Float16 half2_t __attribute__((ext_vector_type(2)));

constexpr int   kD         = 128;
constexpr int   kTile      = 32;             // cached positions per tile
constexpr int   kRowBytes  = 256;
constexpr int   kTileBytes = kTile * kRowBytes;       // 8192: one K or one V tile
constexpr int   kQPerWave  = 32;             // query positions per wave
constexpr float kNegBig    = -1.0e30f;

// s_waitcnt immediate for "at most n vector-memory operations outstanding" (n < 64),
// leaving the other counters unconstrained; & 0xc07f adds "no LDS operation outstanding".
constexpr int vmcnt_imm(int n) { return (n & 15) | (7 << 4) | (15 << 8) | ((n >> 4) << 14); }

union Frag {
    uint4_t u;
    half8_t h;
};

// The running maximum of a query is only raised when a score exceeds it by more than
// this many binary orders of magnitude, and the accumulators are rescaled rarely instead
// of every tile.  Whether a raise is due is read off the sum of a lane's eight weights of
// a tile (no per-tile maximum): a sum of at most kSumBound = 8 * 2^kLazyBits changes
// nothing, so weights stay below 2^11 (exact enough in binary16, whose precision is
// relative); a larger sum means some score lies more than 2^kLazyBits above the maximum.
constexpr float kLazyBits = 8.0f;
constexpr float kSumBound = 8.0f * 256.0f;

// Query tokens of a request: with L cached positions and nq of them queries (the last
// nq; nq = L when no q_lens array is given), query index i is the token at position
// L - nq + i.
__device__ __forceinline__ int request_queries(const SwPrefillArgs &a, int r, int L)
{
    if (!a.q_lens) return L;
    const int cap = L < a.max_q ? L : a.max_q;
    int nq = a.q_lens[r];
    nq = nq < 0 ? 0 : (nq > cap ? cap : nq);
    // a request with a single query token is a token-phase request: when the call runs
    // those through the token-phase kernels, it is none of this kernel's business
    return (a.skip_single && nq == 1) ? 0 : nq;
}

// ---- workgroup -> (request, query block).  How many query blocks a request has depends
// on lengths only the device knows, so the grid is sized by a host-side bound and every
// wave finds its workgroup's item itself (no LDS, no barrier): items are numbered request
// by request, a request's late blocks (which see the most positions) first.  (When the
// bound is no smaller than requests x blocks-per-request anyway, the host asks for the
// direct mapping instead, which puts the late blocks of ALL requests first.)  A request
// owns one item per block of q_block query indices that holds a query whose row exists
// (rows outside [0, n_tokens) are never stored, so blocks of only such rows are no items).
struct QItem {
    int  r;            // request
    int  qb;           // query block: query indices qb * q_block ...
    int  L;            // cached positions of the request
    int  NQ;           // its query tokens (the last NQ positions)
    long long q_first; // row of its query index 0
    bool valid;        // false: nothing to do for this workgroup
};

__device__ __forceinline__ void request_span(const SwPrefillArgs &a, int r, int q_block, int &L, int &NQ,
                                             long long &q_first, int &qb_lo, int &cnt)
{
    L = a.seq_lens[r];
    q_first = a.q_starts[r];
    L = L < 0 ? 0 : (L > a.max_len ? a.max_len : L);
    NQ = request_queries(a, r, L);
    const long long lo = q_first < 0 ? -q_first : 0;                       // first query index with a row
    const long long room = a.n_tokens - q_first;
    const long long hi = room < (long long)NQ ? room : (long long)NQ;      // one past the last
    qb_lo = cnt = 0;
    if (hi > lo) {
        qb_lo = (int)(lo / q_block);
        cnt = (int)((hi - 1) / q_block) - qb_lo + 1;
    }
}

// The largest of the lanes' values (none negative).
__device__ __forceinline__ int wave_max(int x)
{
    x = max(x, __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, true));   // row_shr:1, 2, 4, 8: see the scan
    x = max(x, __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, true));
    x = max(x, __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, true));
    x = max(x, __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, true));
    x = max(x, __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false));  // row_bcast:15, 31
    x = max(x, __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false));
    return __builtin_amdgcn_readlane(x, 63);
}

// The same with the items of all requests numbered by work, longest first (one request per lane,
// n_req <= 64), for the kernels whose workgroups have a compute unit each: their time ends with
// the last workgroups, and with the requests one after the other those were the last request's, its
// longest blocks among them (which batches take it: sw_prefill_blocks_by_work).  A block's work is
// the position it ends at: its level, in blocks.  Levels are taken in up to 64 bands of 2^sh (finer
// ones gain nothing), the band that holds the item is found by bisection, a scan over the requests
// a step, and inside a band the requests follow each other.
// With the cache store, 8 heads on one: 16 prompts of 100 to 1900 tokens 89.5 -> 70.5 us, 4 of 500 to
// 8000 234 -> 207, 3 of 4000 to 9000 343 -> 284; 32 heads on 8, 16 of 48 to 880 90.2 -> 83.3; 16
// heads on one, 12 of 1258 to 3776 388 -> 378.  The key-split kernel's workgroups, two to a compute
// unit and a quarter as long, gain nothing and pay for the steps (6 prompts of 44 to 792 tokens, 8
// heads on 8, up to 0.90): there the requests stay one after the other.  So they do beyond 64 requests.
__device__ __forceinline__ QItem find_item_by_work(const SwPrefillArgs &a, unsigned item, int q_block)
{
    QItem it;
    it.r = it.qb = it.L = it.NQ = 0;
    it.q_first = 0;
    it.valid = false;
    const int lane = threadIdx.x & 63;
    int L = 0, NQ = 0, qb_lo = 0, cnt = 0, top = 0;
    long long qf = 0;
    if (lane < a.n_req) {
        request_span(a, lane, q_block, L, NQ, qf, qb_lo, cnt);
        if (cnt > 0) top = (int)((unsigned)(L - NQ) / (unsigned)q_block) + qb_lo + cnt;
    }
    const int levels = wave_max(top);
    const int sh = levels <= 64 ? 0 : 32 - __builtin_clz((unsigned)(levels - 1) >> 6);      // 64 << sh >= levels
    auto from_band = [&](int x) {                   // items at band x and above
        return (unsigned)__builtin_amdgcn_readlane(sw_wave_inclusive_scan(min(max(top - (x << sh), 0), cnt)), 63);
    };
    if (from_band(0) <= item) return it;            // past the last item
    int band = 0;
    unsigned above = 0;                             // items above the band
    for (int step = levels > 1 ? 1 << (31 - __builtin_clz((unsigned)((levels - 1) >> sh))) : 0; step > 0; step >>= 1) {
        const unsigned n = from_band(band + step);
        if (n > item) band += step;
        else          above = n;
    }
    const int higher = min(max(top - ((band + 1) << sh), 0), cnt);          // this lane's items above the band ...
    const int mine = min(max(top - (band << sh), 0), cnt) - higher;         // ... and in it
    const int incl = sw_wave_inclusive_scan(mine);
    const unsigned long long hit = __ballot((unsigned)incl > item - above);
    if (hit == 0) return it;                        // cannot happen when the counts are right
    const int owner = __builtin_ctzll(hit);
    const int rank = (int)(item - above) - __builtin_amdgcn_readlane(incl - mine - higher, owner);
    it.r = owner;
    it.qb = __builtin_amdgcn_readlane(qb_lo + cnt, owner) - 1 - rank;
    it.L = __builtin_amdgcn_readlane(L, owner);
    it.NQ = __builtin_amdgcn_readlane(NQ, owner);
    const unsigned lo32 = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(unsigned long long)qf, owner);
    const unsigned hi32 = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)((unsigned long long)qf >> 32), owner);
    it.q_first = (long long)(((unsigned long long)hi32 << 32) | lo32);
    it.valid = true;
    return it;
}

// Called by all 64 lanes of a wave; every wave of a workgroup gets the same answer.  BY_WORK: see
// find_item_by_work.
template <bool BY_WORK = false>
__device__ __forceinline__ QItem find_item(const SwPrefillArgs &a, unsigned item, int q_block)
{
    QItem it;
    it.r = it.qb = it.L = it.NQ = 0;
    it.q_first = 0;
    it.valid = false;
    if (!a.compact) {
        // direct mapping: item = (n_qblocks - 1 - qb) * n_req + r, late blocks of all requests first
        const int r = (int)(item % (unsigned)a.n_req);
        int L = a.seq_lens[r];
        it.q_first = a.q_starts[r];          // read together with the length: one wait for both
        L = L < 0 ? 0 : (L > a.max_len ? a.max_len : L);
        it.r = r;
        it.qb = a.n_qblocks - 1 - (int)(item / (unsigned)a.n_req);
        it.L = L;
        it.NQ = request_queries(a, r, L);
        it.valid = it.qb >= 0;
        return it;
    }
    if (BY_WORK && a.compact == kScanByWork) return find_item_by_work(a, item, q_block);
    const int lane = threadIdx.x & 63;
    const int per = (a.n_req + 63) >> 6;            // consecutive requests per lane
    int L = 0, NQ = 0, qb_lo = 0, cnt = 0, mine = 0;
    long long qf = 0;
    for (int j = 0; j < per; ++j) {
        const int r = lane * per + j;
        if (r < a.n_req) {
            request_span(a, r, q_block, L, NQ, qf, qb_lo, cnt);
            mine += cnt;
        }
    }
    const int incl = sw_wave_inclusive_scan(mine);
    const unsigned long long hit = __ballot((unsigned)incl > item);
    if (hit == 0) return it;                        // past the last item
    const int owner = __builtin_ctzll(hit);         // first lane whose requests reach the item
    unsigned before = (unsigned)__builtin_amdgcn_readlane(incl - mine, owner);
    int r = owner;
    if (per == 1) {
        L = __builtin_amdgcn_readlane(L, owner);
        NQ = __builtin_amdgcn_readlane(NQ, owner);
        qb_lo = __builtin_amdgcn_readlane(qb_lo, owner);
        cnt = __builtin_amdgcn_readlane(cnt, owner);
        const unsigned lo32 = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(unsigned long long)qf, owner);
        const unsigned hi32 = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)((unsigned long long)qf >> 32), owner);
        qf = (long long)(((unsigned long long)hi32 << 32) | lo32);
    } else {
        // walk the owner lane's requests again (wave-uniform loads, served from cache)
        cnt = 0;
        for (int j = 0; j < per; ++j) {
            before += (unsigned)cnt;
            r = min(owner * per + j, a.n_req - 1);
            request_span(a, r, q_block, L, NQ, qf, qb_lo, cnt);
            if (before + (unsigned)cnt > item) break;
        }
    }
    const unsigned local = item - before;
    if (local >= (unsigned)cnt) return it;          // cannot happen when the scan is right
    // wave-uniform by construction; say so, so that everything derived stays in scalar registers
    it.r = __builtin_amdgcn_readfirstlane(r);
    it.qb = __builtin_amdgcn_readfirstlane(qb_lo + cnt - 1 - (int)local);
    it.L = __builtin_amdgcn_readfirstlane(L);
    it.NQ = __builtin_amdgcn_readfirstlane(NQ);
    const unsigned lo32 = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)(unsigned long long)qf);
    const unsigned hi32 = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)((unsigned long long)qf >> 32));
    it.q_first = (long long)(((unsigned long long)hi32 << 32) | lo32);
    it.valid = true;
    return it;
}

// What a workgroup of the shared-tile kernels computes of its item: `cols` columns (query head, 32 query
// positions), wave by wave.
struct Columns {
    int width, first, head0;       // column c: head head0 + c % width, positions 32 * (c / width) .. +31 of the item
    __device__ __forceinline__ Columns(const SwPrefillArgs &a, int part, int cols)
        : width(a.hp ? a.hp : a.group), first(a.hp ? 0 : part * cols), head0(a.hp ? part * a.hp : 0) {}
    __device__ __forceinline__ int head(int i) const { return head0 + (first + i) % width; }
    __device__ __forceinline__ int block(int i) const { return (first + i) / width; }
};

// Q^T operands of a wave: lane (n16, gq) holds dims 32kk + 8gq .. +7 of the query with
// index q0 + 16nb + n16 (of nq).  Indices past the last query repeat it (never stored);
// row indices are clamped into [0, n_tokens).
__device__ __forceinline__ void load_q(const SwPrefillArgs &a, long long q_first, int q0, int nq, int h,
                                       int n16, int gq, Frag (&qreg)[2][4])
{
#pragma unroll
    for (int nb = 0; nb < 2; ++nb) {
        int qpos = q0 + 16 * nb + n16;
        qpos = qpos < nq ? qpos : nq - 1;
        long long row = q_first + qpos;
        row = row < 0 ? 0 : (row >= a.n_tokens ? a.n_tokens - 1 : row);
        const uint16_t *src = a.q + (row * a.n_qh + h) * kD + 8 * gq;
#pragma unroll
        for (int kk = 0; kk < 4; ++kk)
            qreg[nb][kk].u = *reinterpret_cast<const uint4_t *>(src + 32 * kk);
    }
}

// S^T = K Q^T for one tile staged at kb (rows XOR-swizzled by 16-byte piece):
// two 16-position blocks x two 16-query blocks, four 32-dim steps.
__device__ __forceinline__ void qk_tile(const unsigned char *kb, const Frag (&qreg)[2][4], int n16, int gq,
                                        float4_t (&sacc)[2][2])
{
#pragma unroll
    for (int nb = 0; nb < 2; ++nb)
#pragma unroll
        for (int tb = 0; tb < 2; ++tb) sacc[nb][tb] = float4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
        const int off = n16 * kRowBytes + (((4 * kk + gq) ^ n16) << 4);   // row n16, piece 4kk+gq
        Frag k0, k1;
        k0.u = *reinterpret_cast<const uint4_t *>(kb + off);
        k1.u = *reinterpret_cast<const uint4_t *>(kb + 16 * kRowBytes + off);
#pragma unroll
        for (int nb = 0; nb < 2; ++nb) {
            sacc[nb][0] = __builtin_amdgcn_mfma_f32_16x16x32_f16(k0.h, qreg[nb][kk].h, sacc[nb][0], 0, 0, 0);
            sacc[nb][1] = __builtin_amdgcn_mfma_f32_16x16x32_f16(k1.h, qreg[nb][kk].h, sacc[nb][1], 0, 0, 0);
        }
    }
}

// The same product in two steps, so that work of the two query blocks can be interleaved:
// the K operands of a tile (both 16-position blocks, four 32-dim steps) ...
__device__ __forceinline__ void load_k_ops(const unsigned char *kb, int n16, int gq, Frag (&kop)[2][4])
{
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
        const int off = n16 * kRowBytes + (((4 * kk + gq) ^ n16) << 4);
        kop[0][kk].u = *reinterpret_cast<const uint4_t *>(kb + off);
        kop[1][kk].u = *reinterpret_cast<const uint4_t *>(kb + 16 * kRowBytes + off);
    }
}

// ... and S^T of one query block from them.
__device__ __forceinline__ void qk_block(int nb, const Frag (&kop)[2][4], const Frag (&qreg)[2][4],
                                         float4_t (&sacc)[2][2])
{
    sacc[nb][0] = float4_t{0.f, 0.f, 0.f, 0.f};
    sacc[nb][1] = float4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
        sacc[nb][0] = __builtin_amdgcn_mfma_f32_16x16x32_f16(kop[0][kk].h, qreg[nb][kk].h, sacc[nb][0], 0, 0, 0);
        sacc[nb][1] = __builtin_amdgcn_mfma_f32_16x16x32_f16(kop[1][kk].h, qreg[nb][kk].h, sacc[nb][1], 0, 0, 0);
    }
}

typedef short short4_t __attribute__((ext_vector_type(4)));
typedef short4_t __attribute__((address_space(3))) *lds_short4_ptr;

// A staged V row keeps its sixteen 16-byte pieces XOR-swizzled by row, in pairs:
// piece p of row rho sits in slot p ^ v_swizzle(rho).  (Pairs, because the transposing
// read below takes 8 bytes per lane and two neighbouring lanes share a piece.)
__device__ __forceinline__ int v_swizzle(int rho) { return (rho & 7) << 1; }

// Byte offsets, inside a staged V tile, of this lane's sixteen transposing reads: entry
// [hk][e] serves keys 16hk + 4gq .. +3 and dims 16e .. 16e+15.  They depend on the lane
// only, so a kernel computes them once.
__device__ __forceinline__ void vt_offsets(int n16, int gq, unsigned (&off)[8])
{
    // rows 4gq + n16/4 (keys 0..15 of the tile); the rows 16 further on (keys 16..31) share
    // the swizzle and lie exactly 16 rows = 4096 bytes behind: an immediate offset of the read
    const int rho = 4 * gq + (n16 >> 2);                      // the row whose 8 bytes this lane addresses
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const int piece = 2 * e + ((n16 >> 1) & 1);           // dims 16e + 4(n16 % 4) .. +3 live in this piece
        off[e] = (unsigned)(rho * kRowBytes + ((piece ^ v_swizzle(rho)) << 4) + 8 * (n16 & 1));
    }
}

// V^T operands of the second product straight from LDS with the transposing read of
// gfx950 (ds_read_b64_tr_b16).  Within 16 lanes, result j of lane l is element l % 4 of
// the 8 bytes that lane 4j + l / 4 addresses; with the addresses of vt_offsets lane
// (n16, gq) therefore receives V[key 16hk + 4gq + j][dim 16e + n16], j = 0..3 -- exactly
// the A operand (row = dim 16e + n16, k-slots = the keys this lane group's P operand
// holds).  Block e covers dims 16e .. 16e+15 (row = MFMA row).
__device__ __forceinline__ void load_vt(const unsigned char *vb, const unsigned (&off)[8], Frag (&va)[8])
{
#pragma unroll
    for (int e = 0; e < 8; ++e)
#pragma unroll
        for (int hk = 0; hk < 2; ++hk) {
            union { short4_t s; unsigned int u[2]; } x;
            x.s = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4_ptr)(vb + off[e] + hk * 16 * kRowBytes));
            va[e].u[2 * hk] = x.u[0];
            va[e].u[2 * hk + 1] = x.u[1];
        }
}

// ---- pieces of the kernels that run a tile's softmax beside the next tile's first product

__device__ __forceinline__ void copy_scores(const float4_t (&from)[2][2], float4_t (&to)[2][2])
{
#pragma unroll
    for (int nb = 0; nb < 2; ++nb)
#pragma unroll
        for (int tb = 0; tb < 2; ++tb) to[nb][tb] = from[nb][tb];
}

// Causal mask of the scores of the tile at t0 (q0 = position of the wave's first query).
__device__ __forceinline__ void mask_tile(float4_t (&s)[2][2], int q0, int t0, int n16, int gq)
{
#pragma unroll
    for (int nb = 0; nb < 2; ++nb)
#pragma unroll
        for (int tb = 0; tb < 2; ++tb)
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (t0 + 16 * tb + 4 * gq + i > q0 + 16 * nb + n16) s[nb][tb][i] = -INFINITY;
}

// Sum of two binary16 values onto a binary32 one, each taken as it is and the sum rounded to binary32
// (v_fma_mix_f32 with one for the other factor; opaque, or the compiler takes the product away and
// converts by itself).  Not one more matrix product with ones in V's place, which the shared-tile kernel
// took before: two of 34 matrix instructions a tile, on a chip whose clock gives way under them (one prompt
// of 32768 tokens, 8 heads on one, with its cache store: 5 to 6 % in three sessions, 2043 -> 1945 us in one; of
// 16384 532 -> 503; 16 of 100 to 1900 96 -> 90.5).
// DOT: the two-element dot product, one instruction for two, in the key-split kernel.  The bits were the same
// in 500 calls of 1 to 64 heads, 1 to 20000 tokens; time without it over time with it 0.97 to 1.02, in the mean
// 1.002, and 1.008 where eight waves walk long chains.
template <bool DOT>
__device__ __forceinline__ float add_halves(half2_t w, float one, float sum)
{
    if constexpr (DOT) return __builtin_amdgcn_fdot2(w, half2_t{(_Float16)1.f, (_Float16)1.f}, sum, false);
    sum = __builtin_fmaf((float)w[0], one, sum);
    return __builtin_fmaf((float)w[1], one, sum);
}

__device__ __forceinline__ float opaque_one()
{
    float one = 1.f;
    asm("" : "+s"(one));
    return one;
}

// A tile's weights of one query block against the maximum behind neg_m (= -m * scale_log2e):
// rounded to binary16 (the second product's operand), and the lane's sum of the ROUNDED values in
// binary32: numerator and denominator of a row are built from the same rounded weights, w~_i =
// w_i (1 + d_i).  The row's error is then sum_i w_i d_i (v_i - out), which vanishes where one key
// dominates (its v is the row) -- with the exact sum as denominator it would be sum_i w_i d_i v_i, up
// to 2^-11 |v| for such a row, which alone exceeds the error bound once |v| reaches 4.
template <bool DOT = false>
__device__ __forceinline__ void weights_block(const float4_t (&s)[2], float scale_log2e, float neg_m, Frag &p, float &psum)
{
    const float one = opaque_one();
    psum = 0.f;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const float x = __builtin_amdgcn_exp2f(fmaf(s[j >> 1][2 * (j & 1)], scale_log2e, neg_m));
        const float y = __builtin_amdgcn_exp2f(fmaf(s[j >> 1][2 * (j & 1) + 1], scale_log2e, neg_m));
        const half2_t w = __builtin_convertvector((float2_t){x, y}, half2_t);
        p.h[2 * j] = w[0];
        p.h[2 * j + 1] = w[1];
        psum = add_halves<DOT>(w, one, psum);
    }
}

// The same, and what the rounding left of the weights, in binary16 again, with the lane's sum of it: with it the
// weights are good to about 22 bits.
struct Rest {
    Frag w;
    float sum;
};

__device__ __forceinline__ void weights_rest_block(const float4_t (&s)[2], float scale_log2e, float neg_m, Frag &p, float &psum,
                                                   Rest &rest)
{
    const float one = opaque_one();
    psum = rest.sum = 0.f;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const float x = __builtin_amdgcn_exp2f(fmaf(s[j >> 1][2 * (j & 1)], scale_log2e, neg_m));
        const float y = __builtin_amdgcn_exp2f(fmaf(s[j >> 1][2 * (j & 1) + 1], scale_log2e, neg_m));
        const half2_t w = __builtin_convertvector((float2_t){x, y}, half2_t);
        p.h[2 * j] = w[0];
        p.h[2 * j + 1] = w[1];
        psum = add_halves<false>(w, one, psum);
        const half2_t left = __builtin_convertvector((float2_t){x - (float)w[0], y - (float)w[1]}, half2_t);
        rest.w.h[2 * j] = left[0];
        rest.w.h[2 * j + 1] = left[1];
        rest.sum = add_halves<false>(left, one, rest.sum);
    }
}

// A tile's largest score of each query.
__device__ __forceinline__ float tile_max(const float4_t (&s)[2])
{
    return quad_rows_max(fmaxf(fmaxf(fmaxf(s[0][0], s[0][1]), fmaxf(s[0][2], s[0][3])),
                               fmaxf(fmaxf(s[1][0], s[1][1]), fmaxf(s[1][2], s[1][3]))));
}

// Raises the running maximum of one query block where a score of the tile lies more than kLazyBits above it, and
// rescales what has been accumulated.
__device__ __forceinline__ void raise_max(const float4_t (&s)[2], float scale_log2e, float lazy_raw, float &m, float &l,
                                          float4_t (&o)[8])
{
    const float mt = tile_max(s);
    const float m_new = mt > m + lazy_raw ? mt : m;
    const float alpha = __builtin_amdgcn_exp2f((m - m_new) * scale_log2e);
    m = m_new;
    l *= alpha;
#pragma unroll
    for (int e = 0; e < 8; ++e) o[e] *= alpha;
}

// The exact pass of one query block: that, and the tile's weights again.  (weights_block takes the
// maximum as it stands.)
template <bool DOT = false>
__device__ __forceinline__ void raise_block(const float4_t (&s)[2], float scale_log2e, float lazy_raw,
                                            float &m, float &l, float4_t (&o)[8], Frag &p, float &psum)
{
    raise_max(s, scale_log2e, lazy_raw, m, l, o);
    weights_block<DOT>(s, scale_log2e, -m * scale_log2e, p, psum);
}

// Both of a wave's first tile, where there is no maximum yet (m is kNegBig, l and o are zero).
__device__ __forceinline__ void first_weights(const float4_t (&s)[2][2], float scale_log2e, float lazy_raw, float (&m)[2],
                                              Frag (&p)[2], float (&psum)[2], Rest (&rest)[2])
{
#pragma unroll
    for (int nb = 0; nb < 2; ++nb) {
        const float mt = tile_max(s[nb]);
        m[nb] = mt > kNegBig + lazy_raw ? mt : kNegBig;        // (no position of the tile may be visible)
        weights_rest_block(s[nb], scale_log2e, -m[nb] * scale_log2e, p[nb], psum[nb], rest[nb]);
    }
}

// One operand of load_vt: dims 16e .. 16e+15 of the tile's V rows.
__device__ __forceinline__ Frag v_operand(const unsigned char *vb, const unsigned (&off)[8], int e)
{
    Frag v;
#pragma unroll
    for (int hk = 0; hk < 2; ++hk) {
        union { short4_t s; unsigned int u[2]; } x;
        x.s = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4_ptr)(vb + off[e] + hk * 16 * kRowBytes));
        v.u[2 * hk] = x.u[0];
        v.u[2 * hk + 1] = x.u[1];
    }
    return v;
}

// O^T += V^T rest^T behind the second product of one of a wave's first tiles.  An infinity in V stays out, where its
// sign would be the rest's.  It (or a NaN in V) has left a dim of the accumulators without a finite value in every
// query, which one block of queries tells; a query that is itself not finite has lost all its dims and no other's.
// 0.5 us a tile for two waves to a SIMD (without the rests of both tiles 32 prompts of 128 tokens, 8 heads on one,
// 12.9 -> 11.8 us; 8 of 1000, 8 on 8, 36.0 -> 35.0), where a second look at V's operands, the weights computed anew and a
// pass over the operands for each block of queries took 1.4.
__device__ __forceinline__ void add_rest(const unsigned char *vb, const unsigned (&vt_off)[8], const Rest (&rest)[2],
                                         float (&l)[2], float4_t (&o)[2][8])
{
    constexpr int kAhead = 2;                    // operands read ahead of their products
    Frag v[kAhead];
#pragma unroll
    for (int e = 0; e < kAhead; ++e) v[e] = v_operand(vb, vt_off, e);
    float top[2] = {0.f, 0.f};                   // (v_maximum3_f32, which hands a NaN on)
#pragma unroll
    for (int e = 0; e < 8; ++e)
#pragma unroll
        for (int i = 0; i < 2; ++i)
            top[i] = __builtin_elementwise_maximum(__builtin_elementwise_maximum(__builtin_fabsf(o[0][e][2 * i]),
                                                                                 __builtin_fabsf(o[0][e][2 * i + 1])), top[i]);
    unsigned long long lost = __builtin_amdgcn_ballot_w64(!(__builtin_elementwise_maximum(top[0], top[1]) < INFINITY));
    if (lost != 0) {                             // all sixteen queries of a lane group?
        for (int i = 1; i < 16; i *= 2) lost &= lost >> i;
        if (lost & 0x0001000100010001ull) return;
    }
    l[0] += rest[0].sum;
    l[1] += rest[1].sum;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
#pragma unroll
        for (int nb = 0; nb < 2; ++nb)
            o[nb][e] = __builtin_amdgcn_mfma_f32_16x16x32_f16(v[e % kAhead].h, rest[nb].w.h, o[nb][e], 0, 0, 0);
        if (e + kAhead < 8) v[e % kAhead] = v_operand(vb, vt_off, e + kAhead);
        __builtin_amdgcn_sched_barrier(0);
    }
}

// 64 lanes x 16 bytes, global -> LDS, asynchronously: lane l's bytes (at base + off, base
// wave-uniform) land at LDS offset lds_at + 16 l.  Inline assembly, because the compiler's
// wait-count pass holds an LDS read that may alias a pending request of the builtin form (every
// transposing read does) until all of them have landed; the kernels' own waits count exactly.
// (No output register: nothing of the instruction is outstanding for the register allocator.)
// The compiler's hazard pass does not know the instruction either.  The wait state it needs after
// M0 is written is here; the five after a vector instruction (v_readfirstlane) wrote the scalar
// base are here unless SETTLED, whose bases have passed settled(): they stay the same from tile to
// tile.  (All five in each request cost 2 to 7 % of the key-split kernel's time over dense caches;
// over block tables, where every request has a base of its own, they cost nothing measurable.)
// (M0 is a register the compiler keeps for itself; it takes the clobber, and so no value of its own
// across the statement, with a warning.)
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
template <bool SETTLED>
__device__ __forceinline__ void request_1k(const char *base, unsigned off, unsigned lds_at)
{
    if constexpr (SETTLED) {
        asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %0"
                     :: "s"(base), "v"(off), "s"(lds_at) : "m0", "memory");
    } else {
        asm volatile("s_mov_b32 m0, %2\n\ts_nop 3\n\tglobal_load_lds_dwordx4 %1, %0"
                     :: "s"(base), "v"(off), "s"(lds_at) : "m0", "memory");
    }
}

// (the same with a full address per lane, in vector registers)
__device__ __forceinline__ void request_1k_at(const void *src, unsigned lds_at)
{
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off"
                 :: "v"(src), "s"(lds_at) : "m0", "memory");
}
#pragma clang diagnostic pop

// Bases for the requests above, in scalar registers and long enough ago: whatever instruction
// computed them, requests may use them from here on.
__device__ __forceinline__ void settled(const char *&base) { asm volatile("s_nop 4" : "+s"(base)); }

// LDS offset of a __shared__ object, for the requests above.
__device__ __forceinline__ unsigned lds_offset(const void *p)
{
    return (unsigned)(uintptr_t)(__attribute__((address_space(3))) const unsigned char *)p;
}

// The block table is read-only for the whole launch; reading it through the constant
// address space lets wave-uniform entries come in over the scalar path.
typedef const __attribute__((address_space(4))) int32_t *const_table_t;

// A moving wave of the kernels that share staged tiles: it requests tiles and does nothing else.
// Requests are dealt to MOVERS such waves and not to the waves that compute, because these walk in step
// behind a barrier: dealt to them, every wave stands at the 16-cycle issue of all the others' requests before
// its first product (a tile's 16 requests took 7 % of the shared-tile kernel's time, in the form with
// two tiles a step twice that), and does the address arithmetic and the table reads between its products.
// A step is TILES consecutive tiles of K and of V.  Row group j of a step is rows 4(j%8) .. +3 of tile j/8:
// one request for K (16-byte pieces XOR-swizzled by row), one for V (by pairs of rows).
template <bool PAGED, int MOVERS, int TILES>
struct TileMover {
    static constexpr int C = 8 * TILES / MOVERS;       // row groups of a step that are this wave's
    static constexpr int kRequests = 2 * C;            // requests of a step
    static_assert(C * MOVERS == 8 * TILES, "row groups go round");
    const SwPrefillArgs &a;
    const char *kslab, *vslab;                         // settled
    const_table_t table;
    int L, mover, gq, n16, in_block;
    // this lane's byte offsets where a tile lies in the context whole: dense, inside the step's
    // tiles; block table, inside a pool block.  And where a request lands behind the step's first byte.
    unsigned k_off[C], v_off[C], at[C];

    __device__ __forceinline__ TileMover(const SwPrefillArgs &args, const char *k, const char *v, const_table_t t, int len,
                                         int which, int lane)
        : a(args), kslab(k), vslab(v), table(t), L(len), mover(which), gq(lane >> 4), n16(lane & 15),
          in_block(PAGED ? (1 << args.block_shift) - 1 : ~0)
    {
#pragma unroll
        for (int c = 0; c < C; ++c) {
            const int j = mover + MOVERS * c;
            const int rho = 4 * (j & 7) + gq;
            const unsigned row = PAGED ? (unsigned)(rho & in_block) * kRowBytes
                                       : (unsigned)((j >> 3) * kTileBytes + rho * kRowBytes);
            k_off[c] = row | (unsigned)((n16 ^ (rho & 15)) << 4);
            v_off[c] = row | (unsigned)((n16 ^ v_swizzle(rho)) << 4);
            at[c] = (unsigned)__builtin_amdgcn_readfirstlane(j * 1024);
            asm volatile("" : "+s"(at[c]));
        }
    }

    // This wave's share of step st -> LDS, K tiles from k_to on, V tiles from v_to on.
    __device__ __forceinline__ void request(int st, unsigned k_to, unsigned v_to) const
    {
        const bool whole = (st + 1) * (TILES * kTile) <= L;
        if (!PAGED && whole) {
            const unsigned tile = (unsigned)st * (TILES * kTileBytes);
#pragma unroll
            for (int c = 0; c < C; ++c) {
                request_1k<true>(kslab, tile + k_off[c], at[c] + k_to);
                request_1k<true>(vslab, tile + v_off[c], at[c] + v_to);
            }
            return;
        }
        // block table: the four rows of a request share a pool block (blocks hold a multiple of four
        // positions, tiles start at multiples of 32): one wave-uniform table read for K and V, the id
        // clamped into the pool
        long long block_off[C];
#pragma unroll
        for (int c = 0; c < C; ++c) {
            const int j = mover + MOVERS * c;
            block_off[c] = PAGED ? table[min((st * TILES + (j >> 3)) * kTile + 4 * (j & 7), L - 1) >> a.block_shift] : 0;
        }
#pragma unroll
        for (int c = 0; c < C; ++c) {
            if (!PAGED) continue;
            int id = (int)block_off[c];
            id = id < 0 ? 0 : (id >= a.n_blocks ? a.n_blocks - 1 : id);
            block_off[c] = 2 * (long long)id * a.stride_block;
        }
        if (PAGED && whole) {
            // row (t0 + rho) % block_size of a block is t0 % block_size + rho % block_size: t0 is a multiple of 32
#pragma unroll
            for (int c = 0; c < C; ++c) {
                const int t0 = (st * TILES + ((mover + MOVERS * c) >> 3)) * kTile;
                const long long off = block_off[c] + (long long)(((unsigned)t0 & (unsigned)in_block) * kRowBytes);
                request_1k<false>(kslab + off, k_off[c], at[c] + k_to);
                request_1k<false>(vslab + off, v_off[c], at[c] + v_to);
            }
            return;
        }
#pragma unroll
        for (int c = 0; c < C; ++c) {
            const int j = mover + MOVERS * c;
            const int rho = 4 * (j & 7) + gq;
            const int t = min((st * TILES + (j >> 3)) * kTile + rho, L - 1);       // rows past the prompt repeat its last row
            const unsigned row = ((unsigned)t & (unsigned)in_block) << 8;
            request_1k<!PAGED>(kslab + block_off[c], row | (unsigned)((n16 ^ (rho & 15)) << 4), at[c] + k_to);
            request_1k<!PAGED>(vslab + block_off[c], row | (unsigned)((n16 ^ v_swizzle(rho)) << 4), at[c] + v_to);
        }
    }

    // All n_steps of them, three ring slots: of step i, K lands at k_ring + (i % 3) * stride, V likewise.
    // One barrier a step, behind which every wave may read step i and this one fills the slot of step i - 1.
    __device__ __forceinline__ void walk(int n_steps, unsigned k_ring, unsigned v_ring, unsigned stride) const
    {
        request(0, k_ring, v_ring);
        if (n_steps > 1) request(1, k_ring + stride, v_ring + stride);
        unsigned ahead = 2 * stride;                   // slot of step i + 2
        for (int i = 0; i < n_steps; ++i) {
            // this wave's requests of step i have landed (those of step i + 1 may be in flight)
            if (i + 1 < n_steps) __builtin_amdgcn_s_waitcnt(vmcnt_imm(kRequests));
            else                 __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
            if (i + 2 < n_steps) request(i + 2, k_ring + ahead, v_ring + ahead);
            ahead = ahead == 2 * stride ? 0 : ahead + stride;
        }
    }
};

}  // namespace sw_prefill
