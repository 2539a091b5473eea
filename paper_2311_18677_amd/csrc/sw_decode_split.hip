// Token-phase (decode) attention on the matrix cores, split over context length, one launch
// (gfx950, wave64), head_dim 128 or 64, 16 query heads of a key/value head per workgroup
// (larger groups, up to 64 heads, in head tiles of 16).
//
// The step the paper's token machines run for every generated token (sections 2.2 and
// 3.5): the newest token's query attends over the whole cached context, which is read
// exactly once.  S^T = K Q^T and O^T = V^T P^T run on v_mfma_f32_16x16x32_f16 with the
// group's heads on the 16-wide N axis (head = lane % 16), so the first product's output
// layout is the second product's B-operand layout, P never moves between lanes and every
// softmax scalar lives in the lane that owns the head.
//
// A workgroup handles one item: one chunk of one (request, key/value head), found from a
// scan of the lengths (sw_worklist.h).  A request of L positions is cut into
// nc = ceil(L / chunk) items of (nearly) equal numbers of 32-position tiles.  K and V tiles
// go global->LDS directly (no registers held while data is in flight, all of a wave's
// loads of one kind, so the waits count exactly); a wave keeps the next tile's K and V
// requests in flight while it computes the current tile:
//
//   wait K(i) | QK(i) from LDS | request K(i+1) | softmax(i) |
//   wait V(i) | V(i) LDS->registers | request V(i+1) | transpose, PV(i)
//
// The item's result is merged with the request's other items in the same launch
// (sw_fused.h), or -- FUSED = false -- left in the workspace for a merge kernel.
//
// Append variant (the newest token's rows join the cache in the same pass): the one wave
// whose tile holds the new position overwrites that row of its staged K and V tiles with
// the new rows (brought into LDS once per workgroup) and stores them to the cache in
// global memory; no other wave or workgroup reads that position.
//
// At head_dim 128 each wave owns 16 KB of LDS (K tile + V tile), so two 4-wave workgroups fit a
// compute unit; at 64 it owns 8 KB and four (three in the single-launch form, whose merge needs
// registers) fit, so as many bytes are in flight.  At head_dim 64 the vector-ALU kernel, which
// served it before, spends 30 lane instructions per row and head and is bound by them for groups
// of two heads and more.  A call, this kernel after that one: 64 requests of up to 3000 positions, 12
// heads on 4: 32.4 -> 22.1 us (3.2 -> 4.8 TB/s); 200 of 1500, 16 heads on one: 75.6 -> 19.7; 64 of
// 3000, 8 on 8: 66.9 -> 62.7 (6.3 TB/s); 4 of 128, 8 on 8: 5.3 -> 5.3.
// A weight is a binary32 value there and a binary16 pair here (about 22 bits): over two dozen shapes
// of 75 to 26000 positions both are 2.03e-4 to 2.16e-4 off 64 bits in the 2-norm, the same to five
// digits, which is the rounding of the results.
//
// The kernel's leading arguments repeat what the length scan needs: they arrive in
// registers with the wave (kernel-argument preload), so the lengths are requested before
// the rest of the arguments has been fetched.
#include "sw_internal.h"
#include "sw_worklist.h"
#include "sw_fused.h"
#include "sw_lane_ops.h"
#include "sw_prefill_split_body.h"

#include <type_traits>

namespace {

typedef _Float16 half8_t __attribute__((ext_vector_type(8)));
typedef float float4_t __attribute__((ext_vector_type(4)));
typedef unsigned int uint4_t __attribute__((ext_vector_type(4)));
typedef unsigned int uint2_t __attribute__((ext_vector_type(2)));

constexpr int   kTile     = 32;            // tokens per wave per iteration
constexpr float kNegBig   = -1.0e30f;
// A running maximum is raised only when a score exceeds it by more than this many
// binary orders of magnitude: weights then stay below 2^kLazyBits.
constexpr float kLazyBits = 8.0f;

typedef float float2_t __attribute__((ext_vector_type(2)));
typedef _Float16 half2_t __attribute__((ext_vector_type(2)));
// Cache policy of the K/V stream: non-temporal (read once; must not push the
// partial results, which are written and read back, out of L2).
constexpr int   kStream   = 2;

// s_waitcnt immediate for "at most n vector-memory operations outstanding" (n < 64),
// leaving the other counters unconstrained.
constexpr int vmcnt_imm(int n) { return (n & 15) | (7 << 4) | (15 << 8) | ((n >> 4) << 14); }

// Block-table variant: byte offset of the pool block behind each four rows of a tile.
struct TileBlocks { long long off[kTile / 4]; };

// The block table is read-only for the whole launch; reading it through the constant
// address space lets wave-uniform entries come in over the scalar path.
typedef const __attribute__((address_space(4))) int32_t *const_table_t;

union Frag {
    uint4_t u;
    half8_t h;
};

// 64 lanes x 16 bytes, global -> LDS, asynchronously; stream_lds (a base and an offset per lane)
// with the K/V stream's cache policy.  (Functions of their own: with builtin arguments whose types
// depend on a template parameter the compiler leaves the kernel without its host side.)
template <bool ASM>
__device__ __forceinline__ void load_lds(const void *src, unsigned char *to)
{
    if constexpr (ASM) sw_prefill::request_1k_at(src, sw_prefill::lds_offset(to));
    else               __builtin_amdgcn_global_load_lds(src, to, 16, 0, 0);
}

#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
template <bool ASM>
__device__ __forceinline__ void stream_lds(const char *base, unsigned off, unsigned char *to)
{
    if constexpr (ASM) {
        // (wait states: see request_1k)
        asm volatile("s_mov_b32 m0, %2\n\ts_nop 3\n\tglobal_load_lds_dwordx4 %1, %0 nt"
                     :: "s"(base), "v"(off), "s"(sw_prefill::lds_offset(to)) : "m0", "memory");
    } else {
        __builtin_amdgcn_global_load_lds(base + off, to, 16, 0, kStream);
    }
}
#pragma clang diagnostic pop

// No LDS read moves above a wait for assembly requests, which the compiler does not know of.
template <bool ASM>
__device__ __forceinline__ void landed()
{
    if constexpr (ASM) asm volatile("" ::: "memory");
}

// Two binary16 values, those that are not finite replaced by zero.
__device__ __forceinline__ unsigned finite_halves(unsigned u)
{
    if ((u & 0x00007c00u) == 0x00007c00u) u &= 0xffff0000u;
    if ((u & 0x7c000000u) == 0x7c000000u) u &= 0x0000ffffu;
    return u;
}

// Keeps a wave-uniform value in scalar registers from here on: whatever it is computed or
// loaded from has been waited for at this point.
template <typename T>
__device__ __forceinline__ void sw_pin(T &x)
{
    asm volatile("" : "+s"(x));
}

// D = head_dim.  A staged K or V row is 2 * D bytes and one load instruction (64 lanes x 16
// bytes) brings kRowsPerLoad whole rows: four at D = 128, eight at D = 64, where a wave's two
// tiles are half as large and twice the waves fit a compute unit.
// ASM: the rows are requested by inline assembly (see request_1k), for a kernel whose LDS
// arrays are one object: the compiler would hold every LDS read until all requests have landed.
// `block`: the workgroup's number among the token-phase workgroups; lds, sm_q, sm_m, sm_l, sm_flag:
// WAVES * kWaveLds bytes, 16 * kRowBytes + 1024 bytes (Q rows, then the append variant's new K row
// and new V row), and what the waves exchange.
template <int D, int WAVES, int PER, bool FUSED, bool PAGED, bool ASM>
__device__ __forceinline__ void decode_workgroup(const int32_t *seq_lens, int n_req, int max_len, int chunk_shift, int n_kvh,
                                                 const SwArgs &a_rest, unsigned block, unsigned char *lds, unsigned char *sm_q,
                                                 float (*sm_m)[16], float (*sm_l)[16], int *sm_flag)
{
    constexpr int kRowBytes    = 2 * D;                    // a staged row (K pieces XOR-swizzled, no padding)
    constexpr int kRowShift    = D == 128 ? 8 : 7;
    constexpr int kPieces      = kRowBytes / 16;           // 16-byte pieces (lanes) per row
    constexpr int kRowsPerLoad = 64 / kPieces;
    constexpr int kLoads       = kTile / kRowsPerLoad;     // load instructions of a tile
    constexpr int kBlocks      = D / 16;                   // 16-row blocks of the second product's output
    constexpr int kHeadStride  = D + 4;                    // floats; merge buffer row = head, D dims + padding
    constexpr int kTileBytes   = kTile * kRowBytes;
    constexpr int kWaveLds     = 2 * kTileBytes;           // K tile + V tile; the merge buffer reuses it
    static_assert(D == 128 || D == 64, "head_dim");
    static_assert(16 * kHeadStride * 4 <= kWaveLds, "merge buffer must fit in the wave's LDS area");
    SwArgs a = a_rest;
    a.seq_lens = seq_lens;
    a.n_req = n_req;
    a.max_len = max_len;
    a.chunk_shift = chunk_shift;
    a.chunk = 1 << chunk_shift;
    a.n_kvh = n_kvh;

    // -- phase: workgroup started
    // First of all the lengths: asking for them needs nothing but the leading arguments, which
    // arrive in registers.  While they travel, every other argument the workgroup will need is
    // read from the argument block in one go: left to itself the compiler reads each one where
    // it is first used, past the early exit below, which puts several scalar-memory round trips
    // in a row between knowing the item and asking for its first tile.
    const SwRawLens<PER> raw_lens = sw_scan_issue<PER>(a);
    sw_pin(a.q);
    sw_pin(a.k);
    sw_pin(a.v);
    sw_pin(a.q_rows);
    sw_pin(a.k_new);
    sw_pin(a.stride_req);
    sw_pin(a.stride_kvh);
    sw_pin(a.group);
    sw_pin(a.n_qh);
    sw_pin(a.n_chunks);
    sw_pin(a.scale_log2e);
    if (FUSED) {
        sw_pin(a.out);
        sw_pin(a.units);
        sw_pin(a.ws_tag);
        sw_pin(a.ws_tag_bytes);
    } else {
        sw_pin(a.ws_o);
        sw_pin(a.ws_ml);
    }
    if (PAGED) {
        sw_pin(a.block_table);
        sw_pin(a.stride_block);
        sw_pin(a.block_shift);
        sw_pin(a.max_blocks);
        sw_pin(a.n_blocks);
    }

    // ... and everything that does not depend on the item is done now, under the lengths' latency.
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // wave-uniform, kept in a scalar register
    const int n16  = lane & 15;     // head (B operand / output column), token (A operand of QK), dim chunk (A operand of PV)
    const int gq   = lane >> 4;     // k-slot group
    const int piece = lane % kPieces;       // a load instruction's lane: which 16 bytes ...
    const int lrow  = lane / kPieces;       // ... of which of its rows
    // the piece swizzle: sixteen rows' reads of one piece hit all banks once
    auto swizzle = [](int row) { return D == 128 ? row & 15 : (row >> 1) & 7; };
    unsigned char *wlds = lds + wave * kWaveLds;

    // A group of more than 16 query heads is served in head tiles of 16, one workgroup per
    // tile and chunk.  Consecutive workgroups go to different XCDs (eight L2s), so the tiles
    // of one chunk are numbered eight apart: they start almost together behind the SAME L2,
    // where the second and later readers of the chunk find it.  With x = id % 8, y = id / 8:
    // tile y % n_ht of item (y / n_ht) * 8 + x (the host rounds the items up to a multiple
    // of eight; numbers past the last item find no work).
    // h0 = the tile's first head within the group, gn = how many it has.
    const unsigned n_ht = (unsigned)(a.group + 15) >> 4;
    unsigned item = block;
    int ht = 0;
    if (n_ht > 1) {
        const unsigned x = block & 7u, y = block >> 3;
        ht = (int)(y % n_ht);
        item = (y / n_ht) * 8u + x;
    }
    const int h0 = 16 * ht;
    const int gn = min(16, a.group - h0);
    // Q^T rows of heads past the group are zero columns of the B operands.  Stored before any
    // global->LDS load is issued: no LDS store may follow a pending one.
    {
        const int row = kRowsPerLoad * wave + lrow;
        if (row < 16 && row >= gn)
            *reinterpret_cast<uint4_t *>(sm_q + row * kRowBytes + piece * 16) = uint4_t{0u, 0u, 0u, 0u};
    }
    float m = kNegBig, l = 0.f;                        // m in raw score units
    const float lazy_raw = kLazyBits / a.scale_log2e;  // the raise threshold in raw score units
    float4_t o[kBlocks];
#pragma unroll
    for (int e = 0; e < kBlocks; ++e) o[e] = float4_t{0.f, 0.f, 0.f, 0.f};

    const SwScan<PER> scan = sw_scan_finish<PER>(a, raw_lens);

    // Rows of requests with no cached position get +0; no item exists for them, so
    // workgroup b < n_req looks after request b.
    if (FUSED && block < (unsigned)a.n_req && sw_scanned_len<PER>(a, scan, (int)block) == 0)
        sw_zero_rows<D>(a, (int)block);
    const SwWork w = sw_lookup<PER>(a, scan, item);
    // -- phase: item known
    if (!w.valid) return;
    const int r = w.r, g = w.g, c = w.c;
    // the request's tiles of 32 positions, dealt evenly to its nc items: n_all = q * nc + rem
    // tiles, the first rem items take q + 1 of them.  (One division; both numbers are below
    // 2^24, so the single-precision quotient is off by at most one and one look at the
    // remainder settles it.)
    const unsigned n_all = (unsigned)(w.L + kTile - 1) / kTile;
    const unsigned nc = (unsigned)(w.L + a.chunk - 1) >> a.chunk_shift;
    unsigned quot = (unsigned)((float)n_all * __builtin_amdgcn_rcpf((float)nc));
    quot = __builtin_amdgcn_readfirstlane(quot);
    if (quot * nc > n_all) --quot;
    if ((quot + 1) * nc <= n_all) ++quot;
    const unsigned rem = n_all - quot * nc;
    const unsigned tile_begin = (unsigned)c * quot + min((unsigned)c, rem);
    const unsigned tile_count = quot + ((unsigned)c < rem ? 1u : 0u);
    const int t_begin = (int)(tile_begin * kTile);
    const int t_end = min(w.L, (int)((tile_begin + tile_count) * kTile));
    const bool alone = FUSED && nc == 1;            // the whole request: finished here, no merge
    const long long unit = ((long long)r * a.n_kvh + g) * n_ht + ht;
    SwFused fz;
    if (FUSED) {
        sw_fused_begin(a, fz, unit);
        fz.nc = (int)nc;
        fz.c = c;
        fz.merger = false;
    }

    // ---- Q^T for the B operands goes to LDS once per workgroup (row = head, chunks
    // swizzled like K's).  Wave w covers kRowsPerLoad rows with one global->LDS load: a lane
    // lands in slot `piece` of its row and therefore fetches piece slot ^ swizzle(row).
    {
        const int row = kRowsPerLoad * wave + lrow;
        if (row < gn) {            // at most 16 rows: the later waves may stage nothing
            const uint16_t *src = a.q + (sw_q_row(a, r) * a.n_qh + g * a.group + h0 + row) * D + 8 * (piece ^ swizzle(row));
            load_lds<ASM>(src, sm_q + wave * 1024);
        }
    }

    // Append variant: position the new rows go to if it lies in this chunk, else -1
    // (workgroup-uniform).  Wave 0 brings both rows into LDS with one load: the first kPieces
    // lanes the K row's 16-byte pieces, the next the V row's (the others repeat them).
    unsigned char *sm_new = sm_q + 16 * kRowBytes;
    const int new_pos = (w.new_pos >= t_begin && w.new_pos < t_end) ? w.new_pos : -1;
    if (new_pos >= 0 && wave == 0) {
        const uint16_t *src = ((lrow & 1) ? a.v_new : a.k_new) + ((long long)r * a.n_kvh + g) * D + 8 * piece;
        load_lds<ASM>(src, sm_new);
    }

    // Row addressing: a wave-uniform 64-bit base plus a 32-bit byte offset per lane.
    // Dense layout: the base is the (request, head) slab (below 4 GiB: max_len <= 2^23
    // rows of 256 bytes).  Block-table layout: the base is the pool block of the
    // instruction's rows.  Four aligned rows always share one block (blocks hold a multiple of
    // four positions and tiles start at multiples of 32), so the block id is a scalar table read;
    // ids are clamped into the pool.  At D = 64 an instruction brings eight rows: with blocks
    // of four positions, and only then, its two halves have bases of their own.
    const char *kslab = reinterpret_cast<const char *>(a.k) + 2 * ((long long)r * a.stride_req + (long long)g * a.stride_kvh);
    const char *vslab = reinterpret_cast<const char *>(a.v) + 2 * ((long long)r * a.stride_req + (long long)g * a.stride_kvh);
    // the table is read-only for the whole launch: read it through the constant address
    // space so that wave-uniform entries come in over the scalar path
    const_table_t table = PAGED ? (const_table_t)(a.block_table + (long long)r * a.max_blocks) : nullptr;
    const int in_block = PAGED ? (1 << a.block_shift) - 1 : ~0;
    const int n_tiles = (int)((unsigned)(t_end - t_begin + kTile - 1) / (unsigned)kTile);   // t_end > t_begin

    // byte offset, from the block-table base, of the block that holds row 4n of tile t0
    // (clamped like the rows themselves); unused in the dense layout
    auto find_blocks = [&](int t0) {
        TileBlocks tb;
        if (PAGED && a.block_shift >= 5) {
            // blocks of 32 positions or more hold the whole tile: one table read
            int id = table[min(t0, t_end - 1) >> a.block_shift];
            id = id < 0 ? 0 : (id >= a.n_blocks ? a.n_blocks - 1 : id);
            const long long off = 2 * (long long)id * a.stride_block;
#pragma unroll
            for (int n = 0; n < kTile / 4; ++n) tb.off[n] = off;
            return tb;
        }
        if (PAGED && a.block_shift == 4) {
            // blocks of 16 positions: one read per half tile
            int id0 = table[min(t0, t_end - 1) >> 4];
            int id1 = table[min(t0 + 16, t_end - 1) >> 4];
            id0 = id0 < 0 ? 0 : (id0 >= a.n_blocks ? a.n_blocks - 1 : id0);
            id1 = id1 < 0 ? 0 : (id1 >= a.n_blocks ? a.n_blocks - 1 : id1);
            const long long off0 = 2 * (long long)id0 * a.stride_block;
            const long long off1 = 2 * (long long)id1 * a.stride_block;
#pragma unroll
            for (int n = 0; n < kTile / 4; ++n) tb.off[n] = n < kTile / 8 ? off0 : off1;
            return tb;
        }
#pragma unroll
        for (int n = 0; n < kTile / 4; ++n) {
            tb.off[n] = 0;
            if (PAGED) {
                const int tu = min(t0 + 4 * n, t_end - 1);            // wave-uniform
                int id = table[tu >> a.block_shift];
                id = id < 0 ? 0 : (id >= a.n_blocks ? a.n_blocks - 1 : id);
                tb.off[n] = 2 * (long long)id * a.stride_block;
            }
        }
        return tb;
    };

    // K tile -> LDS, asynchronously.  Rows past the chunk's end re-read its last
    // row (in bounds, result masked below).  HALVES: blocks of four positions at D = 64, where
    // the lane's half of the load selects the block (a base per lane instead of per wave: its
    // own branch, because it makes every load's address a 64-bit sum per lane -- 29.4 us against
    // 22.0 for 64 requests over blocks of 16 positions).
    constexpr int kQuads = kRowsPerLoad / 4;
    const bool halves = PAGED && kQuads == 2 && a.block_shift == 2;
    auto issue_k_from = [&](int t0, const TileBlocks &tb, auto halves_c) {
        constexpr bool HALVES = decltype(halves_c)::value;
#pragma unroll
        for (int n = 0; n < kLoads; ++n) {
            const int rho = kRowsPerLoad * n + lrow;
            const int tk  = min(t0 + rho, t_end - 1);
            const char *from = kslab + (HALVES && lrow >= 4 ? tb.off[kQuads * n + kQuads - 1] : tb.off[kQuads * n]);
            stream_lds<ASM>(from, (((unsigned)tk & (unsigned)in_block) << kRowShift) | (unsigned)((piece ^ swizzle(rho)) << 4),
                            wlds + n * 1024);
        }
    };
    // V tile -> LDS, asynchronously, whole rows in token order; at D = 64, where a row covers
    // half of the banks, rows 4-7 of every eight swap places in pairs, so that the rows 4gq + n
    // of neighbouring lane groups lie in different halves.
    unsigned char *vlds = wlds + kTileBytes;
    auto v_slot = [](int row) { return D == 128 ? row : row ^ ((row >> 2) & 1); };      // its own inverse
    auto issue_v_from = [&](int t0, const TileBlocks &tb, auto halves_c) {
        constexpr bool HALVES = decltype(halves_c)::value;
#pragma unroll
        for (int n = 0; n < kLoads; ++n) {
            const int tv = min(t0 + v_slot(kRowsPerLoad * n + lrow), t_end - 1);
            const char *from = vslab + (HALVES && lrow >= 4 ? tb.off[kQuads * n + kQuads - 1] : tb.off[kQuads * n]);
            stream_lds<ASM>(from, (((unsigned)tv & (unsigned)in_block) << kRowShift) | (unsigned)(piece << 4), vlds + n * 1024);
        }
    };
    auto issue_k = [&](int t0, const TileBlocks &tb) {
        if (PAGED && kQuads == 2 && halves) issue_k_from(t0, tb, std::true_type{});
        else                                issue_k_from(t0, tb, std::false_type{});
    };
    auto issue_v = [&](int t0, const TileBlocks &tb) {
        if (PAGED && kQuads == 2 && halves) issue_v_from(t0, tb, std::true_type{});
        else                                issue_v_from(t0, tb, std::false_type{});
    };

    // One tile: the wave's loads for this tile are in flight on entry (K first,
    // then V).  MORE says whether the wave has a further tile, whose loads are
    // then issued from here; it is a compile-time flag so that the waits in
    // between can count exactly which loads are still outstanding.
    // CAREFUL: infinities in V, see the second walk below.
    auto process_tile = [&](int t0, int t0_next, auto more_c, auto careful_c) {
        constexpr bool MORE = decltype(more_c)::value;
        constexpr bool CAREFUL = decltype(careful_c)::value;
        // block ids of the next tile: requested first, needed only after QK
        TileBlocks nb;
        if (MORE) nb = find_blocks(t0_next);

        // ---- S^T = K Q^T : two 16-token blocks, four 32-dim steps.
        // Outstanding, oldest first: K(t0), V(t0), kLoads each.
        __builtin_amdgcn_s_waitcnt(vmcnt_imm(kLoads));
        landed<ASM>();
        // -- phase: K tile landed
        // the new position lies in the chunk's last tile, which is some wave's last tile
        const bool has_new = !MORE && new_pos >= t0 && new_pos < t0 + kTile;     // wave-uniform
        if (has_new && lrow == 0) {
            const int rho = new_pos - t0;
            *reinterpret_cast<uint4_t *>(wlds + rho * kRowBytes + ((piece ^ swizzle(rho)) << 4)) =
                *reinterpret_cast<const uint4_t *>(sm_new + piece * 16);
        }
        float4_t sacc[2];
        sacc[0] = float4_t{0.f, 0.f, 0.f, 0.f};
        sacc[1] = float4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int kk = 0; kk < D / 32; ++kk) {
            const int off = n16 * kRowBytes + (((4 * kk + gq) ^ swizzle(n16)) << 4);   // row n16, piece 4kk+gq
            Frag qb, k0, k1;
            qb.u = *reinterpret_cast<const uint4_t *>(sm_q + off);
            k0.u = *reinterpret_cast<const uint4_t *>(wlds + off);
            k1.u = *reinterpret_cast<const uint4_t *>(wlds + 16 * kRowBytes + off);
            sacc[0] = __builtin_amdgcn_mfma_f32_16x16x32_f16(k0.h, qb.h, sacc[0], 0, 0, 0);
            sacc[1] = __builtin_amdgcn_mfma_f32_16x16x32_f16(k1.h, qb.h, sacc[1], 0, 0, 0);
        }
        // The K tile's LDS area is refilled only once every read of it has RETURNED:
        // the global->LDS writes arrive outside the LDS instruction queue, so a
        // refill requested while reads are still queued can overtake them when the
        // rows come back quickly (cache-resident data).
        if (MORE) {
            __builtin_amdgcn_s_waitcnt(0xc07f);   // lgkmcnt(0)
            issue_k(t0_next, nb);
        }

        // ---- online softmax, base 2; this lane: head n16, tokens t0 + 16tb + 4gq + i.
        // m is kept in raw score units (the scale enters through one fused multiply-add) and
        // is only raised when a score exceeds it by more than kLazyBits binary orders of
        // magnitude, so the accumulators are rescaled rarely instead of every tile.
        float s[8];
#pragma unroll
        for (int tb = 0; tb < 2; ++tb)
#pragma unroll
            for (int i = 0; i < 4; ++i) s[4 * tb + i] = sacc[tb][i];
        // only a wave's last tile can reach past the chunk's end
        const bool ragged = !MORE && t0 + kTile > t_end;
        if (ragged) {
#pragma unroll
            for (int tb = 0; tb < 2; ++tb)
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (t0 + 16 * tb + 4 * gq + i >= t_end) s[4 * tb + i] = -INFINITY;
        }
        float mt = fmaxf(fmaxf(fmaxf(s[0], s[1]), fmaxf(s[2], s[3])),
                         fmaxf(fmaxf(s[4], s[5]), fmaxf(s[6], s[7])));
        mt = quad_rows_max(mt);
        const bool raise = mt > m + lazy_raw;
        if (__builtin_amdgcn_ballot_w64(raise) != 0) {
            const float m_new = raise ? mt : m;
            const float alpha = __builtin_amdgcn_exp2f((m - m_new) * a.scale_log2e);
            m = m_new;
            l *= alpha;
#pragma unroll
            for (int e = 0; e < kBlocks; ++e) o[e] *= alpha;
        }
        const float neg_m = -m * a.scale_log2e;
        float p[8];
        float psum = 0.f;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            p[j] = __builtin_amdgcn_exp2f(fmaf(s[j], a.scale_log2e, neg_m));
            psum += p[j];
        }
        l += psum;
        // weights as a binary16 pair hi + lo (together ~22 bits)
        Frag phi, plo;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            half2_t hi = __builtin_convertvector((float2_t){p[2 * j], p[2 * j + 1]}, half2_t);
            if (CAREFUL) {
                // a weight below binary16's range is a weight all the same where its row is infinite
                if (p[2 * j] > 0.f && hi[0] == (_Float16)0.f) hi[0] = (_Float16)0x1p-24f;
                if (p[2 * j + 1] > 0.f && hi[1] == (_Float16)0.f) hi[1] = (_Float16)0x1p-24f;
            }
            const half2_t lo = __builtin_convertvector(
                (float2_t){p[2 * j] - (float)hi[0], p[2 * j + 1] - (float)hi[1]}, half2_t);
            phi.h[2 * j] = hi[0];
            phi.h[2 * j + 1] = hi[1];
            plo.h[2 * j] = lo[0];
            plo.h[2 * j + 1] = lo[1];
        }

        // ---- V(t0): LDS -> registers.  Lane group gq takes the 8 tokens its P operand
        // holds, 4gq .. 4gq+3 and 16+4gq .. 16+4gq+3.
        // Outstanding, oldest first: V(t0), then K(next) if there is a next tile, kLoads each.
        if (MORE) __builtin_amdgcn_s_waitcnt(vmcnt_imm(kLoads));
        else      __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
        landed<ASM>();
        // -- phase: V tile landed
        if (has_new) {
            // all of the wave's loads have landed: patch the staged V row, then store
            // both rows to the cache (the first kPieces lanes the K row, the next the V row)
            if (lrow == 0)
                *reinterpret_cast<uint4_t *>(vlds + v_slot(new_pos - t0) * kRowBytes + piece * 16) =
                    *reinterpret_cast<const uint4_t *>(sm_new + kRowBytes + piece * 16);
            if (lrow < 2 && ht == 0) {       // every head tile patches its staged rows, the first one stores
                long long boff = 0;
                if (PAGED) {
                    int id = table[new_pos >> a.block_shift];
                    id = id < 0 ? 0 : (id >= a.n_blocks ? a.n_blocks - 1 : id);
                    boff = 2 * (long long)id * a.stride_block;
                }
                char *dst = const_cast<char *>(lrow ? vslab : kslab) + boff +
                            ((((unsigned)new_pos & (unsigned)in_block) << kRowShift) | (unsigned)(piece << 4));
                *reinterpret_cast<uint4_t *>(dst) = *reinterpret_cast<const uint4_t *>(sm_new + lrow * kRowBytes + piece * 16);
            }
        }
        // (this lane's kBlocks dims of every one of them: 16 bytes at D = 128, 8 at D = 64)
        typedef typename std::conditional<D == 128, uint4_t, uint2_t>::type vpiece_t;
        vpiece_t vreg[8];
#pragma unroll
        for (int n = 0; n < 8; ++n) {
            const int row = n < 4 ? 4 * gq + n : 16 + 4 * gq + (n - 4);
            vreg[n] = *reinterpret_cast<const vpiece_t *>(vlds + v_slot(row) * kRowBytes + n16 * (D / 8));
        }
        if (ragged) {
            // weights of the re-read rows are exactly 0; clear the rows too so that
            // a non-finite value in the last valid row cannot turn 0 * x into NaN
#pragma unroll
            for (int n = 0; n < 8; ++n)
                if (t0 + (n < 4 ? 4 * gq + n : 16 + 4 * gq + (n - 4)) >= t_end) vreg[n] = vpiece_t(0u);
        }
        // the V tile is in registers: its LDS area may be refilled
        if (MORE) {
            __builtin_amdgcn_s_waitcnt(0xc07f);   // lgkmcnt(0): the LDS reads above have returned
            issue_v(t0_next, nb);
        }

        // ---- O^T += V^T P^T : block e covers dims kBlocks*row + e (row = MFMA row)
#pragma unroll
        for (int e = 0; e < kBlocks; ++e) {
            const int w2 = e >> 1;
            const unsigned sel = (e & 1) ? 0x07060302u : 0x05040100u;
            Frag va;
#pragma unroll
            for (int j = 0; j < 4; ++j)
                va.u[j] = __builtin_amdgcn_perm(vreg[2 * j + 1][w2], vreg[2 * j][w2], sel);
            o[e] = __builtin_amdgcn_mfma_f32_16x16x32_f16(va.h, phi.h, o[e], 0, 0, 0);
            if (CAREFUL) {
#pragma unroll
                for (int j = 0; j < 4; ++j) va.u[j] = finite_halves(va.u[j]);
            }
            o[e] = __builtin_amdgcn_mfma_f32_16x16x32_f16(va.h, plo.h, o[e], 0, 0, 0);
        }
    };


    int ti = wave;
    auto issue_tile = [&](int t0) {
        const TileBlocks fb = find_blocks(t0);
        issue_k(t0, fb);
        issue_v(t0, fb);
    };
    if (ti < n_tiles) issue_tile(t_begin + ti * kTile);
    // -- phase: first loads issued
    // Q (and the new rows) must be in LDS before any wave goes on; the tile loads stay in flight
    // across the barrier.  Vector-memory operations complete in issue order, so
    // "at most the 2 * kLoads tile loads outstanding" means this wave's Q load is done.
    if (ti < n_tiles) __builtin_amdgcn_s_waitcnt(vmcnt_imm(2 * kLoads) & 0xc07f);   // and lgkmcnt(0)
    else              __builtin_amdgcn_s_waitcnt(vmcnt_imm(0) & 0xc07f);    // vmcnt(0),  lgkmcnt(0)
    __builtin_amdgcn_s_barrier();
    landed<ASM>();

    if (ti < n_tiles) {
        while (ti + WAVES < n_tiles) {
            process_tile(t_begin + ti * kTile, t_begin + (ti + WAVES) * kTile, std::true_type{}, std::false_type{});
            ti += WAVES;
        }
        process_tile(t_begin + ti * kTile, 0, std::false_type{}, std::false_type{});
        if constexpr (D == 64) {
            // An infinity in V times hi + lo is NaN wherever lo is not positive.  Finite rows leave
            // finite sums (a weight is at most 2^kLazyBits), so where a sum is not finite the wave
            // walks its tiles again, one at a time, with infinities in the hi product only: weight
            // times value as the vector unit has it, which served this head size before.  (At
            // head_dim 128 the pair's NaN is what the library has always given.)
            float4_t spoiled = o[0] * 0.f;
#pragma unroll
            for (int e = 1; e < kBlocks; ++e) spoiled += o[e] * 0.f;
            const float any = (spoiled[0] + spoiled[1]) + (spoiled[2] + spoiled[3]);
            if (__builtin_expect(__builtin_amdgcn_ballot_w64(any != 0.f) != 0, 0)) {
                m = kNegBig;
                l = 0.f;
#pragma unroll
                for (int e = 0; e < kBlocks; ++e) o[e] = float4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
                for (ti = wave; ti < n_tiles; ti += WAVES) {
                    __builtin_amdgcn_s_waitcnt(0);      // nothing outstanding on the areas that are refilled
                    issue_tile(t_begin + ti * kTile);
                    process_tile(t_begin + ti * kTile, 0, std::false_type{}, std::true_type{});
                }
            }
        }
    }

    // -- phase: tiles done
    // ---- the lane groups summed disjoint tokens into l
    l = quad_rows_sum(l);

    // ---- merge the waves through LDS (each wave reuses its own K staging area):
    // row = head (stride kHeadStride floats), column = dim; this lane owns dims
    // kBlocks * (4gq + i) + e, i.e. for each i one or two aligned groups of four consecutive dims
    float *mo = reinterpret_cast<float *>(wlds);
    if (n16 < gn) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int hf = 0; hf < kBlocks / 4; ++hf)
                *reinterpret_cast<float4_t *>(mo + n16 * kHeadStride + kBlocks * (4 * gq + i) + 4 * hf) =
                    float4_t{o[4 * hf][i], o[4 * hf + 1][i], o[4 * hf + 2][i], o[4 * hf + 3][i]};
        if (gq == 0) {
            sm_m[wave][n16] = m * a.scale_log2e;       // from here on in scaled (base-2 exponent) units
            sm_l[wave][n16] = l;
        }
    }
    __syncthreads();
    // Single launch: every wave's tiles are done.  One lane takes the unit's ticket; while the
    // answer travels, the threads merge the waves and send the chunk's pieces off.
    unsigned ticket = 0;
    if (FUSED && !alone && threadIdx.x == 0) ticket = sw_fused_ticket(a, unit);
    // (a group of more than 8 heads gives a thread two rows' worth of dims)
    constexpr int kMine = (16 * (D / 4) + 64 * WAVES - 1) / (64 * WAVES);
    float4_t my_num[kMine];
    float my_den[kMine], my_mx[kMine];
#pragma unroll
    for (int k = 0; k < kMine; ++k) {
        const int idx = threadIdx.x + k * 64 * WAVES;
        if (idx >= gn * (D / 4)) break;
        const int hh = idx / (D / 4);
        const int j4 = idx % (D / 4);
        float mx = sm_m[0][hh];
#pragma unroll
        for (int w = 1; w < WAVES; ++w) mx = fmaxf(mx, sm_m[w][hh]);
        float4_t num = float4_t{0.f, 0.f, 0.f, 0.f};
        float den = 0.f;
#pragma unroll
        for (int w = 0; w < WAVES; ++w) {
            const float f = __builtin_amdgcn_exp2f(sm_m[w][hh] - mx);
            const float4_t x = *reinterpret_cast<const float4_t *>(
                reinterpret_cast<const float *>(lds + w * kWaveLds) + hh * kHeadStride + 4 * j4);
#pragma unroll
            for (int t = 0; t < 4; ++t) num[t] = fmaf(f, x[t], num[t]);
            den = fmaf(f, sm_l[w][hh], den);
        }
        if (alone) {
            sw_store_final4<D>(a, sw_q_row(a, r) * a.n_qh + g * a.group + h0 + hh, j4, num, den);
            continue;
        }
        if (FUSED) {
            sw_fused_send<D>(a, fz, r, g, h0 + hh, j4, num, den, mx);
            my_num[k] = num;
            my_den[k] = den;
            my_mx[k] = mx;
            continue;
        }
        const long long slot = sw_ws_slot(a, r, g, c, h0 + hh);
        *reinterpret_cast<float4_t *>(a.ws_o + slot * D + 4 * j4) = num;
        if (j4 == 0) *reinterpret_cast<float2_t *>(a.ws_ml + slot * 2) = float2_t{mx, den};
    }
    // -- phase: results stored
    if (FUSED && !alone) {
        // the workgroup that drew the unit's last ticket folds the chunks: every other one has
        // sent its pieces before it drew its own
        if (threadIdx.x == 0) *sm_flag = sw_fused_is_merger(a, unit, ticket, (int)nc) ? 1 : 0;
        __syncthreads();
        if (*sm_flag == 0) return;
#pragma unroll
        for (int k = 0; k < kMine; ++k) {
            const int idx = threadIdx.x + k * 64 * WAVES;
            if (idx < gn * (D / 4))
                sw_fused_fold<D>(a, fz, r, g, h0 + idx / (D / 4), idx % (D / 4), my_num[k], my_den[k], my_mx[k]);
        }
    }
    // -- phase: merged
}

template <int D, int WAVES, int PER, bool FUSED, bool PAGED>
__global__ __launch_bounds__(64 * WAVES, D == 128 ? 2 : (FUSED ? 3 : 4))
void sw_decode_split_kernel(const int32_t *seq_lens, int n_req, int max_len, int chunk_shift, int n_kvh, SwArgs a)
{
    constexpr int kRowBytes = 2 * D;
    __shared__ __attribute__((aligned(16))) unsigned char lds[WAVES * 2 * kTile * kRowBytes];
    // Q rows, then (append variant) the new K row and the new V row.  One array: the
    // compiler sees no ordinary store into the new rows' part -- they arrive by
    // global->LDS load only -- and must not take it for never written.
    __shared__ __attribute__((aligned(16))) unsigned char sm_q[16 * kRowBytes + 1024];
    __shared__ float sm_m[WAVES][16];
    __shared__ float sm_l[WAVES][16];
    __shared__ int sm_flag;
    decode_workgroup<D, WAVES, PER, FUSED, PAGED, false>(seq_lens, n_req, max_len, chunk_shift, n_kvh, a, blockIdx.x,
                                                         lds, sm_q, sm_m, sm_l, &sm_flag);
}

// A mixed batch's two phases in one launch (paper section 2.4): workgroups 0 .. n_prompt - 1 are the
// key-split prompt kernel's, the others the token phase's.  The prompt's workgroups are few
// and each a long chain of dependent tiles that leaves memory idle, the token phase's stream the
// caches: in two launches the one waited for the other.  Prompt first, since a workgroup of
// it runs four times as long.  Both kinds use one LDS area (the sum of their arrays would leave
// one workgroup per compute unit).  63 token-phase requests of 1000 to 2600 cached tokens, 8
// heads over one, beside a prompt of 1500: 30.0 -> 26.8 us with the combine kernel; 10
// requests of 1800 to 11100, 8 heads over 8, beside two prompts of 103: 77.6 -> 53.5.
union MixedLds {
    sw_split::SplitLds<4> prompt;
    struct {
        __attribute__((aligned(16))) unsigned char lds[4 * 2 * kTile * 256];
        __attribute__((aligned(16))) unsigned char q[16 * 256 + 1024];
        float m[4][16], l[4][16];
        int flag;
    } token;
};

template <int PER, bool PAGED>
__global__ __launch_bounds__(256, 2)
void sw_mixed_kernel(const int32_t *seq_lens, int n_req, int max_len, int chunk_shift, int n_kvh, unsigned n_prompt,
                     SwArgs d, SwPrefillArgs p)
{
    __shared__ MixedLds sm;
    if (blockIdx.x < n_prompt)
        sw_split::prompt_workgroup<4, PAGED>(p, blockIdx.x, sm.prompt);
    else
        decode_workgroup<128, 4, PER, false, PAGED, true>(seq_lens, n_req, max_len, chunk_shift, n_kvh, d, blockIdx.x - n_prompt,
                                                          sm.token.lds, sm.token.q, sm.token.m, sm.token.l, &sm.token.flag);
}

}  // namespace

bool sw_decode_split_supported(const SwArgs &a)
{
    return (a.head_dim == 128 || a.head_dim == 64) && a.group <= 64 && (a.waves == 4 || a.waves == 8);
}

template <int D, int W, int P, bool FUSED, bool PAGED>
static hipError_t launch_form(const SwArgs &a, dim3 grid, hipStream_t stream, const SwLaunchEvents *ev)
{
    return sw_launch(sw_decode_split_kernel<D, W, P, FUSED, PAGED>, grid, dim3(64 * W), 0, stream, ev,
                     a.seq_lens, a.n_req, a.max_len, a.chunk_shift, a.n_kvh, a);
}

template <int D, int W, int P>
static hipError_t launch_split(const SwArgs &a, dim3 grid, hipStream_t stream, const SwLaunchEvents *ev)
{
    if (a.block_table)
        return a.units ? launch_form<D, W, P, true, true>(a, grid, stream, ev) : launch_form<D, W, P, false, true>(a, grid, stream, ev);
    return a.units ? launch_form<D, W, P, true, false>(a, grid, stream, ev) : launch_form<D, W, P, false, false>(a, grid, stream, ev);
}

template <int D, int W>
static hipError_t launch_per(const SwArgs &a, dim3 grid, hipStream_t stream, const SwLaunchEvents *ev)
{
    switch (sw_worklist_per(a.n_req)) {
    case 1:  return launch_split<D, W, 1>(a, grid, stream, ev);
    case 4:  return launch_split<D, W, 4>(a, grid, stream, ev);
    case 16: return launch_split<D, W, 16>(a, grid, stream, ev);
    default: return launch_split<D, W, 0>(a, grid, stream, ev);
    }
}

static long long decode_blocks(const SwArgs &a)
{
    const long long blocks = (long long)a.n_req * a.n_kvh * a.n_chunks;
    const int n_ht = (a.group + 15) / 16;
    return n_ht > 1 ? (blocks + 7) / 8 * 8 * n_ht : blocks;      // see the kernel's numbering of head tiles
}

hipError_t sw_launch_decode_split(const SwArgs &a, hipStream_t stream, const SwLaunchEvents *ev)
{
    if (!sw_decode_split_supported(a)) return hipErrorNotSupported;
    const long long blocks = decode_blocks(a);
    if (blocks > 0x7fffffffLL) return hipErrorInvalidValue;
    const dim3 grid((unsigned)blocks);
    if (a.head_dim == 128)
        return a.waves == 4 ? launch_per<128, 4>(a, grid, stream, ev) : launch_per<128, 8>(a, grid, stream, ev);
    return a.waves == 4 ? launch_per<64, 4>(a, grid, stream, ev) : launch_per<64, 8>(a, grid, stream, ev);
}

// Workgroups of the mixed kernel's prompt part (the prompt kernel's own grid), and whether its
// (request, query block) items are numbered compactly.
static long long mixed_prompt_blocks(const SwPrefillArgs &p, int *compact)
{
    const long long pairs = sw_prefill_items(p, sw_prefill::kQPerWave, sw_split_scans_early(p), compact) * p.n_kvh;
    return (pairs + 7) / 8 * 8 * p.group;
}

bool sw_mixed_supported(const SwArgs &d, const SwPrefillArgs &p)
{
    int compact;
    const long long n_prompt = mixed_prompt_blocks(p, &compact);
    return d.head_dim == 128 && p.head_dim == 128 && sw_decode_split_supported(d) && d.waves == 4 && !d.units && !d.k_new
        && sw_worklist_per(d.n_req) > 0 && n_prompt > 0 && n_prompt + decode_blocks(d) <= 0x7fffffffLL;
}

hipError_t sw_launch_mixed(const SwArgs &d, const SwPrefillArgs &p_in, hipStream_t stream, const SwLaunchEvents *ev)
{
    if (!sw_mixed_supported(d, p_in)) return hipErrorNotSupported;
    SwPrefillArgs p = p_in;
    int compact;
    const unsigned np = (unsigned)mixed_prompt_blocks(p, &compact);
    p.compact = compact;
    const dim3 grid((unsigned)(np + decode_blocks(d)));
#define SW_MIXED_CASE(P) \
    if (sw_worklist_per(d.n_req) == P) \
        return d.block_table \
            ? sw_launch(sw_mixed_kernel<P, true>, grid, dim3(256), 0, stream, ev, d.seq_lens, d.n_req, d.max_len, d.chunk_shift, d.n_kvh, np, d, p) \
            : sw_launch(sw_mixed_kernel<P, false>, grid, dim3(256), 0, stream, ev, d.seq_lens, d.n_req, d.max_len, d.chunk_shift, d.n_kvh, np, d, p);
    SW_MIXED_CASE(1) SW_MIXED_CASE(4) SW_MIXED_CASE(16)
#undef SW_MIXED_CASE
    return hipErrorInvalidValue;
}
