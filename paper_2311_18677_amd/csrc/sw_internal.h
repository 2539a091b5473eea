// Internal interface between the host dispatcher (sw_api.hip) and the kernel
// translation units.  Not installed; the public ABI is include/sw_decode.h.
#pragma once
#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>
#include <stdint.h>

// State of one (request, key/value head, head tile) unit of the single-launch variant,
// kept between calls: the ticket counter is zero outside a launch, the epoch counts the
// calls in which the unit merged.
struct SwUnitState {
    unsigned ticket;
    unsigned epoch;
};

// Everything a kernel needs, passed by value.
//
// Split over context length: positions [0, L) of a request are cut into
// chunks of `chunk` positions; a workgroup of the partial kernel handles chunk
// c of key/value head g of request r for the query heads that head serves,
// and leaves per query head an unnormalised partial result in the workspace.
// The workspace is item-major, so that one workgroup writes one contiguous
// block: with slot(r, g, c, hh) = ((r*n_kvh + g)*n_chunks + c)*group + hh for
// the hh-th head of the group,
//   ws_o [slot*head_dim + j] = sum_t 2^(s2_t - m2) * V[t][j]
//   ws_ml[slot*2 + {0,1}]    = m2, sum_t 2^(s2_t - m2)
// where s2 = score * log2(e) (so that the exponentials are exp2) and m2 is
// the chunk's maximum of s2.  Chunks at or past L are never written nor read.
struct SwArgs {
    const uint16_t *q;
    const uint16_t *k;
    const uint16_t *v;
    const int32_t  *seq_lens;
    uint16_t       *out;
    float          *ws_o;
    float          *ws_ml;
    // single-launch variant (else units is null): per-unit ticket and epoch, the tagged
    // 16-byte pieces (see sw_fused.h), and a word the device sets if a merge gave up
    // waiting for a piece
    SwUnitState    *units;
    void           *ws_tag;
    unsigned        ws_tag_bytes;
    unsigned       *dev_err;
    const uint16_t *k_new;              // append variant: the newest token's K rows [n_req][n_kvh][head_dim], else null
    const uint16_t *v_new;              //                 and V rows
    const int32_t  *block_table;        // block-table variant: [n_req][max_blocks] pool block ids, else null
    // Token-phase part of a mixed batch (all null / 0 otherwise): request r takes part only
    // if exactly one of its tokens is a query (q_lens[r] clamped to [0, min(L, max_q)] is 1)
    // and q_rows[r] is a row of q and out ([n_rows][n_qh][head_dim]); its query and result
    // are that row instead of row r.  The other requests are neither read nor written.
    const int32_t  *q_rows;
    const int32_t  *q_lens;
    long long       n_rows;
    int             max_q;
    int   n_req, n_qh, n_kvh, group;   // group = n_qh / n_kvh
    int   head_dim, max_len;
    int   chunk, chunk_shift, n_chunks; // chunk = 1 << chunk_shift; n_chunks = ceil(max_len / chunk)
    int   waves;                        // waves per workgroup of the matrix-core partial kernel (4 or 8)
    long long stride_req, stride_kvh;  // elements; the token stride is head_dim
    // block-table variant: k, v are pools; row t of request r is row t % block_size of pool
    // block block_table[r*max_blocks + t / block_size]; stride_req is unused
    long long stride_block;
    int   block_shift, max_blocks, n_blocks;   // block_size = 1 << block_shift
    float scale_log2e;                 // log2(e) / sqrt(head_dim)
};

// Arguments of the prompt-phase (causal) kernel.
struct SwPrefillArgs {
    const uint16_t *q;                  // [n_tokens][n_qh][head_dim]
    const uint16_t *k;                  // caches in the dense layout
    const uint16_t *v;
    const int32_t  *seq_lens;           // prompt lengths
    const int32_t  *q_starts;           // row of each request's first query token
    const int32_t  *q_lens;             // query tokens per request (the last ones), or null: all of them
    uint16_t       *out;                // [n_tokens][n_qh][head_dim]
    long long n_tokens;
    int   n_req, n_qh, n_kvh, group;
    int   head_dim, max_len;
    int   max_q;                        // bound on the query tokens of a request (sizes the grid)
    int   skip_single;                  // non-zero: requests with exactly one query token are left out
    int   compact;                      // how workgroups find their (request, query block): see sw_prefill_items
    int   hp;                           // query heads (of one group) per workgroup; 0: the columns are dealt flat (sw_prefill_flat)
    int   qw;                           // waves per query head in a workgroup; flat: blocks of 32 query positions an item has
    int   n_qblocks;                    // query blocks (of 32 * qw positions) that cover max_len
    long long stride_req, stride_kvh;   // in elements
    // block-table variant: k, v are pools, row t of request r is row
    // t % block_size of pool block block_table[r*max_blocks + t / block_size]; stride_req unused
    const int32_t *block_table;         // null for the dense layout
    long long stride_block;
    int   block_shift, max_blocks, n_blocks;
    float scale_log2e;
};

// Arguments of the pools <-> dense copy of the KV hand-off.
struct SwHandoffArgs {
    uint16_t *k_pool, *v_pool;          // block pools
    uint16_t *k_dense, *v_dense;        // dense caches
    const int32_t *block_table;
    const int32_t *seq_lens;
    int   n_req, n_kvh, head_dim;
    int   cap;                          // positions copied at most: min(max_len, max_blocks * block_size)
    int   n_tiles;                      // workgroups per (request, head)
    int   block_shift, max_blocks, n_blocks;
    long long stride_block, p_stride_kvh;       // pools, in elements
    long long d_stride_req, d_stride_kvh;       // dense, in elements
};

// Number of cached positions request r attends over, with a flag.  seq_lens[r]
// is clamped to [0, max_len]; in the append variant it counts the positions
// cached BEFORE the newest token, whose K/V rows this call stores at that
// position (and attends over) unless the cache is already full.  Bit
// kSwAppendedBit of the result says that the rows are stored, i.e. that
// position L - 1 is the new one; the bits below it hold L (max_len <= 2^23).
// kSwSkip (negative, length bits 0) marks a request that takes no part in the call:
// it has no work item and its output row is left alone.
constexpr int kSwAppendedBit = 30;
constexpr int kSwLenMask     = (1 << kSwAppendedBit) - 1;
constexpr int kSwSkip        = (int)0x80000000u;

// (sw_flag_len: the same from a seq_lens[r] value that has already been read)
__device__ inline int sw_flag_len(const SwArgs &a, int r, int L)
{
    L = L < 0 ? 0 : (L > a.max_len ? a.max_len : L);
    if (a.q_lens) {
        const int cap = L < a.max_q ? L : a.max_q;
        const int nq = a.q_lens[r] < cap ? a.q_lens[r] : cap;
        const long long row = a.q_rows[r];
        if (nq != 1 || row < 0 || row >= a.n_rows) return kSwSkip;
    }
    if (a.k_new && L < a.max_len) L += 1 + (1 << kSwAppendedBit);
    return L;
}

__device__ inline int sw_request_len_flagged(const SwArgs &a, int r)
{
    return sw_flag_len(a, r, a.seq_lens[r]);
}

// Row of q and out that belongs to request r (valid for requests that take part).
__device__ inline long long sw_q_row(const SwArgs &a, int r)
{
    return a.q_rows ? (long long)a.q_rows[r] : (long long)r;
}

__device__ inline int sw_request_len(const SwArgs &a, int r)
{
    return sw_request_len_flagged(a, r) & kSwLenMask;
}

__host__ __device__ inline long long sw_ws_slot(const SwArgs &a, int r, int g, int c, int hh)
{
    return (((long long)r * a.n_kvh + g) * a.n_chunks + c) * a.group + hh;
}

// Optional per-kernel timing: when both are non-null the launch attaches them
// to the dispatch so that their difference is the kernel's device time.
struct SwLaunchEvents {
    hipEvent_t start;
    hipEvent_t stop;
};

// Vector-ALU partial kernel: any group size (looped in tiles of up to 8 heads).
hipError_t sw_launch_partial_valu(const SwArgs &a, hipStream_t stream, const SwLaunchEvents *ev);
// Matrix-core kernel, K and V staged through LDS (head_dim 128 or 64, groups up to 64, 4 or 8 waves).
bool       sw_decode_split_supported(const SwArgs &a);
hipError_t sw_launch_decode_split(const SwArgs &a, hipStream_t stream, const SwLaunchEvents *ev);
// A mixed batch's token phase (two-kernel form, partial results to the workspace) and prompt phase in one launch.
bool       sw_mixed_supported(const SwArgs &d, const SwPrefillArgs &p);
hipError_t sw_launch_mixed(const SwArgs &d, const SwPrefillArgs &p, hipStream_t stream, const SwLaunchEvents *ev);
// Merge of the chunks' partial results, normalisation and rounding to binary16.
hipError_t sw_launch_combine(const SwArgs &a, hipStream_t stream, const SwLaunchEvents *ev);
// Bound on the (request, block of q_block query tokens) items of a prompt-phase call, which
// sizes its grid: no request has more than n_qblocks of them, and requests whose rows of q
// and out do not overlap have at most n_tokens / q_block + 2 per request between them.
// *compact: how workgroups find their items: kDirect, or by a scan of the lengths, which costs each a little
// (every wave reads all the lengths, ceil(n_req / 64) per lane): it pays once it removes a good part
// of the grid, and never for huge batches.  `early`: also where it removes less.
enum { kDirect = 0, kScan = 1, kScanByWork = 2 };
static inline long long sw_prefill_items(const SwPrefillArgs &a, int q_block, bool early, int *compact)
{
    const long long by_shape = (long long)a.n_req * a.n_qblocks;
    const long long by_rows = a.n_tokens / q_block + 2LL * a.n_req;
    *compact = early || (by_rows * 4 < by_shape * 3 && a.n_req <= 4096) ? kScan : kDirect;
    return *compact ? by_rows : by_shape;
}
// Flat dealing of the shared-tile kernels' columns (query head, 32 query positions): the columns of an item, which
// is as many blocks of 32 positions as make the columns of all the group's heads a multiple of the `cols` that a
// workgroup computes, are numbered block by block, and a workgroup takes the next `cols` of them.  For groups
// of a power of two it is the dealing by whole heads; groups of three, five, six and seven have no idle waves.
static inline int sw_prefill_flat_blocks(int group, int cols)
{
    int common = cols;                                  // (cols is a power of two)
    while (group % common) common /= 2;
    return cols / common;
}
// Workgroups of `cols` columns that serve one item of one key/value head.
static inline int sw_prefill_parts(const SwPrefillArgs &a, int cols)
{
    return a.hp ? a.group / a.hp : a.group * a.qw / cols;
}
// The same for the kernels that can number a batch's items by work, with a compute unit to each of their
// workgroups, `cols` columns each; the number of these.  The numbering takes its workgroup a scan of the requests per step of
// the search, and shortens the call by a part of one chain: it wins where chains are long against the number
// of rounds of 256 workgroups.  Time without it over time with it, batches of 1 to 64 heads that are scanned either
// way: 0.95 to 1.60, in the mean 1.14, where a request has three blocks of 32 tokens a round; 0.90 to 1.16, in
// the mean 1.00, below (20 prompts of 490 tokens, 32 heads on 8: 92 -> 102 us; 24 of 250, 64 on 16: 94 -> 103).  There
// the scan also pays from a tenth of the grid on (two prompts of 2133 and 1066 tokens, 32 heads on
// 8: 86 -> 65 us): 0.94 to 1.47, in the mean 1.07 (19 of these 565 batches below 0.97); elsewhere 0.92 to 1.31, in
// the mean 1.02, a seventh of them below 0.97.
//   How much of the grid the scan removes is counted in blocks of whole heads also where the columns are dealt flat: items are
// up to eight times as long there, and the two blocks a request by which the rows' bound is too large hide what
// tells uneven batches (10 pieces of up to 1944 tokens behind up to 7400, 14 heads on 2: 405 -> 315 us).
static inline long long sw_prefill_blocks_by_work(const SwPrefillArgs &a, int cols, int *compact)
{
    const int q_block = 32 * a.qw;
    const long long per_item = (long long)a.n_kvh * sw_prefill_parts(a, cols);
    const long long by_rows = a.n_tokens / q_block + 2LL * a.n_req;
    const long long rows = a.n_tokens / (a.n_req > 0 ? a.n_req : 1);        // of a request, the host's estimate
    const bool by_work = a.n_req > 1 && a.n_req <= 64 && rows * (256 / 32) >= 3 * by_rows * per_item;
    int unit = q_block;
    if (a.hp == 0) {
        int heads = a.group < cols ? a.group : cols;
        while (a.group % heads) --heads;
        unit = 32 * (cols / heads);
    }
    const long long grid = (long long)a.n_req * ((a.max_q + unit - 1) / unit), left = a.n_tokens / unit + 2LL * a.n_req;
    const bool early = by_work ? left * 10 < grid * 9 : left * 4 < grid * 3 && a.n_req <= 4096;
    const long long items = sw_prefill_items(a, q_block, early, compact);
    if (by_work && *compact) *compact = kScanByWork;
    return items * per_item;
}
// Whether the key-split prompt kernel takes the scan of the lengths already where it removes 15 % of the grid.
// Without the scan the (query block, key/value head) pairs are numbered block by block, late blocks first, over
// all requests, and the blocks that a shorter request does not have are empty workgroups.  Where a
// request's pairs reach all eight XCDs these cost little (three prompts of about 500 tokens, 8 heads on one:
// 9.6 us against 10.5 with the scan); where they miss some XCDs, the others alone get the missing work.  The scan
// mends that but takes the requests one after the other, which costs a batch of many requests more than
// the empty ones do.  Time without it over time with it, 1300 batches of 1 to 24 heads: two to four requests
// whose heads come in groups, on a grid beyond the chip's 512 places that shrinks by 15 % or more, 0.96 to 1.47,
// in the mean 1.16 (3200 and 1600 tokens, 8 heads on one: 57.6 -> 44.9 us); 10 to 15 % of the grid 0.89 to 1.2, less
// 0.9 to 1.25; one head on one 0.87 to 1.26 at up to four requests; five and more requests 0.72 to 1.52, in
// the mean 0.96 (18 of about 960 tokens, one head: 14.3 -> 20.0); grids that the chip holds at once 0.78 to 1.2,
// in the mean 0.96.
static inline bool sw_split_scans_early(const SwPrefillArgs &a)
{
    const long long by_shape = (long long)a.n_req * a.n_qblocks;
    const long long by_rows = a.n_tokens / 32 + 2LL * a.n_req;          // (blocks of 32 query tokens)
    if (a.n_req < 2 || a.n_req > 4 || a.group < 2) return false;
    if (by_rows * 20 >= by_shape * 17 || by_shape * a.n_qh <= 512) return false;
    const long long stride = (long long)a.n_req * a.n_kvh;
    int common = 8;
    while (stride % common) common /= 2;
    return common > a.n_kvh;                                            // a request's pairs miss some XCDs
}
bool       sw_prefill_mfma_supported(const SwPrefillArgs &a);
void       sw_prefill_shape(int group, int *hp, int *qw);
// merge != null (mixed batches, four waves): extra workgroups merge the token-phase chunks that the
// partial kernel launched before on the same stream left in the workspace (instead of the combine kernel)
hipError_t sw_launch_prefill_split(const SwPrefillArgs &a, int waves, hipStream_t stream, const SwLaunchEvents *ev,
                                   const SwArgs *merge = nullptr);
hipError_t sw_launch_prefill_mfma(const SwPrefillArgs &a, hipStream_t stream, const SwLaunchEvents *ev);
// the shared-tile form with the key range in two halves (columns dealt flat: hp 0, group * qw a multiple of 4)
hipError_t sw_launch_prefill_halves(const SwPrefillArgs &a, hipStream_t stream, const SwLaunchEvents *ev);
int        sw_kv_copy_rows_per_group();
hipError_t sw_launch_kv_copy(const SwHandoffArgs &a, bool to_dense, hipStream_t stream, const SwLaunchEvents *ev);
hipError_t sw_launch_kv_span_plan(const int32_t *block_table, const int32_t *seq_lens,
                                  int32_t *span_first, int32_t *span_blocks, int32_t *n_spans,
                                  int n_req, int block_shift, int max_blocks, int n_blocks,
                                  hipStream_t stream);
hipError_t sw_launch_kv_store(const SwPrefillArgs &a, const uint16_t *k_rows, const uint16_t *v_rows,
                              uint16_t *k_out, uint16_t *v_out, hipStream_t stream, const SwLaunchEvents *ev);
hipError_t sw_launch_stream_read(const void *src, unsigned long long n_bytes, unsigned *sink,
                                 int workgroups, hipStream_t stream, const SwLaunchEvents *ev);
hipError_t sw_launch_advance_lens(int32_t *seq_lens, int n_req, int max_len, hipStream_t stream);

// Granularity the chunk length must be a multiple of (all kernels).
constexpr int SW_CHUNK_QUANTUM = 64;

template <typename... KArgs, typename... Args>
static inline hipError_t sw_launch(void (*kernel)(KArgs...), dim3 grid, dim3 block, size_t lds,
                                   hipStream_t stream, const SwLaunchEvents *ev, Args... args)
{
    if (ev && ev->start && ev->stop) {
        hipExtLaunchKernelGGL(kernel, grid, block, lds, stream, ev->start, ev->stop, 0, args...);
    } else {
        hipLaunchKernelGGL(kernel, grid, block, lds, stream, args...);
    }
    return hipGetLastError();
}
