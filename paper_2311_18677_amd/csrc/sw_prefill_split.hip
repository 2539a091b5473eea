// Prompt-phase (causal) attention, key-split form for short and medium prompts
// (gfx950, wave64), head_dim 128.
//
// A prompt batch on a prompt machine is capped at about two thousand tokens
// (paper section 4.2), which at one GPU's share of the heads is only a few
// hundred (query block, head) pairs: with one wave per pair the chip is mostly
// idle and every wave walks a long chain of key tiles.  Here the waves of a
// workgroup share ONE pair -- 32 query positions of one head -- and split its
// key range instead: wave w takes tiles w, w + W, ...  Each wave stages its own
// K and V tiles global->LDS and waits on its own counters (no barrier in the
// loop), exactly like the token-phase kernel; at the end the waves' partial
// (maximum, sum, accumulator) triples are merged through LDS and the rows are
// normalised and stored.  The first product of a wave's next tile runs beside the softmax of
// the current one: a tile's chain of product, maximum, exponentials and product is what bounds a
// wave (two waves per SIMD issue in turn, and the chip is far from its matrix and memory rates).
// Measured against one tile at a time, with 8 query heads over one key/value head: prompts of 548 and
// 1500 tokens 16.3 -> 15.5 us, one of 1024 tokens 11.1 -> 10.5; 2 heads over one, 4096 tokens, 28.9
// -> 27.3 (22.0 with eight waves, which serve few and long chains: split_waves_for in
// sw_api.hip).  (The 32x32x16 product gains more on short chains, but loses 3 to 6 % from
// 4096 tokens on.)  The workgroup's code is in sw_prefill_split_body.h.
#include "sw_prefill_split_body.h"
#include "sw_merge.h"

namespace {

using namespace sw_split;

// MERGE (mixed batches): the workgroups from number n_prompt on do not belong to the prompt
// phase at all.  They merge the chunks of the token-phase requests that the partial kernel
// of the same call, launched just before on the same stream, has left in the workspace
// (arguments d) -- the work of the combine kernel, riding along here so that the call is
// two launches instead of three.  Eight output rows per workgroup, one thread per four dims.
template <int WAVES, bool PAGED, bool MERGE>
__global__ __launch_bounds__(64 * WAVES, WAVES >= 4 ? 8 / WAVES : 2)
void sw_prefill_split_kernel(SwPrefillArgs a, SwArgs d, unsigned n_prompt)
{
    if (MERGE && blockIdx.x >= n_prompt) {
        const long long rh = (long long)(blockIdx.x - n_prompt) * (64 * WAVES / (kD / 4)) + (threadIdx.x / (kD / 4));
        if (rh < (long long)d.n_req * d.n_qh) sw_merge::merge_row_serial<kD>(d, (int)rh, (int)(threadIdx.x % (kD / 4)));
        return;
    }
    __shared__ SplitLds<WAVES> sm;
    prompt_workgroup<WAVES, PAGED>(a, blockIdx.x, sm);
}

}  // namespace

hipError_t sw_launch_prefill_split(const SwPrefillArgs &a_in, int waves, hipStream_t stream, const SwLaunchEvents *ev,
                                   const SwArgs *merge)
{
    if (a_in.head_dim != kD) return hipErrorNotSupported;
    SwPrefillArgs a = a_in;
    int compact;
    const long long pairs = sw_prefill_items(a, kQPerWave, sw_split_scans_early(a), &compact) * a.n_kvh;
    const long long n_prompt = (pairs + 7) / 8 * 8 * a.group;      // see the kernel's numbering of the heads
    if (n_prompt <= 0 || n_prompt > 0x7fffffffLL) return hipErrorInvalidValue;
    a.compact = compact;
    if (merge) {
        // the token-phase rows to merge: 256 threads = 8 rows of 32 four-dim pieces
        if (waves != 4 || merge->head_dim != kD) return hipErrorInvalidValue;
        const long long rows = (long long)merge->n_req * merge->n_qh;
        const long long blocks = n_prompt + (rows + 7) / 8;
        if (blocks > 0x7fffffffLL) return hipErrorInvalidValue;
        const dim3 grid((unsigned)blocks);
        return a.block_table
            ? sw_launch(sw_prefill_split_kernel<4, true, true>, grid, dim3(256), 0, stream, ev, a, *merge, (unsigned)n_prompt)
            : sw_launch(sw_prefill_split_kernel<4, false, true>, grid, dim3(256), 0, stream, ev, a, *merge, (unsigned)n_prompt);
    }
    const dim3 grid((unsigned)n_prompt);
    const SwArgs none = {};
    const unsigned np = (unsigned)n_prompt;
    if (a.block_table) {
        if (waves == 8) return sw_launch(sw_prefill_split_kernel<8, true, false>, grid, dim3(512), 0, stream, ev, a, none, np);
        if (waves == 4) return sw_launch(sw_prefill_split_kernel<4, true, false>, grid, dim3(256), 0, stream, ev, a, none, np);
        if (waves == 2) return sw_launch(sw_prefill_split_kernel<2, true, false>, grid, dim3(128), 0, stream, ev, a, none, np);
        return hipErrorInvalidValue;
    }
    if (waves == 8) return sw_launch(sw_prefill_split_kernel<8, false, false>, grid, dim3(512), 0, stream, ev, a, none, np);
    if (waves == 4) return sw_launch(sw_prefill_split_kernel<4, false, false>, grid, dim3(256), 0, stream, ev, a, none, np);
    if (waves == 2) return sw_launch(sw_prefill_split_kernel<2, false, false>, grid, dim3(128), 0, stream, ev, a, none, np);
    return hipErrorInvalidValue;
}
