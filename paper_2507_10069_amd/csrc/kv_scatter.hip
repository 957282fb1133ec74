// KV scatter: the new tokens' K/V rows go to the pool slots that follow each request's cached
// prefix (Section 2.2 of the paper: prefill yields the KV cache of every input token; the copy
// must be exact in the sense of Appendix B.5).
//
// Pure data movement: 4 * T * Hkv * d * elt bytes (read K,V + write K,V), HBM bound on a large batch and bound by its
// chain of memory round trips on a small one.  One wave moves one token: the lanes move the token's K row and V row
// (all KV heads, Hkv * d * elt bytes each) in 16-byte chunks.  The packed source [T][Hkv][d] is read fully
// coalesced; a (token, head) row of d*elt bytes lands contiguously in its page.  The chain is three round trips long:
// kernel arguments; the batch's offsets and lengths (64 of each at once, one per lane, the token's request found by a
// ballot) together with the rows to be moved, whose place does not depend on them; the page id.
// Measured against a binary search by scalar loads with the rows asked for last: 5.1 -> 3.9 us for 36 tokens, 48.4 ->
// 46.2 us (6.4 TB/s) for 36336 tokens of 8 heads; a kernel that does nothing takes 1.7 us.  (The kernel arguments were three round
// trips of their own until all were asked for at once: 5.2 -> 4.0 us behind a call that keeps the chip busy.)
#include "emm_internal.h"

namespace emm {

namespace {

constexpr int WAVES = 4;                                 // tokens per workgroup

// row_shift: a (token, head) row is 1 << row_shift chunks of 16 bytes (head_dim * element size / 16)
__global__ __launch_bounds__(64 * WAVES) void kv_scatter_kernel(BatchView b, const uint4* __restrict__ k_new,
                                                                const uint4* __restrict__ v_new,
                                                                uint4* __restrict__ k_cache, uint4* __restrict__ v_cache,
                                                                int row_shift)
{
    const int t = blockIdx.x * WAVES + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // packed token, wave-uniform
    // every argument in one round trip: the compiler asks for some where they are first used.  (Behind the asm it takes scalar loads only
    // from the constant address space.)
    typedef const __attribute__((address_space(4))) int32_t* scalar_ints;
    const scalar_ints cu_s = (scalar_ints)(uintptr_t)b.cu_new_lens, table_s = (scalar_ints)(uintptr_t)b.page_table;
    asm volatile("" ::"s"(k_new), "s"(v_new), "s"(k_cache), "s"(v_cache), "s"(b.cu_new_lens), "s"(b.prefix_lens), "s"(b.page_table), "s"(row_shift),
                 "s"(b.num_reqs), "s"(b.num_kv_heads), "s"(b.page_shift), "s"(b.max_pages));
    if (t >= b.total_new_tokens) return;
    const int lane = threadIdx.x & 63;

    // the token's rows, asked for before it is known where they go
    const int token_chunks = b.num_kv_heads << row_shift;                 // chunks of the token's K (or V) row, all heads
    const long long src = (long long)t * token_chunks;
    constexpr int HELD = 2;                                               // chunks per lane and pool held in registers (8 heads of 128 bf16)
    uint4 k_held[HELD], v_held[HELD];
#pragma unroll
    for (int u = 0; u < HELD; ++u) {
        const int c = min(lane + 64 * u, token_chunks - 1);               // past the row: its last chunk, which is not stored
        k_held[u] = k_new[src + c];
        v_held[u] = v_new[src + c];
    }

    // request that owns packed token t: last r with cu[r] <= t, among 64 that the lanes look at together
    int lo = 0, hi = b.num_reqs;
    while (hi - lo > 64) {
        const int mid = (lo + hi) >> 1;
        if (cu_s[mid] <= t) lo = mid; else hi = mid;
    }
    const int mine = min(lo + lane, hi - 1);
    const int cu_mine = b.cu_new_lens[mine], prefix_mine = b.prefix_lens[mine];
    const unsigned long long not_after = __builtin_amdgcn_ballot_w64(lo + lane < hi && cu_mine <= t);
    const int at = not_after == 0 ? 0 : 63 - __builtin_clzll(not_after);
    const int r = lo + at;
    const long long pos64 = (long long)__builtin_amdgcn_readlane(prefix_mine, at) + (t - __builtin_amdgcn_readlane(cu_mine, at));
    // inconsistent lengths or a corrupt table: drop the write, never stray
    const int pos = (int)min(max(pos64, 0ll), (long long)b.max_pages * b.page_size - 1);
    const int page = table_s[(long long)r * b.max_pages + (pos >> (4 + b.page_shift))];
    // (the rows are waited for here, with the page id: left to itself the compiler asks for them where they are stored)
#pragma unroll
    for (int u = 0; u < HELD; ++u)
        asm volatile("" ::"v"(k_held[u].x), "v"(k_held[u].y), "v"(k_held[u].z), "v"(k_held[u].w), "v"(v_held[u].x), "v"(v_held[u].y),
                     "v"(v_held[u].z), "v"(v_held[u].w));
    if (pos64 != pos || page < 0 || page >= b.num_pages) return;

    // chunk c of the token is chunk c % row of head c / row; heads are page_size rows apart in the pool
    const long long dst = ((long long)page * b.num_kv_heads * b.page_size + (pos & (b.page_size - 1))) << row_shift;
    const int head_stride = (b.page_size - 1) << row_shift;               // extra chunks between consecutive heads
    auto place = [&](int c) -> long long { return dst + c + (long long)(c >> row_shift) * head_stride; };
#pragma unroll
    for (int u = 0; u < HELD; ++u)
        if (lane + 64 * u < token_chunks) {
            k_cache[place(lane + 64 * u)] = k_held[u];
            v_cache[place(lane + 64 * u)] = v_held[u];
        }
    for (int c = lane + 64 * HELD; c < token_chunks; c += 64) {
        k_cache[place(c)] = k_new[src + c];
        v_cache[place(c)] = v_new[src + c];
    }
}

}  // namespace

hipError_t launch_kv_scatter(const BatchView& b, const void* k_new, const void* v_new, void* k_cache,
                             void* v_cache, int elt_bytes, hipStream_t stream)
{
    if (b.total_new_tokens == 0 || b.num_reqs == 0) return hipSuccess;
    const int chunks_per_row = b.head_dim * elt_bytes / 16;              // 8, 16 or 32: a power of two
    int row_shift = 0;
    while ((1 << row_shift) < chunks_per_row) ++row_shift;
    if ((1 << row_shift) != chunks_per_row) return hipErrorInvalidValue;
    const long long blocks = ((long long)b.total_new_tokens + WAVES - 1) / WAVES;
    hipLaunchKernelGGL(kv_scatter_kernel, dim3((unsigned)blocks), dim3(64 * WAVES), 0, stream, b,
                       (const uint4*)k_new, (const uint4*)v_new, (uint4*)k_cache, (uint4*)v_cache, row_shift);
    return hipGetLastError();
}

}  // namespace emm
