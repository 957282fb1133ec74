// Merging two attention results of the same query rows over DISJOINT key sets (bf16, head_dim 128), for gfx950.
//
// Prefill with shared prefixes (Section 3.3 of the paper: requests repeat system prompts, images and videos, so
// several requests of a prefill batch hold the same physical pages at the head of their page tables) is done
// in two attention passes: one over the shared keys, with the query rows of all the requests of a sharing group
// packed into common row tiles, and one over each request's own remaining keys.  Softmax attention over a union
// of key sets is the convex combination of the parts' results with weights exp(lse_part - lse_all), which this
// kernel forms, row by row:
//     out = (e^{lse_a} out_a + e^{lse_b} out_b) / (e^{lse_a} + e^{lse_b}),   lse = log(e^{lse_a} + e^{lse_b}).
// Rows of requests that are in no sharing group have no first part and stay as they are.  This kernel is for own passes whose units may be cut along the
// keys (attn_bf16_d128_takes_parts); the others merge in the attention kernel.
//
// Pure data movement, HBM bound: per row two 256-byte reads, one 256-byte write and three floats.  A row is done
// by 16 lanes (8 channels, 16 bytes each), a workgroup does 16 rows.
#include "emm_internal.h"

namespace emm {

namespace {

constexpr int THREADS = 256;
constexpr int D = 128;
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

// the request that packed token t belongs to: the last r with cu_new_lens[r] <= t among requests that have tokens
// (what the array holds is forced into range wherever an index depends on it).  Among up to 64 requests the lanes look at one
// offset each and a ballot for each of the wave's four rows counts them (all lanes must be there): one round trip
// instead of one per search step.
__device__ inline int request_of_token(const BatchView& b, int t)
{
    if (b.num_reqs <= 64) {
        const int lane = threadIdx.x & 63;
        const int cu = b.cu_new_lens[min(lane, b.num_reqs - 1)];
        int r = 0;
#pragma unroll
        for (int k = 0; k < 4; ++k) {                        // the row of lanes 16 k .. 16 k + 15
            const int tk = __builtin_amdgcn_readlane(t, 16 * k);
            const int n = __builtin_popcountll(__builtin_amdgcn_ballot_w64(lane < b.num_reqs && cu <= tk));
            if ((lane >> 4) == k) r = max(n - 1, 0);
        }
        return r;
    }
    int lo = 0, hi = b.num_reqs - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (b.cu_new_lens[mid] <= t) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

__global__ __launch_bounds__(THREADS) void attn_merge_parts_kernel(BatchView b, const int32_t* __restrict__ req_shared_len,
                                                                   const __bf16* __restrict__ out_shared,
                                                                   const float* __restrict__ lse_shared,
                                                                   const float* __restrict__ lse_own, __bf16* __restrict__ out,
                                                                   float* __restrict__ lse, Divisor by_heads)
{
    // (every argument in one round trip: the compiler asks for some where they are first used)
    asm volatile("" ::"s"(req_shared_len), "s"(out_shared), "s"(lse_shared), "s"(lse_own), "s"(out), "s"(lse), "s"(b.cu_new_lens), "s"(b.num_reqs));
    const long long n_rows = (long long)b.total_new_tokens * b.num_q_heads;
    const long long my_row = (long long)blockIdx.x * (THREADS / 16) + (threadIdx.x >> 4);
    const long long row = my_row < n_rows ? my_row : n_rows - 1;          // every lane stays for the ballots: left below
    const int t = n_rows <= 0x7fffffff ? by_heads.quotient((int)row) : (int)(row / b.num_q_heads);   // (a 64-bit division is 150 instructions)
    const float lo = lse_own[row];
    const int r = request_of_token(b, t);
    float merged = lo;
    // The parts are read for members only: a batch may hold a group of short questions beside long prompts that are in no group.
    // (Asked for in every row, before it is known, they take no time off a batch of members: 91.5 us both ways for 64 short questions on
    // 8 videos; beside a group of 16, a prompt of 4096 tokens 202 -> 197 us, four of them 556 -> 534.)
    if (req_shared_len[r] > 0 && my_row < n_rows) {
        const long long at = row * D + (threadIdx.x & 15) * 8;
        const float ls = lse_shared[row];
        const bf16x8 a = *(const bf16x8*)(out_shared + at);
        const bf16x8 c = *(const bf16x8*)(out + at);
        asm volatile("" ::"v"(ls), "v"(a), "v"(c));          // all three at once (left to itself the compiler asks for two when it has looked at ls)
        const float m = fmaxf(ls, lo);
        if (m > -INFINITY) {
            const float ws = __expf(ls - m), wo = __expf(lo - m);
            const float inv = 1.f / (ws + wo);
            bf16x8 o;
#pragma unroll
            for (int i = 0; i < 8; ++i) o[i] = (__bf16)merged_channel((float)a[i], ws, (float)c[i], wo, inv);
            *(bf16x8*)(out + at) = o;
            merged = m + __logf(ws + wo);
        }
    }
    if (lse != nullptr && (threadIdx.x & 15) == 0 && my_row < n_rows) lse[row] = merged;
}

}  // namespace

hipError_t launch_attn_merge_parts(const BatchView& b, const int32_t* req_shared_len, const void* out_shared,
                                   const float* lse_shared, const float* lse_own, void* out, float* lse, hipStream_t stream)
{
    const long long n_rows = (long long)b.total_new_tokens * b.num_q_heads;
    if (n_rows == 0 || b.num_reqs == 0) return hipSuccess;
    const long long grid = (n_rows + THREADS / 16 - 1) / (THREADS / 16);
    if (grid > 0x7fffffff) return hipErrorInvalidValue;
    hipLaunchKernelGGL(attn_merge_parts_kernel, dim3((unsigned)grid), dim3(THREADS), 0, stream, b, req_shared_len,
                       (const __bf16*)out_shared, lse_shared, lse_own, (__bf16*)out, lse, divisor_of(b.num_q_heads));
    return hipGetLastError();
}

}  // namespace emm
