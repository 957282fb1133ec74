// KV page migration primitive, the part one GPU can show (Appendix B.5 of the paper: on scaling, a request's
// KV cache moves to another instance by exact copy, verified with checksums).  pack gathers a request's pages
// from the two pools into a contiguous staging buffer -- what would be handed to the transport -- and unpack
// scatters a received staging buffer into whatever free pages the destination pool has; both take the
// Adler-32 (RFC 1950) of every page as it passes, so the two sides can be compared.
//
// Pure data movement, HBM bound: 2 * page_bytes read and written per page.  One workgroup per page; a lane
// moves 16 bytes at a time, fully coalesced on both sides (a page is contiguous in its pool and in the
// staging buffer).  The checksum rides along on the integer dot-product instruction: for the four bytes of a
// word at offset i of the n-byte page, sum(d) and sum(k * d[k]) (v_dot4_u32_u8 with constants), from which
//   A = 1 + sum over the page of d            B = n + sum over the page of (n - position) * d,  both mod 65521.
//
// A large move (STREAM) goes past the caches, loads and stores with the non-temporal hint: neither side is read again
// here, and lines that wait to be written back hold up the reads.  8 requests of 18432 tokens (302 MB each way, pack +
// unpack) 239 -> 219 us = 5.5 TB/s read + write, where the runtime's own copy of 2 GiB reaches 4.9; loads alone 203 of 227, stores
// alone 220.  What the last-level cache holds is left there, where the transport or the next kernel finds it: the line is drawn
// where pages and staging together pass its 256 MiB (a staging buffer unpacked after it was packed: 134 MB of pages, 268 MB
// in all, 94 us and 99 with the hint; 302 in all 114 and 110; 134 in all 42 and 49; 67 in all 23 and 25.  Pages and buffers
// that nobody had touched before: 108 and 100, 121 and 111, 50 and 51, 31 and 28).
#include "emm_internal.h"

#include <type_traits>

namespace emm {

namespace {

constexpr int THREADS = 256;
constexpr unsigned ADLER_MOD = 65521;
constexpr long long STREAM_BYTES = 256ll << 20;

// wave sum of a 64-bit value
__device__ inline unsigned long long wave_sum_u64(unsigned long long x)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const unsigned lo = __shfl_xor((unsigned)x, o, 64), hi = __shfl_xor((unsigned)(x >> 32), o, 64);
        x += ((unsigned long long)hi << 32) | lo;
    }
    return x;
}

typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
template <bool STREAM>
__device__ inline u32x4 load16(const unsigned char* p)
{
    if constexpr (STREAM) return __builtin_nontemporal_load((const u32x4*)p);
    else return *(const u32x4*)p;
}
template <bool STREAM>
__device__ inline void store16(unsigned char* p, u32x4 w)
{
    if constexpr (STREAM) __builtin_nontemporal_store(w, (u32x4*)p);
    else *(u32x4*)p = w;
}

// UNPACK = false: pools -> staging; true: staging -> pools.  page_bytes: one page of ONE pool.
template <bool UNPACK, bool STREAM>
__global__ __launch_bounds__(THREADS) void kv_pages_kernel(unsigned char* __restrict__ k_cache,
                                                           unsigned char* __restrict__ v_cache,
                                                           unsigned char* __restrict__ staging,
                                                           const int32_t* __restrict__ page_ids, int num_pages,
                                                           long long page_bytes, uint32_t* __restrict__ checksums,
                                                           const uint32_t* __restrict__ expected,
                                                           uint32_t* __restrict__ mismatches)
{
    __shared__ unsigned long long part[2][THREADS / 64];
    const int p = blockIdx.x;
    const int page = min(max(page_ids[p], 0), num_pages - 1);             // never leaves the pool
    const long long n = 2 * page_bytes;                                   // bytes of the page in the staging buffer
    unsigned char* kp = k_cache + (long long)page * page_bytes;
    unsigned char* vp = v_cache + (long long)page * page_bytes;
    unsigned char* sp = staging + (long long)p * n;
    unsigned long long sum_d = 0, sum_w = 0;                              // sum of bytes, sum of (n - position) * byte
    constexpr int BATCH = 8;                                              // loads in flight per lane
    for (long long off0 = (long long)threadIdx.x * 16; off0 < n; off0 += (long long)BATCH * THREADS * 16) {
        u32x4 w[BATCH];
#pragma unroll
        for (int u = 0; u < BATCH; ++u) {
            const long long off = off0 + (long long)u * THREADS * 16;
            if (off < n) {
                const unsigned char* pool = off < page_bytes ? kp + off : vp + (off - page_bytes);
                w[u] = load16<STREAM>(UNPACK ? sp + off : pool);
            }
        }
#pragma unroll
        for (int u = 0; u < BATCH; ++u) {
            const long long off = off0 + (long long)u * THREADS * 16;
            if (off < n) {
                unsigned char* pool = off < page_bytes ? kp + off : vp + (off - page_bytes);
                store16<STREAM>(UNPACK ? pool : sp + off, w[u]);
                const unsigned words[4] = {w[u][0], w[u][1], w[u][2], w[u][3]};
                unsigned s_all = 0;                                       // of the 16 bytes: at most 4080
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const unsigned s = __builtin_amdgcn_udot4(words[j], 0x01010101u, 0u, false);   // d0 + d1 + d2 + d3
                    const unsigned t = __builtin_amdgcn_udot4(words[j], 0x03020100u, 0u, false);   // d1 + 2 d2 + 3 d3
                    s_all += s;
                    // one word's term fits 32 bits ((n - position) <= 2^21, s <= 1020: below 2^31.1), the four of a
                    // chunk together need not (pages above 512 KiB), so each goes into the 64-bit sum by itself
                    sum_w += (unsigned)(n - off - 4 * j) * s - t;
                }
                sum_d += s_all;
            }
        }
    }
    sum_d = wave_sum_u64(sum_d);
    sum_w = wave_sum_u64(sum_w);
    const int wave = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) {
        part[0][wave] = sum_d;
        part[1][wave] = sum_w;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned long long d = 0, w = 0;
        for (int i = 0; i < THREADS / 64; ++i) {
            d += part[0][i];
            w += part[1][i];
        }
        const unsigned a = (unsigned)((1 + d) % ADLER_MOD), b = (unsigned)(((unsigned long long)n + w) % ADLER_MOD);
        const uint32_t sum = (b << 16) | a;
        if (checksums != nullptr) checksums[p] = sum;
        if (UNPACK && expected != nullptr && mismatches != nullptr && expected[p] != sum) atomicAdd(mismatches, 1u);
    }
}

}  // namespace

hipError_t launch_kv_pages(bool unpack, void* k_cache, void* v_cache, void* staging, const int32_t* page_ids, int n,
                           int num_pages, long long page_bytes, uint32_t* checksums, const uint32_t* expected,
                           uint32_t* mismatches, hipStream_t stream)
{
    if (n == 0) return hipSuccess;
    auto go = [&](auto unpack_c, auto stream_c) {
        hipLaunchKernelGGL((kv_pages_kernel<decltype(unpack_c)::value, decltype(stream_c)::value>), dim3((unsigned)n), dim3(THREADS), 0, stream,
                           (unsigned char*)k_cache, (unsigned char*)v_cache, (unsigned char*)staging, page_ids, num_pages, page_bytes,
                           checksums, expected, mismatches);
    };
    const bool streamed = 4 * page_bytes * n > STREAM_BYTES;            // K and V pages and their staging
    if (unpack && streamed) go(std::true_type{}, std::true_type{});
    else if (unpack) go(std::true_type{}, std::false_type{});
    else if (streamed) go(std::false_type{}, std::true_type{});
    else go(std::false_type{}, std::false_type{});
    return hipGetLastError();
}

}  // namespace emm
