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
// What goes past the caches (the non-temporal hint): unpack's loads, which are the last use of the staging buffer; unpack's stores, unless the
// move is small enough for the next kernel to find the pages in the last-level cache; pack's loads of a large move.  Pack's stores do not.
// What a hint gains depends on what the caches hold; us on one GPU, MB of K and V pages, nothing streamed / everything / this:
//   pack, caches full of what was read last        67: 26.6 / 27.6 / 26.6   101: 36.8 / 39.6 / 37.0   302: 99.7 / 107.0 / 91.4   604: 211 / 208 / 185
//   pack of pages just written                     101: 33.7 / 33.4 / 34.0   302: 112.6 / 105.7 / 94.3   604: 243 / 216 / 211
//   unpack of a buffer just received, otherwise the same   67: 24.3 / 24.4 / 24.6   101: 34.2 / 33.9 / 34.3   134: 48.7 / 43.4 / 43.8
//   and the pages read after that                  67: 56.0 / 61.6 / 56.0   101: 70.0 / 78.9 / 70.1   134: 89.8 / 95.8 / 83.8
//   pack and unpack in turn on three sets          34: 27.3 / 28 / 23.2   67: 49.8 / 53 / 48.6   101: 79.3 / 75 / 71.1   134: 107.4 / 99 / 93.3
//                                                  201: 159 / 146.2 / 124.9   302: 237 / 218.8 / 189.2 (6.4 TB/s read + write)   604: 469 / 437.5 / 420.7
// It costs where the caches are full of lines to be written back: pack after a fill of 768 MB, everything streamed and this, 302: 107.5 and 116.6,
// 604: 208.9 and 223.9, and so packs in turn, which leave their own staging buffers (302: 103.3 and 109.5); and where the same buffer is unpacked again
// out of the caches (34: nothing streamed 11.7, this 13.8).  A copy to another buffer between the two, in place of a transport, takes away what the unpack
// gained (302: 319 and 326 for the three, 201: 206 and 234; 134: 168 with nothing streamed, 136); a transport to another GPU was not measured.
// The lines: pack's loads in turn, streamed or not, 45.4 and 43.7 at 64 MB, 66.5 and 66.7 at 96.  Unpack's stores streamed from 40 MB on were a gain in
// turn (67: 44.0 and 48.6, 134: 85.0 and 93.3) and a loss on pages that nothing had touched (67: 28.3 and 26.6, 101: 41.8 and 36.9), and leave the pages
// to be fetched again; above 128 MB they are as the move in turn has them (302: 189 and 212; on untouched pages 117 and 92).
#include "emm_internal.h"

#include <type_traits>

namespace emm {

namespace {

constexpr int THREADS = 256;
constexpr unsigned ADLER_MOD = 65521;
constexpr long long STREAM_LOADS = 80ll << 20, STREAM_STORES = 128ll << 20;          // pack's loads, unpack's stores: of K and V pages

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
template <bool UNPACK, bool LOADS, bool STORES>
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
                w[u] = load16<LOADS>(UNPACK ? sp + off : pool);
            }
        }
#pragma unroll
        for (int u = 0; u < BATCH; ++u) {
            const long long off = off0 + (long long)u * THREADS * 16;
            if (off < n) {
                unsigned char* pool = off < page_bytes ? kp + off : vp + (off - page_bytes);
                store16<STORES>(UNPACK ? pool : sp + off, w[u]);
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
    auto go = [&](auto unpack_c, auto loads_c, auto stores_c) {
        hipLaunchKernelGGL((kv_pages_kernel<decltype(unpack_c)::value, decltype(loads_c)::value, decltype(stores_c)::value>), dim3((unsigned)n),
                           dim3(THREADS), 0, stream, (unsigned char*)k_cache, (unsigned char*)v_cache, (unsigned char*)staging, page_ids,
                           num_pages, page_bytes, checksums, expected, mismatches);
    };
    const std::true_type streamed;
    const std::false_type cached;
    const long long bytes = 2 * page_bytes * n;
    if (unpack && bytes > STREAM_STORES) go(std::true_type{}, streamed, streamed);
    else if (unpack) go(std::true_type{}, streamed, cached);
    else if (bytes > STREAM_LOADS) go(std::false_type{}, streamed, cached);
    else go(std::false_type{}, cached, cached);
    return hipGetLastError();
}

}  // namespace emm
