// fp32 attention over the paged pool on the fp32 matrix instruction (head_dim 64 or 128), for gfx950.
//
// This is the fp32 path of the library (small correctness configurations and fp32 models of small heads).
// It follows the same definition as the bf16 kernels -- causal over absolute positions for the prefix-cached
// prefill (Section 3.3 / Appendix B.7 of the paper), unmasked for cross-attention (Section 2.1).
//
// What bounds it: such calls are small (a few hundred rows, up to a few thousand keys), so it is the chain of
// memory and instruction latencies from the launch to the last store, not a rate.  The work is therefore cut
// finely: a workgroup takes 16 query rows of one (request, KV head) -- row j * G + g is head g of new token j, so
// the heads that share a KV head are neighbours -- and its waves, 8 of them in a small call, take the keys in turn, 16 at
// a time (16 keys lie in one page, so a chunk's K and V are one contiguous run each and its page a scalar).  Every wave
// keeps its own online softmax; the results are combined through LDS.  There is no LDS in the loop: K and
// V go straight to registers, the next chunk's K and this chunk's V while this chunk's scores are computed.
//
// v_mfma_f32_16x16x4_f32 takes one A and one B value per lane (row or column lane % 16, k = lane / 16 =: g) and
// returns column lane % 16, rows 4 g .. 4 g + 3.  The sums over k may run in any order, so the operands are laid
// out for the loads:
//   S^T = K Q^T   lane (key i, g) reads 16-byte pieces 16 j + 4 g of row i, j = 0, 1, ...; Q likewise.  A lane then
//                 holds the scores of row lane % 16 with keys 4 g .. 4 g + 3: the row maximum is two lane exchanges.
//   O^T += V^T P^T  step v takes key 4 g + v from lane group g, which is where that weight already is; as the A
//                 operand lane i stands for channels 4 i .. 4 i + 3 of the four products of a 64-channel block, so V
//                 rows are read whole, 16 bytes per lane, and a lane ends up with 16 consecutive channels of its row.
// Measured, scatter and attention per step, against one wave per row with lanes owning keys (no matrix instruction):
// 4 heads on 1 KV head of 64, 256 cached + 64 new tokens 38.8 -> 9.5 us (11.1 before the loads overlapped, the lengths came in one
// round trip and the channels were split: see SPLIT_WORKGROUPS); the same
// heads, 4 x (1024 + 256) tokens 254 -> 26 us; 8 heads on 2 of 128, 4096 new tokens 5.59 -> 0.44 ms (78 TFLOP/s of the
// 154 that a large fp32 matrix product reaches).  Relative error against 64 bits 4.2e-7 -> 3.0e-7 on the first.
#include "emm_internal.h"

#include <type_traits>

namespace emm {

namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int ROWS = 16;                              // query rows per workgroup
constexpr int KEYS = 16;                              // keys per chunk; a page holds a whole number of chunks

// max or sum of a value over the four lanes that share lane % 16
__device__ inline float group_max(float x)
{
    uint32_t u = __float_as_uint(x);
    const auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
    u = __float_as_uint(fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1])));
    const auto t = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    return fmaxf(__uint_as_float(t[0]), __uint_as_float(t[1]));
}
__device__ inline float group_sum(float x)
{
    uint32_t u = __float_as_uint(x);
    const auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
    u = __float_as_uint(__uint_as_float(r[0]) + __uint_as_float(r[1]));
    const auto t = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    return __uint_as_float(t[0]) + __uint_as_float(t[1]);
}
__device__ inline bool is_finite(float x) { return (__float_as_uint(x) & 0x7f800000u) != 0x7f800000u; }

// First row-tile slot of request r: its ceil(rows / 16) tiles fit between this and the next request's, whatever
// cu_new_lens[r] is, so the grid needs no more than T G / 16 + B slots and no prefix sums over row tiles.
__device__ inline long long first_slot(int cu_new, int G, int r) { return (long long)max(cu_new, 0) * G / ROWS + r; }

// NW: waves per workgroup; SPLIT: workgroups that share a row tile's channels; APART: fewer workgroups fit a compute unit (see PLACES)
template <int D, int NW, int SPLIT, bool APART>
__global__ __launch_bounds__(64 * NW, 2) void attn_f32_kernel(AttnArgs a, int G, Divisor by_G, Divisor by_kv_heads)
{
    constexpr int QK = D / 16;                        // 16-byte pieces of a Q or K row per lane
    constexpr int CH = D / SPLIT;                     // channels of the output that this workgroup makes
    constexpr int NB = CH < 64 ? 1 : CH / 64;         // blocks of V
    constexpr int VE = CH / NB / 16;                  // channels of a block that a lane reads: VE l16 .. VE l16 + VE - 1
    constexpr int STRIDE = APART ? 164 : CH + 4;      // floats between rows of the LDS records: spreads the banks (APART: and takes more LDS)
    static_assert(!APART || (CH <= 160 && NW * ROWS * STRIDE * 4 > (NW == 8 ? 80 << 10 : 40 << 10)), "more than a half or a quarter of 160 KB");
    typedef float vec __attribute__((ext_vector_type(VE)));
    __shared__ __attribute__((aligned(16))) float o_s[NW][ROWS][STRIDE];
    __shared__ float m_s[NW][ROWS], l_s[NW][ROWS];
    const BatchView& b = a.b;
    const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int tile = blockIdx.x / SPLIT;
    const int ch0 = blockIdx.x % SPLIT * CH;          // first of this workgroup's channels
    const int slot = by_kv_heads.quotient(tile);
    const int kvh = tile - slot * b.num_kv_heads;

    int lo = 0, hi = b.num_reqs;                      // the request of this slot: the last one that starts at or before it
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (first_slot(b.cu_new_lens[mid], G, mid) <= slot) lo = mid; else hi = mid;
    }
    const int r = lo;
    const int pg_log2 = 4 + b.page_shift, ps = b.page_size;
    // The page of this wave's i-th chunk, wave + NW i, by a scalar load, which does not count among the loads of K and V.  (With the
    // pages in a vector register every chunk waited for all loads on their way.)
    const __attribute__((address_space(4))) int32_t* pt =
        (const __attribute__((address_space(4))) int32_t*)(uintptr_t)(b.page_table + (long long)r * b.max_pages);
    auto page_of = [&](int i) -> int { return pt[min((int)(((uint32_t)(wave + NW * i) * KEYS) >> pg_log2), b.max_pages - 1)]; };
    // all lengths in one round trip, and with it every argument that is needed further down
    const int new_len = b.new_lens[r], prefix_len = b.prefix_lens[r], cu_new = b.cu_new_lens[r];
    int page = page_of(0);                            // (an entry past the request's pages is read and not used)
    asm volatile("" ::"s"(page), "s"(new_len), "s"(prefix_len), "s"(cu_new), "s"(a.q), "s"(a.k_cache), "s"(a.v_cache), "s"(a.out), "s"(a.lse), "s"(a.causal));
    __builtin_amdgcn_sched_barrier(0);

    // (lengths forced into what the page table and the packed tensors can hold: see clamp_new_len)
    const int N = clamp_new_len(b, new_len, a.causal != 0);
    const int n_rows = N * G;
    const long long row0_wide = ((long long)slot - first_slot(cu_new, G, r)) * ROWS;
    if (row0_wide < 0 || row0_wide >= n_rows) return;                       // uniform over the workgroup
    const int row0 = (int)row0_wide;
    const int P = clamp_prefix_len(b, prefix_len, a.causal ? N : 0);
    const int kv_len = a.causal ? P + by_G.quotient(min(row0 + ROWS - 1, n_rows - 1)) + 1 : P;   // keys that some row here sees
    const int n_chunks = (kv_len + KEYS - 1) / KEYS;
    const int min_limit = a.causal ? P + by_G.quotient(row0) : P - 1;               // last key that every row here sees
    const int row = min(row0 + l16, n_rows - 1);
    const int tok = by_G.quotient(row);
    const int limit = a.causal ? P + tok : P - 1;                           // last key of this lane's row
    const long long first_row = clamp_first_row(b, cu_new, N);

    const float* __restrict__ qp = (const float*)a.q + ((first_row + tok) * b.num_q_heads + kvh * G + (row - tok * G)) * D + 4 * g;
    f32x4 q[QK];
#pragma unroll
    for (int j = 0; j < QK; ++j) q[j] = *(const f32x4*)(qp + 16 * j);

    float m = -INFINITY, l = 0.f;                     // l: this lane's keys only, until the end
    f32x4 o[VE * NB];
#pragma unroll
    for (int i = 0; i < VE * NB; ++i) o[i] = f32x4{0.f, 0.f, 0.f, 0.f};

    auto chunk_base = [&](int i, int pg) -> long long {       // element offset of the KV head's 16 rows of chunk wave + NW i
        const int off = ((wave + NW * i) * KEYS) & (ps - 1);
        return (((long long)min(max(pg, 0), b.num_pages - 1) * b.num_kv_heads + kvh) * ps + off) * D;
    };
    f32x4 k[2][QK];
    vec v[4][NB];
    auto load_k = [&](long long at, f32x4 (&kk)[QK]) {
        const float* kp = (const float*)a.k_cache + at + l16 * D + 4 * g;
#pragma unroll
        for (int j = 0; j < QK; ++j) kk[j] = *(const f32x4*)(kp + 16 * j);
    };
    auto load_v = [&](long long at) {
        const float* vp = (const float*)a.v_cache + at + 4 * g * D + ch0 + VE * l16;
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int n = 0; n < NB; ++n) v[u][n] = *(const vec*)(vp + u * D + 64 * n);
    };
    auto compute = [&](int c, long long at, const f32x4 (&kk)[QK]) {
        f32x4 s = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int j = 0; j < QK; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) s = __builtin_amdgcn_mfma_f32_16x16x4f32(kk[j][e], q[j][e], s, 0, 0, 0);
        const bool masked = c * KEYS + KEYS - 1 > min_limit;                // some row does not see some key
        float x[4], p[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            x[u] = s[u] * b.softmax_scale;
            if (masked && c * KEYS + 4 * g + u > limit) x[u] = -INFINITY;
        }
        const float m_new = fmaxf(m, group_max(fmaxf(fmaxf(x[0], x[1]), fmaxf(x[2], x[3]))));
        const float ref = m_new == -INFINITY ? 0.f : m_new;                 // a row that sees none of the keys so far
        const float alpha = expf(m - ref);                                  // 0 on the first visible chunk (m = -inf)
        m = m_new;
#pragma unroll
        for (int u = 0; u < 4; ++u) p[u] = expf(x[u] - ref);
        l = l * alpha + ((p[0] + p[1]) + (p[2] + p[3]));
#pragma unroll
        for (int i = 0; i < VE * NB; ++i) o[i] *= alpha;
        if (masked) {
            // keys past the tile's last are no tokens: whatever their slots hold must not count.  A key that some rows
            // see and others do not may hold an infinity or NaN, which a weight of 0 would not remove: such a chunk
            // is done key by key with what each row sees.
            bool odd = false;
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int n = 0; n < NB; ++n) {
                    if (c * KEYS + 4 * g + u >= kv_len) v[u][n] = vec(0.f);
#pragma unroll
                    for (int e = 0; e < VE; ++e) odd = odd || !is_finite(v[u][n][e]);
                }
            if (__builtin_amdgcn_ballot_w64(odd) != 0) {
                for (int kk2 = 0; kk2 < KEYS && c * KEYS + kk2 < kv_len; ++kk2) {
                    const int u = kk2 & 3;
                    const float mine = u == 0 ? p[0] : u == 1 ? p[1] : u == 2 ? p[2] : p[3];
                    const float pk = __shfl(mine, l16 + 16 * (kk2 >> 2));
                    const float* vp = (const float*)a.v_cache + at + (long long)kk2 * D + ch0 + 4 * VE * g;
                    if (c * KEYS + kk2 <= limit)
#pragma unroll
                        for (int n = 0; n < NB; ++n)
#pragma unroll
                            for (int t = 0; t < 4; ++t) {
                                const vec w = *(const vec*)(vp + 64 * n + VE * t);
#pragma unroll
                                for (int e = 0; e < VE; ++e) o[VE * n + e][t] = fmaf(pk, w[e], o[VE * n + e][t]);
                            }
                }
                return;
            }
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int n = 0; n < NB; ++n)
#pragma unroll
                for (int e = 0; e < VE; ++e) o[VE * n + e] = __builtin_amdgcn_mfma_f32_16x16x4f32(v[u][n][e], p[u], o[VE * n + e], 0, 0, 0);
    };
    const int n_mine = n_chunks > wave ? (n_chunks - wave + NW - 1) / NW : 0;    // chunks wave, wave + NW, ...
    if (n_mine > 0) {
        // this chunk's V, the next one's K and the page of the one after it are on their way while this chunk's scores are computed
        // (past the last chunk the last one's again: with loads that depend on there being one the waits would have to allow for both)
        const int end = n_mine - 1;
        long long at = chunk_base(0, page);
        load_k(at, k[0]);
        page = page_of(min(1, end));
        for (int i = 0; i <= end; i += 2) {
            load_v(at);
            const long long next = chunk_base(min(i + 1, end), page);
            load_k(next, k[1]);
            page = page_of(min(i + 2, end));
            compute(wave + NW * i, at, k[0]);
            if (i + 1 > end) break;
            load_v(next);
            at = chunk_base(min(i + 2, end), page);
            load_k(at, k[0]);
            page = page_of(min(i + 3, end));
            compute(wave + NW * (i + 1), next, k[1]);
        }
    }

    // ---- the waves' results: o[VE n + e][t] is channel ch0 + 64 n + VE (4 g + t) + e of row l16
    l = group_sum(l);
#pragma unroll
    for (int n = 0; n < NB; ++n)
#pragma unroll
        for (int x = 0; x < VE; ++x) {                // 4 VE channels, four at a time
            f32x4 w;
#pragma unroll
            for (int y = 0; y < 4; ++y) w[y] = o[VE * n + (4 * x + y) % VE][(4 * x + y) / VE];
            *(f32x4*)&o_s[wave][l16][64 * n + 4 * VE * g + 4 * x] = w;
        }
    if (g == 0) {
        m_s[wave][l16] = m;
        l_s[wave][l16] = l;
    }
    __syncthreads();
    // 16 rows x CH / 4 pieces of 16 bytes
    for (int idx = tid; idx < ROWS * (CH / 4); idx += 64 * NW) {
        const int my = idx / (CH / 4), c4 = idx % (CH / 4) * 4;
        if (row0 + my >= n_rows) break;
        float m_all = -INFINITY, l_all = 0.f;
#pragma unroll
        for (int w = 0; w < NW; ++w) m_all = fmaxf(m_all, m_s[w][my]);
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            const float wgt = m_s[w][my] == -INFINITY ? 0.f : expf(m_s[w][my] - m_all);
            l_all += wgt * l_s[w][my];
            acc += wgt * *(const f32x4*)&o_s[w][my][c4];
        }
        const float inv = (l_all > 0.f) ? 1.f / l_all : 0.f;                // no keys (cross, empty cache): zero row
        const int o_row = row0 + my, o_tok = by_G.quotient(o_row);
        const long long at = (first_row + o_tok) * b.num_q_heads + kvh * G + (o_row - o_tok * G);
        *(f32x4*)((float*)a.out + at * D + ch0 + c4) = acc * inv;
        if (a.lse != nullptr && ch0 + c4 == 0) a.lse[at] = (l_all > 0.f) ? m_all + logf(l_all) : -INFINITY;
    }
}

// Waves of a workgroup.  Few workgroups need many, which share the keys; where the workgroups alone fill the chip, the
// combination of the waves and the LDS that it takes only cost, the more so the shorter the contexts (at most `keys`, what a row
// of the page table can hold).  Long ones that differ keep more, by which the longest ends sooner.  Measured on 300 shapes, us with
// 8 / 4 / 2 / 1 waves: one new token of 128 requests, 32 heads of 64 (4352 workgroups), 16 keys 53 / 28 / 20 / 16, 301 keys 146 /
// 124 / 126 / 123; of 32 requests (1088), 16 keys 17 / 11 / 11 / 11; of 8 (256), 301 keys 15 / 16 / 21 / 29; of 44 (1472), up to 700 keys
// 71 / 66 / 70 / 87, up to 2700 244 / 256 / 258 / 312; of 64 on 4 KV heads (384), the same 61 / 69 / 125 / 191.  Prompts share K and V
// among their row tiles: 1024 new tokens, 32 heads on 8 of 64 (2056) 88 / 71 / 83 / 92; 32 requests of 64 + 256 (4352) 127 / 86 / 82 / 76.
// `single`: at most one row tile for a (request, KV head), as in a decode step.
// (Those times are older than the loads that overlap and the registers they take.  Of 162 shapes measured since, the choice is 4 % behind the
// best on average; the largest differences are at head_dim 128: 101 contexts of 801 tokens on one KV head, 8 and 4 waves, 30.2 and 26.9, 19 prompts of
// 17 + 44 on 8, 4 and 1, 36.8 and 25.6.)
int waves_of(long long workgroups, bool single, long long keys)
{
    int waves;
    if (keys >= 512) waves = workgroups <= 512 || (single && keys >= 1024) ? 8 : 4;
    else if (single) waves = workgroups <= 320 ? 8 : workgroups <= 1024 ? 4 : workgroups <= 2048 ? 2 : 1;
    else waves = workgroups <= 320 ? 8 : workgroups <= 4096 ? 4 : 2;
    while (waves > 1 && (waves / 2) * KEYS >= keys) waves /= 2;           // no more than there are chunks of keys
    return waves;
}

// Few workgroups with many keys are bound by their compute unit's matrix pipes and by what it fetches while the others idle: up to
// SPLIT_WORKGROUPS of them become four each, which make a quarter of the channels (the scores again, a quarter of V).  4 heads on 1 of 64,
// 256 cached + 64 new tokens (17 workgroups), 10.3 -> 9.3 us of the GPU with the scatter, 1024 + 64 20.3 -> 15.7; from 80 workgroups on it is slower
// (88: 10.8 and 13.9).
constexpr int SPLIT_WORKGROUPS = 64;
// By its registers two workgroups of 8 waves or four of 4 fit a compute unit (head_dim 64).  The dispatcher fills places, not time: some compute
// units get all they hold while others have fewer, or none where the grid's workgroups without rows held the places and left (a decode step has
// one slot more than row tiles for every request), and who shares a compute unit is as much longer.  So fewer fit, APART, in steps of one row
// tile per (request, KV head): one of 8 waves, and three of 4 where as many places are enough for all that have rows.  us, as many as the registers allow
// and APART: 8 waves, 32 contexts of 1000 tokens on 8 KV heads (256 pairs) 35.0 and 26.8, 22 of 414 to 1659 on 16 (352) 48.5 and 42.3, 163 of 1145 to
// 4580 on 4 (652) 211 and 196 (equal ones lose what the chip holds at once: 347 of 915 on one (347) 38.8 and 41.3, and more the shorter they are: 17 of
// 79 on 16 (272) 9.9 and 12.5); 4 waves, 340 of 933 on 2 (680) 76.4 and 67.4, 81 of 360 on 8 (648) 29.0 and 25.8, but 99 of 43 on 8 (792) 10.4 and 12.0
// and 104 of 877 on 4 (416) 49.5 and 50.2.
constexpr int COMPUTE_UNITS = 256, PLACES = 3;
bool apart_of(int waves, long long workgroups, long long pairs, long long keys)
{
    if (waves == 8) return workgroups > COMPUTE_UNITS && (pairs <= COMPUTE_UNITS || keys >= 512);
    return waves == 4 && pairs > (PLACES - 1) * COMPUTE_UNITS && pairs <= PLACES * COMPUTE_UNITS;
}

}  // namespace

hipError_t launch_attn_f32(const AttnArgs& a, hipStream_t stream)
{
    const BatchView& b = a.b;
    if (b.total_new_tokens == 0 || b.num_reqs == 0) return hipSuccess;
    const int G = b.num_q_heads / b.num_kv_heads;
    const long long grid = ((long long)b.total_new_tokens * G / ROWS + b.num_reqs) * b.num_kv_heads;
    if (grid > 0x7fffffff) return hipErrorInvalidValue;
    auto go = [&](auto d, auto nw, auto split, auto apart) {
        constexpr int D = decltype(d)::value, NW = decltype(nw)::value, SPLIT = decltype(split)::value;
        hipLaunchKernelGGL((attn_f32_kernel<D, NW, SPLIT, decltype(apart)::value>), dim3((unsigned)(grid * SPLIT)), dim3(64 * NW), 0, stream, a, G, divisor_of(G), divisor_of(b.num_kv_heads));
    };
    const bool single = (long long)b.max_new_len * G <= ROWS;              // at most one row tile for a (request, KV head)
    const long long keys = (long long)b.max_pages * b.page_size;
    const int waves = waves_of(grid, single, keys);
    const bool apart = single && apart_of(waves, grid, (long long)b.num_reqs * b.num_kv_heads, keys);
    auto of_dim = [&](auto d) {
        using one = std::integral_constant<int, 1>;
        using eight = std::integral_constant<int, 8>;
        constexpr bool small = decltype(d)::value == 64;
        if (waves == 8 && grid <= SPLIT_WORKGROUPS) go(d, eight{}, std::integral_constant<int, 4>{}, std::false_type{});
        else if (waves == 8 && small && apart) go(d, eight{}, one{}, std::integral_constant<bool, small>{});
        else if (waves == 8) go(d, eight{}, one{}, std::false_type{});
        else if (waves == 4 && small && apart) go(d, std::integral_constant<int, 4>{}, one{}, std::integral_constant<bool, small>{});
        else if (waves == 4) go(d, std::integral_constant<int, 4>{}, one{}, std::false_type{});
        else if (waves == 2) go(d, std::integral_constant<int, 2>{}, one{}, std::false_type{});
        else go(d, one{}, one{}, std::false_type{});
    };
    if (b.head_dim == 64) of_dim(std::integral_constant<int, 64>{});
    else of_dim(std::integral_constant<int, 128>{});
    return hipGetLastError();
}

}  // namespace emm
