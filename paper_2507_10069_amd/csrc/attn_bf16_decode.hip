// Decode-step attention over the paged KV pool (bf16, head_dim 128, pages of 16 to 256 tokens) for gfx950: every
// request has at most ONE query token, which attends to its whole context -- the stage that follows
// prefill and produces one token per iteration (Section 2.2 of the paper; memory bound, as it says).
// Same operation as the prefill kernel restricted to one row tile of G = H / Hkv rows per (request,
// KV head) pair; what differs is where the parallelism comes from: the K/V bytes of a pair are read
// exactly once, so the work is cut along the KEY axis, first into pieces of `tiles_per_piece` 32-key
// tiles (one workgroup each), then, inside a workgroup, block by block of 16 keys over its 4 waves.
//
//   workgroup = one piece of one pair, 4 waves, 64 KB of LDS, two on a compute unit.  Wave w takes blocks w, w+4, ... of
//               the piece and does everything for them by itself: it fetches them by LDS-DMA into a ring of its
//               own (two blocks of K and V: one is computed while the other is on its way), waits for its own
//               fetches only, and keeps its own online softmax.  There is no barrier before the end.  (With
//               tiles that all waves fetch and one of them computes, a barrier per tile, the waves' computing was
//               one chain: 0.6 us per 32 keys, which bound every batch too small to fill the chip: one context
//               of 1500 tokens 10.6 -> 7.3 us for both kernels, of 16384 17.1 -> 13.6.)
//   matrix    = v_mfma_f32_16x16x32 for S^T = K Q^T and 16x16x16 for O^T += V^T P^T: 16 query rows, the most a KV head
//               has here, so half the accumulators and half the exponentials of the 32-column shape, and a lane's
//               four scores are the four keys that the value product expects from it.  The matrix pipe is mostly
//               idle; the kernel is bound by the rate at which blocks arrive from HBM.
//   merge 1   = the 4 waves' (maximum, row sum, accumulator) are combined through LDS;
//   merge 2   = a pair with several pieces leaves one record per piece in the workspace, and the last of its workgroups
//               (small batches: see FOLD_PIECES), attn_bf16_decode_merge_kernel or, where rows have few pieces,
//               attn_bf16_decode_merge_rows_kernel combines them; a pair with one piece writes its output directly.  All derive
//               the piece count from the lengths.
//
// Shared prefixes (Section 3.3: requests repeat system prompts and images).  Requests whose leading pages
// are the same physical pages can be given as a UNIT: up to 32 / G consecutive requests and the length they
// share.  The shared keys are then read once per unit instead of once per request: extra workgroups at the
// end of the grid take the shared part, with the query rows of all the unit's requests side by side in the
// two groups of 16 rows, while the requests' own workgroups start behind the shared part; the merge
// kernel adds the records of both.  Built as a second instantiation (SHARED) so that the plain path pays
// nothing for it.  Units of a batch that the L2s can hold are left aside: see better_alone.
//
// Fused step (FUSED instantiation, emm_decode_step): the query token's own K/V row need not be in the pool
// beforehand.  The wave whose block holds the token's slot asks for the row in k_new / v_new before its first fetch and
// puts it into the LDS block once the block has landed (into the swizzled places the loads would have put it) and into
// the pool, so a decode step is one launch less than scatter + attention.  (Stored in the pool before the first fetch, as
// it was, the row cost its wave two round trips: 32 contexts of 1500 tokens 20.9 -> 20.0 us, 8 of 4000 17.3 -> 16.4.)
#include "attn_bf16_common.h"

#include <algorithm>
#include <atomic>
#include <chrono>
#include <climits>
#include <mutex>
#include <type_traits>

namespace emm {

namespace {

using namespace bf16attn;

constexpr int MAX_G = 16;                        // query heads per KV head this kernel takes
constexpr int REC_FLOATS = D + 2;                // per row of a record: 128 accumulator values, m, l (folded: the rows' values, then their m, l)
constexpr int RED_FLOATS = D + 4;                // per row in LDS: 128 accumulator values, m, l, and the next row 16 bytes aligned
constexpr int NW = 4;                            // waves per workgroup
constexpr int NT = NW * 64;
constexpr int BK = 32;                           // keys per tile, the unit in which pieces are measured
constexpr int BLK = 16;                          // keys per block, what a wave fetches and computes at a time (a page holds 1 to 16)
constexpr int BLOCKS_PER_TILE = BK / BLK;
constexpr int BLOCK_BYTES = BLK * D * 2;         // one K or V block in LDS: 16 rows of 256 bytes
constexpr int NSLOT = 2;                         // blocks a wave's ring holds; block i of a wave lives in slot i % NSLOT
constexpr int RING_BYTES = NSLOT * 2 * BLOCK_BYTES;      // of one wave: slots of a K block and a V block
constexpr int PAIR_TILES = 2 * NW / BLOCKS_PER_TILE;     // up to so many tiles of a piece a wave has two blocks at most, which it does side by side
constexpr int MIN_TILES_PER_PIECE = 4, MAX_TILES_PER_PIECE = 124;  // a wave's blocks of a piece: at most 62, one page id per lane
constexpr int WORKGROUPS_PER_ROUND = 2 * 256;    // two workgroups on each of 256 CUs
constexpr int WORKGROUPS_PER_ROUND_ONE_REQUEST = 384;    // see attn_bf16_decode_shape
constexpr int MAX_ROWS = 32;                     // query rows of a shared-prefix unit
static_assert(MAX_G * RED_FLOATS * 4 <= RING_BYTES, "the merge across waves reuses the rings, each wave its own");
static_assert(MAX_TILES_PER_PIECE * BLOCKS_PER_TILE <= NW * 64, "a wave's page ids sit in one register");

// What a launch adds to its arguments: the ticket of a folded merge (0: none) and quotients that every workgroup would have to work out
// (with every argument asked for at the start a call is 0.3 us shorter than with divisions).
struct LaunchInfo {
    unsigned long long ticket;
    int32_t G, grid_y;
    Divisor by_kv_heads, by_piece /* tiles_per_piece */, by_pairs, by_unit_pairs;
};
constexpr int MAX_GRID_Y = 32768;
__device__ inline int up_to_pieces(int n_tiles, int tiles_per_piece) { return (n_tiles + tiles_per_piece - 1) / tiles_per_piece; }
__device__ inline int up_to_pieces(int n_tiles, const Divisor& by_piece) { return by_piece.quotient(n_tiles - 1) + 1; }    // n_tiles > 0
template <typename PIECE> __device__ inline int pieces_of(int kv_len, const PIECE& tiles_per_piece)
{
    const int n_tiles = (kv_len + BK - 1) / BK;
    return n_tiles == 0 ? 1 : up_to_pieces(n_tiles, tiles_per_piece);
}
// pieces of a request's own part when its first t_off tiles belong to a unit's shared part: possibly none
template <typename PIECE> __device__ inline int own_pieces_of(int kv_len, int t_off, const PIECE& tiles_per_piece, bool in_unit)
{
    if (!in_unit) return pieces_of(kv_len, tiles_per_piece);
    const int n_tiles = (kv_len + BK - 1) / BK - t_off;
    return n_tiles <= 0 ? 0 : up_to_pieces(n_tiles, tiles_per_piece);
}
// max or sum over the four lanes that hold a query row (lane % 16)
__device__ inline float quad_max(float x)
{
    const uint32_t u = __float_as_uint(x);
    const auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
    return pair_max(fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1])));
}
__device__ inline float quad_sum(float x)
{
    const uint32_t u = __float_as_uint(x);
    const auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
    return pair_sum(__uint_as_float(r[0]) + __uint_as_float(r[1]));
}
// what the lane N places further on holds, of the 16 of a row of lanes, which go round
template <int N> __device__ inline float from_lane(float x)
{
    return __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(x), 0x120 + 16 - N, 0xf, 0xf, false));
}
// workspace: the requests' own records first, [pair][piece][MAX_G rows], then the units', [unit][KV head][piece][MAX_ROWS]
__device__ __host__ inline size_t unit_records_offset(const DecodeShape& S)
{
    return (size_t)S.n_pairs * S.pieces_max * MAX_G * REC_FLOATS;
}

// K and V are fetched past the caches (non-temporal) when a call reads more of them than the last-level cache would keep
// until they are read again: 6.6 instead of 5.7 TB/s (64 x 8192 tokens 196 -> 173 us, 262 MB ragged 56 -> 48, 102 MB in
// one context 25.5 -> 23.6); below, where a repeated call finds them there, it costs up to 12 % (66 MB: 15.7 -> 17.7).
// The line lies between.  Pages that several requests read would lose what the first of them brought into the L2 (32
// requests on 8 videos without units: 115 -> 154 us): each wave looks whether another request holds its first page.
constexpr long long STREAM_BYTES = 96ll << 20;
constexpr int STREAM_TILES = (int)(STREAM_BYTES / (BK * D * 4));

// Does a request other than r .. r + n - 1 hold page `id` at entry `at` of its row of the page table?  (Shared pages are
// leading pages, so a shared one stands at the same entry everywhere.)  The whole wave asks, 64 requests at a time; with
// more than SHARE_LOOKUP of them the answer is yes, unasked.  What is found decides how the page is fetched and nothing
// else, so entries past a request's own pages do no harm.  The entries of the first 64 requests (`first`, one per lane) are
// asked for together with the lengths, the answer is formed when the workgroups without work have left.
constexpr int SHARE_LOOKUP = 512;
__device__ inline int first_holders(const BatchView& b, int at)
{
    // (an atomic load of the weakest kind, which is an ordinary one, but which the compiler leaves where it is written)
    return __hip_atomic_load(b.page_table + (long long)min((int)threadIdx.x & 63, b.num_reqs - 1) * b.max_pages + at, __ATOMIC_RELAXED,
                             __HIP_MEMORY_SCOPE_WAVEFRONT);
}
__device__ inline bool holds_page(const BatchView& b, int first, int at, int id, int r, int n)
{
    if (b.num_reqs > SHARE_LOOKUP) return true;
    const int lane = threadIdx.x & 63;
    bool found = first == id && lane < b.num_reqs && (lane < r || lane >= r + n);
    for (int k = lane + 64; k < b.num_reqs; k += 64)
        found = found || (b.page_table[(long long)k * b.max_pages + at] == id && (k < r || k >= r + n));
    return __builtin_amdgcn_ballot_w64(found) != 0;
}

// The waits of the block loop, written out because the compiler does not see the LDS-DMA fetches: all but the newest
// PENDING of this wave's fetches have landed.  The clobber keeps reads of LDS behind it.
template <int PENDING>
__device__ inline void wait_fetches()
{
    static_assert(PENDING < 16, "the low four bits of the count");
    asm volatile("s_waitcnt vmcnt(%0)" ::"i"(PENDING) : "memory");
}

// Where a context and a unit have at most ROW_PIECES pieces and there are rows for every compute unit, a wave of its own merges each row: see
// attn_bf16_decode_merge_rows_kernel.
constexpr int ROW_PIECES = 8, ROW_ROWS = 256;
// waves of the merge kernel by the pieces of a context (see there)
constexpr int MANY_PIECES = 32, MANY_WAVES = 16, FEW_WAVES = 4;

// ---- Folded merge: where a context has few pieces (fold_applies), the last of its workgroups to finish combines them and the second
// kernel is not launched.  Nobody waits for anybody: a workgroup stores its record, counts itself in and leaves unless it is the one that
// completes the count.  Records and counts are stored, counted and read with agent scope (past what the XCDs do not share), a wave's
// stores are awaited before its workgroup counts, and pieces are combined in their order, so the result does not depend on who is last.
// The count of a (request, KV head) lies in the last row of its first record, which FOLD_ROWS query heads leave unused, and needs no
// zero to start from: it is the launch's ticket (48 bits that no other launch of this process has) above the number of workgroups.
// Each workgroup asks for it with the lengths and, unless the ticket is there, puts it there before its first fetch; whoever completes
// the count takes the ticket away, so that a replay of a captured launch starts again.  Every workgroup that the grid has for a context
// counts, whatever the device arrays hold, so the count is completed in every launch.
constexpr int FOLD_PIECES = 16, FOLD_ROWS = 8, FOLD_COUNT_BITS = 16;
__device__ inline unsigned long long* fold_count(const AttnArgs& a, const DecodeShape& S, int pair)
{
    return (unsigned long long*)((float*)a.workspace + ((size_t)pair * S.pieces_max * MAX_G) * REC_FLOATS + (MAX_G - 1) * D);
}

typedef float f32x2_rec __attribute__((ext_vector_type(2)));
__device__ inline void put_record(float* at, f32x2_rec x)
{
    __hip_atomic_store((unsigned long long*)at, __builtin_bit_cast(unsigned long long, x), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ inline f32x2_rec get_record(const float* at)
{
    return __builtin_bit_cast(f32x2_rec, __hip_atomic_load((const unsigned long long*)at, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
}

// The same, 16 bytes of a record at a time (buffer instructions, whose cache policy can be stated; `record` is the same in all lanes).
typedef uint32_t u32x4_rec __attribute__((ext_vector_type(4)));
typedef float f32x4_rec __attribute__((ext_vector_type(4)));
constexpr int AGENT_SCOPE = 16, RAW_BUFFER = 0x00020000;     // cache policy sc1; a buffer without a format
__device__ inline void put_record4(float* record, int at, f32x4_rec x)
{
    const auto all = __builtin_amdgcn_make_buffer_rsrc(record, 0, MAX_G * REC_FLOATS * 4, RAW_BUFFER);
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4_rec, x), all, at * 4, 0, AGENT_SCOPE);
}

// A piece's two channels, weighted, in either merge.  What is fused is written out, so that both round alike: left to the compiler it is this
// in the one and both channels in the other.
__device__ inline void add_weighted(f32x2_rec& acc, float wgt, f32x2_rec x)
{
#pragma clang fp contract(off)
    acc[0] = fmaf(wgt, x[0], acc[0]);
    acc[1] += wgt * x[1];
}

// The same for a sum of weights: the first of some pieces, which scales what there is already, and the others.
__device__ inline float add_weight(bool first, float l, float alpha, float wgt, float x)
{
#pragma clang fp contract(off)
    return first ? fmaf(l, alpha, wgt * x) : fmaf(wgt, x, l);
}

// a launch without units passes none: arguments that lie closer together arrive sooner (16 contexts of 500 tokens, 28 / 4 heads, 8.46 and 8.25 us)
struct NoUnits {};
template <bool SHARED> using UnitsOf = std::conditional_t<SHARED, SharedPrefixView, NoUnits>;

// FOLD: the launch has a ticket.  (With the folded merge in one kernel for all, calls that do not use it were 0.3 us longer: 32 / 8 heads,
// one context of 60 tokens 3.65 us and 3.34.)
template <bool CAUSAL, bool SHARED, bool FUSED, bool FOLD>
__global__ __launch_bounds__(NT, 2) void attn_bf16_decode_kernel(AttnArgs a, DecodeShape S, LaunchInfo info, UnitsOf<SHARED> units)
{
    static_assert(CAUSAL || !FUSED, "only a causal step has a new token to store");
    static_assert(!SHARED || !FOLD, "units have the second kernel");
    __shared__ __attribute__((aligned(1024))) unsigned char smem[NW * RING_BYTES];
    typedef short s16x4 __attribute__((ext_vector_type(4)));
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    SharedPrefixView sv = {};
    if constexpr (SHARED) sv = units;

    const BatchView& b = a.b;
    const int G = info.G;
    const int n_own_blocks = S.n_pairs * S.pieces_max;
    const bool unit_mode = SHARED && (int)blockIdx.x >= n_own_blocks;     // this workgroup: a unit's shared part
    // piece-major: the first pieces of all contexts come first in the grid, the workgroups that find their
    // context too short for their piece number (they exit at once) gather at its end
    const int n_items = unit_mode ? S.n_unit_pairs : S.n_pairs;
    // (without units the grid has a dimension for the pieces, which saves a division; the third is for more than MAX_GRID_Y)
    const int blk = unit_mode ? blockIdx.x - n_own_blocks : blockIdx.x;
    const int piece = SHARED ? (unit_mode ? info.by_unit_pairs : info.by_pairs).quotient(blk) : blockIdx.y + info.grid_y * blockIdx.z;
    const int pair = SHARED ? blk - piece * n_items : blk;                // unit mode: (unit, KV head)
    const int unit = info.by_kv_heads.quotient(pair);                     // own part: this is the request itself
    const int kvh = pair - unit * b.num_kv_heads;
    // (what the device arrays hold is forced into range wherever an address depends on it: see clamp_new_len)
    const int r = unit_mode ? min(max(sv.unit_first_req[unit], 0), b.num_reqs - 1) : unit;   // the request whose page table is read
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lane = tid & 63;
    const int l16 = lane & 15, g = lane >> 4;
    // everything that is needed of the lengths, asked for together (and before any of it decides on a branch)
    const int new_len = b.new_lens[r], prefix_len = b.prefix_lens[r], cu_new = b.cu_new_lens[r];
    const int req_unit = SHARED ? sv.req_unit[r] : -1, req_shared = SHARED ? sv.req_shared_len[r] : 0;
    const int t_off = (SHARED && !unit_mode) ? max(req_shared, 0) / BK : 0;   // tiles a unit computes for this request
    const int t_begin = t_off + piece * S.tiles_per_piece;
    // Wave w does blocks w, w + 4, ... of the piece; lane k holds where in the pool its k-th one lies.  Asked for before
    // the lengths are known, so that the two loads overlap: entries past the request's pages are read (the row
    // has max_pages of them) and forced into the pool, but never fetched from.  (S.late: after them, so that workgroups without
    // work do not stay for the answer.)
    const int32_t* __restrict__ pt = b.page_table + (long long)r * b.max_pages;
    const int blk16 = t_begin * BLOCKS_PER_TILE + wave + NW * lane;       // logical 16-key block of the request
    const int pg_first = __builtin_amdgcn_readfirstlane(min(blk16 >> b.page_shift, b.max_pages - 1));    // of the wave's first block
    int pg_raw = 0, holders = 0;
    auto ask_pages = [&]() {
        pg_raw = pt[min(blk16 >> b.page_shift, b.max_pages - 1)];         // (max_pages > 0: checked on the host)
        if (S.stream != DecodeShape::STREAM_NEVER) holders = first_holders(b, pg_first);
    };
    if (!S.late) ask_pages();
    constexpr int SPEAKER = NW - 1;                          // the wave that counts for the workgroup: see FOLD_PIECES
    unsigned long long seen = 0;
    if (FOLD && wave == SPEAKER)
        seen = __hip_atomic_load(fold_count(a, S, pair), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    asm volatile("" ::"s"(new_len), "s"(prefix_len), "s"(cu_new));
    // and every argument that is needed further down, which the compiler would ask for where it is first used
    asm volatile("" ::"s"(a.q), "s"(a.k_cache), "s"(a.v_cache), "s"(a.out), "s"(a.lse), "s"(a.workspace), "s"(info.by_piece.mul), "s"(S.n_pairs));
    if (FUSED) asm volatile("" ::"s"(a.k_new), "s"(a.v_new));
    if (FOLD) asm volatile("" ::"s"(info.ticket));
    __builtin_amdgcn_sched_barrier(0);
    int kv_len, n_pieces, n_rows;
    bool direct;                                             // one piece and no unit: this workgroup writes the output
    if (!unit_mode) {
        if (new_len <= 0) return;                            // no query token
        const int P = clamp_prefix_len(b, prefix_len, CAUSAL ? 1 : 0);
        kv_len = CAUSAL ? P + 1 : P;                         // keys the query sees = slots that hold tokens
        const bool in_unit = SHARED && req_unit >= 0;
        n_pieces = own_pieces_of(kv_len, t_off, info.by_piece, in_unit);
        n_rows = G;
        direct = n_pieces == 1 && !in_unit;
    } else {
        // a multiple of the tile: no mask, no ragged tail
        kv_len = (int)min((long long)max(sv.unit_shared_len[unit], 0), (long long)b.max_pages * b.page_size) / BK * BK;
        n_pieces = kv_len > 0 ? up_to_pieces(kv_len / BK, info.by_piece) : 0;
        n_rows = min(max(sv.unit_num_reqs[unit], 1) * G, MAX_ROWS);
        direct = false;
    }
    // (a grid of several z may have workgroups past the last piece that the workspace has room for)
    if (piece >= (SHARED ? n_pieces : min(n_pieces, S.pieces_max))) return;
    if (S.late) ask_pages();
    const bool folded = FOLD && !direct;                     // see FOLD_PIECES
    unsigned long long* const count = fold_count(a, S, pair);
    if (folded && wave == SPEAKER && lane == 0 && ((seen ^ info.ticket) >> FOLD_COUNT_BITS) != 0)
        __hip_atomic_compare_exchange_strong(count, &seen, info.ticket, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const int n_blocks = min(S.tiles_per_piece * BLOCKS_PER_TILE, (kv_len + BLK - 1) / BLK - t_begin * BLOCKS_PER_TILE);    // of the piece; 0 only for an empty context
    const int n_mine = n_blocks > wave ? (n_blocks - wave + NW - 1) / NW : 0;
    // in units of 4096 bytes (one block of one KV head): (page, KV head, block within the page)
    const int pg_vec = ((min(max(pg_raw, 0), b.num_pages - 1) * b.num_kv_heads + kvh) << b.page_shift) +
                       (blk16 & ((1 << b.page_shift) - 1));

    // ---- global -> LDS by LDS-DMA (lane i lands at base + 16 i), four rows of 256 bytes per instruction, rows = keys,
    //      16-byte chunks XOR-swizzled; the hardware fixes where a lane's bytes land, so the swizzle is on the source
    //      side: the lane that lands on (row, physical chunk p) fetches logical chunk p ^ f(row).
    //        K: f(row) = row          read with ds_read_b128, 16 rows of one chunk at a time
    //        V: f(row) = (row & 3) << 2   read with ds_read_tr16_b64, four rows of two chunks
    const uint32_t ring = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)smem + wave * RING_BYTES;
    unsigned char* my_ring = smem + wave * RING_BYTES;
    int k_goff[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) k_goff[j] = (4 * j + g) * 256 + ((l16 ^ (4 * j + g)) << 4);
    const int v_goff = g * 256 + ((l16 ^ (g << 2)) << 4);
    const unsigned char* __restrict__ kcb = (const unsigned char*)a.k_cache;
    const unsigned char* __restrict__ vcb = (const unsigned char*)a.v_cache;
    constexpr int FETCHES = 8;                               // instructions per block
    // (what the host does not know it takes from this context: the others are as long)
    const bool long_enough = S.stream == DecodeShape::STREAM_PRIVATE || (long long)(kv_len / BK - t_off) * n_items >= STREAM_TILES;
    const bool streamed = S.stream != DecodeShape::STREAM_NEVER && long_enough &&
                          !holds_page(b, holders, pg_first, __builtin_amdgcn_readfirstlane(pg_raw), r, unit_mode ? sv.unit_num_reqs[unit] : 1);
    auto fetch = [&](int i, int slot) {                      // this wave's block i into its ring
        const long long off = (long long)__builtin_amdgcn_readlane(pg_vec, i) * BLOCK_BYTES;
        const uint32_t to = __builtin_amdgcn_readfirstlane(ring + slot * (2 * BLOCK_BYTES));
        if (streamed) {
#pragma unroll
            for (int j = 0; j < 4; ++j) lds_dma16_streamed(kcb + off, k_goff[j], to + j * 1024);
#pragma unroll
            for (int j = 0; j < 4; ++j) lds_dma16_streamed(vcb + off, v_goff + j * 1024, to + BLOCK_BYTES + j * 1024);
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j) lds_dma16(kcb + off, k_goff[j], to + j * 1024);
#pragma unroll
            for (int j = 0; j < 4; ++j) lds_dma16(vcb + off, v_goff + j * 1024, to + BLOCK_BYTES + j * 1024);
        }
    };
    const int limit = kv_len - 1;                            // last visible key (the query's own slot if causal)
    auto first_key = [&](int i) { return t_begin * BK + (wave + NW * i) * BLK; };
    // V rows (keys) past the context are zeroed in LDS: 0 * NaN would poison the output; K rows past it only give
    // scores that the mask removes
    auto zero_v_tail = [&](int i, int slot) {
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (first_key(i) + 4 * j + g >= kv_len)
                *(uint4*)(my_ring + slot * (2 * BLOCK_BYTES) + BLOCK_BYTES + j * 1024 + lane * 16) = make_uint4(0, 0, 0, 0);
    };
    // FUSED: the query token's own K/V row (K by lanes 0..15, V by 16..31) comes from k_new / v_new into the places the fetches
    // would have put it, and into its slot in the pool for the steps to come (the block fetched from there is patched, so the order of the
    // two does not matter).  Only its wave asks for it, before its fetches: the row is in registers when the block has landed.
    const long long first_row = clamp_first_row(b, cu_new, 1);
    const bool row_is_mine = FUSED && !unit_mode && n_mine > 0 && limit >= first_key(0) && (limit - first_key(0)) % (NW * BLK) < BLK &&
                             (limit - first_key(0)) / (NW * BLK) < n_mine;
    const int row_block = row_is_mine ? (limit - first_key(0)) / (NW * BLK) : -1;
    uint4 new_row = make_uint4(0, 0, 0, 0);
    if (row_is_mine && lane < 32)
        new_row = *(const uint4*)((const unsigned char*)(lane < 16 ? a.k_new : a.v_new) + (first_row * b.num_kv_heads + kvh) * (D * 2) + l16 * 16);
    auto patch_new_row = [&](int i, int slot) {
        const int row = limit - first_key(i);
        if (lane < 32) {
            const int chunk = l16 ^ (lane < 16 ? row : (row & 3) << 2);
            *(uint4*)(my_ring + slot * (2 * BLOCK_BYTES) + (lane < 16 ? 0 : BLOCK_BYTES) + row * 256 + (chunk << 4)) = new_row;
            unsigned char* pool = (unsigned char*)const_cast<void*>(lane < 16 ? a.k_cache : a.v_cache);
            *(uint4*)(pool + (long long)__builtin_amdgcn_readlane(pg_vec, i) * BLOCK_BYTES + row * 256 + l16 * 16) = new_row;
        }
    };

    // ---- LDS read addresses.  K: lane (key l16, g) reads chunk 4 st + g; V: lane j of a 16-lane group points at four
    //      channels of key 4 g + j / 4 and receives the group's four keys of channel 16 nb + j.
    const int k_rd0 = l16 * 256 + ((g ^ l16) << 4);
    const int v_rd0 = BLOCK_BYTES + (4 * g + (l16 >> 2)) * 256 + ((((l16 >> 1) & 1) ^ ((l16 >> 2) << 2)) << 4) + (l16 & 1) * 8;
    const float c_log2 = b.softmax_scale * 1.44269504088896340736f;

    // after the loop: each wave's results in its own ring, [16 rows][132], so that no wave has to wait until the others are past theirs
    auto partial = [&](int w, int row) { return (float*)(smem + w * RING_BYTES) + row * RED_FLOATS; };
    // The piece with NR groups of 16 query rows: the G heads of the request or, in unit mode, the G heads of each of
    // the unit's requests; columns of the MFMA past them repeat the last row and are discarded.
    auto attend = [&](auto nr_c) {
        constexpr int NR = decltype(nr_c)::value;
        bf16x8 qf[NR][4];
#pragma unroll
        for (int q = 0; q < NR; ++q) {
            const int my_row = min(16 * q + l16, n_rows - 1);
            const int hq = kvh * G + (unit_mode ? my_row % G : my_row);
            const long long q_row = unit_mode ? clamp_first_row(b, b.cu_new_lens[min(r + my_row / G, b.num_reqs - 1)], 1) : first_row;
            const __bf16* __restrict__ qp = (const __bf16*)a.q + (q_row * b.num_q_heads + hq) * D + 8 * g;
#pragma unroll
            for (int st = 0; st < 4; ++st) qf[q][st] = *(const bf16x8*)(qp + 32 * st);
        }
        f32x4 o_acc[NR][8];
        float m_run[NR], l_run[NR];
#pragma unroll
        for (int q = 0; q < NR; ++q) {
            m_run[q] = -INFINITY;
            l_run[q] = 0.f;
#pragma unroll
            for (int nb = 0; nb < 8; ++nb) o_acc[q][nb] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
        // one block, start to finish: S^T = K Q^T, mask, online softmax, O^T += V^T P^T
        auto compute = [&](int i, int slot) {
            const unsigned char* at = my_ring + slot * (2 * BLOCK_BYTES);
            bf16x8 kf[4];
#pragma unroll
            for (int st = 0; st < 4; ++st) kf[st] = *(const bf16x8*)(at + (k_rd0 ^ (st << 6)));
            s16x4 vf[8];
#pragma unroll
            for (int nb = 0; nb < 8; ++nb)
                vf[nb] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(at + (v_rd0 ^ (nb << 5))));
            f32x4 s[NR];
#pragma unroll
            for (int q = 0; q < NR; ++q) {
                s[q] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int st = 0; st < 4; ++st) s[q] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[st], qf[q][st], s[q], 0, 0, 0);
            }
            const int key0 = first_key(i);
            if (key0 + BLK > kv_len) {
#pragma unroll
                for (int q = 0; q < NR; ++q)
#pragma unroll
                    for (int v = 0; v < 4; ++v) s[q][v] = (key0 + 4 * g + v > limit) ? -INFINITY : s[q][v];
            }
#pragma unroll
            for (int q = 0; q < NR; ++q) {
                // The reference of a row (the same in its four lanes) is its running maximum: the largest weight is then exactly
                // 1 and carries no rounding error.  (Raised only when passed by 2^8, as with tiles of 32 keys before, the error
                // against 64 bits is 6 % larger where a wave has two blocks.)
                const float mx = fmaxf(fmaxf(s[q][0], s[q][1]), fmaxf(s[q][2], s[q][3]));
                if (__builtin_amdgcn_ballot_w64(mx > m_run[q]) != 0) {
                    const float m_new = fmaxf(quad_max(mx), m_run[q]);
                    const float alpha = m_run[q] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f((m_run[q] - m_new) * c_log2);
                    m_run[q] = m_new;
                    l_run[q] *= alpha;
#pragma unroll
                    for (int nb = 0; nb < 8; ++nb) o_acc[q][nb] *= alpha;
                }
                // every block has a visible key, but all its scores may be -infinity (products past the largest float): weights of 0
                const float mc = m_run[q] == -INFINITY ? 0.f : m_run[q] * c_log2;
                bf16x4 p;
                float psum = 0.f;
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    p[v] = (__bf16)__builtin_amdgcn_exp2f(fmaf(s[q][v], c_log2, -mc));
                    psum += (float)p[v];                     // the rounded value, as in the numerator
                }
                l_run[q] += psum;
#pragma unroll
                for (int nb = 0; nb < 8; ++nb)
                    o_acc[q][nb] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(vf[nb], __builtin_bit_cast(s16x4, p), o_acc[q][nb], 0, 0, 0);
            }
        };
        // Both blocks of a wave that has no more (pieces of four tiles, which small batches are cut into), side by side: a block is a chain of latencies, 0.43 us
        // where its wave has a SIMD to itself.  The sums are those of the two in turn, the first one's reference
        // included (one maximum for both: 0.1 us quicker, error against 64 bits 2.0e-3 -> 2.1e-3).  One context of 1500 tokens 6.68 -> 6.36 us, 8 of 900 8.09 -> 7.74, 28 / 4
        // heads, one of 2032 on 32 / 8 6.58 -> 6.33.
        // Longer pieces keep one block on its way while the other is computed.
        auto compute_pair = [&]() {
            f32x4 s[2];
            s16x4 vf[2][8];
            float mx[2], psum[2];
            bf16x4 p[2];
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const unsigned char* at = my_ring + i * (2 * BLOCK_BYTES);
                bf16x8 kf[4];
#pragma unroll
                for (int st = 0; st < 4; ++st) kf[st] = *(const bf16x8*)(at + (k_rd0 ^ (st << 6)));
                s[i] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int st = 0; st < 4; ++st) s[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[st], qf[0][st], s[i], 0, 0, 0);
            }
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int nb = 0; nb < 8; ++nb)
                    vf[i][nb] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(my_ring + i * (2 * BLOCK_BYTES) + (v_rd0 ^ (nb << 5))));
            if (first_key(1) + BLK > kv_len) {
#pragma unroll
                for (int v = 0; v < 4; ++v) s[1][v] = (first_key(1) + 4 * g + v > limit) ? -INFINITY : s[1][v];
            }
#pragma unroll
            for (int i = 0; i < 2; ++i) mx[i] = quad_max(fmaxf(fmaxf(s[i][0], s[i][1]), fmaxf(s[i][2], s[i][3])));
            const float m_all = fmaxf(mx[1], mx[0]);
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const float m_ref = i == 0 ? mx[0] : m_all;
                const float mc = m_ref == -INFINITY ? 0.f : m_ref * c_log2;
                psum[i] = 0.f;
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    p[i][v] = (__bf16)__builtin_amdgcn_exp2f(fmaf(s[i][v], c_log2, -mc));
                    psum[i] += (float)p[i][v];
                }
            }
            const float alpha = mx[0] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f((mx[0] - m_all) * c_log2);
            const bool raised = __builtin_amdgcn_ballot_w64(mx[1] > mx[0]) != 0;
            m_run[0] = m_all;
            l_run[0] = (raised ? psum[0] * alpha : psum[0]) + psum[1];
#pragma unroll
            for (int nb = 0; nb < 8; ++nb)
                o_acc[0][nb] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(vf[0][nb], __builtin_bit_cast(s16x4, p[0]), o_acc[0][nb], 0, 0, 0);
            if (raised)
#pragma unroll
                for (int nb = 0; nb < 8; ++nb) o_acc[0][nb] *= alpha;
#pragma unroll
            for (int nb = 0; nb < 8; ++nb)
                o_acc[0][nb] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(vf[1][nb], __builtin_bit_cast(s16x4, p[1]), o_acc[0][nb], 0, 0, 0);
        };
        if (NR == 1 && n_mine == 2) {
            fetch(0, 0);
            fetch(1, 1);
            wait_fetches<0>();
#pragma unroll
            for (int st = 0; st < 4; ++st) asm volatile("" ::"v"(qf[0][st]));
            if (FUSED) asm volatile("" ::"v"(new_row.x), "v"(new_row.y), "v"(new_row.z), "v"(new_row.w));
            if (first_key(1) + BLK > kv_len) zero_v_tail(1, 1);          // (the piece's first block is whole: the second holds tokens)
            if (row_block >= 0) patch_new_row(row_block, row_block);
            compute_pair();
        } else if (n_mine > 0) {
            fetch(0, 0);
            if (n_mine > 1) fetch(1, 1);
            for (int i = 0; i < n_mine; ++i) {
                const int slot = i & 1;
                if (i + 1 < n_mine) wait_fetches<FETCHES>(); // the next block's stay on their way
                else wait_fetches<0>();
                // (the query rows, asked for first, have landed as well; used here so that the compiler, which does not
                // count the fetches, has no wait of its own to place inside the loop)
                if (i == 0)
#pragma unroll
                    for (int q = 0; q < NR; ++q)
#pragma unroll
                        for (int st = 0; st < 4; ++st) asm volatile("" ::"v"(qf[q][st]));
                if (FUSED && i == 0) asm volatile("" ::"v"(new_row.x), "v"(new_row.y), "v"(new_row.z), "v"(new_row.w));
                if (first_key(i) + BLK > kv_len) zero_v_tail(i, slot);
                if (i == row_block) patch_new_row(i, slot);
                compute(i, slot);
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");       // every read of the slot is done before it is filled again
                if (i + NSLOT < n_mine) fetch(i + NSLOT, slot);
            }
        }
        // ---- merge 1: the waves' partial results, 16 rows at a time, through LDS
        float* __restrict__ rec =
            unit_mode ? (float*)a.workspace + unit_records_offset(S) + (size_t)(pair * S.pieces_unit + piece) * MAX_ROWS * REC_FLOATS
                      : (float*)a.workspace + (size_t)(pair * S.pieces_max + piece) * MAX_G * REC_FLOATS;
#pragma unroll
        for (int q = 0; q < NR; ++q) {
            if (q > 0) __syncthreads();                      // the pass before has been read
            const int row0 = 16 * q, rows_here = min(MAX_G, n_rows - row0);
            const float l_row = quad_sum(l_run[q]);
            if (l16 < rows_here) {
                float* dst = partial(wave, l16);
#pragma unroll
                for (int nb = 0; nb < 8; ++nb) *(f32x4*)(dst + 16 * nb + 4 * g) = o_acc[q][nb];
                if (g == 0) *(f32x2*)(dst + D) = f32x2{m_run[q], l_row};
            }
            __syncthreads();
            // A wave takes a row and a lane two of its channels, or, with more rows than waves, half a wave and four: up to 8 rows at
            // once.  (Four for all left half of the waves idle over twice the divisions where a KV head has 4 query heads or fewer:
            // 32 / 8 heads, one context of 60 tokens 3.7 us and 3.5.)
            auto combine = [&](auto width_c) {
                constexpr int W = decltype(width_c)::value;  // channels of a lane
                typedef float vec __attribute__((ext_vector_type(W)));
                typedef __bf16 out_vec __attribute__((ext_vector_type(W)));
                for (int lrow = tid / (D / W); lrow < rows_here; lrow += NT / (D / W)) {
                    const int ch = W * (lane & (D / W - 1)), row = row0 + lrow;
                    f32x2 ml[NW];
                    vec x[NW];
#pragma unroll
                    for (int w = 0; w < NW; ++w) {
                        const float* src = partial(w, lrow);
                        ml[w] = *(const f32x2*)(src + D);
                        x[w] = *(const vec*)(src + ch);
                    }
                    float m_all = -INFINITY;
#pragma unroll
                    for (int w = 0; w < NW; ++w) m_all = fmaxf(m_all, ml[w][0]);
                    vec acc = vec(0.f);
                    float l_tot = 0.f;
#pragma unroll
                    for (int w = 0; w < NW; ++w) {
                        const float wgt = (ml[w][0] == -INFINITY) ? 0.f : __builtin_amdgcn_exp2f((ml[w][0] - m_all) * c_log2);
#pragma unroll
                        for (int v = 0; v < W; ++v) acc[v] += wgt * x[w][v];
                        l_tot += wgt * ml[w][1];
                    }
                    if (direct) {
                        const int head = kvh * G + row;
                        out_vec o;
#pragma unroll
                        for (int v = 0; v < W; ++v) o[v] = (__bf16)(l_tot > 0.f ? acc[v] / l_tot : 0.f);
                        *(out_vec*)((__bf16*)a.out + (first_row * b.num_q_heads + head) * D + ch) = o;
                        if (ch == 0 && a.lse != nullptr)
                            a.lse[first_row * b.num_q_heads + head] = (l_tot > 0.f) ? m_all * b.softmax_scale + logf(l_tot) : -INFINITY;
                    } else if (folded) {
#pragma unroll
                        for (int v = 0; v < W; v += 2)
                            if constexpr (W == 2) put_record(rec + row * D + ch + v, f32x2{acc[v], acc[v + 1]});
                        if constexpr (W == 4) put_record4(rec, row * D + ch, acc);
                        if (ch == 0) put_record(rec + MAX_G * D + row * 2, f32x2{m_all, l_tot});
                    } else {
#pragma unroll
                        for (int v = 0; v < W; v += 2) *(f32x2*)(rec + row * REC_FLOATS + ch + v) = f32x2{acc[v], acc[v + 1]};
                        if (ch == 0) *(f32x2*)(rec + row * REC_FLOATS + D) = f32x2{m_all, l_tot};
                    }
                }
            };
            if (rows_here <= NW) combine(std::integral_constant<int, 2>{});
            else combine(std::integral_constant<int, 4>{});
        }
    };

    if (SHARED && unit_mode && n_rows > 16) attend(std::integral_constant<int, 2>{});
    else attend(std::integral_constant<int, 1>{});
    if (!folded) return;

    // ---- merge 2, folded
    const int n = min(n_pieces, S.pieces_max);               // workgroups of this pair that the grid has
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");         // this wave's part of the record is where every XCD sees it
    __syncthreads();
    if (wave == SPEAKER) {
        unsigned long long before = 0;
        if (lane == 0) before = __hip_atomic_fetch_add(count, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const bool last = lane == 0 && (int)(before & ((1 << FOLD_COUNT_BITS) - 1)) + 1 == n;
        if (lane == 0) *(int*)smem = last ? 1 : 0;
        // no ticket, so that the same launch replayed from a graph starts again
        if (last) __hip_atomic_store(count, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();
    if (*(volatile __attribute__((address_space(3))) int*)smem == 0) return;
    const float* rec0 = (const float*)a.workspace + (size_t)pair * S.pieces_max * MAX_G * REC_FLOATS;
    // A wave takes a row and a lane two channels of it, or, with more rows than waves, two rows, half of the lanes each, and a lane four; the weights are made
    // with a lane for each record, of the first row in lanes 0 .. 15, of the second in 16 .. 31, and go to all lanes through LDS.  (A wave has a SIMD to
    // itself here and is bound by the instructions that it issues: with two rows in turn, 7 heads, it was 1.0 us from the count to the records and 1.1 to the
    // result, of 7.2; now 0.85 and 0.75.)  The sums are those of attn_bf16_decode_merge_kernel term by
    // term, its FEW_WAVES partial ones of every fourth piece first: a context's result does not tell which of the two merged it.
    constexpr int ROWS = FOLD_ROWS / NW, PARTS = FEW_WAVES;
    static_assert(ROWS == 2 && ROWS * FOLD_PIECES == 32 && PARTS == 4, "a lane for every weight; the rotations by which partial sums are made");
    if (wave >= G) return;
    auto merge = [&](auto width_c) {
        constexpr int W = decltype(width_c)::value;          // channels of a lane
        typedef float vec __attribute__((ext_vector_type(W)));
        typedef __bf16 out_vec __attribute__((ext_vector_type(W)));
        const int u_lane = lane & (FOLD_PIECES - 1), row_lane = min(wave + (lane / FOLD_PIECES & (ROWS - 1)) * NW, G - 1);
        const f32x2 ml = get_record(rec0 + min(u_lane, n - 1) * (MAX_G * REC_FLOATS) + MAX_G * D + 2 * row_lane);
        const int half = W == 4 ? lane >> 5 : 0, row = wave + NW * half, ch = W * (lane & (D / W - 1));
        const auto records = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(rec0), 0, n * (MAX_G * REC_FLOATS * 4), RAW_BUFFER);
        const int at_row = (min(row, G - 1) * D + ch) * 4;
        vec val[FOLD_PIECES];
#pragma unroll
        for (int u0 = 0; u0 < FOLD_PIECES; u0 += PARTS)
            if (u0 < n)
#pragma unroll
                for (int u = u0; u < u0 + PARTS; ++u) {
                    const int at_piece = min(u, n - 1) * (MAX_G * REC_FLOATS * 4);
                    if constexpr (W == 4) val[u] = __builtin_bit_cast(vec, __builtin_amdgcn_raw_buffer_load_b128(records, at_row, at_piece, AGENT_SCOPE));
                    else val[u] = __builtin_bit_cast(vec, __builtin_amdgcn_raw_buffer_load_b64(records, at_row, at_piece, AGENT_SCOPE));
                }
        const float m = u_lane < n ? ml[0] : -INFINITY, l = u_lane < n ? ml[1] : 0.f;
        float m_part = fmaxf(m, from_lane<4>(m));            // of the pieces that leave the same remainder by 4
        m_part = fmaxf(m_part, from_lane<8>(m_part));
        const float wgt = __builtin_amdgcn_exp2f((m - (m_part == -INFINITY ? 0.f : m_part)) * c_log2);
        float l_part = wgt * l;                              // lanes 0 .. 3 of the row: from the first piece to the last
        l_part = fmaf(from_lane<4>(wgt), from_lane<4>(l), l_part);
        l_part = fmaf(from_lane<8>(wgt), from_lane<8>(l), l_part);
        l_part = fmaf(from_lane<12>(wgt), from_lane<12>(l), l_part);
        float m_all = fmaxf(m_part, from_lane<1>(m_part));
        m_all = fmaxf(m_all, from_lane<2>(m_all));
        const float w_part = m_part == -INFINITY ? 0.f : __builtin_amdgcn_exp2f((m_part - m_all) * c_log2);
        float l_tot = w_part * l_part;                       // lane 0 of the row
        l_tot = fmaf(from_lane<1>(w_part), from_lane<1>(l_part), l_tot);
        l_tot = fmaf(from_lane<2>(w_part), from_lane<2>(l_part), l_tot);
        l_tot = fmaf(from_lane<3>(w_part), from_lane<3>(l_part), l_tot);
        // to every lane what is its row's: the pieces' weights, the partial sums', l and m
        float* own = (float*)smem + 256 + wave * 128;        // (clear of the word that says who is last)
        if (lane < ROWS * FOLD_PIECES) {
            own[lane] = wgt;
            own[32 + lane] = w_part;
            own[64 + lane] = l_tot;
            own[96 + lane] = m_all;
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // the wave's own LDS writes are visible to its own reads
        const f32x4 w_parts = *(const f32x4*)(own + 32 + FOLD_PIECES * half);
        const float l_row = own[64 + FOLD_PIECES * half], m_row = own[96 + FOLD_PIECES * half];
        vec part[PARTS] = {}, acc = vec(0.f);
#pragma unroll
        for (int u0 = 0; u0 < FOLD_PIECES; u0 += PARTS)
            if (u0 < n) {
                const f32x4 w_u = *(const f32x4*)(own + FOLD_PIECES * half + u0);
                if (u0 + PARTS > n)                          // (past the last record its value again: 0, lest it be infinite)
#pragma unroll
                    for (int w = 1; w < PARTS; ++w)
                        if (u0 + w >= n) val[u0 + w] = vec(0.f);
#pragma unroll
                for (int w = 0; w < PARTS; ++w)
#pragma unroll
                    for (int v = 0; v < W; v += 2) {
                        f32x2 p = {part[w][v], part[w][v + 1]};
                        add_weighted(p, w_u[w], f32x2{val[u0 + w][v], val[u0 + w][v + 1]});
                        part[w][v] = p[0];
                        part[w][v + 1] = p[1];
                    }
            }
#pragma unroll
        for (int w = 0; w < PARTS; ++w)
#pragma unroll
            for (int v = 0; v < W; ++v) acc[v] = fmaf(w_parts[w], part[w][v], acc[v]);
        if (row >= G) return;
        const long long at_out = first_row * b.num_q_heads + kvh * G + row;
        out_vec o;
#pragma unroll
        for (int v = 0; v < W; ++v) o[v] = (__bf16)(l_row > 0.f ? acc[v] / l_row : 0.f);
        *(out_vec*)((__bf16*)a.out + at_out * D + ch) = o;
        if (ch == 0 && a.lse != nullptr) a.lse[at_out] = (l_row > 0.f) ? m_row * b.softmax_scale + logf(l_row) : -INFINITY;
    };
    if (G <= NW) merge(std::integral_constant<int, 2>{});
    else merge(std::integral_constant<int, 4>{});
}

// merge 2: one workgroup per (pair, query row); wave w takes pieces w, w + WAVES, ..., a lane two channels of each.
// The kernel is a few microseconds long and bound by its chain of memory round trips, so there is one (AHEAD): every wave
// asks for its first LOADS pieces (a record's 128 values and its m, l) before it knows how many the context has --
// the workspace holds S.pieces_max of them whatever the lengths are -- and drops what turns out not to be a piece.  A
// wave holds the m of all its pieces itself, so weights need no exchange; the waves meet in LDS once.
// Measured against lengths first, then all (m, l), then the values, with two barriers: 4.7 -> 3.1 us for the 12 pieces of
// one request of 1500 tokens, 6.3 -> 5.1 us for 64 requests of 3 pieces (behind a kernel that streams 1 GB).
// Where most of those records are none (short contexts behind a page table that is wide, or of which a few are long) asking
// for them all costs more than the round trip: see AHEAD_BYTES.  The lengths come first then.
// 16 waves when a row has many pieces (a single long context), 4 when it has few (a big batch, where 1024-thread
// workgroups would only crowd the chip).
constexpr int LOADS = 8;                                     // pieces of a wave in flight at a time
inline bool many_pieces(const DecodeShape& S) { return S.pieces_max + (S.n_unit_pairs > 0 ? S.pieces_unit : 0) > MANY_PIECES; }

template <bool CAUSAL, bool SHARED, int WAVES, bool AHEAD>
__global__ __launch_bounds__(64 * WAVES) void attn_bf16_decode_merge_kernel(AttnArgs a, DecodeShape S, SharedPrefixView sv, Divisor by_piece)
{
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    __shared__ f32x2 acc_s[WAVES][D / 2], ml_s[WAVES];
    const BatchView& b = a.b;
    const int G = gridDim.z, row = blockIdx.z, kvh = blockIdx.y, r = blockIdx.x;
    const int pair = r * b.num_kv_heads + kvh;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const float* __restrict__ rec_own = (const float*)a.workspace + ((size_t)pair * S.pieces_max * MAX_G + row) * REC_FLOATS;

    // pieces j0 + wave, j0 + wave + WAVES, ... of a list of records, `stride` floats apart, that holds `room` of them
    struct Asked {
        f32x2 val[LOADS], ml[LOADS];
    } own, of_unit;
    auto ask = [&](Asked& to, const float* __restrict__ rec, size_t stride, int j0, int room) {
#pragma unroll
        for (int u = 0; u < LOADS; ++u) {
            const float* __restrict__ src = rec + (size_t)min(j0 + wave + u * WAVES, room - 1) * stride;
            to.val[u] = *(const f32x2*)(src + 2 * lane);
            to.ml[u] = *(const f32x2*)(src + D);
        }
    };
    const int n_new = b.new_lens[r], prefix_len = b.prefix_lens[r], cu_new = b.cu_new_lens[r];
    const int req_unit = SHARED ? sv.req_unit[r] : -1, req_shared = SHARED ? sv.req_shared_len[r] : 0;
    if (AHEAD) {
        ask(own, rec_own, MAX_G * REC_FLOATS, 0, S.pieces_max);
        __builtin_amdgcn_sched_barrier(0);
        // needed further down only, but asked for here
        asm volatile("" ::"s"(n_new), "s"(cu_new), "s"(by_piece.mul), "s"(a.out), "s"(a.lse));
        if (SHARED) asm volatile("" ::"s"(sv.unit_shared_len), "s"(sv.unit_first_req), "s"(sv.num_units));
    }

    const int P = clamp_prefix_len(b, prefix_len, CAUSAL ? 1 : 0);
    // the records of this row: n_own from the request's own workgroups, then n_unit from its unit's
    // (counts and positions forced into what the workspace holds, whatever the device arrays say)
    const int unit = SHARED ? min(max(req_unit, -1), sv.num_units - 1) : -1;
    const int n_own = min(own_pieces_of(CAUSAL ? P + 1 : P, SHARED ? max(req_shared, 0) / BK : 0, by_piece, unit >= 0),
                          S.pieces_max);
    const bool nothing = n_new <= 0 || (unit < 0 && n_own == 1);          // no query token, or finished by the main kernel
    // (with the loads on their way left only where the result would be stored: a branch here would have them wait behind it)
    if (!AHEAD) {
        if (nothing) return;
        ask(own, rec_own, MAX_G * REC_FLOATS, 0, max(n_own, 1));
    }
    // the unit's first records too, before the first use of any
    int n_unit = 0;
    const float* __restrict__ rec_unit = rec_own;
    if (SHARED && unit >= 0) {
        const int unit_len = sv.unit_shared_len[unit], unit_first = sv.unit_first_req[unit];
        const int shared_len = (int)min((long long)max(unit_len, 0), (long long)b.max_pages * b.page_size) / BK * BK;
        n_unit = shared_len > 0 ? min(up_to_pieces(shared_len / BK, by_piece), S.pieces_unit) : 0;
        const int member = min(max(r - unit_first, 0), MAX_ROWS / G - 1);                  // position of the request in its unit
        rec_unit = (const float*)a.workspace + unit_records_offset(S) +
                   ((size_t)(unit * b.num_kv_heads + kvh) * S.pieces_unit * MAX_ROWS + member * G + row) * REC_FLOATS;
        if (n_unit > 0) ask(of_unit, rec_unit, MAX_ROWS * REC_FLOATS, 0, S.pieces_unit);
    }

    const float c_log2 = b.softmax_scale * 1.44269504088896340736f;
    float m = -INFINITY, l = 0.f;                            // of this wave's pieces (every piece has a visible key)
    f32x2 acc = {0.f, 0.f};
    auto add = [&](Asked& from, int j0, int n) {             // the pieces asked for, those below n
        f32x2 (&val)[LOADS] = from.val, (&ml)[LOADS] = from.ml;
        float m_new = m;
#pragma unroll
        for (int u = 0; u < LOADS; ++u) {
            ml[u][0] = j0 + wave + u * WAVES < n ? ml[u][0] : -INFINITY;
            m_new = fmaxf(m_new, ml[u][0]);
        }
        const float ref = m_new == -INFINITY ? 0.f : m_new;  // no piece of this wave so far: all weights are 0
        const float alpha = __builtin_amdgcn_exp2f((m - ref) * c_log2);
        acc *= alpha;
        m = m_new;
#pragma unroll
        for (int u = 0; u < LOADS; ++u) {
            const bool in = j0 + wave + u * WAVES < n;       // what is no piece may hold anything, infinities and NaN included
            const float wgt = __builtin_amdgcn_exp2f((ml[u][0] - ref) * c_log2);
            l = add_weight(u == 0, l, alpha, wgt, in ? ml[u][1] : 0.f);
            add_weighted(acc, wgt, in ? val[u] : f32x2{0.f, 0.f});
        }
    };
    add(own, 0, n_own);
    for (int j0 = LOADS * WAVES; j0 < n_own; j0 += LOADS * WAVES) {
        ask(own, rec_own, MAX_G * REC_FLOATS, j0, S.pieces_max);
        add(own, j0, n_own);
    }
    if (SHARED && n_unit > 0) {
        add(of_unit, 0, n_unit);
        for (int j0 = LOADS * WAVES; j0 < n_unit; j0 += LOADS * WAVES) {
            ask(of_unit, rec_unit, MAX_ROWS * REC_FLOATS, j0, S.pieces_unit);
            add(of_unit, j0, n_unit);
        }
    }
    acc_s[wave][lane] = acc;
    if (lane == 0) ml_s[wave] = f32x2{m, l};
    __syncthreads();
    if (wave > 0 || nothing) return;
    float m_all = -INFINITY;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) m_all = fmaxf(m_all, ml_s[w][0]);
    float l_tot = 0.f;
    acc = f32x2{0.f, 0.f};
#pragma unroll
    for (int w = 0; w < WAVES; ++w) {
        const f32x2 x = ml_s[w];
        const float wgt = x[0] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f((x[0] - m_all) * c_log2);
        l_tot += wgt * x[1];
        acc += wgt * acc_s[w][lane];
    }
    const long long q_row = clamp_first_row(b, cu_new, 1);
    const int head = kvh * G + row;
    bf16x2 o;
    o[0] = (__bf16)(l_tot > 0.f ? acc[0] / l_tot : 0.f);
    o[1] = (__bf16)(l_tot > 0.f ? acc[1] / l_tot : 0.f);
    *(bf16x2*)((__bf16*)a.out + (q_row * b.num_q_heads + head) * D + 2 * lane) = o;
    if (lane == 0 && a.lse != nullptr)
        a.lse[q_row * b.num_q_heads + head] = (l_tot > 0.f) ? m_all * b.softmax_scale + logf(l_tot) : -INFINITY;
}

// The same where a row has few pieces: a wave takes a row, all its pieces, of the request and of its unit, asked for at once, without LDS and barriers and
// with a quarter of the waves, which is what bounds the kernel above where there are many rows of few pieces.  The sums are those of the four waves above,
// term by term.  Both kernels, four waves for a row and one, us: units of 4 contexts, 40 of 1758 to 2414 tokens in 10 units, 28 / 4 heads, 25.6 and 23.2,
// 36 of 2974 to 3573 in 6, 32 / 8, 32.8 and 29.6, 32 of 18432 in 8 75.3 and 73.8; no units, 64 of 8192 174.5 and 173.4, 32 of 350 to 4600, 32 / 8, 46.3 and 45.8.
// With 16 pieces at once 4 contexts of 1822 to 3574 in one unit take 12.9 instead of 11.2, and 7 of 2078 to 3794 in two (196 rows) with 8 13.5
// instead of 13.3: hence ROW_PIECES and ROW_ROWS.
template <bool CAUSAL, bool SHARED, int PIECES, bool AHEAD>
__global__ __launch_bounds__(64 * FEW_WAVES) void attn_bf16_decode_merge_rows_kernel(AttnArgs a, DecodeShape S, SharedPrefixView sv, Divisor by_piece, Divisor by_heads,
                                                                                     Divisor by_G, int G)
{
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    constexpr int PARTS = FEW_WAVES;
    static_assert(PIECES % PARTS == 0, "every fourth piece");
    const BatchView& b = a.b;
    const int lane = threadIdx.x & 63;
    const int head_row = blockIdx.x * FEW_WAVES + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);      // request * query heads + query head
    const int r = by_heads.quotient(head_row);
    if (r >= b.num_reqs) return;
    const int head = head_row - r * b.num_q_heads;
    const int kvh = by_G.quotient(head), row = head - kvh * G;
    const int pair = r * b.num_kv_heads + kvh;
    const float* __restrict__ rec_own = (const float*)a.workspace + ((size_t)pair * S.pieces_max * MAX_G + row) * REC_FLOATS;
    struct Asked {
        f32x2 val[PIECES], ml[PIECES];
    } own, of_unit;
    auto ask = [&](Asked& to, const float* __restrict__ rec, size_t stride, int room) {
#pragma unroll
        for (int u = 0; u < PIECES; ++u) {
            const float* __restrict__ src = rec + (size_t)min(u, room - 1) * stride;
            to.val[u] = *(const f32x2*)(src + 2 * lane);
            to.ml[u] = *(const f32x2*)(src + D);
        }
    };
    const int n_new = b.new_lens[r], prefix_len = b.prefix_lens[r], cu_new = b.cu_new_lens[r];
    const int req_unit = SHARED ? sv.req_unit[r] : -1, req_shared = SHARED ? sv.req_shared_len[r] : 0;
    if (AHEAD) {
        ask(own, rec_own, MAX_G * REC_FLOATS, S.pieces_max);
        __builtin_amdgcn_sched_barrier(0);
        // needed further down only, but asked for here
        asm volatile("" ::"s"(n_new), "s"(cu_new), "s"(by_piece.mul), "s"(a.out), "s"(a.lse));
        if (SHARED) asm volatile("" ::"s"(sv.unit_shared_len), "s"(sv.unit_first_req), "s"(sv.num_units));
    }
    // the counts, forced into what the workspace holds: as in the kernel above
    const int P = clamp_prefix_len(b, prefix_len, CAUSAL ? 1 : 0);
    const int unit = SHARED ? min(max(req_unit, -1), sv.num_units - 1) : -1;
    const int n_own = min(own_pieces_of(CAUSAL ? P + 1 : P, SHARED ? max(req_shared, 0) / BK : 0, by_piece, unit >= 0),
                          S.pieces_max);
    const bool nothing = n_new <= 0 || (unit < 0 && n_own == 1);          // no query token, or finished by the main kernel
    if (!AHEAD) {
        if (nothing) return;
        ask(own, rec_own, MAX_G * REC_FLOATS, max(n_own, 1));
    }
    int n_unit = 0;
    if (SHARED && unit >= 0) {
        const int unit_len = sv.unit_shared_len[unit], unit_first = sv.unit_first_req[unit];
        const int shared_len = (int)min((long long)max(unit_len, 0), (long long)b.max_pages * b.page_size) / BK * BK;
        n_unit = shared_len > 0 ? min(up_to_pieces(shared_len / BK, by_piece), S.pieces_unit) : 0;
        const int member = min(max(r - unit_first, 0), MAX_ROWS / G - 1);                  // position of the request in its unit
        const float* __restrict__ rec_unit = (const float*)a.workspace + unit_records_offset(S) +
                                             ((size_t)(unit * b.num_kv_heads + kvh) * S.pieces_unit * MAX_ROWS + member * G + row) * REC_FLOATS;
        if (n_unit > 0) ask(of_unit, rec_unit, MAX_ROWS * REC_FLOATS, S.pieces_unit);
    }
    if (nothing) return;

    const float c_log2 = b.softmax_scale * 1.44269504088896340736f;
    float m[PARTS], l[PARTS];                                // of the pieces that leave the same remainder by 4 (every piece has a visible key)
    f32x2 acc[PARTS];
#pragma unroll
    for (int w = 0; w < PARTS; ++w) {
        m[w] = -INFINITY;
        l[w] = 0.f;
        acc[w] = f32x2{0.f, 0.f};
    }
    auto add = [&](const Asked& from, int n) {
#pragma unroll
        for (int w = 0; w < PARTS; ++w) {
            float m_new = m[w];
#pragma unroll
            for (int u = w; u < PIECES; u += PARTS) m_new = fmaxf(m_new, u < n ? from.ml[u][0] : -INFINITY);
            const float ref = m_new == -INFINITY ? 0.f : m_new;          // no piece so far: all weights are 0
            const float alpha = __builtin_amdgcn_exp2f((m[w] - ref) * c_log2);
            acc[w] *= alpha;
            m[w] = m_new;
#pragma unroll
            for (int u = w; u < PIECES; u += PARTS) {
                const bool in = u < n;                       // what is no piece may hold anything, infinities and NaN included
                const float wgt = __builtin_amdgcn_exp2f(((in ? from.ml[u][0] : -INFINITY) - ref) * c_log2);
                l[w] = add_weight(u == w, l[w], alpha, wgt, in ? from.ml[u][1] : 0.f);
                add_weighted(acc[w], wgt, in ? from.val[u] : f32x2{0.f, 0.f});
            }
        }
    };
    add(own, n_own);
    if (SHARED && n_unit > 0) add(of_unit, n_unit);
    float m_all = -INFINITY;
#pragma unroll
    for (int w = 0; w < PARTS; ++w) m_all = fmaxf(m_all, m[w]);
    float l_tot = 0.f;
    f32x2 sum = {0.f, 0.f};
#pragma unroll
    for (int w = 0; w < PARTS; ++w) {
        const float wgt = m[w] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f((m[w] - m_all) * c_log2);
        l_tot = fmaf(wgt, l[w], l_tot);
        sum[0] = fmaf(wgt, acc[w][0], sum[0]);
        sum[1] = fmaf(wgt, acc[w][1], sum[1]);
    }
    const long long at = clamp_first_row(b, cu_new, 1) * (long long)b.num_q_heads + head;
    bf16x2 o;
    o[0] = (__bf16)(l_tot > 0.f ? sum[0] / l_tot : 0.f);
    o[1] = (__bf16)(l_tot > 0.f ? sum[1] / l_tot : 0.f);
    *(bf16x2*)((__bf16*)a.out + at * D + 2 * lane) = o;
    if (lane == 0 && a.lse != nullptr) a.lse[at] = (l_tot > 0.f) ? m_all * b.softmax_scale + logf(l_tot) : -INFINITY;
}

// How a decode batch is cut: the piece length with the least time by a model of the main kernel (times in us, measured).
//   START           from the launch to the first block and from the last block to the end
//   TILE_HBM        one 32-key tile of one KV head (16 KB) at the rate at which the whole chip streams, 6.6 TB/s
//   TILE_CU         the same on one compute unit of a chip that has one piece on each: about 36 bytes per ns, so the longest
//                   piece, twice where a compute unit gets two full ones, bounds the time as well (8 x 18432 tokens: 288
//                   workgroups of 64 tiles 66 us, 448 of 43 53 us, 800 of 24 55 us).  Measured over 66 batches of equal contexts:
//                   .49 us a tile of 192 to 255 workgroups, .78 to .93 of 256 to 447.  Of fewer than 64 it is .26, of 64 to
//                   127 .34; the model has one figure for all
//   two workgroups fit a compute unit, 512 the chip; what does not fit starts when others end, and a last round that is
//   nearly empty lasts as long as a full one: half of its emptiness is charged (608 workgroups of 32 tiles: 58 us)
//   equal contexts are cut evenly: of the lengths that give the same number of pieces the shortest, so that no sliver takes the
//   place of a workgroup with work (64 contexts of 2048 to 8191 tokens behind a table of 256 tiles: 85 + 85 + 85 + 1 133 us, 64 four
//   times 125; where all have 8192 tokens both take 176)
//   MERGE           the second kernel, which a batch cut in single pieces does without (128 contexts of 1000 tokens: 15.7 us
//                   in single pieces, 18.3 in four each), and WORKGROUP what every further piece adds.  (Where the last workgroup merges there is
//                   no second kernel, but the pieces are chosen as if there were: the constants are fitted to two.)
//   PAIR            what pieces of four tiles save beyond their length where each has a compute unit to itself: a wave's two blocks are then
//                   done side by side.  (Contexts told to be equal, plan before and after, us: 28 / 4 heads, 8 of 900 tokens 7.37 and 6.83, with K and V not
//                   in the caches 8.41 and 7.99, 16 of 400 7.07 and 6.32, 8.16 and 7.65, 2 of 3500 7.71 and 7.08; 32 / 8, 5 of 720 7.06 and 6.23, one of
//                   3889 7.46 and 6.85.  A figure of its own for a chip that is half empty, .34 a tile, gained 3 to 10 % on single
//                   pieces of 100 contexts of 500 to 1000 tokens and lost as much on 130 of 3400: not used.)  Contexts of up to 10 tiles are
//                   in one piece or several as without it: 300 tokens in one piece and in three, 32 / 4 heads 5.3 and 5.7, 8 on 40 / 8 5.4 and 5.8, 16 / 8 5.1 and 5.4
// What the host is told (SharedPrefixView) sharpens the plan: `max_own_tiles` / `max_unit_tiles` bound the
// longest own part / shared part and with it the pieces per context that the grid must provide; `planned_tiles` is the
// amount of work there is (32-key tiles per KV head, summed over contexts), by which contexts are known to DIFFER: half a piece
// is then lost per context.  Their workgroups are dealt in the order of the grid, the empty ones among them, so as soon
// as the grid has more than one for every compute unit some of those get two that are long.  (Told by the workgroups that have
// work, that came too late: 25 contexts of 800 to 8000 tokens on 4 KV heads, pieces of 77 tiles, 232 workgroups of a grid of 400,
// 59.6 us, pieces of 41 43.3; 19 of them 48.5, 34.8.  The two constants with _DIFFER are fitted to 189 such batches at 20 piece
// lengths each: the piece taken is 3 % behind the best one, by the constants for equal contexts 8 %.)  32 contexts of 350 to
// 4600 tokens, 8 KV heads, 262 MB: pieces of 48 tiles 48.5 us, of 45 46.7, of 40, which do not fit at once, 49.8.
// Without them the host knows only the longest possible context (the width of the page table) and plans for every context
// being that long.
// Without the amount of work the contexts may differ and may share pages, and both do better in shorter pieces: of the
// lengths within 3 % of the best that fit the chip at once the shortest is taken (8 requests on one video without units:
// pieces of 45 tiles 35 us, of 36 30 us; 40 contexts of 1000 to 4000 tokens: of 63 55 us, of 43 48 us).  And where the
// longest piece bounds the time, not HBM, those of one and a half rounds count as well, up to 12 % more by the model of equal ones
// (22 contexts of 1200 to 4900 tokens, 8 KV heads: of 77 tiles 67 us, of 39 52).  A batch of one request
// is kept to 384 workgroups: its contexts cannot differ (131072 tokens: 48 us, 47 in 256 workgroups, 53 in 512).
// Records are kept to what fits the library's own array (attn_bf16_decode_static_scratch_bytes) wherever longer pieces
// can do that, so that batches do not outgrow it.  A batch that needs more at any length has its pairs fill the chip several times
// over, and is best left to the longest pieces (300 contexts of 4120 tokens on 8 KV heads, 129 tiles: 124 + 5 804 us, 65 + 64 819).
constexpr double START_US = 6.0, TILE_HBM_US = 0.00248, TILE_CU_US = 0.45, MERGE_US = 3.0, WORKGROUP_US = 0.003;
constexpr double TILE_CU_DIFFER_US = 0.42, WORKGROUP_DIFFER_US = 0.004;
constexpr double PAIR_US = 0.5;
constexpr int PAIR_FROM_TILES = 11;
constexpr long long STATIC_RECORDS = (16ll << 20) / (MAX_G * REC_FLOATS * 4);

// The merge kernel asks for records before it knows which of them there are when they are few in all, or when the amount of
// work says that at least half of them are.  (28 / 4 heads, both kernels: 200 contexts of 333 to 500 tokens behind a table of
// 131072 68 us, 89 with all records asked for; 16 of 1000 to 1500 behind a table of that length, 1.9 MB, 15.0 and 14.4.)
constexpr long long AHEAD_BYTES = 2ll << 20;
// Without the amount of work a grid of several rounds is mostly one of a page table wider than the contexts.  Its workgroups without
// work leave on the lengths alone then (64 / 8 heads, 73 contexts of 50 to 500 tokens behind a table of 131072: 50 -> 43 us, 128 of 300 to
// 900 on 32 / 8 heads 99 -> 88); a workgroup with work starts half a microsecond later for it (64 contexts that do have 8192: 177 -> 180).
constexpr long long LATE_GRID = 4 * WORKGROUPS_PER_ROUND;

// Hints never make a plan without units need more records than the same batch without hints, so that a caller may allocate once, by
// the batch alone.  Room is therefore left for the shorter pieces of contexts that are known to differ: what a batch without
// hints reports is at least as many records as the library's own array holds, up to RESERVED_PIECES for a context, and hints
// are planned within that.  (Room for 768 records only: 52 of 87 such batches would get longer pieces, and 5 to 16 % slower for it.)
constexpr int RESERVED_PIECES = 96;

long long table_tiles_of(const BatchView& b) { return ((long long)b.max_pages * b.page_size + BK - 1) / BK; }

// most_allowed: records (own pieces, without units) that the plan may need, unless even the longest pieces need more; us: the plan's time by the model
DecodeShape plan(const BatchView& b, const SharedPrefixView& sv, long long most_allowed, double* us = nullptr)
{
    DecodeShape S;
    S.n_pairs = b.num_reqs * b.num_kv_heads;
    S.n_unit_pairs = sv.num_units * b.num_kv_heads;
    const long long table_tiles = table_tiles_of(b);         // longest possible context
    const long long own_tiles = sv.max_own_tiles > 0 ? std::min<long long>(sv.max_own_tiles, table_tiles) : table_tiles;
    const long long unit_tiles = sv.num_units == 0 ? 0
                                 : sv.max_unit_tiles > 0 ? std::min<long long>(sv.max_unit_tiles, table_tiles) : table_tiles;
    const long long items = (long long)S.n_pairs + S.n_unit_pairs;
    auto pieces = [](long long tiles, int tpp) { return tiles > 0 ? (tiles + tpp - 1) / tpp : 1; };
    const long long most = (long long)S.n_pairs * own_tiles + (long long)S.n_unit_pairs * unit_tiles;
    const long long total = sv.planned_tiles > 0 ? std::min(most, (long long)sv.planned_tiles * b.num_kv_heads) : most;
    const bool known = sv.planned_tiles > 0 && total < most;             // contexts differ
    const long long longest = std::max(own_tiles, unit_tiles);
    const bool one = b.num_reqs == 1 && sv.num_units == 0;
    const bool may_differ = sv.planned_tiles == 0 && sv.num_units == 0 && !one;
    const int at_once = one ? WORKGROUPS_PER_ROUND_ONE_REQUEST : WORKGROUPS_PER_ROUND;
    // the cut into pieces of tpp tiles
    struct Cut {
        int tpp;
        long long own, unit, grid;                           // pieces of the longest own part and of the longest shared part, workgroups
    };
    auto cut_of = [&](int tpp) {
        Cut c = {tpp, pieces(own_tiles, tpp), S.n_unit_pairs > 0 ? pieces(unit_tiles, tpp) : 1, 0};
        c.grid = S.n_pairs * c.own + S.n_unit_pairs * c.unit;
        return c;
    };
    // those of n pieces of a part that are worth counting: not a last one of under a quarter
    auto full = [](long long tiles, long long n, int tpp) { return tiles > 0 && 4 * (tiles - (n - 1) * tpp) <= tpp ? n - 1 : n; };
    // workgroups that have work worth counting
    auto busy_of = [&](const Cut& c) {
        return std::max<long long>(1, known ? std::min(c.grid, (total + c.tpp - 1) / c.tpp + items / 2)
                                            : S.n_pairs * full(own_tiles, c.own, c.tpp) + S.n_unit_pairs * full(unit_tiles, c.unit, c.tpp));
    };
    auto cost_of = [&](const Cut& c) {
        const long long busy = busy_of(c);
        const bool doubled = (known ? c.grid : busy) > WORKGROUPS_PER_ROUND / 2;
        const double piece = std::min<long long>(c.tpp, longest) * (known ? TILE_CU_DIFFER_US : TILE_CU_US);
        double cost = START_US + std::max(total * TILE_HBM_US, piece * (doubled ? 2 : 1));
        const long long last_round = busy % WORKGROUPS_PER_ROUND;
        if (busy > WORKGROUPS_PER_ROUND)
            cost += START_US * 0.25 * (busy / WORKGROUPS_PER_ROUND) +
                    (last_round ? 0.5 * piece * (1.0 - (double)last_round / WORKGROUPS_PER_ROUND) : 0.0);
        if (S.n_unit_pairs > 0 || c.own > 1) cost += MERGE_US;
        if (c.tpp <= PAIR_TILES && own_tiles >= PAIR_FROM_TILES && S.n_unit_pairs == 0 && c.grid <= WORKGROUPS_PER_ROUND / 2) cost -= PAIR_US;
        return cost + (known ? WORKGROUP_DIFFER_US : WORKGROUP_US) * c.grid;
    };
    const int longest_piece = (int)std::max<long long>(MIN_TILES_PER_PIECE, std::min<long long>(MAX_TILES_PER_PIECE, longest));
    int best = longest_piece;
    double least = -1;
    bool best_is_bound_by_its_longest = false;
    Cut next = cut_of(longest_piece);
    for (int tpp = longest_piece; tpp >= MIN_TILES_PER_PIECE; --tpp) {
        const Cut c = next;
        if (tpp > MIN_TILES_PER_PIECE) next = cut_of(tpp - 1);
        if (tpp < longest_piece && ((sv.num_units == 0 && c.grid > STATIC_RECORDS) || (one && c.grid > at_once) || c.grid > most_allowed)) break;
        if (!known && tpp > MIN_TILES_PER_PIECE && next.grid == c.grid) continue;           // the same number of pieces, more alike
        const double cost = cost_of(c);
        // what contexts that may differ are to be taken for the better one at: see above
        const bool at_a_time = c.grid <= at_once, nearly = c.grid <= at_once + at_once / 2 && best_is_bound_by_its_longest;
        // ties: the longer piece, but of contexts that differ the shorter one that fits at once, by which they differ less
        if (least < 0 || cost < least || (known && cost == least && busy_of(c) <= at_once) ||
            (sv.planned_tiles == 0 && ((at_a_time && cost <= 1.03 * least) || (nearly && cost <= 1.12 * least)))) {
            best = tpp;
            best_is_bound_by_its_longest = may_differ && c.grid > WORKGROUPS_PER_ROUND / 2 && 2 * tpp * TILE_CU_US >= 0.9 * total * TILE_HBM_US;
        }
        if (least < 0 || cost < least) least = cost;
    }
    if (us != nullptr) *us = cost_of(cut_of(best));
    S.tiles_per_piece = best;
    S.pieces_max = (int)pieces(own_tiles, best);
    S.pieces_unit = (int)pieces(unit_tiles, best);
    const long long asked = std::min<long long>(S.pieces_max, LOADS * (many_pieces(S) ? MANY_WAVES : FEW_WAVES));      // per row
    const long long grid = (long long)S.n_pairs * S.pieces_max + (long long)S.n_unit_pairs * S.pieces_unit;
    S.ahead = (asked * S.n_pairs * (b.num_q_heads / b.num_kv_heads) * REC_FLOATS * 4 <= AHEAD_BYTES ||
               (sv.planned_tiles > 0 && 2 * std::min(grid, (total + best - 1) / best + items / 2) >= grid)) ? 1 : 0;
    S.late = sv.planned_tiles == 0 && grid > LATE_GRID ? 1 : 0;
    S.stream = total < STREAM_TILES ? DecodeShape::STREAM_NEVER
               : sv.planned_tiles > 0 ? DecodeShape::STREAM_PRIVATE : DecodeShape::STREAM_BY_LENGTHS;
    return S;
}

bool has_hints(const BatchView& b, const SharedPrefixView& sv)
{
    return sv.planned_tiles > 0 || (sv.max_own_tiles > 0 && sv.max_own_tiles < table_tiles_of(b));
}

// Units save reading the shared keys again, but a unit's pieces are longer to compute (two groups of rows), its rows have more records to merge and a
// small batch with units has no folded merge.  Where all there is to read, shared keys once, fits the L2s (8 of 4 MiB), the members after the first find it
// there, and every context by itself is mostly quicker, unless that reads shared keys too often or cuts pieces for contexts that are not there: it is planned with nothing
// known but the two bounds, every context as long as the longest could be, and taken where even that amount is done in less time than the plan of the units.
//   ALONE           from the launch to the end, with the folded merge
//   REREAD          a tile of one KV head out of the caches, by the whole chip; FEW with one or two query heads per KV head, whose units are one group of
//                   rows and quicker than the model has them
// 380 batches of 2 to 65 contexts, 1 to 16 query heads on 1 to 8 KV heads, groups beside private contexts and alone, up to 400 MiB of that amount, both ways, K and V in the
// caches and not: .83 of the time with units in the mean (always one by one .83, the better of both .82), 1.09 at most (1.80).  One by one and units: 3 of 2432 shared tokens, 28 / 4
// heads, 7.7 and 10.5 us, 8 of 1856 in two 7.7 and 11.2; two of 6016 beside 40 of 100 27.3 and 11.6, 32 of 2048 on 8 / 8 heads 18.7 and 12.7.  190 others, with which nothing was
// fitted: .83, 1.07 at most.  By a line on the amount (88 MiB, 64 with one or two heads) .86 and 1.09.  Only where the caller says how much there is and how long the longest parts are.
constexpr long long ALONE_BYTES = 26ll << 20;
constexpr double ALONE_US = 7.0, REREAD_US = 0.0010, REREAD_FEW_US = 0.0013;
constexpr int REREAD_FEW_HEADS = 2;
// us_of_units: of the plan with the units
bool better_alone(const BatchView& b, const SharedPrefixView& sv, double us_of_units)
{
    if (sv.planned_tiles <= 0 || sv.max_own_tiles <= 0 || sv.max_unit_tiles <= 0 || (long long)sv.planned_tiles * b.num_kv_heads * (BK * D * 4) > ALONE_BYTES) return false;
    const double most = ((double)sv.max_own_tiles + sv.max_unit_tiles) * b.num_reqs * b.num_kv_heads;
    return ALONE_US + most * (b.num_q_heads / b.num_kv_heads <= REREAD_FEW_HEADS ? REREAD_FEW_US : REREAD_US) < us_of_units;
}

// pieces of a context that the workspace of the batch without units and hints has room for at least
long long pieces_reserved(const BatchView& b)
{
    const long long n_pairs = std::max<long long>(1, (long long)b.num_reqs * b.num_kv_heads);
    return std::min({(long long)RESERVED_PIECES, STATIC_RECORDS / n_pairs, (table_tiles_of(b) + MIN_TILES_PER_PIECE - 1) / MIN_TILES_PER_PIECE});
}

}  // namespace

DecodeShape attn_bf16_decode_shape(const BatchView& b, const SharedPrefixView& sv, size_t* bytes)
{
    double us = 0;
    const DecodeShape S = plan(b, sv, LLONG_MAX, &us);
    if (sv.num_units > 0) {
        *bytes = attn_bf16_decode_workspace_bytes(S);
        if (!better_alone(b, sv, us)) return S;
        // contexts up to the longest own part behind the longest shared one, within the records that the units would take
        SharedPrefixView alone = {};
        alone.max_own_tiles = (int32_t)std::min<long long>(INT32_MAX, (long long)sv.max_own_tiles + sv.max_unit_tiles);
        const long long room = (long long)S.n_pairs * S.pieces_max + (long long)S.n_unit_pairs * S.pieces_unit * (MAX_ROWS / MAX_G);
        DecodeShape A = plan(b, alone, room);
        if ((long long)A.n_pairs * A.pieces_max > room) return S;
        A.late = S.late;                                     // (by the amount of work, which the plan of its own was not told)
        A.stream = S.stream;
        return A;
    }
    const long long room = !has_hints(b, sv) || S.pieces_max <= pieces_reserved(b) ? LLONG_MAX
                           : std::max<long long>(pieces_reserved(b), plan(b, SharedPrefixView{}, LLONG_MAX).pieces_max);
    const DecodeShape within = S.pieces_max <= room ? S : plan(b, sv, room * S.n_pairs);
    *bytes = attn_bf16_decode_workspace_bytes(within);
    return within;
}

DecodeShape attn_bf16_decode_shape(const BatchView& b, const SharedPrefixView& sv)
{
    size_t bytes = 0;
    return attn_bf16_decode_shape(b, sv, &bytes);
}

bool attn_bf16_decode_applies(const BatchView& b)
{
    return b.max_new_len <= 1 && b.num_q_heads / b.num_kv_heads <= MAX_G;
}

size_t attn_bf16_decode_workspace_bytes(const DecodeShape& S)
{
    return (unit_records_offset(S) + (size_t)S.n_unit_pairs * S.pieces_unit * MAX_ROWS * REC_FLOATS) * sizeof(float);
}

size_t attn_bf16_decode_reserve_bytes(const BatchView& b, const SharedPrefixView& sv)
{
    size_t bytes = 0;
    DecodeShape S = attn_bf16_decode_shape(b, sv, &bytes);
    if (sv.num_units > 0 || has_hints(b, sv)) return bytes;
    S.pieces_max = (int)std::max<long long>(S.pieces_max, pieces_reserved(b));
    return attn_bf16_decode_workspace_bytes(S);
}

namespace {

// Folded where the batch fits the chip at once (grid of at most 512), its pieces are short, so that the second launch is a good part
// of the call, and what the last workgroup has to read is little: it reads all records of its context, through one compute unit, while
// the second kernel has a workgroup for each row.  us of the GPU for two kernels and one:
//   (one: before its last workgroup read 16 bytes a lane; since then 7 heads are .3 to .5 us quicker: one context of 1500 6.7, 4 of 1000 7.0 -> 6.6,
//   8 of 900 8.7 -> 8.1, 16 of 500 8.8 -> 8.3; up to 4 heads as they were or .1)
//   4 pieces    28 / 4 heads, one context of 500 tokens 6.7 and 6.6, 16 of 500 9.0 and 8.6, 32 / 8 heads, 4 of 500 7.0 and 6.5
//   8           32 / 8 heads, 4 of 1500 9.4 and 9.0
//   12          28 / 4, one of 1500 6.7 and 7.2, 4 7.9 and 8.2; 32 / 8, one 6.6 and 6.8; 8 / 8, one 6.4 and 6.4
//   16          28 / 4, one of 2000 6.8 and 7.5, 4 8.7 and 9.3; 32 / 8, one 6.7 and 7.0
//   15 heads on 1: 3 pieces 6.9 and 7.8, 16 7.2 and 9.9
// The host is a launch quicker, and it bounds such calls where they are not replayed from a graph (28 / 4, one of 1500, a call after the
// other: 9.0 and 7.3), so the line lies where one launch takes the GPU half a microsecond more.  Not folded: more than 512
// workgroups (32 of 2000 to 8000, 32 / 8 heads: 119.6 and 121.2) and more than 8 longer pieces (4 of 1500 to 6000: 13.4 and 13.9).
constexpr int FOLD_SHORT = 6, FOLD_READS = 24;               // pieces x rows of a wave
bool fold_applies(const BatchView& b, const DecodeShape& S)
{
    const int G = b.num_q_heads / b.num_kv_heads;
    const int most = S.tiles_per_piece <= FOLD_SHORT ? std::min(FOLD_PIECES, FOLD_READS / ((G + NW - 1) / NW)) : S.tiles_per_piece <= 16 ? FOLD_PIECES / 2 : 0;
    return S.n_unit_pairs == 0 && S.pieces_max > 1 && S.pieces_max <= most && (long long)S.n_pairs * S.pieces_max <= WORKGROUPS_PER_ROUND &&
           G <= FOLD_ROWS;
}

// 48 bits that no other launch of this process has, above FOLD_COUNT_BITS bits of count.  They start from a number that is another in
// every process, so that what an uninitialised workspace holds is a ticket with a chance of 2^-48 only.  Never 0.
unsigned long long next_ticket()
{
    static std::atomic<unsigned long long> next{[] {
        unsigned long long x = (unsigned long long)std::chrono::steady_clock::now().time_since_epoch().count() ^ (unsigned long long)(uintptr_t)&next;
        x = (x ^ (x >> 30)) * 0xbf58476d1ce4e5b9ull;         // the finaliser of splitmix64
        x = (x ^ (x >> 27)) * 0x94d049bb133111ebull;
        return x ^ (x >> 31);
    }()};
    const unsigned long long t = next.fetch_add(1, std::memory_order_relaxed) << FOLD_COUNT_BITS;
    return t != 0 ? t : next.fetch_add(1, std::memory_order_relaxed) << FOLD_COUNT_BITS;
}

template <bool SHARED, bool FUSED>
hipError_t launch_decode(const AttnArgs& a, const SharedPrefixView& sv, const DecodeShape& S, hipStream_t stream)
{
    const BatchView& b = a.b;
    if (b.total_new_tokens == 0 || b.num_reqs == 0) return hipSuccess;
    // the requests' own workgroups first, then (SHARED) those of the units' shared parts
    const long long grid = (long long)S.n_pairs * S.pieces_max + (long long)S.n_unit_pairs * S.pieces_unit;
    if (grid > 0x3fffffff) return hipErrorInvalidValue;
    dim3 dims((unsigned)grid);
    if (!SHARED) {
        dims.x = (unsigned)S.n_pairs;
        dims.z = (unsigned)((S.pieces_max + MAX_GRID_Y - 1) / MAX_GRID_Y);
        dims.y = (unsigned)((S.pieces_max + dims.z - 1) / dims.z);
    }
    const LaunchInfo info = {fold_applies(b, S) ? next_ticket() : 0, b.num_q_heads / b.num_kv_heads, (int32_t)dims.y, divisor_of(b.num_kv_heads), divisor_of(S.tiles_per_piece),
                             SHARED ? divisor_of(S.n_pairs) : Divisor{}, SHARED ? divisor_of(std::max(S.n_unit_pairs, 1)) : Divisor{}};
    if (!a.causal && FUSED) return hipErrorInvalidValue;
    UnitsOf<SHARED> units = {};
    if constexpr (SHARED) units = sv;
    auto attend = [&](auto fold) {
        constexpr bool FOLD = decltype(fold)::value;
        if (a.causal)
            hipLaunchKernelGGL((attn_bf16_decode_kernel<true, SHARED, FUSED, FOLD>), dims, dim3(NT), 0, stream, a, S, info, units);
        else if constexpr (!FUSED)
            hipLaunchKernelGGL((attn_bf16_decode_kernel<false, SHARED, false, FOLD>), dims, dim3(NT), 0, stream, a, S, info, units);
    };
    if (!SHARED && info.ticket != 0) attend(std::integral_constant<bool, !SHARED>{});
    else attend(std::false_type{});
    hipError_t err = hipGetLastError();
    if (err != hipSuccess || info.ticket != 0 || (!SHARED && S.pieces_max == 1)) return err;    // merged, or one piece each: already written
    const dim3 mgrid((unsigned)b.num_reqs, (unsigned)b.num_kv_heads, (unsigned)(b.num_q_heads / b.num_kv_heads));
    auto merge = [&](auto causal, auto waves, auto ahead) {
        hipLaunchKernelGGL((attn_bf16_decode_merge_kernel<decltype(causal)::value, SHARED, decltype(waves)::value, decltype(ahead)::value>), mgrid,
                           dim3(64 * decltype(waves)::value), 0, stream, a, S, sv, info.by_piece);
    };
    // a wave for each row where one can ask for all its pieces at once
    const int most = std::max(S.pieces_max, S.n_unit_pairs > 0 ? S.pieces_unit : 0);
    auto rows = [&](auto causal, auto pieces, auto ahead) {
        const long long waves = (long long)b.num_reqs * b.num_q_heads;
        hipLaunchKernelGGL((attn_bf16_decode_merge_rows_kernel<decltype(causal)::value, SHARED, decltype(pieces)::value, decltype(ahead)::value>),
                           dim3((unsigned)((waves + FEW_WAVES - 1) / FEW_WAVES)), dim3(64 * FEW_WAVES), 0, stream, a, S, sv, info.by_piece,
                           divisor_of(b.num_q_heads), divisor_of(info.G), info.G);
    };
    auto rows_of = [&](auto causal) {
        auto of = [&](auto pieces) {
            if (S.ahead) rows(causal, pieces, std::true_type{});
            else rows(causal, pieces, std::false_type{});
        };
        if (most <= ROW_PIECES / 2) of(std::integral_constant<int, ROW_PIECES / 2>{});
        else of(std::integral_constant<int, ROW_PIECES>{});
    };
    if (most <= ROW_PIECES && (long long)b.num_reqs * b.num_q_heads >= ROW_ROWS) {
        if (a.causal) rows_of(std::true_type{});
        else rows_of(std::false_type{});
        return hipGetLastError();
    }
    auto merge_of = [&](auto causal) {
        using few = std::integral_constant<int, FEW_WAVES>;
        using many = std::integral_constant<int, MANY_WAVES>;
        if (many_pieces(S) && S.ahead) merge(causal, many{}, std::true_type{});
        else if (many_pieces(S)) merge(causal, many{}, std::false_type{});
        else if (S.ahead) merge(causal, few{}, std::true_type{});
        else merge(causal, few{}, std::false_type{});
    };
    if (a.causal) merge_of(std::true_type{});
    else merge_of(std::false_type{});
    return hipGetLastError();
}

}  // namespace

hipError_t launch_attn_bf16_decode(const AttnArgs& a, const SharedPrefixView& sv, const DecodeShape& S, bool fused, hipStream_t stream)
{
    // without units only the bounds matter: the plain kernels, cut by the sharper plan
    // (a shape without unit pairs: the contexts by themselves, see better_alone)
    if (sv.num_units > 0 && S.n_unit_pairs > 0) return fused ? launch_decode<true, true>(a, sv, S, stream) : launch_decode<true, false>(a, sv, S, stream);
    return fused ? launch_decode<false, true>(a, sv, S, stream) : launch_decode<false, false>(a, sv, S, stream);
}

// ---- The same launch for callers that cannot allocate (code under HIP graph capture, serving loops, harnesses
// that forbid hipMalloc): the piece records go to a fixed array in the library's own device image instead of a
// workspace of the caller's.  Every GPU the library runs on holds the array (EMM_DECODE_STATIC_SCRATCH_BYTES) until the
// process ends, at an address of its own, which is looked up once per device with that device current.  In host
// code the array's name is only a handle for that lookup, never a device address: kernels get the looked-up pointer.
namespace {

constexpr size_t STATIC_SCRATCH_BYTES = 16u << 20;
static __device__ __align__(256) unsigned char scratch[STATIC_SCRATCH_BYTES];
constexpr int MAX_DEVICES = 64;
void* scratch_ptr[MAX_DEVICES];                              // per device; nullptr until first use there
std::mutex scratch_lock;

}  // namespace

size_t attn_bf16_decode_static_scratch_bytes() { return STATIC_SCRATCH_BYTES; }

hipError_t launch_attn_bf16_decode_static(AttnArgs a, const DecodeShape& S, hipStream_t stream)
{
    if (attn_bf16_decode_workspace_bytes(S) > STATIC_SCRATCH_BYTES) return hipErrorInvalidValue;
    int dev = -1;
    hipError_t err = hipGetDevice(&dev);
    if (err != hipSuccess) return err;
    if (dev < 0 || dev >= MAX_DEVICES) return hipErrorInvalidDevice;
    void* ptr = nullptr;
    {
        std::lock_guard<std::mutex> guard(scratch_lock);
        if (scratch_ptr[dev] == nullptr) {
            err = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
            if (err != hipSuccess) return err;
            if (ptr == nullptr) return hipErrorInvalidSymbol;
            scratch_ptr[dev] = ptr;
        }
        ptr = scratch_ptr[dev];
    }
    // The kernels write every record they later read, and a count starts from whatever is there (see FOLD_PIECES), so what an
    // earlier call left in the array does not matter.
    a.workspace = ptr;
    return launch_decode<false, false>(a, SharedPrefixView{}, S, stream);
}

}  // namespace emm
