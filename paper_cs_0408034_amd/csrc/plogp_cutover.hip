// gfx950 kernels of the cut-over extraction: each row (table, operation, P)
// of a decision table, read along the message sizes, is compressed into its
// runs of equal decision.  This is the form in which the tuned decisions are
// applied (paper, Section 3.1: above some message size a collective is
// segmented, below it is not; Section 1: one technique per pattern, message
// size and node count).
//
// Integer and index work only; the result is unique, so it must equal the
// plain definition bit for bit.
//
// Three steps, all bound by HBM traffic:
//   k_cut_mark  one thread per (row, tile of CUT_TM sizes): compares the key of
//               every cell with the key of the cell before it, keeps the start
//               flags of the tile as a bit mask and their count;
//   k_cut_scan1 / k_cut_scan2  exclusive prefix of the counts in (row, tile)
//               order: per workgroup of CUT_SCAN_WG counts, then over the
//               workgroup totals;
//   k_cut_emit  one thread per (row, tile) again: writes a run record for every
//               flagged cell at its place, and the row offsets.
// The decision table is stored [table][operation][m][P] with P fastest, so the
// lanes of a wave run over consecutive P (coalesced) and, when the grid has
// fewer than 64 process counts, over consecutive tiles as well.
//
// Grids of at most CUT_ROWS_MAX_M sizes take two launches instead, which read the table once:
//   k_cut_rows   a workgroup takes 64 or 16 rows, finds their starts and leaves them packed, in the order
//                of the output, in scratch, with the number of them;
//   k_cut_place  adds up the numbers of the groups before and moves the packed starts to their
//                place, as run records.
// A batch whose packed starts would take more than CUT_SCRATCH_MOST goes through them slice by slice.
#include "plogp_internal.hpp"

namespace plogp {
namespace {

typedef unsigned long long u64;

struct CutShape {
    int n_tables, n_ops, n_m, n_P;
    int n_tiles;      // tiles of CUT_TM sizes per row
    int lp;           // lanes of a wave along P: a power of two, at most 64
    int n_pg;         // groups of lp process counts
    long n_items;     // n_tables * n_ops * n_pg * n_tiles * lp threads
};

// Thread -> (row, tile).  Returns false for the padding lanes past n_P.
__device__ __forceinline__ bool cut_item(const CutShape &sh, long item, int &t, int &op, int &pi,
                                         int &tile)
{
    const int pl = (int)(item % sh.lp);
    item /= sh.lp;
    tile = (int)(item % sh.n_tiles);
    item /= sh.n_tiles;
    const int pg = (int)(item % sh.n_pg);
    item /= sh.n_pg;
    op = (int)(item % sh.n_ops);
    t = (int)(item / sh.n_ops);
    pi = pg * sh.lp + pl;
    return pi < sh.n_P;
}

// (s, strategy) of a cell: the second half of its 16-byte record.  STREAM: the table is far
// larger than the caches and every record is read once, so the loads carry the non-temporal
// hint (3 % off the pass over a 2 GB table; on a table that fits the caches the hint costs 24 %).
template <bool STREAM>
__device__ __forceinline__ uint2 cell_key(const plogp_cell_dev *cells, size_t idx)
{
    if (STREAM) {
        typedef unsigned u32x2_t __attribute__((ext_vector_type(2)));
        const u32x2_t k = __builtin_nontemporal_load(reinterpret_cast<const u32x2_t *>(cells) + idx * 2 + 1);
        return make_uint2(k.x, k.y);
    }
    return reinterpret_cast<const uint2 *>(cells)[idx * 2 + 1];
}

template <bool STREAM>
__global__ void __launch_bounds__(256) k_cut_mark(CutShape sh, const plogp_cell_dev *cells, int key_mode,
                                                  uint32_t *counts, uint32_t *flags)
{
    const long item = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (item >= sh.n_items)
        return;
    int t, op, pi, tile;
    if (!cut_item(sh, item, t, op, pi, tile))
        return;
    const int m0 = tile * CUT_TM;
    const int len = sh.n_m - m0 < CUT_TM ? sh.n_m - m0 : CUT_TM;
    const size_t base = ((size_t)(t * sh.n_ops + op) * sh.n_m + m0) * sh.n_P + pi;
    // all keys of the tile and the one before it are fetched before any is compared
    uint2 key[CUT_TM + 1];
    key[0] = m0 > 0 ? cell_key<STREAM>(cells, base - sh.n_P) : make_uint2(0u, 0u);
#pragma unroll
    for (int k = 0; k < CUT_TM; ++k)
        key[k + 1] = k < len ? cell_key<STREAM>(cells, base + (size_t)k * sh.n_P) : make_uint2(0u, 0u);
    uint32_t bits = 0u;
#pragma unroll
    for (int k = 0; k < CUT_TM; ++k) {
        bool differs = key[k + 1].y != key[k].y;              // strategy
        if (key_mode == 1)
            differs = differs || key[k + 1].x != key[k].x;    // and segment size
        if (k < len && (differs || (m0 == 0 && k == 0)))      // the first cell of a row starts a run
            bits |= 1u << k;
    }
    const size_t row = (size_t)(t * sh.n_ops + op) * sh.n_P + pi;
    counts[row * sh.n_tiles + tile] = (uint32_t)__builtin_popcount(bits);
    flags[row * sh.n_tiles + tile] = bits;
}

// Exclusive prefix inside each group of CUT_SCAN_WG counts and the group
// totals.  A thread takes CUT_SCAN_PER consecutive counts.
__global__ void __launch_bounds__(CUT_SCAN_THREADS) k_cut_scan1(const uint32_t *counts, uint32_t *local,
                                                                 size_t n, u64 *group_total)
{
    __shared__ uint32_t wave_sum[CUT_SCAN_THREADS / 64];
    const size_t first = ((size_t)blockIdx.x * CUT_SCAN_THREADS + threadIdx.x) * CUT_SCAN_PER;
    uint32_t v[CUT_SCAN_PER];
    uint32_t sum = 0u;
#pragma unroll
    for (int k = 0; k < CUT_SCAN_PER; ++k) {
        v[k] = first + k < n ? counts[first + k] : 0u;
        sum += v[k];
    }
    // inclusive scan of the thread sums over the wave (log steps through the lanes)
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint32_t inc = sum;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const uint32_t up = (uint32_t)__shfl_up((int)inc, d, 64);
        if (lane >= d)
            inc += up;
    }
    if (lane == 63)
        wave_sum[wave] = inc;
    __syncthreads();
    uint32_t before = 0u, total = 0u;
#pragma unroll
    for (int w = 0; w < CUT_SCAN_THREADS / 64; ++w) {
        before += w < wave ? wave_sum[w] : 0u;
        total += wave_sum[w];
    }
    uint32_t run = before + inc - sum;
#pragma unroll
    for (int k = 0; k < CUT_SCAN_PER; ++k) {
        if (first + k < n)
            local[first + k] = run;
        run += v[k];
    }
    if (threadIdx.x == 0)
        group_total[blockIdx.x] = total;
}

// Exclusive prefix of the group totals (in place), one workgroup; the grand
// total goes to *total_out (the entry after the last row offset).
__global__ void __launch_bounds__(1024) k_cut_scan2(u64 *group_total, size_t n_groups, u64 *total_out)
{
    __shared__ u64 wave_sum[16];
    __shared__ u64 carry_s;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (threadIdx.x == 0)
        carry_s = 0ull;
    __syncthreads();
    for (size_t g0 = 0; g0 < n_groups; g0 += 1024) {
        const size_t i = g0 + threadIdx.x;
        const u64 v = i < n_groups ? group_total[i] : 0ull;
        u64 inc = v;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const u64 up = (u64)__shfl_up((long long)inc, d, 64);
            if (lane >= d)
                inc += up;
        }
        if (lane == 63)
            wave_sum[wave] = inc;
        __syncthreads();
        u64 before = carry_s, all = 0ull;
        for (int w = 0; w < 16; ++w) {
            before += w < wave ? wave_sum[w] : 0ull;
            all += wave_sum[w];
        }
        if (i < n_groups)
            group_total[i] = before + inc - v;
        __syncthreads();
        if (threadIdx.x == 0)
            carry_s += all;
        __syncthreads();
    }
    if (threadIdx.x == 0)
        *total_out = carry_s;
}

struct plogp_run_dev {
    u64 m_from;
    uint32_t s;
    uint32_t strategy;
};

// n_fused > 0: group_before still holds the n_fused (at most CUT_FUSE_MAX) group totals; every
// workgroup forms their exclusive prefix itself in LDS, workgroup 0 also writes the grand
// total to *total_out - one launch fewer for the small jobs, which are bound by launches.
constexpr int CUT_FUSE_MAX = 1024;

__global__ void __launch_bounds__(256) k_cut_emit(CutShape sh, const plogp_cell_dev *cells, const u64 *m,
                                                  const uint32_t *local, const uint32_t *flags,
                                                  const u64 *group_before, u64 *row_offsets,
                                                  plogp_run_dev *runs, u64 capacity, int n_fused,
                                                  u64 *total_out)
{
    __shared__ u64 gpre[CUT_FUSE_MAX];
    __shared__ u64 wsum[4];
    if (n_fused > 0) {
        // four totals per thread, in order; scan over the wave, then over the four waves
        const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
        u64 v[4], sum = 0ull;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int g = (int)threadIdx.x * 4 + k;
            v[k] = g < n_fused ? group_before[g] : 0ull;
            sum += v[k];
        }
        u64 inc = sum;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const u64 up = (u64)__shfl_up((long long)inc, d, 64);
            if (lane >= d)
                inc += up;
        }
        if (lane == 63)
            wsum[wave] = inc;
        __syncthreads();
        u64 before = 0ull, all = 0ull;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            before += w < wave ? wsum[w] : 0ull;
            all += wsum[w];
        }
        u64 run = before + inc - sum;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            gpre[threadIdx.x * 4 + k] = run;
            run += v[k];
        }
        if (blockIdx.x == 0 && threadIdx.x == 0)
            *total_out = all;
        __syncthreads();
    }
    const long item = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (item >= sh.n_items)
        return;
    int t, op, pi, tile;
    if (!cut_item(sh, item, t, op, pi, tile))
        return;
    const size_t row = (size_t)(t * sh.n_ops + op) * sh.n_P + pi;
    const size_t idx = row * sh.n_tiles + tile;
    u64 at = (n_fused > 0 ? gpre[idx / CUT_SCAN_WG] : group_before[idx / CUT_SCAN_WG]) + local[idx];
    if (tile == 0)
        row_offsets[row] = at;
    uint32_t bits = flags[idx];
    const int m0 = tile * CUT_TM;
    const size_t base = ((size_t)(t * sh.n_ops + op) * sh.n_m + m0) * sh.n_P + pi;
    while (bits != 0u) {
        const int k = __builtin_ctz(bits);
        bits &= bits - 1u;
        if (at < capacity) {
            const uint2 key = cell_key<false>(cells, base + (size_t)k * sh.n_P);
            union {
                plogp_run_dev r;
                uint4 v;
            } u;
            u.r.m_from = m[m0 + k];
            u.r.s = key.x;
            u.r.strategy = key.y;
            reinterpret_cast<uint4 *>(runs)[at] = u.v;
        }
        ++at;
    }
}

// ---- one pass over the table, a group of rows to a workgroup ----------------------
//
// A workgroup takes 64 rows, or 16 where there are few, and a thread `seg` sizes of one (a multiple of
// 16): rows along the lanes, then sizes along the rest of the wave and the waves.  Every start goes to a
// pool in LDS with its key and where it was found; once the counts are known the pool leaves in the order
// of the output, whole cache lines at a time.  A group whose starts do not fit leaves the counts only, and
// k_cut_place reads its rows once more.
//
// Nothing waits for another workgroup: 480 000 rows x 256 sizes (1.97 GB) take 335 + 15 us, of which
// the bare read is 318, 6.2 TB/s.  With the place of a group's runs learnt from status words of the
// groups before it, in one launch, a workgroup holds its slot for a trip through the loaded memory
// system per 64 groups looked at: 397 us with 256 rows to a workgroup and records written by the
// thread of their row, 436 with 64 rows and packed records (334 without the look-back), 462 with
// persistent workgroups that look back one group late.  Two or eight waves to a group: 354, 350;
// 16-byte loads 371; eight or 32 keys in flight: 351, 356.
// Small jobs: 254 rows x 256 sizes 9.8 us in groups of 16 rows (11.5 in groups of 64; 13 as mark,
// prefix and emit).
struct CutRowsArgs {
    u64 row0, n_rows;      // the slice: n_rows rows from row0 on; everything but the cells counts from there
    int row_bits;          // log2 of the rows of a group
    int seg, cap;          // sizes of a thread; starts that fit the pool
    uint2 *keys;           // [groups][cap] starts in the order of the output: (s, strategy), ...
    uint16_t *sizes;       // [groups][cap] ... and the index of the size
    uint32_t *row_first;   // [rows] starts of the group before each row
    uint32_t *count;       // [groups]
};

static int cut_rows_lds(int cap, int threads) { return cap * 14 + threads * 4; }
constexpr int CUT_ROWS_STATIC_LDS = 512;      // more than k_cut_rows has beside that

__device__ __forceinline__ u64 wave_sum_u64(u64 v)
{
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1)
        v += (u64)__shfl_xor((long long)v, d, 64);
    return v;
}

template <bool STREAM>
__global__ void __launch_bounds__(64 * CUT_ROWS_MAX_WAVES)
k_cut_rows(CutShape sh, const plogp_cell_dev *cells, int key_mode, CutRowsArgs A)
{
    extern __shared__ __align__(16) char cut_lds[];
    __shared__ unsigned n_pool;
    __shared__ unsigned wave_total[CUT_ROWS_MAX_WAVES];
    const int threads = (int)blockDim.x, n_waves = threads >> 6;
    const int tid = (int)threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int rows = 1 << A.row_bits, parts = threads >> A.row_bits;           // parts: of a row's sizes
    const int my_row = tid & (rows - 1), my_part = tid >> A.row_bits;
    uint2 *key_of = reinterpret_cast<uint2 *>(cut_lds);                        // [cap]
    uint32_t *found = reinterpret_cast<uint32_t *>(key_of + A.cap);            // [cap] thread, its start, its size
    uint32_t *first = found + A.cap;                                           // [threads] starts before (row, part)
    unsigned short *place = reinterpret_cast<unsigned short *>(first + threads);   // [cap] by order of output
    const u64 group = blockIdx.x, row = (group << A.row_bits) + my_row;
    const bool live = row < A.n_rows;
    const u64 rr = A.row0 + (live ? row : A.n_rows - 1);       // padding threads read a valid row
    const size_t base = (size_t)(rr / (u64)sh.n_P) * sh.n_m * sh.n_P + (size_t)(rr % (u64)sh.n_P);
    const int m_lo = my_part * A.seg, m_hi = m_lo + A.seg < sh.n_m ? m_lo + A.seg : sh.n_m;
    uint2 prev = make_uint2(0u, 0u);
    if (m_lo > 0 && m_lo < sh.n_m)
        prev = cell_key<STREAM>(cells, base + (size_t)(m_lo - 1) * sh.n_P);
    if (tid == 0)
        n_pool = 0u;
    __syncthreads();
    unsigned starts = 0;
    // (as often for every lane: its first lane has the wave's lowest sizes)
    const int m_wave = __builtin_amdgcn_readfirstlane(m_lo);
    for (int m0 = m_lo; m_wave + (m0 - m_lo) < sh.n_m && m0 - m_lo < A.seg; m0 += 16) {
        uint2 key[16];                                 // sixteen keys are fetched before any is compared
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            const int mi = m0 + k < sh.n_m ? m0 + k : sh.n_m - 1;
            key[k] = cell_key<STREAM>(cells, base + (size_t)mi * sh.n_P);
        }
        unsigned bits = 0u;
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            const uint2 before = k > 0 ? key[k > 0 ? k - 1 : 0] : prev;
            const bool differs = key[k].y != before.y || (key_mode == 1 && key[k].x != before.x);
            if (m0 + k < m_hi && (differs || m0 + k == 0))
                bits |= 1u << k;
        }
        prev = key[15];
        bits = live ? bits : 0u;
        if (__ballot(bits != 0u) == 0)
            continue;
        const unsigned mine = (unsigned)__builtin_popcount(bits);
        unsigned inc = mine;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const unsigned up = (unsigned)__shfl_up((int)inc, d, 64);
            inc += lane >= d ? up : 0u;
        }
        unsigned at = 0;
        if (lane == 63)
            at = atomicAdd(&n_pool, inc);
        at = (unsigned)__builtin_amdgcn_readlane((int)at, 63) + inc - mine;
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            if ((bits >> k) & 1u) {
                if (at < (unsigned)A.cap) {
                    key_of[at] = key[k];
                    found[at] = (unsigned)tid | starts << 10 | (unsigned)(m0 + k) << 20;
                }
                ++at;
                ++starts;
            }
        }
    }

    // the starts before each (row, part), rows first
    first[my_row * parts + my_part] = starts;
    __syncthreads();
    const unsigned count = first[tid];
    unsigned inc = count;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const unsigned up = (unsigned)__shfl_up((int)inc, d, 64);
        inc += lane >= d ? up : 0u;
    }
    if (lane == 63)
        wave_total[wave] = inc;
    __syncthreads();
    unsigned inside = inc - count, total = 0;
    for (int w = 0; w < n_waves; ++w) {
        inside += w < wave ? wave_total[w] : 0u;
        total += wave_total[w];
    }
    first[tid] = inside;                               // (every thread replaces the entry it read)
    __syncthreads();
    if (tid < rows && live)
        A.row_first[row] = first[tid * parts];
    if (tid == 0)
        A.count[group] = total;
    uint2 *keys = A.keys + group * A.cap;
    if (total > (unsigned)A.cap) {
        // (there are at most two threads to a start that is kept where a group can have more, so they fit)
        reinterpret_cast<uint32_t *>(keys)[tid] = inside;
        return;
    }
    for (unsigned i = (unsigned)tid; i < total; i += (unsigned)threads) {
        const unsigned f = found[i], who = f & 1023u;
        place[first[(who & (unsigned)(rows - 1)) * parts + (who >> A.row_bits)] + ((f >> 10) & 1023u)] = (unsigned short)i;
    }
    __syncthreads();
    for (unsigned d = (unsigned)tid; d < total; d += (unsigned)threads) {
        const unsigned i = place[d];
        keys[d] = key_of[i];
        A.sizes[group * A.cap + d] = (uint16_t)(found[i] >> 20);
    }
}

// `per_wg` groups to a workgroup.  ALONE: no more groups than compute units, so that nothing hides the loads
// of a group with many runs (48 rows x 512 sizes, every cell a run: 17.7 us, 20.4 one by one; 32 000 rows x
// 28 sizes would lose 1 us of 12 to the registers this takes).  local, before: the prefix of the counts in
// two levels, or null: then the workgroup adds up the counts before its first group itself.  The number of
// runs in the slices before is what the one before left in row_offsets[0]; this one writes it there again.
template <bool ALONE>
__global__ void __launch_bounds__(256) k_cut_place(CutShape sh, const plogp_cell_dev *cells, const u64 *m, int key_mode,
                                                   CutRowsArgs A, unsigned n_groups, int parts, int per_wg,
                                                   const uint32_t *local, const u64 *before_of, u64 *row_offsets,
                                                   plogp_run_dev *runs, u64 capacity)
{
    __shared__ u64 size_of[CUT_ROWS_MAX_M];
    __shared__ u64 wave_sum[4];
    const int tid = (int)threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const unsigned g0 = blockIdx.x * (unsigned)per_wg;
    for (int i = tid; i < sh.n_m; i += 256)
        size_of[i] = m[i];
    u64 acc = 0;
    if (local == nullptr) {
#pragma unroll 8
        for (unsigned g = (unsigned)tid; g < g0; g += 256)
            acc += A.count[g];
        acc = wave_sum_u64(acc);
    }
    if (lane == 0)
        wave_sum[wave] = acc;
    __syncthreads();
    u64 before = local == nullptr ? wave_sum[0] + wave_sum[1] + wave_sum[2] + wave_sum[3]
                                  : before_of[g0 / CUT_SCAN_WG] + local[g0];
    before += A.row0 > 0 ? row_offsets[0] : 0ull;
    auto emit = [&](u64 at, int mi, const uint2 &key) {
        union {
            plogp_run_dev r;
            uint4 v;
        } u;
        u.r.m_from = size_of[mi];
        u.r.s = key.x;
        u.r.strategy = key.y;
        reinterpret_cast<uint4 *>(runs)[at] = u.v;
    };
    for (unsigned g = g0; g < g0 + (unsigned)per_wg && g < n_groups; ++g) {
        const unsigned total = A.count[g];
        const uint2 *keys = A.keys + (size_t)g * A.cap;
        if (tid < 1 << A.row_bits) {
            const u64 row = ((u64)g << A.row_bits) + tid;
            if (row < A.n_rows)
                row_offsets[row] = before + A.row_first[row];
            if (row == A.n_rows - 1)
                row_offsets[A.n_rows] = before + total;        // the grand total, or the next slice's first
        }
        if (total <= (unsigned)A.cap) {
            const uint16_t *sizes = A.sizes + (size_t)g * A.cap;
            const u64 room = capacity > before ? capacity - before : 0ull;
            const unsigned n = total < room ? total : (unsigned)room;
            unsigned d = (unsigned)tid;
            for (; ALONE && d + 768 < n; d += 1024) {  // four loads before the first store
                uint2 key[4];
                int mi[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    key[u] = keys[d + 256 * u];
                    mi[u] = sizes[d + 256 * u];
                }
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    emit(before + d + 256 * u, mi[u], key[u]);
            }
            for (; d < n; d += 256)
                emit(before + d, sizes[d], keys[d]);
        } else {
            // a (row, part) of k_cut_rows to a thread: its sizes are read again
            for (int t = tid; t < parts << A.row_bits; t += 256) {
                const u64 row = ((u64)g << A.row_bits) + t / parts, rr = A.row0 + row;
                if (row >= A.n_rows)
                    continue;
                const size_t base = (size_t)(rr / (u64)sh.n_P) * sh.n_m * sh.n_P + (size_t)(rr % (u64)sh.n_P);
                const int m_lo = t % parts * A.seg, m_hi = m_lo + A.seg < sh.n_m ? m_lo + A.seg : sh.n_m;
                u64 at = before + reinterpret_cast<const uint32_t *>(keys)[t];
                uint2 prev = make_uint2(0u, 0u);
                if (m_lo > 0 && m_lo < sh.n_m)
                    prev = cell_key<false>(cells, base + (size_t)(m_lo - 1) * sh.n_P);
                for (int m0 = m_lo; m0 < m_hi; m0 += 8) {
                    uint2 key[8];
#pragma unroll
                    for (int k = 0; k < 8; ++k)
                        key[k] = cell_key<false>(cells, base + (size_t)(m0 + k < m_hi ? m0 + k : m_hi - 1) * sh.n_P);
#pragma unroll
                    for (int k = 0; k < 8; ++k) {
                        const bool differs = key[k].y != prev.y || (key_mode == 1 && key[k].x != prev.x);
                        if (m0 + k < m_hi && (differs || m0 + k == 0)) {
                            if (at < capacity)
                                emit(at, m0 + k, key[k]);
                            ++at;
                        }
                        prev = key[k];
                    }
                }
            }
        }
        before += total;
    }
}

}  // namespace

static bool cutover_by_rows(const DeviceGrid &G) { return G.n_m <= CUT_ROWS_MAX_M; }

// Few rows: groups of 64 would not fill the chip (254 rows x 256 sizes: 10.9 us in groups of 64).
static size_t cut_few_rows() { return (size_t)256 * device_info().n_cu; }

// Starts that are kept.  Tuned tables hold 2 to 8 a row (groups of 64 rows up to 12 on 250 sizes, groups of
// 16 up to 8 on 20 sizes and 41 on 500), but a key that holds the segment size changes far more often where
// the candidates are dense.  A group with more is read again, its records go out a row to a thread, and the
// call takes twice as long: 480 000 rows x 256 sizes with 18 starts a row 868 us read again, 407 kept; 39 a
// row 993 and 551; 19 200 rows x 512 sizes with 77 a row 71 and 38.  Room for them costs little, down to
// three workgroups of four waves per compute unit (480 000 rows x 256 sizes with 6 starts a row: room for 16
// 358.8 us, for 48 359.8; 384 000 x 512 for 16 585, for 80 590).
// Where all groups are on the chip at once they share its LDS, whatever that gives: 96 000 rows x 16 sizes,
// half of the cells starts, 16.6 us (25.7 with room for 6), 48 rows x 512 12.0 (15.5 with room for 64).
CutRowsShape cutover_rows_shape(const DeviceGrid &G, size_t n_rows, size_t entries)
{
    CutRowsShape c;
    const bool few = n_rows < cut_few_rows();
    const size_t n_cu = (size_t)device_info().n_cu;
    c.row_bits = few ? 4 : 6;
    c.groups = (n_rows + (1u << c.row_bits) - 1) >> c.row_bits;
    // 16 sizes to a thread, 64 and more on many long rows
    const int tiles = (G.n_m + 15) / 16, most = few ? 32 : 4, per = (tiles + most - 1) / most;
    const int wave_parts = 64 >> c.row_bits;
    c.seg = 16 * per;
    c.waves = ((tiles + per - 1) / per + wave_parts - 1) / wave_parts;
    c.parts = c.waves * wave_parts;
    const int half = (G.n_m + 1) / 2, quarter = (G.n_m + 3) / 4;
    int row = few ? (half < 12 ? 12 : half < 64 ? half : 64)
                  : (quarter < 6 ? 6 : quarter < 32 ? quarter : 16 + G.n_m / 8);
    if (row > G.n_m) row = G.n_m;
    c.least = row << c.row_bits;
    // (a group more than each has on average, for compute units that get more of them)
    const size_t per_cu = c.groups <= n_cu ? 1 : c.groups / n_cu + 2, share = device_info().lds_per_cu / per_cu;
    const size_t other = CUT_ROWS_STATIC_LDS + (size_t)cut_rows_lds(0, 64 * c.waves);
    if (share > other) {
        const size_t fit = (share - other) / (size_t)cut_rows_lds(1 << c.row_bits, 0);
        if (fit > (size_t)row) row = fit < (size_t)G.n_m ? (int)fit : G.n_m;
    }
    c.cap = row << c.row_bits;
    if (c.groups && (size_t)c.cap > entries / c.groups) c.cap = (int)(entries / c.groups);
    return c;
}

hipError_t cutover_init()
{
    for (const bool stream : {false, true}) {
        const void *k = reinterpret_cast<const void *>(stream ? k_cut_rows<true> : k_cut_rows<false>);
        const hipError_t e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize,
                                                 (int)device_info().lds_per_cu - CUT_ROWS_STATIC_LDS);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

size_t cutover_items(const DeviceGrid &G, int n_tables)
{
    const size_t n_tiles = ((size_t)G.n_m + CUT_TM - 1) / CUT_TM;
    return (size_t)n_tables * G.n_ops * G.n_P * n_tiles;
}

static size_t cut_layout(const DeviceGrid &G, int n_tables, size_t n_rows, size_t most, void *base, CutScratch *C)
{
    size_t at = 0;
    auto take = [&](size_t bytes) {
        const size_t here = at;
        at += (bytes + 255) & ~(size_t)255;
        return reinterpret_cast<void *>(reinterpret_cast<uintptr_t>(base) + here);
    };
    CutScratch c = {};
    c.slice_rows = n_rows;
    const size_t few = n_rows < cut_few_rows() ? n_rows : cut_few_rows();
    // (for either size of group; fewer tables on the same block share out its room for starts)
    size_t counts = (n_rows + 63) / 64;
    if (counts < (few + 15) / 16) counts = (few + 15) / 16;
    if (!cutover_by_rows(G)) counts = cutover_items(G, n_tables);
    c.counts = static_cast<uint32_t *>(take(counts * sizeof(uint32_t)));
    c.local = static_cast<uint32_t *>(take(counts * sizeof(uint32_t)));
    c.group_total = static_cast<uint64_t *>(take((counts + CUT_SCAN_WG - 1) / CUT_SCAN_WG * sizeof(uint64_t)));
    if (cutover_by_rows(G)) {
        const CutRowsShape shape = cutover_rows_shape(G, n_rows, SIZE_MAX);
        constexpr size_t each = sizeof(uint2) + sizeof(uint16_t);
        c.entries = shape.groups * (shape.groups * shape.cap <= most / each ? shape.cap : shape.least);
        c.keys = take(c.entries * sizeof(uint2));
        c.sizes = static_cast<uint16_t *>(take(c.entries * sizeof(uint16_t)));
        c.row_first = static_cast<uint32_t *>(take(n_rows * sizeof(uint32_t)));
    } else {
        c.flags = static_cast<uint32_t *>(take(counts * sizeof(uint32_t)));
    }
    if (C) *C = c;
    return at;
}

size_t cutover_scratch(const DeviceGrid &G, int n_tables, size_t most, void *base, CutScratch *C)
{
    const size_t n_rows = (size_t)n_tables * G.n_ops * G.n_P;
    size_t rows = n_rows;
    if (cutover_by_rows(G)) {
        const size_t all = cut_layout(G, n_tables, n_rows, most, nullptr, nullptr);
        if (all > most) rows = n_rows / (all / (most ? most : 1) + 1) & ~(size_t)63;
        if (rows < CUT_SLICE_LEAST) rows = CUT_SLICE_LEAST;
        if (rows > n_rows) rows = n_rows;
    }
    return cut_layout(G, n_tables, rows, most, base, C);
}

// Rows taken whole: one stage of rows row0 .. row1 - 1.
static hipError_t launch_cut_rows(int stage, const CutShape &sh, const DeviceGrid &G, size_t row0, size_t row1,
                                  const plogp_cell_dev *d_cells, int key_mode, const CutScratch &C,
                                  u64 *d_row_offsets, void *d_runs, u64 capacity, hipStream_t st)
{
    const size_t n_rows = row1 - row0;
    const CutRowsShape shape = cutover_rows_shape(G, n_rows, C.entries);
    const size_t n_wg = shape.groups;
    if (n_wg > 0x7FFFFFFFull) return hipErrorInvalidValue;
    const int threads = 64 * shape.waves;
    CutRowsArgs A;
    A.row0 = row0;
    A.n_rows = n_rows;
    A.row_bits = shape.row_bits;
    A.seg = shape.seg;
    A.cap = shape.cap;
    A.keys = reinterpret_cast<uint2 *>(C.keys);
    A.sizes = C.sizes;
    A.row_first = C.row_first;
    A.count = C.counts;
    const bool own_sums = n_wg <= (size_t)CUT_OWN_SUMS;
    if (stage == 0) {
        const bool stream = n_rows * G.n_m * sizeof(plogp_cell_dev) > ((size_t)256 << 20);
        hipLaunchKernelGGL(stream ? k_cut_rows<true> : k_cut_rows<false>, dim3((unsigned)n_wg), dim3(threads),
                           cut_rows_lds(A.cap, threads), st, sh, d_cells, key_mode, A);
    } else if (stage == 1) {
        if (!own_sums) {
            const size_t n_sums = (n_wg + CUT_SCAN_WG - 1) / CUT_SCAN_WG;
            u64 *sums = reinterpret_cast<u64 *>(C.group_total);
            hipLaunchKernelGGL(k_cut_scan1, dim3((unsigned)n_sums), dim3(CUT_SCAN_THREADS), 0, st, C.counts, C.local,
                               n_wg, sums);
            // (the closing entry, which k_cut_place writes too, with the slices before)
            hipLaunchKernelGGL(k_cut_scan2, dim3(1), dim3(1024), 0, st, sums, n_sums, d_row_offsets + row1);
        }
    } else {
        // four groups of 64 rows to a workgroup; one where few of them have short rows, as four in turn
        // would leave most of the chip idle (96 000 rows x 16 sizes 11.9 us, 14.6 with four; x 6 11.0, 13.5)
        const bool few = shape.row_bits < 6;
        const int per_wg = few || (G.n_m <= 32 && n_wg < (size_t)8 * device_info().n_cu) ? 1 : 4;
        const bool alone = n_wg <= (size_t)device_info().n_cu;
        hipLaunchKernelGGL(alone ? k_cut_place<true> : k_cut_place<false>,
                           dim3((unsigned)((n_wg + per_wg - 1) / per_wg)), dim3(256), 0, st, sh, d_cells,
                           reinterpret_cast<const u64 *>(G.m), key_mode, A, (unsigned)n_wg, shape.parts, per_wg,
                           own_sums ? nullptr : C.local, reinterpret_cast<const u64 *>(C.group_total),
                           d_row_offsets + row0, reinterpret_cast<plogp_run_dev *>(d_runs), capacity);
    }
    return hipGetLastError();
}

hipError_t launch_cutovers_stage(int stage, const DeviceGrid &G, int n_tables, const plogp_cell_dev *d_cells,
                                 int key_mode, const CutScratch &C, uint64_t *d_row_offsets, void *d_runs,
                                 uint64_t capacity, hipStream_t st)
{
    CutShape sh;
    sh.n_tables = n_tables;
    sh.n_ops = G.n_ops;
    sh.n_m = G.n_m;
    sh.n_P = G.n_P;
    sh.n_tiles = (G.n_m + CUT_TM - 1) / CUT_TM;
    int lp = 1;
    while (lp < 64 && lp < G.n_P) lp <<= 1;
    sh.lp = lp;
    sh.n_pg = (G.n_P + lp - 1) / lp;
    sh.n_items = (long)n_tables * G.n_ops * sh.n_pg * sh.n_tiles * lp;
    const size_t n_counts = cutover_items(G, n_tables);
    const size_t n_groups = (n_counts + CUT_SCAN_WG - 1) / CUT_SCAN_WG;
    const size_t n_rows = (size_t)n_tables * G.n_ops * G.n_P;
    // one thread per (row, tile), padded to whole waves along P: must fit one launch
    if ((sh.n_items + 255) / 256 > 0x7FFFFFFFL || n_groups > 0x7FFFFFFFull) return hipErrorInvalidValue;
    const unsigned blocks = (unsigned)((sh.n_items + 255) / 256);
    const bool fuse = n_groups <= (size_t)CUT_FUSE_MAX;     // the prefix of the group totals inside the last step
    if (cutover_by_rows(G)) {
        // the slices before the last go through all stages in the first
        size_t row0 = 0;
        for (; row0 + C.slice_rows < n_rows; row0 += C.slice_rows)
            for (int k = 0; stage == 0 && k < CUT_STAGES; ++k) {
                const hipError_t e = launch_cut_rows(k, sh, G, row0, row0 + C.slice_rows, d_cells, key_mode, C,
                                                     reinterpret_cast<u64 *>(d_row_offsets), d_runs, capacity, st);
                if (e != hipSuccess) return e;
            }
        return launch_cut_rows(stage, sh, G, row0, n_rows, d_cells, key_mode, C,
                               reinterpret_cast<u64 *>(d_row_offsets), d_runs, capacity, st);
    }
    if (stage == 0) {
        // a table beyond the 256 MB of the last-level cache is streamed
        const bool stream = n_counts * CUT_TM * sizeof(plogp_cell_dev) > ((size_t)256 << 20);
        hipLaunchKernelGGL(stream ? k_cut_mark<true> : k_cut_mark<false>, dim3(blocks), dim3(256), 0, st, sh,
                           d_cells, key_mode, C.counts, C.flags);
    } else if (stage == 1) {
        hipLaunchKernelGGL(k_cut_scan1, dim3((unsigned)n_groups), dim3(CUT_SCAN_THREADS), 0, st,
                           C.counts, C.local, n_counts, reinterpret_cast<u64 *>(C.group_total));
        if (!fuse)
            hipLaunchKernelGGL(k_cut_scan2, dim3(1), dim3(1024), 0, st,
                               reinterpret_cast<u64 *>(C.group_total), n_groups,
                               reinterpret_cast<u64 *>(d_row_offsets) + n_rows);
    } else {
        hipLaunchKernelGGL(k_cut_emit, dim3(blocks), dim3(256), 0, st, sh, d_cells,
                           reinterpret_cast<const u64 *>(G.m), C.local, C.flags,
                           reinterpret_cast<const u64 *>(C.group_total),
                           reinterpret_cast<u64 *>(d_row_offsets),
                           reinterpret_cast<plogp_run_dev *>(d_runs), (u64)capacity, fuse ? (int)n_groups : 0,
                           reinterpret_cast<u64 *>(d_row_offsets) + n_rows);
    }
    return hipGetLastError();
}

}  // namespace plogp
