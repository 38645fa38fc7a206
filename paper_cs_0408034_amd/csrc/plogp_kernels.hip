// gfx950 kernels of the pLogP tuning sweep.
//
// Arithmetic contract (what makes the decision table reproducible bit for
// bit): IEEE binary64, no contraction (-ffp-contract=off), a fused
// multiply-add only where __builtin_fma is written, integers (m, s, k, P-1,
// floor/ceil log2 P, j*m, 2^j*m) below 2^53 and therefore exact as doubles.
//
// The models are the rows of the paper's Table 1 (Broadcast) and Table 2
// (Scatter); g() is the measured gap of Section 2 read as piecewise linear.
#include "plogp_internal.hpp"

#include <math.h>

namespace plogp {
namespace {

typedef unsigned long long u64;

// ---------------------------------------------------------------- g()

// Table of one cluster staged in LDS: sizes, gaps, interval slopes.
struct LdsTable {
    const double *x;
    const double *y;
    const double *sl;
    int n;
};

// Index of the last sample with x <= z, 0 if z is below every sample.
__device__ __forceinline__ int last_not_above(const double *x, int n, double z)
{
    int lo = 0, len = n;
    while (len > 1) {
        const int half = len >> 1;
        lo = (x[lo + half] <= z) ? lo + half : lo;
        len -= half;
    }
    return lo;
}

// g(z), Section 2: linear inside the interval that starts at the last sample
// not above z; clamped to the first gap below the first sample; the last
// interval's line continues above the last sample (slope[n-1] = slope[n-2]).
__device__ __forceinline__ double gap_at(const LdsTable &t, double z)
{
    const int i = last_not_above(t.x, t.n, z);
    const double x0 = t.x[0];
    const double zc = z > x0 ? z : x0;
    return __builtin_fma(t.sl[i], zc - t.x[i], t.y[i]);
}

// g() at four points at once: the four searches run side by side, so that the
// LDS latencies of one halving step overlap (the step sequence depends on n only).
__device__ __forceinline__ void gap_at4(const LdsTable &t, const double (&z)[4], double (&g)[4])
{
    int lo[4] = {0, 0, 0, 0};
    int len = t.n;
    while (len > 1) {
        const int half = len >> 1;
        double xv[4];
#pragma unroll
        for (int u = 0; u < 4; ++u)
            xv[u] = t.x[lo[u] + half];
#pragma unroll
        for (int u = 0; u < 4; ++u)
            lo[u] = xv[u] <= z[u] ? lo[u] + half : lo[u];
        len -= half;
    }
    const double x0 = t.x[0];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const double zc = z[u] > x0 ? z[u] : x0;
        g[u] = __builtin_fma(t.sl[lo[u]], zc - t.x[lo[u]], t.y[lo[u]]);
    }
}

__device__ __forceinline__ double interval_slope(const double *x, const double *y, int n, int i)
{
    const int a = i < n - 1 ? i : n - 2;
    const double dy = y[a + 1] - y[a];
    const double dx = x[a + 1] - x[a];
    return dy / dx;
}

// Copies table t (sizes, gaps, slopes) from global memory into LDS.
__device__ __forceinline__ LdsTable stage_table(double *lds, const DeviceTables &T, int t)
{
    const int n = T.n;
    double *x = lds, *y = lds + n, *sl = lds + 2 * n;
    const double *gx = T.x + (size_t)t * n, *gy = T.y + (size_t)t * n;
    const double *gs = T.slope + (size_t)t * n;
    for (int i = threadIdx.x; i < n; i += blockDim.x) {
        x[i] = gx[i];
        y[i] = gy[i];
        sl[i] = gs[i];
    }
    __syncthreads();
    LdsTable tab = {x, y, sl, n};
    return tab;
}

// ---------------------------------------------------------------- integer terms

__device__ __forceinline__ int floor_log2(uint32_t P) { return 31 - __clz((int)P); }
// P >= 1: the bit length of P - 1 (__clz(0) is 32)
__device__ __forceinline__ int ceil_log2(uint32_t P) { return 32 - __clz((int)(P - 1u)); }

// k = ceil(m / s) for integers below 2^53: the rounded quotient of two such
// integers cannot reach or cross an integer it is not equal to (its error is
// below 1/s, the smallest possible distance), so ceil() of it is exact.
__device__ __forceinline__ double segments(u64 m, u64 s) { return ceil((double)m / (double)s); }

// The terms of the segmented rows of Table 1 that depend on (m, s) only:
//   k = ceil(m/s), A = g(s) k, B = g(s) (k-1), C = g(s) + L.
// k comes from one multiplication by the rounded reciprocal of s, which can be
// off by one, and one exact remainder m - k s (an fma) that corrects it.
__device__ __forceinline__ void segment_terms(double md, double sd, double rcp_s, double gs,
                                              double L, double &A, double &B, double &C)
{
    double k = ceil(md * rcp_s);
    const double r = __builtin_fma(-k, sd, md);        // exact: m - k s
    // 1, -1 or 0 (their low words are all 0): two selects and an addition
    k += __hiloint2double(r > 0.0 ? 0x3FF00000 : (r <= -sd ? (int)0xBFF00000 : 0), 0);
    A = gs * k;
    B = gs * (k - 1.0);
    C = gs + L;
}

// Minimum of two doubles that are never NaN: a single v_min_f64 (the builtin
// adds a canonicalising v_max_f64 per operand in IEEE mode).
__device__ __forceinline__ double min_f64(double a, double b)
{
    double r;
    asm("v_min_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}

template <int CTRL, int ROW_MASK>
__device__ __forceinline__ double dpp_move(double v)
{
    int lo = __double2loint(v), hi = __double2hiint(v);
    lo = __builtin_amdgcn_update_dpp(lo, lo, CTRL, ROW_MASK, 0xf, false);
    hi = __builtin_amdgcn_update_dpp(hi, hi, CTRL, ROW_MASK, 0xf, false);
    return __hiloint2double(hi, lo);
}

// Minimum over the 64 lanes of a fully active wave, returned in every lane.
// DPP butterflies inside each row of 16 lanes (quad permutes, half-row and row
// mirrors), then the row broadcasts 15 and 31 fold the four rows into lane 63.
__device__ __forceinline__ double wave_min(double v)
{
    v = min_f64(v, dpp_move<0xB1, 0xf>(v));            // quad_perm [1,0,3,2]
    v = min_f64(v, dpp_move<0x4E, 0xf>(v));            // quad_perm [2,3,0,1]
    v = min_f64(v, dpp_move<0x141, 0xf>(v));           // row_half_mirror
    v = min_f64(v, dpp_move<0x140, 0xf>(v));           // row_mirror
    v = min_f64(v, dpp_move<0x142, 0xa>(v));           // row_bcast:15 into rows 1, 3
    v = min_f64(v, dpp_move<0x143, 0xc>(v));           // row_bcast:31 into rows 2, 3
    const int lo = __builtin_amdgcn_readlane(__double2loint(v), 63);
    const int hi = __builtin_amdgcn_readlane(__double2hiint(v), 63);
    return __hiloint2double(hi, lo);
}

// min_f64(a of one half or of the even rows, of the other half or of the odd rows) of two values at
// once: ROWS = false: the lower lanes get the fold of a over the two halves, the upper ones that of
// b; ROWS = true: even rows of 16 lanes get the fold of a over pairs of rows, odd ones that of b.
// (The compiler keeps the two wait states that these permutes need after a vector instruction, but
// does not see the one inside min_f64's assembly: hence the explicit ones.)
template <bool ROWS>
__device__ __forceinline__ double fold_two(double a, double b)
{
    asm("s_nop 1" : "+v"(a), "+v"(b));
    const auto swap = [](int x, int y) {
        return ROWS ? __builtin_amdgcn_permlane16_swap(x, y, false, false)
                    : __builtin_amdgcn_permlane32_swap(x, y, false, false);
    };
    const auto lo = swap(__double2loint(a), __double2loint(b)), hi = swap(__double2hiint(a), __double2hiint(b));
    return min_f64(__hiloint2double((int)hi[0], (int)lo[0]), __hiloint2double((int)hi[1], (int)lo[1]));
}

// v[p] becomes the minimum of v[p] over the 64 lanes, in every lane, for N values at once: the
// first two steps fold two values into one register pair, which halves the instructions of N
// wave_min one after the other.
template <int N>
__device__ __forceinline__ void wave_min_each(double (&v)[N])
{
    constexpr int N2 = (N + 1) / 2, N4 = (N2 + 1) / 2;
    double half[N2], row[N4];
#pragma unroll
    for (int i = 0; i < N2; ++i)
        half[i] = fold_two<false>(v[2 * i], v[2 * i + 1 < N ? 2 * i + 1 : 2 * i]);
#pragma unroll
    for (int i = 0; i < N4; ++i) {
        double r = fold_two<true>(half[2 * i], half[2 * i + 1 < N2 ? 2 * i + 1 : 2 * i]);
        r = min_f64(r, dpp_move<0xB1, 0xf>(r));            // within each row of 16 lanes
        r = min_f64(r, dpp_move<0x4E, 0xf>(r));
        r = min_f64(r, dpp_move<0x141, 0xf>(r));
        row[i] = min_f64(r, dpp_move<0x140, 0xf>(r));
    }
#pragma unroll
    for (int p = 0; p < N; ++p) {
        const int from = 32 * (p % 2) + 16 * (p / 2 % 2);
        v[p] = __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(row[p / 4]), from),
                                __builtin_amdgcn_readlane(__double2loint(row[p / 4]), from));
    }
}

__device__ __forceinline__ double lane_value(double v, int lane)
{
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), lane),
                            __builtin_amdgcn_readlane(__double2loint(v), lane));
}

// Row 5, min over s of fma(q, C, B), for all q between q_lo and q_hi at once: which of 64 candidates, one per
// lane (lane < nv; elsewhere B = +inf), can be the first to attain the minimum for some q.  Before rounding a
// value is a line in q, so a candidate above another at either end by a margin is above it by that in between:
// the two that are least at the ends leave out nearly all others.  The margin makes it certain after rounding
// too: nothing between the ends is larger than M, the largest magnitude at the ends, the values at the ends and
// in between are each off by up to 2^-53 M, and it is 2^-49 M.  (Values that are not finite stay in.)
// 70 instructions, where a pass over 64 process counts, eight candidates at a time, took 35 for every eight: 1024
// sizes x 1023 process counts, 34 candidates 16.0 -> 13.2 us, x 600, 8 candidates (2000 sizes) 17.0 -> 16.5; 4096
// sizes x 976, 43 candidates (k_sweep_p) the call 126.5 -> 121.  Where the pass is the shorter: row_few, sweep_few.
__device__ __forceinline__ u64 row5_candidates(double C, double B, int nv, double q_lo, double q_hi)
{
    const u64 there = nv >= 64 ? ~0ull : (1ull << nv) - 1ull;
    const double at_lo = __builtin_fma(q_lo, C, B), at_hi = __builtin_fma(q_hi, C, B);
    double least[2] = {at_lo, at_hi};
    wave_min_each<2>(least);
    const int a = __builtin_ctzll(__ballot(at_lo == least[0]) | 1ull << 63);
    const int b = __builtin_ctzll(__ballot(at_hi == least[1]) | 1ull << 63);
    const double a_hi = lane_value(at_hi, a), b_lo = lane_value(at_lo, b);
    const double mine = fmax(fabs(at_lo), fabs(at_hi));
    const double over_a = 0x1p-49 * fmax(mine, fmax(fabs(least[0]), fabs(a_hi)));
    const double over_b = 0x1p-49 * fmax(mine, fmax(fabs(b_lo), fabs(least[1])));
    const bool out = (at_lo - least[0] > over_a && at_hi - a_hi > over_a) ||
                     (at_lo - b_lo > over_b && at_hi - least[1] > over_b);
    return there & ~__ballot(out);
}

// The minimum over the candidates `which`, in ascending order, and the first that attains it.
template <int PPL>
__device__ __forceinline__ void row5_least(double C, double B, u64 which, const double (&q)[PPL],
                                           double (&least)[PPL], int (&at)[PPL])
{
    for (; which != 0; which &= which - 1) {
        const int c = __builtin_ctzll(which);
        const double Cv = lane_value(C, c), Bv = lane_value(B, c);
#pragma unroll
        for (int h = 0; h < PPL; ++h) {
            const double v = __builtin_fma(q[h], Cv, Bv);
            at[h] = v < least[h] ? c : at[h];
            least[h] = min_f64(least[h], v);
        }
    }
}

// The minimum over the first nv, eight per round trip to LDS, and the eight among which it first appeared.  B comes
// from there (the same address in every lane), C from the lane that holds it, which halves the traffic.
template <int PPL>
__device__ __forceinline__ void row5_all(double C, const double *sB, int nv, const double (&q)[PPL], double (&least)[PPL],
                                         int (&at)[PPL])
{
    for (int s0 = 0; s0 < nv; s0 += 8) {
        double Bv[8], Cv[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            Bv[u] = sB[s0 + u];
            Cv[u] = lane_value(C, s0 + u);
        }
#pragma unroll
        for (int h = 0; h < PPL; ++h) {
            double cur = INFINITY;
#pragma unroll
            for (int u = 0; u < 8; ++u)
                cur = min_f64(cur, __builtin_fma(q[h], Cv[u], Bv[u]));
            at[h] = cur < least[h] ? s0 : at[h];
            least[h] = min_f64(least[h], cur);
        }
    }
}

// ---------------------------------------------------------------- slopes (table load)

__global__ void __launch_bounds__(256) k_slopes(DeviceTables T, double *slope_out)
{
    const int t = blockIdx.x, n = T.n;
    const double *x = T.x + (size_t)t * n, *y = T.y + (size_t)t * n;
    for (int i = threadIdx.x; i < n; i += blockDim.x)
        slope_out[(size_t)t * n + i] = interval_slope(x, y, n, i);
}

// The same for tables that come as the argument (448 numbers: a kernel's arguments are 4 KB at most), written out
// beside their slopes.
__global__ void __launch_bounds__(256) k_load_packed(PackedTables packed, double *block, int n, int n_tables)
{
    const int count = n * n_tables, last = 2 * count + n_tables;
    for (int i = threadIdx.x; i < last; i += blockDim.x)
        block[i] = packed.v[i];
    for (int i = threadIdx.x; i < count; i += blockDim.x) {
        const int t = i / n;
        block[last + i] = interval_slope(packed.v + t * n, packed.v + count + t * n, n, i - t * n);
    }
}

// ---------------------------------------------------------------- g() at arbitrary sizes

__global__ void __launch_bounds__(256) k_interp(DeviceTables T, int t, const u64 *z, size_t n,
                                                double *out)
{
    extern __shared__ double lds[];
    const LdsTable tab = stage_table(lds, T, t);
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n)
        out[i] = gap_at(tab, (double)z[i]);
}

// ---------------------------------------------------------------- one strategy at n points

// Every row but the Scatter and Gather chains, which add up to P - 1 gaps per point and have a
// kernel of their own (k_eval_chain).
__global__ void __launch_bounds__(256) k_eval(DeviceTables T, int t, int id, const u64 *dm,
                                              const uint32_t *dP, const u64 *ds, size_t n,
                                              double *out)
{
    extern __shared__ double lds[];
    const LdsTable tab = stage_table(lds, T, t);
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n)
        return;
    const u64 m = dm[i];
    const uint32_t P = dP[i];
    const bool seg = (id == 2 || id == 5 || id == 9);
    const u64 s = seg ? ds[i] : 0;
    const u64 lim = 1ull << 53;
    bool ok = m > 0 && m < lim && P >= 2 && (!seg || (s > 0 && s <= m));
    if (ok && (id == 12 || id == 15))
        ok = m <= ((lim - 1) >> (ceil_log2(P) > 0 ? ceil_log2(P) - 1 : 0));
    if (!ok) {
        out[i] = NAN;
        return;
    }
    const double L = T.L[t];
    const double q = (double)(P - 1), fl = (double)floor_log2(P), cl = (double)ceil_log2(P);
    const double gm = gap_at(tab, (double)m);
    const double g1 = gap_at(tab, 1.0);
    const double R = __builtin_fma(3.0, L, 2.0 * g1);
    double gs = 0.0, k = 0.0;
    if (seg) {
        gs = gap_at(tab, (double)s);
        k = segments(m, s);
    }
    double r;
    switch (id) {
    case 0: case 10: case 13: r = __builtin_fma(q, gm, L); break;
    case 1: r = __builtin_fma(q, gm, R); break;
    case 2: r = __builtin_fma(q, gs * k, L); break;
    case 3: r = q * (gm + L); break;
    case 4: r = q * (gm + R); break;
    case 5: r = __builtin_fma(q, gs + L, gs * (k - 1.0)); break;
    case 6: r = cl * __builtin_fma(2.0, gm, L); break;
    case 7: r = __builtin_fma(fl, gm, cl * L); break;
    case 8: r = __builtin_fma(fl, gm, cl * R); break;
    case 9: r = __builtin_fma(fl, gs * k, cl * L); break;
    case 16: r = 2.0 * __builtin_fma(q, g1, L); break;
    case 17: r = 2.0 * __builtin_fma(fl, g1, cl * L); break;
    default: {
        double sum = 0.0;
        const int c = ceil_log2(P);
        for (int j = 0; j < c; ++j)
            sum = sum + gap_at(tab, (double)(m << j));
        r = __builtin_fma(cl, L, sum);
    } break;
    }
    out[i] = r;
}

// ---------------------------------------------------------------- tune, step 1: per-table and per-m terms

constexpr int TERMS_ROWS = 64;       // rows of (m, s) pairs whose minimum of A is formed together

// An image of a double (no NaN) as an unsigned integer that orders the same way.
__device__ __forceinline__ unsigned long long ordered_bits(double v)
{
    const unsigned long long b = (unsigned long long)__double_as_longlong(v);
    return (b >> 63) ? ~b : b | 0x8000000000000000ull;
}

__device__ __forceinline__ double from_ordered_bits(unsigned long long k)
{
    return __longlong_as_double((long long)((k >> 63) ? k & 0x7FFFFFFFFFFFFFFFull : ~k));
}

// One workgroup per (table, chunk of blockDim items); a lane takes one m and
// one s.  Computes the interval slopes from the raw samples (into LDS, for its
// own lookups), g(m), the number of
// candidates that compete for m and the prefix sums over j of g(2^j m) for its
// rows, g(s) for its candidates and (first table only) the reciprocals 1/s used
// to get k = ceil(m/s) without a division per (m, s); chunk 0 also g(1).  (terms_piece does the same on
// the table as intervals, with the same expressions: what changes here changes there.)
__device__ __forceinline__ void terms_body(const DeviceTables &T, const DeviceGrid &G, const Scratch &S,
                                           int n_chunks, int n_mchunks, int with_pairs, int block_id,
                                           double *lds)
{
    // per table: n_chunks workgroups for the candidates and the (m, s) pairs, then n_mchunks
    // that only do the per-size part (0: the first kind does that part as well); the two
    // parts are about equally long chains of dependent steps, side by side they halve
    const int per_table = n_chunks + n_mchunks;
    const int t = block_id / per_table, c_in = block_id % per_table;
    const bool m_role = c_in >= n_chunks;
    const int chunk = m_role ? c_in - n_chunks : c_in;
    const bool first = chunk == 0 && !m_role;
    const int waves = (int)(blockDim.x >> 6);
    const int n = T.n;
    double *x = lds, *y = lds + n, *sl = lds + 2 * n;
    const double *gx = T.x + (size_t)t * n, *gy = T.y + (size_t)t * n;
    for (int i = threadIdx.x; i < n; i += blockDim.x) {
        x[i] = gx[i];
        y[i] = gy[i];
    }
    __syncthreads();
    for (int i = threadIdx.x; i < n; i += blockDim.x)
        sl[i] = interval_slope(x, y, n, i);
    __syncthreads();
    const LdsTable tab = {x, y, sl, n};
    // for the sweep that runs its lanes over P: g(s) and 1/s of every candidate, for this
    // workgroup's own use below
    const bool pairs = (with_pairs & 1) != 0 && !m_role, stage_s = (with_pairs & 2) != 0;
    double *gs_l = lds + 3 * n, *rcp_l = gs_l + G.n_s;
    double *sd_l = lds + 3 * n + ((with_pairs & 1) ? 2 * G.n_s : 0);   // the candidates (exact as doubles)
    if (pairs || stage_s) {
        for (int si = threadIdx.x; si < G.n_s; si += blockDim.x) {
            const double sd = (double)G.s[si];
            if (pairs) {
                gs_l[si] = gap_at(tab, sd);
                rcp_l[si] = 1.0 / sd;
            }
            if (stage_s)
                sd_l[si] = sd;
        }
        __syncthreads();
    }

    // per message size: g(m), the number of candidates, the prefix of g(2^j m).  Groups
    // of 64 sizes are dealt to the waves of this table's workgroups.
    const int n_mw = (G.n_m + 63) / 64;
    // (wave w of chunk c takes group w * chunks + c first: few groups spread over the
    // workgroups, one wave in each, rather than filling the first of them)
    const int m_chunks = n_mchunks > 0 ? n_mchunks : n_chunks;
    const int m_step = m_chunks * waves;
    const int m_first = n_mchunks > 0 && !m_role ? n_mw : (int)(threadIdx.x >> 6) * m_chunks + chunk;
    for (int mw = m_first; mw < n_mw; mw += m_step) {
        const int mi = mw * 64 + (int)(threadIdx.x & 63);
        if (mi >= G.n_m)
            continue;
        const u64 m = G.m[mi];
        S.gm[(size_t)t * G.n_m + mi] = gap_at(tab, (double)m);
        {                              // candidates s <= min(m, s_cap): the list ascends
            const u64 lim = m < G.s_cap ? m : G.s_cap;
            int lo = 0, hi = G.n_s;
            if (stage_s) {             // from LDS: a step is not a round trip to memory
                const double limd = (double)lim;
                while (lo < hi) {
                    const int mid = (lo + hi) >> 1;
                    if (sd_l[mid] <= limd) lo = mid + 1; else hi = mid;
                }
            } else {
                while (lo < hi) {
                    const int mid = (lo + hi) >> 1;
                    if (G.s[mid] <= lim) lo = mid + 1; else hi = mid;
                }
            }
            if (t == 0)
                S.nv[mi] = lo;
        }
        if (G.need & (1u << 12)) {
            double *o = S.sum2 + ((size_t)t * G.n_m + mi) * (G.cl_max + 1);   // [m][d]
            double acc = 0.0;
            o[0] = 0.0;
            for (int j0 = 0; j0 < G.cl_max; j0 += 4) {
                double z[4], g[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int j = j0 + u < G.cl_max ? j0 + u : G.cl_max - 1;
                    z[u] = (double)(m << j);
                }
                gap_at4(tab, z, g);
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    if (j0 + u < G.cl_max) {
                        acc = acc + g[u];
                        o[j0 + u + 1] = acc;
                    }
                }
            }
        }
    }
    if (first && threadIdx.x == 0)
        S.g1[t] = gap_at(tab, 1.0);
    if (m_role)
        return;
    // per candidate: g(s), 1/s, C = g(s) + L; shared out over the chunks of this table
    const double L = T.L[t];
    for (int s0 = chunk * blockDim.x + (threadIdx.x & ~63u); s0 < G.n_s; s0 += n_chunks * blockDim.x) {
        const int si = s0 + (int)(threadIdx.x & 63u);
        double gs = INFINITY;
        if (si < G.n_s) {
            const double sd = (double)G.s[si];
            gs = gap_at(tab, sd);
            S.gs[(size_t)t * G.n_s + si] = gs;
            if (with_pairs & 1)
                S.segC[(size_t)t * G.n_s + si] = gs + L;
            if (t == 0)
                S.rcp[si] = 1.0 / sd;
        }
        if (with_pairs & 4) {              // for the sweep over s: the least g(s) of 64 consecutive candidates
            gs = wave_min(gs);
            if ((threadIdx.x & 63u) == 0u)
                S.minG[(size_t)t * ((G.n_s + 63) / 64) + s0 / 64] = gs;
        }
    }
    // per (m, s): A = g(s) k and B = g(s)(k-1) for the sweep that runs its lanes over P
    // (there they are wave-uniform), +inf where s does not compete; per m the minimum of A
    // over the candidates (rows 2 and 9 of Table 1 are monotone in A).  A chunk takes whole
    // rows of (m, s) pairs, TERMS_ROWS at a time, and forms the minima in LDS on an
    // order-preserving integer image of the doubles.
    if (pairs) {
        __shared__ unsigned long long amin_l[TERMS_ROWS];
        const int rows = (G.n_m + n_chunks - 1) / n_chunks;        // rows of a chunk
        for (int r0 = chunk * rows; r0 < (chunk + 1) * rows && r0 < G.n_m; r0 += TERMS_ROWS) {
            int nr = (chunk + 1) * rows - r0;
            nr = nr < TERMS_ROWS ? nr : TERMS_ROWS;
            nr = nr < G.n_m - r0 ? nr : G.n_m - r0;
            if ((int)threadIdx.x < TERMS_ROWS)
                amin_l[threadIdx.x] = ordered_bits(INFINITY);
            __syncthreads();
            for (int e = threadIdx.x; e < nr * G.n_s; e += blockDim.x) {
                const int ml = e / G.n_s, si = e % G.n_s;
                const int mi = r0 + ml;
                const u64 m = G.m[mi], sv = G.s[si];
                const u64 lim = m < G.s_cap ? m : G.s_cap;
                double A = INFINITY, B = INFINITY, C;
                if (sv <= lim) {
                    segment_terms((double)m, (double)sv, rcp_l[si], gs_l[si], L, A, B, C);
                    atomicMin(&amin_l[ml], ordered_bits(A));
                }
                const size_t o = ((size_t)t * G.n_m + mi) * G.n_s + si;
                S.segA[o] = A;
                S.segB[o] = B;
            }
            __syncthreads();
            if ((int)threadIdx.x < nr)
                S.amin[(size_t)t * G.n_m + r0 + threadIdx.x] = from_ordered_bits(amin_l[threadIdx.x]);
            __syncthreads();
        }
    }
}

__global__ void __launch_bounds__(256) k_terms(DeviceTables T, DeviceGrid G, Scratch S, int n_chunks,
                                               int n_mchunks, int with_pairs)
{
    extern __shared__ double lds[];
    terms_body(T, G, S, n_chunks, n_mchunks, with_pairs, (int)blockIdx.x, lds);
}

// ---------------------------------------------------------------- tune, step 2: Scatter-chain sum

// sum_{j=1}^{P-1} g(j m) (Table 2, chain row).  One lane per message size.  The
// arguments j*m ascend, so the interval of the table only moves forward: one
// search at the start, then a walk that keeps d = j*m - x_i (exact: integers
// below 2^53) and takes eight terms at a time, each an add, an fma and the
// accumulation; lanes that leave their interval among the eight form those from
// there on once more (walk_terms).  Sizes below the first sample fall into a
// virtual interval of slope 0 and gap y_0 (the clamp).  Emits each block total
// and, for every P of the grid whose P-1 falls inside a block, the running sum at
// that point.

typedef double f64x2 __attribute__((ext_vector_type(2)));

// The table as the chain walk sees it, in LDS, as intervals.  Interval 0 is
// virtual: [0, x_0) with gap y_0 and slope 0 (the clamp below the first
// sample); interval i + 1 starts at sample i; the last one never ends (its
// width is +inf) and starts of +inf follow it.
struct ChainCtx {
    const f64x2 *YS;      // [n + 2] {gap at the start of the interval, slope}
    const double *X;      // [n + 6] interval starts
    const double *W;      // [n + 2] interval widths
    int n;                // samples of the table
    int n_blk;
    size_t n_m;
    const u64 *blk_mask;
    const int *blk_off;
};

// Scratch::blk: [block][m], or, where the totals are turned into their prefix, the sizes of one workgroup
// of that step (k_chain_prefix), or half of them, together: [group of BLK_GROUP sizes][block][m of the group].
constexpr int BLK_GROUP = 8;

struct BlkAt {
    size_t first, stride;      // of block 0, from a block to the next
};

__device__ __forceinline__ BlkAt blk_of(const DeviceGrid &G, int t, int mi)
{
    const size_t table = (size_t)t * G.n_blk * G.n_mu;
    if (!G.blk_is_prefix)
        return {table + mi, (size_t)G.n_mu};
    const int first = mi / BLK_GROUP * BLK_GROUP, width = G.n_mu - first < BLK_GROUP ? G.n_mu - first : BLK_GROUP;
    return {table + (size_t)first * G.n_blk + (mi - first), (size_t)width};
}

// Builds the table as intervals in LDS (4 n + CHAIN_PAD doubles at `lds`).  The caller synchronises.
// The slopes are formed here (the same expression as everywhere) where many tables are staged once
// or twice each, or read (SLOPES) where every workgroup stages the same one, from its cache (one
// point at a table of 64 samples 7.2 us, 7.7 with the divisions; 400 tables of 4096 samples 81 us
// with a third more bytes to read, 73 with the divisions).
constexpr size_t CHAIN_PAD = 14;                                   // entries beside the 4 n of the table

template <bool SLOPES = false>
__device__ __forceinline__ void stage_intervals(ChainCtx &C, double *lds, const DeviceTables &T, int t)
{
    const int n = T.n;
    f64x2 *YS = reinterpret_cast<f64x2 *>(lds);                    // n + 2 entries
    double *X = lds + 2 * (n + 2);                                 // n + 6 entries, +inf from n + 1 on
    double *W = X + (n + 6);                                       // n + 2 entries
    const double *gx = T.x + (size_t)t * n, *gy = T.y + (size_t)t * n, *gs = T.slope + (size_t)t * n;
    for (int i = threadIdx.x; i < n + 6; i += blockDim.x) {
        // interval i starts at sample i - 1; interval 0 is the clamp below the first sample
        const double x0 = i == 0 ? 0.0 : i <= n ? gx[i - 1] : INFINITY;
        X[i] = x0;
        if (i < n + 2) {
            f64x2 ys;
            ys.x = i == 0 ? gy[0] : i <= n ? gy[i - 1] : 0.0;
            ys.y = (i == 0 || i > n) ? 0.0 : SLOPES ? gs[i - 1] : interval_slope(gx, gy, n, i - 1);
            YS[i] = ys;
            W[i] = i < n ? gx[i] - x0 : INFINITY;
        }
    }
    C.YS = YS;
    C.X = X;
    C.W = W;
    C.n = n;
}

// Intervals of U sizes at once: for each the number of samples not above it
// (0 = the virtual interval).  The searches run side by side, so that the LDS
// latencies of one halving step overlap.
template <int U>
__device__ __forceinline__ void chain_locate(const double *X, int n, const double (&z)[U], int (&i)[U])
{
#pragma unroll
    for (int c = 0; c < U; ++c)
        i[c] = 0;
    for (int len = n; len > 1;) {
        const int half = len >> 1;
        double xv[U];
#pragma unroll
        for (int c = 0; c < U; ++c)
            xv[c] = X[1 + i[c] + half];
        // all comparisons first, their results in scalar registers: a select right behind its comparison
        // waits for it (a call of 49 sizes x 26 process counts up to 4096, bound by this, 18.6 and 18.3 us)
        u64 past[U];
#pragma unroll
        for (int c = 0; c < U; ++c) {
            past[c] = __ballot(xv[c] <= z[c]);
            if (U >= 4)
                asm("" : "+s"(past[c]));
        }
#pragma unroll
        for (int c = 0; c < U; ++c)
            i[c] = __builtin_amdgcn_inverse_ballot_w64(past[c]) ? i[c] + half : i[c];
        len -= half;
    }
    const double x_first = X[1];
#pragma unroll
    for (int c = 0; c < U; ++c)
        i[c] += z[c] >= x_first ? 1 : 0;
}

// g at U sizes, each by a search of its own.
template <int U>
__device__ __forceinline__ void gaps_located(const ChainCtx &C, const double (&z)[U], double (&g)[U])
{
    int i[U];
    chain_locate<U>(C.X, C.n, z, i);
#pragma unroll
    for (int c = 0; c < U; ++c) {
        const f64x2 ys = C.YS[i[c]];
        g[c] = __builtin_fma(ys.y, z[c] - C.X[i[c]], ys.x);
    }
}

// Formed again for the lanes that are on: g of the terms of eight that lie at or past `end` (an offset, as d;
// that of the next interval, whose gap and slope ys holds).  d ascends and d[7] >= end in every one of these
// lanes, so that, from the last term down, fewer and fewer are left.  A comparison, a subtraction and an fma
// per term; as selects (the compiler's form) a term costs two more, for both halves of g.
__device__ __forceinline__ void terms_past(const double (&d)[8], double end, f64x2 ys, double (&g)[8])
{
    u64 lanes;
    double e;
    asm volatile("s_mov_b64 %[lanes], exec\n\t"
                 "v_add_f64 %[e], %[d7], -%[end]\n\t"
                 "v_fma_f64 %[g7], %[s], %[e], %[y]\n\t"
#define PLOGP_TERM(k)                                                                                                \
                 "v_cmpx_le_f64_e32 vcc, %[end], %[d" #k "]\n\t"                                                    \
                 "v_add_f64 %[e], %[d" #k "], -%[end]\n\t"                                                          \
                 "v_fma_f64 %[g" #k "], %[s], %[e], %[y]\n\t"
                 PLOGP_TERM(6) PLOGP_TERM(5) PLOGP_TERM(4) PLOGP_TERM(3) PLOGP_TERM(2) PLOGP_TERM(1) PLOGP_TERM(0)
#undef PLOGP_TERM
                 "s_mov_b64 exec, %[lanes]\n\t"
                 "s_nop 4"
                 // (&: a g is written before the last input is read, so that an input of the same value must not
                 // share its registers)
                 : [lanes] "=&s"(lanes), [e] "=&v"(e), [g0] "+&v"(g[0]), [g1] "+&v"(g[1]), [g2] "+&v"(g[2]),
                   [g3] "+&v"(g[3]), [g4] "+&v"(g[4]), [g5] "+&v"(g[5]), [g6] "+&v"(g[6]), [g7] "+&v"(g[7])
                 : [d0] "v"(d[0]), [d1] "v"(d[1]), [d2] "v"(d[2]), [d3] "v"(d[3]), [d4] "v"(d[4]), [d5] "v"(d[5]),
                   [d6] "v"(d[6]), [d7] "v"(d[7]), [end] "v"(end), [y] "v"(ys.x), [s] "v"(ys.y)
                 : "vcc");
}

// Where a lane is in the table: interval, the next term's offset in it (exact: integers below 2^53), its
// width, gap and slope.
struct WalkAt {
    int i;
    double d, w;
    f64x2 ys;
};

__device__ __forceinline__ WalkAt walk_from(const ChainCtx &C, double z)
{
    const double z0[1] = {z};
    int i[1];
    chain_locate<1>(C.X, C.n, z0, i);
    WalkAt at;
    at.i = i[0];
    at.d = z - C.X[i[0]];
    at.w = C.W[i[0]];
    at.ys = C.YS[i[0]];
    return at;
}

// g at the next eight sizes, md apart.  All eight are formed on the line of the interval that the lane is in;
// lanes whose last one lies past its end then form those from there on once more on the next line, and so on.
// Where the sizes of a wave cross an interval every hundred terms, some lane crosses at most of them: a branch
// per term, with the reads of the next interval behind it, cost 8 vector, 4 scalar and 1.3 branch instructions
// a term on average (one table of 4096 samples, 3215 sizes x 65 536 terms), 7.4, 2.9 and 0.5 this way, and 3
// where no lane crosses.
constexpr int WALK_V = 8;
constexpr int WALK_HOPS = 12;        // intervals after which the next is searched for: some may have no term in them

__device__ __forceinline__ void walk_terms(const ChainCtx &C, WalkAt &at, double md, double (&g)[WALK_V])
{
    const double md2 = md + md, md4 = md2 + md2;
    double d[WALK_V];
    d[0] = at.d;
    d[1] = at.d + md;
    d[2] = at.d + md2;
    d[3] = d[1] + md2;
#pragma unroll
    for (int k = 0; k < 4; ++k)
        d[4 + k] = d[k] + md4;
#pragma unroll
    for (int k = 0; k < WALK_V; ++k)
        g[k] = __builtin_fma(at.ys.y, d[k], at.ys.x);
    at.d = d[7] + md;
    if (d[7] >= at.w) {
        double start = 0.0, end = at.w;          // of the interval, as offsets from the first
        int hops = 0;
        do {
            ++at.i;
            double to = end;
            if (hops == WALK_HOPS) {             // to that of the first term not yet in its own
                const double x0 = C.X[at.i] - end;
                double z[1] = {d[7]};
#pragma unroll
                for (int k = 6; k >= 0; --k)
                    z[0] = d[k] >= end ? d[k] : z[0];
                z[0] = x0 + z[0];
                int iz[1];
                chain_locate<1>(C.X, C.n, z, iz);
                at.i = iz[0];
                to = C.X[at.i] - x0;
            } else {
                ++hops;
            }
            at.ys = C.YS[at.i];
            start = to;
            terms_past(d, start, at.ys, g);
            end = start + C.W[at.i];
        } while (d[7] >= end);
        at.d -= start;
        at.w = end - start;
    }
}

// The sum of a block for a lane that is `at` its first term, which moves to that of the next block.  Bit r of
// wanted: the sum before term r goes to *out and on; any: all lanes' wanted or'ed.
__device__ __forceinline__ double walk_block(const ChainCtx &C, WalkAt &at, double md, u64 wanted, u64 any, double *out)
{
    double run = 0.0;
    const double next = __builtin_fma((double)SUM_BLOCK, md, at.d);
    if (__ballot(next - md >= at.w) == 0) {      // no lane leaves its interval: as above the last sample
        double d = at.d;
        int k = 0;
        for (;;) {
            const int hit = any != 0 ? __builtin_ctzll(any) : SUM_BLOCK;
#pragma unroll 1
            for (; k + WALK_V <= hit; k += WALK_V) {
#pragma unroll
                for (int u = 0; u < WALK_V; ++u) {
                    run = run + __builtin_fma(at.ys.y, d, at.ys.x);
                    d += md;
                }
            }
#pragma unroll 1
            for (; k < hit; ++k) {
                run = run + __builtin_fma(at.ys.y, d, at.ys.x);
                d += md;
            }
            if (hit == SUM_BLOCK)
                break;
            if ((wanted >> hit) & 1ull)
                *out++ = run;
            any &= any - 1;
        }
        at.d = next;
        return run;
    }
#pragma unroll 1
    for (int k0 = 0; k0 < SUM_BLOCK; k0 += WALK_V) {
        double g[WALK_V];
        walk_terms(C, at, md, g);
        const unsigned some = (unsigned)(any >> k0) & 0xFFu;
        if (some == 0u) {
#pragma unroll
            for (int k = 0; k < WALK_V; ++k)
                run = run + g[k];
        } else {
            const unsigned mine = (unsigned)(wanted >> k0) & 0xFFu;
#pragma unroll
            for (int k = 0; k < WALK_V; ++k) {
                if ((some >> k) & 1u) {
                    if ((mine >> k) & 1u)
                        *out++ = run;
                }
                run = run + g[k];
            }
        }
    }
    return run;
}

// The tuning's first step (see terms_body) in pieces of a wave, on a table that is there as intervals:
// piece j of workgroup wg of the table; false: it has no more.  sd: the candidates in LDS, or null.
__device__ __forceinline__ bool terms_piece(const ChainCtx &C, const DeviceTables &T, const DeviceGrid &G,
                                            const Scratch &S, int t, int wg, int W, int waves, int terms_mode,
                                            unsigned j, const double *sd)
{
    const int lane = threadIdx.x & 63;
    // 64 message sizes: g(m), the number of candidates, the prefix of g(2^j m)
    const int n_mw = (G.n_m + 63) / 64, my_mw = n_mw > wg ? (n_mw - wg + W - 1) / W : 0;
    if (j < (unsigned)my_mw) {
        const int mi = (wg + (int)j * W) * 64 + lane;
        if (mi < G.n_m) {
            const u64 m = G.m[mi];
            const double z[1] = {(double)m};
            double g[1];
            gaps_located<1>(C, z, g);
            S.gm[(size_t)t * G.n_m + mi] = g[0];
            const u64 lim = m < G.s_cap ? m : G.s_cap;
            int lo = 0, hi = G.n_s;
            if (sd) {                                // from LDS: a step is not a round trip to memory
                const double limd = (double)lim;
                while (lo < hi) {
                    const int mid = (lo + hi) >> 1;
                    if (sd[mid] <= limd) lo = mid + 1; else hi = mid;
                }
            } else {
                while (lo < hi) {
                    const int mid = (lo + hi) >> 1;
                    if (G.s[mid] <= lim) lo = mid + 1; else hi = mid;
                }
            }
            if (t == 0)
                S.nv[mi] = lo;
            if (G.need & (1u << 12)) {
                double *o = S.sum2 + ((size_t)t * G.n_m + mi) * (G.cl_max + 1);   // [m][d]
                double acc = 0.0;
                o[0] = 0.0;
                for (int j0 = 0; j0 < G.cl_max; j0 += 4) {
                    double z4[4], g4[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u)
                        z4[u] = (double)(m << (j0 + u < G.cl_max ? j0 + u : G.cl_max - 1));
                    gaps_located<4>(C, z4, g4);
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        if (j0 + u < G.cl_max) {
                            acc = acc + g4[u];
                            o[j0 + u + 1] = acc;
                        }
                    }
                }
            }
        }
        return true;
    }
    j -= (unsigned)my_mw;
    // 64 candidates: g(s), 1/s, C = g(s) + L; the first of all takes g(1) along
    const double L = T.L[t];
    const int n_sw = G.n_s > 0 ? (G.n_s + 63) / 64 : 1, my_sw = n_sw > wg ? (n_sw - wg + W - 1) / W : 0;
    if (j < (unsigned)my_sw) {
        const int sw = wg + (int)j * W, si = sw * 64 + lane;
        const double s = si < G.n_s ? (double)G.s[si] : 1.0, z[2] = {s, 1.0};
        double g[2];
        gaps_located<2>(C, z, g);
        if (sw == 0 && lane == 0)
            S.g1[t] = g[1];
        if (si < G.n_s) {
            S.gs[(size_t)t * G.n_s + si] = g[0];
            if (terms_mode & 1)
                S.segC[(size_t)t * G.n_s + si] = g[0] + L;
            if (t == 0)
                S.rcp[si] = 1.0 / s;
        }
        if (terms_mode & 4) {              // for the sweep over s: the least g(s) of 64 consecutive candidates
            const double least = wave_min(si < G.n_s ? g[0] : INFINITY);
            if (lane == 0 && G.n_s > 0)
                S.minG[(size_t)t * n_sw + sw] = least;
        }
        return true;
    }
    j -= (unsigned)my_sw;
    // some rows of (m, s) pairs: A = g(s) k and B = g(s)(k-1), +inf where s does not compete, min A
    const int rows = (G.n_m + W - 1) / W, r_end = (wg + 1) * rows < G.n_m ? (wg + 1) * rows : G.n_m;
    const int per = (rows + waves - 1) / waves, r0 = wg * rows + (int)j * per;
    if ((terms_mode & 1) == 0 || (int)j >= waves || r0 >= r_end)
        return false;
    constexpr int SL = SWEEP_M_MAX_S / 64;
    double s[SL], rcp[SL], gs[SL];
#pragma unroll
    for (int c = 0; c < SL; ++c) {
        if (64 * c < G.n_s) {
            const int si = 64 * c + lane;
            s[c] = si < G.n_s ? (double)G.s[si] : INFINITY;
            const double z[1] = {si < G.n_s ? s[c] : 1.0};
            double g[1];
            gaps_located<1>(C, z, g);
            gs[c] = g[0];
            rcp[c] = 1.0 / z[0];
        }
    }
    for (int mi = r0; mi < r0 + per && mi < r_end; ++mi) {
        const u64 m = G.m[mi];
        const double lim = (double)(m < G.s_cap ? m : G.s_cap);
        const size_t o = ((size_t)t * G.n_m + mi) * G.n_s + lane;
        double least = INFINITY;
#pragma unroll
        for (int c = 0; c < SL; ++c) {
            if (64 * c < G.n_s) {
                double A = INFINITY, B = INFINITY, Cs;
                if (s[c] <= lim) {
                    segment_terms((double)m, s[c], rcp[c], gs[c], L, A, B, Cs);
                    least = min_f64(least, A);
                }
                if (64 * c + lane < G.n_s) {
                    S.segA[o + 64 * c] = A;
                    S.segB[o + 64 * c] = B;
                }
            }
        }
        least = wave_min(least);
        if (lane == 0)
            S.amin[(size_t)t * G.n_m + mi] = least;
    }
    return true;
}

// The same sums for a small job (few samples, about a million terms or fewer), where the
// walk above is bound by the latency of one lane's 64 dependent steps and the chip is
// nearly idle: a workgroup takes one (block, 64 sizes) item at a time; its four waves
// evaluate the 64 x 64 terms side by side, each by a search of its own (the same
// expression, so the same gaps), into LDS; one wave then adds the terms of each size in
// order, leaving the sum before every term in place; all waves write the wanted partial
// sums, a row of the output per store.
constexpr int SMALL_LD = 65;          // row stride of the 64 x 64 tile of terms

__device__ __forceinline__ void chain_small_body(const DeviceTables &T, const DeviceGrid &G,
                                                 const Scratch &S, int wg_per_table, int block_id,
                                                 double *chain_lds)
{
    const int t = block_id / wg_per_table, wg = block_id % wg_per_table;
    const int n = T.n;
    f64x2 *YS = reinterpret_cast<f64x2 *>(chain_lds);              // n + 2 entries
    double *X = chain_lds + 2 * (n + 2);                           // n + 6 entries
    double *gl = X + (n + 6);                                      // 64 rows of SMALL_LD
    const int lane = threadIdx.x & 63, wave = (int)(threadIdx.x >> 6);
    const int n_mu = G.n_mu;
    const int n_mg = (n_mu + 63) / 64;
    const int n_items = G.n_blk * n_mg;
    // the first item's size, block mask and offset are on their way while the table is staged
    u64 m_next = 0, wanted_next = 0;
    int off_next = 0;
    if (wg < n_items) {
        const int mi0 = (wg % n_mg) * 64 + lane;
        m_next = G.mu[mi0 < n_mu ? mi0 : n_mu - 1];
        wanted_next = G.blk_mask[wg / n_mg];
        off_next = G.blk_off[wg / n_mg];
    }
    {
        const double *gx = T.x + (size_t)t * n, *gy = T.y + (size_t)t * n;
        for (int i = threadIdx.x; i < n + 6; i += blockDim.x) {
            X[i] = i == 0 ? 0.0 : i <= n ? gx[i - 1] : INFINITY;
            if (i < n + 2) {
                f64x2 ys;
                ys.x = i == 0 ? gy[0] : i <= n ? gy[i - 1] : 0.0;
                ys.y = (i == 0 || i > n) ? 0.0 : interval_slope(gx, gy, n, i - 1);
                YS[i] = ys;
            }
        }
    }
    __syncthreads();
    for (int item = wg; item < n_items; item += wg_per_table) {
        const int b = item / n_mg, mg = item % n_mg;
        const int mi = mg * 64 + lane;
        const u64 m = m_next, wanted = wanted_next;
        const int off = off_next;
        if (item + wg_per_table < n_items) {
            const int nxt = item + wg_per_table;
            const int mi1 = (nxt % n_mg) * 64 + lane;
            m_next = G.mu[mi1 < n_mu ? mi1 : n_mu - 1];
            wanted_next = G.blk_mask[nxt / n_mg];
            off_next = G.blk_off[nxt / n_mg];
        }
        const u64 j0 = (u64)b * SUM_BLOCK + 1 + (u64)wave * 16;     // this wave's 16 terms
#pragma unroll
        for (int r0 = 0; r0 < 16; r0 += 8) {                        // eight searches side by side
            double z[8];
            int i[8];
#pragma unroll
            for (int c = 0; c < 8; ++c)
                z[c] = (double)((j0 + r0 + c) * m);
            chain_locate<8>(X, n, z, i);
#pragma unroll
            for (int c = 0; c < 8; ++c) {
                const f64x2 ys = YS[i[c]];
                gl[(wave * 16 + r0 + c) * SMALL_LD + lane] = __builtin_fma(ys.y, z[c] - X[i[c]], ys.x);
            }
        }
        __syncthreads();
        if (wave == 0) {
            const BlkAt at_total = blk_of(G, t, mi < n_mu ? mi : 0);
            double run = 0.0;
            for (int r0 = 0; r0 < SUM_BLOCK; r0 += 8) {
                double g[8];
#pragma unroll
                for (int c = 0; c < 8; ++c)
                    g[c] = gl[(r0 + c) * SMALL_LD + lane];
#pragma unroll
                for (int c = 0; c < 8; ++c) {
                    gl[(r0 + c) * SMALL_LD + lane] = run;          // the sum before term r0 + c
                    run = run + g[c];
                }
            }
            if (mi < n_mu && b < G.n_blk - 1)
                S.blk[at_total.first + b * at_total.stride] = run;
        }
        __syncthreads();
        {
            // lane r holds term r's place: bit r of the mask = the sum before term r is wanted
            const bool want = ((wanted >> lane) & 1ull) != 0;
            const int at = off + __popcll(wanted & ((1ull << lane) - 1ull));
            for (int row = wave; row < 64; row += 4) {
                const int mrow = mg * 64 + row;
                if (mrow < n_mu && want)
                    S.part[((size_t)t * n_mu + mrow) * G.n_P + at] = gl[lane * SMALL_LD + row];
            }
        }
        __syncthreads();
    }
}

// ---------------------------------------------------------------- block sums of the chain row, a block per lane

// The points at which the running sum of some lane of the wave is wanted (bit r: after r terms): the
// lanes' masks or'ed together (all lanes active; 24 instructions, where a loop over the different blocks
// of the lanes took a dozen for each).
__device__ __forceinline__ u64 wave_any_wanted(u64 wanted)
{
    auto all = [](int v) {
        v |= __builtin_amdgcn_update_dpp(v, v, 0x111, 0xf, 0xf, false);      // row_shr:1
        v |= __builtin_amdgcn_update_dpp(v, v, 0x112, 0xf, 0xf, false);      // row_shr:2
        v |= __builtin_amdgcn_update_dpp(v, v, 0x114, 0xf, 0xf, false);      // row_shr:4
        v |= __builtin_amdgcn_update_dpp(v, v, 0x118, 0xf, 0xf, false);      // row_shr:8
        v |= __builtin_amdgcn_update_dpp(v, v, 0x142, 0xa, 0xf, false);      // row_bcast:15
        v |= __builtin_amdgcn_update_dpp(v, v, 0x143, 0xc, 0xf, false);      // row_bcast:31
        return (u64)(unsigned)__builtin_amdgcn_readlane(v, 63);
    };
    return all((int)(unsigned)wanted) | all((int)(unsigned)(wanted >> 32)) << 32;
}

// A power of two of intervals, or the whole table, the same in every lane: none enters so many.
__device__ __forceinline__ int wave_reach(const ChainCtx &C, int enters)
{
    int reach = 1;
    while (__ballot(enters >= reach) != 0)
        reach <<= 1;
    return reach < C.n + 2 ? reach : C.n + 2;
}

// That of a block's terms, the first of which is z0 in interval i0.
__device__ __forceinline__ int block_reach(const ChainCtx &C, double z0, double md, int i0)
{
    const double last[1] = {__builtin_fma((double)(SUM_BLOCK - 1), md, z0)};
    int il[1];
    chain_locate<1>(C.X, C.n, last, il);
    return wave_reach(C, il[0] - i0);
}

// From so many intervals on, a power of two, that some lane's block enters, a wave's blocks are searched for, term
// by term, not walked: a walk takes as many turns over its eight terms as some lane enters intervals (1000 sizes x P
// up to 8192 on 4000 samples: all blocks walked 65 us, 50 with this; 16 or 32 make no difference, 64 56).
constexpr int WALK_REACH = 32;

constexpr bool power_of_two(int v) { return v > 0 && (v & (v - 1)) == 0; }
static_assert(power_of_two(WALK_REACH), "compared with what wave_reach gives");

// Addresses in LDS as numbers: a step of a search is then an addition, a read, a comparison and a select.
typedef __attribute__((address_space(3))) const double lds_double;
typedef __attribute__((address_space(3))) const f64x2 lds_f64x2;
__device__ __forceinline__ unsigned lds_address(const double *p) { return (unsigned)(uintptr_t)(lds_double *)p; }
__device__ __forceinline__ double lds_read(unsigned at) { return *(lds_double *)(uintptr_t)at; }

// g(z), z in the interval whose start is at `at`.
__device__ __forceinline__ double gap_in(const ChainCtx &C, unsigned at, double z)
{
    const unsigned ys_at = 2u * at + (lds_address((const double *)C.YS) - 2u * lds_address(C.X));
    const f64x2 ys = *(lds_f64x2 *)(uintptr_t)ys_at;
    return __builtin_fma(ys.y, z - lds_read(at), ys.x);
}

// Where the intervals of V sizes start, which lie in i0 .. i0 + reach - 1 (reach: at most n + 2, the
// same in every lane): the searches run side by side.
template <int V>
__device__ __forceinline__ void starts_within(const ChainCtx &C, int i0, int reach, const double (&z)[V], unsigned (&at)[V])
{
    // from further below where the table ends before i0 + reach (+inf past the last interval)
    const unsigned first = lds_address(C.X + (i0 < C.n + 2 - reach ? i0 : C.n + 2 - reach));
#pragma unroll
    for (int c = 0; c < V; ++c)
        at[c] = first;
    for (int len = reach; len > 1;) {
        const unsigned half = (unsigned)(len >> 1) * 8u;
        double x[V];
#pragma unroll
        for (int c = 0; c < V; ++c)
            x[c] = lds_read(at[c] + half);
#pragma unroll
        for (int c = 0; c < V; ++c)
            at[c] = x[c] <= z[c] ? at[c] + half : at[c];
        len -= len >> 1;
    }
}

// g at V such sizes.
template <int V>
__device__ __forceinline__ void gaps_within(const ChainCtx &C, int i0, int reach, const double (&z)[V], double (&g)[V])
{
    unsigned at[V];
    starts_within<V>(C, i0, reach, z, at);
#pragma unroll
    for (int c = 0; c < V; ++c)
        g[c] = gap_in(C, at[c], z[c]);
}

// g at V ascending sizes, the first not below interval i, which becomes that of the last (it lies below
// i + reach, as above).  Bound by instructions, the search's above all: a step of it is five vector
// instructions and a read of LDS per term, over all the intervals that some lane's block enters.  Of eight
// terms, few enter more than three intervals: then the bounds between these are read once for all eight
// and compared with; else there is a search each, over as many intervals as the eight span in some lane.
// Which of the two is decided for the wave (333 tables of 57 samples x 203 sizes x 37 process counts up to
// 1500: 76.7 us with a search over the whole block's intervals per term, 68.2 so; 100 tables of 120
// samples x 200 sizes: 44.5 and 37.0).
template <int V>
__device__ __forceinline__ void gaps_ascending(const ChainCtx &C, int &i, int reach, const double (&z)[V], double (&g)[V])
{
    const double *X = C.X + i;
    const double x1 = X[1], x2 = X[2], x3 = X[3];
    if (__ballot(z[V - 1] >= X[4]) == 0) {
        const unsigned here = lds_address(X);
        unsigned at[V];
#pragma unroll
        for (int c = 0; c < V; ++c)
            at[c] = here + (z[c] >= x3 ? 24u : z[c] >= x2 ? 16u : z[c] >= x1 ? 8u : 0u);
#pragma unroll
        for (int c = 0; c < V; ++c)
            g[c] = gap_in(C, at[c], z[c]);
        i += (int)((at[V - 1] - here) >> 3);
        return;
    }
    const double last[1] = {z[V - 1]};
    unsigned at[1];
    starts_within<1>(C, i, reach, last, at);
    const int il = (int)((at[0] - lds_address(C.X)) >> 3);
    int span = 4;
    while (__ballot(il - i >= span) != 0)
        span <<= 1;
    gaps_within<V>(C, i, span < reach ? span : reach, z, g);
    i = il;
}

// The same for a block whose terms enter several intervals.
__device__ __forceinline__ double block_search(const ChainCtx &C, int i, int reach, double md, double zb, u64 wanted,
                                               u64 any, double *out)
{
    constexpr int V = 8;
    double run = 0.0;
#pragma unroll 1
    for (int k = 0; k < SUM_BLOCK; k += V) {
        double z[V], g[V];
#pragma unroll
        for (int c = 0; c < V; ++c)
            z[c] = __builtin_fma((double)c, md, zb);
        gaps_ascending<V>(C, i, reach, z, g);
        if (((any >> k) & 0xFFull) != 0) {
#pragma unroll
            for (int c = 0; c < V; ++c) {
                if ((wanted >> (k + c)) & 1ull)
                    *out++ = run;
                run = run + g[c];
            }
        } else {
#pragma unroll
            for (int c = 0; c < V; ++c)
                run = run + g[c];
        }
        zb = __builtin_fma((double)V, md, zb);
    }
    return run;
}

// ---------------------------------------------------------------- chain sums of a big table

// `n` consecutive blocks from block b on, one after the other, for the size m of this lane.  part: this
// size's row of in-block partial sums; tot: its block totals, `stride` apart.
__device__ __forceinline__ void chain_item(const ChainCtx &C, int b, int n, u64 m, double *part, double *tot,
                                           size_t stride)
{
    const double md = (double)m;
    const double ends[2] = {(double)(((u64)b * SUM_BLOCK + 1) * m), (double)(((u64)b * SUM_BLOCK + SUM_BLOCK) * m)};
    int i[2];
    chain_locate<2>(C.X, C.n, ends, i);
    WalkAt at = {i[0], ends[0] - C.X[i[0]], C.W[i[0]], C.YS[i[0]]};
    const int b_end = C.n_blk - b < n ? C.n_blk : b + n;
    if (wave_reach(C, i[1] - i[0]) > WALK_REACH) {
        for (; b < b_end; ++b) {
            const WalkAt from = walk_from(C, (double)(((u64)b * SUM_BLOCK + 1) * m));
            const double z0 = C.X[from.i] + from.d;
            // bit r (wave-uniform): some grid P needs the running sum after r terms
            const u64 wanted = C.blk_mask[b];
            const double run = block_search(C, from.i, block_reach(C, z0, md, from.i), md, z0, wanted, wanted,
                                            part + C.blk_off[b]);
            if (b < C.n_blk - 1)                          // the last block is never complete
                tot[b * stride] = run;
        }
        return;
    }
    for (; b < b_end; ++b) {
        const u64 wanted = C.blk_mask[b];
        const double run = walk_block(C, at, md, wanted, wanted, part + C.blk_off[b]);
        if (b < C.n_blk - 1)
            tot[b * stride] = run;
    }
}

// Work items of one table, in this order: (block b, group of 64 sizes mg) for the
// n_single leading blocks, one block each -- small j, which enter many intervals
// per term, so that an item takes longest -- then (unit u, mg) with CHAIN_U blocks each.  The items are
// dealt to the workgroups of the table in rounds, every other round in reverse
// order, so that every workgroup gets its share of the heavy items and meets
// them first; inside a workgroup the waves take the next item of its list from
// a counter in LDS, because how long an item takes depends on how often its
// sizes cross an interval.
// TERMS: the workgroups do the tuning's first step as well, in pieces of a wave that come after the
// items: chains of dependent steps, which leave the vector units idle, for waves that have nothing left
// while others finish their last item, on the table that is there.  (Behind a barrier, on the table
// staged and its slopes formed once more, they took 5 to 8 us of a call: 4000 samples, 300 sizes x P up
// to 65 536 63.6 us, 57.6 now; 4000 x P up to 4000 51 and 45.6; 4096 sizes x 976 process counts 137.4 and
// 132.1.  A launch of their own takes 13.)
// Bound by vector instructions, 24.7 million (27.1 with a branch per term, see walk_terms): one table of 4096
// samples, 4096 sizes x 976 process counts up to 65 536 the call 132 -> 125 us, 1000 x up to 8192 56 -> 50.5, 300
// sizes x up to 65 536 59 -> 55; 300 samples, 3000 sizes 96 -> 89.  (Units of one, two or four blocks make no
// difference.)
constexpr int CHAIN_U = 4;           // blocks walked one after the other by a lane in the sparse part
constexpr int CHAIN_MAX_S = 1024;    // candidates kept in LDS for these pieces

template <bool TERMS>
__device__ __forceinline__ void chain_body(const DeviceTables &T, const DeviceGrid &G, const Scratch &S,
                                           int wg_per_table, int n_single, int terms_mode,
                                           int block_id, double *chain_lds)
{
    __shared__ unsigned next_item;
    const int t = block_id / wg_per_table, wg = block_id % wg_per_table;
    ChainCtx C;
    stage_intervals(C, chain_lds, T, t);
    double *const sd = chain_lds + 4 * T.n + CHAIN_PAD;
    if (TERMS && (terms_mode & 2))
        for (int si = threadIdx.x; si < G.n_s; si += blockDim.x)
            sd[si] = (double)G.s[si];
    if (threadIdx.x == 0)
        next_item = 0u;
    __syncthreads();
    const int lane = threadIdx.x & 63;
    const int n_mg = (G.n_mu + 63) / 64;      // groups of 64 distinct sizes
    const unsigned n_single_items = (unsigned)n_single * (unsigned)n_mg;
    const unsigned n_units = (unsigned)((G.n_blk - n_single + CHAIN_U - 1) / CHAIN_U);
    const unsigned n_items = n_single_items + n_units * (unsigned)n_mg;
    const unsigned W_ = (unsigned)wg_per_table;
    C.n_blk = G.n_blk;
    C.n_m = (size_t)G.n_mu;
    C.blk_mask = G.blk_mask;
    C.blk_off = G.blk_off;
    for (;;) {
        unsigned k = 0;
        if (lane == 0)
            k = atomicAdd(&next_item, 1u);
        k = __builtin_amdgcn_readfirstlane(k);
        // round k of the deal: this workgroup's place is wg, or W_ - 1 - wg in odd rounds
        const unsigned item = k * W_ + ((k & 1u) ? W_ - 1u - (unsigned)wg : (unsigned)wg);
        if (item >= n_items) {            // later rounds lie further on still
            const unsigned rounds = n_items / W_, in_last = (rounds & 1u) ? W_ - 1u - (unsigned)wg : (unsigned)wg;
            const unsigned my_items = rounds + (in_last < n_items - rounds * W_ ? 1u : 0u);
            if (TERMS && terms_piece(C, T, G, S, t, wg, wg_per_table, (int)(blockDim.x >> 6), terms_mode, k - my_items,
                                     (terms_mode & 2) ? sd : nullptr))
                continue;
            break;
        }
        const bool single = item < n_single_items;
        const unsigned rest = single ? item : item - n_single_items;
        const int u = (int)(rest / (unsigned)n_mg), mg = (int)(rest % (unsigned)n_mg);
        const int mi = mg * 64 + lane;
        if (mi >= G.n_mu)
            continue;
        const u64 m = G.mu[mi];
        double *part = S.part + ((size_t)t * C.n_m + mi) * G.n_P;     // [m][P index]
        const BlkAt at_total = blk_of(G, t, mi);
        chain_item(C, single ? u : n_single + u * CHAIN_U, single ? 1 : CHAIN_U, m, part,
                   S.blk + at_total.first, at_total.stride);
    }
}

__global__ void __launch_bounds__(1024) k_chain_blocks(DeviceTables T, DeviceGrid G, Scratch S, int wg_per_table,
                                                       int n_single, int terms_mode)
{
    extern __shared__ __align__(16) double chain_lds[];   // the table as intervals, the candidates
    chain_body<true>(T, G, S, wg_per_table, n_single, terms_mode, (int)blockIdx.x, chain_lds);
}

// ---------------------------------------------------------------- the chain row at n points

// Sums of g((64 b + 1) m), ..., g((64 b + 64) m) added in ascending j from +0.0.

// After moving into interval i the size is
// still at or past its end (d >= w), i.e. several intervals on.  Looks four
// intervals ahead a few times, then searches the rest of the table for the size
// itself (exact: integers below 2^53).  Leaves i, d and the interval's terms.
__device__ __forceinline__ void chain_skip_ahead(const ChainCtx &C, int &i, double &d, double &w,
                                                 double &yi, double &si)
{
    const double *X = C.X;
    double xb = X[i + 1];         // end of interval i
    double e = d - w;             // size - end of interval i
    int hops = 0;
    for (;;) {
        const double r1 = X[i + 2] - xb, r2 = X[i + 3] - xb;
        const double r3 = X[i + 4] - xb, r4 = X[i + 5] - xb;
        if (e >= r4) {
            if (++hops == 3) {
                const double z[1] = {xb + e};
                int iz[1];
                chain_locate<1>(X, C.n, z, iz);
                i = iz[0];
                d = z[0] - X[i];
                break;
            }
            i += 4;
            e -= r4;
            xb += r4;
            continue;
        }
        const int c = (e >= r1 ? 1 : 0) + (e >= r2 ? 1 : 0) + (e >= r3 ? 1 : 0);
        const double lo = c == 0 ? 0.0 : (c == 1 ? r1 : (c == 2 ? r2 : r3));
        d = e - lo;
        i += 1 + c;
        break;
    }
    const f64x2 ys = C.YS[i];
    w = C.W[i];
    yi = ys.x;
    si = ys.y;
}

// The first `terms` of them in this lane (0: none; FULL: all 64), a step per term (the loop runs to the wave's
// largest), with a branch where some lane enters an interval: eight at a time, as walk_block does, is no faster
// where most lanes have left before the last term (100 000 points with P up to 300 on 100 samples 31.7 us this way,
// 35.9 so; 290 000 with P up to 1024 on 256 samples 99, 117).  The sum and the distance are pinned to their
// registers after every term: left to itself the compiler carries a copy of every state variable past each
// branch.
template <bool FULL>
__device__ __forceinline__ double chain_step_walk(const ChainCtx &C, u64 b, u64 m, int terms)
{
    const double md = (double)m;
    WalkAt at = walk_from(C, (double)((b * SUM_BLOCK + 1) * m));
    double run = 0.0;
    const auto step = [&](bool use) {
        if (use && at.d >= at.w) {
            at.d -= at.w;
            ++at.i;
            at.w = C.W[at.i];
            at.ys = C.YS[at.i];
            if (at.d >= at.w) {                       // several intervals on
                double yi, si;
                chain_skip_ahead(C, at.i, at.d, at.w, yi, si);
                at.ys.x = yi;
                at.ys.y = si;
            }
        }
        const double g = run + __builtin_fma(at.ys.y, at.d, at.ys.x);
        run = use ? g : run;
        at.d += md;
        asm volatile("" : "+v"(run), "+v"(at.d));
    };
    if (FULL) {
#pragma unroll 1
        for (int k = 0; k < SUM_BLOCK; k += 8) {
#pragma unroll
            for (int u = 0; u < 8; ++u)
                step(true);
        }
    } else {
        for (int k = 0; __ballot(k < terms) != 0; ++k)
            step(k < terms);
    }
    return run;
}

// All 64.  Bound by the number of instructions, or, for few points, by the time that a wave takes.  What matters is
// the first block, whose sizes are six octaves apart; the others are walked eight terms at a time (or searched for
// where they enter many intervals all the same).  On a table of few samples the first is walked too, without a look
// at how many intervals it enters.  On others a wave with some lane's first block searches for its terms, unless
// there are so many points that their instructions count, not the wait: then it walks a term at a time (122 samples,
// P up to 122: 290 000 points 30.0 us so, 32.3 searched for, 38.0 walked eight terms at a time; 3500 points 23.1,
// 20.9 and 23.2; 72 samples 20.2, 20.0 and 18.2).  The rule: launch_eval.
enum EvalBlocks : int { EVAL_WALK, EVAL_SEARCH, EVAL_STEP };
constexpr int EVAL_LOOK_N = 128;         // up to which blocks other than the first are walked without a look
constexpr int EVAL_REACH = 16;           // intervals entered from which on it searches in the first block
static_assert(power_of_two(EVAL_REACH), "compared with what wave_reach gives");

// BIG: more than EVAL_SEARCH_N samples (without the walk that is not looked for there, the kernel for these keeps
// to 80 registers, with which two workgroups of 768 threads share a compute unit: 900 samples, 290 000 points with
// P up to 70 76 us, 91 with 85).
template <int BLOCKS, bool BIG>
__device__ __forceinline__ double chain_block_sum(const ChainCtx &C, u64 b, u64 m)
{
    const bool first = BLOCKS != EVAL_WALK && __ballot(b == 0) != 0;
    if (BLOCKS == EVAL_STEP && first)
        return chain_step_walk<true>(C, b, m, SUM_BLOCK);
    const double md = (double)m, z0 = (double)((b * SUM_BLOCK + 1) * m);
    if (BLOCKS == EVAL_WALK || (!BIG && C.n <= EVAL_LOOK_N && !first)) {
        WalkAt at = walk_from(C, z0);
        return walk_block(C, at, md, 0, 0, nullptr);
    }
    const double ends[2] = {z0, (double)((b * SUM_BLOCK + SUM_BLOCK) * m)};
    int i[2];
    chain_locate<2>(C.X, C.n, ends, i);
    const int reach = wave_reach(C, i[1] - i[0]);
    if (reach > (!BIG && C.n <= EVAL_LOOK_N ? EVAL_REACH : WALK_REACH))
        return block_search(C, i[0], reach, md, z0, 0, 0, nullptr);
    WalkAt at = {i[0], z0 - C.X[i[0]], C.W[i[0]], C.YS[i[0]]};
    return walk_block(C, at, md, 0, 0, nullptr);
}

// As gaps_within, on indices in place of addresses (reach: a power of two).
template <int V>
__device__ __forceinline__ void gaps_within_by_index(const ChainCtx &C, int i0, int reach, const double (&z)[V],
                                                     double (&g)[V])
{
    int i[V];
#pragma unroll
    for (int c = 0; c < V; ++c)
        i[c] = i0;
    for (int half = reach >> 1; half > 0; half >>= 1) {
        double x[V];
#pragma unroll
        for (int c = 0; c < V; ++c) {
            const int at = i[c] + half;
            x[c] = C.X[at < C.n + 1 ? at : C.n + 1];       // +inf past the last interval
        }
#pragma unroll
        for (int c = 0; c < V; ++c)
            i[c] = x[c] <= z[c] ? i[c] + half : i[c];
    }
#pragma unroll
    for (int c = 0; c < V; ++c) {
        const f64x2 ys = C.YS[i[c]];
        g[c] = __builtin_fma(ys.y, z[c] - C.X[i[c]], ys.x);
    }
}

// g((64 b + 1) m) + ... + g((64 b + terms) m), terms < 64 of them in this lane (0: none).  BY_INDEX: where
// there are many points, of which a workgroup takes 768, or 256 up to 640 samples.  The search on addresses
// makes those of 768 slower (300 000 points: 2000 samples with P up to 300 218 us by index, 239; 1500 with P
// up to 64 65 and 82) and those of 256 mostly faster, but not all (600 samples with P up to 64 48.0 by index,
// 44.5; 512 with P up to 300 83.4 and 87.3).  Few points gain (3000 with P up to 64: 600 samples 24.4 us by
// index, 19.2; 4000 samples 34.3 and 29.1).
template <bool BY_INDEX>
__device__ __forceinline__ double chain_rest_sum(const ChainCtx &C, u64 b, u64 m, int terms)
{
    constexpr int V = 8;
    const double md = (double)m;
    double zb = (double)((b * SUM_BLOCK + 1) * m);
    const double ends[2] = {zb, terms > 0 ? __builtin_fma((double)(terms - 1), md, zb) : zb};
    int at[2], reach = 1;
    chain_locate<2>(C.X, C.n, ends, at);
    while (__ballot(at[1] - at[0] >= reach) != 0)
        reach <<= 1;
    if (!BY_INDEX)
        reach = reach < C.n + 2 ? reach : C.n + 2;
    double run = 0.0;
#pragma unroll 1
    for (int k = 0; __ballot(k < terms) != 0; k += V) {
        double z[V], g[V];
#pragma unroll
        for (int c = 0; c < V; ++c)
            z[c] = __builtin_fma((double)c, md, zb);
        if (BY_INDEX)
            gaps_within_by_index<V>(C, at[0], reach, z, g);
        else
            gaps_within<V>(C, at[0], reach, z, g);
#pragma unroll
        for (int c = 0; c < V; ++c)
            run = k + c < terms ? run + g[c] : run;
        zb = __builtin_fma((double)V, md, zb);
    }
    return run;
}

// Table 2, chain row (and its Gather twin) at n independent points: fma(P-1, L, sum_{j<P} g(j m)).
// A sum is blocks of SUM_BLOCK terms that do not depend on one another, and points ask for very
// different numbers of them: a workgroup takes as many points as it has threads, sorts them by
// the number of complete blocks, and deals (block index, point) pairs to the lanes, equal block
// indices side by side (they cross about as many intervals of the table per term).  Block totals
// go to LDS, LEVELS block indices at a time; the thread of a point adds its totals in ascending
// order, then the incomplete block it forms itself: on a table of few samples by the same walk, else
// with a search per term, eight side by side, because nearly every term enters another interval
// there (300 000 points with P up to 64: 64 samples 19 us walked, 35 searched; 4096 samples 291 and
// 88; at 512 as fast, and with P up to 16 30 and 20).
//
// Bound by the vector instructions of the walk (300 000 points with P up to 1024, 64 samples: 71 us, 76
// with a branch per term, which few lanes take but some nearly always; 555 with a thread that walks its
// point alone and searches the table per term).  Few points, where a wave's latency counts, gain most by
// the walk of eight terms at a time: 30 000 points 56 -> 42 us, 3000 51 -> 39, 30 000 with P up to 5000
// 183 -> 126; on 2000 samples, of which blocks are searched for, 290 000 with P up to 300 214 -> 165.
// LEVELS: eight when there are few points, whose blocks would not fill the chip otherwise, four when
// there are many on a table that leaves LDS for few waves (512 samples: 142 us, 185 with eight).
constexpr int EVAL_SEARCH_N = 256;       // more samples: the rest of a sum is searched for

template <int LEVELS, int BLOCKS>
__global__ void __launch_bounds__(LEVELS == 4 ? 768 : 384)
k_eval_chain(DeviceTables T, int t, const u64 *dm, const uint32_t *dP, size_t n, double *out)
{
    extern __shared__ __align__(16) double eval_lds[];
    __shared__ unsigned above[LEVELS + 2], slot[LEVELS + 1], most;
    const int threads = (int)blockDim.x, tid = (int)threadIdx.x;
    double *tot = eval_lds;                                        // [LEVELS][threads]
    u64 *m_of = reinterpret_cast<u64 *>(tot + (size_t)LEVELS * threads);
    unsigned short *order = reinterpret_cast<unsigned short *>(m_of + threads);
    ChainCtx C;
    stage_intervals<true>(C, reinterpret_cast<double *>(order + threads), T, t);
    const size_t i = (size_t)blockIdx.x * threads + tid;
    const u64 m = i < n ? dm[i] : 0;
    const uint32_t P = i < n ? dP[i] : 0;
    const u64 lim = 1ull << 53;
    const bool ok = m > 0 && m < lim && P >= 2 && (u64)(P - 1) <= (lim - 1) / m;
    const uint32_t full = ok ? (P - 1u) / SUM_BLOCK : 0u;
    const int tail = ok ? (int)((P - 1u) % SUM_BLOCK) : 0;
    m_of[tid] = ok ? m : 1;
    if (tid == 0)
        most = 0u;
    __syncthreads();
    atomicMax(&most, full);
    __syncthreads();
    const uint32_t levels = most;
    double done = 0.0;
    for (uint32_t b0 = 0; b0 < levels; b0 += LEVELS) {
        // complete blocks of this point among b0 .. b0 + LEVELS - 1
        const int mine = full <= b0 ? 0 : (full - b0 < LEVELS ? (int)(full - b0) : LEVELS);
        if (tid <= LEVELS)
            slot[tid] = 0u;
        __syncthreads();
        const unsigned rank = atomicAdd(&slot[mine], 1u);          // among the points with as many
        __syncthreads();
        if (tid == 0) {                                            // above[k]: points with k or more
            unsigned acc = 0;
            above[LEVELS + 1] = 0u;
            for (int k = LEVELS; k >= 0; --k) {
                acc += slot[k];
                above[k] = acc;
            }
        }
        __syncthreads();
        order[above[mine + 1] + rank] = (unsigned short)tid;       // most blocks first
        __syncthreads();
        // level k's pairs are the first above[k + 1] points of that order
        unsigned total = 0;
#pragma unroll
        for (int k = 0; k < LEVELS; ++k)
            total += above[k + 1];
        for (unsigned e0 = (unsigned)tid & ~63u; e0 < total; e0 += (unsigned)threads) {
            unsigned r = e0 + ((unsigned)tid & 63u);
            const bool real = r < total;
            r = real ? r : total - 1u;
            int k = 0;
#pragma unroll
            for (int u = 0; u < LEVELS - 1; ++u) {
                const unsigned c = above[u + 1];
                if (k == u && r >= c) {
                    r -= c;
                    k = u + 1;
                }
            }
            const int p = order[r];
            const double v = chain_block_sum<BLOCKS, LEVELS == 4>(C, (u64)b0 + k, m_of[p]);
            if (real)
                tot[(size_t)k * threads + p] = v;
        }
        __syncthreads();
        for (int k = 0; k < mine; ++k)
            done = done + tot[(size_t)k * threads + tid];
    }
    const double rest = C.n > EVAL_SEARCH_N ? chain_rest_sum<LEVELS == 4>(C, full, m_of[tid], tail)
                                            : chain_step_walk<false>(C, full, m_of[tid], tail);
    if (i < n)
        out[i] = ok ? __builtin_fma((double)(P - 1u), T.L[t], done + rest) : NAN;
}

static size_t eval_chain_lds(int n, int levels, int threads)
{
    return ((size_t)levels * threads + threads + threads / 4 + 4 * (size_t)n + CHAIN_PAD) * sizeof(double);
}

// The Scatter-chain sums of one (table, distinct m) in one workgroup, for tables of few
// samples and sums of few blocks: what k_chain_blocks and k_chain_prefix leave in device
// memory (the in-block sums at the grid's process counts, and the totals of the finished
// blocks or their prefix), without a lane that walks a block alone.  A thread evaluates 16
// consecutive terms g(j m) (one search, then a walk: the sizes ascend), into a tile in LDS;
// a lane per block adds its 64 terms in order and leaves the sum before every term in
// place; one lane adds the block totals in order; all threads write the sums out, the
// process counts along the lanes.
constexpr int CROW_THREADS = 256;
constexpr int CROW_MAX_BLK = 96;         // 6144 terms at most
constexpr int CROW_TPT = 16;             // consecutive terms per thread
constexpr int CROW_LD = SUM_BLOCK + SUM_BLOCK / CROW_TPT + 1;     // 69: a block's row in the tile

// term r (0-based) sits at r + r / 64 + r / 16: rows of 69, so that neither the threads
// that write runs of 16 nor the lanes that read one row each meet in a bank
__device__ __forceinline__ int crow_at(int r) { return r + r / SUM_BLOCK + r / CROW_TPT; }

static size_t chain_row_lds(int n, int n_blk)
{
    return ((size_t)3 * n + (size_t)n_blk * CROW_LD + 2 * CROW_MAX_BLK) * sizeof(double);
}

__device__ __forceinline__ void chain_row_body(const DeviceTables &T, const DeviceGrid &G, const Scratch &S,
                                               int block_id, double *lds)
{
    const int n = T.n, n_blk = G.n_blk, n_mu = G.n_mu, n_P = G.n_P;
    const int tid = threadIdx.x;
    const int t = block_id / n_mu, mu_i = block_id % n_mu;
    double *x = lds, *y = x + n, *sl = y + n;
    double *pre = sl + n;                                  // the terms, then the sums before each
    double *tot = pre + (size_t)n_blk * CROW_LD, *done = tot + CROW_MAX_BLK;
    const u64 m = G.mu[mu_i];
    const uint32_t P_first = tid < n_P ? G.P[tid] : 2u;    // asked for now, used at the very end
    {
        const double *gx = T.x + (size_t)t * n, *gy = T.y + (size_t)t * n;
        for (int i = tid; i < n; i += CROW_THREADS) {
            x[i] = gx[i];
            y[i] = gy[i];
        }
        __syncthreads();
        for (int i = tid; i < n; i += CROW_THREADS)
            sl[i] = interval_slope(x, y, n, i);
        __syncthreads();
    }
    const double md = (double)m, x0 = x[0];
    const int n_terms = SUM_BLOCK * (n_blk - 1) + G.last_terms;
    for (int r0 = tid * CROW_TPT; r0 < n_blk * SUM_BLOCK; r0 += CROW_THREADS * CROW_TPT) {
        // g((r + 1) m) for r = r0 .. r0 + 15: the same expression as gap_at, with the interval
        // carried along (i: the last sample not above the size, 0 below the first)
        double z = (double)((u64)(r0 + 1) * m);
        int i = last_not_above(x, n, z);
        double xi = x[i], yi = y[i], si = sl[i];
        double xn = i + 1 < n ? x[i + 1] : INFINITY;
#pragma unroll 4
        for (int k = 0; k < CROW_TPT; ++k) {
            double v = 0.0;
            if (r0 + k < n_terms) {
                while (z >= xn) {
                    ++i;
                    xi = xn;
                    yi = y[i];
                    si = sl[i];
                    xn = i + 1 < n ? x[i + 1] : INFINITY;
                }
                const double zc = z > x0 ? z : x0;
                v = __builtin_fma(si, zc - xi, yi);
            }
            pre[crow_at(r0 + k)] = v;
            z += md;                                       // exact: integers below 2^53
        }
    }
    __syncthreads();
    if (tid < n_blk) {
        // sixteen terms at a time: read, add in order, write the sums before each
        double *p = pre + tid * CROW_LD;
        double run = 0.0;
        for (int r0 = 0; r0 < SUM_BLOCK; r0 += CROW_TPT) {
            double v[CROW_TPT];
            double *q = p + r0 + r0 / CROW_TPT;
#pragma unroll
            for (int u = 0; u < CROW_TPT; ++u)
                v[u] = q[u];
#pragma unroll
            for (int u = 0; u < CROW_TPT; ++u) {
                q[u] = run;
                run = run + v[u];
            }
        }
        tot[tid] = run;
    } else if (tid < CROW_MAX_BLK) {
        tot[tid] = 0.0;
    }
    __syncthreads();
    if (tid == 0) {
        // the finished blocks, in ascending order; sixteen totals per round trip to LDS
        double acc = 0.0;
        for (int b0 = 0; b0 < n_blk; b0 += 16) {
            double v[16];
#pragma unroll
            for (int u = 0; u < 16; ++u)
                v[u] = tot[b0 + u];
#pragma unroll
            for (int u = 0; u < 16; ++u) {
                done[b0 + u] = acc;
                acc = acc + v[u];
            }
        }
    }
    __syncthreads();
    const size_t row = (size_t)t * n_mu + mu_i;
    for (int pi = tid; pi < n_P; pi += CROW_THREADS) {
        const int r = (int)((pi == tid ? P_first : G.P[pi]) - 1u), blk = r / SUM_BLOCK;
        S.part[row * n_P + pi] = pre[crow_at(r)];
        if (G.blk_is_prefix)
            S.pre[row * n_P + pi] = done[blk];
    }
    if (!G.blk_is_prefix)
        for (int b = tid; b < n_blk - 1; b += CROW_THREADS)        // the last block is never complete
            S.blk[((size_t)t * n_blk + b) * n_mu + mu_i] = tot[b];
}

__global__ void __launch_bounds__(CROW_THREADS) k_chain_row(DeviceTables T, DeviceGrid G, Scratch S)
{
    extern __shared__ double lds[];
    chain_row_body(T, G, S, (int)blockIdx.x, lds);
}

// The terms and the sums above in one launch, side by side: both are short chains of
// dependent steps.  The (few) terms workgroups come first, so that they are on the chip at
// once.
__global__ void __launch_bounds__(CROW_THREADS) k_terms_chain_row(DeviceTables T, DeviceGrid G, Scratch S,
                                                                  int terms_wg, int n_chunks, int n_mchunks,
                                                                  int with_pairs)
{
    extern __shared__ __align__(16) double both_lds[];
    if ((int)blockIdx.x < terms_wg)
        terms_body(T, G, S, n_chunks, n_mchunks, with_pairs, (int)blockIdx.x, both_lds);
    else
        chain_row_body(T, G, S, (int)blockIdx.x - terms_wg, both_lds);
}

// Both first steps in one launch: they do not depend on each other (each stages the
// table from the raw samples), so the workgroups of the chain sums (the longer job, first
// in the grid) and those of the terms run side by side.  For tables small enough that
// workgroups of both kinds share a CU.  SMALL: a small job, terms by search, side by side (a kernel
// of its own: 49 sizes x 26 process counts up to 4096 took 0.5 us of 8 longer beside the walk's code).
template <bool SMALL>
__global__ void __launch_bounds__(256) k_terms_chain(DeviceTables T, DeviceGrid G, Scratch S, int n_chain_wg,
                                                     int wg_per_table, int n_single,
                                                     int n_chunks, int n_mchunks, int with_pairs)
{
    extern __shared__ __align__(16) double both_lds[];
    if ((int)blockIdx.x < n_chain_wg) {
        if (SMALL)
            chain_small_body(T, G, S, wg_per_table, (int)blockIdx.x, both_lds);
        else
            chain_body<false>(T, G, S, wg_per_table, n_single, 0, (int)blockIdx.x, both_lds);
    } else
        terms_body(T, G, S, n_chunks, n_mchunks, with_pairs, (int)blockIdx.x - n_chain_wg, both_lds);
}

// Turns the block totals of M message sizes into their exclusive prefix in
// ascending block order (the sum of all finished blocks before block b) and
// writes, per process count of the grid, the prefix of the block it ends in:
// pre[m][P index], which the sweeps read side by side with the partial sums.  The sum is
// sequential per m: one wave adds (lane m, two blocks per access to LDS, the next sixteen on their
// way), the others meanwhile write out the tile before, put the next one into LDS and ask for the one
// after next two steps ahead; three tiles of PFX_TILE blocks take turns, so that a step is one barrier.
//
// 3215 distinct sizes x 1024 blocks, 976 process counts: 18.7 us in the trace for 51 MB, 300 sizes 15.0
// (20.0 and 17.3 with sixteen sizes to a workgroup, whose totals lay 128 bytes at a time among those of all
// sizes, and each sixteen asked for when those before had been added; 19.9 and 16.2 with eight sizes, their
// totals together, alone; 32 and 14.7 with four; tiles of 64 blocks 20.2 and 16.7; 25.7 for the first when a
// workgroup of four waves loaded, added and wrote in turn).  What bounds it is the way of the adding wave through
// LDS: of the 14.8 us of 300 sizes 13.0 remain with nothing loaded and nothing written out by the others (14.2
// without the loads, 13.5 without the stores; of 18.9 with 3215 sizes 14.3), and with the totals passed on in place
// of sums, no addition waiting for another, it takes no less (17.1).
constexpr int PFX_TILE = 128;
constexpr int PFX_THREADS = 512;
constexpr int PFX_LD = PFX_TILE + 2;     // row of a size: the lanes' pairs lie in different banks
constexpr int PFX_WG_PER_CU = 4;         // at once, of eight sizes (the line at 2 or 8: 60 x 200 sizes 171 and 183 us)
constexpr int PFX_MAX_P = 4096;          // process counts whose block index is kept in LDS

__host__ __device__ inline bool pfx_in_lds(const DeviceGrid &G) { return G.n_P <= PFX_MAX_P && G.n_blk <= 65536; }

template <int M>
__global__ void __launch_bounds__(PFX_THREADS) k_chain_prefix(DeviceGrid G, Scratch S, int n_mgroups)
{
    __shared__ __align__(16) double tile[3][M * PFX_LD];     // [m][block]
    extern __shared__ unsigned short pfx_blk_of[];               // [n_P] if pfx_in_lds
    const int t = blockIdx.x / n_mgroups, mg = blockIdx.x % n_mgroups;
    const int tid = threadIdx.x, hid = tid - 64;         // hid: thread of the helping waves
    constexpr int HELPERS = PFX_THREADS - 64, ROWS = HELPERS / M, N = (PFX_TILE + ROWS - 1) / ROWS;
    const int ml = tid % M, br = hid / M;
    const int mi = mg * M + ml;
    const bool active = mi < G.n_mu;
    const size_t n_m = (size_t)G.n_mu;       // rows: the distinct sizes
    const BlkAt from = blk_of(G, t, active ? mi : mg * M);
    const double *src = S.blk + from.first;
    const int full = G.n_blk - 1;                        // blocks that have a total
    const int n_tiles = (G.n_blk + PFX_TILE - 1) / PFX_TILE;
    const bool p_in_lds = pfx_in_lds(G);
    const int m_valid = G.n_mu - mg * M < M ? G.n_mu - mg * M : M;   // sizes of this group
    double v[2][N], done = 0.0;
    auto load = [&](int k, double (&r)[N]) {             // totals of tile k (0 where there is none)
#pragma unroll
        for (int u = 0; u < N; ++u) {
            const int row = br + ROWS * u, b = k * PFX_TILE + row;
            r[u] = (active && row < PFX_TILE && b < full) ? src[b * from.stride] : 0.0;
        }
    };
    auto put = [&](int k, const double (&r)[N]) {
#pragma unroll
        for (int u = 0; u < N; ++u) {
            const int row = br + ROWS * u;
            if (row < PFX_TILE)
                tile[k % 3][ml * PFX_LD + row] = r[u];
        }
    };
    // only the blocks in which some process count of the grid ends are wanted: the sums
    // go out per process count, pre[m][P index], a run of the output per m and store
    auto write = [&](int k) {
        const int b0 = k * PFX_TILE, b1 = b0 + PFX_TILE < G.n_blk ? b0 + PFX_TILE : G.n_blk;
        const int pi_hi = G.blk_off[b1];
        for (int pi = G.blk_off[b0] + hid; pi < pi_hi; pi += HELPERS) {
            const int bb = (p_in_lds ? (int)pfx_blk_of[pi] : (int)((G.P[pi] - 1u) / SUM_BLOCK)) - b0;
            // all the sums of the row first (one wait for LDS), then the stores
            double row[M];
#pragma unroll
            for (int mm = 0; mm < M; ++mm)
                row[mm] = tile[k % 3][mm * PFX_LD + bb];
            double *o = S.pre + ((size_t)t * n_m + (size_t)mg * M) * G.n_P + pi;
#pragma unroll
            for (int mm = 0; mm < M; ++mm) {
                if (mm < m_valid)
                    o[(size_t)mm * G.n_P] = row[mm];
            }
        }
    };
    // Step k: tile k is added up, k - 1 written out, k + 1 put into LDS, k + 3 asked for.
    auto step = [&](int k, double (&next)[N]) {
        if (hid < 0) {
            if (k < n_tiles && tid < M) {
                f64x2 *row = reinterpret_cast<f64x2 *>(&tile[k % 3][tid * PFX_LD]);
                const int left = G.n_blk - k * PFX_TILE, nb = left < PFX_TILE ? left : PFX_TILE;
                // sixteen at a time, the next sixteen on their way (blocks past the last hold zeros)
                f64x2 tot[2][8];
#pragma unroll
                for (int u = 0; u < 8; ++u)
                    tot[0][u] = row[u];
#pragma unroll
                for (int h = 0; h < PFX_TILE / 16; ++h) {
                    if (16 * h >= nb)
                        break;
                    if (h + 1 < PFX_TILE / 16) {
#pragma unroll
                        for (int u = 0; u < 8; ++u)
                            tot[(h + 1) & 1][u] = row[8 * (h + 1) + u];
                    }
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int u = 0; u < 8; ++u) {
                        f64x2 before;
                        before.x = done;
                        done = done + tot[h & 1][u].x;
                        before.y = done;
                        done = done + tot[h & 1][u].y;
                        row[8 * h + u] = before;
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
        } else {
            if (k + 1 < n_tiles)
                put(k + 1, next);
            if (k + 3 < n_tiles)
                load(k + 3, next);
            if (k > 0)
                write(k - 1);
        }
        __syncthreads();
    };
    if (hid >= 0) {
        load(0, v[0]);
        if (1 < n_tiles)
            load(1, v[1]);
        if (p_in_lds)
            for (int pi = hid; pi < G.n_P; pi += HELPERS)
                pfx_blk_of[pi] = (unsigned short)((G.P[pi] - 1u) / SUM_BLOCK);
        put(0, v[0]);
        if (2 < n_tiles)
            load(2, v[0]);
    }
    __syncthreads();
    for (int k = 0; k <= n_tiles; k += 2) {
        step(k, v[1]);
        if (k + 1 <= n_tiles)
            step(k + 1, v[0]);
    }
}

// ---------------------------------------------------------------- tune, step 3: sweep, arg-min, write

struct Best {
    double t;
    uint32_t s;
    uint32_t id;
};

__device__ __forceinline__ void consider(Best &b, double T, uint32_t id, uint32_t s)
{
    if (T < b.t) {
        b.t = T;
        b.id = id;
        b.s = s;
    }
}

// A 16-byte record of an output that no kernel of the call reads again: stored with the
// non-temporal hint, so that the stream of cells does not push the tables and terms out of the
// caches (measured on the 1.97 GB table of 10 000 clusters: 5 % off the whole kernel).
__device__ __forceinline__ void stream_out(void *p, uint4 v)
{
    typedef unsigned u32x4_t __attribute__((ext_vector_type(4)));
    u32x4_t w = {v.x, v.y, v.z, v.w};
    __builtin_nontemporal_store(w, reinterpret_cast<u32x4_t *>(p));
}

__device__ __forceinline__ void store_cell(plogp_cell_dev *p, const Best &b)
{
    union {
        plogp_cell_dev c;
        uint4 v;
    } u;
    u.c.time = b.t;
    u.c.s = b.s;
    u.c.strategy = b.id;
    stream_out(p, u.v);
}

// Broadcast: the ten rows of Table 1 in id order, strict '<' (ties: lowest id).
// t2/t5/t9 are the minima over s of the segmented rows (+inf if none), s2/s5/s9
// the segment sizes that attain them.
__device__ __forceinline__ Best decide_bcast(uint32_t mask, double q, double fl, double cl,
                                             double gm, double L, double g1, double t2,
                                             uint32_t s2, double t5, uint32_t s5, double t9,
                                             uint32_t s9)
{
    const double clL = cl * L;
    // A rendezvous row adds R - L = 2 g(1) + 2 L to its plain twin's latency term.  Gaps
    // and latencies are checked to be non-negative when a table is loaded and g(1) is the
    // first gap (size 1 is never above the first sample), so R >= L, and as rounding is
    // monotone a rendezvous row is never below its twin; with the twin enabled (lower id:
    // it also wins ties) the rendezvous row cannot be chosen and is not evaluated.
    if ((mask & 0x3FFu) == 0x3FFu) {
        // the usual case, every row enabled: rows 0, 2, 3, 5, 6, 7, 9 compete; the minimum,
        // then the lowest id that attains it (the compares do not depend on one another and
        // no partial minimum stays live)
        const double v0 = __builtin_fma(q, gm, L), v3 = q * (gm + L);
        const double v6 = cl * __builtin_fma(2.0, gm, L), v7 = __builtin_fma(fl, gm, clL);
        const double best =
            min_f64(min_f64(min_f64(v0, t2), min_f64(v3, t5)), min_f64(min_f64(v6, v7), t9));
        uint32_t id = 9u;
        id = v7 == best ? 7u : id;
        id = v6 == best ? 6u : id;
        id = t5 == best ? 5u : id;
        id = v3 == best ? 3u : id;
        id = t2 == best ? 2u : id;
        id = v0 == best ? 0u : id;
        Best b;
        b.t = best;
        b.id = id;
        b.s = id == 2u ? s2 : (id == 5u ? s5 : (id == 9u ? s9 : 0u));
        return b;
    }
    const double R = __builtin_fma(3.0, L, 2.0 * g1);   // rendezvous: 2 g(1) + 3 L
    Best b = {INFINITY, 0u, 0xFFFFFFFFu};
    // a rendezvous row (1, 4, 8) is evaluated only when its plain twin (0, 3, 7) is masked out
    if (mask & (1u << 0)) consider(b, __builtin_fma(q, gm, L), 0, 0);
    if ((mask & 3u) == 2u) consider(b, __builtin_fma(q, gm, R), 1, 0);
    if (mask & (1u << 2)) consider(b, t2, 2, s2);
    if (mask & (1u << 3)) consider(b, q * (gm + L), 3, 0);
    if ((mask & 0x18u) == 0x10u) consider(b, q * (gm + R), 4, 0);
    if (mask & (1u << 5)) consider(b, t5, 5, s5);
    if (mask & (1u << 6)) consider(b, cl * __builtin_fma(2.0, gm, L), 6, 0);
    if (mask & (1u << 7)) consider(b, __builtin_fma(fl, gm, clL), 7, 0);
    if ((mask & 0x180u) == 0x100u) consider(b, __builtin_fma(fl, gm, cl * R), 8, 0);
    if (mask & (1u << 9)) consider(b, t9, 9, s9);
    return b;
}

// Scatter: the three rows of Table 2, given the two sums for this (m, P).
__device__ __forceinline__ Best decide_scatter(uint32_t mask, double q, double cl, double gm,
                                               double L, double s11, double s12)
{
    if ((mask & 0x1C00u) == 0x1C00u) {
        // every row enabled: the minimum, then the lowest id that attains it
        const double v10 = __builtin_fma(q, gm, L), v11 = __builtin_fma(q, L, s11);
        const double v12 = __builtin_fma(cl, L, s12);
        Best b;
        b.t = min_f64(min_f64(v10, v11), v12);
        b.s = 0u;
        b.id = v10 == b.t ? 10u : (v11 == b.t ? 11u : 12u);
        return b;
    }
    Best b = {INFINITY, 0u, 0xFFFFFFFFu};
    if (mask & (1u << 10)) consider(b, __builtin_fma(q, gm, L), 10, 0);
    if (mask & (1u << 11)) consider(b, __builtin_fma(q, L, s11), 11, 0);
    if (mask & (1u << 12)) consider(b, __builtin_fma(cl, L, s12), 12, 0);
    return b;
}

// Barrier: a one-byte fan-in and fan-out, flat or binomial (bits 3 and 4 of `extra`).
__device__ __forceinline__ Best decide_barrier(uint32_t extra, double q, double fl, double cl, double L, double g1)
{
    Best b = {INFINITY, 0u, 0xFFFFFFFFu};
    if (extra & 8u) consider(b, 2.0 * __builtin_fma(q, g1, L), 16, 0);
    if (extra & 16u) consider(b, 2.0 * __builtin_fma(fl, g1, cl * L), 17, 0);
    return b;
}

// sum_{j=1}^{P-1} g(j m) for (m index mi, P index pi) from the block sums
__device__ __forceinline__ double chain_sum_of(const DeviceGrid &G, const Scratch &S, int t, int mi,
                                               int pi, uint32_t P)
{
    const size_t n_m = (size_t)G.n_mu;      // the chain sums are kept per distinct size
    mi = G.m_map[mi];
    const int blk = (int)((P - 1u) / SUM_BLOCK);
    double done;
    if (G.blk_is_prefix) {
        done = S.pre[((size_t)t * n_m + mi) * G.n_P + pi];
    } else {                           // few blocks: add the finished ones here, in ascending order
        const double *tot = S.blk + (size_t)t * G.n_blk * n_m + mi;
        done = 0.0;
        for (int b = 0; b < blk; ++b)
            done = done + tot[(size_t)b * n_m];
    }
    return done + S.part[((size_t)t * n_m + mi) * G.n_P + pi];
}

// Rows 2 and 9 of Table 1 are monotone in A = g(s) k for a fixed P (q >= 1,
// floor(log2 P) >= 1, rounding is monotone), so their minima over s are
//   min_s T2 = fma(q, min_s A, L),   min_s T9 = fma(fl, min_s A, cl L)
// exactly, and only min_s A (one v_min per (m, s)) is tracked in the sweeps.
// The segment size is then needed only in the cells that row 2 or 9 wins: there
// the candidates are walked once more, in ascending order, for the first s whose
// value equals the minimum (several A can round to the same time, so this is
// not simply the s of the smallest A).
//
// One lane per m, PC process counts per lane.  want[p]: 0 = nothing to find,
// else the row (2 or 9) that won cell p; V[p] its time.  cand(si, sd, rcp, gs)
// supplies the wave-uniform scalars of candidate si.  found[p] receives s.
template <int PC, class Cand>
__device__ __forceinline__ void first_s_of_flat_or_binomial(
    int n_cand, double limd, double md, double L, const double (&q)[PC], const double (&fl)[PC],
    const double (&clL)[PC], const int (&want)[PC], const double (&V)[PC], uint32_t (&found)[PC],
    Cand cand)
{
    bool open[PC];
#pragma unroll
    for (int p = 0; p < PC; ++p)
        open[p] = want[p] != 0;
    for (int si = 0; si < n_cand; ++si) {
        double sd, rcp_s, gs;
        cand(si, sd, rcp_s, gs);
        if (sd <= limd) {
            double A, B, C;
            segment_terms(md, sd, rcp_s, gs, L, A, B, C);
#pragma unroll
            for (int p = 0; p < PC; ++p) {
                const double Tv = want[p] == 2 ? __builtin_fma(q[p], A, L)
                                               : __builtin_fma(fl[p], A, clL[p]);
                if (open[p] && Tv == V[p]) {
                    found[p] = (uint32_t)sd;
                    open[p] = false;
                }
            }
        }
    }
}

// ---- sweep, few candidates: one lane per message size ------------------------
//
// A wave takes 64 consecutive m of one table and PC consecutive process counts.
// P and s are wave-uniform loop variables (their terms live in scalar
// registers); A, B are computed in the lane once per (m, s) and shared by the PC
// process counts.  Per (P, s) and segmented row: one fma, one compare, the
// running minimum and the index of the candidate that attained it (strict '<'
// in ascending s: ties go to the smallest s).

template <int PC>
__global__ void __launch_bounds__(256) k_sweep_m(DeviceTables T, DeviceGrid G, Scratch S,
                                                 plogp_cell_dev *out, int n_mg, int n_pcg)
{
    // the four waves of a workgroup share the table and the m group and take four
    // consecutive chunks of PC process counts; the per-candidate scalars (s, 1/s,
    // g(s)) are staged in LDS once for all of them
    __shared__ double sS[SWEEP_M_MAX_S], sR[SWEEP_M_MAX_S], sG[SWEEP_M_MAX_S];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    int bid = blockIdx.x;
    const int pcg = bid % n_pcg;
    bid /= n_pcg;
    const int mg = bid % n_mg;
    const int t = bid / n_mg;
    const int pc = pcg * 4 + wave;
    for (int si = threadIdx.x; si < G.n_s; si += blockDim.x) {
        sS[si] = (double)G.s[si];
        sR[si] = S.rcp[si];
        sG[si] = S.gs[(size_t)t * G.n_s + si];
    }
    __syncthreads();
    if (pc * PC >= G.n_P)
        return;

    const int mi = mg * 64 + lane;
    const bool active = mi < G.n_m;
    const u64 m = active ? G.m[mi] : 1;
    const double md = (double)m;
    const u64 lim = active ? (m < G.s_cap ? m : G.s_cap) : 0;
    const double limd = (double)lim;         // exact: at most m < 2^53 (0 for an idle lane)
    const double L = T.L[t];
    const uint32_t mask = G.mask;

    uint32_t Pv[PC];
    double q[PC], fl[PC], clL[PC];
#pragma unroll
    for (int p = 0; p < PC; ++p) {
        const int pi = pc * PC + p;
        Pv[p] = pi < G.n_P ? G.P[pi] : 2u;
        q[p] = (double)(Pv[p] - 1);
        fl[p] = (double)floor_log2(Pv[p]);
        clL[p] = (double)ceil_log2(Pv[p]) * L;
    }
    double b5[PC];
    int i5[PC];
#pragma unroll
    for (int p = 0; p < PC; ++p) {
        b5[p] = INFINITY;
        i5[p] = 0;
    }
    double amin = INFINITY;                  // min over s of A = g(s) k (rows 2 and 9)
    int n_seen = 0;                          // candidates walked (wave-uniform)
    if ((mask & 0x224u) && G.n_s > 0) {
        // the scalars of the next candidate are read from LDS while this one computes
        double sd_n = sS[0], rcp_n = sR[0], gs_n = sG[0];
        for (int si = 0; si < G.n_s; ++si) {
            const double sd = sd_n, rcp_s = rcp_n, gsv = gs_n;
            const int nx = si + 1 < G.n_s ? si + 1 : si;
            sd_n = sS[nx];
            rcp_n = sR[nx];
            gs_n = sG[nx];
            const bool valid = sd <= limd;
            if (__ballot(valid) == 0)
                break;                       // the candidates ascend: nothing further competes
            n_seen = si + 1;
            if (valid) {
                double A, B, C;
                segment_terms(md, sd, rcp_s, gsv, L, A, B, C);
                amin = min_f64(amin, A);
#pragma unroll
                for (int p = 0; p < PC; ++p) {
                    const double T5 = __builtin_fma(q[p], C, B);
                    i5[p] = T5 < b5[p] ? si : i5[p];
                    b5[p] = min_f64(b5[p], T5);
                }
            }
        }
    }
    if (!active)
        return;
    const size_t n_m = (size_t)G.n_m;
    const double gm = S.gm[(size_t)t * n_m + mi];
    const double g1 = S.g1[t];
    const size_t plane = n_m * G.n_P;

    // everything the PC cells read is fetched before the first of them is stored
    double s11[PC], s12[PC];
    uint32_t s5[PC];
    double done[PC];                         // finished blocks of the chain sum before each P
#pragma unroll
    for (int p = 0; p < PC; ++p)
        done[p] = 0.0;
    const size_t n_mu = (size_t)G.n_mu;      // the chain sums are kept per distinct size
    const int um = G.m_map[mi];
    if (mask & (1u << 11)) {
        const double *tot = S.blk + (size_t)t * G.n_blk * n_mu + um;
        if (G.blk_is_prefix) {
            const double *pre = S.pre + ((size_t)t * n_mu + um) * G.n_P;
#pragma unroll
            for (int p = 0; p < PC; ++p)
                done[p] = pre[pc * PC + p < G.n_P ? pc * PC + p : G.n_P - 1];
        } else {
            // few blocks (at most 32): the totals are added here, in ascending order; the
            // P of the chunk ascend, so one pass over the blocks serves all of them, and
            // the loads of eight blocks are in flight together
            int last = 0;
#pragma unroll
            for (int p = 0; p < PC; ++p) {
                const int blk = (int)((Pv[p] - 1u) / SUM_BLOCK);
                last = blk > last ? blk : last;
            }
            double acc = 0.0;
            for (int b0 = 0; b0 < last; b0 += 8) {
                double tv[8];
#pragma unroll
                for (int u = 0; u < 8; ++u)
                    tv[u] = b0 + u < last ? tot[(size_t)(b0 + u) * n_mu] : 0.0;
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    if (b0 + u < last) {
                        acc = acc + tv[u];
#pragma unroll
                        for (int p = 0; p < PC; ++p)
                            if ((int)((Pv[p] - 1u) / SUM_BLOCK) == b0 + u + 1)
                                done[p] = acc;
                    }
                }
            }
        }
    }
#pragma unroll
    for (int p = 0; p < PC; ++p) {
        const int pi = pc * PC + p < G.n_P ? pc * PC + p : G.n_P - 1;
        s11[p] = s12[p] = 0.0;
        if (mask & (1u << 11))
            s11[p] = done[p] + S.part[((size_t)t * n_mu + um) * G.n_P + pi];
        if (mask & (1u << 12))
            s12[p] = S.sum2[((size_t)t * n_m + mi) * (G.cl_max + 1) + ceil_log2(Pv[p])];
        s5[p] = b5[p] < INFINITY ? (uint32_t)sS[i5[p]] : 0u;
    }
    Best bc[PC];
    if (mask & 0x3FFu) {
        int want[PC];
        double V[PC];
        uint32_t found[PC];
        bool any = false;
#pragma unroll
        for (int p = 0; p < PC; ++p) {
            const double t2 = amin < INFINITY ? __builtin_fma(q[p], amin, L) : INFINITY;
            const double t9 = amin < INFINITY ? __builtin_fma(fl[p], amin, clL[p]) : INFINITY;
            bc[p] = decide_bcast(mask, q[p], fl[p], (double)ceil_log2(Pv[p]), gm, L, g1, t2, 0u,
                                 b5[p], s5[p], t9, 0u);
            want[p] = (bc[p].id == 2u || bc[p].id == 9u) ? (int)bc[p].id : 0;
            V[p] = bc[p].t;
            found[p] = 0u;
            any = any || want[p] != 0;
        }
        if (__ballot(any) != 0) {
            first_s_of_flat_or_binomial<PC>(
                n_seen, limd, md, L, q, fl, clL, want, V, found,
                [&](int si, double &sd, double &rcp_s, double &g) {
                    sd = sS[si];
                    rcp_s = sR[si];
                    g = sG[si];
                });
#pragma unroll
            for (int p = 0; p < PC; ++p)
                if (want[p] != 0)
                    bc[p].s = found[p];
        }
    }
#pragma unroll
    for (int p = 0; p < PC; ++p) {
        const int pi = pc * PC + p;
        if (pi >= G.n_P)
            break;
        plogp_cell_dev *o = out + (size_t)t * G.n_ops * plane + (size_t)mi * G.n_P + pi;
        const double cl = (double)ceil_log2(Pv[p]);
        if (mask & 0x3FFu) {
            store_cell(o, bc[p]);
            o += plane;
        }
        if (mask & 0x1C00u)
            store_cell(o, decide_scatter(mask, q[p], cl, gm, L, s11[p], s12[p]));
    }
}

// ---- sweep, few candidates, many process counts: one lane per P -----------------
//
// A wave takes 64 consecutive process counts of the grid (its lanes) and walks
// over message sizes.  Everything that depends on (m, s) only -- A, B (from
// k_terms), C, the candidate count, g(m) -- is the same in all lanes then: per
// candidate the lanes do one fma, one compare, the index select and the running
// minimum for row 5 of Table 1; min_s A for rows 2 and 9 is one reduction over the
// wave per m.  A cell
// costs two coalesced 16-byte stores.  The sizes of a wave lie n_w apart, so every
// wave meets the same mix of short and long candidate lists; the loads for the next
// size are issued before the current one is worked on.
// NSV: candidates per lane when a row of (m, s) terms is moved (n_s <= 64 NSV).
// FEW (NSV 1): row 5 for the candidates alone that can win it for some process count of
// the wave (row5_candidates), in place of a loop over all, eight a round trip to LDS.
// Which calls: sweep_few.
template <int NSV, bool ALL, int PPL, bool FEW>
__global__ void __launch_bounds__(256) k_sweep_p(DeviceTables T, DeviceGrid G, Scratch S,
                                                 plogp_cell_dev *out, int t0, int n_w)
{
    // the loops below read up to 7 entries past the last candidate: rows are 8 longer
    constexpr int ROW = 64 * NSV + 8;
    __shared__ uint32_t sSv[ROW];                    // s
    __shared__ double sC[FEW ? 1 : ROW];             // g(s) + L (0 past the end)
    __shared__ double rowB[4][FEW ? 1 : ROW];        // B of the current size (+inf past the end)
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    // grid: x = group of four waves, y = group of 64 PPL process counts, z = table (from t0)
    const int wq = (int)blockIdx.x, pg = (int)blockIdx.y, t = t0 + (int)blockIdx.z;
    const int w = wq * 4 + wave;
    const bool has_work = w < n_w && w < G.n_m;
    const uint32_t mask = ALL ? 0x1FFFu : G.mask;      // ALL: every strategy competes
    const int n_P = G.n_P, n_s = G.n_s, n_blk = G.n_blk;
    const size_t n_m = (size_t)G.n_m;
    const double L = T.L[t];
    const double g1 = S.g1[t];
    const bool chain = (mask & (1u << 11)) != 0, binom = (mask & (1u << 12)) != 0;
    const bool seg = (mask & 0x224u) != 0 && n_s > 0;
    const size_t plane = n_m * n_P;
    // a lane takes PPL process counts, 64 apart (so that every store of a wave is one run)
    int pi[PPL], cli[PPL], blk[PPL], bmin[PPL], bmax[PPL];
    bool active[PPL];
    double q[PPL], fl[PPL], cl[PPL], clL[PPL];
#pragma unroll
    for (int h = 0; h < PPL; ++h) {
        const int base = (pg * PPL + h) * 64;
        pi[h] = base + lane;
        active[h] = pi[h] < n_P;
        const uint32_t Pv = G.P[active[h] ? pi[h] : n_P - 1];
        q[h] = (double)(Pv - 1u);
        cli[h] = ceil_log2(Pv);
        fl[h] = (double)floor_log2(Pv);
        cl[h] = (double)cli[h];
        clL[h] = cl[h] * L;
        blk[h] = (int)((Pv - 1u) / SUM_BLOCK);
        // the smallest and the largest block index among the lanes (the P of the grid ascend;
        // an empty half repeats the last P of the grid)
        const int here = n_P - base < 64 ? n_P - base : 64;
        bmin[h] = __builtin_amdgcn_readfirstlane(blk[h]);
        bmax[h] = __builtin_amdgcn_readlane(blk[h], here > 0 ? here - 1 : 0);
    }
    plogp_cell_dev *const obase = out + (size_t)t * G.n_ops * plane + pi[0];

    // what is fetched one size ahead
    double fB[NSV], f_part[PPL], f_s12[PPL], f_done[PPL], f_gm, f_amin = INFINITY;
    int f_nv;
#pragma unroll
    for (int h = 0; h < PPL; ++h)
        f_part[h] = f_s12[h] = f_done[h] = 0.0;
#pragma unroll
    for (int k = 0; k < NSV; ++k)
        fB[k] = INFINITY;                // of a grid without candidates, which fetches none
    // row of the chain sums (kept per distinct size) of the size fetched next: read one size
    // earlier still, so that the fetch does not wait for it
    int um_next = chain && has_work ? G.m_map[w] : 0;
    // the sizes of a wave lie n_w apart: the rows of the per-size arrays are reached by adding
    // a stride to running pointers (no multiplications per size); the chain sums are kept per
    // distinct size and go through the row map
    const double *p_gm = S.gm + (size_t)t * n_m + w;
    const double *p_amin = S.amin + (size_t)t * n_m + w;
    const int *p_nv = S.nv + w;
    const double *p_B = S.segB + ((size_t)t * n_m + w) * n_s + lane;
    const double *p_s12 = S.sum2 + ((size_t)t * n_m + w) * (G.cl_max + 1);
    const size_t stride_B = (size_t)n_w * n_s, stride_s12 = (size_t)n_w * (G.cl_max + 1);
    const double *const part_t = S.part + (size_t)t * G.n_mu * n_P;
    const double *const pre_t = S.pre + (size_t)t * G.n_mu * n_P;
    const double *const blk_t = S.blk + ((size_t)t * n_blk + lane) * G.n_mu;
    auto fetch = [&](int mi) {
        f_gm = *p_gm;
        f_nv = *p_nv;
        p_gm += n_w;
        p_nv += n_w;
        if (seg) {
            f_amin = *p_amin;
            p_amin += n_w;
#pragma unroll
            for (int k = 0; k < NSV; ++k)
                fB[k] = lane + 64 * k < n_s ? p_B[64 * k] : INFINITY;
            p_B += stride_B;
        }
        if (chain) {
            const uint32_t um = (uint32_t)um_next;
            um_next = G.m_map[mi + n_w < (int)n_m ? mi + n_w : mi];
            const double *row = part_t + (u64)um * (uint32_t)n_P;
#pragma unroll
            for (int h = 0; h < PPL; ++h)
                f_part[h] = row[active[h] ? pi[h] : n_P - 1];
            if (G.blk_is_prefix) {
                const double *prow = pre_t + (u64)um * (uint32_t)n_P;
#pragma unroll
                for (int h = 0; h < PPL; ++h)
                    f_done[h] = prow[active[h] ? pi[h] : n_P - 1];
            } else {                   // few blocks: lane b holds the total of block b
                f_done[0] = lane < n_blk - 1 ? blk_t[um] : 0.0;
            }
        }
        if (binom) {
#pragma unroll
            for (int h = 0; h < PPL; ++h)
                f_s12[h] = p_s12[cli[h]];
            p_s12 += stride_s12;
        }
    };
    // the first size's inputs are on their way while the candidates go to LDS
    if (has_work)
        fetch(w);
    for (int si = threadIdx.x; si < ROW; si += blockDim.x) {
        sSv[si] = si < G.n_s ? (uint32_t)G.s[si] : 0u;
        if (!FEW) {
            sC[si] = si < G.n_s ? S.segC[(size_t)t * G.n_s + si] : 0.0;
            if (si >= 64 * NSV) {
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    rowB[k][si] = INFINITY;
            }
        }
    }
    // a candidate per lane (0 past the end)
    const double C = FEW && seg && lane < n_s ? S.segC[(size_t)t * n_s + lane] : 0.0;
    const double q_lo = lane_value(q[0], 0), q_hi = lane_value(q[PPL - 1], 63);
    __syncthreads();
    if (!has_work)
        return;
    for (int mi = w; mi < (int)n_m; mi += n_w) {
        const double gm = f_gm;
        double part[PPL], s12[PPL], dn[PPL];
#pragma unroll
        for (int h = 0; h < PPL; ++h) {
            part[h] = f_part[h];
            s12[h] = f_s12[h];
            dn[h] = f_done[h];
        }
        const int nv = f_nv;
        const double amin = f_amin;      // min over s of A = g(s) k, from k_terms
        const size_t row_now = (size_t)t * n_m + mi;
        const double B = FEW ? fB[0] : 0.0;
        if (!FEW && seg) {
#pragma unroll
            for (int k = 0; k < NSV; ++k)
                rowB[wave][lane + 64 * k] = fB[k];
        }
        if (!FEW) {
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
        }
        if (mi + n_w < (int)n_m)
            fetch(mi + n_w);

        // row 5: min over s of fma(q, C, B), and where it first appeared (FEW: the candidate, else
        // the batch of eight; the candidate itself is then looked for, where row 5 wins the cell)

        double b5[PPL];
        int i5[PPL];
#pragma unroll
        for (int h = 0; h < PPL; ++h) {
            b5[h] = INFINITY;
            i5[h] = 0;
        }
        if (mask & 0x20u) {
            if (FEW) {
                row5_least<PPL>(C, B, row5_candidates(C, B, nv, q_lo, q_hi), q, b5, i5);
            } else {
                // eight candidates per round trip to LDS; past the last competing one B is
                // +inf (and C is finite), so the value is +inf and never taken
                for (int s0 = 0; s0 < nv; s0 += 8) {
                    double Bv[8], Cv[8];
#pragma unroll
                    for (int u = 0; u < 8; ++u) {
                        Bv[u] = rowB[wave][s0 + u];
                        Cv[u] = sC[s0 + u];
                    }
#pragma unroll
                    for (int h = 0; h < PPL; ++h) {
                        double cur = INFINITY;
#pragma unroll
                        for (int u = 0; u < 8; ++u)
                            cur = min_f64(cur, __builtin_fma(q[h], Cv[u], Bv[u]));
                        i5[h] = cur < b5[h] ? s0 : i5[h];
                        b5[h] = min_f64(b5[h], cur);
                    }
                }
            }
        }

        plogp_cell_dev *o = obase + (size_t)mi * n_P;
        if (mask & 0x3FFu) {
#pragma unroll
            for (int h = 0; h < PPL; ++h) {
                const double t2 = amin < INFINITY ? __builtin_fma(q[h], amin, L) : INFINITY;
                const double t9 = amin < INFINITY ? __builtin_fma(fl[h], amin, clL[h]) : INFINITY;
                Best bc = decide_bcast(mask, q[h], fl[h], cl[h], gm, L, g1, t2, 0u, b5[h], 0u, t9, 0u);
                if (FEW) {
                    if (bc.id == 5u)
                        bc.s = sSv[i5[h]];
                } else if (__ballot(active[h] && bc.id == 5u) != 0) {
                    // the first candidate of the remembered batch that attains the minimum (lanes
                    // differ in their batch: per-lane LDS reads of its eight candidates)
                    double Bv[8], Cv[8];
#pragma unroll
                    for (int u = 0; u < 8; ++u) {
                        Bv[u] = rowB[wave][i5[h] + u];
                        Cv[u] = sC[i5[h] + u];
                    }
                    int at5 = i5[h];
#pragma unroll
                    for (int u = 7; u >= 0; --u)        // descending: the first match stays
                        at5 = __builtin_fma(q[h], Cv[u], Bv[u]) == b5[h] ? i5[h] + u : at5;
                    const uint32_t s_at = sSv[at5];
                    bc.s = bc.id == 5u ? s_at : bc.s;
                }
                // a winning row 2 or 9: the first candidate whose value equals the minimum
                bool open = active[h] && (bc.id == 2u || bc.id == 9u);
                if (__ballot(open) != 0) {
                    const double mul = bc.id == 2u ? q[h] : fl[h], add = bc.id == 2u ? L : clL[h];
                    uint32_t found = 0u;
                    for (int s0 = 0; s0 < nv; s0 += 4) {     // past the last candidate A is +inf
                        double Av[4];
                        uint32_t Sv[4];
#pragma unroll
                        for (int u = 0; u < 4; ++u) {
                            Av[u] = s0 + u < n_s ? S.segA[row_now * n_s + s0 + u] : INFINITY;
                            Sv[u] = sSv[s0 + u];
                        }
#pragma unroll
                        for (int u = 0; u < 4; ++u) {
                            const bool hit = open && __builtin_fma(mul, Av[u], add) == bc.t;
                            found = hit ? Sv[u] : found;
                            open = open && !hit;
                        }
                        if (__ballot(open) == 0)
                            break;
                    }
                    if (bc.id == 2u || bc.id == 9u)
                        bc.s = found;
                }
                if (active[h])
                    store_cell(o + 64 * h, bc);
            }
            o += plane;
        }
        if (mask & 0x1C00u) {
            double s11[PPL];
#pragma unroll
            for (int h = 0; h < PPL; ++h)
                s11[h] = 0.0;
            if (chain) {
                double done[PPL];
                if (!G.blk_is_prefix) {
                    // the finished blocks are added in ascending order, the same sum in every
                    // lane; a lane keeps, per process count, the value that belongs to its block
                    const double tot = dn[0];
                    double acc = 0.0;
                    for (int b = 0; b < bmin[0]; ++b)
                        acc = acc + __hiloint2double(
                                        __builtin_amdgcn_readlane(__double2hiint(tot), b),
                                        __builtin_amdgcn_readlane(__double2loint(tot), b));
#pragma unroll
                    for (int h = 0; h < PPL; ++h)
                        done[h] = acc;               // lanes of block bmin[0]
                    for (int b = bmin[0]; b < bmax[PPL - 1]; ++b) {
                        acc = acc + __hiloint2double(
                                        __builtin_amdgcn_readlane(__double2hiint(tot), b),
                                        __builtin_amdgcn_readlane(__double2loint(tot), b));
#pragma unroll
                        for (int h = 0; h < PPL; ++h)
                            done[h] = blk[h] == b + 1 ? acc : done[h];
                    }
                } else {
#pragma unroll
                    for (int h = 0; h < PPL; ++h)
                        done[h] = dn[h];
                }
#pragma unroll
                for (int h = 0; h < PPL; ++h)
                    s11[h] = done[h] + part[h];
            }
#pragma unroll
            for (int h = 0; h < PPL; ++h)
                if (active[h])
                    store_cell(o + 64 * h, decide_scatter(mask, q[h], cl[h], gm, L, s11[h], s12[h]));
        }
        if (!FEW)
            __builtin_amdgcn_wave_barrier();
    }
}

// ---- sweep, many candidates: lanes over s, most of them never evaluated --------
//
// A workgroup takes one (table, m) and up to SWEEP_S_WAVES groups of GP process counts, one group
// per wave.  For row 5, min over s of fma(P-1, C, B), the candidates are cut into chunks of 64
// consecutive ones: rounding is monotone, so fma(P-1, min C, min B) over a chunk is not above any
// of its values, and a chunk whose bound lies above a value already found cannot hold the minimum
// (nor tie with it).  The workgroup computes A and B of every candidate of a pass once (B to LDS),
// the minimum of B per chunk (that of C does not depend on m and comes from the tuning's first
// step) and the minima of A; a wave then takes, per process count, the smallest of the chunks'
// first candidates as an upper bound, compares it with the bounds of all chunks (two per lane),
// and evaluates the chunks that some process count of its group still needs.  On 8192 candidates
// and 69 process counts that is 7 of 128 chunks per wave on average (1024 sizes up to 1 GiB, one
// table: kernel 76 -> about 40 us, the call 89 -> 51; with every candidate evaluated it was bound
// by its fp64 instructions).  What is left, in us of the call: the step before 10, A and B of
// every candidate 18, upper bounds and bounds 9, the chunks 10, rows 2 and 9 3.  It is bound by
// latency at 16 waves per compute unit (64 KB of B per workgroup, 110 registers); passes of 4096
// (100 us), groups of six process counts in two workgroups (67) and loads one step ahead in the
// filling (56, spills) are slower.
constexpr int SWEEP_S_WAVES = 8;
constexpr int SWEEP_S_PASS = 8192;      // candidates per pass: 64 KB of LDS, two workgroups per CU
constexpr int SWEEP_S_CHUNKS = SWEEP_S_PASS / 64;
constexpr int SWEEP_S_RANGE = SWEEP_S_PASS / SWEEP_S_WAVES;   // candidates of a whole pass that a wave fills
constexpr int SWEEP_S_RANGES = 64;      // ranges whose minimum of A is remembered

template <int GP, int OCC>
__global__ void __launch_bounds__(64 * SWEEP_S_WAVES, OCC)
k_sweep_s(DeviceTables T, DeviceGrid G, Scratch S, plogp_cell_dev *out, int n_ptiles)
{
    extern __shared__ __align__(16) double sweep_lds[];          // B of the candidates of a pass
    __shared__ double minB[SWEEP_S_CHUNKS], firstB[SWEEP_S_CHUNKS], firstC[SWEEP_S_CHUNKS];
    __shared__ double rangeMinA[SWEEP_S_RANGES];                  // min of A over each of the first ranges
    __shared__ double fillMinA[SWEEP_S_WAVES];                    // per wave: over the ranges it filled
    double *sB = sweep_lds;

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    int bid = blockIdx.x;
    const int ptile = bid % n_ptiles;
    bid /= n_ptiles;
    const int mi = bid % G.n_m;
    const int t = bid / G.n_m;
    const int p0 = (ptile * SWEEP_S_WAVES + wave) * GP;           // first P index of this wave
    const bool has_work = p0 < G.n_P;

    const double md = (double)G.m[mi];
    const double L = T.L[t];
    const uint32_t mask = G.mask;
    const double *gs = S.gs + (size_t)t * G.n_s;
    const double *minG = S.minG + (size_t)t * ((G.n_s + 63) / 64);
    const int nv = S.nv[mi];                                      // candidates s <= min(m, s_cap)

    double q[GP];                                                 // wave-uniform: kept in scalar registers
#pragma unroll
    for (int p = 0; p < GP; ++p) {
        const uint32_t Pv = (p0 + p < G.n_P) ? G.P[p0 + p] : 2u;
        const double qv = (double)(Pv - 1);
        q[p] = __hiloint2double(__builtin_amdgcn_readfirstlane(__double2hiint(qv)),
                                __builtin_amdgcn_readfirstlane(__double2loint(qv)));
    }
    // What lane p < GP needs at the end to decide its cells is asked for now, so that the end
    // of the wave does not wait for device memory: its process count, g(m), g(1), the two
    // Scatter sums.
    const int pi = p0 + lane;
    const bool mine = lane < GP && pi < G.n_P;
    uint32_t Pv = 2u;
    double gm = 0.0, g1 = 0.0, s11 = 0.0, s12 = 0.0;
    if (has_work) {
        Pv = G.P[mine ? pi : G.n_P - 1];
        gm = S.gm[(size_t)t * G.n_m + mi];
        g1 = S.g1[t];
        if (mine && (mask & (1u << 11)))
            s11 = chain_sum_of(G, S, t, mi, pi, Pv);
        if (mine && (mask & (1u << 12)))
            s12 = S.sum2[((size_t)t * G.n_m + mi) * (size_t)(G.cl_max + 1) + ceil_log2(Pv)];
    }

    double least_A = INFINITY;                                    // over the candidates this thread filled
    // The minimum of row 5 per process count, the same in every lane.  (The +inf at the start goes
    // through a vector register: as a constant this compiler moves it into a scalar pair with one
    // 64-bit literal, which the hardware does not have - it reads as 0.)
    double V5p[GP], unset = INFINITY;
    asm("" : "+v"(unset));
#pragma unroll
    for (int p = 0; p < GP; ++p)
        V5p[p] = unset;
    int at5 = 0;                                                  // lane p: the first candidate that attains V5p[p]
    for (int s0 = 0; s0 < nv; s0 += SWEEP_S_PASS) {
        const int n_here = nv - s0 < SWEEP_S_PASS ? nv - s0 : SWEEP_S_PASS;
        const int n_chunks = (n_here + 63) >> 6;
        if (s0 > 0)
            __syncthreads();                                      // every wave is done with the pass before
        // this wave's range of the pass, four chunks at a time (their loads side by side): an eighth
        // of the chunks when one pass takes them all (1000 candidates x 250 sizes x 69 process counts:
        // 18.2 us, 19.3 when the first wave fills all 1000), SWEEP_S_RANGE candidates else, so that a
        // range whose minimum is remembered below has a place of its own
        const int per_wave = nv <= SWEEP_S_PASS ? (n_chunks + SWEEP_S_WAVES - 1) / SWEEP_S_WAVES : SWEEP_S_RANGE / 64;
        const int c_end = (wave + 1) * per_wave < n_chunks ? (wave + 1) * per_wave : n_chunks;
        double range_A = INFINITY;
        for (int c0 = wave * per_wave; c0 < c_end; c0 += 4) {
            const int first = s0 + 64 * c0;
            auto fill = [&](bool whole) {                         // whole: all 256 candidates compete
                uint32_t f_s[4];
                double f_rcp[4], f_gs[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    if (!whole && c0 + u >= c_end)
                        continue;
                    const int si = first + 64 * u + lane, idx = whole || si < nv ? si : nv - 1;
                    f_s[u] = *reinterpret_cast<const uint32_t *>(G.s + idx);               // below 2^32
                    f_rcp[u] = S.rcp[idx];
                    f_gs[u] = gs[idx];
                }
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int c = c0 + u;
                    if (!whole && c >= c_end)
                        continue;
                    double A, B, C;
                    segment_terms(md, (double)f_s[u], f_rcp[u], f_gs[u], L, A, B, C);
                    range_A = min_f64(range_A, A);                // (past the end: the last one again)
                    sB[64 * c + lane] = whole || first + 64 * u + lane < nv ? B : INFINITY;
                    if (lane == 0) {
                        firstB[c] = B;
                        firstC[c] = C;
                    }
                }
            };
            if (c0 + 4 <= c_end && first + 256 <= nv)
                fill(true);
            else
                fill(false);
        }
        if (mask & 0x204u) {
            const double r = wave_min(range_A);
            least_A = min_f64(least_A, r);
            const int range = s0 / SWEEP_S_RANGE + wave;
            if (lane == 0 && range < SWEEP_S_RANGES)
                rangeMinA[range] = r;
        }
        __syncthreads();
        // the minimum of B per chunk: four threads to a chunk, each its quarter from an offset of
        // its own (no two chunks of a wave in one bank)
        {
            const int c = (int)threadIdx.x >> 2, part = (int)threadIdx.x & 3;
            double least = INFINITY;
            if (c < n_chunks) {
#pragma unroll
                for (int k = 0; k < 16; ++k)
                    least = min_f64(least, sB[64 * c + 16 * part + ((k + c) & 15)]);
            }
            least = min_f64(least, __shfl_xor(least, 1));
            least = min_f64(least, __shfl_xor(least, 2));
            if (part == 0)
                minB[c] = least;
        }
        __syncthreads();
        if (!has_work || (mask & 0x20u) == 0)
            continue;
        // the chunks that some process count of this wave needs
        u64 need[SWEEP_S_CHUNKS / 64];
        {
            double up[GP];
#pragma unroll
            for (int p = 0; p < GP; ++p)
                up[p] = INFINITY;
#pragma unroll
            for (int h = 0; h < SWEEP_S_CHUNKS / 64; ++h) {
                const int c = 64 * h + lane;
                if (64 * h < n_chunks) {
                    const double fb = c < n_chunks ? firstB[c] : INFINITY, fc = c < n_chunks ? firstC[c] : 0.0;
#pragma unroll
                    for (int p = 0; p < GP; ++p)
                        up[p] = min_f64(up[p], __builtin_fma(q[p], fc, fb));
                }
            }
#pragma unroll
            for (int p = 0; p < GP; ++p)
                up[p] = min_f64(up[p], V5p[p]);
            wave_min_each<GP>(up);
#pragma unroll
            for (int h = 0; h < SWEEP_S_CHUNKS / 64; ++h) {
                need[h] = 0;
                const int c = 64 * h + lane;
                if (64 * h < n_chunks) {
                    const double lb = minB[c], lc = c < n_chunks ? minG[s0 / 64 + c] + L : 0.0;
#pragma unroll
                    for (int p = 0; p < GP; ++p)
                        need[h] |= __ballot(__builtin_fma(q[p], lc, lb) <= up[p]);
                    if (n_chunks - 64 * h < 64)
                        need[h] &= (1ull << (n_chunks - 64 * h)) - 1ull;
                }
            }
        }
        double best5[GP], V[GP];
        int chunk5[GP];                                           // in which chunk this lane's minimum first appeared
#pragma unroll
        for (int p = 0; p < GP; ++p) {
            best5[p] = INFINITY;
            chunk5[p] = 0;
        }
#pragma unroll
        for (int h = 0; h < SWEEP_S_CHUNKS / 64; ++h) {
            for (u64 left = need[h]; left != 0; left &= left - 1) {
                const int c = 64 * h + __builtin_ctzll(left), e = 64 * c + lane;
                const double B = sB[e], C = gs[s0 + e < nv ? s0 + e : nv - 1] + L;
#pragma unroll
                for (int p = 0; p < GP; ++p) {
                    const double T5 = __builtin_fma(q[p], C, B);
                    chunk5[p] = T5 < best5[p] ? c : chunk5[p];
                    best5[p] = min_f64(best5[p], T5);
                }
            }
        }
#pragma unroll
        for (int p = 0; p < GP; ++p)
            V[p] = best5[p];
        wave_min_each<GP>(V);
        // the process counts whose minimum this pass lowers: the first candidate that attains it
#pragma unroll
        for (int p = 0; p < GP; ++p) {
            if (!(V[p] < V5p[p]))
                continue;
            V5p[p] = V[p];
            int first = 0x7FFFFFFF;
            for (u64 holders = __ballot(best5[p] == V[p]); holders != 0; holders &= holders - 1) {
                const int l = __builtin_ctzll(holders);           // more than one lane only on exact ties
                const int at = s0 + 64 * __builtin_amdgcn_readlane(chunk5[p], l) + l;
                first = at < first ? at : first;
            }
            at5 = lane == p ? first : at5;
        }
    }
    double V5 = INFINITY;                                         // lane p: of process count p0 + p
#pragma unroll
    for (int p = 0; p < GP; ++p)
        V5 = lane == p ? V5p[p] : V5;
    if (mask & 0x204u) {
        if (lane == 0)
            fillMinA[wave] = least_A;
        __syncthreads();
    }
    if (!has_work)
        return;
    double Aw = INFINITY;
    if (mask & 0x204u)
#pragma unroll
        for (int w = 0; w < SWEEP_S_WAVES; ++w)
            Aw = min_f64(Aw, fillMinA[w]);
    const bool haveA = Aw < INFINITY;

    // lanes 0..GP-1 decide one Broadcast cell each: the segmented rows' minima, the
    // unsegmented rows, arg-min.  The segment size of rows 2 and 9 is looked for afterwards, and
    // only in the cells that they win.
    const double qv = (double)(Pv - 1);
    const int fli = floor_log2(Pv), cli = ceil_log2(Pv);
    const size_t plane = (size_t)G.n_m * G.n_P;
    plogp_cell_dev *o = out + (size_t)t * G.n_ops * plane + (size_t)mi * G.n_P + (mine ? pi : 0);
    if (mask & 0x3FFu) {
        const double t2 = ((mask & (1u << 2)) && haveA) ? __builtin_fma(qv, Aw, L) : INFINITY;
        const double t9 = ((mask & (1u << 9)) && haveA)
                              ? __builtin_fma((double)fli, Aw, (double)cli * L) : INFINITY;
        Best bc = decide_bcast(mask, qv, (double)fli, (double)cli, gm, L, g1, t2, 0u, V5, 0u, t9, 0u);
        if (mine && bc.id == 5u)
            bc.s = (uint32_t)G.s[at5];
        u64 seek = __ballot(mine && (bc.id == 2u || bc.id == 9u));
        if (seek != 0) {
            // The first candidate whose value equals the minimum, for all these cells at once.
            // With a single pass the chunks' minima of B are still there: exactly, g(s) k is
            // g(s) (k - 1) + g(s), so A is not below min B + min g of its chunk but for roundings, and
            // few chunks can hold it.  g(s) has either sign (a falling table goes on falling past its
            // last sample).  Where it is not negative, A >= (B + g)(1 - 2u), u = 2^-53, and a sum below
            // zero is below A anyhow; where it is, A >= B + g - 2u(|B| + |g|), and neither of these two
            // is larger than that of the minimum, which is not above it.  So A needs 2u(|min B| +
            // |min g|) of room and the two roundings of the bound itself half of that each; it is given
            // 8u.  After several passes the first range whose minimum of A gives the value is walked
            // from its start.
            auto from_lane = [&](double v, int l) {
                return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), l),
                                        __builtin_amdgcn_readlane(__double2loint(v), l));
            };
            const double mul_l = bc.id == 2u ? qv : (double)fli, add_l = bc.id == 2u ? L : (double)cli * L;
            const int n_chunks = (nv + 63) >> 6;
            u64 may[SWEEP_S_CHUNKS / 64];
            int c_first = 0;
            const bool single = nv <= SWEEP_S_PASS;
            if (single) {
#pragma unroll
                for (int h = 0; h < SWEEP_S_CHUNKS / 64; ++h) {
                    const int c = 64 * h + lane;
                    may[h] = 0;
                    if (64 * h >= n_chunks)
                        continue;
                    const double lb = c < n_chunks ? minB[c] : INFINITY, lg = c < n_chunks ? minG[c] : 0.0;
                    const double low = (lb + lg) - 0x1p-50 * (fabs(lb) + fabs(lg));
                    for (u64 k = seek; k != 0; k &= k - 1) {
                        const int p = __builtin_ctzll(k);
                        may[h] |= __ballot(__builtin_fma(from_lane(mul_l, p), low, from_lane(add_l, p)) <=
                                           from_lane(bc.t, p));
                    }
                }
            } else {
                const int n_ranges = (nv + SWEEP_S_RANGE - 1) / SWEEP_S_RANGE;
                const int known = n_ranges < SWEEP_S_RANGES ? n_ranges : SWEEP_S_RANGES;
                u64 holds = 0;
                for (u64 k = seek; k != 0; k &= k - 1) {
                    const int p = __builtin_ctzll(k);
                    const u64 in = __ballot(lane < known && __builtin_fma(from_lane(mul_l, p), rangeMinA[lane],
                                                                          from_lane(add_l, p)) == from_lane(bc.t, p));
                    holds |= in != 0 ? in : 1ull << (known - 1);   // beyond the ranges remembered
                }
                c_first = __builtin_ctzll(holds) * (SWEEP_S_RANGE / 64);
            }
            while (c_first < n_chunks && seek != 0) {
                int c[2];                                         // the next two chunks
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    if (single) {
                        while (c_first < n_chunks && ((may[c_first >> 6] >> (c_first & 63)) & 1ull) == 0) {
                            const u64 rest = may[c_first >> 6] >> (c_first & 63);
                            c_first = rest != 0 ? c_first + __builtin_ctzll(rest) : (c_first | 63) + 1;
                        }
                    }
                    c[u] = c_first < n_chunks ? c_first : n_chunks - 1;
                    ++c_first;
                }
                double sdv[2], A[2];
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    const int si = 64 * c[u] + lane, idx = si < nv ? si : nv - 1;
                    sdv[u] = (double)*reinterpret_cast<const uint32_t *>(G.s + idx);
                    double B, C;
                    segment_terms(md, sdv[u], S.rcp[idx], gs[idx], L, A[u], B, C);
                    A[u] = si < nv ? A[u] : INFINITY;
                }
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    for (u64 k = seek; k != 0; k &= k - 1) {
                        const int p = __builtin_ctzll(k);
                        const u64 hits = __ballot(__builtin_fma(from_lane(mul_l, p), A[u], from_lane(add_l, p)) ==
                                                  from_lane(bc.t, p));
                        if (hits != 0) {
                            const uint32_t sv = (uint32_t)from_lane(sdv[u], __builtin_ctzll(hits));
                            bc.s = lane == p ? sv : bc.s;
                            seek &= ~(1ull << p);
                        }
                    }
                }
            }
        }
        if (mine)
            store_cell(o, bc);
        o += plane;
    }
    if (!mine)
        return;
    if (mask & 0x1C00u)
        store_cell(o, decide_scatter(mask, qv, (double)cli, gm, L, s11, s12));
}

// The kernel for gp process counts per wave.  Few process counts go two or four to a wave, so that
// more waves take part (10 of them, 1000 candidates x 1500 sizes: the call 28 us by two, 34 by
// six).  Up to four, registers allow three workgroups per CU; six fit only if four registers are
// spilled, which pays where three workgroups find work and room in LDS (`dense`; 40 process counts,
// 1000 candidates x 1500 sizes: 39 us with two workgroups, 36 with three; 8192 candidates, two
// workgroups either way: 60 without the spilling, 62 with it).
static auto sweep_s_kernel(int gp, bool dense)
{
    return gp == 2 ? k_sweep_s<2, 6> : gp == 4 ? k_sweep_s<4, 6> : gp == 6 ? (dense ? k_sweep_s<6, 6> : k_sweep_s<6, 4>)
           : gp == 9 ? k_sweep_s<9, 4> : k_sweep_s<12, 4>;
}

// LDS of a workgroup: B of the candidates of a pass; with_static: the arrays the kernel declares too.
static size_t sweep_s_lds(int n_s, bool with_static)
{
    const int pass = n_s < SWEEP_S_PASS ? (n_s + 63) / 64 * 64 : SWEEP_S_PASS;
    return ((size_t)pass + (with_static ? 3 * SWEEP_S_CHUNKS + SWEEP_S_RANGES + SWEEP_S_WAVES : 0)) * sizeof(double);
}

// ---- whole path of a tile of message sizes of one table in one workgroup -------
//
// Batches of tables that do not share their sample sizes (or are too few for lanes over
// tables).  A workgroup takes one table and up to TILE_MAX_M message sizes and does every step
// for them with LDS between the steps: the table as intervals; the candidates; the terms of
// every (m, s); the Scatter-chain sums; then the cells, lanes over (m, P) in the order of the
// output, so that a wave stores whole cache lines.
//
// The chain sums are half of the work.  Their items are (block of SUM_BLOCK terms, m); within a
// block most items stay inside one interval of the table or enter one other, and only the first
// blocks enter many.  A wave that mixes the kinds pays for the worst.  So every item is first
// placed (one search) and sorted: by whether it enters no interval (three fp64 instructions per
// term), one, and among which eight of its terms (lanes that enter together cost a walk one turn
// more over these eight, see walk_terms, and none elsewhere), or more; and the waves take 64 of
// that order at a time, from its end, whatever the kind: a list per kind left lanes idle in the
// last wave of each.  Waves of which some item enters as many intervals as TILE_REACH says search for
// eight terms side by side (gaps_ascending).
//
// 333 tables of 57 samples x 203 sizes x 37 process counts up to 1500, 19 candidates, 80 MB of
// cells: 63 us a call (68 with the change of interval as six selects per term of the items that
// enter one, a list per kind and the mask of rows read at run time; a lane per message size that
// walks its whole row alone took 175; 10 000 rows x 1000 process counts 2500 us, now the row path's
// 82); 1000 tables 178 -> 168; 300 tables of 30 samples x 150 sizes x 20 process counts up to 300
// 31.4 -> 28.3.  Bound by vector instruction issue (25.8 million, 29.8 before), a third of it the
// cells.  With few process counts a tile has few items, often less than a wave of the slowest kind, which the
// other waves wait for: eight lanes share each of these then, where the chip waits too (see tile_shared), and
// the items that enter one interval, a wave of walks of many turns, go first, so that the shared ones fill up
// the time of the other waves (227 tables of 20 samples x 22 sizes x 7 process counts up to 667, 242 items of
// a tile, 25 of them shared: 12.6 us, 13.9 with the shared ones first, 15.1 with a lane per item, 13.4
// shared before lists of one interval's items as selects; on 50 samples, 40 shared of 176 and 8 up to 455, 14.6,
// 16.0 and 16.2).
// Tried: the cells of the Broadcast plane handed out with the items, for waves that have nothing left
// of these (the same time: there is no idle time to fill, and a lane has to find its cell by a
// division); the searched terms of large jobs spread over all threads through LDS (94 us).
constexpr int TILE_THREADS = 256;
constexpr int TILE_MAX_M = TILE_THREADS / 8;
constexpr int TILE_NS = 24;              // candidates at most
constexpr int TILE_MAX_BLK = 32;         // blocks of the chain sum at most
constexpr size_t TILE_STATIC_LDS = 256;  // room for the counters
constexpr long TILE_MIN_ROWS = 16;       // (table, m) rows per compute unit at least (more than TILE_FEW_N samples: twice)
constexpr int TILE_FEW_N = 512;
constexpr int TILE_WG_PER_CU = 6;        // that their registers leave room for
constexpr int TILE_DENSE_N = 40;         // from so many samples on a table's blocks enter more intervals
// Intervals entered by some lane's block from which on a wave searches (as WALK_REACH): the second from TILE_DENSE_N
// samples on, where the blocks of the last kind enter many (95 samples, 32 tables x 137 sizes 21.9 us with 16, 20.2 so,
// 300 tables 31.9 and 30.5; 57 samples, 333 tables no difference), the first else (25 samples, 60 tables x 95 sizes 17.2,
// 18.1 with 4).
constexpr int TILE_REACH = 16, TILE_REACH_DENSE = 4;
static_assert(power_of_two(TILE_REACH) && power_of_two(TILE_REACH_DENSE), "compared with what wave_reach gives");

// Where the arrays of a workgroup start in LDS, in 8-byte slots.  The lists of the chain items lie
// where A and B of every (m, s) go afterwards.
struct TileLds {
    int ab, list, c, gs, rcp, gm, amin, md, sum2, tot, part, mask, sv, sp, off, slots;
    int nsp;             // candidates, padded to a multiple of four
    __host__ __device__ TileLds(int n, int n_s, int n_P, int n_blk, int cl_max, int M)
    {
        nsp = (n_s + 3) & ~3;
        int at = 4 * n + (int)CHAIN_PAD;
        ab = list = at;
        const int after = list + (M * n_blk + 1) / 2;
        at += 2 * M * nsp;
        at = at > after ? at : after;
        c = at; at += nsp;
        gs = at; at += nsp;
        rcp = at; at += nsp;
        gm = at; at += M;
        amin = at; at += M;
        md = at; at += M;
        sum2 = at; at += M * (cl_max + 1);
        tot = at; at += M * n_blk;
        part = at; at += M * n_P;
        mask = at; at += n_blk;
        sv = at; at += (nsp + 1) / 2;
        sp = at; at += (n_P + 1) / 2;
        off = at; at += (n_blk + 1) / 2;
        slots = at;
    }
};

constexpr int TILE_KINDS = 10;           // no interval entered, one at the 8k-th term or after, more

// An item of the chain sums on a list: size within the tile, block, interval of its first term.
__device__ __forceinline__ unsigned tile_item(int ml, int b, int i)
{
    return (unsigned)ml | (unsigned)b << 5 | (unsigned)i << 10;
}

// One item per lane; dense: some lane's enters several intervals.  `real` lanes store.
__device__ __forceinline__ void tile_sum(const ChainCtx &C, unsigned item, bool real, bool dense, const double *m_of, int M,
                                         const u64 *blk_mask, const int *blk_off, int n_P, double *part, double *tot)
{
    const int ml = (int)(item & 31u), b = (int)((item >> 5) & 31u), i = (int)(item >> 10);
    const double md = m_of[ml];
    const double z0 = (double)(b * SUM_BLOCK + 1) * md;                      // exact: an integer below 2^53
    const u64 wanted = real ? blk_mask[b] : 0ull;
    double *out = part + ml * n_P + blk_off[b];
    const u64 any = wave_any_wanted(wanted);
    double run;
    if (dense) {
        const int reach = block_reach(C, z0, md, i);
        if (reach > (C.n >= TILE_DENSE_N ? TILE_REACH_DENSE : TILE_REACH)) {
            run = block_search(C, i, reach, md, z0, wanted, any, out);
            if (real)
                tot[b * M + ml] = run;
            return;
        }
    }
    WalkAt at = {i, z0 - C.X[i], C.W[i], C.YS[i]};
    run = walk_block(C, at, md, wanted, any, out);
    if (real)
        tot[b * M + ml] = run;
}

// The same for few items: eight lanes to an item, a lane searches for eight of the terms.  The sum is
// handed from lane to lane (every lane adds its terms in every round; in round r the r-th lane of an
// item holds the sum of the terms before its own).
__device__ __forceinline__ void tile_search_shared(const ChainCtx &C, unsigned item, bool real, const double *m_of, int M,
                                                   const u64 *blk_mask, const int *blk_off, int n_P, double *part,
                                                   double *tot)
{
    constexpr int V = SUM_BLOCK / 8;
    const int q = (int)threadIdx.x & 7;
    const int ml = (int)(item & 31u), b = (int)((item >> 5) & 31u), i0 = (int)(item >> 10);
    const double md = m_of[ml], zb = (double)(b * SUM_BLOCK + 1) * md;
    const int reach = block_reach(C, zb, md, i0);
    const double zq = __builtin_fma((double)(V * q), md, zb);
    double z[V], g[V];
#pragma unroll
    for (int c = 0; c < V; ++c)
        z[c] = __builtin_fma((double)c, md, zq);
    gaps_within<V>(C, i0, reach, z, g);
    const u64 wanted = real ? blk_mask[b] : 0ull;
    // (32-bit shifts: a 64-bit one whose amount sits in the last register of the wave's allocation does
    // not read that register on this hardware, and the compiler does not know)
    const unsigned lo = (unsigned)wanted, hi = (unsigned)(wanted >> 32), shift = V * (q & 3);
    const unsigned half = q < 4 ? lo : hi;
    const unsigned mine = half >> shift & 0xFFu;
    double *out = part + ml * n_P + blk_off[b] + __builtin_popcount(half & ((1u << shift) - 1u)) +
                  (q < 4 ? 0 : __builtin_popcount(lo));
    double run = 0.0;
#pragma unroll 1
    for (int r = 0; r < 8; ++r) {
        if (r > 0)
            run = dpp_move<0x111, 0xf>(run);       // row_shr:1
        if (__ballot(q == r && mine != 0u) != 0) {
#pragma unroll
            for (int c = 0; c < V; ++c) {
                if (q == r && ((mine >> c) & 1u))
                    *out++ = run;
                run = run + g[c];
            }
        } else {
#pragma unroll
            for (int c = 0; c < V; ++c)
                run = run + g[c];
        }
    }
    if (real && q == 7)
        tot[b * M + ml] = run;
}

template <bool ALL>
__global__ void __launch_bounds__(TILE_THREADS, TILE_WG_PER_CU)
k_tile(DeviceTables T, DeviceGrid G, plogp_cell_dev *out, int n_tiles, int M, int shared)
{
    // (a name of its own: under a name that another kernel declares without it the alignment is lost,
    // and 16-byte reads of misaligned LDS take twice the kernel's time)
    extern __shared__ __align__(16) double tile_lds[];
    __shared__ unsigned count[TILE_KINDS], next_wave, nv_tile;
    __shared__ double sh_g1;
    const int n_s = G.n_s, n_P = G.n_P, n_blk = G.n_blk, cl_max = G.cl_max;
    const TileLds A(T.n, n_s, n_P, n_blk, cl_max, M);
    const int tid = (int)threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int t = (int)blockIdx.x / n_tiles, m0 = (int)blockIdx.x % n_tiles * M;
    const int n_m = G.n_m - m0 < M ? G.n_m - m0 : M;           // sizes of this tile
    const uint32_t mask = ALL ? 0x1FFFu : G.mask;
    const bool chain = (mask & (1u << 11)) != 0, binom = (mask & (1u << 12)) != 0;
    f64x2 *sAB = reinterpret_cast<f64x2 *>(tile_lds + A.ab);
    double *sC = tile_lds + A.c, *sG = tile_lds + A.gs, *sR = tile_lds + A.rcp, *sGm = tile_lds + A.gm, *sM = tile_lds + A.md;
    double *sAmin = tile_lds + A.amin;
    double *sum2 = tile_lds + A.sum2, *tot = tile_lds + A.tot, *part = tile_lds + A.part;
    u64 *sMask = reinterpret_cast<u64 *>(tile_lds + A.mask);
    unsigned *list = reinterpret_cast<unsigned *>(tile_lds + A.list);
    uint32_t *sSv = reinterpret_cast<uint32_t *>(tile_lds + A.sv), *sP = reinterpret_cast<uint32_t *>(tile_lds + A.sp);
    int *sOff = reinterpret_cast<int *>(tile_lds + A.off);
    const double L = T.L[t];
    ChainCtx C;
    stage_intervals(C, tile_lds, T, t);
    for (int p = tid; p < n_P; p += TILE_THREADS)
        sP[p] = G.P[p];
    for (int b = tid; b < n_blk; b += TILE_THREADS) {
        sMask[b] = G.blk_mask[b];
        sOff[b] = G.blk_off[b];
    }
    if (tid < n_m)
        sM[tid] = (double)G.m[m0 + tid];
    if (tid < TILE_KINDS)
        count[tid] = 0u;
    if (tid == 64)
        next_wave = 0u;
    if (tid == 65)
        nv_tile = 0u;
    __syncthreads();

    // what needs the table only: g(s), g(m), g(1), the terms g(2^j m), the places of the chain items
    auto gap = [&](double z) {
        const double zz[1] = {z};
        int i[1];
        chain_locate<1>(C.X, C.n, zz, i);
        const f64x2 ys = C.YS[i[0]];
        return __builtin_fma(ys.y, z - C.X[i[0]], ys.x);
    };
    if (tid < A.nsp) {
        const bool there = tid < n_s;
        const double sd = there ? (double)G.s[tid] : 1.0;
        const double gs = there ? gap(sd) : 0.0;
        sG[tid] = gs;
        sR[tid] = 1.0 / sd;
        sC[tid] = gs + L;
        sSv[tid] = there ? (uint32_t)sd : 0u;
    }
    if (tid >= 64 && tid < 64 + n_m)
        sGm[tid - 64] = gap(sM[tid - 64]);
    if (tid == 128)
        sh_g1 = gap(1.0);
    if (binom)
        for (int ml = tid >> 3; ml < n_m; ml += TILE_THREADS / 8)
            for (int j = tid & 7; j < cl_max; j += 8)
                sum2[ml * (cl_max + 1) + j + 1] = gap(sM[ml] * (double)(1ull << j));  // exact: below 2^53
    const int n_items = chain ? n_m * n_blk : 0;
    constexpr int PER = TILE_MAX_M * TILE_MAX_BLK / TILE_THREADS;              // items of a thread at most
    unsigned item[PER], place[PER];                                            // kind, its place among those of its kind
    {
        const int step_b = TILE_THREADS / n_m, step_m = TILE_THREADS % n_m;
        int b = tid / n_m, ml = tid % n_m;     // the next item of this thread: b n_m + ml
#pragma unroll
        for (int h = 0; h < PER; h += 2) {
            place[h] = place[h + 1] = ~0u;
            if (wave * 64 + h * TILE_THREADS >= n_items)
                continue;
            double z[2], md[2];                                                // two searches side by side
            int i[2], bb[2], mm[2];
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                bb[c] = b;
                mm[c] = ml;
                md[c] = sM[ml];
                z[c] = (double)(b * SUM_BLOCK + 1) * md[c];
                b += step_b;
                ml += step_m;
                if (ml >= n_m) {
                    ml -= n_m;
                    ++b;
                }
            }
            chain_locate<2>(C.X, C.n, z, i);
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                if (bb[c] >= n_blk)
                    continue;
                const double last = __builtin_fma((double)(SUM_BLOCK - 1), md[c], z[c]), x1 = C.X[i[c] + 1];
                unsigned kind = 0;
                if (last >= x1) {
                    // terms before the next interval, near enough
                    int before = (int)((float)(x1 - z[c]) * __builtin_amdgcn_rcpf((float)md[c]));
                    before = before < 0 ? 0 : before >= SUM_BLOCK ? SUM_BLOCK - 1 : before;
                    kind = last >= C.X[i[c] + 2] ? TILE_KINDS - 1 : 1u + (unsigned)before / 8u;
                }
                item[h + c] = tile_item(mm[c], bb[c], i[c]);
                place[h + c] = kind << 16 | atomicAdd(&count[kind], 1u);
            }
        }
    }
    __syncthreads();
    unsigned n0 = 0, n1 = 0, n2 = 0;
    if (chain) {
        // in the order of their kinds
        unsigned at = 0;
        unsigned first[TILE_KINDS];                                           // in scalar registers: nothing spills
#pragma unroll
        for (int k = 0; k < TILE_KINDS; ++k) {
            first[k] = at;
            at += (unsigned)__builtin_amdgcn_readfirstlane((int)count[k]);
        }
        n0 = first[1];
        n2 = at - first[TILE_KINDS - 1];
        n1 = at - n0 - n2;
#pragma unroll
        for (int h = 0; h < PER; ++h) {
            if (place[h] != ~0u) {
                unsigned to = 0;
#pragma unroll
                for (int k = 1; k < TILE_KINDS; ++k)
                    to = place[h] >> 16 == (unsigned)k ? first[k] : to;
                list[to + (place[h] & 0xFFFFu)] = item[h];
            }
        }
        __syncthreads();
    }

    // the prefix of g(2^j m)
    if (binom && tid >= TILE_THREADS - 64 && tid - (TILE_THREADS - 64) < n_m) {
        double *p = sum2 + (tid - (TILE_THREADS - 64)) * (cl_max + 1), acc = 0.0;
        p[0] = 0.0;
        for (int j = 1; j <= cl_max; ++j) {
            acc = acc + p[j];
            p[j] = acc;
        }
    }
    if (chain) {
        // 64 items at a time, the slowest first
        const bool share = n2 <= 64u && n_items <= shared;
        const unsigned w1 = share ? (n1 + 63) / 64 : 0u, w2 = share ? (n2 + 7) / 8 : 0u;
        const unsigned rest = w2 != 0u ? n0 + n1 : (unsigned)n_items;
        for (;;) {
            unsigned k = 0;
            if (lane == 0)
                k = atomicAdd(&next_wave, 1u);
            k = __builtin_amdgcn_readfirstlane(k);
            if (k >= w2 + (rest + 63) / 64)
                break;
            if (k - w1 < w2) {                                                // (k >= w1)
                const unsigned e = (k - w1) * 8 + (lane >> 3);
                tile_search_shared(C, list[n0 + n1 + (e < n2 ? e : n2 - 1)], e < n2, sM, M, sMask, sOff, n_P, part, tot);
            } else {
                const unsigned e = (k < w1 ? k : k - w2) * 64, at = e + lane;
                tile_sum(C, list[at < rest ? rest - 1 - at : 0u], at < rest, rest - e > n0 + n1, sM, M, sMask, sOff, n_P,
                         part, tot);
            }
        }
        __syncthreads();
        if (tid >= TILE_THREADS - 64 && tid - (TILE_THREADS - 64) < n_m) {     // the finished blocks, in ascending order
            double *p = tot + (tid - (TILE_THREADS - 64)), acc = 0.0;
            for (int b = 0; b < n_blk; ++b) {
                const double v = p[b * M];
                p[b * M] = acc;
                acc = acc + v;
            }
        }
    }
    // the terms of every (m, s): eight threads per message size, TILE_MAX_M sizes at once
    {
        const int ml = tid >> 3;
        double least = INFINITY;
        int top = 0;
        if (ml < n_m) {
            const double md = sM[ml];
            const double lim = (double)(G.s_cap < (1ull << 53) ? G.s_cap : (1ull << 53));
            for (int si = tid & 7; si < A.nsp; si += 8) {
                f64x2 ab = {INFINITY, INFINITY};
                const double sd = (double)sSv[si];
                if (si < n_s && sd <= md && sd <= lim) {
                    double a, bb, cc;
                    segment_terms(md, sd, sR[si], sG[si], L, a, bb, cc);
                    ab.x = a;
                    ab.y = bb;
                    least = min_f64(least, a);
                    top = si + 1;
                }
                sAB[ml * A.nsp + si] = ab;
            }
        }
#pragma unroll
        for (int x = 1; x < 8; x <<= 1) {
            least = min_f64(least, __shfl_xor(least, x));
            const int other = __shfl_xor(top, x);
            top = other > top ? other : top;
        }
        if (ml < n_m && (tid & 7) == 0) {
            sAmin[ml] = least;
            atomicMax(&nv_tile, (unsigned)top);
        }
    }
    __syncthreads();

    // the cells, in the order of the output
    const double g1 = sh_g1;
    const int nv = (int)nv_tile;
    const size_t plane = (size_t)G.n_m * n_P;
    plogp_cell_dev *const o0 = out + (size_t)t * G.n_ops * plane + (size_t)m0 * n_P;
    const bool has_b = (mask & 0x3FFu) != 0, has_s = (mask & 0x1C00u) != 0;
    const int dm = TILE_THREADS / n_P, dp = TILE_THREADS % n_P;
    int ml = tid / n_P, pi = tid % n_P;
    for (int e0 = tid - lane; e0 < n_m * n_P; e0 += TILE_THREADS) {
        const bool active = ml < n_m;
        const int mr = active ? ml : n_m - 1, pr = active ? pi : n_P - 1, e = mr * n_P + pr;
        const uint32_t P = sP[pr];
        const int cli = ceil_log2(P);
        const double q = (double)(P - 1u), fl = (double)floor_log2(P), cl = (double)cli, gm = sGm[mr];
        plogp_cell_dev *o = o0 + e;
        if (has_b) {
            const f64x2 *ab = sAB + mr * A.nsp;
            const double clL = cl * L, amin = sAmin[mr];
            double b5 = INFINITY;
            int at5 = 0;
            if (mask & 0x20u) {
                // four candidates at a time; the four in which the minimum first appeared are
                // remembered
                for (int s0 = 0; s0 < nv; s0 += 4) {
                    double cur = INFINITY;
#pragma unroll
                    for (int u = 0; u < 4; ++u)
                        cur = min_f64(cur, __builtin_fma(q, sC[s0 + u], ab[s0 + u].y));
                    at5 = cur < b5 ? s0 : at5;
                    b5 = min_f64(b5, cur);
                }
            }
            const double t2 = amin < INFINITY ? __builtin_fma(q, amin, L) : INFINITY;
            const double t9 = amin < INFINITY ? __builtin_fma(fl, amin, clL) : INFINITY;
            Best bc = decide_bcast(mask, q, fl, cl, gm, L, g1, t2, 0u, b5, 0u, t9, 0u);
            if (bc.id == 5u) {
                int s_at = at5;
#pragma unroll
                for (int u = 3; u >= 0; --u)
                    s_at = __builtin_fma(q, sC[at5 + u], ab[at5 + u].y) == b5 ? at5 + u : s_at;
                bc.s = sSv[s_at];
            } else if (bc.id == 2u || bc.id == 9u) {
                // the first candidate whose value equals the minimum
                const double mul = bc.id == 2u ? q : fl, add = bc.id == 2u ? L : clL;
                int si = 0;
                while (si < nv - 1 && __builtin_fma(mul, ab[si].x, add) != bc.t)
                    ++si;
                bc.s = sSv[si];
            }
            if (active)
                store_cell(o, bc);
            o += plane;
        }
        const double s11 = chain ? tot[(int)((P - 1u) / SUM_BLOCK) * M + mr] + part[e] : 0.0;
        const double s12 = binom ? sum2[mr * (cl_max + 1) + cli] : 0.0;
        if (has_s && active)
            store_cell(o, decide_scatter(mask, q, cl, gm, L, s11, s12));
        ml += dm;
        pi += dp;
        if (pi >= n_P) {
            pi -= n_P;
            ++ml;
        }
    }
}

// ---- whole path of one (table, m) row in one workgroup ------------------------
//
// Few candidates (one per lane of a wave) and few blocks of the Scatter-chain sum:
// a workgroup takes one (table, m) and does every step for it, with LDS between
// the steps instead of device memory and launches: the table and its slopes; wave
// 0 the candidates (g(s), k, A, B, C, min A: one lane each), wave 1 g(m), g(1)
// and the prefix of g(2^j m); all threads the terms g(j m) of the chain sum, one
// search each; wave 0 the sums inside the blocks (a lane per block, 64 dependent
// additions) and then over the blocks; then the waves run their lanes over the
// process counts as in k_sweep_p: the few candidates that can win row 5 of Table 1
// for some process count of the group (or all: row_few), min_s A for rows 2 and 9, whose
// candidate is looked for only where one of them wins, two coalesced stores per cell.
// The slopes are read, as they were formed when the table was loaded, beside the
// samples: a division and a barrier less in a chain of dependent steps that is all
// of a small call (64 sizes x 49 process counts, 21 samples: 4.24 us in a graph of
// such calls, 4.03 so, where an empty kernel takes 1.6; 200 x 100 5.16 and 5.05).
constexpr int ROW_THREADS = 512;
constexpr int ROW_MAX_BLK = 32;          // at most 2048 terms of the chain sum
constexpr int ROW_NS = 64;               // candidates at most (the loops over them read up to the next eight)
constexpr int ROW_MAX_N = 512;           // samples at most (LDS per workgroup stays small)
constexpr long ROW_MAX_ROWS = 32;        // (table, m) rows per compute unit: 256 to 511 process counts (fewer: half, or less)

static size_t row_lds_bytes(int n, int n_blk, int n_P)
{
    return ((size_t)3 * n + 3 * ROW_NS + 36 + 36 + (size_t)n_blk * (SUM_BLOCK + 1) + 2 * ROW_MAX_BLK +
            ROW_NS / 2 + (size_t)(n_P + 1) / 2) * sizeof(double);
}

// PPL: process counts per lane in the Broadcast plane.  EXTRA: the planes of Gather and Barrier too,
// the first from the sums that are in LDS, the second by the waves that wait for them (501 sizes x
// 300 process counts, 37 candidates, all 18 rows: 10.6 us; terms and sums, sweep and planes in three
// launches 20.8).  FEW: row 5 for the candidates alone that can win it (see row_few).
template <bool ALL, int PPL, bool EXTRA, bool FEW>
__global__ void __launch_bounds__(ROW_THREADS) k_row(DeviceTables T, DeviceGrid G, plogp_cell_dev *out)
{
    extern __shared__ __align__(16) double row_lds[];
    __shared__ double sh_gm, sh_g1, sh_amin;
    __shared__ int sh_nv;
    __shared__ unsigned next_group;
    const int n = T.n, n_s = G.n_s, n_P = G.n_P, n_blk = G.n_blk;
    const uint32_t mask = ALL ? 0x1FFFu : G.mask;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // the rows of large sizes (the most candidates) first when the sizes ascend
    const int t = (int)blockIdx.x / G.n_m, mi = G.n_m - 1 - (int)blockIdx.x % G.n_m;
    f64x2 *ys = reinterpret_cast<f64x2 *>(row_lds);                    // {gap, slope} of every sample
    double *x = row_lds + 2 * n;
    double *sA = x + n, *sB = sA + ROW_NS, *sC = sB + ROW_NS;          // per candidate (past the last: +inf, +inf, 0)
    double *sum2 = sC + ROW_NS, *g2 = sum2 + 36;                       // prefix of g(2^j m); its terms
    double *pre = g2 + 36;                     // [block][65]: the terms, then the sums before each
    double *tot = pre + (size_t)n_blk * (SUM_BLOCK + 1), *done = tot + ROW_MAX_BLK;
    uint32_t *sSv = reinterpret_cast<uint32_t *>(done + ROW_MAX_BLK);  // the candidates
    uint32_t *sP = sSv + ROW_NS;                                       // the process counts
    // everything that comes from device memory is asked for at once
    const u64 m = G.m[mi];
    const double L = T.L[t];
    const u64 my_s = wave == 0 && lane < n_s ? G.s[lane] : 0ull;
    // (the division does not wait for the table: it runs while the samples are on their way)
    const double my_sd = (double)my_s, my_rcp = 1.0 / my_sd;
    {
        const double *gx = T.x + (size_t)t * n, *gy = T.y + (size_t)t * n, *gs = T.slope + (size_t)t * n;
        for (int i = tid; i < n; i += ROW_THREADS) {
            x[i] = gx[i];
            const f64x2 v = {gy[i], gs[i]};
            ys[i] = v;
        }
        for (int i = tid; i < n_P; i += ROW_THREADS)
            sP[i] = G.P[i];
        if (tid == 0)
            next_group = 0u;
        __syncthreads();
    }
    const auto gap = [&](double z) {
        const int i = last_not_above(x, n, z);
        const f64x2 v = ys[i];
        const double x0 = x[0];
        return __builtin_fma(v.y, (z > x0 ? z : x0) - x[i], v.x);
    };
    const double md = (double)m;
    const uint32_t need = EXTRA ? G.need : mask;       // the sums that some row adds up
    const bool chain = (need & (1u << 11)) != 0, binom = (need & (1u << 12)) != 0;

    if (wave == 0) {
        double A = INFINITY, B = INFINITY, C = 0.0;
        bool valid = false;
        if (lane < n_s) {
            const u64 lim = m < G.s_cap ? m : G.s_cap;
            const double sd = my_sd, gs = gap(sd);
            C = gs + L;
            valid = my_s <= lim;
            if (valid) {
                double Cx;
                segment_terms(md, sd, my_rcp, gs, L, A, B, Cx);
            }
        }
        sA[lane] = A;
        sB[lane] = B;
        sC[lane] = C;
        sSv[lane] = (uint32_t)my_s;
        const double amin = wave_min(A);
        const int nv = __builtin_popcountll(__ballot(valid));       // the candidates ascend
        if (lane == 0) {
            sh_amin = amin;
            sh_nv = nv;
        }
    } else if (wave == 1) {
        if (binom && lane < G.cl_max)
            g2[lane] = gap((double)(m << lane));
        if (lane == 63) {
            sh_gm = gap(md);
            sh_g1 = gap(1.0);
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        if (binom && lane == 0) {
            double acc = 0.0;
            sum2[0] = 0.0;
            for (int j = 0; j < G.cl_max; ++j) {
                acc = acc + g2[j];
                sum2[j + 1] = acc;
            }
        }
    }
    if (chain) {
        const int n_terms = SUM_BLOCK * (n_blk - 1) + G.last_terms;
        for (int r = tid; r < n_blk * SUM_BLOCK; r += ROW_THREADS) {
            double v = 0.0;
            if (r < n_terms)
                v = gap((double)((u64)(r + 1) * m));
            pre[r + r / SUM_BLOCK] = v;
        }
    }
    __syncthreads();
    // wave 0 adds the chain sums up while the others start on the Broadcast plane, which
    // does not need them; it joins them afterwards (the groups of 64 process counts are
    // handed out through a counter)
    if (chain && wave == 0) {
        if (lane < n_blk) {
            // sixteen terms at a time: read, add in order, write the sums before each
            double *p = pre + lane * (SUM_BLOCK + 1);
            double run = 0.0;
            for (int r0 = 0; r0 < SUM_BLOCK; r0 += 16) {
                double v[16];
#pragma unroll
                for (int u = 0; u < 16; ++u)
                    v[u] = p[r0 + u];
#pragma unroll
                for (int u = 0; u < 16; ++u) {
                    p[r0 + u] = run;
                    run = run + v[u];
                }
            }
            tot[lane] = run;
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        if (lane == 0) {
            double acc = 0.0;
            for (int b = 0; b < n_blk; ++b) {      // the finished blocks, in ascending order
                done[b] = acc;
                acc = acc + tot[b];
            }
        }
    }

    const double gm = sh_gm, g1 = sh_g1, amin = sh_amin;
    const int nv = __builtin_amdgcn_readfirstlane(sh_nv);
    const size_t plane = (size_t)G.n_m * n_P;
    plogp_cell_dev *const orow = out + (size_t)t * G.n_ops * plane + (size_t)mi * n_P;
    // lane si keeps candidate si (lanes past the candidates: B is +inf)
    const double c_mine = sC[lane], b_mine = sB[lane];
    // a lane takes PPL process counts, 64 apart: a candidate read serves them all
    const unsigned n_groups = (unsigned)((n_P + 64 * PPL - 1) / (64 * PPL));
    if (mask & 0x3FFu) {
        for (;;) {
            unsigned grp = 0u;
            if (lane == 0)
                grp = atomicAdd(&next_group, 1u);
            grp = __builtin_amdgcn_readfirstlane(grp);
            if (grp >= n_groups)
                break;
            int pi[PPL];
            bool active[PPL];
            double q[PPL], fl[PPL], cl[PPL], clL[PPL], b5[PPL];
            int i5[PPL];
#pragma unroll
            for (int h = 0; h < PPL; ++h) {
                pi[h] = ((int)grp * PPL + h) * 64 + lane;
                active[h] = pi[h] < n_P;
                const uint32_t Pv = sP[active[h] ? pi[h] : n_P - 1];
                q[h] = (double)(Pv - 1u);
                fl[h] = (double)floor_log2(Pv);
                cl[h] = (double)ceil_log2(Pv);
                clL[h] = cl[h] * L;
                b5[h] = INFINITY;
                i5[h] = 0;
            }
            if (mask & 0x20u) {
                if (FEW)
                    row5_least<PPL>(c_mine, b_mine,
                                    row5_candidates(c_mine, b_mine, nv, lane_value(q[0], 0), lane_value(q[PPL - 1], 63)),
                                    q, b5, i5);
                else
                    row5_all<PPL>(c_mine, sB, nv, q, b5, i5);
            }
#pragma unroll
            for (int h = 0; h < PPL; ++h) {
                const double t2 = amin < INFINITY ? __builtin_fma(q[h], amin, L) : INFINITY;
                const double t9 = amin < INFINITY ? __builtin_fma(fl[h], amin, clL[h]) : INFINITY;
                Best bc = decide_bcast(mask, q[h], fl[h], cl[h], gm, L, g1, t2, 0u, b5[h], 0u, t9, 0u);
                int at5 = i5[h];
                if (!FEW && __ballot(active[h] && bc.id == 5u) != 0) {
                    // the first candidate of the remembered eight that attains the minimum
#pragma unroll
                    for (int u = 7; u >= 0; --u)        // descending: the first match stays
                        at5 = __builtin_fma(q[h], sC[i5[h] + u], sB[i5[h] + u]) == b5[h] ? i5[h] + u : at5;
                }
                if (bc.id == 5u)
                    bc.s = sSv[at5];
                bool open = active[h] && (bc.id == 2u || bc.id == 9u);
                if (__ballot(open) != 0) {
                    // a winning row 2 or 9: the first candidate whose value equals the minimum
                    const double mul = bc.id == 2u ? q[h] : fl[h], add = bc.id == 2u ? L : clL[h];
                    uint32_t found = 0u;
                    for (int s0 = 0; s0 < nv; s0 += 4) {     // past the last candidate A is +inf
#pragma unroll
                        for (int u = 0; u < 4; ++u) {
                            const bool hit = open && __builtin_fma(mul, sA[s0 + u], add) == bc.t;
                            found = hit ? sSv[s0 + u] : found;
                            open = open && !hit;
                        }
                        if (__ballot(open) == 0)
                            break;
                    }
                    if (bc.id == 2u || bc.id == 9u)
                        bc.s = found;
                }
                if (active[h])
                    store_cell(orow + pi[h], bc);
            }
        }
    }
    plogp_cell_dev *const srow = orow + ((mask & 0x3FFu) ? plane : 0);
    const uint32_t gather = EXTRA ? (G.extra & 7u) << 10 : 0u;         // under the ids of its Scatter twins
    plogp_cell_dev *const grow = srow + ((mask & 0x1C00u) ? plane : 0);
    if (EXTRA && (G.extra & 0x18u) && wave > 0) {
        plogp_cell_dev *const brow = grow + (gather ? plane : 0);
        for (int pi = tid - 64; pi < n_P; pi += ROW_THREADS - 64) {
            const uint32_t Pv = sP[pi];
            store_cell(brow + pi, decide_barrier(G.extra, (double)(Pv - 1u), (double)floor_log2(Pv),
                                                 (double)ceil_log2(Pv), L, g1));
        }
    }
    __syncthreads();                   // the chain sums are complete
    if ((mask & 0x1C00u) || gather) {
        for (int pi = tid; pi < n_P; pi += ROW_THREADS) {
            const uint32_t Pv = sP[pi];
            const int cli = ceil_log2(Pv), blk = (int)((Pv - 1u) / SUM_BLOCK);
            const double q = (double)(Pv - 1u), cl = (double)cli;
            const double s11 = chain ? done[blk] + pre[(Pv - 1u) + blk] : 0.0;
            const double s12 = binom ? sum2[cli] : 0.0;
            if (mask & 0x1C00u)
                store_cell(srow + pi, decide_scatter(mask, q, cl, gm, L, s11, s12));
            if (EXTRA && gather) {
                Best b = decide_scatter(gather, q, cl, gm, L, s11, s12);
                b.id += 3u;
                store_cell(grow + pi, b);
            }
        }
    }
}

// ---- whole path for batches of tables that share their sample sizes ----------
//
// Measured tables of many clusters are normally taken at the same list of
// message sizes.  Then, for a fixed m, everything that depends on where a size
// falls among the samples -- the interval of m, of 2^j m, of every j m of the
// Scatter-chain sum, the candidates that compete, k = ceil(m / s) -- is the same
// for all tables, and only the gaps, slopes and L differ.  So here the lanes of a
// wave run over 64 tables and the wave walks over message sizes: all control
// flow is wave-uniform (no lane ever waits for another lane's interval
// crossing), the table entries are read as coalesced rows of a copy laid out
// [interval][table], and the per-m facts come from small tables prepared once
// per call by k_batch_setup.

// One thread per entry of the prepared facts.  Uses table 0's sample sizes.
// Intervals are numbered as in the chain walk: 0 = [0, x_0) (the clamp: gap y_0,
// slope 0), i + 1 = [x_i, x_{i+1}), n = [x_{n-1}, inf).  Everything about one
// message size sits in one record of B.rec (layout: BatchRec).
__device__ __forceinline__ void batch_prep_body(const DeviceTables &T, const DeviceGrid &G,
                                                const BatchPrep &B, int block, int n_blocks, double *lds)
{
    const int n = T.n;
    double *x = lds;                              // samples of table 0
    for (int i = threadIdx.x; i < n; i += blockDim.x)
        x[i] = T.x[i];
    __syncthreads();
    // interval of size z and z minus the start of that interval (exact)
    auto locate = [&](double z, int &iv, double &dz) {
        const int cnt = last_not_above(x, n, z) + (z >= x[0] ? 1 : 0);     // samples not above z
        iv = cnt;
        dz = cnt == 0 ? z : z - x[cnt - 1];
    };
    const BatchRec R(n, G.n_s, G.cl_max);
    const long tid = (long)block * blockDim.x + threadIdx.x;
    const long stride = (long)n_blocks * blockDim.x;
    for (long e = tid; e < G.n_m; e += stride) {
        double *rec = B.rec + (size_t)e * R.slots;
        const u64 m = G.m[e];
        int iv;
        double dz;
        locate((double)m, iv, dz);
        const u64 lim = m < G.s_cap ? m : G.s_cap;          // candidates s <= min(m, s_cap) ascend
        int lo = 0, hi = G.n_s;
        while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if (G.s[mid] <= lim) lo = mid + 1; else hi = mid;
        }
        rec[R.DM] = dz;
        rec[R.MD] = (double)m;
        reinterpret_cast<int *>(rec + R.IM_NV)[0] = iv;
        reinterpret_cast<int *>(rec + R.IM_NV)[1] = lo;
    }
    for (long e = tid; e < (long)G.n_m * G.cl_max; e += stride) {
        const long mi = e / G.cl_max;
        const int j = (int)(e % G.cl_max);
        double *rec = B.rec + (size_t)mi * R.slots;
        int iv;
        double dz;
        locate((double)(G.m[mi] << j), iv, dz);
        rec[R.D2 + j] = dz;
        reinterpret_cast<int *>(rec + R.I2)[j] = iv;
    }
    for (long e = tid; e < (long)G.n_m * (n + 1); e += stride) {
        // last j whose size j m still lies in interval i of this m: below the next sample
        const long mi = e / (n + 1);
        const int i = (int)(e % (n + 1));
        const u64 m = G.m[mi];
        u64 last = 0xFFFFFFFFull;
        if (i < n) {
            last = ((u64)x[i] - 1ull) / m;
            last = last < 0xFFFFFFFFull ? last : 0xFFFFFFFFull;
        }
        reinterpret_cast<unsigned *>(B.rec + (size_t)mi * R.slots + R.JEND)[i] = (unsigned)last;
    }
    for (long e = tid; e < (long)G.n_m * G.n_s; e += stride) {
        const long mi = e / G.n_s;
        const int si = (int)(e % G.n_s);
        const u64 m = G.m[mi], sv = G.s[si];
        B.rec[(size_t)mi * R.slots + R.K + si] = (double)((m + sv - 1ull) / sv);   // k = ceil(m / s), exact
    }
    // B.tab: interval of size 1 and 1 minus its start; widths of the intervals; per candidate
    // s minus the start of its interval, then its interval; per process count three doubles
    for (long e = tid; e < G.n_s; e += stride) {
        int iv;
        double dz;
        locate((double)G.s[e], iv, dz);
        B.tab[2 + (n + 1) + e] = dz;
        B.tab[2 + (n + 1) + G.n_s + e] = (double)iv;
    }
    for (long e = tid; e <= n; e += stride)
        B.tab[2 + e] = e == 0 ? x[0] : (e < n ? x[e] - x[e - 1] : INFINITY);
    // per process count 32 bytes: P - 1, floor(log2 P), ceil(log2 P) as doubles, then P - 1 and
    // ceil(log2 P) as integers; the list is filled up to a multiple of eight, plus one, with
    // copies of its last entry (the kernel takes eight at a time and fetches one ahead)
    for (long e = tid; e < batch_padded_P(G.n_P); e += stride) {
        double *pt = B.tab + 2 + (n + 1) + 2 * (size_t)G.n_s + 4 * e;
        const uint32_t P = G.P[e < G.n_P ? e : G.n_P - 1];
        pt[0] = (double)(P - 1u);
        pt[1] = (double)floor_log2(P);
        pt[2] = (double)ceil_log2(P);
        reinterpret_cast<uint32_t *>(pt + 3)[0] = P - 1u;
        reinterpret_cast<uint32_t *>(pt + 3)[1] = (uint32_t)ceil_log2(P);
    }
    if (tid == 0) {
        int i1;
        double d1;
        locate(1.0, i1, d1);
        B.tab[0] = (double)i1;
        B.tab[1] = d1;
    }
}

// The tables laid out by interval: ysT[i][t] = {gap, slope} of interval i of table t
// (i = 0: the clamp {y_0, 0}; i = n + 1: zeros, only ever fetched ahead).  The slopes
// are formed here from the raw samples.  A workgroup takes BATCH_STAGE_TT tables: their
// gaps are read as whole rows into LDS (rows padded by one), then written with the
// tables along the lanes.  The sample sizes are those of table 0 (shared by all).
constexpr int BATCH_STAGE_TT = 32;

__device__ __forceinline__ void batch_stage_body(const DeviceTables &T, f64x2 *ysT, int block, double *lds)
{
    const int n = T.n, t0 = block * BATCH_STAGE_TT;
    const int nt = T.n_tables - t0 < BATCH_STAGE_TT ? T.n_tables - t0 : BATCH_STAGE_TT;
    for (int e = threadIdx.x; e < nt * n; e += blockDim.x) {
        const int tl = e / n, i = e - tl * n;
        lds[tl * (n + 1) + i] = T.y[(size_t)(t0 + tl) * n + i];
    }
    __syncthreads();
    for (int e = threadIdx.x; e < (n + 2) * BATCH_STAGE_TT; e += blockDim.x) {
        const int i = e / BATCH_STAGE_TT, tl = e % BATCH_STAGE_TT;
        if (tl >= nt)
            continue;
        const double *y = lds + tl * (n + 1);
        f64x2 v = {0.0, 0.0};
        if (i == 0)
            v = f64x2{y[0], 0.0};
        else if (i <= n)
            v = f64x2{y[i - 1], interval_slope(T.x, y, n, i - 1)};
        ysT[(size_t)i * T.n_tables + t0 + tl] = v;
    }
}

// One launch for both preparations: the first n_stage workgroups lay out the tables, the
// others prepare the per-size facts.
__global__ void __launch_bounds__(256) k_batch_setup(DeviceTables T, DeviceGrid G, BatchPrep B,
                                                     f64x2 *ysT, int n_stage)
{
    extern __shared__ double lds[];
    if ((int)blockIdx.x < n_stage)
        batch_stage_body(T, ysT, (int)blockIdx.x, lds);
    else
        batch_prep_body(T, G, B, (int)blockIdx.x - n_stage, (int)gridDim.x - n_stage, lds);
}

constexpr size_t BATCH_T_LDS_MAX = 160 * 1024;     // LDS of a compute unit

// A wave-uniform read of data that no kernel writes while this one runs, through the
// scalar cache (constant address space).  Unlike a vector load it does not queue behind
// the wave's outstanding stores.
template <class V>
__device__ __forceinline__ V uniform_load(const V *p)
{
    typedef const V __attribute__((address_space(4))) *const_ptr;
    return *(const_ptr)(p);
}
constexpr int BATCH_T_WAVES = 16;      // waves of a workgroup; they share the 64 tables
constexpr int BATCH_T_PC = 4;          // process counts decided together (in registers)
constexpr int BATCH_T_PS = 8;          // process counts per pass over the candidates, and the
                                       // cells of a table written together (128 bytes)
// Output staging of a wave, used in turn as 64 rows of 8 times + 8 one-byte ids (Scatter)
// and as 32 rows of 8 cells padded to 9 (Broadcast).
constexpr int BATCH_T_STAGE = 64 * 72;
static_assert(BATCH_T_STAGE >= 32 * (BATCH_T_PS + 1) * 16 && BATCH_T_STAGE % 16 == 0, "both layouts fit");

struct BatchDims {
    int n, n_tables, n_m, n_P, n_s, cl_max, n_ops, n_mchunks, m_per_wave;
    uint32_t mask;
    uint32_t extra;   // rows beyond the tables: bits 0..2 Gather, bits 3, 4 Barrier (see DeviceGrid)
};

// A workgroup stages its 64 tables by interval in LDS (YS[i][lane] = {gap, slope}
// of interval i of the lane's table) together with their g(s); every later
// access to a table is one conflict-free LDS read of a whole row.  All other
// inputs are wave-uniform and come through the scalar cache.  The cells of PS = 8
// process counts are turned round in LDS so that eight neighbouring lanes store
// the 128 contiguous bytes of one table (whole cache lines when n_P is a multiple
// of 8: measured 5.2 TB/s against 3.3 TB/s for 64-byte runs).  LDS has room for
// 4.5 KB of staging per wave, not for 64 rows of 8 cells: a Scatter cell is staged
// as its time and a one-byte id (s is 0), the Broadcast cells go out in two halves
// of 32 tables, the second half waiting in registers.
// ALL: every strategy of Tables 1 and 2 is enabled (the mask is a compile-time constant).
// EXTRA: rows beyond the tables are enabled as well (their planes cost nothing otherwise).
template <int PC, int PS, bool ALL, bool EXTRA>
__global__ void __launch_bounds__(64 * BATCH_T_WAVES)
k_batch_t(BatchDims D, const f64x2 *__restrict__ ysT, const double *__restrict__ Lt,
          const double *__restrict__ recs, const double *__restrict__ tab,
          const u64 *__restrict__ p_s, plogp_cell_dev *__restrict__ out)
{
    extern __shared__ __align__(16) double batch_lds[];
    const int n = D.n, n_s = D.n_s, n_P = D.n_P;
    const BatchRec R(n, n_s, D.cl_max);
    f64x2 *YS = reinterpret_cast<f64x2 *>(batch_lds);          // [n + 2][64]
    double *GS = batch_lds + (size_t)2 * (n + 2) * 64;         // [n_s][64]
    // per wave: the PC cells of 64 tables on their way out, rows padded by one cell
    char *stage_all = reinterpret_cast<char *>(GS + (size_t)(n_s ? n_s : 1) * 64);
    uint32_t *sS = reinterpret_cast<uint32_t *>(stage_all + (size_t)BATCH_T_WAVES * BATCH_T_STAGE);   // [n_s]
    unsigned &next_m = *reinterpret_cast<unsigned *>(sS + (n_s ? n_s : 1));   // next size of this workgroup's chunk
    // the chunks of large sizes (more candidates, the longest) are handed out first, so that
    // the launch ends with short workgroups
    const int n_tg = (D.n_tables + 63) / 64;
    const int tg = blockIdx.x % n_tg, mc = D.n_mchunks - 1 - (int)(blockIdx.x / n_tg);
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int t = tg * 64 + lane;
    const int tc = t < D.n_tables ? t : D.n_tables - 1;
    const double L = Lt[tc];
    const uint32_t mask = ALL ? 0x1FFFu : D.mask;
    for (int si = threadIdx.x; si < n_s; si += blockDim.x)
        sS[si] = (uint32_t)p_s[si];
    for (int i = wave; i < n + 2; i += BATCH_T_WAVES)
        YS[i * 64 + lane] = ysT[(size_t)i * D.n_tables + tc];
    if (threadIdx.x == 0)
        next_m = 0u;
    __syncthreads();
    const f64x2 *ys = YS + lane;                               // this lane's table: ys[64 i]
    const double *tab_ds = tab + 2 + (n + 1), *tab_is = tab_ds + n_s, *Wd = tab + 2;
    // per process count {P - 1, floor log2 P, ceil log2 P, {P - 1, ceil log2 P} as integers}
    typedef double f64x4 __attribute__((ext_vector_type(4)));
    const f64x4 *tab_P = reinterpret_cast<const f64x4 *>(tab_is + n_s);
    for (int si = wave; si < n_s; si += BATCH_T_WAVES) {
        const f64x2 v = ys[64 * (int)uniform_load(tab_is + si)];
        GS[si * 64 + lane] = __builtin_fma(v.y, uniform_load(tab_ds + si), v.x);
    }
    double g1;
    {
        const f64x2 v = ys[64 * (int)uniform_load(tab)];
        g1 = __builtin_fma(v.y, uniform_load(tab + 1), v.x);
    }
    __syncthreads();
    const double *gsl = GS + lane;                             // g(s) of this lane's table: gsl[64 si]
    char *stage = stage_all + (size_t)wave * BATCH_T_STAGE;
    // A store instruction writes the PS cells (PS x 16 contiguous bytes) of 64 / PS tables:
    // lane l takes cell l % PS of table row l / PS + (64 / PS) it.
    static_assert(PC == 4 && PS == 8, "128-byte runs, decided four at a time");
    const int out_p = lane % PS, out_row = lane / PS;
    const size_t plane = (size_t)D.n_m * n_P;
    const size_t table_cells = (size_t)D.n_ops * plane;
    // Where the staged cells go: a wave-uniform 64-bit part (table group, row step, plane, m,
    // first process count) plus a per-lane 32-bit byte offset, so that the stores need no
    // per-lane 64-bit addresses (the host checks that the offset fits).
    const unsigned lane_off = (unsigned)(((size_t)out_row * table_cells + out_p) * sizeof(plogp_cell_dev));
    char *const o_grp = reinterpret_cast<char *>(out + (size_t)tg * 64 * table_cells);
    const int rows_left = D.n_tables - tg * 64 - out_row;      // table rows r0 + out_row with r0 < rows_left exist
    typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
    // wave-uniform base in scalar registers + 32-bit lane offset
    auto store_run = [&](char *ubase, u32x4 cell) {
        asm volatile("global_store_dwordx4 %0, %1, %2 nt" : : "v"(lane_off), "v"(cell), "s"(ubase) : "memory");
    };
    const size_t run_step = (size_t)(64 / PS) * table_cells * sizeof(plogp_cell_dev);   // 8 tables on
    const bool whole_group = tg * 64 + 64 <= D.n_tables;       // wave-uniform: no row of tables is missing
    // cell0: index of cell (plane, mi, p0) inside a table.  Scatter layout: row r of the stage
    // holds 8 times, then 8 ids as signed bytes (-1 = no strategy).
    // id_add: 0, or 3 when the staged Scatter decisions go out as their Gather twins
    auto scatter_cell = [&](int r0, int id_add) {
        const char *row = stage + (r0 + out_row) * 72;
        const double tv = *reinterpret_cast<const double *>(row + 8 * out_p);
        const int id = *reinterpret_cast<const signed char *>(row + 64 + out_p);
        u32x4 cell;
        cell.x = (unsigned)__double2loint(tv);
        cell.y = (unsigned)__double2hiint(tv);
        cell.z = 0u;
        cell.w = (unsigned)(id < 0 ? id : id + id_add);
        return cell;
    };
    auto flush_times = [&](size_t cell0, int p0, int id_add) {
        __builtin_amdgcn_wave_barrier();
        if (p0 + out_p < n_P) {
            char *ubase = o_grp + cell0 * sizeof(plogp_cell_dev);
            if (whole_group) {
                // (four rows are read before their four stores go out: a store keeps the reads
                // that follow it behind itself)
#pragma unroll
                for (int it = 0; it < 64 / PS; it += 4) {
                    u32x4 c[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u)
                        c[u] = scatter_cell((64 / PS) * (it + u), id_add);
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        store_run(ubase, c[u]);
                        ubase += run_step;
                    }
                }
            } else {
                // (the limit is made opaque here: its sixteen compares would otherwise be kept
                // in scalar registers across the whole kernel)
                int rl = rows_left;
                asm volatile("" : "+v"(rl));
#pragma unroll
                for (int it = 0; it < 64 / PS; ++it) {
                    if ((64 / PS) * it < rl)
                        store_run(ubase, scatter_cell((64 / PS) * it, id_add));
                    ubase += run_step;
                }
            }
        }
        __builtin_amdgcn_wave_barrier();
    };
    // Broadcast layout: row r of the stage holds the 8 cells of table 32 half + r, padded to 9.
    auto flush_cells = [&](int half, size_t cell0, int p0) {
        __builtin_amdgcn_wave_barrier();
        if (p0 + out_p < n_P) {
            char *ubase = o_grp + ((size_t)32 * half * table_cells + cell0) * sizeof(plogp_cell_dev);
            const u32x4 *rows = reinterpret_cast<const u32x4 *>(stage) + out_row * (PS + 1) + out_p;
            if (whole_group) {
                u32x4 c[32 / PS];
#pragma unroll
                for (int it = 0; it < 32 / PS; ++it)
                    c[it] = rows[(64 / PS) * it * (PS + 1)];
#pragma unroll
                for (int it = 0; it < 32 / PS; ++it) {
                    store_run(ubase, c[it]);
                    ubase += run_step;
                }
            } else {
                int rl = rows_left;
                asm volatile("" : "+v"(rl));
#pragma unroll
                for (int it = 0; it < 32 / PS; ++it) {
                    if (32 * half + (64 / PS) * it < rl)
                        store_run(ubase, rows[(64 / PS) * it * (PS + 1)]);
                    ubase += run_step;
                }
            }
        }
        __builtin_amdgcn_wave_barrier();
    };
    auto pack = [](const Best &b) {
        union { plogp_cell_dev c; uint4 v; } u;
        u.c.time = b.t; u.c.s = b.s; u.c.strategy = b.id;
        return u.v;
    };
    // The Gather rows (ids 13..15) are the Scatter rows on the same sums: this kernel takes them
    // when they are enabled exactly as the Scatter rows are, or without any Scatter row (the host
    // sees to that), decides once and writes the decisions to both planes.  The Barrier rows
    // (16, 17) need g(1), L and the process count only.
    const uint32_t extra = EXTRA ? D.extra : 0u;
    const uint32_t gather_rows = (extra & 7u) << 10;               // as the Scatter rows they mirror
    const uint32_t sg_rows = (mask & 0x1C00u) | gather_rows;
    const bool want_chain = (sg_rows & (1u << 11)) != 0, want_binom = (sg_rows & (1u << 12)) != 0;
    const bool has_b = (mask & 0x3FFu) != 0, has_s = sg_rows != 0;
    const bool has_scatter = (mask & 0x1C00u) != 0, has_gather = gather_rows != 0;
    const bool has_barrier = (extra & 0x18u) != 0;
    const size_t scatter_at = (has_b ? plane : 0), gather_at = scatter_at + (has_scatter ? plane : 0);
    const size_t barrier_at = gather_at + (has_gather ? plane : 0);

    // The waves take the sizes of the workgroup's chunk one at a time from a counter, the largest
    // first (a size's cost grows with its number of candidates): the one workgroup that fits a
    // compute unit then ends with all its waves busy, whatever the mix.
    const int chunk = BATCH_T_WAVES * D.m_per_wave;
    for (;;) {
        unsigned k = 0u;
        if (lane == 0)
            k = atomicAdd(&next_m, 1u);
        k = (unsigned)__builtin_amdgcn_readfirstlane((int)k);
        if (k >= (unsigned)chunk)
            break;
        const int mi = mc * chunk + chunk - 1 - (int)k;                      // wave-uniform
        if (mi >= D.n_m)
            continue;
        const double *rec = recs + (size_t)mi * R.slots;
        const double md = uniform_load(rec + R.MD);
        const int nvm = uniform_load(reinterpret_cast<const int *>(rec + R.IM_NV) + 1);
        const double *Krow = rec + R.K;
        const unsigned *jend = reinterpret_cast<const unsigned *>(rec + R.JEND);
        // g(m); the chain sum starts at j = 1 in the same interval
        int ci = uniform_load(reinterpret_cast<const int *>(rec + R.IM_NV));
        f64x2 cur = ys[64 * ci];
        double d = uniform_load(rec + R.DM);                    // size - start of its interval
        const double gm = __builtin_fma(cur.y, d, cur.x);
        unsigned je = uniform_load(jend + ci);                  // last j inside interval ci
        // fetched one crossing ahead: the next interval's entries, its last j, this one's width
        f64x2 nxt = ys[64 * (ci + 1)];
        unsigned je_n = uniform_load(jend + (ci < n ? ci + 1 : n));
        double w_n = uniform_load(Wd + ci);
        double run = 0.0, done = 0.0;
        unsigned j_done = 0;
        double s12 = 0.0;
        int cl_done = 0;
        int i2_n = uniform_load(reinterpret_cast<const int *>(rec + R.I2));
        double d2_n = uniform_load(rec + R.D2);
        f64x4 P_n = uniform_load(tab_P);
        // minimum over s of A = g(s) k (rows 2 and 9 of Table 1 are monotone in A), the first
        // candidate that attains it, and the least A before that candidate (+inf if none)
        double amin = INFINITY, abefore = INFINITY;
        int imin = 0;
        if (mask & 0x204u) {
            // (the next candidate's g(s) and k are fetched while this one is worked on)
            double gs_n = gsl[0], k_n = uniform_load(Krow);
            for (int si = 0; si < nvm; ++si) {
                const double A = gs_n * k_n;
                const int nx = si + 1 < nvm ? si + 1 : si;
                gs_n = gsl[64 * nx];
                k_n = uniform_load(Krow + nx);
                const bool lower = A < amin;
                abefore = lower ? amin : abefore;
                imin = lower ? si : imin;
                amin = min_f64(amin, A);
            }
        }

        // PS process counts per pass over the candidates (the per-candidate terms are formed
        // once for all of them), then PC cells at a time are decided and written
        for (int q0 = 0; q0 < n_P; q0 += PS) {
            const size_t cell0 = (size_t)mi * n_P + q0;
            if (has_s) {
                // Scatter plane, one process count after the other: the chain sum is walked
                // along j while P ascends, the binomial sum grows with ceil(log2 P)
#pragma nounroll
                for (int p = 0; p < PS; ++p) {
                    const f64x4 Pv = P_n;                       // (fetched one step ahead, like i2_n and d2_n)
                    P_n = uniform_load(tab_P + q0 + p + 1);
                    if (want_chain) {
                        const unsigned target = (unsigned)__double2loint(Pv.w);
                        while (j_done < target) {
                            // up to the next process count, block end or interval end
                            const unsigned block_end = (j_done / SUM_BLOCK + 1u) * SUM_BLOCK;
                            unsigned stop = target < block_end ? target : block_end;
                            stop = stop < je ? stop : je;
                            unsigned j = j_done;
                            for (; j + 4u <= stop; j += 4u) {
#pragma unroll
                                for (int r = 0; r < 4; ++r) {
                                    run = run + __builtin_fma(cur.y, d, cur.x);
                                    d += md;
                                }
                            }
                            for (; j < stop; ++j) {
                                run = run + __builtin_fma(cur.y, d, cur.x);
                                d += md;
                            }
                            j_done = stop;
                            if (j_done % SUM_BLOCK == 0u) {
                                done = done + run;
                                run = 0.0;
                            }
                            while (je <= j_done) {              // the next size lies further on
                                d -= w_n;
                                ++ci;
                                cur = nxt;
                                je = je_n;
                                nxt = ys[64 * (ci + 1)];
                                je_n = uniform_load(jend + (ci < n ? ci + 1 : n));
                                w_n = uniform_load(Wd + ci);
                            }
                        }
                    }
                    if (want_binom) {
                        const int cli = __double2hiint(Pv.w);
                        while (cl_done < cli) {
                            const f64x2 v = ys[64 * i2_n];
                            s12 = s12 + __builtin_fma(v.y, d2_n, v.x);
                            ++cl_done;
                            const int nx = cl_done < D.cl_max ? cl_done : cl_done - 1;
                            i2_n = uniform_load(reinterpret_cast<const int *>(rec + R.I2) + nx);
                            d2_n = uniform_load(rec + R.D2 + nx);
                        }
                    }
                    const Best r = decide_scatter(ALL ? mask : sg_rows, Pv.x, Pv.z, gm, L, done + run, s12);
                    *reinterpret_cast<double *>(stage + lane * 72 + 8 * p) = r.t;
                    *reinterpret_cast<signed char *>(stage + lane * 72 + 64 + p) = (signed char)r.id;
                }
                if (has_scatter)
                    flush_times(scatter_at + cell0, q0, 0);
                if (has_gather)
                    flush_times(gather_at + cell0, q0, 3);
            }
            if (has_barrier) {
                // twice the flat-tree and the binomial row of Table 1 at one byte; the same for
                // every message size, formed again for each (what it would take to keep them
                // costs more than the few instructions)
#pragma unroll
                for (int p = 0; p < PS; ++p) {
                    const f64x4 Pv = uniform_load(tab_P + q0 + p);
                    Best b = {INFINITY, 0u, 0xFFFFFFFFu};
                    if (extra & 8u) consider(b, 2.0 * __builtin_fma(Pv.x, g1, L), 16, 0);
                    if (extra & 16u) consider(b, 2.0 * __builtin_fma(Pv.y, g1, Pv.z * L), 17, 0);
                    *reinterpret_cast<double *>(stage + lane * 72 + 8 * p) = b.t;
                    *reinterpret_cast<signed char *>(stage + lane * 72 + 64 + p) = (signed char)b.id;
                }
                flush_times(barrier_at + cell0, q0, 0);
            }
            if (!has_b)
                continue;
            double b5[PS];
            int i5[PS];
#pragma unroll
            for (int p = 0; p < PS; ++p) {
                b5[p] = INFINITY;
                i5[p] = 0;
            }
            if (has_b && (mask & (1u << 5))) {
                double q[PS];                                   // wave-uniform
#pragma unroll
                for (int p = 0; p < PS; ++p)
                    q[p] = uniform_load(reinterpret_cast<const double *>(tab_P + q0 + p));
                double gs_n = gsl[0], k_n = uniform_load(Krow);
                for (int si = 0; si < nvm; ++si) {
                    const double gs = gs_n, k = k_n;
                    const int nx = si + 1 < nvm ? si + 1 : si;
                    gs_n = gsl[64 * nx];
                    k_n = uniform_load(Krow + nx);
                    const double Bv = gs * (k - 1.0), Cv = gs + L;
#pragma unroll
                    for (int p = 0; p < PS; ++p) {
                        const double T5 = __builtin_fma(q[p], Cv, Bv);
                        i5[p] = T5 < b5[p] ? si : i5[p];
                        b5[p] = min_f64(b5[p], T5);
                    }
                }
            }
            Best held[PC];                                      // the first four cells of tables 32..63
#pragma unroll
            for (int g = 0; g < PS / PC; ++g) {
                const int p0 = q0 + g * PC;                     // may lie past the end: indices are clamped
                double q[PC], fl[PC], clL[PC], cl[PC];          // q, fl, cl: wave-uniform
#pragma unroll
                for (int p = 0; p < PC; ++p) {
                    const double *pt = reinterpret_cast<const double *>(tab_P + p0 + p);
                    q[p] = uniform_load(pt);
                    fl[p] = uniform_load(pt + 1);
                    cl[p] = uniform_load(pt + 2);
                    clL[p] = cl[p] * L;
                }
                Best bc[PC];
                bool any = false;
#pragma unroll
                for (int p = 0; p < PC; ++p) {
                    // without a candidate amin is +inf, and so are both values (q, fl >= 1)
                    const double t2 = __builtin_fma(q[p], amin, L);
                    const double t9 = __builtin_fma(fl[p], amin, clL[p]);
                    const double t5 = b5[g * PC + p];
                    const uint32_t s5 = t5 < INFINITY ? sS[i5[g * PC + p]] : 0u;
                    bc[p] = decide_bcast(mask, q[p], fl[p], cl[p], gm, L, g1, t2, 0u, t5, s5, t9, 0u);
                    any = any || bc[p].id == 2u || bc[p].id == 9u;
                }
                if (__ballot(any) != 0) {
                    // A winning row 2 or 9: the first candidate whose value equals the minimum.
                    // The rows grow with A, so that is the candidate of the least A, unless a
                    // larger A before it rounds to the same time: only the least of those can.
                    bool open[PC];
                    bool tie = false;
                    const uint32_t smin = nvm > 0 ? sS[imin] : 0u;
#pragma unroll
                    for (int p = 0; p < PC; ++p) {
                        open[p] = bc[p].id == 2u || bc[p].id == 9u;
                        const double Tb = bc[p].id == 2u ? __builtin_fma(q[p], abefore, L)
                                                         : __builtin_fma(fl[p], abefore, clL[p]);
                        tie = tie || (open[p] && Tb == bc[p].t);
                        bc[p].s = open[p] ? smin : bc[p].s;
                    }
                    if (__ballot(tie) != 0) {
                        // (rare) the search itself, for every lane
                        for (int si = 0; si < nvm; ++si) {
                            const double A = gsl[64 * si] * uniform_load(Krow + si);
                            const uint32_t sv = sS[si];
#pragma unroll
                            for (int p = 0; p < PC; ++p) {
                                const double Tv = bc[p].id == 2u ? __builtin_fma(q[p], A, L)
                                                                 : __builtin_fma(fl[p], A, clL[p]);
                                if (open[p] && Tv == bc[p].t) {
                                    bc[p].s = sv;
                                    open[p] = false;
                                }
                            }
                        }
                    }
                }
                uint4 *rows = reinterpret_cast<uint4 *>(stage);
                if (g == 0) {
                    if (lane < 32) {
#pragma unroll
                        for (int p = 0; p < PC; ++p)
                            rows[lane * (PS + 1) + p] = pack(bc[p]);
                    }
#pragma unroll
                    for (int p = 0; p < PC; ++p)
                        held[p] = bc[p];
                } else {
                    if (lane < 32) {
#pragma unroll
                        for (int p = 0; p < PC; ++p)
                            rows[lane * (PS + 1) + PC + p] = pack(bc[p]);
                    }
                    flush_cells(0, cell0, q0);
                    if (lane >= 32) {
#pragma unroll
                        for (int p = 0; p < PC; ++p) {
                            rows[(lane - 32) * (PS + 1) + p] = pack(held[p]);
                            rows[(lane - 32) * (PS + 1) + PC + p] = pack(bc[p]);
                        }
                    }
                    flush_cells(1, cell0, q0);
                }
            }
        }
    }
}

// ---- prediction against measurement ------------------------------------------
//
// The step after the tuning in the paper (Section 4): every implementation is
// measured, the measurements are set against the predictions of Tables 1 and
// 2, and the question is whether the technique the models choose is the one
// that is fastest in the measurement.  k_score: one thread per (m, P), lanes
// along P (the measured times meas[r][m][P] and the predictions are read and
// written coalesced); r runs over the enabled strategies in ascending id.
// g(m), g(1) and the two Scatter sums come from the tuning's own first stages.

struct plogp_verdict_dev {
    double regret;
    uint32_t pred_best;
    uint32_t meas_best;
};

// The prediction of strategy `id` (rows of Tables 1 and 2 as the scoring evaluates them) at one
// point: a segmented row at the segment size the point was measured with (gs, k; NaN if that
// size is not usable), the Scatter rows from the tuning's sums.
__device__ __forceinline__ double score_predict(int id, double q, double fl, double cl, double gm, double L,
                                                double R, const double (&gs)[3], const double (&k)[3],
                                                const bool (&ok)[3], const DeviceGrid &G, const Scratch &S,
                                                int mi, int pi, uint32_t P)
{
    switch (id) {
    case 0: case 10: return __builtin_fma(q, gm, L);
    case 1: return __builtin_fma(q, gm, R);
    case 2: return ok[0] ? __builtin_fma(q, gs[0] * k[0], L) : NAN;
    case 3: return q * (gm + L);
    case 4: return q * (gm + R);
    case 5: return ok[1] ? __builtin_fma(q, gs[1] + L, gs[1] * (k[1] - 1.0)) : NAN;
    case 6: return cl * __builtin_fma(2.0, gm, L);
    case 7: return __builtin_fma(fl, gm, cl * L);
    case 8: return __builtin_fma(fl, gm, cl * R);
    case 9: return ok[2] ? __builtin_fma(fl, gs[2] * k[2], cl * L) : NAN;
    case 11: return __builtin_fma(q, L, chain_sum_of(G, S, 0, mi, pi, P));
    default: return __builtin_fma(cl, L, S.sum2[(size_t)mi * (G.cl_max + 1) + ceil_log2(P)]);
    }
}

// Workgroups walk the (m, chunk of P) items with a stride, so that a big table is
// staged once per workgroup; the measured times and segment sizes of a point are
// fetched before any arithmetic (13 + 3 independent loads per lane in flight).
__global__ void __launch_bounds__(1024) k_score_points(DeviceTables T, DeviceGrid G, Scratch S,
                                                const double *__restrict__ meas,
                                                const uint32_t *__restrict__ seg,
                                                double *__restrict__ pred,
                                                plogp_verdict_dev *__restrict__ verdict, int n_pchunks,
                                                int n_items)
{
    extern __shared__ double lds[];
    const uint32_t mask = G.mask;
    const bool any_seg = (mask & 0x224u) != 0;
    LdsTable tab = {nullptr, nullptr, nullptr, T.n};
    if (any_seg)
        tab = stage_table(lds, T, 0);                 // for g(s) at the measured segment sizes
    const double L = T.L[0];
    const double g1 = S.g1[0];
    const double R = __builtin_fma(3.0, L, 2.0 * g1);
    const size_t plane = (size_t)G.n_m * G.n_P;
    for (int item = blockIdx.x; item < n_items; item += gridDim.x) {
        const int mi = item / n_pchunks;
        const int pi = (item % n_pchunks) * blockDim.x + threadIdx.x;
        if (pi >= G.n_P)
            continue;
        const size_t cell = (size_t)mi * G.n_P + pi;
        double tm[13];
        uint32_t sv[3] = {0u, 0u, 0u};
        {
            int r = 0;
#pragma unroll
            for (int id = 0; id < 13; ++id) {
                tm[id] = 0.0;
                if ((mask >> id) & 1u) {
                    const size_t at = (size_t)r * plane + cell;
                    tm[id] = meas[at];
                    if (id == 2) sv[0] = seg[at];
                    if (id == 5) sv[1] = seg[at];
                    if (id == 9) sv[2] = seg[at];
                    ++r;
                }
            }
        }
        const u64 m = G.m[mi];
        const uint32_t P = G.P[pi];
        const double q = (double)(P - 1), fl = (double)floor_log2(P), cl = (double)ceil_log2(P);
        const double gm = S.gm[mi];
        double gs[3] = {0.0, 0.0, 0.0}, k[3] = {0.0, 0.0, 0.0};
        bool ok[3] = {true, true, true};
#pragma unroll
        for (int u = 0; u < 3; ++u) {
            if (!((mask >> (u == 0 ? 2 : u == 1 ? 5 : 9)) & 1u))
                continue;
            const u64 sz = sv[u];
            ok[u] = sz > 0 && sz <= m;
            if (ok[u]) {
                gs[u] = gap_at(tab, (double)sz);
                k[u] = segments(m, sz);
            }
        }
        double best_p[2] = {INFINITY, INFINITY}, best_m[2] = {INFINITY, INFINITY};
        double meas_of_pred_best[2] = {NAN, NAN};
        uint32_t id_p[2] = {0xFFFFFFFFu, 0xFFFFFFFFu}, id_m[2] = {0xFFFFFFFFu, 0xFFFFFFFFu};
        int r = 0;
#pragma unroll
        for (int id = 0; id < 13; ++id) {
            if (!((mask >> id) & 1u))
                continue;
            const size_t at = (size_t)r * plane + cell;
            ++r;
            const double v = score_predict(id, q, fl, cl, gm, L, R, gs, k, ok, G, S, mi, pi, P);
            __builtin_nontemporal_store(v, pred + at);
            const double t_meas = tm[id];
            const int op = id < 10 ? 0 : 1;
            if (v < best_p[op]) {
                best_p[op] = v;
                id_p[op] = (uint32_t)id;
                meas_of_pred_best[op] = t_meas;
            }
            if (t_meas < best_m[op]) {
                best_m[op] = t_meas;
                id_m[op] = (uint32_t)id;
            }
        }
        plogp_verdict_dev *o = verdict + cell;
#pragma unroll
        for (int op = 0; op < 2; ++op) {
            if (!(mask & (op == 0 ? 0x3FFu : 0x1C00u)))
                continue;
            union {
                plogp_verdict_dev vd;
                uint4 v;
            } u;
            u.vd.regret = meas_of_pred_best[op] / best_m[op] - 1.0;
            u.vd.pred_best = id_p[op];
            u.vd.meas_best = id_m[op];
            stream_out(o, u.v);
            o += plane;
        }
    }
}

// e = |(pred - meas) / meas| per point; per (strategy row r, m): the sum over P in
// ascending order from +0.0 and the maximum.  rows[(r * n_m + mi) * 2] = {sum, max}.
// A wave takes SCORE_RT rows of n_P points: per chunk of 64 process counts every lane
// loads one point of each row (coalesced) and leaves e in LDS; then lane i < SCORE_RT
// adds the 64 values of row i in order, while the loads of the next chunk are in
// flight.  The running sums stay in those lanes.
constexpr int SCORE_RT = 8;
constexpr int SCORE_WAVES = 4;

__global__ void __launch_bounds__(64 * SCORE_WAVES) k_score_rows(DeviceGrid G, int n_ids,
                                                                  const double *__restrict__ meas,
                                                                  const double *__restrict__ pred,
                                                                  double *__restrict__ rows)
{
    __shared__ double tile[SCORE_WAVES][SCORE_RT][65];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const long n_rows = (long)n_ids * G.n_m;
    const long row0 = ((long)blockIdx.x * SCORE_WAVES + w) * SCORE_RT;
    if (row0 >= n_rows)
        return;
    const int n_here = n_rows - row0 < SCORE_RT ? (int)(n_rows - row0) : SCORE_RT;
    const int n_P = G.n_P;
    double vp[SCORE_RT], vm[SCORE_RT];
    auto fetch = [&](int p0) {
        const int pi = p0 + lane;
#pragma unroll
        for (int i = 0; i < SCORE_RT; ++i) {
            vp[i] = 1.0;                  // padding: e = 0, below every real maximum
            vm[i] = 1.0;
            if (i < n_here && pi < n_P) {
                vp[i] = pred[(size_t)(row0 + i) * n_P + pi];
                vm[i] = meas[(size_t)(row0 + i) * n_P + pi];
            }
        }
    };
    fetch(0);
    // the maximum does not depend on the order: every lane keeps its own per row and the
    // lanes are combined once at the end, so that only the sum is a serial chain
    double sum = 0.0;
    double wmax[SCORE_RT];
#pragma unroll
    for (int i = 0; i < SCORE_RT; ++i)
        wmax[i] = 0.0;
    for (int p0 = 0; p0 < n_P; p0 += 64) {
#pragma unroll
        for (int i = 0; i < SCORE_RT; ++i) {
            const double err = fabs((vp[i] - vm[i]) / vm[i]);
            wmax[i] = err > wmax[i] ? err : wmax[i];
            tile[w][i][lane] = err;
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        if (p0 + 64 < n_P)
            fetch(p0 + 64);
        if (lane < n_here) {
            const int cnt = n_P - p0 < 64 ? n_P - p0 : 64;
            int j = 0;
            for (; j + 16 <= cnt; j += 16) {           // 16 LDS reads in flight, added in order
                double err[16];
#pragma unroll
                for (int u = 0; u < 16; ++u)
                    err[u] = tile[w][lane][j + u];
#pragma unroll
                for (int u = 0; u < 16; ++u)
                    sum = sum + err[u];
            }
            for (; j < cnt; ++j)
                sum = sum + tile[w][lane][j];
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
#pragma unroll
    for (int i = 0; i < SCORE_RT; ++i)
        tile[w][i][lane] = wmax[i];
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    if (lane < n_here) {
        double worst = 0.0;
#pragma unroll 16
        for (int j = 0; j < 64; ++j) {
            const double v = tile[w][lane][j];
            worst = v > worst ? v : worst;
        }
        rows[2 * (row0 + lane)] = sum;
        rows[2 * (row0 + lane) + 1] = worst;
    }
}

// A wave takes one message size at a time and walks over its process counts, 64 (its lanes)
// at a time: the measured times and segment sizes of a point are fetched before any
// arithmetic (13 + 3 independent loads per lane in flight), the predictions and the verdicts
// go out, and the relative errors e = |(pred - meas) / meas| stay in the wave for the
// statistics, so that nothing is read a second time.  Per (strategy row r, m) the sum of e
// over P is one serial chain in ascending P from +0.0: the lanes leave their e in an LDS tile
// (SCORE_TILE_ROWS strategy rows at a time), then lane j adds the 64 values of row j in
// order, sixteen LDS reads at a time, and keeps the running sum for the next 64 process
// counts; the maximum does not depend on the order, every lane keeps its own per row and the
// lanes are combined once per message size.  rows[(r * n_m + mi) * 2] = {sum, max}.
// A big table is staged once per workgroup, and the waves take sizes with a stride.
// Bound by memory: 1.01 GB for 4096 sizes x 976 process counts x 13 strategies in 215 us, 4.7 TB/s
// where a large copy reaches 4.9; without the divisions, the serial sums or the searches it is at
// most 3 % faster.  (225 us before g(s) and k were kept while the segment sizes stay the same.)
constexpr int SCORE_TILE_ROWS = 7;                     // 13 strategy rows go through the tile in two halves
constexpr int SCORE_TILE_LD = 65;

// BIG: workgroups of 1024 threads (128 registers a lane); otherwise 256, and the measured times
// of the next 64 process counts are fetched while the current ones are worked on.
template <bool BIG>
__global__ void __launch_bounds__(BIG ? 1024 : 256) k_score_fused(DeviceTables T, DeviceGrid G, Scratch S,
                                                const double *__restrict__ meas,
                                                const uint32_t *__restrict__ seg,
                                                double *__restrict__ pred,
                                                plogp_verdict_dev *__restrict__ verdict,
                                                double *__restrict__ rows)
{
    extern __shared__ double lds[];
    const uint32_t mask = G.mask;
    const bool any_seg = (mask & 0x224u) != 0;
    LdsTable tab = {nullptr, nullptr, nullptr, T.n};
    if (any_seg)
        tab = stage_table(lds, T, 0);                 // for g(s) at the measured segment sizes
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int n_waves = blockDim.x >> 6;
    double *tile = lds + (any_seg ? 3 * T.n : 0) + (size_t)wave * SCORE_TILE_ROWS * SCORE_TILE_LD;
    const double L = T.L[0];
    const double g1 = S.g1[0];
    const double R = __builtin_fma(3.0, L, 2.0 * g1);
    const int n_P = G.n_P;
    const size_t plane = (size_t)G.n_m * n_P;
    int n_ids = 0;
#pragma unroll
    for (int id = 0; id < 13; ++id)
        n_ids += (mask >> id) & 1u;
    auto wave_sync = [&]() {
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    };
    for (int mi = blockIdx.x * n_waves + wave; mi < G.n_m; mi += gridDim.x * n_waves) {
        const u64 m = G.m[mi];
        const double gm = S.gm[mi];
        double wmax[13];                               // this lane's largest e per strategy
#pragma unroll
        for (int id = 0; id < 13; ++id)
            wmax[id] = 0.0;
        double sum_lo = 0.0, sum_hi = 0.0;             // lane j: rows j and SCORE_TILE_ROWS + j
        double gs[3] = {0.0, 0.0, 0.0}, k[3] = {0.0, 0.0, 0.0};
        uint32_t sv_had[3] = {0u, 0u, 0u};             // the segment sizes they belong to (0: none)
        double tm_n[13];
        uint32_t sv_n[3] = {0u, 0u, 0u};
        auto fetch = [&](int p0, double (&tmv)[13], uint32_t (&svv)[3]) {
            const int pi = p0 + lane < n_P ? p0 + lane : n_P - 1;
            const size_t cell = (size_t)mi * n_P + pi;
            int r = 0;
#pragma unroll
            for (int id = 0; id < 13; ++id) {
                tmv[id] = 0.0;
                if ((mask >> id) & 1u) {
                    const size_t at = (size_t)r * plane + cell;
                    tmv[id] = __builtin_nontemporal_load(meas + at);
                    if (id == 2) svv[0] = seg[at];
                    if (id == 5) svv[1] = seg[at];
                    if (id == 9) svv[2] = seg[at];
                    ++r;
                }
            }
        };
        if (!BIG)
            fetch(0, tm_n, sv_n);
        for (int p0 = 0; p0 < n_P; p0 += 64) {
            const bool valid = p0 + lane < n_P;
            const int pi = valid ? p0 + lane : n_P - 1;     // padding lanes work on a valid point, quietly
            const size_t cell = (size_t)mi * n_P + pi;
            double tm[13];
            uint32_t sv[3] = {0u, 0u, 0u};
            if (BIG) {
                fetch(p0, tm, sv);
            } else {
#pragma unroll
                for (int id = 0; id < 13; ++id)
                    tm[id] = tm_n[id];
#pragma unroll
                for (int u = 0; u < 3; ++u)
                    sv[u] = sv_n[u];
                if (p0 + 64 < n_P)
                    fetch(p0 + 64, tm_n, sv_n);
            }
            const uint32_t P = G.P[pi];
            const double q = (double)(P - 1), fl = (double)floor_log2(P), cl = (double)ceil_log2(P);
            bool ok[3] = {true, true, true};
            int before = -1;                           // the segmented row before this one
#pragma unroll
            for (int u = 0; u < 3; ++u) {
                if (!((mask >> (u == 0 ? 2 : u == 1 ? 5 : 9)) & 1u))
                    continue;
                const u64 sz = sv[u];
                ok[u] = sz > 0 && sz <= m;
                // g(s) and k from the 64 process counts before, or from the row before, where the
                // segment sizes are the same in every lane
                if (__ballot(sv[u] != sv_had[u]) != 0) {
                    if (u > 0 && before == u - 1 && __ballot(sv[u] != sv[u > 0 ? u - 1 : 0]) == 0) {
                        gs[u] = gs[u > 0 ? u - 1 : 0];
                        k[u] = k[u > 0 ? u - 1 : 0];
                    } else if (ok[u]) {
                        gs[u] = gap_at(tab, (double)sz);
                        k[u] = segments(m, sz);
                    }
                    sv_had[u] = sv[u];
                }
                before = u;
            }
            double best_p[2] = {INFINITY, INFINITY}, best_m[2] = {INFINITY, INFINITY};
            double meas_of_pred_best[2] = {NAN, NAN};
            uint32_t id_p[2] = {0xFFFFFFFFu, 0xFFFFFFFFu}, id_m[2] = {0xFFFFFFFFu, 0xFFFFFFFFu};
            double ev[13];                             // e of this point per strategy (0 in padding lanes)
            int r = 0;
#pragma unroll
            for (int id = 0; id < 13; ++id) {
                ev[id] = 0.0;
                if (!((mask >> id) & 1u))
                    continue;
                const size_t at = (size_t)r * plane + cell;
                ++r;
                const double v = score_predict(id, q, fl, cl, gm, L, R, gs, k, ok, G, S, mi, pi, P);
                if (valid)
                    __builtin_nontemporal_store(v, pred + at);
                const double t_meas = tm[id];
                const double e = fabs((v - t_meas) / t_meas);
                ev[id] = valid ? e : 0.0;
                wmax[id] = ev[id] > wmax[id] ? ev[id] : wmax[id];
                const int op = id < 10 ? 0 : 1;
                if (v < best_p[op]) {
                    best_p[op] = v;
                    id_p[op] = (uint32_t)id;
                    meas_of_pred_best[op] = t_meas;
                }
                if (t_meas < best_m[op]) {
                    best_m[op] = t_meas;
                    id_m[op] = (uint32_t)id;
                }
            }
            if (valid) {
                plogp_verdict_dev *o = verdict + cell;
#pragma unroll
                for (int op = 0; op < 2; ++op) {
                    if (!(mask & (op == 0 ? 0x3FFu : 0x1C00u)))
                        continue;
                    union {
                        plogp_verdict_dev vd;
                        uint4 v;
                    } u;
                    u.vd.regret = meas_of_pred_best[op] / best_m[op] - 1.0;
                    u.vd.pred_best = id_p[op];
                    u.vd.meas_best = id_m[op];
                    stream_out(o, u.v);
                    o += plane;
                }
            }
            // the sums: the strategy rows go through the tile in two halves; a padding lane
            // holds +0.0, which leaves a sum as it is
#pragma unroll
            for (int half = 0; half < 2; ++half) {
                int rr = 0;
#pragma unroll
                for (int id = 0; id < 13; ++id) {
                    if (!((mask >> id) & 1u))
                        continue;
                    if (rr / SCORE_TILE_ROWS == half)
                        tile[(rr % SCORE_TILE_ROWS) * SCORE_TILE_LD + lane] = ev[id];
                    ++rr;
                }
                wave_sync();
                if (half * SCORE_TILE_ROWS + lane < n_ids && lane < SCORE_TILE_ROWS) {
                    double acc = half == 0 ? sum_lo : sum_hi;
                    const double *mine = tile + lane * SCORE_TILE_LD;
#pragma unroll
                    for (int j = 0; j < 64; j += 16) {     // 16 LDS reads in flight, added in order
                        double err[16];
#pragma unroll
                        for (int u = 0; u < 16; ++u)
                            err[u] = mine[j + u];
#pragma unroll
                        for (int u = 0; u < 16; ++u)
                            acc = acc + err[u];
                    }
                    if (half == 0)
                        sum_lo = acc;
                    else
                        sum_hi = acc;
                }
                wave_sync();
            }
        }
        // the maxima over the lanes, the same way, and the two results of every row
#pragma unroll
        for (int half = 0; half < 2; ++half) {
            int rr = 0;
#pragma unroll
            for (int id = 0; id < 13; ++id) {
                if (!((mask >> id) & 1u))
                    continue;
                if (rr / SCORE_TILE_ROWS == half)
                    tile[(rr % SCORE_TILE_ROWS) * SCORE_TILE_LD + lane] = wmax[id];
                ++rr;
            }
            wave_sync();
            const int row = half * SCORE_TILE_ROWS + lane;
            if (row < n_ids && lane < SCORE_TILE_ROWS) {
                const double *mine = tile + lane * SCORE_TILE_LD;
                double worst = 0.0;
#pragma unroll 16
                for (int j = 0; j < 64; ++j) {
                    const double v = mine[j];
                    worst = v > worst ? v : worst;
                }
                rows[2 * ((size_t)row * G.n_m + mi)] = half == 0 ? sum_lo : sum_hi;
                rows[2 * ((size_t)row * G.n_m + mi) + 1] = worst;
            }
            wave_sync();
        }
    }
}

struct plogp_score_dev {
    double sum_abs_err;
    double max_abs_err;
    unsigned long long count;
    unsigned long long reserved;
};

// Per strategy row: the per-m sums added in ascending m from +0.0.  One workgroup
// per row: 1024 per-m results are loaded side by side into LDS and thread 0 adds them
// in order while the next 1024 are in flight.
__global__ void __launch_bounds__(1024) k_score_final(DeviceGrid G, const double *rows,
                                                      plogp_score_dev *score)
{
    __shared__ double part[1024];
    __shared__ double wave_max[16];
    const int r = blockIdx.x, tid = threadIdx.x;
    const double *mine = rows + 2 * (size_t)r * G.n_m;
    double total = 0.0, worst = 0.0;        // worst: this thread's own maximum
    double a = 0.0, b = 0.0;
    if (tid < G.n_m) {
        a = mine[2 * tid];
        b = mine[2 * tid + 1];
    }
    for (int m0 = 0; m0 < G.n_m; m0 += 1024) {
        part[tid] = a;
        worst = b > worst ? b : worst;
        __syncthreads();
        const int nxt = m0 + 1024 + tid;
        b = 0.0;
        if (nxt < G.n_m) {
            a = mine[2 * (size_t)nxt];
            b = mine[2 * (size_t)nxt + 1];
        }
        if (tid == 0) {
            const int cnt = G.n_m - m0 < 1024 ? G.n_m - m0 : 1024;
            int j = 0;
            for (; j + 16 <= cnt; j += 16) {           // 16 LDS reads in flight, added in order
                double sv[16];
#pragma unroll
                for (int u = 0; u < 16; ++u)
                    sv[u] = part[j + u];
#pragma unroll
                for (int u = 0; u < 16; ++u)
                    total = total + sv[u];
            }
            for (; j < cnt; ++j)
                total = total + part[j];
        }
        __syncthreads();
    }
    // the maximum over all threads (any order gives the same value)
    for (int off = 32; off > 0; off >>= 1) {
        const double o = __shfl_xor(worst, off, 64);
        worst = o > worst ? o : worst;
    }
    if ((tid & 63) == 0)
        wave_max[tid >> 6] = worst;
    __syncthreads();
    if (tid == 0) {
        double top = 0.0;
        for (int i = 0; i < 16; ++i)
            top = wave_max[i] > top ? wave_max[i] : top;
        plogp_score_dev sc;
        sc.sum_abs_err = total;
        sc.max_abs_err = top;
        sc.count = (unsigned long long)G.n_m * (unsigned long long)G.n_P;
        sc.reserved = 0ull;
        score[r] = sc;
    }
}

// ---- the planes beyond Tables 1 and 2 -------------------------------------------
//
// Section 3 of the paper names Gather and Barrier as patterns that are built like
// Broadcast and Scatter.  In pLogP a Gather is its Scatter with every message
// reversed (the same sends, the other way round, over the same span of time; the
// root's receptions lie a gap apart as its sends did): rows 13..15 are the
// expressions of Table 2, on the same two sums.  A Barrier carries no payload: a
// one-byte fan-in to the root and a one-byte fan-out, flat (row 16: twice the flat
// row of Table 1 at g(1)) or binomial (row 17: twice its binomial row at g(1)); it
// does not depend on the message size.  One thread per (table, m, P), lanes along
// P; g(m), g(1) and the sums come from the staged path's first steps.
__global__ void __launch_bounds__(256) k_more_planes(DeviceTables T, DeviceGrid G, Scratch S,
                                                     plogp_cell_dev *out, int n_pchunks)
{
    int bid = (int)blockIdx.x;
    const int pi = (bid % n_pchunks) * 256 + (int)threadIdx.x;
    bid /= n_pchunks;
    const int mi = bid % G.n_m, t = bid / G.n_m;
    if (pi >= G.n_P)
        return;
    const uint32_t P = G.P[pi];
    const double L = T.L[t];
    const double q = (double)(P - 1u), fl = (double)floor_log2(P), cl = (double)ceil_log2(P);
    const size_t plane = (size_t)G.n_m * G.n_P;
    const int first = ((G.mask & 0x3FFu) ? 1 : 0) + ((G.mask & 0x1C00u) ? 1 : 0);   // planes before these
    plogp_cell_dev *o = out + ((size_t)t * G.n_ops + first) * plane + (size_t)mi * G.n_P + pi;
    if (G.extra & 7u) {
        // the rows of Table 2 under the ids of their Gather twins
        const uint32_t as_scatter = (G.extra & 7u) << 10;
        const double gm = S.gm[(size_t)t * G.n_m + mi];
        const double s11 = (as_scatter & (1u << 11)) ? chain_sum_of(G, S, t, mi, pi, P) : 0.0;
        const double s12 = (as_scatter & (1u << 12))
                               ? S.sum2[((size_t)t * G.n_m + mi) * (size_t)(G.cl_max + 1) + ceil_log2(P)] : 0.0;
        Best b = decide_scatter(as_scatter, q, cl, gm, L, s11, s12);
        b.id += 3u;
        store_cell(o, b);
        o += plane;
    }
    if (G.extra & 0x18u) {
        store_cell(o, decide_barrier(G.extra, q, fl, cl, L, S.g1[t]));
    }
}

}  // namespace

// ---------------------------------------------------------------- launch wrappers

static const size_t kMaxTableLds = (size_t)3 * 4096 * sizeof(double) + 96 +
                                   (size_t)2 * SWEEP_M_MAX_S * sizeof(double);   // + g(s), 1/s in k_terms
static const size_t kMaxChainLds = ((size_t)4 * 4096 + CHAIN_PAD + CHAIN_MAX_S) * sizeof(double);   // + interval widths

static DeviceInfo g_device = {256, (size_t)160 * 1024};

const DeviceInfo &device_info() { return g_device; }

hipError_t kernels_init()
{
    hipError_t e;
    {
        int dev = 0;
        hipDeviceProp_t prop;
        if ((e = hipGetDevice(&dev)) != hipSuccess) return e;
        if ((e = hipGetDeviceProperties(&prop, dev)) != hipSuccess) return e;
        if (prop.multiProcessorCount > 0) g_device.n_cu = prop.multiProcessorCount;
        // the kernels that fill a compute unit's LDS were laid out for 160 KB; a device that
        // reports less gets fewer workgroups per unit from the same formulas
        if (prop.maxSharedMemoryPerMultiProcessor >= (size_t)64 * 1024)
            g_device.lds_per_cu = prop.maxSharedMemoryPerMultiProcessor;
    }
    e = hipFuncSetAttribute(reinterpret_cast<const void *>(k_interp),
                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)kMaxTableLds);
    if (e != hipSuccess) return e;
    e = hipFuncSetAttribute(reinterpret_cast<const void *>(k_eval),
                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)kMaxTableLds);
    if (e != hipSuccess) return e;
    for (const void *k : {reinterpret_cast<const void *>(k_eval_chain<4, EVAL_SEARCH>),
                          reinterpret_cast<const void *>(k_eval_chain<4, EVAL_STEP>)}) {
        e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)eval_chain_lds(4096, 4, 768));
        if (e != hipSuccess) return e;
    }
    for (const void *k : {reinterpret_cast<const void *>(k_eval_chain<8, EVAL_WALK>),
                          reinterpret_cast<const void *>(k_eval_chain<8, EVAL_SEARCH>),
                          reinterpret_cast<const void *>(k_eval_chain<8, EVAL_STEP>)}) {
        e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)eval_chain_lds(4096, 8, 384));
        if (e != hipSuccess) return e;
    }
    e = hipFuncSetAttribute(reinterpret_cast<const void *>(k_terms),
                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)kMaxTableLds);
    if (e != hipSuccess) return e;
    e = hipFuncSetAttribute(reinterpret_cast<const void *>(k_chain_blocks),
                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)kMaxChainLds);
    if (e != hipSuccess) return e;
    e = hipFuncSetAttribute(reinterpret_cast<const void *>(k_terms_chain<false>),
                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)kMaxTableLds);
    if (e != hipSuccess) return e;
    e = hipFuncSetAttribute(reinterpret_cast<const void *>(k_terms_chain<true>),
                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)kMaxTableLds);
    if (e != hipSuccess) return e;
    for (const void *k : {reinterpret_cast<const void *>(k_tile<false>), reinterpret_cast<const void *>(k_tile<true>)}) {
        e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)(g_device.lds_per_cu - TILE_STATIC_LDS));
        if (e != hipSuccess) return e;
    }
    e = hipFuncSetAttribute(reinterpret_cast<const void *>(k_score_points),
                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)kMaxTableLds);
    if (e != hipSuccess) return e;
    // (the table plus the waves' tiles; the launch checks the sum against the device's LDS)
    e = hipFuncSetAttribute(reinterpret_cast<const void *>(k_score_fused<true>),
                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)g_device.lds_per_cu);
    if (e != hipSuccess) return e;
    e = hipFuncSetAttribute(reinterpret_cast<const void *>(k_score_fused<false>),
                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)g_device.lds_per_cu);
    if (e != hipSuccess) return e;
    for (const int gp : {2, 4, 6, 9, 12})
        for (const bool dense : {false, true}) {
            const void *k = reinterpret_cast<const void *>(sweep_s_kernel(gp, dense));
            e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, SWEEP_S_PASS * (int)sizeof(double));
            if (e != hipSuccess) return e;
        }
    const void *batch_kernels[4] = {
        reinterpret_cast<const void *>(k_batch_t<BATCH_T_PC, BATCH_T_PS, false, false>),
        reinterpret_cast<const void *>(k_batch_t<BATCH_T_PC, BATCH_T_PS, false, true>),
        reinterpret_cast<const void *>(k_batch_t<BATCH_T_PC, BATCH_T_PS, true, false>),
        reinterpret_cast<const void *>(k_batch_t<BATCH_T_PC, BATCH_T_PS, true, true>)};
    for (const void *k : batch_kernels) {
        e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)BATCH_T_LDS_MAX);
        if (e != hipSuccess) return e;
    }
    return e;
}

hipError_t launch_slopes(const DeviceTables &T, double *slope_out, hipStream_t st)
{
    hipLaunchKernelGGL(k_slopes, dim3(T.n_tables), dim3(256), 0, st, T, slope_out);
    return hipGetLastError();
}

hipError_t launch_load_packed(const PackedTables &packed, double *d_block, int n, int n_tables, hipStream_t st)
{
    hipLaunchKernelGGL(k_load_packed, dim3(1), dim3(256), 0, st, packed, d_block, n, n_tables);
    return hipGetLastError();
}

hipError_t launch_interp(const DeviceTables &T, int table, const uint64_t *d_z, size_t n,
                         double *d_out, hipStream_t st)
{
    if (n == 0) return hipSuccess;
    if ((n + 255) / 256 > 0x7FFFFFFFull) return hipErrorInvalidValue;
    const size_t lds = (size_t)3 * T.n * sizeof(double);
    const unsigned blocks = (unsigned)((n + 255) / 256);
    hipLaunchKernelGGL(k_interp, dim3(blocks), dim3(256), lds, st, T, table,
                       reinterpret_cast<const u64 *>(d_z), n, d_out);
    return hipGetLastError();
}

hipError_t launch_eval(const DeviceTables &T, int table, int strategy, const uint64_t *d_m,
                       const uint32_t *d_P, const uint64_t *d_s, size_t n, double *d_out,
                       hipStream_t st)
{
    if (n == 0) return hipSuccess;
    if ((n + 255) / 256 > 0x7FFFFFFFull) return hipErrorInvalidValue;
    if (strategy == 11 || strategy == 14) {
        // many: a full chip with one workgroup of 384 points per compute unit, as a big table leaves
        // room for (a small one leaves room for enough waves anyhow: 256 samples 103 us, 107 as many).
        // More points per workgroup then stage the table less often (300 000 points with P up to 1024,
        // 1500 samples: 313 us with 768, 468 with 384; 600 samples 203 with 256, 227 with 384)
        const bool many = n > (size_t)384 * device_info().n_cu && T.n > EVAL_SEARCH_N;
        const int levels = many ? 4 : 8, threads = T.n <= (many ? 640 : 512) ? 256 : many ? 768 : 384;
        // (step: 450 samples, 290 000 points with P up to 300 80 us, 85 searched for, up to 70 65 and 62; 600: 108
        // and 104, 74 and 62; 256 samples, 100 000 points up to 122 30 and 28)
        const bool step = n >= (size_t)768 * device_info().n_cu && T.n <= 512;
        const auto kern = T.n <= (step ? 64 : 72) ? k_eval_chain<8, EVAL_WALK>
                          : many ? (step ? k_eval_chain<4, EVAL_STEP> : k_eval_chain<4, EVAL_SEARCH>)
                                 : (step ? k_eval_chain<8, EVAL_STEP> : k_eval_chain<8, EVAL_SEARCH>);
        hipLaunchKernelGGL(kern, dim3((unsigned)((n + threads - 1) / threads)), dim3(threads),
                           eval_chain_lds(T.n, levels, threads), st, T, table, reinterpret_cast<const u64 *>(d_m), d_P,
                           n, d_out);
        return hipGetLastError();
    }
    const size_t lds = (size_t)3 * T.n * sizeof(double);
    const unsigned blocks = (unsigned)((n + 255) / 256);
    hipLaunchKernelGGL(k_eval, dim3(blocks), dim3(256), lds, st, T, table, strategy,
                       reinterpret_cast<const u64 *>(d_m), d_P,
                       reinterpret_cast<const u64 *>(d_s), n, d_out);
    return hipGetLastError();
}

// Message sizes per workgroup of the tile path (k_tile): 0 = the path does not take this job.
// Few candidates, few blocks of the chain sum, enough (table, m) rows: a workgroup takes about 20
// us from its first load to its last store, however many of them run (tables of 57 samples, 36
// process counts up to 1500: 1200 rows 24 us against 16 on the staged path, 3600 rows 24 against
// 27, 12 000 rows 30 against 59).  Smaller tiles to fill the chip do not help: what a workgroup
// does once per table outweighs them (4000 rows: 27 us with 32 sizes a tile, 43 with eight).
static int tile_sizes(const DeviceTables &T, const DeviceGrid &G, bool only_where_faster)
{
    const bool few = T.n <= TILE_FEW_N;
    if ((long)T.n_tables * G.n_m < (few ? 1 : 2) * TILE_MIN_ROWS * device_info().n_cu || G.n_s > TILE_NS ||
        G.n_blk > TILE_MAX_BLK)
        return 0;
    const size_t lds_per_cu = device_info().lds_per_cu;
    const size_t table = ((size_t)4 * T.n + CHAIN_PAD) * sizeof(double);
    // a small table: six workgroups per compute unit (333 tables of 57 samples x 203 sizes: 79 us, 80
    // with four, 90 with eight); a table of up to about 640 samples: three (500 samples, 200 process
    // counts: 274 us, 563 with one); a bigger one: all the LDS
    const size_t most = table <= lds_per_cu / 16 ? lds_per_cu / 6 : table <= lds_per_cu / 8 ? lds_per_cu / 3 : lds_per_cu;
    int M = TILE_MAX_M < G.n_m ? TILE_MAX_M : G.n_m;
    auto bytes = [&](int m) {
        return (size_t)TileLds(T.n, G.n_s, G.n_P, G.n_blk, G.cl_max, m).slots * sizeof(double) + TILE_STATIC_LDS;
    };
    // (half the LDS where that makes one tile of all sizes: 400 tables of 500 samples x 21 sizes x 200
    // process counts 65 us, 72 in two tiles)
    const bool one_tile = table > lds_per_cu / 16 && M == G.n_m && bytes(M) <= lds_per_cu / 2;
    while (M > 1 && bytes(M) > most && !one_tile)
        --M;
    if (bytes(M) > lds_per_cu)
        return 0;
    const int tiles = (G.n_m + M - 1) / M;               // then the same for every tile, but the last
    // Every tile stages its table, and a big table leaves room for one workgroup per compute unit: the
    // staged path, which stages it once for all sizes, takes these (333 tables x 203 sizes, staged and
    // in tiles: 4096 samples, 37 process counts up to 300 213 and 416 us, without the chain 79 and 204;
    // 600 samples, 200 up to 2000 297 and 604), except
    // - where one tile holds all of a table's sizes (400 tables x 21 sizes: 1500 samples, 37 process
    //   counts 81 and 48, 200 109 and 122, without the chain 19 and 15, 4096 samples 31 and 43; 600
    //   samples, 200 process counts 80 and 65);
    // - without chain sums up to 1024 samples (600: 60 and 45) or few rows (60 tables x 140 sizes, 1500
    //   samples 19 and 16);
    // - few process counts and few blocks, up to two of which let the lanes share the searches (12 up to
    //   64: 1100 samples 120 and 74, 1500 124 and 101, 2500 130 and 213; 1500 samples, 6 up to 100 95 and
    //   108; 12 up to 200 1100 samples 144 and 109; 10 000 sizes of one table of 2500 samples, 12 up to 64
    //   62 and 41, of 600 samples, 12 up to 200 25 and 28);
    // - short sums, few rows and between 1024 and 2048 samples, where the staged path has launches of
    //   their own for terms and sums (60 tables x 140 sizes, 37 up to 300: 1100 samples 57 and 40, 1000
    //   samples 35 and 39, 2500 60 and 71; 37 up to 1500, 1500 samples 50 and 64).
    const bool chain = (G.mask & (1u << 11)) != 0;
    const bool few_rows = (long)T.n_tables * G.n_m < 4 * TILE_MIN_ROWS * device_info().n_cu;
    if (!few && only_where_faster) {
        const bool worth = tiles == 1 ? (chain ? G.n_P <= 64 || T.n <= 1024 : T.n <= 2048)
                           : !chain ? T.n <= 1024 || (few_rows && T.n <= 2048)
                                    : (G.n_P < 32 && T.n <= 1280 && G.n_blk <= (few_rows ? 2 : 4)) ||
                                          (few_rows && G.n_P < 32 && G.n_blk <= 2) ||
                                          (few_rows && T.n > 1024 && T.n <= 2048 && G.n_blk <= 8);
        if (!worth)
            return 0;
    }
    return (G.n_m + tiles - 1) / tiles;
}

// Few candidates, few blocks of the chain sum, few samples: one workgroup per (table, m) can do
// the whole path (k_row).
static bool use_row_path(const DeviceTables &T, const DeviceGrid &G)
{
    return G.n_s <= ROW_NS && G.n_blk <= ROW_MAX_BLK && T.n <= ROW_MAX_N &&
           (long)T.n_tables * G.n_m <= 65535 * 16;
}

// Masks with Gather or Barrier rows: (table, m) rows per compute unit up to which one workgroup per row beats
// the staged path, which for these masks has one launch more and reads its terms more often.  How far that
// carries depends on what the staged path has to do anyway: most where Broadcast, Scatter and Gather share
// launches and sums, least where there are Broadcast rows and no sums; further with many process counts (of
// which the staged path makes more passes) and with many candidates for few process counts (a lane of its
// sweep then takes all of a size); not as far where a table of more than 128 samples has to be staged per
// row.  Every line lies where whole calls on 16, 64 and 300 samples, 5 to 50 candidates, 5 to 1500 process
// counts and 250 to 50 000 rows cross, to 4 % on the staged side (us per row and staged in brackets; 64
// samples, 15 candidates):
//   all 18 rows            5 process counts up to 6     4100 rows  21  (25)    8100  38  (33)
//                         36 up to 1500                 6000       43  (46)    8100  56  (54)
//                        100 up to 1500                 8100       56  (62)  16 000 105  (97)
//                        300 up to 1500               16 000      118 (155)
//   Gather                12 up to 200                  2000       14  (17)    4100  26  (22)
//                        255 up to 1500                 8100       65  (69)  16 000 124 (109)
//   Barrier                5 up to 6                    3000       11  (13)    6000  20  (13)  16 000 47 (16)
//                        300 up to 1500                 8100       30  (39)  16 000  54  (62)
//   Tables 1, 2, Barrier  36 up to 1500                 2000       16  (19)    6000  42  (34)
//   Broadcast, Barrier    36 up to 60                   2000       11  (14)    4100  21  (16)
//                        512 up to 513                  8100       54  (59)  16 000 102  (89)
static long row_path_most(const DeviceTables &T, const DeviceGrid &G)
{
    constexpr long kAny = 1L << 40;
    const bool bcast = (G.mask & 0x3FFu) != 0, scatter = (G.mask & 0x1C00u) != 0;
    const bool chain = (G.need & (1u << 11)) != 0, gather_chain = (G.extra & 2u) != 0;
    const bool big = T.n > 128, long_sums = G.n_blk >= 16, wide = G.n_P >= 256;
    const bool candidates = bcast && G.n_s > 32 && G.n_P < 32;
    const long n_P = G.n_P;
    const auto at_least = [](long a, long b) { return a > b ? a : b; };
    if (n_P >= 1024 || (n_P >= 512 && gather_chain && (scatter || !bcast)))
        return kAny;
    if (gather_chain && scatter) {
        if (wide) return 64;
        if (bcast) return n_P >= 64 ? 32 : candidates ? 28 : long_sums ? 24 : 17;
        return at_least(12, n_P / 6);
    }
    if (gather_chain) {
        const long most = candidates ? 20 : at_least(big ? 10 : 11, (big ? 9 : 12) * n_P / 100);
        return wide && (!bcast || n_P >= 512) ? most * 3 / 2 : most;
    }
    if (chain)
        return candidates ? 22 : at_least(bcast ? (n_P < 32 || !long_sums ? 12 : 10) : long_sums ? 7 : 10,
                                          (big ? 6 : 9) * n_P / 128 * (wide ? 2 : 1));
    if (bcast || scatter)
        return candidates ? 15 : at_least(8, big || !wide ? n_P / 21 : n_P / 14);
    return at_least(big ? 10 : n_P < 32 ? 12 : 13, big ? (wide ? n_P / 10 : n_P / 15) : wide ? n_P / 6 : n_P / 9);
}

// LDS of a k_batch_t workgroup: 64 tables by interval, their g(s), the output staging.
static size_t batch_t_lds(int n, int n_s)
{
    return ((size_t)2 * (n + 2) + (n_s ? n_s : 1)) * 64 * sizeof(double) +
           (size_t)BATCH_T_WAVES * BATCH_T_STAGE + (size_t)(n_s ? n_s : 1) * 4 + 16;
}

// Batches whose tables share their sample sizes, with enough tables to fill waves and
// few enough samples and candidates for the LDS staging: lanes over tables.
static bool use_table_lane_path(const DeviceTables &T, const DeviceGrid &G)
{
    // a lane's byte offset inside a store (up to 7 tables + 7 cells on) is kept in 32 bits
    const size_t table_cells = (size_t)G.n_ops * G.n_m * G.n_P;
    return T.shared_x && T.n_tables >= 64 && (long)T.n_tables * G.n_m >= 8192 &&
           table_cells <= ((size_t)1 << 24) && batch_t_lds(T.n, G.n_s) <= BATCH_T_LDS_MAX;
}

namespace {

// Lays the arrays of a plan out one after the other, each on a 256-byte boundary; the first
// 256 bytes stay free (arrays of size 0 point there).
struct LayoutBuilder {
    size_t at = 256;
    bool too_big = false;          // a size did not fit: the plan is refused
    // an array of a * b * c * d elements of `elem` bytes (a factor of 0 makes it empty)
    size_t take(size_t elem, size_t a, size_t b = 1, size_t c = 1, size_t d = 1)
    {
        constexpr size_t kMaxBytes = (size_t)1 << 46;       // no single array beyond 64 TiB: sizes stay far from wrapping
        size_t count = a;
        for (size_t f : {b, c, d}) {
            if (f != 0 && count > kMaxBytes / f) too_big = true;
            count *= f;
        }
        if (count > kMaxBytes / elem) too_big = true;
        if (too_big || count == 0) return 0;
        const size_t here = at;
        at += (count * elem + 255) & ~(size_t)255;
        return here;
    }
};

constexpr long kMaxLaunch = 0x7FFFFFFFL;      // workgroups of one launch, and int indices inside the kernels

}  // namespace

Scratch bind_scratch(void *base, const ScratchLayout &lay)
{
    char *b = static_cast<char *>(base);
    Scratch S = {};
    S.g1 = reinterpret_cast<double *>(b + lay.g1);
    S.gs = reinterpret_cast<double *>(b + lay.gs);
    S.gm = reinterpret_cast<double *>(b + lay.gm);
    S.sum2 = reinterpret_cast<double *>(b + lay.sum2);
    S.blk = reinterpret_cast<double *>(b + lay.blk);
    S.pre = reinterpret_cast<double *>(b + lay.pre);
    S.part = reinterpret_cast<double *>(b + lay.part);
    S.rcp = reinterpret_cast<double *>(b + lay.rcp);
    S.segC = reinterpret_cast<double *>(b + lay.segC);
    S.segA = reinterpret_cast<double *>(b + lay.segA);
    S.segB = reinterpret_cast<double *>(b + lay.segB);
    S.amin = reinterpret_cast<double *>(b + lay.amin);
    S.minG = reinterpret_cast<double *>(b + lay.minG);
    S.nv = reinterpret_cast<int *>(b + lay.nv);
    S.batch.rec = reinterpret_cast<double *>(b + lay.rec);
    S.batch.tab = reinterpret_cast<double *>(b + lay.tab);
    S.batch_ys = reinterpret_cast<double *>(b + lay.batch_ys);
    return S;
}

// Up to how many chain items of a tile eight lanes share each of those that enter several intervals (if these
// are no more than a wave).  It saves a workgroup the wait for its slowest wave and costs instructions, so it
// depends on whether the workgroups are on the chip at once, or, where a table has several tiles, some of which
// have little to wait for, two thirds of what is.  If so, up to 312: 7 process counts up to 667, 30 samples, 1136
// tables x 22 sizes, 242 items, 20.7 us shared, 22.9 with a lane per item; 12 samples, 250 x 56 sizes, 308, 15.0
// and 16.2, 70 x 200 sizes, 319, 15.9 and 15.5; and with few process counts, sums at which cost the shared ones
// most, and one or two tiles as long as a lane per item takes the four waves no more than two turns (12 up to
// 1480, 30 samples, 350 x 20 sizes, 480 items 17.3 and 19.0, 12 samples, 233 x 30, 720 18.1 and 16.9; 30 up to
// 1174, 20 samples, 1136 x 22, 418 28.2 and 27.2).  If not, few: 12 samples, 300 x 200 sizes x 8 up to 455, 232
// items, 31.5 and 30.0; 30 samples, 150 sizes x 20 up to 300, 300 tables 28.4 and 27.5, 166 19.0 and 19.0, 93
// 14.8 and 15.8; more of up to eight blocks on tables from TILE_DENSE_N samples on, which enter more intervals (49
// samples, 300 tables x 66 sizes, 176 items 24.7 and 26.0).
static int tile_shared(const DeviceTables &T, const DeviceGrid &G, const TunePlan &p)
{
    const long by_lds = (long)(device_info().lds_per_cu / (p.tile_lds + TILE_STATIC_LDS));
    const long at_once = device_info().n_cu * (by_lds < TILE_WG_PER_CU ? by_lds : TILE_WG_PER_CU);
    const long wg = (long)T.n_tables * p.n_tiles, most = at_once * 2 / 3;
    if (wg <= most && p.n_tiles <= 2 && G.n_P <= 16)
        return 2 * TILE_THREADS;
    if (wg <= (p.n_tiles == 1 ? at_once : most))
        return 312;
    return G.n_blk <= 8 && T.n >= TILE_DENSE_N ? 256 : 128;
}

// The tile path's part of a plan: one launch, and no scratch beside the spare.
static bool plan_tiles(const DeviceTables &T, const DeviceGrid &G, int tile_m, TunePlan &p)
{
    p.path = TUNE_TILE;
    p.tile_m = tile_m;
    p.n_tiles = (G.n_m + tile_m - 1) / tile_m;
    p.tile_lds = (size_t)TileLds(T.n, G.n_s, G.n_P, G.n_blk, G.cl_max, tile_m).slots * sizeof(double);
    p.tile_shared = tile_shared(T, G, p);
    p.lay.total = LayoutBuilder().at;
    return (long)T.n_tables * p.n_tiles <= kMaxLaunch;
}

// Whether a workgroup per row leaves out the candidates that cannot win row 5 (row5_candidates) or evaluates all.
// The former is 70 instructions that wait for one another and a candidate at a time after them, the latter two
// round trips for 16 candidates.  The latter is the shorter wait where a call waits for nothing else, which is where no
// chain sum is needed, beside which the others wait: up to 24 candidates for a few waves of process counts (64 sizes
// of up to 8 MB, 30 samples, the Broadcast rows: 13 candidates x 64 up to 640 4.53 us, 4.84 with those left out that
// cannot win; 4000 sizes x 200, 26 candidates 14.1 and 13.8), up to 8 for any number (1000 x 1000, 5 candidates 10.4
// and 10.7), and for a wave of process counts far apart, for which many can win, any number (2000 sizes x 64 up to
// 2047, 48 candidates 11.7 and 12.6; x 6 up to 30, 26, 60 sizes 4.3 and 4.0).  Beside chain sums for such process
// counts alone (30 tables x 24 sizes x 10 up to 512, 18 candidates 7.1 and 7.3; 35 sizes x 14 up to 2048, 35, 8.7 and
// 9.1; 60 x 20 up to 100, 26 5 % slower; 49 up to 50, 13, 4.05 and 4.12, left as it is; 300 sizes x 100 up to 101, 17,
// 5.5 and 5.35).
static bool row_few(const DeviceGrid &G)
{
    const int P_top = SUM_BLOCK * (G.n_blk - 1) + G.last_terms + 1;
    if ((G.need & (1u << 11)) != 0) {
        const int apart = G.n_s > 24 ? 500 : G.n_P > 32 ? 4 * G.n_P : 128;
        return G.n_s <= 12 || G.n_P > 64 || P_top < apart;
    }
    return G.n_s > 8 && (G.n_s > 24 || G.n_P > 256) && (G.n_P > 64 || P_top < 256);
}

// The same for the sweep over process counts.  With two of them per lane it is the faster to leave candidates out
// (4096 sizes x 976, 43 candidates: 38 us, 33), with one where the list is close (at least half of all counts up to
// the largest; 9000 x 300 up to 301, 34 candidates: the call 63.6, 58.0), and not where a wave's counts lie far apart
// (1638 x 100 up to 2612, 40: 8.1 us, 9.2; 5000 x 40 up to 1500, 34: the call 31.9, 33.1); not for a few candidates
// (700 samples, 6000 sizes x 1000 up to 1800: 3 candidates 2 % slower, 8 the same); and where no chain sum is read,
// so that a wave waits for little else, for many candidates and process counts alone (the Broadcast rows, 6000 x
// 300: 3 candidates 8 % slower, 8 3 %, 17 to 24 the same, 34 3 % faster; 34 x 64 3 % slower).
static bool sweep_few(const DeviceGrid &G, int ppl)
{
    const bool close = 2L * G.n_P >= (long)G.n_blk * SUM_BLOCK;
    if ((G.need & (1u << 11)) != 0)
        return G.n_s > 4 && (ppl == 2 || close);
    return G.n_s > 24 && G.n_P >= 256 && close;
}

// The row path's part, the same.
static bool plan_rows(const DeviceTables &T, const DeviceGrid &G, TunePlan &p)
{
    p.path = TUNE_ROW;
    // two process counts per lane when there are more groups of 64 than waves
    p.row_two = G.n_P > 64 * (ROW_THREADS / 64);
    p.row_few = row_few(G);
    p.row_lds = row_lds_bytes(T.n, G.n_blk, G.n_P);
    p.lay.total = LayoutBuilder().at;
    return true;
}

static bool plan_fastest(const DeviceTables &T, const DeviceGrid &G, bool terms_only, TunePlan &p)
{
    p = TunePlan{};
    p.terms_only = terms_only ? 1 : 0;
    const DeviceInfo &dev = device_info();
    const long n_cu = dev.n_cu;
    const size_t D = sizeof(double);
    const size_t nt = (size_t)T.n_tables, n_m = (size_t)G.n_m, n_mu = (size_t)G.n_mu;
    const size_t n_P = (size_t)G.n_P, n_s = (size_t)G.n_s;
    LayoutBuilder lb;
    // the planes of the rows beyond Tables 1 and 2 are written by the staged path's last launch, by
    // k_row, or by the table-lane kernel, that one only when the Gather rows are enabled exactly as
    // the Scatter rows are (or one of the two patterns is absent): it decides once for both
    const bool fast_ok = !terms_only && G.extra == 0;
    const uint32_t scatter_rows = G.mask & 0x1C00u, gather_rows = (G.extra & 7u) << 10;
    const bool lanes_ok = !terms_only && (gather_rows == 0 || scatter_rows == 0 || gather_rows == scatter_rows);
    if (lanes_ok && use_table_lane_path(T, G)) {
        p.path = TUNE_TABLE_LANES;
        // tables by interval and the per-m facts, then everything else in one kernel
        p.n_stage = (T.n_tables + BATCH_STAGE_TT - 1) / BATCH_STAGE_TT;
        long prep_items = (long)G.n_m * (T.n + 1);
        if ((long)G.n_m * G.n_s > prep_items) prep_items = (long)G.n_m * G.n_s;
        long prep_wg = (prep_items + 255) / 256;
        if (prep_wg > 1024) prep_wg = 1024;
        p.prep_wg = (int)prep_wg;
        p.setup_lds = (size_t)BATCH_STAGE_TT * (T.n + 1) * D;
        // a workgroup: 64 tables x (BATCH_T_WAVES waves x m_per_wave sizes)
        p.n_tg = (T.n_tables + 63) / 64;
        const int per = BATCH_T_WAVES;
        int m_per_wave = 8;
        while (m_per_wave > 1 && (long)p.n_tg * ((G.n_m + per * m_per_wave - 1) / (per * m_per_wave)) < 4 * n_cu)
            m_per_wave >>= 1;
        p.m_per_wave = m_per_wave;
        p.batch_mchunks = (G.n_m + per * m_per_wave - 1) / (per * m_per_wave);
        p.batch_lds = batch_t_lds(T.n, G.n_s);
        if ((long)p.n_tg * p.batch_mchunks > kMaxLaunch) return false;
        const BatchRec R(T.n, G.n_s, G.cl_max);
        p.lay.rec = lb.take(D, n_m, (size_t)R.slots);
        p.lay.tab = lb.take(D, 2 + ((size_t)T.n + 1) + 2 * (n_s ? n_s : 1) + 4 * (size_t)batch_padded_P(G.n_P));
        p.lay.batch_ys = lb.take(D, (size_t)T.n + 2, nt, 2);
        p.lay.total = lb.at;
        return !lb.too_big;
    }
    // A row per workgroup while there are few rows or many process counts.  It is one launch where
    // the staged path has two or three, and a small job is their latency.  Whole calls on tables of 64
    // samples, all 13 rows, staged in brackets (1000 rows and more: sums up to 64 terms for 12, 1500
    // for 36, 256 for 255 process counts): 64 sizes x 49 process counts x 13 candidates 5.3 us (12),
    // 20 x 16 x 34 7.5 (28), 1000 x 12 x 13 6.4 (15), 1000 x 36 x 37 9.7 (16), 3000 x 12 x 37 15 (32),
    // 4000 x 255 x 13 23 (28), 6000 x 36 x 37 39 (34), 10 000 61 (45).  Tables of 512 samples gain more
    // (4000 x 12 x 13 20 (34)).  Against tiles: 4000 rows x 12 process counts 18 (21), x 127 22 (22), 6000 x 36
    // 37 (22); 4000 x 300 24 (30), 10 000 x 300 51 (34); 10 000 x 1000 78 (96).
    // Chain sums for few cells are the one kind of row that the staged path does cheaper from fewer
    // rows on, the longer the sums the fewer, where neither the table nor the candidates are many (36
    // process counts, 13 candidates: up to 1500 2000 rows 14 (15), 3000 20 (19), 4000 26 (22); up to 700
    // 3000 rows 17 (18), 4000 22 (20); up to 1500, 2000 rows, 256 samples 16 (17), 37 candidates 16 (18), 12
    // process counts 3000 rows 20 (23)).
    const long rows = (long)T.n_tables * G.n_m;
    const long few_cells = G.n_P >= 32 && G.n_P < 64 && T.n <= 128 && G.n_s <= 16 ? G.n_blk / 4 : 0;
    // Masks with Gather or Barrier rows take the same launch up to a number of rows of their own (64 sizes x
    // 49 process counts, all 18 rows 5.8 us (16.4)).
    const bool few_rows = G.extra != 0 ? rows < row_path_most(T, G) * n_cu
                                       : G.n_P >= 512 || rows < (G.n_P >= 256 ? ROW_MAX_ROWS : ROW_MAX_ROWS / 2 - few_cells) * n_cu;
    const bool by_row = !terms_only && use_row_path(T, G) && few_rows;
    const int tile_m = fast_ok && !by_row ? tile_sizes(T, G, true) : 0;
    if (by_row)
        return plan_rows(T, G, p);
    if (tile_m > 0)
        return plan_tiles(T, G, tile_m, p);
    p.path = TUNE_STAGED;
    const size_t tab_lds = (size_t)3 * T.n * D;
    // which sweep runs: lanes over s for many candidates, else lanes over P if the grid
    // has enough process counts to fill a wave, else lanes over m
    const bool lanes_s = G.n_s > SWEEP_M_MAX_S;
    const bool lanes_p = !terms_only && !lanes_s && G.n_P >= 32 && G.n_P <= 65535 * 64;   // grid.y
    // the per-(m, s) terms A, B and min_s A in device memory: only for the sweep that runs its
    // lanes over P, and only when there is a candidate at all
    const bool pairs = lanes_p && G.n_s > 0;
    p.lanes_s = lanes_s;
    p.lanes_p = lanes_p;
    p.pairs = pairs;
    long n_items = G.n_m > G.n_s ? G.n_m : G.n_s;          // a lane takes one m and one s ...
    if (pairs && (long)G.n_m * G.n_s > n_items)
        n_items = (long)G.n_m * G.n_s;                     // ... and one (m, s) pair
    long n_chunks_l = (n_items + 255) / 256;
    // the candidates go to LDS too (for the count per m) if they fit beside the table and are
    // few: every workgroup stages them all, and for 8192 of them that takes longer (11.8 us)
    // than the thirteen dependent loads of a search in device memory (6.9 us)
    const size_t pair_lds = pairs ? (size_t)2 * G.n_s * D : 0;
    const bool stage_s = G.n_s > 0 && G.n_s <= 1024 && tab_lds + pair_lds + (size_t)G.n_s * D <= kMaxTableLds;
    p.terms_mode = (pairs ? 1 : 0) | (stage_s ? 2 : 0) | (lanes_s && !terms_only ? 4 : 0);
    p.terms_lds = tab_lds + pair_lds + (stage_s ? (size_t)G.n_s * D : 0);
    // a workgroup stages the whole table: with a big table one workgroup fits a CU, so no
    // more workgroups than CUs
    const long wg_cap = p.terms_lds > 65536 ? n_cu : 2 * n_cu;
    const long chunk_cap = wg_cap / T.n_tables > 1 ? wg_cap / T.n_tables : 1;
    if (n_chunks_l > chunk_cap) n_chunks_l = chunk_cap;
    // the per-size part in workgroups of its own, beside the others: freely for small tables;
    // for a big table (one workgroup per CU) out of the same budget of workgroups
    int n_mchunks = 0;
    if (p.terms_lds <= 16384) {
        n_mchunks = ((G.n_m + 63) / 64 + 3) / 4;
        const int cap = n_cu / T.n_tables > 1 ? (int)(n_cu / T.n_tables) : 1;
        if (n_mchunks > cap) n_mchunks = cap;
    } else if (T.n_tables == 1 && n_chunks_l >= 64) {
        n_mchunks = ((G.n_m + 63) / 64 + 3) / 4;
        if (n_mchunks > n_chunks_l / 8) n_mchunks = (int)(n_chunks_l / 8);
        if (n_chunks_l + n_mchunks > chunk_cap) n_chunks_l = chunk_cap - n_mchunks;
    }
    p.n_chunks = (int)n_chunks_l;
    p.n_mchunks = n_mchunks;
    const long terms_wg = (long)T.n_tables * (p.n_chunks + n_mchunks);
    if (terms_wg > kMaxLaunch) return false;
    p.terms_wg = (int)terms_wg;
    const bool chain = (G.need & (1u << 11)) != 0;
    p.chain = chain;
    // a big table fills most of the LDS of a CU: one large workgroup per CU then, which
    // stays for its whole share of the work (the table is staged once)
    p.chain_lds = ((size_t)4 * T.n + CHAIN_PAD) * D;
    const bool big = p.chain_lds > 32768;
    // few samples, few blocks, enough distinct sizes: a workgroup per (table, m) forms all
    // its sums, the prefix over the blocks included
    p.crow_lds = chain_row_lds(T.n, G.n_blk);
    p.chain_row = chain && T.n <= 512 && G.n_blk <= CROW_MAX_BLK && p.crow_lds <= 65536 &&
                  (long)T.n_tables * G.n_mu >= 128 && (long)T.n_tables * G.n_mu <= (1L << 24);
    // small tables: the terms and the chain sums in one launch, side by side
    p.together = chain && !big && !p.chain_row;
    // (terms beside the per-row chain sums: when the terms need little LDS)
    p.row_together = p.chain_row && p.terms_lds <= 65536;
    // a big table: the workgroups of the chain sums do the terms when they run out of sums, with the
    // candidates in LDS beside the table
    if (big && stage_s)
        p.chain_lds += n_s * D;
    if (p.chain_row) {
        if ((long)p.terms_wg + (long)T.n_tables * G.n_mu > kMaxLaunch) return false;
    } else if (chain) {
        p.chain_threads = big ? 1024 : 256;
        const int n_mg = (G.n_mu + 63) / 64;
        // leading blocks that are items of their own: the dense part of a table with many
        // samples, the first blocks of one of which they enter so many intervals that a unit that begins
        // with them is searched for as a whole (100 tables of 150 samples x 3 sizes x 100 process counts
        // up to 8000 56 -> 27 us, one x 1500 sizes x 300 up to 30 000 44 -> 37; 30 samples, 100 tables x 3
        // x 40 up to 20 000 33 and 35), or every block when the whole sum is too small to fill the chip
        // with units of CHAIN_U blocks
        int n_single = T.n > 256 ? 32 : T.n > 64 ? CHAIN_U : 0;
        if ((long)T.n_tables * n_mg * ((G.n_blk + CHAIN_U - 1) / CHAIN_U) < 8 * n_cu) n_single = G.n_blk;
        if (n_single > G.n_blk) n_single = G.n_blk;
        const long items = (long)n_mg * (n_single + (G.n_blk - n_single + CHAIN_U - 1) / CHAIN_U);
        if (items > kMaxLaunch) return false;
        long wg = (big ? n_cu : 4 * n_cu) / T.n_tables;
        const long wg_need = (items + p.chain_threads / 64 - 1) / (p.chain_threads / 64);
        if (wg > wg_need) wg = wg_need;
        if (wg < 1) wg = 1;
        // a small job (the walk would be bound by one lane's latency): every term by a search
        const double n_terms = (double)T.n_tables * G.n_mu * G.n_blk * SUM_BLOCK;
        const bool small = p.together && n_single == G.n_blk && n_terms <= (double)(3L << 20);
        p.both_lds = p.chain_lds > p.terms_lds ? p.chain_lds : p.terms_lds;
        if (small) {
            const size_t small_lds = ((size_t)3 * T.n + 10 + 64 * SMALL_LD) * D;
            if (small_lds > p.both_lds) p.both_lds = small_lds;
            n_single = -1;
            wg = (long)n_mg * G.n_blk;
            // the chain workgroups come first in the grid: they must leave the terms
            // workgroups room on the chip, or those would only start when these are done
            long room = n_cu * (long)(dev.lds_per_cu / (p.both_lds + 512)) - (long)p.terms_wg;
            // (but a workgroup per CU at least: a table of 1000 samples leaves room for two, and terms of
            // 512 workgroups left the chain sums of 10 000 sizes to one: 1230 us, 17 now)
            if (room < n_cu) room = n_cu;
            if (room > 2 * n_cu) room = 2 * n_cu;
            if (wg > room / T.n_tables) wg = room / T.n_tables;
            if (wg < 1) wg = 1;
        }
        p.n_single = n_single;
        p.chain_wg = (int)wg;
        if ((long)T.n_tables * wg + p.terms_wg > kMaxLaunch) return false;
        p.n_chain_wg = (int)(T.n_tables * wg);
        // eight sizes to a workgroup of the prefix, sixteen where the workgroups of eight would not be on the
        // chip at once: their adding waves then use twice the lanes for the same time (100 tables x 1000 sizes x
        // P up to 20 000: the kernel 111 us with eight, 60 so; the call 20 x 3000 224 and 201, 300 x 200 317 and 289)
        p.prefix_m = (long)T.n_tables * ((G.n_mu + 7) / 8) > PFX_WG_PER_CU * n_cu ? 16 : 8;
        p.n_mgroups = (G.n_mu + p.prefix_m - 1) / p.prefix_m;
        if ((long)T.n_tables * p.n_mgroups > kMaxLaunch) return false;
    }
    if (!terms_only) {
        if (lanes_s) {
            // 8 waves per workgroup (two per SIMD, so that two or three workgroups share a CU);
            // as few process counts per wave as let one workgroup cover all of them, if it can
            const int waves = SWEEP_S_WAVES;
            p.sweep_gp = 12;
            for (int gp : {9, 6, 4, 2})
                if (G.n_P <= gp * waves) p.sweep_gp = gp;
            // three workgroups per CU where there are enough of them and their LDS leaves room
            p.sweep_dense = (long)T.n_tables * G.n_m > 2 * n_cu && 3 * sweep_s_lds(G.n_s, true) <= dev.lds_per_cu;
            p.sweep_ptiles = p.sweep_gp == 12 ? (G.n_P + 12 * waves - 1) / (12 * waves) : 1;
            if ((long)T.n_tables * G.n_m * p.sweep_ptiles > kMaxLaunch) return false;
        } else if (lanes_p) {
            // as many waves as the chip holds at four per SIMD, shared out over the tables and
            // the groups of 64 process counts; each walks over every n_w-th message size;
            // two process counts per lane when the grid has at least 512 of them
            const bool all = G.mask == 0x1FFFu;
            p.ppl = G.n_P >= 512 && G.n_s <= 64 && all ? 2 : 1;
            p.n_pg = (G.n_P + 64 * p.ppl - 1) / (64 * p.ppl);
            // (a big job - 6 x 4096 groups of cells - runs best with one size per wave:
            // 33.5 us against 37.8 with six)
            const long wave_budget = (long)T.n_tables * p.n_pg * G.n_m >= 64 * n_cu ? 256 * n_cu * p.ppl : 32 * n_cu;
            long n_w = wave_budget / p.ppl / ((long)T.n_tables * p.n_pg);
            if (n_w > G.n_m) n_w = G.n_m;
            if (n_w < 1) n_w = 1;
            n_w = (n_w + 3) / 4 * 4;
            p.n_w = (int)n_w;
        } else {
            constexpr int PC = 4;
            p.n_mg = (G.n_m + 63) / 64;
            p.n_pcg = (G.n_P + 4 * PC - 1) / (4 * PC);
            if ((long)T.n_tables * p.n_mg * p.n_pcg > kMaxLaunch) return false;
        }
    }
    if (!terms_only && G.extra != 0 && (long)T.n_tables * G.n_m * ((G.n_P + 255) / 256) > kMaxLaunch) return false;
    // scratch: what the kernels of this path index (m-fastest arrays per distinct size where noted)
    const bool binom = (G.need & (1u << 12)) != 0;
    p.lay.g1 = lb.take(D, nt);
    p.lay.gs = lb.take(D, nt, n_s);
    p.lay.gm = lb.take(D, nt, n_m);
    p.lay.sum2 = lb.take(D, binom ? nt : 0, n_m, (size_t)(G.cl_max + 1));
    p.lay.blk = lb.take(D, chain ? nt : 0, (size_t)G.n_blk, n_mu);
    p.lay.part = lb.take(D, chain ? nt : 0, n_mu, n_P);
    p.lay.pre = lb.take(D, chain && G.blk_is_prefix ? nt : 0, n_mu, n_P);
    p.lay.rcp = lb.take(D, n_s);
    p.lay.segC = lb.take(D, pairs ? nt : 0, n_s);
    p.lay.segA = lb.take(D, pairs ? nt : 0, n_m, n_s);
    p.lay.segB = lb.take(D, pairs ? nt : 0, n_m, n_s);
    p.lay.amin = lb.take(D, pairs ? nt : 0, n_m);
    p.lay.minG = lb.take(D, lanes_s && !terms_only ? nt : 0, (n_s + 63) / 64);
    p.lay.nv = lb.take(sizeof(int), n_m);
    if (terms_only)
        p.lay.score_rows = lb.take(D, 13, n_m, 2);
    p.lay.total = lb.at;
    return !lb.too_big;
}

bool plan_tune(const DeviceTables &T, const DeviceGrid &G, bool terms_only, TunePlan &p, size_t most_scratch)
{
    const bool ok = plan_fastest(T, G, terms_only, p);
    if (terms_only || (ok && p.lay.total <= most_scratch))
        return ok;
    // jobs that the staged path is faster for but has no room for: rows and tiles need no scratch
    if (G.extra != 0) {
        if (ok && p.path == TUNE_STAGED && use_row_path(T, G)) {
            p = TunePlan{};
            return plan_rows(T, G, p);
        }
        return ok;
    }
    if (T.n <= TILE_FEW_N)
        return ok;
    const int tile_m = tile_sizes(T, G, false);
    TunePlan tiles = {};
    if (tile_m > 0 && plan_tiles(T, G, tile_m, tiles)) {
        p = tiles;
        return true;
    }
    return ok;
}

hipError_t launch_tune_stage(const TunePlan &p, int stage, const DeviceTables &T, const DeviceGrid &G,
                             const Scratch &S, plogp_cell_dev *d_out, hipStream_t st)
{
    if (p.path == TUNE_TABLE_LANES) {
        if (stage == TUNE_STAGE_TERMS) {
            hipLaunchKernelGGL(k_batch_setup, dim3((unsigned)(p.n_stage + p.prep_wg)), dim3(256), p.setup_lds,
                               st, T, G, S.batch, reinterpret_cast<f64x2 *>(S.batch_ys), p.n_stage);
        } else if (stage == TUNE_STAGE_SWEEP) {
            BatchDims D;
            D.n = T.n; D.n_tables = T.n_tables; D.n_m = G.n_m; D.n_P = G.n_P; D.n_s = G.n_s;
            D.cl_max = G.cl_max; D.n_ops = G.n_ops; D.n_mchunks = p.batch_mchunks; D.m_per_wave = p.m_per_wave;
            D.mask = G.mask;
            D.extra = G.extra;
            const bool all = G.mask == 0x1FFFu, more = G.extra != 0;
            const auto kern = all ? (more ? k_batch_t<BATCH_T_PC, BATCH_T_PS, true, true>
                                          : k_batch_t<BATCH_T_PC, BATCH_T_PS, true, false>)
                                  : (more ? k_batch_t<BATCH_T_PC, BATCH_T_PS, false, true>
                                          : k_batch_t<BATCH_T_PC, BATCH_T_PS, false, false>);
            hipLaunchKernelGGL(kern, dim3((unsigned)p.n_tg * p.batch_mchunks), dim3(64 * BATCH_T_WAVES),
                               p.batch_lds, st, D, reinterpret_cast<const f64x2 *>(S.batch_ys), T.L,
                               S.batch.rec, S.batch.tab, reinterpret_cast<const u64 *>(G.s), d_out);
        }
        return hipGetLastError();
    }
    if (p.path == TUNE_ROW) {
        if (stage == TUNE_STAGE_SWEEP) {
            const bool all = G.mask == 0x1FFFu, two = p.row_two != 0;
            const bool more = G.extra != 0;
            // (all 13 rows and two process counts to a lane: always those that can win alone)
            const auto kern = p.row_few || (all && two)
                                  ? (all ? (two ? (more ? k_row<true, 2, true, true> : k_row<true, 2, false, true>)
                                                : (more ? k_row<true, 1, true, true> : k_row<true, 1, false, true>))
                                         : (two ? (more ? k_row<false, 2, true, true> : k_row<false, 2, false, true>)
                                                : (more ? k_row<false, 1, true, true> : k_row<false, 1, false, true>)))
                              : all ? (more ? k_row<true, 1, true, false> : k_row<true, 1, false, false>)
                                    : (two ? (more ? k_row<false, 2, true, false> : k_row<false, 2, false, false>)
                                           : (more ? k_row<false, 1, true, false> : k_row<false, 1, false, false>));
            hipLaunchKernelGGL(kern, dim3((unsigned)(T.n_tables * G.n_m)), dim3(ROW_THREADS), p.row_lds, st,
                               T, G, d_out);
        }
        return hipGetLastError();
    }
    if (p.path == TUNE_TILE) {
        if (stage == TUNE_STAGE_SWEEP)
            hipLaunchKernelGGL(G.mask == 0x1FFFu ? k_tile<true> : k_tile<false>, dim3((unsigned)T.n_tables * p.n_tiles),
                               dim3(TILE_THREADS), p.tile_lds, st, T, G, d_out, p.n_tiles, p.tile_m,
                               p.tile_shared);
        return hipGetLastError();
    }
    if (stage == TUNE_STAGE_MORE) {
        if (!p.terms_only && G.extra != 0) {
            const int n_pchunks = (G.n_P + 255) / 256;
            hipLaunchKernelGGL(k_more_planes, dim3((unsigned)((long)T.n_tables * G.n_m * n_pchunks)), dim3(256), 0,
                               st, T, G, S, d_out, n_pchunks);
        }
        return hipGetLastError();
    }
    switch (stage) {
    case TUNE_STAGE_TERMS:
        if (!p.chain || (p.chain_row && !p.row_together))      // else they come with the chain sums
            hipLaunchKernelGGL(k_terms, dim3((unsigned)p.terms_wg), dim3(256), p.terms_lds, st, T, G, S,
                               p.n_chunks, p.n_mchunks, p.terms_mode);
        break;
    case TUNE_STAGE_CHAIN:
        if (p.chain_row) {
            if (p.row_together)
                hipLaunchKernelGGL(k_terms_chain_row, dim3((unsigned)(p.terms_wg + T.n_tables * G.n_mu)),
                                   dim3(CROW_THREADS), p.crow_lds > p.terms_lds ? p.crow_lds : p.terms_lds, st,
                                   T, G, S, p.terms_wg, p.n_chunks, p.n_mchunks, p.terms_mode);
            else
                hipLaunchKernelGGL(k_chain_row, dim3((unsigned)(T.n_tables * G.n_mu)), dim3(CROW_THREADS),
                                   p.crow_lds, st, T, G, S);
        } else if (p.chain) {
            if (p.together)
                hipLaunchKernelGGL(p.n_single < 0 ? k_terms_chain<true> : k_terms_chain<false>,
                                   dim3((unsigned)(p.n_chain_wg + p.terms_wg)), dim3(256), p.both_lds, st, T, G, S,
                                   p.n_chain_wg, p.chain_wg, p.n_single, p.n_chunks, p.n_mchunks, p.terms_mode);
            else
                hipLaunchKernelGGL(k_chain_blocks, dim3((unsigned)p.n_chain_wg), dim3(p.chain_threads), p.chain_lds, st,
                                   T, G, S, p.chain_wg, p.n_single, p.terms_mode);
        }
        break;
    case TUNE_STAGE_PREFIX:
        if (p.chain && !p.chain_row && G.blk_is_prefix)
            hipLaunchKernelGGL(p.prefix_m == 16 ? k_chain_prefix<16> : k_chain_prefix<8>, dim3((unsigned)T.n_tables * p.n_mgroups), dim3(PFX_THREADS),
                               pfx_in_lds(G) ? (size_t)G.n_P * sizeof(unsigned short) : 0, st, G, S, p.n_mgroups);
        break;
    default:
        if (p.terms_only)
            break;
        if (p.lanes_s) {
            const unsigned rows = (unsigned)T.n_tables * G.n_m;
            const dim3 threads(64 * SWEEP_S_WAVES);
            const auto kern = sweep_s_kernel(p.sweep_gp, p.sweep_dense != 0);
            hipLaunchKernelGGL(kern, dim3(rows * p.sweep_ptiles), threads, sweep_s_lds(G.n_s, false), st, T, G, S, d_out,
                               p.sweep_ptiles);
        } else if (p.lanes_p) {
            const bool all = G.mask == 0x1FFFu;
            for (int t0 = 0; t0 < T.n_tables; t0 += 65535) {
                const int nt = T.n_tables - t0 < 65535 ? T.n_tables - t0 : 65535;
                const dim3 blocks((unsigned)(p.n_w / 4), (unsigned)p.n_pg, (unsigned)nt);
                const bool few = sweep_few(G, p.ppl);
                const auto kern = G.n_s > 64   ? k_sweep_p<4, false, 1, false>
                                  : !all       ? (few ? k_sweep_p<1, false, 1, true> : k_sweep_p<1, false, 1, false>)
                                  : p.ppl == 2 ? (few ? k_sweep_p<1, true, 2, true> : k_sweep_p<1, true, 2, false>)
                                               : (few ? k_sweep_p<1, true, 1, true> : k_sweep_p<1, true, 1, false>);
                hipLaunchKernelGGL(kern, blocks, dim3(256), 0, st, T, G, S, d_out, t0, p.n_w);
            }
        } else {
            hipLaunchKernelGGL(k_sweep_m<4>, dim3((unsigned)T.n_tables * p.n_mg * p.n_pcg), dim3(256), 0, st, T, G,
                               S, d_out, p.n_mg, p.n_pcg);
        }
        break;
    }
    return hipGetLastError();
}

hipError_t launch_score_stage(int stage, const TunePlan &plan, const DeviceTables &T1, const DeviceGrid &G,
                              const Scratch &S, double *rows, const double *d_meas, const uint32_t *d_seg,
                              double *d_pred, void *d_verdict, void *d_scores, hipStream_t st)
{
    int n_ids = 0;
    for (int id = 0; id < 13; ++id) n_ids += (G.mask >> id) & 1u;
    if (stage == 0)      // g(m), g(1), the Scatter sums: the first stages of the tuning
        return launch_tune(plan, T1, G, S, nullptr, st);
    // With many message sizes a wave takes a whole size and forms the error sums on the way
    // (one pass over the measurements); with fewer there would be too few waves to hide the
    // memory latency of their serial walks, and the points go one to a thread with the sums
    // formed by a second pass.
    const bool fused = G.n_m >= 8 * device_info().n_cu;
    const size_t tab_lds = (G.mask & 0x224u) ? (size_t)3 * T1.n * sizeof(double) : 0;
    // a small table is staged by every workgroup of 256; a big one by as few workgroups of 1024
    // as fill the compute units, which then walk their items with a stride
    const bool big = tab_lds > 16384;
    const int threads = big ? 1024 : 256;
    const DeviceInfo &dev = device_info();
    if (stage == 1 && fused) {
        const int waves = threads / 64;
        const size_t lds = tab_lds + (size_t)waves * SCORE_TILE_ROWS * SCORE_TILE_LD * sizeof(double);
        if (lds > dev.lds_per_cu) return hipErrorInvalidValue;
        long n_wg = ((long)G.n_m + waves - 1) / waves;
        if (big) {
            const long fit = (long)dev.n_cu * (long)(dev.lds_per_cu / lds);
            if (n_wg > fit) n_wg = fit;
        }
        hipLaunchKernelGGL(big ? k_score_fused<true> : k_score_fused<false>, dim3((unsigned)n_wg), dim3(threads),
                           lds, st, T1, G, S, d_meas, d_seg, d_pred,
                           reinterpret_cast<plogp_verdict_dev *>(d_verdict), rows);
        return hipGetLastError();
    }
    if (stage == 1) {
        const int n_pchunks = (G.n_P + threads - 1) / threads;
        const long n_items = (long)G.n_m * n_pchunks;
        long n_wg = n_items;
        if (big) {
            const long fit = (long)dev.n_cu * (long)(dev.lds_per_cu / tab_lds);
            if (n_wg > fit) n_wg = fit;
        }
        if (n_items > kMaxLaunch) return hipErrorInvalidValue;
        hipLaunchKernelGGL(k_score_points, dim3((unsigned)n_wg), dim3(threads), tab_lds, st, T1, G, S, d_meas,
                           d_seg, d_pred, reinterpret_cast<plogp_verdict_dev *>(d_verdict), n_pchunks,
                           (int)n_items);
        return hipGetLastError();
    }
    if (!fused) {
        const long n_rows = (long)n_ids * G.n_m;
        const long row_wg = (n_rows + SCORE_RT * SCORE_WAVES - 1) / (SCORE_RT * SCORE_WAVES);
        hipLaunchKernelGGL(k_score_rows, dim3((unsigned)row_wg), dim3(64 * SCORE_WAVES), 0, st, G, n_ids, d_meas,
                           d_pred, rows);
    }
    // the per-m sums of every strategy added in ascending m
    hipLaunchKernelGGL(k_score_final, dim3((unsigned)n_ids), dim3(1024), 0, st, G, rows,
                       reinterpret_cast<plogp_score_dev *>(d_scores));
    return hipGetLastError();
}

}  // namespace plogp
