// The full gradient of the log (pseudo-)likelihood with respect to eta, for
// every subject, in O(N) (the vector delta - P delta of Sec. 2.9, which a
// proximal-gradient step multiplies by X'; Sec. 2.9 notes the prefix-sum
// form of Sec. 2.7 applies).  With the subjects by decreasing time and d_k
// the events of the tie run ending at k (Breslow):
//
//   S0_k   = prefix(e)_k [+ G(Y_k) * (sum of e w after k's run), Fine-Gray]
//   dl/deta_m = delta_m - e_m * ( sum_{run ends k >= m} d_k / S0_k
//               [+ w_m * sum_{run ends k < m} d_k G(Y_k) / S0_k, Fine-Gray] )
//   l      = sum_m delta_m eta_m - sum_k d_k log S0_k
//
// with w = I(status = 2) / G(y) the competing-event weight.  Three passes over
// tiles of ST sorted positions, tile t the same positions in each of them:
//   k_adj_sums   the tile's sums of e and (Fine-Gray) of e w;
//   k_adj_terms  prefix of e, suffix of e w, S0 and q = d/S0 at run ends, and
//                the tile's sums of l, of q and of q G;
//   k_adj_grad   suffix of q, prefix of q G, and the gradient in sorted order.
// A tile's carry is the sum over the tiles before (after) it: with few tiles
// each workgroup adds them itself, otherwise k_adj_spine scans them once.
// The gradient reaches subject order by one gather through the inverse
// permutation.  Every sum is taken in a fixed order.
//
// Bound: HBM (each pass at the copy rate; 51 B per subject for Cox, 83 for
// Fine-Gray) and, at small N, the launches (5; scans of their own for e w,
// d/S0 and d G/S0 had taken 7 and 13).
#include <math.h>

#include <type_traits>

#include "scan_device.h"
#include "ss_internal.h"

namespace ss {

namespace {

__device__ __forceinline__ bool is_event(int32_t model, int8_t s)
{
    return model == SS_FINE_GRAY ? s == 1 : s != 0;
}

constexpr int kAdjGrid = 2048;  // workgroups of the element-wise passes

// Eight consecutive bytes of a thread's scan items (memory order).
__device__ __forceinline__ void load_bytes8(const uint8_t *p, int64_t k0, int64_t n,
                                            uint8_t (&b)[SI])
{
    if (k0 + SI <= n && ((uintptr_t)(p + k0) & 7u) == 0) {
        const uint2 v = *reinterpret_cast<const uint2 *>(p + k0);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            b[i] = (uint8_t)(v.x >> (8 * i));
            b[4 + i] = (uint8_t)(v.y >> (8 * i));
        }
        return;
    }
#pragma unroll
    for (int i = 0; i < SI; ++i) b[i] = k0 + i < n ? p[k0 + i] : 0;
}

// Fixed-order sum of one value per thread of the workgroup; thread 0 gets it.
__device__ __forceinline__ double block_total(double v, double *s_red)
{
    for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o);
    if ((threadIdx.x & 63) == 0) s_red[threadIdx.x >> 6] = v;
    __syncthreads();
    return ((s_red[0] + s_red[1]) + s_red[2]) + s_red[3];
}

// Inclusive suffix scan of SI items per thread (thread t holds the t-th run
// of SI items of the tile) with the sum of everything after the tile.
__device__ __forceinline__ void block_suffix_scan(double (&it)[SI], double after, double *s_w)
{
    constexpr int NW = SB / kWave;
    const int lane = lane_id();
    const int w = threadIdx.x / kWave;
    double run = 0.0;
#pragma unroll
    for (int i = SI - 1; i >= 0; --i) {
        run += it[i];
        it[i] = run;
    }
    double inc = run;
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) {
        const double y = __shfl_down(inc, off, kWave);
        if (lane + off < kWave) inc += y;
    }
    if (lane == 0) s_w[w] = inc;
    __syncthreads();
    double pre = after;
#pragma unroll
    for (int q = NW - 1; q >= 0; --q)
        if (q > w) pre += s_w[q];
    __syncthreads();
    const double lanes_after = __shfl_down(inc, 1, kWave);
    if (lane < kWave - 1) pre += lanes_after;
#pragma unroll
    for (int i = 0; i < SI; ++i) it[i] += pre;
}

// Carries of the tiles.  Up to kSelfCarry tiles every workgroup adds the
// sums of the tiles before (after) its own; above, k_adj_spine has turned
// the sums into carries and the workgroup reads its own.  (N = 1e6, 489
// tiles: a spine launch costs 4.3 us and the gap before it, the additions
// below 1 us; at 2048 tiles they read 16 MB from L2 over all workgroups.)
constexpr int64_t kSelfCarry = 2048;

template <bool AFTER>
__device__ __forceinline__ double tile_carry(const double *sums, int64_t tiles, double *s_red)
{
    const int64_t t = blockIdx.x;
    if (tiles > kSelfCarry) return sums[t];
    double v = 0.0;
    const int64_t lo = AFTER ? t + 1 : 0, hi = AFTER ? tiles : t;
#pragma unroll 4
    for (int64_t i = lo + threadIdx.x; i < hi; i += SB) v += sums[i];
    v = dpp_wave_sum(v);
    __syncthreads();
    if (lane_id() == 0) s_red[threadIdx.x / kWave] = v;
    __syncthreads();
    double c = 0.0;
#pragma unroll
    for (int q = 0; q < SB / kWave; ++q) c += s_red[q];
    return c;
}

// Exclusive scan of the tile sums in place, one workgroup per array:
// workgroup 0 `fwd` from the first tile, workgroup 1 `bwd` from the last.
constexpr int kSpineBlock = 1024;

__global__ __launch_bounds__(kSpineBlock) void k_adj_spine(int64_t tiles, double *fwd,
                                                           double *bwd)
{
    constexpr int NW = kSpineBlock / kWave;
    constexpr int PT = 8;
    __shared__ double s_w[NW];
    const bool rev = blockIdx.x != 0;
    double *a = rev ? bwd : fwd;
    if (!a) return;
    const int lane = lane_id(), w = threadIdx.x / kWave;
    double carry = 0.0;
    for (int64_t c0 = 0; c0 < tiles; c0 += kSpineBlock * PT) {
        const int64_t base = c0 + (int64_t)threadIdx.x * PT;
        double it[PT], run = 0.0;
#pragma unroll
        for (int i = 0; i < PT; ++i) {
            const int64_t l = base + i;
            it[i] = l < tiles ? a[rev ? tiles - 1 - l : l] : 0.0;
        }
#pragma unroll
        for (int i = 0; i < PT; ++i) {
            const double x = it[i];
            it[i] = run;  // exclusive within the thread
            run += x;
        }
        const double inc = dpp_incl_scan(run);
        if (lane == kWave - 1) s_w[w] = inc;
        __syncthreads();
        double before = carry, all = 0.0;
#pragma unroll
        for (int q = 0; q < NW; ++q) {
            if (q < w) before += s_w[q];
            all += s_w[q];
        }
        // the lanes before this one (not inc - run: it would round)
        const double lanes_before = __shfl_up(inc, 1, kWave);
        if (lane > 0) before += lanes_before;
        carry += all;
        __syncthreads();
#pragma unroll
        for (int i = 0; i < PT; ++i) {
            const int64_t l = base + i;
            if (l < tiles) a[rev ? tiles - 1 - l : l] = before + it[i];
        }
    }
}

template <bool FG>
__global__ __launch_bounds__(SB) void k_adj_sums(int64_t n, const double *e, const double *w_comp,
                                                 double *sum_e, double *sum_ew)
{
    __shared__ double s_red[SB / kWave];
    const int64_t k0 = (int64_t)blockIdx.x * ST + (int64_t)threadIdx.x * SI;
    double ev[SI], wv[FG ? SI : 1];
    load_items<double, OpAdd<double>>(e, k0, n, ev);
    if constexpr (FG) load_items<double, OpAdd<double>>(w_comp, k0, n, wv);
    double a = 0.0, b = 0.0;
#pragma unroll
    for (int i = 0; i < SI; ++i) {
        a += ev[i];
        if constexpr (FG) b += ev[i] * wv[i];
    }
    const double ta = block_total(a, s_red);
    if (threadIdx.x == 0) sum_e[blockIdx.x] = ta;
    if constexpr (FG) {
        __syncthreads();
        const double tb = block_total(b, s_red);
        if (threadIdx.x == 0) sum_ew[blockIdx.x] = tb;
    }
}

// S0 at k is the prefix of e (Fine-Gray: plus G(Y_k) times the e w after
// k); q = d/S0 at run ends, and the tile's sums of delta eta - d log S0, of
// q and (Fine-Gray) of q G.
template <bool FG>
__global__ __launch_bounds__(SB) void k_adj_terms(int64_t n, int64_t tiles, const double *e,
                                                  const double *w_comp, const double *sum_e,
                                                  const double *sum_ew, const int8_t *status_s,
                                                  const double *eta, const uint8_t *d8,
                                                  const int32_t *d32, const double *g_end,
                                                  double *q, double *lpart, double *sum_q,
                                                  double *sum_qg)
{
    static_assert(SB == 4 * kWave, "block_total sums four waves");
    __shared__ double s_w[SB / kWave];
    __shared__ double s_red[SB / kWave];
    const int64_t k0 = (int64_t)blockIdx.x * ST + (int64_t)threadIdx.x * SI;
    double s0[SI], et[SI], r[FG ? SI : 1], gv[FG ? SI : 1];
    load_items<double, OpAdd<double>>(e, k0, n, s0);
    load_items<double, OpAdd<double>>(eta, k0, n, et);
    uint8_t dd[SI], st[SI];
    load_bytes8(d8, k0, n, dd);
    load_bytes8(reinterpret_cast<const uint8_t *>(status_s), k0, n, st);
    if constexpr (FG) {
        load_items<double, OpAdd<double>>(w_comp, k0, n, r);
        load_items<double, OpAdd<double>>(g_end, k0, n, gv);
        const double after = tile_carry<true>(sum_ew, tiles, s_red);
#pragma unroll
        for (int i = 0; i < SI; ++i) r[i] *= s0[i];
        block_suffix_scan(r, after, s_w);
        // the weighted sum starts after the position: one position on
        const double next = __shfl_down(r[0], 1, kWave);
        __shared__ double s_first[SB / kWave];
        if (lane_id() == 0) s_first[threadIdx.x / kWave] = r[0];
        __syncthreads();
        const int w = threadIdx.x / kWave;
        const double past = lane_id() < kWave - 1 ? next
                            : w < SB / kWave - 1  ? s_first[w + 1]
                                                  : after;
#pragma unroll
        for (int i = 0; i < SI - 1; ++i) r[i] = r[i + 1];
        r[SI - 1] = past;
    }
    block_scan<double, OpAdd<double>>(s0, tile_carry<false>(sum_e, tiles, s_red), s_w);
    double qv[SI];
    double lsum = 0.0, qsum = 0.0, qgsum = 0.0;
#pragma unroll
    for (int i = 0; i < SI; ++i) {
        const int64_t k = k0 + i;
        qv[i] = 0.0;
        if (k < n) {
            int d = dd[i];
            if (d == 255) d = d32[k];
            double l = is_event(FG ? SS_FINE_GRAY : SS_COX, (int8_t)st[i]) ? et[i] : 0.0;
            if (d != 0) {
                double S0 = s0[i];
                if constexpr (FG) S0 += gv[i] * r[i];
                qv[i] = (double)d / S0;
                qsum += qv[i];
                if constexpr (FG) qgsum += qv[i] * gv[i];
                l -= (double)d * log(S0);
            }
            lsum += l;
        }
    }
    store_items<double>(q, k0, n, qv);
    __syncthreads();
    const double tl = block_total(lsum, s_red);
    if (threadIdx.x == 0) lpart[blockIdx.x] = tl;
    __syncthreads();
    const double tq = block_total(qsum, s_red);
    if (threadIdx.x == 0) sum_q[blockIdx.x] = tq;
    if constexpr (FG) {
        __syncthreads();
        const double tg = block_total(qgsum, s_red);
        if (threadIdx.x == 0) sum_qg[blockIdx.x] = tg;
    }
}

// R at k is the suffix of q, Q (Fine-Gray) the prefix of q G before k:
// dl/deta_k = delta_k - e_k (R + w_k Q) goes to grad_s in sorted order.
// Workgroup 0 also adds the likelihood partials in order.
template <bool FG>
__global__ __launch_bounds__(SB) void k_adj_grad(int64_t n, int64_t tiles, const double *q,
                                                 const double *sum_q, const double *sum_qg,
                                                 const int8_t *status_s, const double *e,
                                                 const double *w_comp, const double *g_end,
                                                 const double *lpart, double *grad_s,
                                                 double *loglik)
{
    __shared__ double s_w[SB / kWave];
    __shared__ double s_red[SB / kWave];
    __shared__ double s_last[SB / kWave];
    const int64_t k0 = (int64_t)blockIdx.x * ST + (int64_t)threadIdx.x * SI;
    double r[SI], ev[SI], qg[FG ? SI : 1], wv[FG ? SI : 1];
    load_items<double, OpAdd<double>>(q, k0, n, r);
    load_items<double, OpAdd<double>>(e, k0, n, ev);
    uint8_t st[SI];
    load_bytes8(reinterpret_cast<const uint8_t *>(status_s), k0, n, st);
    if constexpr (FG) {
        load_items<double, OpAdd<double>>(g_end, k0, n, qg);
        load_items<double, OpAdd<double>>(w_comp, k0, n, wv);
#pragma unroll
        for (int i = 0; i < SI; ++i) qg[i] *= r[i];
        const double before = tile_carry<false>(sum_qg, tiles, s_red);
        block_scan<double, OpAdd<double>>(qg, before, s_w);
        inclusive_to_exclusive<double>(qg, before, s_last);
    }
    block_suffix_scan(r, tile_carry<true>(sum_q, tiles, s_red), s_w);
    double gv[SI];
#pragma unroll
    for (int i = 0; i < SI; ++i) {
        double inner = r[i];
        if constexpr (FG) inner += wv[i] * qg[i];
        gv[i] = (is_event(FG ? SS_FINE_GRAY : SS_COX, (int8_t)st[i]) ? 1.0 : 0.0) - ev[i] * inner;
    }
    store_items<double>(grad_s, k0, n, gv);
    if (blockIdx.x == 0) {
        double v = 0.0;
        for (int64_t b = threadIdx.x; b < tiles; b += SB) v += lpart[b];
        __syncthreads();
        const double t = block_total(v, s_red);
        if (threadIdx.x == 0) *loglik = t;
    }
}

// Subject order: a gather through the inverse permutation (random reads
// cost less than random partial-line writes).
__global__ __launch_bounds__(256) void k_adj_to_subjects(int64_t n, const int32_t *inv_perm,
                                                         const double *grad_s, double *grad)
{
    for (int64_t i = blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256)
        grad[i] = grad_s[inv_perm[i]];
}

// X' g over the sorted-position CSC design, cut along the positions into
// spans of kspan chunks (kspan * SS_CHUNK positions): one wave sums column
// j's non-zeros inside span c, found through the chunk index, into
// part[j * nspan + c].  A wave's unit is (span, column group); the waves of
// one span sit next to each other in launch order, so the stretch of g a
// span gathers from stays in L2 while its columns are summed.  Every sum is
// in a fixed order (four interleaved accumulators, then the wave), so the
// result is deterministic.
constexpr int kXtWaves = 4;

__global__ __launch_bounds__(256) void k_xt_span(int64_t p, int64_t nspan, int64_t kspan,
                                                 int64_t nchunk, int64_t groups,
                                                 const int64_t *col_ptr,
                                                 const int32_t *chunk_ptr,
                                                 const int32_t *rows_sorted,
                                                 const double *vals_sorted, const double *g,
                                                 double *part)
{
    const int lane = threadIdx.x & (kWave - 1);
    const int64_t unit = (int64_t)blockIdx.x * kXtWaves + (threadIdx.x >> 6);
    if (unit >= nspan * groups) return;  // the whole wave
    const int64_t c = unit / groups;
    const int64_t t0 = c * kspan, t1 = min(t0 + kspan, nchunk);
    for (int64_t j = unit - c * groups; j < p; j += groups) {
        const int32_t *cp = chunk_ptr + j * (nchunk + 1);
        const int64_t base = col_ptr[j];
        const int64_t hi = base + cp[t1];
        int64_t q = base + cp[t0] + lane;
        double a0 = 0.0, a1 = 0.0, a2 = 0.0, a3 = 0.0;
        if (vals_sorted) {
            for (; q + 3 * kWave < hi; q += 4 * kWave) {
                a0 += vals_sorted[q] * g[rows_sorted[q]];
                a1 += vals_sorted[q + kWave] * g[rows_sorted[q + kWave]];
                a2 += vals_sorted[q + 2 * kWave] * g[rows_sorted[q + 2 * kWave]];
                a3 += vals_sorted[q + 3 * kWave] * g[rows_sorted[q + 3 * kWave]];
            }
            for (; q < hi; q += kWave) a0 += vals_sorted[q] * g[rows_sorted[q]];
        } else {
            for (; q + 3 * kWave < hi; q += 4 * kWave) {
                a0 += g[rows_sorted[q]];
                a1 += g[rows_sorted[q + kWave]];
                a2 += g[rows_sorted[q + 2 * kWave]];
                a3 += g[rows_sorted[q + 3 * kWave]];
            }
            for (; q < hi; q += kWave) a0 += g[rows_sorted[q]];
        }
        const double v = dpp_wave_sum((a0 + a1) + (a2 + a3));
        if (lane == 0) part[j * nspan + c] = v;
    }
}

// The same for larger designs: a workgroup keeps a span of g in LDS (kXtSpan
// positions at a time where the span is longer) and its waves sum the pieces
// of a group of columns from there.  A random 8-byte read takes a cache
// line's worth of L2 bandwidth, which bounded the gather (N = 1e6, P = 1000,
// 5e7 non-zeros: 194 us); from LDS it costs a bank access and the row indices
// stream from HBM (43 us, 4.6 TB/s).  A wave takes the bounds of its columns
// in one set of loads, and loads a column's first kXtAhead * 64 row indices
// while it sums the column before.  Short pieces would leave most of those
// lanes and loads idle: batches of them put several columns in flight at once
// (up to 128 entries) or give each lane a column (up to kXtFew); in long
// spans, which wide designs get, short columns are gathered from L2 at once.
//
// The line between the two, whole beta gradients, us from L2 / from LDS: 5%
// density N = 1e6, P = 16 40 / 32, P = 256 69.8 / 40.9; N = 1e5, P = 512 25.4 /
// 25.3 (valued 28.3 / 29), P = 1024 32.7 / 27.8 (37.8 / 33.6), P = 2048 50.5 /
// 32.5; 100 non-zeros a column N = 1e6, P = 2000 70 / 36; N = 1000, P = 1e5,
// 5% 91 / 78.  Below 16 columns a span loaded is hardly read; with 16 columns
// of 100 non-zeros N = 2e7 281 / 287.
constexpr int kXtBlock = 512;
constexpr int kXtSpan = 8192;
constexpr int kXtAhead = 8;
constexpr int kXtFew = 8;  // entries of a piece that a lane sums by itself
constexpr int64_t kXtLdsCols = 16;
constexpr int64_t kXtLdsSize = 100'000'000;  // positions times columns

template <bool VALS>
__global__ __launch_bounds__(kXtBlock) void k_xt_lds(int64_t n, int64_t p, int64_t nspan,
                                                     int64_t kspan, int64_t nchunk, int64_t groups,
                                                     int64_t group_cols, const int64_t *col_ptr,
                                                     const int32_t *chunk_ptr,
                                                     const int32_t *rows_sorted,
                                                     const double *vals_sorted, const double *g,
                                                     double *part)
{
    constexpr int NW = kXtBlock / kWave;
    constexpr int kSub = kXtSpan / SS_CHUNK;  // chunks held at a time
    __shared__ double s_g[kXtSpan + 1];
    __shared__ double s_t[NW][kXtAhead];
    const int lane = lane_id();
    const int w = threadIdx.x / kWave;
    const int64_t c = blockIdx.x / groups;
    const int64_t j0 = (blockIdx.x - c * groups) * group_cols;
    const int64_t j1 = min(j0 + group_cols, p);
    const int64_t t_end = min((c + 1) * kspan, nchunk);
    // columns of this wave: a contiguous share of the group's
    const int64_t share = (group_cols + NW - 1) / NW;
    const int64_t ja = min(j0 + w * share, j1), jz = min(ja + share, j1);
    // a batch of up to 64 columns from jb on: column jb + x has its piece
    // [lo, lo + len) between chunks ta and tb in lane x, which also adds its
    // sum to part
    int64_t lo = 0;
    int32_t len = 0;
    auto batch = [&](int64_t jb, int m, int64_t ta, int64_t tb) {
        lo = 0;
        len = 0;
        if (lane < m) {
            const int32_t *cp = chunk_ptr + (jb + lane) * (nchunk + 1);
            const int32_t a = cp[ta], b = cp[tb];
            lo = col_ptr[jb + lane] + a;
            len = b - a;
        }
    };
    // piece x of the batch: entries [at, at + l)
    auto bounds = [&](int x, int64_t &at, int32_t &l) {
        const uint32_t l0 = __builtin_amdgcn_readlane((int)(lo & 0xffffffff), x);
        const uint32_t l1 = __builtin_amdgcn_readlane((int)(lo >> 32), x);
        at = (int64_t)(((uint64_t)l1 << 32) | l0);
        l = __builtin_amdgcn_readlane(len, x);
    };
    auto put = [&](int64_t jb, bool first, double t) {
        double *dst = part + (jb + lane) * nspan + c;
        *dst = first ? t : *dst + t;
    };
    // Batches of short pieces; get(in, r): the gradient at row r, 0 if !in
    // (an entry past the end reads the design's first).  True: all done.
    auto short_pieces = [&](int64_t jb, int m, bool first, int32_t most, auto get) -> bool {
        if (__any(len > most)) return false;
        // a lane for each column
        if (!__any(len > kXtFew)) {
            double acc = 0.0;
            for (int32_t i0 = 0; __any(i0 < len); i0 += kXtFew / 2) {
                int32_t r[kXtFew / 2];
                double v[VALS ? kXtFew / 2 : 1];
#pragma unroll
                for (int i = 0; i < kXtFew / 2; ++i) {
                    const int64_t o = i0 + i < len ? lo + i0 + i : 0;
                    r[i] = rows_sorted[o];
                    if constexpr (VALS) v[i] = vals_sorted[o];
                }
#pragma unroll
                for (int i = 0; i < kXtFew / 2; ++i) {
                    const double gv = get(i0 + i < len, r[i]);
                    if constexpr (VALS) acc += i0 + i < len ? v[i] * gv : 0.0;
                    else acc += gv;
                }
            }
            if (lane < m) put(jb, first, acc);
            return true;
        }
        // kXtAhead loads in flight over several columns, D for each
        auto several = [&](auto depth) {
            constexpr int D = decltype(depth)::value, C = kXtAhead / D;
            for (int x0 = 0; x0 < m; x0 += C) {
                int32_t r[kXtAhead], left[kXtAhead];
                double v[VALS ? kXtAhead : 1], acc[C];
#pragma unroll
                for (int u = 0; u < kXtAhead; ++u) {
                    int64_t at;
                    int32_t l;
                    bounds(min(x0 + u / D, kWave - 1), at, l);  // (none past m)
                    left[u] = l - u % D * kWave;
                    const int64_t o = lane < left[u] ? at + u % D * kWave + lane : 0;
                    r[u] = rows_sorted[o];
                    if constexpr (VALS) v[u] = vals_sorted[o];
                }
#pragma unroll
                for (int u = 0; u < kXtAhead; ++u) {
                    double gv = get(lane < left[u], r[u]);
                    if constexpr (VALS) gv = lane < left[u] ? v[u] * gv : 0.0;
                    acc[u / D] = u % D == 0 ? gv : acc[u / D] + gv;
                }
                wave_sums_to<C>(acc, s_t[w]);
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                if (lane >= x0 && lane < min(x0 + C, m)) put(jb, first, s_t[w][lane - x0]);
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            }
        };
        if (!__any(len > kWave)) several(std::integral_constant<int, 1>{});
        else several(std::integral_constant<int, 2>{});
        return true;
    };
    // A span of several stretches: batches with up to 128 entries a column in
    // all of it gather from L2, at once.
    uint64_t direct = 0;  // the wave's batches (the first 64) that did
    if (kspan > kSub) {
        bool all = jz - ja <= 64 * kWave;
        int64_t q = 0;
        for (int64_t jb = ja; jb < jz && q < 64; jb += kWave, ++q) {
            const int m = (int)min((int64_t)kWave, jz - jb);
            batch(jb, m, c * kspan, t_end);
            const bool done = short_pieces(jb, m, true, 2 * kWave, [&](bool in, int32_t row) {
                const double x = g[row];
                return in ? x : 0.0;
            });
            if (done) direct |= 1ull << q;
            all = all && done;
        }
        if (__syncthreads_and(all)) return;
    }
    for (int64_t t0 = c * kspan; t0 < t_end; t0 += kSub) {
        const int64_t t1 = min(t0 + kSub, t_end);
        const int64_t k0 = t0 * SS_CHUNK;
        const int32_t cnt = (int32_t)(min(t1 * SS_CHUNK, n) - k0);
        const bool first = t0 == c * kspan;
        __syncthreads();
        for (int32_t i = threadIdx.x; i < cnt; i += kXtBlock) s_g[i] = g[k0 + i];
        if (threadIdx.x == 0) s_g[kXtSpan] = 0.0;
        __syncthreads();
        int64_t q = 0;
        for (int64_t jb = ja; jb < jz; jb += kWave, ++q) {
            if (q < 64 && (direct >> q) & 1u) continue;
            const int m = (int)min((int64_t)kWave, jz - jb);
            batch(jb, m, t0, t1);
            if (short_pieces(jb, m, first, 2 * kWave, [&](bool in, int32_t row) {
                    return s_g[in ? row - (int32_t)k0 : kXtSpan];
                }))
                continue;
            // entries o .. of a piece (the last one again past the end; of an
            // empty one the design's first)
            auto load = [&](int64_t at, int32_t l, int32_t o, int32_t (&r)[kXtAhead],
                            double (&v)[VALS ? kXtAhead : 1]) {
                const int32_t *rp = rows_sorted + (l > 0 ? at : 0);
                const double *vp = VALS ? vals_sorted + (l > 0 ? at : 0) : nullptr;
#pragma unroll
                for (int u = 0; u < kXtAhead; ++u) {
                    const uint32_t i = (uint32_t)min(o + u * kWave + lane, max(l - 1, 0));
                    r[u] = rp[i];
                    if constexpr (VALS) v[u] = vp[i];
                }
            };
            int64_t at;
            int32_t l;
            bounds(0, at, l);
            int32_t r[kXtAhead];
            double v[VALS ? kXtAhead : 1];
            load(at, l, 0, r, v);
            for (int x = 0; x < m; ++x) {
                double acc[4] = {0.0, 0.0, 0.0, 0.0};
                // (an entry past the end reads the 0 after the span)
                auto take = [&](int32_t left) {
                    double gv[kXtAhead];
#pragma unroll
                    for (int u = 0; u < kXtAhead; ++u)
                        gv[u] = s_g[u * kWave + lane < left ? r[u] - (int32_t)k0 : kXtSpan];
#pragma unroll
                    for (int u = 0; u < kXtAhead; ++u) {
                        if constexpr (VALS)
                            acc[u & 3] += u * kWave + lane < left ? v[u] * gv[u] : 0.0;
                        else
                            acc[u & 3] += gv[u];
                    }
                };
                const int64_t at0 = at;
                int32_t done = 0;
                const int32_t l0 = l;
                for (int32_t o = kXtAhead * kWave; o < l0; o += kXtAhead * kWave) {
                    int32_t r2[kXtAhead];
                    double v2[VALS ? kXtAhead : 1];
                    load(at0, l0, o, r2, v2);
                    take(l0 - done);
                    done = o;
#pragma unroll
                    for (int u = 0; u < kXtAhead; ++u) {
                        r[u] = r2[u];
                        if constexpr (VALS) v[u] = v2[u];
                    }
                }
                int32_t r2[kXtAhead];
                double v2[VALS ? kXtAhead : 1];
                bounds(min(x + 1, m - 1), at, l);
                load(at, l, 0, r2, v2);
                take(l0 - done);
                const double t = dpp_wave_sum((acc[0] + acc[1]) + (acc[2] + acc[3]));
                if (lane == x) put(jb, first, t);
#pragma unroll
                for (int u = 0; u < kXtAhead; ++u) {
                    r[u] = r2[u];
                    if constexpr (VALS) v[u] = v2[u];
                }
            }
        }
    }
}

// grad_beta[j] = the sum of column j's span partials, one workgroup per
// column: four interleaved accumulators per thread, then the workgroup's
// fixed-order sum.
__global__ __launch_bounds__(256) void k_xt_cols(int64_t nspan, const double *part, double *out)
{
    __shared__ double s_red[4];
    const double *pj = part + (int64_t)blockIdx.x * nspan;
    double a0 = 0.0, a1 = 0.0, a2 = 0.0, a3 = 0.0;
    int64_t c = threadIdx.x;
    for (; c + 768 < nspan; c += 1024) {
        a0 += pj[c];
        a1 += pj[c + 256];
        a2 += pj[c + 512];
        a3 += pj[c + 768];
    }
    for (; c < nspan; c += 256) a0 += pj[c];
    const double t = block_total((a0 + a1) + (a2 + a3), s_red);
    if (threadIdx.x == 0) out[blockIdx.x] = t;
}

struct AdjWs {
    double *a, *q, *lpart;                   // the gradient in sorted order, d/S0
    double *sum_e, *sum_ew, *sum_q, *sum_qg; // per tile: sums, then carries
};

size_t adj_layout(int64_t n, void *ws, AdjWs *w)
{
    char *p = (char *)ws;
    size_t off = 0;
    auto take = [&](size_t bytes) {
        void *r = p ? p + off : nullptr;
        off = align_up(off + bytes, 256);
        return r;
    };
    const size_t tiles = (size_t)ceil_div(n, ST);
    AdjWs t;
    t.a = (double *)take(8 * (size_t)n);
    t.q = (double *)take(8 * (size_t)n);
    (void)take(16 * (size_t)n);  // the interface promises a size of four N-vectors
    t.lpart = (double *)take(8 * tiles);
    t.sum_e = (double *)take(8 * tiles);
    t.sum_ew = (double *)take(8 * tiles);
    t.sum_q = (double *)take(8 * tiles);
    t.sum_qg = (double *)take(8 * tiles);
    if (w) *w = t;
    return off;
}

int grid_of(int64_t n) { return (int)std::min<int64_t>(kAdjGrid, ceil_div(n, 256)); }

__global__ __launch_bounds__(256) void k_gather_u8(int64_t n, const int32_t *perm,
                                                   const uint8_t *src, uint8_t *dst)
{
    for (int64_t k = blockIdx.x * 256 + threadIdx.x; k < n; k += (int64_t)gridDim.x * 256)
        dst[k] = src[perm[k]];
}

}  // namespace

int32_t launch_gather_u8(int64_t n, const int32_t *perm, const uint8_t *src, uint8_t *dst,
                         hipStream_t s)
{
    hipLaunchKernelGGL(k_gather_u8, dim3(grid_of(n)), dim3(256), 0, s, n, perm, src, dst);
    SS_LAUNCH_CHECK();
    return SS_OK;
}

size_t adjoint_ws_bytes(int64_t n) { return adj_layout(n, nullptr, nullptr); }

// The gradient in eta in sorted order into w.a (and l into *loglik).
template <bool FG>
static int32_t eta_gradient_passes(int64_t n, const int8_t *status_s, const double *eta,
                                   const double *e, const uint8_t *d8, const int32_t *d32,
                                   const double *w_comp, const double *g_end, double *loglik,
                                   const AdjWs &w, hipStream_t s)
{
    const int64_t tiles = ceil_div(n, (int64_t)ST);
    const dim3 grid((unsigned)tiles);
    hipLaunchKernelGGL(k_adj_sums<FG>, grid, dim3(SB), 0, s, n, e, w_comp, w.sum_e, w.sum_ew);
    SS_LAUNCH_CHECK();
    if (tiles > kSelfCarry) {
        hipLaunchKernelGGL(k_adj_spine, dim3(FG ? 2 : 1), dim3(kSpineBlock), 0, s, tiles, w.sum_e,
                           w.sum_ew);
        SS_LAUNCH_CHECK();
    }
    hipLaunchKernelGGL(k_adj_terms<FG>, grid, dim3(SB), 0, s, n, tiles, e, w_comp, w.sum_e,
                       w.sum_ew, status_s, eta, d8, d32, g_end, w.q, w.lpart, w.sum_q, w.sum_qg);
    SS_LAUNCH_CHECK();
    if (tiles > kSelfCarry) {
        hipLaunchKernelGGL(k_adj_spine, dim3(2), dim3(kSpineBlock), 0, s, tiles,
                           FG ? w.sum_qg : (double *)nullptr, w.sum_q);
        SS_LAUNCH_CHECK();
    }
    hipLaunchKernelGGL(k_adj_grad<FG>, grid, dim3(SB), 0, s, n, tiles, w.q, w.sum_q, w.sum_qg,
                       status_s, e, w_comp, g_end, w.lpart, w.a, loglik);
    SS_LAUNCH_CHECK();
    return SS_OK;
}

static int32_t eta_gradient_sorted(int32_t model, int64_t n, const int8_t *status_s,
                                   const double *eta, const double *e, const uint8_t *d8,
                                   const int32_t *d32, const double *w_comp,
                                   const double *g_end, double *loglik, const AdjWs &w,
                                   hipStream_t s)
{
    return model == SS_FINE_GRAY
               ? eta_gradient_passes<true>(n, status_s, eta, e, d8, d32, w_comp, g_end, loglik, w, s)
               : eta_gradient_passes<false>(n, status_s, eta, e, d8, d32, w_comp, g_end, loglik, w,
                                            s);
}

int32_t launch_eta_gradient(int32_t model, int64_t n, const int32_t *inv_perm,
                            const int8_t *status_s, const double *eta, const double *e,
                            const uint8_t *d8, const int32_t *d32, const double *w_comp,
                            const double *g_end, double *grad, double *loglik, void *ws,
                            hipStream_t s)
{
    AdjWs w;
    adj_layout(n, ws, &w);
    const int32_t rc = eta_gradient_sorted(model, n, status_s, eta, e, d8, d32, w_comp, g_end,
                                           loglik, w, s);
    if (rc) return rc;
    hipLaunchKernelGGL(k_adj_to_subjects, dim3(grid_of(n)), dim3(256), 0, s, n, inv_perm, w.a,
                       grad);
    SS_LAUNCH_CHECK();
    return SS_OK;
}

// Span length (in chunks) of the X' pass: 8 chunks (8192 positions), longer
// where p * spans would pass 2 (n + p) partials (designs much wider than
// long), which bounds the workspace.
int64_t xt_span_chunks(int64_t n, int64_t p)
{
    const int64_t nchunk = ceil_div(n, (int64_t)SS_CHUNK);
    int64_t k = 8;
    while (k < nchunk && p * ceil_div(nchunk, k) > 2 * (n + p)) k *= 2;
    return k;
}

// Columns per workgroup of k_xt_lds: the fewest groups that fill at least
// 90% of the workgroup slots (two per CU) over the rounds they take, else the
// fullest; at least 16 columns for each span loaded.  (N = 1e6, P = 1000,
// 123 spans: 4 groups are one round of 492 workgroups; 9 groups, 2.2 rounds,
// took 155 us.  N = 1000, P = 1e5, one span: 461 groups 78 us, 64 groups, as a
// limit once had it, 205.)
int64_t xt_group_cols(int64_t p, int64_t nspan)
{
    constexpr int64_t slots = 2 * 256;
    int64_t best = 1;
    double full = 0.0;
    for (int64_t g = 1; g <= std::min<int64_t>(p / 16, slots); ++g) {
        const int64_t wgs = nspan * g;
        const double f = (double)wgs / (double)(slots * ceil_div(wgs, slots));
        if (f > full) {
            full = f;
            best = g;
        }
        if (full >= 0.9) break;
    }
    return ceil_div(p, best);
}

size_t beta_ws_bytes(int64_t n, int64_t p)
{
    const int64_t nspan = ceil_div(ceil_div(n, (int64_t)SS_CHUNK), xt_span_chunks(n, p));
    return adjoint_ws_bytes(n) + align_up(8 * (size_t)p * (size_t)nspan, 256);
}

int32_t launch_beta_gradient(int32_t model, int64_t n, int64_t p, const int32_t *inv_perm,
                             const int8_t *status_s, const double *eta, const double *e,
                             const uint8_t *d8, const int32_t *d32, const double *w_comp,
                             const double *g_end, const int64_t *col_ptr,
                             const int32_t *rows_sorted, const double *vals_sorted,
                             const int32_t *chunk_ptr, double *grad_beta, double *grad_eta,
                             double *loglik, void *ws, hipStream_t s)
{
    AdjWs w;
    adj_layout(n, ws, &w);
    int32_t rc = eta_gradient_sorted(model, n, status_s, eta, e, d8, d32, w_comp, g_end, loglik,
                                     w, s);
    if (rc) return rc;
    const int64_t nchunk = ceil_div(n, (int64_t)SS_CHUNK);
    const int64_t kspan = xt_span_chunks(n, p);
    const int64_t nspan = ceil_div(nchunk, kspan);
    double *part = reinterpret_cast<double *>(static_cast<char *>(ws) + adjoint_ws_bytes(n));
    if (p >= kXtLdsCols && p >= ceil_div(kXtLdsSize, n)) {
        const int64_t cols = xt_group_cols(p, nspan), groups = ceil_div(p, cols);
        if (vals_sorted)
            hipLaunchKernelGGL(k_xt_lds<true>, dim3((unsigned)(nspan * groups)), dim3(kXtBlock), 0,
                               s, n, p, nspan, kspan, nchunk, groups, cols, col_ptr, chunk_ptr,
                               rows_sorted, vals_sorted, w.a, part);
        else
            hipLaunchKernelGGL(k_xt_lds<false>, dim3((unsigned)(nspan * groups)), dim3(kXtBlock),
                               0, s, n, p, nspan, kspan, nchunk, groups, cols, col_ptr, chunk_ptr,
                               rows_sorted, vals_sorted, w.a, part);
    } else {
        // about 16K waves when the design allows: column groups per span
        const int64_t groups = std::max<int64_t>(1, std::min<int64_t>(p, ceil_div(16384, nspan)));
        hipLaunchKernelGGL(k_xt_span, dim3((unsigned)ceil_div(nspan * groups, kXtWaves)),
                           dim3(256), 0, s, p, nspan, kspan, nchunk, groups, col_ptr, chunk_ptr,
                           rows_sorted, vals_sorted, w.a, part);
    }
    SS_LAUNCH_CHECK();
    hipLaunchKernelGGL(k_xt_cols, dim3((unsigned)p), dim3(256), 0, s, nspan, part, grad_beta);
    SS_LAUNCH_CHECK();
    if (grad_eta) {
        hipLaunchKernelGGL(k_adj_to_subjects, dim3(grid_of(n)), dim3(256), 0, s, n, inv_perm,
                           w.a, grad_eta);
        SS_LAUNCH_CHECK();
    }
    return SS_OK;
}

}  // namespace ss
