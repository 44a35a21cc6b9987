// Persistent cyclic-coordinate-descent sweep for gfx950: the workflow of
// Fig. 3 (sparse update -> fused gradient/Hessian -> conditional update,
// for j = 1..P) in ONE cooperative launch, with no host round trip and no
// per-coordinate launch.
//
// Every workgroup owns a segment of S = BLOCK*IPT consecutive sorted
// positions for the whole sweep; e (and, for Fine-Gray, w and G) of its
// segment stay on chip, and only the rows that an update touches are
// patched.  Per coordinate the workgroups exchange the tuple aggregates of
// their segments (Sec. 2.7), from which each takes its exclusive prefix and,
// for Fine-Gray, the weighted suffix sum (eq. fg_g), and their partial sums
// of d*G, d*(H - G^2), d*log S0, from which comes the coordinate update
// (Secs. 2.3-2.4) -- in a fixed order, so results are deterministic:
//   k_sweep1        0/1 designs, both in one all-to-all exchange;
//   k_sweep_valued  valued designs, two all-to-all exchanges;
//   k_sweep         valued Cox designs of over 2^20 positions, whose segments
//                   of 8192 leave no LDS for eta: two exchanges through
//                   workgroup 0, which scans the aggregates in segment order
//                   and hands out prefixes, adds the partials, takes the
//                   update and broadcasts the step.
// Every exchanged value travels under an epoch tag in 16-byte words with one
// agent-scope access each (no L2 flush or invalidate, no separate flag), so
// nothing is cleared between steps and O(segments) values move per
// exchange.
// Every wait is bounded; a timed-out wait sets the workspace error word and
// every workgroup leaves at its next wait.
#include "exchange.h"

namespace ss {

namespace {

using namespace dev;

// Phase timestamps of the first 8 coordinates per workgroup, for
// performance-analysis builds only (-DSS_TRACE_TIMES).
#ifdef SS_TRACE_TIMES
#define SW_TRACE(a, b, jj, slot)                                                    \
    do {                                                                            \
        if (threadIdx.x == 0 && (jj) - (a).j_begin < 8)                             \
            trace_base((a).ws)                                                      \
                [((b) * 8 + ((jj) - (a).j_begin)) * 8 + (slot)] =                   \
                __builtin_amdgcn_s_memrealtime();                                   \
    } while (0)
#else
#define SW_TRACE(a, b, jj, slot) do { } while (0)
#endif

// Positions per group of the branch-free transform of k_sweep1.
#ifndef SS_SW_GROUP
#define SS_SW_GROUP 8
#endif
constexpr int kSwGroup = SS_SW_GROUP;
#ifndef SS_SW_FG_GROUP
#define SS_SW_FG_GROUP 4
#endif
constexpr int kSwFgGroup = SS_SW_FG_GROUP;  // the same for Fine-Gray

struct SweepArgs {
    int64_t n;
    int32_t j_begin;
    int32_t j_end;
    int32_t nblk;
    double *eta;
    double *e;
    const uint8_t *d8;
    const int32_t *d32;
    const double *w_comp;
    const double *g_end;
    Column col;
    const double *c;
    double *beta;
    double *delta;
    double *steps;
    double *g12_out;
    int32_t penalty;
    double lambda;
    int32_t want_log;
    WsView ws;
};

// Applies `st` times column jc to eta and e inside the segment; with LDS
// (s_ep, s_flag) also patches the registers of the owners.
template <int BLOCK, bool PATCH_LDS>
__device__ __forceinline__ void apply_step(const SweepArgs &a, int32_t jc, double st,
                                           int64_t seg0, int64_t chunk0, int64_t chunk1,
                                           double *s_ep, uint8_t *s_flag)
{
    const ColTile cp = col_tile(a.col, jc, chunk0, chunk1);
    for (int32_t o = cp.lo + (int32_t)threadIdx.x; o < cp.hi; o += BLOCK) {
        const int32_t k = a.col.rows[cp.cb + o];
        const double x = a.col.vals[cp.cb + o];
        const double et = a.eta[k] + x * st;
        const double en = exp(et);
        a.eta[k] = et;
        a.e[k] = en;
        if (PATCH_LDS) {
            s_ep[k - seg0] = en;
            lds_flag_or(s_flag, (int32_t)(k - seg0), kFlagPatch);
        }
    }
}


template <int BLOCK, int IPT>
__global__ __launch_bounds__(BLOCK) void k_sweep(SweepArgs a)
{
    constexpr int S = BLOCK * IPT;
    constexpr int NC = 3;
    constexpr int NW = BLOCK / kWave;
    static_assert(S % SS_CHUNK == 0, "segment must be whole chunks");

    __shared__ __attribute__((aligned(16))) uint8_t s_flag[S];
    __shared__ double s_xv[S];
    __shared__ double s_ep[S];
    __shared__ double s_wsum[NW][NC];
    __shared__ double s_wred[NW][3];
    __shared__ double s_bc[NC];
    __shared__ uint64_t s_ep0;
    __shared__ double s_step;
    __shared__ int s_abort;

    const int tid = threadIdx.x;
    const int lane = lane_id();
    const int w = tid / kWave;
    const int64_t b = blockIdx.x;
    const int G = a.nblk;
    WsHeader *hdr = a.ws.hdr;
    const int64_t seg0 = b * S;
    const int64_t cnt = min((int64_t)S, a.n - seg0);
    const int64_t nchunk = a.col.nchunk1 - 1;
    const int64_t chunk0 = seg0 / SS_CHUNK;
    const int64_t chunk1 = min(chunk0 + S / SS_CHUNK, nchunk);
    const int64_t base = seg0 + (int64_t)tid * IPT;

    if (tid == 0) {
        s_ep0 = ld_relaxed_u64(&hdr->epoch);
        s_abort = 0;
    }

    // ---- the segment's data, kept for the whole sweep
    double ev[IPT];
    int dk[IPT];
    if (cnt == S) {
        const double2 *ep = reinterpret_cast<const double2 *>(a.e + base);
#pragma unroll
        for (int q = 0; q < IPT / 2; ++q) {
            const double2 v = ep[q];
            ev[2 * q] = v.x;
            ev[2 * q + 1] = v.y;
        }
    } else {
#pragma unroll
        for (int i = 0; i < IPT; ++i) {
            const bool ok = base + i < a.n;
            ev[i] = ok ? a.e[base + i] : 0.0;
        }
    }
#pragma unroll
    for (int i = 0; i < IPT; ++i) {
        const int64_t k = base + i;
        const bool ok = k < a.n;
        int d = ok ? (int)a.d8[k] : 0;
        if (d == 255) d = a.d32[k];
        dk[i] = d;
    }
    __syncthreads();
    const uint64_t ep0 = s_ep0;

    for (int32_t j = a.j_begin; j < a.j_end; ++j) {
        const uint64_t ep = ep0 + (uint64_t)(j - a.j_begin);
        const uint64_t tag = (ep << 1) | 1u;
        SW_TRACE(a, b, j, 0);

        // ---- column j and the pending step of column j-1 into LDS
        {
            uint32_t *f32 = reinterpret_cast<uint32_t *>(s_flag);
            for (int i = tid; i < S / 4; i += BLOCK) f32[i] = 0u;
        }
        __syncthreads();
        {
            const ColTile cj = col_tile(a.col, j, chunk0, chunk1);
            for (int32_t o = cj.lo + tid; o < cj.hi; o += BLOCK) {
                const int32_t r = (int32_t)(a.col.rows[cj.cb + o] - seg0);
                s_xv[r] = a.col.vals[cj.cb + o];
                lds_flag_or(s_flag, r, kFlagX);
            }
        }
        if (j > a.j_begin) {
            if (tid == 0) {
                u32x4 r[1];
                if (wait_pairs<1>(a.ws.sw_step + b, ((ep - 1) << 1) | 1u, hdr, r))
                    s_step = pair_value(r[0]);
                else
                    s_abort = 1;
            }
            __syncthreads();
            SW_TRACE(a, b, j, 1);
            if (s_abort) return;
            const double st = s_step;
            if (st != 0.0)
                apply_step<BLOCK, true>(a, j - 1, st, seg0, chunk0, chunk1, s_ep, s_flag);
        }
        __syncthreads();
        SW_TRACE(a, b, j, 2);
        double xv[IPT];
        {
            uint8_t fl[IPT];
            lds_bytes<IPT>(s_flag + tid * IPT, fl);
#pragma unroll
            for (int i = 0; i < IPT; ++i) {
                xv[i] = (fl[i] & kFlagX) ? s_xv[tid * IPT + i] : 0.0;
                if (fl[i] & kFlagPatch) ev[i] = s_ep[tid * IPT + i];
            }
        }

        // ---- thread totals, wave scans (DPP), segment aggregate
        double texcl[NC];
        {
            double run[NC];
#pragma unroll
            for (int c = 0; c < NC; ++c) run[c] = 0.0;
#pragma unroll
            for (int i = 0; i < IPT; ++i) {
                const double ex = ev[i] * xv[i];
                run[0] += ev[i];
                run[1] += ex;
                run[2] += ex * xv[i];
            }
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                const double inc = dpp_incl_scan(run[c]);
                texcl[c] = inc - run[c];
                if (lane == kWave - 1) s_wsum[w][c] = inc;
            }
        }
        __syncthreads();
        if (tid == 0) {
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                double t = 0.0;
#pragma unroll
                for (int q = 0; q < NW; ++q) t += s_wsum[q][c];
                st_pair(a.ws.sw_agg + b * 8 + c, t, tag);
            }
        }
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            double before = 0.0;
#pragma unroll
            for (int q = 0; q < NW; ++q)
                if (q < w) before += s_wsum[q][c];
            texcl[c] += before;
        }
        SW_TRACE(a, b, j, 3);

        // ---- exchange 1: workgroup 0 gathers every segment aggregate, scans
        // them in segment order and hands each workgroup its exclusive
        // prefix.
        if (b == 0) {
            constexpr int K = (kMaxSweepBlocks + BLOCK - 1) / BLOCK;
            double v[K][NC];
            bool bad = false;
#pragma unroll
            for (int k = 0; k < K; ++k) {
                const int q = tid * K + k;
#pragma unroll
                for (int c = 0; c < NC; ++c) v[k][c] = 0.0;
                if (q < G && !bad) {
                    u32x4 r[NC];
                    if (wait_pairs<NC>(a.ws.sw_agg + (int64_t)q * 8, tag, hdr, r)) {
#pragma unroll
                        for (int c = 0; c < NC; ++c) v[k][c] = pair_value(r[c]);
                    } else {
                        bad = true;
                    }
                }
            }
            if (__syncthreads_or(bad)) return;
            // exclusive scan over q = tid*K + k: thread-serial, DPP across
            // lanes, LDS across waves
            double tsum[NC];
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                double t = 0.0;
#pragma unroll
                for (int k = 0; k < K; ++k) t += v[k][c];
                tsum[c] = t;
                const double inc = dpp_incl_scan(t);
                tsum[c] = inc - t;  // exclusive within the wave
                if (lane == kWave - 1) s_wsum[w][c] = inc;
            }
            __syncthreads();
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                double before = 0.0;
#pragma unroll
                for (int q = 0; q < NW; ++q)
                    if (q < w) before += s_wsum[q][c];
                tsum[c] += before;
            }
#pragma unroll
            for (int k = 0; k < K; ++k) {
                const int q = tid * K + k;
                if (q < G) {
#pragma unroll
                    for (int c = 0; c < NC; ++c)
                        st_pair(a.ws.sw_pre + (int64_t)q * 8 + c, tsum[c], tag);
                }
#pragma unroll
                for (int c = 0; c < NC; ++c) tsum[c] += v[k][c];
            }
        }
        if (tid == 0) {
            u32x4 r[NC];
            if (wait_pairs<NC>(a.ws.sw_pre + b * 8, tag, hdr, r)) {
#pragma unroll
                for (int c = 0; c < NC; ++c) s_bc[c] = pair_value(r[c]);
            } else {
                s_abort = 1;
            }
        }
        __syncthreads();
        SW_TRACE(a, b, j, 4);
        if (s_abort) return;

        // ---- running prefix, transform at run ends, reduction
        double acc[3] = {0.0, 0.0, 0.0};
        {
            double Sr[3];
#pragma unroll
            for (int c = 0; c < 3; ++c) Sr[c] = texcl[c] + s_bc[c];
#pragma unroll
            for (int i = 0; i < IPT; ++i) {
                const double ex = ev[i] * xv[i];
                Sr[0] += ev[i];
                Sr[1] += ex;
                Sr[2] += ex * xv[i];
                const int d = dk[i];
                if (d != 0) {
                    const double S0 = Sr[0];
                    const double r = 1.0 / S0;
                    const double Gk = Sr[1] * r;
                    const double Hk = Sr[2] * r;
                    const double dd = (double)d;
                    acc[0] += dd * Gk;
                    acc[1] += dd * (Hk - Gk * Gk);
                    if (a.want_log) acc[2] += dd * log(S0);
                }
            }
        }
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            acc[c] = dpp_wave_sum(acc[c]);
            if (lane == 0) s_wred[w][c] = acc[c];
        }
        __syncthreads();

        // ---- exchange 2: partials to workgroup 0, step back to everyone
        if (tid == 0) {
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                double t = 0.0;
#pragma unroll
                for (int q = 0; q < NW; ++q) t += s_wred[q][c];
                st_pair(a.ws.sw_part + b * 4 + c, t, tag);
            }
        }
        SW_TRACE(a, b, j, 5);
        if (b == 0) {
            constexpr int K = (kMaxSweepBlocks + BLOCK - 1) / BLOCK;
            double sum[3] = {0.0, 0.0, 0.0};
            bool bad = false;
#pragma unroll
            for (int k = 0; k < K; ++k) {
                const int q = tid * K + k;
                if (q < G && !bad) {
                    u32x4 r[3];
                    if (wait_pairs<3>(a.ws.sw_part + (int64_t)q * 4, tag, hdr, r)) {
#pragma unroll
                        for (int c = 0; c < 3; ++c) sum[c] += pair_value(r[c]);
                    } else {
                        bad = true;
                    }
                }
            }
            if (__syncthreads_or(bad)) return;
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                sum[c] = dpp_wave_sum(sum[c]);
                if (lane == 0) s_wred[w][c] = sum[c];
            }
            __syncthreads();
            if (tid == 0) {
                double tot[3];
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    double t = 0.0;
#pragma unroll
                    for (int q = 0; q < NW; ++q) t += s_wred[q][c];
                    tot[c] = t;
                }
                const double g1 = a.c[j] - tot[0];
                const double g2 = -tot[1];
                double bj = a.beta[j], dj = a.delta[j], st = 0.0;
                ccd_apply(g1, g2, a.penalty, a.lambda, &bj, &dj, &st);
                a.beta[j] = bj;
                a.delta[j] = dj;
                a.steps[j] = st;
                if (a.g12_out) {
                    a.g12_out[3 * j] = g1;
                    a.g12_out[3 * j + 1] = g2;
                    a.g12_out[3 * j + 2] = tot[2];
                }
                s_step = st;
            }
            __syncthreads();
            SW_TRACE(a, b, j, 6);
            const double st = s_step;
#pragma unroll
            for (int k = 0; k < K; ++k) {
                const int q = tid * K + k;
                if (q < G) st_pair(a.ws.sw_step + q, st, tag);
            }
            SW_TRACE(a, b, j, 7);
        }
    }

    // ---- the last coordinate's update of eta and e
    const int32_t jl = a.j_end - 1;
    const uint64_t ep_last = ep0 + (uint64_t)(jl - a.j_begin);
    if (tid == 0) {
        u32x4 r[1];
        if (wait_pairs<1>(a.ws.sw_step + b, (ep_last << 1) | 1u, hdr, r))
            s_step = pair_value(r[0]);
        else
            s_abort = 1;
    }
    __syncthreads();
    if (s_abort) return;
    if (s_step != 0.0)
        apply_step<BLOCK, false>(a, jl, s_step, seg0, chunk0, chunk1, s_ep, s_flag);
    // every workgroup read the epoch before exchange 1 of the first
    // coordinate, which workgroup 0 waited for
    if (b == 0 && tid == 0)
        st_relaxed_u64(&hdr->epoch, ep0 + (uint64_t)(a.j_end - a.j_begin));
}

// ------------------------------------------------------------------------
// The exchange of the kernels below (exchange.h): a slot is in one of two
// areas of the publication buffer (ss_internal.h), by round parity.
template <bool LATE>
__device__ __forceinline__ u32x4 *pub_area(const WsView &ws, uint64_t round, int copy)
{
    return ws.sw_pub +
           (((int64_t)copy * 2 + (round & 1u)) * kPubSlotWords + (LATE ? 0 : kPubLateWords)) *
               kMaxSweepBlocks;
}
// Words from one segment's slot to the next.
template <bool LATE, int N>
__host__ __device__ constexpr int pub_stride()
{
    return LATE ? kPubLateWords : pub_words<N>() <= 4 ? 4 : kPubEarlyWords;
}

// Publishes t as segment q of the round, in every copy.
template <bool LATE, int N>
__device__ __forceinline__ void publish(const WsView &ws, const double (&t)[N], uint64_t round,
                                        int64_t q, uint64_t tag)
{
    static_assert(kPubLateWords + kPubEarlyWords <= kPubSlotWords, "both slots fit");
    constexpr int64_t copy_words = 2 * (int64_t)kPubSlotWords * kMaxSweepBlocks;
    publish_slots<N, kPubCopies>(pub_area<LATE>(ws, round, 0) + q * pub_stride<LATE, N>(),
                                 copy_words, t, tag);
}

// The sums of gather_sums over a round's publications, from one copy.
template <bool LATE, int N, int NS, int K>
__device__ __forceinline__ bool gather_round(const WsView &ws, uint64_t round, int copy, int t,
                                             int span, int G, int64_t b, uint64_t tag,
                                             const int (&from)[NS], const int (&mode)[NS],
                                             double *dst)
{
    constexpr int words = kMaxSweepBlocks * (LATE ? kPubLateWords : kPubEarlyWords);
    return gather_sums<N, pub_stride<LATE, N>(), NS, K>(pub_area<LATE>(ws, round, copy), words,
                                                        ws.hdr, t, span, G, b, tag, from, mode,
                                                        dst);
}

// ------------------------------------------------------------------------
// One exchange per coordinate, for 0/1 (indicator) designs.
//
// With x in {0, 1}, the update of column j multiplies e by exp(s_j) at the
// rows of column j, so a segment's tuple aggregate for the next coordinate
// is  A + expm1(s_j) D  with  A = sum e (1, x_{j+1})  over the segment and D
// the same sum over the rows of column j -- both known before s_j is.  Every
// workgroup therefore publishes A and D for coordinate j+1 as soon as it has
// them (early: before the transform) and its partial sums for coordinate j
// after the transform (late), then reads all G publications itself, forms
// the sums in the same fixed order, takes the same coordinate update
// (bit-identical everywhere) and its own prefix scan(A) + expm1(s) scan(D)
// over the segments before it.
//
// Bound: the round trip of the late values.  The first half of the waves
// polls them: two 16-byte words per segment, four segments to a cache line
// (with A and D in the same publication, a line per segment polled: N = 1e6,
// P = 1000 5.96 / 10.2 ms Cox / Fine-Gray); the second half meanwhile reads
// and sums A and D, which have arrived.
//
// Between its publication and the next coordinate's a workgroup touches
// global memory only for the exchange itself: e in registers, eta of its
// segment in LDS, the previous column patched in place (eta += s,
// e *= exp(s)), the rows of column j+2 scattered into LDS while the
// publications arrive.  Column c's rows live in bit (c mod 3) of the LDS
// flag bytes.  eta and e = exp(eta) go back to global memory once, at the
// end of the sweep.  c_j, beta_j and delta_j are read before publishing
// round j, and workgroup 0 writes beta_j and delta_j only after it has read
// every publication of that round, so no workgroup can see the updated
// values for the same coordinate.
//
// SOLO: the whole problem in one workgroup, no exchange.
template <int BLOCK, int IPT, int MODEL, bool LOG, bool SOLO>
__global__ __launch_bounds__(BLOCK) void k_sweep1(SweepArgs a)
{
    constexpr int S = BLOCK * IPT;
    constexpr bool FG = MODEL == SS_FINE_GRAY;
    // With x in {0, 1}, e x^2 = e x: the tuple is (e, e x) for Cox and
    // (e, e x, e w, e w x) for Fine-Gray.
    constexpr int NT = FG ? 4 : 2;
    constexpr int NW = BLOCK / kWave;
    // partial sums: sum d G, sum d (G - G^2) and, with LOG, sum d log S0
    constexpr int P0 = LOG ? 3 : 2;
    constexpr int NAD = 2 * NT;             // A, D
    // sums over the segments of A and D: before this one and, for
    // Fine-Gray, the totals of the weighted components (A 2, 3, D 2, 3)
    constexpr int NAS = NAD + (FG ? 4 : 0);
    constexpr int NH = NW / 2;              // waves that gather each kind
    constexpr int K = SOLO ? 1 : (kMaxSweepBlocks + BLOCK / 2 - 1) / (BLOCK / 2);
    static_assert(S % SS_CHUNK == 0, "segment must be whole chunks");

    __shared__ __attribute__((aligned(16))) uint8_t s_flag[S];
    __shared__ double s_eta[S];          // [i * BLOCK + tid]
    __shared__ double s_g[FG ? S : 1];   // G(y) at each position, same layout
    __shared__ double s_wsum[NW][NT];
    __shared__ double s_wnext[NW][NT];   // sums over the rows of column j+1
    __shared__ double s_wred[NW][P0];
    __shared__ double s_sum[2][NW][NAS]; // by round parity
    __shared__ uint64_t s_ep0;
    __shared__ int s_abort;

    const int tid = threadIdx.x;
    const int lane = lane_id();
    const int w = tid / kWave;
    const int64_t b = blockIdx.x;
    const int G = a.nblk;
    WsHeader *hdr = a.ws.hdr;
    const int64_t seg0 = b * S;
    const int64_t cnt = min((int64_t)S, a.n - seg0);
    const int64_t nchunk = a.col.nchunk1 - 1;
    const int64_t chunk0 = seg0 / SS_CHUNK;
    const int64_t chunk1 = min(chunk0 + S / SS_CHUNK, nchunk);
    const int64_t base = seg0 + (int64_t)tid * IPT;
    const int32_t jb = a.j_begin, je = a.j_end;

    if (tid == 0) {
        s_ep0 = ld_relaxed_u64(&hdr->epoch);
        s_abort = 0;
    }
    // ---- the segment's data for the whole sweep
    double ev[IPT];
    int dk[IPT];
    double wv[FG ? IPT : 1];
    if (cnt == S) {
        const double2 *ep = reinterpret_cast<const double2 *>(a.e + base);
        const double2 *hp = reinterpret_cast<const double2 *>(a.eta + base);
#pragma unroll
        for (int q = 0; q < IPT / 2; ++q) {
            const double2 v = ep[q];
            const double2 h = hp[q];
            ev[2 * q] = v.x;
            ev[2 * q + 1] = v.y;
            s_eta[(2 * q) * BLOCK + tid] = h.x;
            s_eta[(2 * q + 1) * BLOCK + tid] = h.y;
        }
        if (FG) {
            const double2 *wp = reinterpret_cast<const double2 *>(a.w_comp + base);
#pragma unroll
            for (int q = 0; q < IPT / 2; ++q) {
                const double2 v = wp[q];
                wv[2 * q] = v.x;
                wv[2 * q + 1] = v.y;
            }
        }
    } else {
#pragma unroll
        for (int i = 0; i < IPT; ++i) {
            const bool ok = base + i < a.n;
            ev[i] = ok ? a.e[base + i] : 0.0;
            s_eta[i * BLOCK + tid] = ok ? a.eta[base + i] : 0.0;
            if (FG) wv[i] = ok ? a.w_comp[base + i] : 0.0;
        }
    }
#pragma unroll
    for (int i = 0; i < IPT; ++i) {
        const int64_t k = base + i;
        const bool ok = k < a.n;
        int d = ok ? (int)a.d8[k] : 0;
        if (d == 255) d = a.d32[k];
        dk[i] = d;
        if (FG) s_g[i * BLOCK + tid] = ok ? a.g_end[k] : 1.0;
    }
    {
        uint32_t *f32 = reinterpret_cast<uint32_t *>(s_flag);
        for (int i = tid; i < S / 4; i += BLOCK) f32[i] = 0u;
    }
    __syncthreads();
    const uint64_t ep0 = s_ep0;

    // Adds column jc's rows of this segment as bit (jc mod 3).
    auto scatter = [&](int32_t jc) {
        const ColTile ct = col_tile(a.col, jc, chunk0, chunk1);
        const uint8_t bit = (uint8_t)(1u << (jc % 3));
        for (int32_t o = ct.lo + tid; o < ct.hi; o += BLOCK)
            lds_flag_or(s_flag, (int32_t)(a.col.rows[ct.cb + o] - seg0), bit);
    };
    // Clears bit (jc mod 3) in the bytes this thread owns.
    auto clear_bit = [&](int32_t jc) {
        const uint32_t keep = ~(0x01010101u << (jc % 3));
        uint32_t *f32 = reinterpret_cast<uint32_t *>(s_flag + tid * IPT);
#pragma unroll
        for (int q = 0; q < IPT / 4; ++q) f32[q] &= keep;
    };
    const int my_copy = (int)(b % kPubCopies);
    // This segment's A and D from the wave sums (all lanes of a wave the
    // same): A = all, on the rows of j+1; D the same on the rows of j.
    auto own_ad = [&](double (&t)[NAD]) {
        double all[NT], next[NT];
#pragma unroll
        for (int c = 0; c < NT; ++c) {
            all[c] = next[c] = 0.0;
#pragma unroll
            for (int q = 0; q < NW; ++q) {
                all[c] += s_wsum[q][c];
                next[c] += s_wnext[q][c];
            }
        }
#pragma unroll
        for (int h = 0; h < NT / 2; ++h) {
            t[2 * h] = all[2 * h];              // A: e (e w)
            t[2 * h + 1] = next[2 * h];         //    on the rows of j+1
            t[NT + 2 * h] = all[2 * h + 1];     // D: on the rows of j
            t[NT + 2 * h + 1] = next[2 * h + 1];//    on the rows of both
        }
    };
    // Publishes the block sums of the partial sums (wave 0).
    auto late = [&](const double (&v)[P0], uint64_t r, uint64_t tag) {
        wave_sums_to<P0>(v, s_wred[w]);
        __syncthreads();
        if (!SOLO && w == 0) {
            double t[P0];
#pragma unroll
            for (int c = 0; c < P0; ++c) {
                t[c] = 0.0;
#pragma unroll
                for (int q = 0; q < NW; ++q) t[c] += s_wred[q][c];
            }
            publish<true, P0>(a.ws, t, r, b, tag);
        }
    };
    // The sums over all segments: `part` the partial sums, `ad` A and D
    // before this segment (then the weighted totals).  False: gave up.
    auto collect = [&](uint64_t r, uint64_t tag, double (&part)[P0], double (&ad)[NAS]) -> bool {
        if constexpr (SOLO) {
            double own[NAD];
            own_ad(own);
#pragma unroll
            for (int c = 0; c < NAS; ++c) ad[c] = 0.0;
            if (FG) {
                ad[NAD] = own[2];
                ad[NAD + 1] = own[3];
                ad[NAD + 2] = own[NT + 2];
                ad[NAD + 3] = own[NT + 3];
            }
#pragma unroll
            for (int c = 0; c < P0; ++c) {
                part[c] = 0.0;
#pragma unroll
                for (int q = 0; q < NW; ++q) part[c] += s_wred[q][c];
            }
            return true;
        } else {
            constexpr int HALF = BLOCK / 2;
            const int par = (int)(r & 1u);
            const int kk = (G + HALF - 1) / HALF;  // segments per thread
            bool ok;
            if (w < NH) {
                int from[P0], mode[P0];
#pragma unroll
                for (int c = 0; c < P0; ++c) {
                    from[c] = c;
                    mode[c] = kAll;
                }
                double *dst = s_sum[par][w];
                ok = kk == 1   ? gather_round<true, P0, P0, 1>(a.ws, r, my_copy, tid, HALF, G, b,
                                                              tag, from, mode, dst)
                     : kk == 2 ? gather_round<true, P0, P0, 2>(a.ws, r, my_copy, tid, HALF, G, b,
                                                              tag, from, mode, dst)
                               : gather_round<true, P0, P0, K>(a.ws, r, my_copy, tid, HALF, G, b,
                                                              tag, from, mode, dst);
            } else {
                int from[NAS], mode[NAS];
#pragma unroll
                for (int c = 0; c < NAD; ++c) {
                    from[c] = c;
                    mode[c] = kBefore;
                }
                if (FG) {
                    const int tot[4] = {2, 3, NT + 2, NT + 3};
#pragma unroll
                    for (int c = 0; c < 4; ++c) {
                        from[NAD + c < NAS ? NAD + c : 0] = tot[c];
                        mode[NAD + c < NAS ? NAD + c : 0] = kAll;
                    }
                }
                double *dst = s_sum[par][w];
                const int t = tid - HALF;
                ok = kk == 1 ? gather_round<false, NAD, NAS, 1>(a.ws, r, my_copy, t, HALF, G, b,
                                                               tag, from, mode, dst)
                             : gather_round<false, NAD, NAS, 2>(a.ws, r, my_copy, t, HALF, G, b,
                                                               tag, from, mode, dst);
            }
            if (__syncthreads_or(!ok)) return false;
#pragma unroll
            for (int c = 0; c < P0; ++c) {
                part[c] = 0.0;
#pragma unroll
                for (int q = 0; q < NH; ++q) part[c] += s_sum[par][q][c];
            }
#pragma unroll
            for (int c = 0; c < NAS; ++c) {
                ad[c] = 0.0;
#pragma unroll
                for (int q = NH; q < NW; ++q) ad[c] += s_sum[par][q][c];
            }
            return true;
        }
    };
    // prefix of this segment (Fine-Gray: plus the suffix starts) for the
    // coordinate after an update s with f = expm1(s)
    auto prefix_from = [&](const double (&ad)[NAS], double f, double (&pre)[NT]) {
#pragma unroll
        for (int c = 0; c < NT; ++c) pre[c] = ad[c] + f * ad[NT + c];
        if (FG) {
#pragma unroll
            for (int c = 2; c < 4; ++c) {
                const double tot = ad[NAD + (c - 2)] + f * ad[NAD + 2 + (c - 2)];
                pre[c] = tot - pre[c];
            }
        }
    };

    // ---- round 0: aggregates of coordinate jb; rows of jb and jb+1
    scatter(jb);
    if (jb + 1 < je) scatter(jb + 1);
    __syncthreads();
    double pre[NT];
    {
        double all[NT], next[NT];
#pragma unroll
        for (int c = 0; c < NT; ++c) all[c] = next[c] = 0.0;
        uint8_t fl[IPT];
        lds_bytes<IPT>(s_flag + tid * IPT, fl);
        const uint8_t bj = (uint8_t)(1u << (jb % 3));
#pragma unroll
        for (int i = 0; i < IPT; ++i) {
            all[0] += ev[i];
            next[0] += (fl[i] & bj) ? ev[i] : 0.0;
            if constexpr (FG) {
                const double ew = ev[i] * wv[i];
                all[2] += ew;
                next[2] += (fl[i] & bj) ? ew : 0.0;
            }
        }
        const uint64_t tag = (ep0 << 1) | 1u;
        wave_sums_to<NT>(all, s_wsum[w]);
        wave_sums_to<NT>(next, s_wnext[w]);
        __syncthreads();
        if (!SOLO && w == NW - 1) {
            double t[NAD];
            own_ad(t);
            publish<false, NAD>(a.ws, t, 0, b, tag);
        }
        double v[P0], part[P0], ad[NAS];
#pragma unroll
        for (int c = 0; c < P0; ++c) v[c] = 0.0;
        late(v, 0, tag);
        if (!collect(0, tag, part, ad)) return;
        prefix_from(ad, 0.0, pre);
        __syncthreads();  // s_wsum, s_wnext have been read
    }
    double st_prev = 0.0, f_prev = 0.0;

    for (int32_t j = jb; j < je; ++j) {
        const uint64_t r = (uint64_t)(j - jb) + 1;  // exchange round of coordinate j
        const uint64_t tag = ((ep0 + r) << 1) | 1u;
        SW_TRACE(a, b, j, 0);
        // the coordinate's constants, read before this round is published
        const double cj = a.c[j];
        double bj = a.beta[j], dj = a.delta[j];
        uint8_t fl[IPT];
        lds_bytes<IPT>(s_flag + tid * IPT, fl);
        const uint8_t bcur = (uint8_t)(1u << (j % 3));
        const uint8_t bnext = (uint8_t)(1u << ((j + 1) % 3));
        const uint8_t bprev = (uint8_t)(1u << ((j + 2) % 3));
        // ---- the update of column j-1, in place
        if (j > jb && st_prev != 0.0) {
            const double fe = exp_from(st_prev, f_prev);
#pragma unroll
            for (int i = 0; i < IPT; ++i) {
                if (fl[i] & bprev) {
                    // LDS atomic add, result unused: no wait for a read
                    // (only this thread touches the position, in order)
                    __hip_atomic_fetch_add(&s_eta[i * BLOCK + tid], st_prev, __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_WORKGROUP);
                    ev[i] *= fe;
                }
            }
        }
        SW_TRACE(a, b, j, 1);
        // ---- in-segment scan of the tuple of coordinate j; A and D of j+1
        const bool has_next = j + 1 < je;
        double texcl[NT];
        {
            double run[NT], next[NT];
#pragma unroll
            for (int c = 0; c < NT; ++c) run[c] = next[c] = 0.0;
#pragma unroll
            for (int i = 0; i < IPT; ++i) {
                const bool xn = has_next && (fl[i] & bnext);
                const double ex = (fl[i] & bcur) ? ev[i] : 0.0;
                run[0] += ev[i];
                run[1] += ex;
                next[0] += xn ? ev[i] : 0.0;
                next[1] += xn ? ex : 0.0;
                if constexpr (FG) {
                    const double ew = ev[i] * wv[i];
                    const double ewx = (fl[i] & bcur) ? ew : 0.0;
                    run[2] += ew;
                    run[3] += ewx;
                    next[2] += xn ? ew : 0.0;
                    next[3] += xn ? ewx : 0.0;
                }
            }
            wave_sums_to<NT>(next, s_wnext[w]);
#pragma unroll
            for (int c = 0; c < NT; ++c) {
                const double inc = dpp_incl_scan(run[c]);
                texcl[c] = inc - run[c];
                if (lane == kWave - 1) s_wsum[w][c] = inc;
            }
        }
        __syncthreads();
        if (!SOLO && w == NW - 1) {
            double t[NAD];
            own_ad(t);
            publish<false, NAD>(a.ws, t, r, b, tag);
        }
        // every thread has read its flags: column j-1's bit is free
        clear_bit(j + 2);
#pragma unroll
        for (int c = 0; c < NT; ++c) {
            double before = 0.0;
#pragma unroll
            for (int q = 0; q < NW; ++q)
                if (q < w) before += s_wsum[q][c];
            texcl[c] += before;
        }
        SW_TRACE(a, b, j, 2);
        // ---- transform and reduction of coordinate j
        double v[P0];
#pragma unroll
        for (int c = 0; c < P0; ++c) v[c] = 0.0;
        {
            double Sr[2], R[2] = {0.0, 0.0};
#pragma unroll
            for (int c = 0; c < 2; ++c) Sr[c] = pre[c] + texcl[c];
            if constexpr (FG) {
#pragma unroll
                for (int c = 0; c < 2; ++c) R[c] = pre[2 + c] - texcl[2 + c];
            }
            // S0 and S1 at a group of positions first, then the transform
            // at all of them at once, masked by the event count: the
            // reciprocals are independent and overlap (one wave per SIMD
            // here, nothing else hides their latency; run by run behind a
            // branch each one waited for the last).
            constexpr int GT = FG ? kSwFgGroup : (IPT < kSwGroup ? IPT : kSwGroup);
#pragma unroll
            for (int i0 = 0; i0 < IPT; i0 += GT) {
                double s0v[GT], s1v[GT];
#pragma unroll
                for (int u = 0; u < GT; ++u) {
                    const int i = i0 + u;
                    const bool xc = fl[i] & bcur;
                    Sr[0] += ev[i];
                    Sr[1] += xc ? ev[i] : 0.0;
                    double S0 = Sr[0], S1 = Sr[1];
                    if constexpr (FG) {
                        const double ew = ev[i] * wv[i];
                        R[0] -= ew;
                        R[1] -= xc ? ew : 0.0;
                        const double g = s_g[i * BLOCK + tid];
                        S0 += g * R[0];
                        S1 += g * R[1];
                    }
                    s0v[u] = S0;
                    s1v[u] = S1;
                }
                // indicator design: S2 = S1, so H = G.  The reciprocal:
                // hardware estimate and Newton steps.  Off the run ends the
                // count is 0, but before the first of them S0 may have
                // underflowed to where the reciprocal is not finite, and
                // 0 times that is no 0: such an S0 counts as kRecipMin.  (N =
                // 1e6, Cox, ms per 1000 coordinates: without a guard 4.62,
                // the maximum 4.66, a select behind the reciprocal 4.75.)
#pragma unroll
                for (int u = 0; u < GT; ++u) {
                    const double Gk = s1v[u] * recip(fmax(s0v[u], kRecipMin));
                    const double dd = (double)dk[i0 + u];  // 0 off the run ends
                    v[0] = fma(dd, Gk, v[0]);
                    v[1] = fma(dd, Gk - Gk * Gk, v[1]);
                }
                if constexpr (LOG) {
#pragma unroll
                    for (int u = 0; u < GT; ++u)
                        if (dk[i0 + u] != 0) v[P0 - 1] += (double)dk[i0 + u] * log(s0v[u]);
                }
            }
            v[0] = fma(0.0, Sr[0] + R[0], v[0]);  // a NaN in e, which the maximum drops
        }
        late(v, r, tag);
        SW_TRACE(a, b, j, 3);
        // ---- rows of column j+2 while the publications arrive
        if (j + 2 < je) scatter(j + 2);
        // ---- every segment's publication: the update of j, the prefix of j+1
        double part[P0], ad[NAS];
        if (!collect(r, tag, part, ad)) return;
        if constexpr (SOLO) __syncthreads();  // the wave sums have been read
        SW_TRACE(a, b, j, 4);
        double st = 0.0;
        {
            const double g1 = cj - part[0];
            const double g2 = -part[1];
            ccd_apply(g1, g2, a.penalty, a.lambda, &bj, &dj, &st);
            if (b == 0 && tid == 0) {
                a.beta[j] = bj;
                a.delta[j] = dj;
                a.steps[j] = st;
                if (a.g12_out) {
                    a.g12_out[3 * j] = g1;
                    a.g12_out[3 * j + 1] = g2;
                    a.g12_out[3 * j + 2] = LOG ? part[P0 - 1] : 0.0;
                }
            }
        }
        f_prev = expm1(st);
        prefix_from(ad, f_prev, pre);
        st_prev = st;
        SW_TRACE(a, b, j, 5);
    }

    // ---- the last coordinate's update, then eta and e back to memory
    {
        uint8_t fl[IPT];
        lds_bytes<IPT>(s_flag + tid * IPT, fl);
        const uint8_t blast = (uint8_t)(1u << ((je - 1) % 3));
#pragma unroll
        for (int i = 0; i < IPT; ++i) {
            const int64_t k = base + i;
            if (k < a.n) {
                double h = s_eta[i * BLOCK + tid];
                if (st_prev != 0.0 && (fl[i] & blast)) h += st_prev;
                a.eta[k] = h;
                a.e[k] = exp(h);
            }
        }
    }
    // every workgroup read the epoch before publishing round 0, which
    // workgroup 0 has gathered
    if (b == 0 && tid == 0)
        st_relaxed_u64(&hdr->epoch, ep0 + (uint64_t)(je - jb) + 1);
}

// ------------------------------------------------------------------------
// Two exchanges per coordinate, for valued designs: exp(x s) is not linear
// in s over the rows of a column, so a segment's aggregate for coordinate j
// is known only after the step of j-1.  Per coordinate: the segment's
// aggregate (early area), every workgroup reads all and takes the sums
// before it (after it for the weighted components); the partial sums (late
// area), every workgroup reads all and takes the same step.
//
// Bound: the two round trips (through workgroup 0 and back they were four,
// k_sweep).  In between: e, eta and the column's values live in LDS as
// [i * BLOCK + tid] (position tid * IPT + i of the segment, so owners read
// without bank conflicts); a column's non-zeros are loaded while the
// aggregates travel, spread evenly over the threads, which keep them for the
// column's own update -- one exponential per non-zero, not per position.
// N = 2e5, P = 200, 30% of the entries non-zero: 2.05 ms per sweep with
// k_sweep.
template <int BLOCK, int IPT, int MODEL, bool SOLO>
__global__ __launch_bounds__(BLOCK) void k_sweep_valued(SweepArgs a)
{
    constexpr int S = BLOCK * IPT;
    constexpr bool FG = MODEL == SS_FINE_GRAY;
    constexpr int NC = FG ? 6 : 3;
    constexpr int NW = BLOCK / kWave;
    constexpr int GT = FG ? 4 : (IPT < 8 ? IPT : 8);  // run ends evaluated together
    // e and x stay in registers across exchange 1, or are read from LDS again
    constexpr bool HOLD = IPT < 16;
    constexpr int NR = HOLD ? IPT : 1;
    static_assert(S % SS_CHUNK == 0, "segment must be whole chunks");

    __shared__ double s_eta[S], s_e[S];
    __shared__ double s_x[2][S];  // column j in buffer j mod 2, 0 off its rows
    __shared__ double s_wsum[NW][NC];
    __shared__ double s_wred[NW][3];
    __shared__ double s_sum[2][NW][NC];  // early, late (3 of NC)
    __shared__ uint64_t s_ep0;

    const int tid = threadIdx.x;
    const int lane = lane_id();
    const int w = tid / kWave;
    const int64_t b = blockIdx.x;
    const int G = a.nblk;
    WsHeader *hdr = a.ws.hdr;
    const int64_t seg0 = b * S;
    const int32_t cnt = (int32_t)min((int64_t)S, a.n - seg0);
    const int64_t nchunk = a.col.nchunk1 - 1;
    const int64_t chunk0 = seg0 / SS_CHUNK;
    const int64_t chunk1 = min(chunk0 + S / SS_CHUNK, nchunk);
    const int32_t jb = a.j_begin, je = a.j_end;
    const int my_copy = (int)(b % kPubCopies);
    auto lds_at = [](int32_t r) { return (r % IPT) * BLOCK + r / IPT; };

    if (tid == 0) s_ep0 = ld_relaxed_u64(&hdr->epoch);
    for (int32_t r = tid; r < S; r += BLOCK) {
        const bool ok = r < cnt;
        s_eta[lds_at(r)] = ok ? a.eta[seg0 + r] : 0.0;
        s_e[lds_at(r)] = ok ? a.e[seg0 + r] : 0.0;
        s_x[0][r] = 0.0;
        s_x[1][r] = 0.0;
    }
    int dk[IPT];
    double wv[FG ? IPT : 1], gv[FG ? IPT : 1];
#pragma unroll
    for (int i = 0; i < IPT; ++i) {
        const int64_t k = seg0 + (int64_t)tid * IPT + i;
        const bool ok = k < a.n;
        int d = ok ? (int)a.d8[k] : 0;
        if (d == 255) d = a.d32[k];
        dk[i] = d;
        if constexpr (FG) {
            wv[i] = ok ? a.w_comp[k] : 0.0;
            gv[i] = ok ? a.g_end[k] : 1.0;
        }
    }
    // a thread's share of a column's non-zeros in the segment: entry
    // tid + u BLOCK at LDS index ei[u]
    int32_t ei[IPT], em = 0;
    double ex[IPT];
    auto load_column = [&](int32_t jc) {
        const ColTile ct = col_tile(a.col, jc, chunk0, chunk1);
        em = ct.hi - ct.lo;
        const int32_t *rp = a.col.rows + ct.cb + ct.lo;
        const double *vp = a.col.vals + ct.cb + ct.lo;
#pragma unroll
        for (int u = 0; u < IPT; ++u) {
            if (u * BLOCK < em) {
                const int32_t o = min(tid + u * BLOCK, em - 1);
                ei[u] = (int32_t)(rp[o] - seg0);
                ex[u] = vp[o];
            }
        }
    };
    auto scatter = [&](double *x) {
#pragma unroll
        for (int u = 0; u < IPT; ++u) {
            if (u * BLOCK < em) {
                ei[u] = lds_at(ei[u]);
                if (tid + u * BLOCK < em) x[ei[u]] = ex[u];
            }
        }
    };
    __syncthreads();
    const uint64_t ep0 = s_ep0;
    load_column(jb);
    scatter(s_x[jb & 1]);
    __syncthreads();

    for (int32_t j = jb; j < je; ++j) {
        const uint64_t r = (uint64_t)(j - jb) + 1;
        const uint64_t tag = ((ep0 + r) << 1) | 1u;
        SW_TRACE(a, b, j, 0);
        // the coordinate's constants, read before this round is published
        const double cj = a.c[j];
        double bj = a.beta[j], dj = a.delta[j];
        // ---- thread totals, wave scans (DPP), segment aggregate
        double ev[NR], xv[NR];
        const double *e_own = s_e + tid;
        double *x_own = s_x[j & 1] + tid;
        if constexpr (HOLD) {
#pragma unroll
            for (int i = 0; i < IPT; ++i) {
                ev[i] = e_own[i * BLOCK];
                xv[i] = x_own[i * BLOCK];
                x_own[i * BLOCK] = 0.0;  // for column j+2
            }
        }
        auto e_at = [&](int i) { return HOLD ? ev[HOLD ? i : 0] : e_own[i * BLOCK]; };
        auto x_at = [&](int i) { return HOLD ? xv[HOLD ? i : 0] : x_own[i * BLOCK]; };
        double texcl[NC], inc[NC];
        {
            double run[NC];
#pragma unroll
            for (int c = 0; c < NC; ++c) run[c] = 0.0;
#pragma unroll
            for (int i = 0; i < IPT; ++i) {
                const double e0 = e_at(i), x = x_at(i);
                const double e1 = e0 * x;
                run[0] += e0;
                run[1] += e1;
                run[2] += e1 * x;
                if constexpr (FG) {
                    const double ew = e0 * wv[i];
                    const double ew1 = ew * x;
                    run[3] += ew;
                    run[4] += ew1;
                    run[5] += ew1 * x;
                }
            }
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                inc[c] = dpp_incl_scan(run[c]);
                texcl[c] = inc[c] - run[c];
                if (lane == kWave - 1) s_wsum[w][c] = inc[c];
            }
        }
        __syncthreads();
        double own[NC];
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            double before = 0.0;
            own[c] = 0.0;
#pragma unroll
            for (int q = 0; q < NW; ++q) {
                if (q < w) before += s_wsum[q][c];
                own[c] += s_wsum[q][c];
            }
            texcl[c] += before;
        }
        if (!SOLO && w == 0) publish<false, NC>(a.ws, own, r, b, tag);
        SW_TRACE(a, b, j, 1);
        // ---- exchange 1, the update's non-zeros of column j kept aside and
        // those of column j+1 loaded meanwhile
        int32_t ui[IPT];
        double ux[IPT];
        const int32_t um = em;
#pragma unroll
        for (int u = 0; u < IPT; ++u) {
            ui[u] = ei[u];
            ux[u] = ex[u];
        }
        if (j + 1 < je) load_column(j + 1);
        double pre[NC];
#pragma unroll
        for (int c = 0; c < NC; ++c) pre[c] = 0.0;
        if constexpr (!SOLO) {
            int from[NC], mode[NC];
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                from[c] = c;
                mode[c] = c < 3 ? kBefore : kAfter;
            }
            const bool ok =
                G <= BLOCK ? gather_round<false, NC, NC, 1>(a.ws, r, my_copy, tid, BLOCK, G, b, tag,
                                                           from, mode, s_sum[0][w])
                           : gather_round<false, NC, NC, 2>(a.ws, r, my_copy, tid, BLOCK, G, b, tag,
                                                           from, mode, s_sum[0][w]);
            if (__syncthreads_or(!ok)) return;
#pragma unroll
            for (int c = 0; c < NC; ++c)
#pragma unroll
                for (int q = 0; q < NW; ++q) pre[c] += s_sum[0][q][c];
        }
        SW_TRACE(a, b, j, 2);
        // ---- running prefix, transform at run ends, reduction.  For
        // Fine-Gray R holds the weighted sums over the positions after the
        // current one.
        double acc[3] = {0.0, 0.0, 0.0};
        {
            double Sr[3], R[3] = {0.0, 0.0, 0.0};
#pragma unroll
            for (int c = 0; c < 3; ++c) Sr[c] = pre[c] + texcl[c];
            if constexpr (FG) {
#pragma unroll
                for (int c = 0; c < 3; ++c) R[c] = (pre[3 + c] + own[3 + c]) - texcl[3 + c];
            }
#pragma unroll
            for (int i0 = 0; i0 < IPT; i0 += GT) {
                double t0[GT], t1[GT], t2[GT];
#pragma unroll
                for (int u = 0; u < GT; ++u) {
                    const int i = i0 + u;
                    const double e0 = e_at(i), x = x_at(i);
                    if constexpr (!HOLD) x_own[i * BLOCK] = 0.0;  // for column j+2
                    const double e1 = e0 * x;
                    Sr[0] += e0;
                    Sr[1] += e1;
                    Sr[2] += e1 * x;
                    t0[u] = Sr[0];
                    t1[u] = Sr[1];
                    t2[u] = Sr[2];
                    if constexpr (FG) {
                        const double ew = e0 * wv[i];
                        const double ew1 = ew * x;
                        R[0] -= ew;
                        R[1] -= ew1;
                        R[2] -= ew1 * x;
                        t0[u] += gv[i] * R[0];
                        t1[u] += gv[i] * R[1];
                        t2[u] += gv[i] * R[2];
                    }
                }
                // all at once, so that the reciprocals overlap; kept at run
                // ends only (S0 may have underflowed to 0 before them)
#pragma unroll
                for (int u = 0; u < GT; ++u) {
                    const double rc = recip(t0[u]);
                    const double Gk = t1[u] * rc;
                    const double dd = (double)dk[i0 + u];
                    const double a0 = fma(dd, Gk, acc[0]);
                    const double a1 = fma(dd, t2[u] * rc - Gk * Gk, acc[1]);
                    acc[0] = dk[i0 + u] != 0 ? a0 : acc[0];
                    acc[1] = dk[i0 + u] != 0 ? a1 : acc[1];
                }
                if (a.want_log) {
#pragma unroll
                    for (int u = 0; u < GT; ++u)
                        if (dk[i0 + u] != 0) acc[2] += (double)dk[i0 + u] * log(t0[u]);
                }
            }
        }
        wave_sums_to<3>(acc, s_wred[w]);
        __syncthreads();
        double tot[3];
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            tot[c] = 0.0;
#pragma unroll
            for (int q = 0; q < NW; ++q) tot[c] += s_wred[q][c];
        }
        if (!SOLO && w == 0) publish<true, 3>(a.ws, tot, r, b, tag);
        SW_TRACE(a, b, j, 3);
        // ---- column j+1 into its buffer, cleared a coordinate ago
        if (j + 1 < je) scatter(s_x[(j + 1) & 1]);
        // ---- exchange 2: the step
        if constexpr (!SOLO) {
            const int from[3] = {0, 1, 2}, mode[3] = {kAll, kAll, kAll};
            const bool ok =
                G <= BLOCK ? gather_round<true, 3, 3, 1>(a.ws, r, my_copy, tid, BLOCK, G, b, tag,
                                                        from, mode, s_sum[1][w])
                           : gather_round<true, 3, 3, 2>(a.ws, r, my_copy, tid, BLOCK, G, b, tag,
                                                        from, mode, s_sum[1][w]);
            if (__syncthreads_or(!ok)) return;
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                tot[c] = 0.0;
#pragma unroll
                for (int q = 0; q < NW; ++q) tot[c] += s_sum[1][q][c];
            }
        }
        SW_TRACE(a, b, j, 4);
        double st = 0.0;
        {
            const double g1 = cj - tot[0];
            const double g2 = -tot[1];
            ccd_apply(g1, g2, a.penalty, a.lambda, &bj, &dj, &st);
            if (b == 0 && tid == 0) {
                a.beta[j] = bj;
                a.delta[j] = dj;
                a.steps[j] = st;
                if (a.g12_out) {
                    a.g12_out[3 * j] = g1;
                    a.g12_out[3 * j + 1] = g2;
                    a.g12_out[3 * j + 2] = tot[2];
                }
            }
        }
        // ---- the update of column j
        if (st != 0.0) {
#pragma unroll
            for (int u = 0; u < IPT; ++u) {
                if (u * BLOCK < um && tid + u * BLOCK < um) {
                    const double h = s_eta[ui[u]] + ux[u] * st;
                    s_eta[ui[u]] = h;
                    s_e[ui[u]] = exp(h);
                }
            }
        }
        __syncthreads();
        SW_TRACE(a, b, j, 5);
    }
    for (int32_t r = tid; r < cnt; r += BLOCK) {
        a.eta[seg0 + r] = s_eta[lds_at(r)];
        a.e[seg0 + r] = s_e[lds_at(r)];
    }
    // every workgroup read the epoch before publishing its first aggregate,
    // which workgroup 0 has gathered
    if (b == 0 && tid == 0) st_relaxed_u64(&hdr->epoch, ep0 + (uint64_t)(je - jb) + 1);
}

// Shapes (workgroup size, positions per thread) of a persistent sweep.
struct Shape {
    int block;
    int ipt;
};

template <int BLOCK, int IPT, bool SOLO>
void *pick_kernel(int model, bool vals, bool log)
{
    if (vals)
        return model == SS_FINE_GRAY
                   ? reinterpret_cast<void *>(&k_sweep_valued<BLOCK, IPT, SS_FINE_GRAY, SOLO>)
                   : reinterpret_cast<void *>(&k_sweep_valued<BLOCK, IPT, SS_COX, SOLO>);
    if (model == SS_FINE_GRAY)
        return log ? reinterpret_cast<void *>(&k_sweep1<BLOCK, IPT, SS_FINE_GRAY, true, SOLO>)
                   : reinterpret_cast<void *>(&k_sweep1<BLOCK, IPT, SS_FINE_GRAY, false, SOLO>);
    return log ? reinterpret_cast<void *>(&k_sweep1<BLOCK, IPT, SS_COX, true, SOLO>)
               : reinterpret_cast<void *>(&k_sweep1<BLOCK, IPT, SS_COX, false, SOLO>);
}

// Indicator designs take the one-exchange kernel (which publishes
// sum d log S0 only when it is asked for), valued ones the two-exchange one.
void *kernel_for(int block, int ipt, int model, bool vals, bool log, bool solo)
{
    if (solo) {
        if (block == 256 && ipt == 4) return pick_kernel<256, 4, true>(model, vals, log);
        if (block == 256 && ipt == 8) return pick_kernel<256, 8, true>(model, vals, log);
        if (block == 256 && ipt == 16) return pick_kernel<256, 16, true>(model, vals, log);
    }
    if (block == 256 && ipt == 4) return pick_kernel<256, 4, false>(model, vals, log);
    if (block == 256 && ipt == 8) return pick_kernel<256, 8, false>(model, vals, log);
    if (block == 256 && ipt == 16) return pick_kernel<256, 16, false>(model, vals, log);
    if (block == 512 && ipt == 8) return pick_kernel<512, 8, false>(model, vals, log);
    // 8192-position segments: Cox only (Fine-Gray would not fit its LDS or
    // would spill registers); valued ones by the kernel that keeps only the
    // column and the patches in LDS
    if (block == 512 && ipt == 16 && model == SS_COX) {
        if (vals) return reinterpret_cast<void *>(&k_sweep<512, 16>);
        return log ? reinterpret_cast<void *>(&k_sweep1<512, 16, SS_COX, true, false>)
                   : reinterpret_cast<void *>(&k_sweep1<512, 16, SS_COX, false, false>);
    }
    return nullptr;
}

// The built-in shape for n positions: one workgroup while its serial part
// is shorter than an exchange, then segments of 1024 (short serial parts)
// while every CU holds at most one workgroup, then longer ones.  us per
// coordinate, Cox 0/1 | Fine-Gray 0/1 | Cox valued | Fine-Gray valued (30%):
//   n = 4000    one workgroup 2.3 | 3.7 | 5.3 | 7.7,  256 x 4  3.1 | 3.9 | 4.2 | 5.3
//   n = 1e5     256 x 4       3.3 | 4.3 | - | -,      256 x 8  3.4 | 4.4 | - | -
//   n = 2e5     256 x 4       3.4 | 5.1 | 5.7 | 7.2,  256 x 8  3.5 | 4.7 | 6.5 | 8.7
//   n = 4e5     256 x 4       5.5 | 6.4 | 9.1 | 16.6, 256 x 8  3.8 | 5.6 | 7.0 | 9.3,
//               256 x 16      4.5 | 6.4 | 9.0 | -
//   n = 1e6     256 x 16 4.85, 512 x 8 4.7 (Cox 0/1)
Shape default_shape(int32_t model, bool vals, int64_t n)
{
    if (n <= 1024) return Shape{256, 4};
    if (n <= 2048) return Shape{256, 8};
    if (n <= 4096 && !vals) return Shape{256, 16};
    if (n <= (model == SS_COX || vals ? 1 << 18 : 1 << 17)) return Shape{256, 4};
    if (n <= 1 << 19) return Shape{256, 8};
    return model == SS_COX && !vals ? Shape{512, 8} : Shape{256, 16};
}

}  // namespace

int32_t launch_sweep_persistent(const SweepCall &call, const WsView &ws, hipStream_t s)
{
    // what is left when the shape of the rule below does not fit the device
    static const Shape others[] = {{256, 16}, {512, 8}, {256, 8}, {512, 16}};
    int dev = 0;
    SS_HIP_CHECK(hipGetDevice(&dev));
    int cus = 0, coop = 0;
    SS_HIP_CHECK(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
    SS_HIP_CHECK(hipDeviceGetAttribute(&coop, hipDeviceAttributeCooperativeLaunch, dev));
    if (!coop) return SS_EUNSUPPORTED;
    const bool vals = call.col.vals != nullptr;
    // a tuned shape first, then the built-in order; a shape forced by a
    // tuning call alone
    Shape order[6];
    int m = 0;
    const int32_t want = tune_lookup(SS_TUNE_SWEEP, call.model, SS_STORAGE_F64, vals, call.n);
    if (want) order[m++] = Shape{want / 100, want % 100};
    if (!(tune_force().choice && tune_force().kind == SS_TUNE_SWEEP)) {
        if (!want) order[m++] = default_shape(call.model, vals, call.n);
        for (const Shape &sh : others)
            if (sh.block != order[0].block || sh.ipt != order[0].ipt) order[m++] = sh;
    }
    for (int o = 0; o < m; ++o) {
        const Shape &sh = order[o];
        const int64_t seg = (int64_t)sh.block * sh.ipt;
        const int64_t G = ceil_div(call.n, seg);
        // a few hundred segments at most: the all-to-all exchange reads G
        // aggregates per workgroup
        if (G > kMaxSweepBlocks || G > ws.max_tiles) continue;
        void *k = kernel_for(sh.block, sh.ipt, call.model, vals, call.g12_out != nullptr, G == 1);
        if (!k) continue;
        int per_cu = 0;
        SS_HIP_CHECK(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k, sh.block, 0));
        if ((int64_t)per_cu * cus < G) continue;
        SweepArgs a;
        a.n = call.n;
        a.j_begin = call.j_begin;
        a.j_end = call.j_end;
        a.nblk = (int32_t)G;
        a.eta = call.eta;
        a.e = call.e;
        a.d8 = call.d8;
        a.d32 = call.d32;
        a.w_comp = call.w_comp;
        a.g_end = call.g_end;
        a.col = call.col;
        a.c = call.c;
        a.beta = call.beta;
        a.delta = call.delta;
        a.steps = call.steps;
        a.g12_out = call.g12_out;
        a.penalty = call.penalty;
        a.lambda = call.lambda;
        a.want_log = call.g12_out != nullptr;
        a.ws = ws;
        void *args[] = {&a};
        SS_HIP_CHECK(hipLaunchCooperativeKernel(k, dim3((unsigned)G), dim3((unsigned)sh.block),
                                                args, 0, s));
        return SS_OK;
    }
    return SS_EUNSUPPORTED;
}

}  // namespace ss
