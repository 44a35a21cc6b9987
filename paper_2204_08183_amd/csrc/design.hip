// The CSC design re-labelled to sorted positions (gfx950): the rows of every
// column as ascending sorted positions, the values in that order, the
// per-column chunk index and c_j = sum over events of x_ij.
//
// The rows of a column are distinct positions, so ordering them needs no
// sort: a workgroup sets one bit per position in an LDS bitmap, takes prefix
// counts over it, and reads the ascending list (and each value's place in
// it) back from the bits.  A column is cut into windows of at most 2^20
// positions (a 128 KB bitmap); one (column, window) piece is one workgroup's
// work.  With one window the rows are read where they are; with more, a
// counting pass and a placement pass first group each column's non-zeros by
// window (in any order: the bitmap orders them).
//
// Bound: per non-zero one random 4-byte read of inv_perm and one LDS atomic;
// 8 bytes of HBM traffic (20 valued) against 24 per pass of the 4-5 pass LSD
// radix sort of (column, position) keys it replaced.  N = 1e6, P = 1000, 5e7
// non-zeros: 288 us against 3.3 ms.  In a build that reads the clock between
// its phases (298 us) the bits take 171 (5e7 random reads, 292 G a second, the
// rate at which the L2s take requests: batches pipelined so that reads and
// atomics overlap gave nothing), the list 103 (a store per entry and lane; a
// wave's run gathered in LDS first took 77, but what followed waited as much
// longer, the preparation unchanged at 617), counts and clearing 24.
#include <algorithm>
#include <vector>

#include "scan_device.h"
#include "ss_internal.h"

namespace ss {

namespace {

constexpr int kMaxWindowBits = 20;
constexpr int kGroupWords = 8;                    // words per prefix count
constexpr int kGroupPos = 32 * kGroupWords;       // 256 positions
constexpr int kSmallMax = 1024;                   // entries the small kernel sorts in LDS
constexpr int kPartChunk = 16384;                 // entries per workgroup of the grouping passes
constexpr int kMaxWindows = 2048;                 // ceil(2^31 / 2^20)

struct DesignArgs {
    int64_t n, p, nchunk;
    int64_t nwin;             // windows per column
    int32_t wbits;            // log2(positions per window) when nwin > 1
    const int64_t *col_ptr;
    const uint32_t *piece;    // nwin > 1: first entry of every piece, then nnz
    const int32_t *rows;      // nwin == 1: the caller's rows and values
    const double *vals;
    const int32_t *inv_perm;
    const uint32_t *pos;      // nwin > 1: positions and values grouped by piece
    const double *pv;
    const uint32_t *ev_bits;  // bit k: the subject at position k had an event
    int32_t *rows_sorted;
    double *vals_sorted;
    int32_t *chunk_ptr;
    double *part;             // event sum of every piece
    uint32_t *err;
};

struct Piece {
    int64_t col, c0, lo, base;
    int32_t m, cnt;  // entries (at most cnt), positions of the window
    bool last;       // the column's last window
    bool over;       // there are more entries than positions
};

__device__ __forceinline__ Piece piece_of(const DesignArgs &a, int64_t q)
{
    Piece r;
    r.col = a.nwin == 1 ? q : q / a.nwin;
    const int64_t win = q - r.col * a.nwin;
    r.c0 = a.col_ptr[r.col];
    r.lo = a.nwin == 1 ? r.c0 : (int64_t)a.piece[q];
    const int64_t hi = a.nwin == 1 ? a.col_ptr[r.col + 1] : (int64_t)a.piece[q + 1];
    r.base = win << (a.nwin == 1 ? 0 : a.wbits);
    const int64_t left = a.n - r.base;
    r.cnt = (int32_t)(a.nwin == 1 ? left : min(left, (int64_t)1 << a.wbits));
    // more entries than positions: some row is there twice, and the others
    // need no look (a count near 2^31 would take the loops' int32 past it)
    r.over = hi - r.lo > r.cnt;
    r.m = (int32_t)min(hi - r.lo, (int64_t)r.cnt);
    r.last = win == a.nwin - 1;
    return r;
}

// A piece with few entries for its window is sorted entry by entry
// (k_design_small); clearing and counting the window's bitmap would cost
// more.  The line: one entry per 512 positions, at most kSmallMax.
__host__ __device__ __forceinline__ bool is_small(int64_t m, int64_t cnt)
{
    return m <= kSmallMax && m < cnt / 512;
}

// Positions of U of a piece's entries, i = first + u * stride (the last entry
// again past the end): U independent loads, and U more through inv_perm.  An
// out-of-range row sets `bad` and is taken as row 0.
template <int U>
__device__ __forceinline__ void entry_pos(const DesignArgs &a, const Piece &pc, int32_t first,
                                          int32_t stride, uint32_t (&k)[U], bool &bad)
{
    if (a.nwin > 1) {
#pragma unroll
        for (int u = 0; u < U; ++u) k[u] = a.pos[pc.lo + min(first + u * stride, pc.m - 1)];
        return;
    }
    int32_t r[U];
#pragma unroll
    for (int u = 0; u < U; ++u) r[u] = a.rows[pc.lo + min(first + u * stride, pc.m - 1)];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const bool out = r[u] < 0 || r[u] >= a.n;
        bad |= out;
        k[u] = (uint32_t)a.inv_perm[out ? 0 : r[u]];
    }
}

template <int BLOCK>
__device__ __forceinline__ double block_sum_all(double v, double *s_red)
{
    v = dpp_wave_sum(v);
    __syncthreads();
    if (lane_id() == 0) s_red[threadIdx.x / kWave] = v;
    __syncthreads();
    double t = 0.0;
#pragma unroll
    for (int i = 0; i < BLOCK / kWave; ++i) t += s_red[i];
    return t;
}

template <int BLOCK, bool VALS>
__global__ __launch_bounds__(BLOCK) void k_design_bits(DesignArgs a, int32_t max_words)
{
    constexpr int NW = BLOCK / kWave;
    constexpr int U = BLOCK == 1024 ? 16 : 8;  // entries in flight per thread
    extern __shared__ __attribute__((aligned(16))) uint32_t s_bits[];
    uint32_t *s_pre = s_bits + max_words;  // entries before every group of words
    __shared__ uint32_t s_w[NW];
    __shared__ double s_red[NW];
    const int tid = threadIdx.x, lane = lane_id(), w = tid / kWave;
    for (int64_t q = blockIdx.x; q < a.p * a.nwin; q += gridDim.x) {
        const Piece pc = piece_of(a, q);
        if (is_small(pc.m, pc.cnt)) continue;
        const int words = (pc.cnt + 31) / 32;
        const int groups = (pc.cnt + kGroupPos - 1) / kGroupPos;
        uint4 *b4 = reinterpret_cast<uint4 *>(s_bits);
        for (int i = tid; i < groups * (kGroupWords / 4); i += BLOCK) b4[i] = uint4{0, 0, 0, 0};
        __syncthreads();

        // ---- one bit per entry
        bool bad = false, twice = false;
        for (int32_t o = tid; o < pc.m; o += U * BLOCK) {
            uint32_t k[U];
            entry_pos<U>(a, pc, o, BLOCK, k, bad);
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (o + u * BLOCK < pc.m) {
                    k[u] -= (uint32_t)pc.base;
                    const uint32_t bit = 1u << (k[u] & 31u);
                    twice |= (atomicOr(&s_bits[k[u] >> 5], bit) & bit) != 0u;
                }
            }
        }
        if (bad) atomicOr(a.err, 8u);
        if (twice || pc.over) atomicOr(a.err, 16u);  // a duplicate row
        __syncthreads();

        // ---- entries per group of words, then their exclusive prefix
        for (int g = tid; g < groups; g += BLOCK) {
            const uint4 x = b4[2 * g], y = b4[2 * g + 1];
            s_pre[g] = __popc(x.x) + __popc(x.y) + __popc(x.z) + __popc(x.w) + __popc(y.x) +
                       __popc(y.y) + __popc(y.z) + __popc(y.w);
        }
        __syncthreads();
        uint32_t carry = 0;
        for (int g0 = 0; g0 < groups; g0 += BLOCK) {
            const int g = g0 + tid;
            const uint32_t own = g < groups ? s_pre[g] : 0u;
            uint32_t inc = own;
#pragma unroll
            for (int off = 1; off < kWave; off <<= 1) {
                const uint32_t y = __shfl_up(inc, off, kWave);
                if (lane >= off) inc += y;
            }
            if (lane == kWave - 1) s_w[w] = inc;
            __syncthreads();
            uint32_t before = carry, all = 0;
#pragma unroll
            for (int i = 0; i < NW; ++i) {
                if (i < w) before += s_w[i];
                all += s_w[i];
            }
            if (g < groups) s_pre[g] = before + inc - own;
            carry += all;
            __syncthreads();
        }

        // ---- the chunk index: a chunk is SS_CHUNK / kGroupPos groups
        {
            int32_t *cp = a.chunk_ptr + pc.col * (a.nchunk + 1) + pc.base / SS_CHUNK;
            const int32_t off = (int32_t)(pc.lo - pc.c0);
            const int chunks = (pc.cnt + SS_CHUNK - 1) / SS_CHUNK;
            for (int t = tid; t < chunks; t += BLOCK)
                cp[t] = off + (int32_t)s_pre[t * (SS_CHUNK / kGroupPos)];
            if (pc.last && tid == 0) cp[chunks] = off + pc.m;
        }

        // ---- the ascending positions, a lane per 64 of them: neighbouring
        // lanes write neighbouring runs
        double evs = 0.0;
        constexpr int kPairs = kGroupWords / 2;  // lanes that share a group
        const uint64_t *b64 = reinterpret_cast<const uint64_t *>(s_bits);
        const uint64_t *e64 = reinterpret_cast<const uint64_t *>(a.ev_bits + pc.base / 32);
        for (int p0 = 0; p0 < (words + 1) / 2; p0 += BLOCK) {
            const int pr = p0 + tid;
            const bool in = pr < (words + 1) / 2;
            uint64_t x = in ? b64[pr] : 0u;
            if (!VALS && in) evs += (double)__popcll(x & e64[pr]);
            uint32_t inc = (uint32_t)__popcll(x);
            const uint32_t own = inc;
#pragma unroll
            for (int off = 1; off < kPairs; off <<= 1) {
                const uint32_t y = __shfl_up(inc, off, kPairs);
                if ((lane & (kPairs - 1)) >= off) inc += y;
            }
            int32_t *dst = a.rows_sorted + pc.lo + (in ? (int32_t)(s_pre[pr / kPairs] + inc - own) : 0);
            const int32_t k0 = (int32_t)(pc.base + 64 * (int64_t)pr);
            while (x != 0u) {
                *dst++ = k0 + (__ffsll((unsigned long long)x) - 1);
                x &= x - 1u;
            }
        }
        if (VALS) {
            // ---- every value to its entry's place, then the event sum in
            // that order
            double *dst = a.vals_sorted + pc.lo;
            constexpr int V = 4;
            for (int32_t o = tid; o < pc.m; o += V * BLOCK) {
                uint32_t k[V];
                double v[V];
                entry_pos<V>(a, pc, o, BLOCK, k, bad);
#pragma unroll
                for (int u = 0; u < V; ++u) {
                    const int64_t i = pc.lo + min(o + u * BLOCK, pc.m - 1);
                    v[u] = a.nwin > 1 ? a.pv[i] : a.vals[i];
                }
#pragma unroll
                for (int u = 0; u < V; ++u) {
                    k[u] -= (uint32_t)pc.base;
                    const uint32_t g = k[u] / kGroupPos, wd = (k[u] >> 5) & (kGroupWords - 1);
                    const uint4 x = b4[2 * g], y = b4[2 * g + 1];
                    const uint32_t ws[kGroupWords] = {x.x, x.y, x.z, x.w, y.x, y.y, y.z, y.w};
                    const uint32_t below = (1u << (k[u] & 31u)) - 1u;
                    uint32_t at = s_pre[g];
#pragma unroll
                    for (int q = 0; q < kGroupWords; ++q)
                        at += __popc(q < (int)wd ? ws[q] : q == (int)wd ? ws[q] & below : 0u);
                    if (o + u * BLOCK < pc.m) dst[at] = v[u];
                }
            }
            __syncthreads();
            for (int32_t i = tid; i < pc.m; i += BLOCK) {
                const int32_t k = a.rows_sorted[pc.lo + i];
                if (k >= 0 && k < a.n && (a.ev_bits[k >> 5] >> (k & 31)) & 1u)
                    evs += a.vals_sorted[pc.lo + i];
            }
        }
        const double t = block_sum_all<BLOCK>(evs, s_red);
        if (tid == 0) a.part[q] = t;
        __syncthreads();
    }
}

// Pieces with few entries: a bitonic sort of (position, entry) in LDS.
constexpr int kSmallBlock = 256;

template <bool VALS>
__global__ __launch_bounds__(kSmallBlock) void k_design_small(DesignArgs a)
{
    constexpr int BLOCK = kSmallBlock;
    __shared__ uint64_t s_k[kSmallMax];
    __shared__ double s_red[BLOCK / kWave];
    const int tid = threadIdx.x;
    for (int64_t q = blockIdx.x; q < a.p * a.nwin; q += gridDim.x) {
        const Piece pc = piece_of(a, q);
        if (!is_small(pc.m, pc.cnt)) continue;
        int size = 2;
        while (size < pc.m) size *= 2;
        bool bad = false;
        for (int i = tid; i < size && pc.m > 0; i += BLOCK) {
            uint32_t k[1];
            entry_pos<1>(a, pc, i, 0, k, bad);
            s_k[i] = i < pc.m ? ((uint64_t)k[0] << 32) | (uint32_t)i : ~0ull;
        }
        if (bad) atomicOr(a.err, 8u);
        __syncthreads();
        for (int k = 2; k <= size; k *= 2) {
            for (int d = k / 2; d > 0; d /= 2) {
                for (int i = tid; i < size / 2; i += BLOCK) {
                    const int x = 2 * i - (i & (d - 1)), y = x + d;
                    const uint64_t u = s_k[x], v = s_k[y];
                    if ((u > v) == ((x & k) == 0)) {
                        s_k[x] = v;
                        s_k[y] = u;
                    }
                }
                __syncthreads();
            }
        }
        double evs = 0.0;
        for (int i = tid; i < pc.m; i += BLOCK) {
            const uint32_t k = (uint32_t)(s_k[i] >> 32);
            if (i > 0 && (uint32_t)(s_k[i - 1] >> 32) == k) atomicOr(a.err, 16u);
            double v = 1.0;
            if (VALS) {
                const int64_t o = pc.lo + (int32_t)(uint32_t)s_k[i];
                v = a.nwin > 1 ? a.pv[o] : a.vals[o];
                a.vals_sorted[pc.lo + i] = v;
            }
            a.rows_sorted[pc.lo + i] = (int32_t)k;
            if ((a.ev_bits[k >> 5] >> (k & 31u)) & 1u) evs += v;
        }
        int32_t *cp = a.chunk_ptr + pc.col * (a.nchunk + 1) + pc.base / SS_CHUNK;
        const int chunks = (pc.cnt + SS_CHUNK - 1) / SS_CHUNK;
        for (int t = tid; t < chunks; t += BLOCK) {
            const uint64_t first = (uint64_t)(pc.base + (int64_t)t * SS_CHUNK) << 32;
            int lo = 0, hi = pc.m;
            while (lo < hi) {
                const int mid = (lo + hi) / 2;
                if (s_k[mid] < first) lo = mid + 1;
                else hi = mid;
            }
            cp[t] = (int32_t)(pc.lo - pc.c0) + lo;
        }
        if (pc.last && tid == 0) cp[chunks] = (int32_t)(pc.lo - pc.c0) + pc.m;
        const double t = block_sum_all<BLOCK>(evs, s_red);
        if (tid == 0) a.part[q] = t;
        __syncthreads();
    }
}

// c_j = the sum of the column's pieces in order.
__global__ void k_design_c(int64_t p, int64_t nwin, const double *part, double *c)
{
    for (int64_t j = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; j < p;
         j += (int64_t)gridDim.x * blockDim.x) {
        double t = 0.0;
        for (int64_t q = j * nwin; q < (j + 1) * nwin; ++q) t += part[q];
        c[j] = t;
    }
}

// ------------------------------------------------------ grouping by window
struct PartChunk {
    int64_t col, begin, end;  // three numbers in the host's list
};

// Positions of a chunk's entries, and its share of the column's counts per
// window.
__global__ __launch_bounds__(256) void k_part_count(const PartChunk *chunks, int64_t nchunks,
                                                    int64_t n, int64_t nwin, int32_t wbits,
                                                    const int32_t *rows, const int32_t *inv_perm,
                                                    uint32_t *pos, uint32_t *cnt, uint32_t *err)
{
    __shared__ uint32_t s_h[kMaxWindows];
    for (int64_t q = blockIdx.x; q < nchunks; q += gridDim.x) {
        const PartChunk ch = chunks[q];
        for (int i = threadIdx.x; i < nwin; i += 256) s_h[i] = 0u;
        __syncthreads();
        for (int64_t o = ch.begin + threadIdx.x; o < ch.end; o += 256) {
            int32_t r = rows[o];
            if (r < 0 || r >= n) {
                atomicOr(err, 8u);
                r = 0;
            }
            const uint32_t k = (uint32_t)inv_perm[r];
            pos[o] = k;
            atomicAdd(&s_h[k >> wbits], 1u);
        }
        __syncthreads();
        for (int i = threadIdx.x; i < nwin; i += 256)
            if (s_h[i] != 0u) atomicAdd(&cnt[ch.col * nwin + i], s_h[i]);
        __syncthreads();
    }
}

// Entries to their pieces: a chunk reserves a run in every piece it has
// entries for (counting `cnt` back down to 0) and fills it in any order.
template <bool VALS>
__global__ __launch_bounds__(256) void k_part_place(const PartChunk *chunks, int64_t nchunks,
                                                    int64_t nwin, int32_t wbits,
                                                    const uint32_t *pos, const double *vals,
                                                    const uint32_t *piece, uint32_t *cnt,
                                                    uint32_t *out_pos, double *out_vals)
{
    __shared__ uint32_t s_h[kMaxWindows];
    for (int64_t q = blockIdx.x; q < nchunks; q += gridDim.x) {
        const PartChunk ch = chunks[q];
        for (int i = threadIdx.x; i < nwin; i += 256) s_h[i] = 0u;
        __syncthreads();
        for (int64_t o = ch.begin + threadIdx.x; o < ch.end; o += 256)
            atomicAdd(&s_h[pos[o] >> wbits], 1u);
        __syncthreads();
        for (int i = threadIdx.x; i < nwin; i += 256) {
            const uint32_t h = s_h[i];
            const int64_t g = ch.col * nwin + i;
            if (h != 0u) s_h[i] = piece[g] + atomicSub(&cnt[g], h) - h;
        }
        __syncthreads();
        for (int64_t o = ch.begin + threadIdx.x; o < ch.end; o += 256) {
            const uint32_t k = pos[o];
            const uint32_t at = atomicAdd(&s_h[k >> wbits], 1u);
            out_pos[at] = k;
            if (VALS) out_vals[at] = vals[o];
        }
        __syncthreads();
    }
}

__global__ void k_zero_u32(uint32_t *p, int64_t m)
{
    for (int64_t k = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; k < m;
         k += (int64_t)gridDim.x * blockDim.x)
        p[k] = 0u;
}

// Windows per column and their size.  Up to 2^20 positions a column is one
// window; fewer, longer columns than the chip has workgroups for are cut
// further while a piece keeps over 16384 entries (below 128 pieces the
// bitmap kernel would leave half the CUs idle).
struct Windows {
    int64_t nwin;
    int32_t wbits;
};

Windows windows_for(int64_t n, int64_t p, int64_t nnz)
{
    int b = kMaxWindowBits;
    while (b > 15 && (int64_t)1 << (b - 1) >= n) --b;
    int64_t nwin = ceil_div(n, (int64_t)1 << b);
    while (b > 15 && p * nwin < 128 && nnz / (p * nwin) > 16384) {
        --b;
        nwin = ceil_div(n, (int64_t)1 << b);
    }
    return Windows{nwin, b};
}

struct DesignWs {
    uint32_t *cnt, *piece, *pos, *out_pos;
    uint64_t *sums;
    double *out_vals, *part;
    PartChunk *chunks;
};

size_t layout(int64_t n, int64_t p, int64_t nnz, char *base, DesignWs *w)
{
    const Windows win = windows_for(n, p, nnz);
    const size_t pieces = (size_t)(p * win.nwin);
    size_t off = 0;
    auto take = [&](size_t bytes) {
        char *r = base ? base + off : nullptr;
        off = align_up(off + bytes, 256);
        return r;
    };
    DesignWs t = {};
    t.part = (double *)take(8 * pieces);
    if (win.nwin > 1) {
        t.cnt = (uint32_t *)take(4 * (pieces + 1));
        t.piece = (uint32_t *)take(4 * (pieces + 1));
        t.sums = (uint64_t *)take(8 * (size_t)(ceil_div((int64_t)pieces + 1, ST) + 1));
        t.pos = (uint32_t *)take(4 * (size_t)nnz);
        t.out_pos = (uint32_t *)take(4 * (size_t)nnz);
        t.out_vals = (double *)take(8 * (size_t)nnz);
        t.chunks = (PartChunk *)take(sizeof(PartChunk) * (size_t)(nnz / kPartChunk + p + 1));
    }
    if (w) *w = t;
    return off;
}

template <int BLOCK>
int32_t launch_bits(const DesignArgs &a, int64_t grid, int32_t max_words, hipStream_t s)
{
    const size_t lds = 4 * (size_t)max_words + 4 * (size_t)(max_words / kGroupWords);
    void *k = a.vals_sorted ? (void *)&k_design_bits<BLOCK, true>
                            : (void *)&k_design_bits<BLOCK, false>;
    // the largest window's, whatever this one's: the attribute belongs to the
    // process, and several threads may be here
    constexpr size_t most = ((size_t)1 << kMaxWindowBits) / 8 * (kGroupWords + 1) / kGroupWords;
    if (BLOCK == 1024)
        SS_HIP_CHECK(hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)most));
    DesignArgs args = a;
    void *ptrs[] = {&args, &max_words};
    SS_HIP_CHECK(hipLaunchKernel(k, dim3((unsigned)grid), dim3(BLOCK), ptrs, lds, s));
    return SS_OK;
}

}  // namespace

size_t design_ws_bytes(int64_t n, int64_t p, int64_t nnz)
{
    return layout(n, p, nnz, nullptr, nullptr);
}

int32_t run_design(int64_t n, int64_t p, int64_t nnz, const int64_t *cp_host,
                   const int64_t *col_ptr, const int32_t *rows, const double *vals,
                   const int32_t *inv_perm, const uint32_t *ev_bits, int32_t *rows_sorted,
                   double *vals_sorted, int32_t *chunk_ptr, double *c, uint32_t *err, void *ws,
                   std::vector<int64_t> &host_list, hipStream_t s)
{
    DesignWs w;
    layout(n, p, nnz, (char *)ws, &w);
    const Windows win = windows_for(n, p, nnz);
    DesignArgs a;
    a.n = n;
    a.p = p;
    a.nchunk = ceil_div(n, SS_CHUNK);
    a.nwin = win.nwin;
    a.wbits = win.wbits;
    a.col_ptr = col_ptr;
    a.piece = w.piece;
    a.rows = rows;
    a.vals = vals;
    a.inv_perm = inv_perm;
    a.pos = w.out_pos;
    a.pv = w.out_vals;
    a.ev_bits = ev_bits;
    a.rows_sorted = rows_sorted;
    a.vals_sorted = vals ? vals_sorted : nullptr;
    a.chunk_ptr = chunk_ptr;
    a.part = w.part;
    a.err = err;
    const int64_t pieces = p * win.nwin;
    const int64_t window = win.nwin == 1 ? n : (int64_t)1 << win.wbits;
    bool any_small = win.nwin > 1, any_bits = win.nwin > 1;
    if (win.nwin == 1) {
        for (int64_t j = 0; j < p && !(any_small && any_bits); ++j)
            (is_small(cp_host[j + 1] - cp_host[j], n) ? any_small : any_bits) = true;
    } else {
        host_list.reserve(3 * (size_t)(nnz / kPartChunk + p + 1));
        for (int64_t j = 0; j < p; ++j)
            for (int64_t o = cp_host[j]; o < cp_host[j + 1]; o += kPartChunk)
                host_list.insert(host_list.end(),
                                 {j, o, std::min(o + kPartChunk, cp_host[j + 1])});
        const int64_t nch = (int64_t)host_list.size() / 3;
        const unsigned grid = (unsigned)std::max<int64_t>(1, std::min<int64_t>(nch, 65536));
        hipLaunchKernelGGL(k_zero_u32, dim3((unsigned)std::min<int64_t>(
                                           8192, ceil_div(pieces + 1, 256))),
                           dim3(256), 0, s, w.cnt, pieces + 1);
        SS_LAUNCH_CHECK();
        if (nch > 0) {
            SS_HIP_CHECK(hipMemcpyAsync(w.chunks, host_list.data(),
                                        sizeof(int64_t) * host_list.size(),
                                        hipMemcpyHostToDevice, s));
            hipLaunchKernelGGL(k_part_count, dim3(grid), dim3(256), 0, s, w.chunks, nch, n,
                               win.nwin, win.wbits, rows, inv_perm, w.pos, w.cnt, err);
            SS_LAUNCH_CHECK();
        }
        const int32_t rc = scan_add_u32_excl(w.cnt, w.piece, pieces + 1, w.sums, s);
        if (rc) return rc;
        if (nch > 0) {
            if (vals)
                hipLaunchKernelGGL(k_part_place<true>, dim3(grid), dim3(256), 0, s, w.chunks, nch,
                                   win.nwin, win.wbits, w.pos, vals, w.piece, w.cnt, w.out_pos,
                                   w.out_vals);
            else
                hipLaunchKernelGGL(k_part_place<false>, dim3(grid), dim3(256), 0, s, w.chunks,
                                   nch, win.nwin, win.wbits, w.pos, vals, w.piece, w.cnt,
                                   w.out_pos, w.out_vals);
            SS_LAUNCH_CHECK();
        }
    }
    const int64_t grid = std::min<int64_t>(pieces, 65536);
    if (any_small) {
        if (vals)
            hipLaunchKernelGGL(k_design_small<true>, dim3((unsigned)grid), dim3(kSmallBlock), 0,
                               s, a);
        else
            hipLaunchKernelGGL(k_design_small<false>, dim3((unsigned)grid), dim3(kSmallBlock), 0,
                               s, a);
        SS_LAUNCH_CHECK();
    }
    if (any_bits) {
        // whole groups of words; a window of over 2^17 positions leaves room
        // for few workgroups per CU, so they are larger
        const int32_t max_words = (int32_t)(ceil_div(window, (int64_t)kGroupPos) * kGroupWords);
        const int32_t rc = window > (1 << 17) ? launch_bits<1024>(a, grid, max_words, s)
                                              : launch_bits<256>(a, grid, max_words, s);
        if (rc) return rc;
    }
    hipLaunchKernelGGL(k_design_c, dim3((unsigned)std::min<int64_t>(8192, ceil_div(p, 256))),
                       dim3(256), 0, s, p, win.nwin, w.part, c);
    SS_LAUNCH_CHECK();
    return SS_OK;
}

}  // namespace ss
