// One-time preparation of a data set on the GPU (gfx950):
//  - stable ordering by decreasing observed time (Sec. 2.7), by an LSD radix
//    sort whose in-tile ranks come from wave64 ballots, so equal times keep
//    increasing subject index;
//  - tie runs, events per run (Cox: status != 0, Fine-Gray: status == 1);
//  - Fine-Gray: Kaplan-Meier estimate of the censoring survival G (Sec. 2.2)
//    as a suffix product over runs, the competing-event weights 1/G(y) and
//    G(y) at every position;
//  - (design.hip) the CSC design re-labelled to sorted positions, the
//    per-column chunk index and c_j = sum over events of x_ij.
// Every integer output is produced with exact integer arithmetic, so it is
// identical from run to run.
#include <utility>
#include <vector>

#include "scan_device.h"
#include "ss_internal.h"

namespace ss {

namespace {

// ------------------------------------------------------------ generic scan
// (block-level pieces in scan_device.h)

__global__ __launch_bounds__(SB) void k_scan_reduce(const uint32_t *in, int64_t m, uint32_t *sums)
{
    __shared__ uint32_t s_w[SB / kWave];
    uint32_t it[SI];
    load_items<uint32_t, OpAdd<uint32_t>>(in, (int64_t)blockIdx.x * ST + (int64_t)threadIdx.x * SI,
                                          m, it);
    const uint32_t tot = block_scan<uint32_t, OpAdd<uint32_t>>(it, 0, s_w);
    if (threadIdx.x == 0) sums[blockIdx.x] = tot;
}

// Single workgroup: exclusive scan of sums[0..nb) in place.
template <typename T, typename Op>
__global__ __launch_bounds__(SB) void k_scan_spine(T *sums, int64_t nb)
{
    __shared__ T s_w[SB / kWave];
    __shared__ T s_last[SB / kWave];
    T carry = Op::id();
    for (int64_t c0 = 0; c0 < nb; c0 += ST) {
        T it[SI];
        const int64_t base = c0 + (int64_t)threadIdx.x * SI;
#pragma unroll
        for (int i = 0; i < SI; ++i) it[i] = base + i < nb ? sums[base + i] : Op::id();
        const T tot = block_scan<T, Op>(it, carry, s_w);
        inclusive_to_exclusive<T>(it, carry, s_last);
#pragma unroll
        for (int i = 0; i < SI; ++i)
            if (base + i < nb) sums[base + i] = it[i];
        carry = Op::op(carry, tot);
    }
}

// Carry of a tile (REV: `sums` are those of the tiles from the last on).  Up
// to ST tiles every workgroup combines the totals of the tiles before its own
// itself, in order; above, k_scan_spine has.  (A launch of one workgroup and
// the gap before it: 3.7 us; the totals of 500 tiles: below 1 us.)
template <typename T, typename Op, bool REV>
__device__ __forceinline__ T tile_carry(const T *sums, int64_t tiles, T *s_w)
{
    const int64_t cnt = REV ? tiles - 1 - (int64_t)blockIdx.x : (int64_t)blockIdx.x;
    if (tiles > ST) return sums[cnt];
    T it[SI];
    load_items<T, Op>(sums, (int64_t)threadIdx.x * SI, cnt, it);
    return block_scan<T, Op>(it, Op::id(), s_w);
}

__global__ __launch_bounds__(SB) void k_scan_down(const uint32_t *in, uint32_t *out, int64_t m,
                                                  int64_t tiles, const uint32_t *sums)
{
    using Op = OpAdd<uint32_t>;
    __shared__ uint32_t s_w[SB / kWave];
    __shared__ uint32_t s_last[SB / kWave];
    uint32_t it[SI];
    const int64_t base = (int64_t)blockIdx.x * ST + (int64_t)threadIdx.x * SI;
    load_items<uint32_t, Op>(in, base, m, it);
    const uint32_t carry = tile_carry<uint32_t, Op, false>(sums, tiles, s_w);
    block_scan<uint32_t, Op>(it, carry, s_w);
    inclusive_to_exclusive<uint32_t>(it, carry, s_last);
    store_items<uint32_t>(out, base, m, it);  // `in` and `out` may alias: a thread's own items
}

// ------------------------------------------------------------ radix sort
// One pass orders (key, value) records by 8 bits of the key, stably.  A tile
// is RB * RI records, wave w of a workgroup its w-th part in rounds of 64,
// so a record's rank among equal digits of the tile is its rank in the
// wave's rounds before (a counter per wave and digit in LDS, no barrier),
// in its round (wave ballots) and the counts of the waves before; the records
// are put in order in LDS and leave as runs.  All of a thread's loads are in
// flight at once.  Bound: at 1e6 records 245 workgroups, one per CU, and in
// each the serial rounds: 8 waves of 8 rounds 16.5 us a pass with the counts
// added up, 4 waves of 16 rounds 19.3, 16 waves of 4 as 8.  (Rounds over the
// whole workgroup with three barriers each, 8-byte values and records stored
// one by one: 22.5 us without them; hist 6.3, now 4.3.)
constexpr int RB = 512;
constexpr int RI = 8;
constexpr int RT = RB * RI;
constexpr int RD = 256;  // digits
// Up to kOwnOffsets tiles a scatter adds the tiles' counts up itself, one row
// of 256 a tile (a tile alone needs none); above, a scan over the counts by
// digit has.  (1e6 records: two launches of 6 us and their gaps a pass against
// 4.7 us more in the scatter, a preparation 609 -> 591 us; the rows read grow
// with the square of the tiles.)
constexpr int64_t kOwnOffsets = 256;

template <bool ROWS>
__global__ __launch_bounds__(RB) void k_radix_hist(const uint64_t *keys, int64_t m,
                                                   int shift, uint32_t *hist,
                                                   int64_t nb)
{
    __shared__ uint32_t cnt[RB / kWave][RD];
    const int w = threadIdx.x / kWave;
#pragma unroll
    for (int q = threadIdx.x; q < RB / kWave * RD; q += RB) (&cnt[0][0])[q] = 0;
    const int64_t base = (int64_t)blockIdx.x * RT;
    uint64_t key[RI];
#pragma unroll
    for (int r = 0; r < RI; ++r) {
        const int64_t idx = base + (int64_t)r * RB + threadIdx.x;
        key[r] = keys[idx < m ? idx : m - 1];
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < RI; ++r)
        if (base + (int64_t)r * RB + threadIdx.x < m)
            atomicAdd(&cnt[w][(key[r] >> shift) & 255u], 1u);
    __syncthreads();
    if (threadIdx.x >= RD) return;
    uint32_t t = 0;
#pragma unroll
    for (int q = 0; q < RB / kWave; ++q) t += cnt[q][threadIdx.x];
    hist[ROWS ? (int64_t)blockIdx.x * RD + threadIdx.x
              : (int64_t)threadIdx.x * nb + blockIdx.x] = t;
}

// Exclusive prefix over a workgroup's threads.
__device__ __forceinline__ uint32_t excl_prefix(uint32_t v, uint32_t *s_wsum)
{
    const int lane = lane_id();
    const int w = threadIdx.x / kWave;
    uint32_t inc = v;
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) {
        const uint32_t y = __shfl_up(inc, off, kWave);
        if (lane >= off) inc += y;
    }
    __syncthreads();
    if (lane == kWave - 1) s_wsum[w] = inc;
    __syncthreads();
    uint32_t pre = inc - v;
#pragma unroll
    for (int q = 0; q < RB / kWave; ++q)
        if (q < w) pre += s_wsum[q];
    return pre;
}

template <bool ROWS>
__global__ __launch_bounds__(RB) void k_radix_scatter(const uint64_t *kin, const uint32_t *vin,
                                                      int64_t m, int shift, const uint32_t *offs,
                                                      int64_t nb, uint64_t *kout, uint32_t *vout,
                                                      uint32_t *err)
{
    constexpr int NW = RB / kWave;
    __shared__ uint32_t s_cnt[NW][RD];    // records of a wave, then of the waves before
    __shared__ uint32_t s_off[RD];        // where a digit's run of the tile goes, less its start
    __shared__ uint32_t s_start[RD];      // a digit's first record in the ordered tile
    __shared__ uint32_t s_wsum[NW];
    __shared__ uint64_t s_key[RT];
    __shared__ uint32_t s_val[RT];
    const int tid = threadIdx.x;
    const int lane = lane_id();
    const int w = tid / kWave;
    const int64_t tile0 = (int64_t)blockIdx.x * RT;
    const int64_t base = tile0 + (int64_t)w * (RI * kWave) + lane;
    uint64_t key[RI];
    uint32_t val[RI];
#pragma unroll
    for (int r = 0; r < RI; ++r) {
        const int64_t idx = base + r * kWave;
        key[r] = kin[idx < m ? idx : m - 1];
    }
#pragma unroll
    for (int r = 0; r < RI; ++r) {
        const int64_t idx = base + r * kWave;
        val[r] = vin[idx < m ? idx : m - 1];
    }
    uint32_t first = 0;  // where the tile's run of digit tid goes
    if constexpr (!ROWS) {
        if (tid < RD) first = offs[(int64_t)tid * nb + blockIdx.x];
    } else if (nb > 1) {
        // wave w adds every NW-th row up, lane l digits 4 l .. 4 l + 3
        const uint4 *row = reinterpret_cast<const uint4 *>(offs) + lane;
        uint4 all = {0, 0, 0, 0}, before = {0, 0, 0, 0};
#pragma unroll 8
        for (int64_t q = w; q < nb; q += NW) {
            const uint4 v = row[q * kWave];
            const uint32_t m_ = q < blockIdx.x ? ~0u : 0u;
            all.x += v.x, all.y += v.y, all.z += v.z, all.w += v.w;
            before.x += v.x & m_, before.y += v.y & m_, before.z += v.z & m_, before.w += v.w & m_;
        }
        uint32_t *t = reinterpret_cast<uint32_t *>(s_key);
        reinterpret_cast<uint4 *>(t)[w * kWave + lane] = all;
        reinterpret_cast<uint4 *>(t + NW * RD)[w * kWave + lane] = before;
        __syncthreads();
        uint32_t sum = 0;
        if (tid < RD) {
#pragma unroll
            for (int q = 0; q < NW; ++q) {
                sum += t[q * RD + tid];
                first += t[(NW + q) * RD + tid];
            }
        }
        first += excl_prefix(sum, s_wsum);
    }
#pragma unroll
    for (int q = tid; q < NW * RD; q += RB) (&s_cnt[0][0])[q] = 0;
    __syncthreads();
    const uint64_t lt_mask = (lane == 0) ? 0ull : ((~0ull) >> (kWave - lane));
    uint32_t rank[RI];  // within the wave
    volatile uint32_t *cnt = s_cnt[w];
#pragma unroll
    for (int r = 0; r < RI; ++r) {
        const bool valid = base + r * kWave < m;
        const uint32_t digit = (uint32_t)(key[r] >> shift) & 255u;
        uint64_t peers = __ballot(valid);
#pragma unroll
        for (int b = 0; b < 8; ++b) {
            const bool bit = (digit >> b) & 1u;
            const uint64_t mb = __ballot(bit);
            peers &= bit ? mb : ~mb;
        }
        // every lane reads its digit's counter before the first of its
        // peers moves it on (one wave: its LDS accesses are in order)
        const uint32_t before = cnt[digit];
        __builtin_amdgcn_wave_barrier();
        rank[r] = before + __popcll(peers & lt_mask);
        if (valid && (peers & lt_mask) == 0) cnt[digit] = before + __popcll(peers);
        __builtin_amdgcn_wave_barrier();
    }
    __syncthreads();
    // thread = digit: the waves' counts become the counts of the waves
    // before, the tile's counts their exclusive prefix over the digits
    uint32_t total = 0;
    if (tid < RD) {
#pragma unroll
        for (int q = 0; q < NW; ++q) {
            const uint32_t c = s_cnt[q][tid];
            s_cnt[q][tid] = total;
            total += c;
        }
    }
    const uint32_t start = excl_prefix(total, s_wsum);
    if (ROWS && nb == 1) first = start;
    if (tid < RD) {
        s_start[tid] = start;
        s_off[tid] = first - start;
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < RI; ++r) {
        if (base + r * kWave < m) {
            const uint32_t digit = (uint32_t)(key[r] >> shift) & 255u;
            const uint32_t at = s_start[digit] + s_cnt[w][digit] + rank[r];
            s_key[at] = key[r];
            s_val[at] = val[r];
        }
    }
    __syncthreads();
    const int cnt_tile = (int)min((int64_t)RT, m - tile0);
    for (int i = tid; i < cnt_tile; i += RB) {
        const uint64_t k = s_key[i];
        const uint32_t off = s_off[(uint32_t)(k >> shift) & 255u] + (uint32_t)i;
        if ((int64_t)off < m) {
            kout[off] = k;
            vout[off] = s_val[i];
        } else {
            atomicOr(err, 32u);
        }
    }
}

// ------------------------------------------------------------ prepare steps
__device__ __forceinline__ uint64_t desc_key(double y)
{
    if (y == 0.0) y = 0.0;  // -0 and +0 are the same time
    uint64_t b = __double_as_longlong(y);
    const uint64_t asc = (b >> 63) ? ~b : (b | 0x8000000000000000ull);
    return ~asc;  // ascending key order = decreasing time
}

// The record of a subject: its key, and its index with the status in the two
// bits above it (PACKED: n <= 2^30), so that the order brings both along and
// nothing is gathered through it.  *vary collects the key bits in which the
// subjects differ.
constexpr int kIdxBits = 30;

template <bool PACKED>
__global__ __launch_bounds__(256) void k_time_keys(const double *y, const int8_t *status,
                                                   int64_t n, uint64_t *keys, uint32_t *vals,
                                                   unsigned long long *vary, uint32_t *err)
{
    __shared__ uint64_t s_v[256 / kWave];
    const uint64_t k0 = desc_key(y[0]);
    uint64_t v = 0;
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x) {
        const uint64_t k = desc_key(y[i]);
        int8_t s = status[i];
        if (s < 0 || s > 2) {
            atomicOr(err, 2u);
            s = 0;
        }
        keys[i] = k;
        vals[i] = (uint32_t)i | (PACKED ? (uint32_t)s << kIdxBits : 0u);
        v |= k ^ k0;
    }
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) v |= __shfl_xor(v, off, kWave);
    if (lane_id() == 0) s_v[threadIdx.x / kWave] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int q = 1; q < 256 / kWave; ++q) v |= s_v[q];
        // 2048 workgroups' atomics on one word took 22 us; most add nothing
        if (v & ~__hip_atomic_load(vary, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
            atomicOr(vary, (unsigned long long)v);
    }
}

// The order from the sorted records.  low > 0: the keys are in order by the
// bits from `low` up only, so a group of records that agree in those is put in
// order here -- by (key, position), which is what the remaining stable passes
// would give -- each record looking at its group once for the place it goes
// to.  (A preparation of 1e6 times in groups of some 8, 16 and 32: 313, 540 and
// 532 us, the last two by all bits in the end; 581 by all bits at once; 434,
// 841 and 969 with every position looking for its record over all pairs.)
// Groups of equal keys are in order already; a group of different ones with
// over kGroupMax records on either side of a change sets err[1], and the
// caller orders all bits instead (1e6 continuous times and one far from them:
// 557 us for a preparation that always ordered all 64 bits, 515 with the
// attempt first; without the far one 571 and 296).
//
// Continuous times differ in sign and exponent, 12 bits at most, and spread
// over the mantissa: 20 bits of it leave groups of below 8 records on average
// up to kFewBits subjects, 28 bits below 8 at any size.  Times in whole units
// vary in few bits and have none left for this.
constexpr int64_t kFewBits = (int64_t)1 << 23;
constexpr int kGroupMax = 32;

template <bool PACKED>
__global__ __launch_bounds__(256) void k_after_sort(int64_t n, int low, const uint64_t *keys,
                                                    const uint32_t *vals, const int8_t *status,
                                                    int32_t *perm, int32_t *inv_perm,
                                                    uint64_t *key_s, int8_t *st_s, uint32_t *err)
{
    for (int64_t k = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; k < n;
         k += (int64_t)gridDim.x * blockDim.x) {
        if (low > 0 &&
            __hip_atomic_load(err + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
            return;
        int64_t at = k;
        const uint64_t key = keys[k];
        const uint64_t prev = k > 0 ? keys[k - 1] : ~key, next = k + 1 < n ? keys[k + 1] : ~key;
        if (low > 0 && ((prev ^ key) >> low == 0 || (next ^ key) >> low == 0)) {
            int64_t a = k, b = k;  // the group, as far as it is looked at
            // one look at the ends of that settles most large groups
            const uint64_t fa = keys[k > kGroupMax ? k - kGroupMax - 1 : k];
            const uint64_t fb = keys[k + kGroupMax + 1 < n ? k + kGroupMax + 1 : k];
            if ((fa != key && (fa ^ key) >> low == 0) || (fb != key && (fb ^ key) >> low == 0)) {
                err[1] = 1u;  // no atomic: thousands of waves may get here
                return;  // all of this is done again
            }
            // records of the group that go elsewhere: larger keys before
            // this one move behind it, smaller ones after it before it
            bool mixed = false;
            while (a > 0 && k - a <= kGroupMax) {
                const uint64_t q = keys[a - 1];
                if ((q ^ key) >> low != 0) break;
                --a;
                mixed = mixed || q != key;
                at -= q > key;
            }
            while (b + 1 < n && b - k <= kGroupMax) {
                const uint64_t q = keys[b + 1];
                if ((q ^ key) >> low != 0) break;
                ++b;
                mixed = mixed || q != key;
                at += q < key;
            }
            if (mixed && (k - a > kGroupMax || b - k > kGroupMax)) {
                err[1] = 1u;
                return;
            }
        }
        const uint32_t v = vals[k];
        int64_t i = PACKED ? v & ((1u << kIdxBits) - 1u) : v;
        if (i >= n) {
            atomicOr(err, 64u);
            i = 0;
        }
        int8_t s = PACKED ? (int8_t)(v >> kIdxBits) : status[i];
        if (s < 0 || s > 2) s = 0;  // reported by k_time_keys
        perm[at] = (int32_t)i;
        inv_perm[i] = (int32_t)at;
        key_s[at] = key;
        st_s[at] = s;
    }
}

__global__ void k_fill_i32(int32_t *p, int64_t m, int32_t v)
{
    for (int64_t k = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; k < m;
         k += (int64_t)gridDim.x * blockDim.x)
        p[k] = v;
}

// A NaN time ties with nothing.
__device__ __forceinline__ bool same_time(uint64_t a, uint64_t b)
{
    const uint64_t inf = 0x000fffffffffffffull;  // +inf; -inf is its complement
    return a == b && a >= inf && a <= ~inf;
}

// Counts since the start of the tie run, as a scan: bit 63 marks a span with
// a run start in it, bits 31..61 count the events and bits 0..30 the censored
// subjects after the last one.
struct OpRun {
    __device__ static uint64_t id() { return 0; }
    __device__ static uint64_t op(uint64_t a, uint64_t b) { return (b >> 63) ? b : a + b; }
};

__device__ __forceinline__ void run_items(int64_t n, int model, const uint64_t *key_s,
                                          const int8_t *st_s, int64_t k0, uint64_t (&key)[SI],
                                          uint64_t (&it)[SI], uint32_t &events)
{
    load_items<uint64_t, OpRun>(key_s, k0, n, key);
    uint64_t prev = k0 > 0 && k0 < n ? key_s[k0 - 1] : 0;
    // st_s is aligned to 256 bytes and holds whole runs of SI
    const uint64_t st = k0 < n ? *reinterpret_cast<const uint64_t *>(st_s + k0) : 0;
    events = 0;  // a bit per item
#pragma unroll
    for (int i = 0; i < SI; ++i) {
        const int64_t k = k0 + i;
        it[i] = 0;
        if (k < n) {
            const int8_t s = (int8_t)(st >> (8 * i));
            const bool ev = model == SS_COX ? (s != 0) : (s == 1);
            it[i] = ((uint64_t)(k == 0 || !same_time(key[i], prev)) << 63) | ((uint64_t)ev << 31) |
                    (uint64_t)(s == 0);
            events |= (uint32_t)ev << i;
            prev = key[i];
        }
    }
}

// Also leaves the events as one bit per position (a thread's items: a byte).
__global__ __launch_bounds__(SB) void k_runs_reduce(int64_t n, int model, const uint64_t *key_s,
                                                    const int8_t *st_s, uint64_t *sums,
                                                    uint8_t *ev_bytes)
{
    static_assert(SI == 8, "a byte of events per thread");
    __shared__ uint64_t s_w[SB / kWave];
    uint64_t key[SI], it[SI];
    uint32_t events;
    const int64_t k0 = (int64_t)blockIdx.x * ST + (int64_t)threadIdx.x * SI;
    run_items(n, model, key_s, st_s, k0, key, it, events);
    if (k0 < n) ev_bytes[k0 / 8] = (uint8_t)events;
    const uint64_t t = block_scan<uint64_t, OpRun>(it, 0, s_w);
    if (threadIdx.x == 0) sums[blockIdx.x] = t;
}

// d at run ends; Fine-Gray also the Kaplan-Meier factor 1 - m_c / #{y >= c} at
// run ends (#{y >= c} = position of the run's last subject + 1), 1 elsewhere,
// and the product of a tile's factors (from the last tile on).
template <bool FG>
__global__ __launch_bounds__(SB) void k_runs_finish(int64_t n, int model, int64_t tiles,
                                                    const uint64_t *key_s, const int8_t *st_s,
                                                    const uint64_t *sums, uint8_t *d8,
                                                    int32_t *d32, double *fac, double *prods)
{
    __shared__ uint64_t s_w[SB / kWave];
    __shared__ double s_p[SB / kWave];
    const int64_t k0 = (int64_t)blockIdx.x * ST + (int64_t)threadIdx.x * SI;
    uint64_t key[SI], it[SI];
    uint32_t events;
    run_items(n, model, key_s, st_s, k0, key, it, events);
    const uint64_t carry = tile_carry<uint64_t, OpRun, false>(sums, tiles, s_w);
    block_scan<uint64_t, OpRun>(it, carry, s_w);
    const uint64_t after = k0 + SI < n ? key_s[k0 + SI] : 0;
    double f[SI], prod = 1.0;
    int32_t d[SI];
    uint64_t d8v = 0;
#pragma unroll
    for (int i = 0; i < SI; ++i) {
        const int64_t k = k0 + i;
        f[i] = 1.0;
        d[i] = 0;
        if (k < n) {
            const bool end = k == n - 1 || !same_time(key[i], i + 1 < SI ? key[(i + 1) % SI] : after);
            if (end) d[i] = (int32_t)((it[i] >> 31) & 0x7fffffffu);
            d8v |= (uint64_t)(d[i] > 255 ? 255 : d[i]) << (8 * i);
            if (FG && end) f[i] = 1.0 - (double)(int32_t)(it[i] & 0x7fffffffu) / (double)(k + 1);
        }
        prod *= f[i];
    }
    store_items<int32_t>(d32, k0, n, d);
    if (k0 + SI <= n && ((uintptr_t)(d8 + k0) & 7u) == 0) {
        *reinterpret_cast<uint64_t *>(d8 + k0) = d8v;
    } else {
        for (int i = 0; i < SI; ++i)
            if (k0 + i < n) d8[k0 + i] = (uint8_t)(d8v >> (8 * i));
    }
    if constexpr (FG) {
        store_items<double>(fac, k0, n, f);
        for (int off = 32; off > 0; off >>= 1) prod *= __shfl_down(prod, off);
        if (lane_id() == 0) s_p[threadIdx.x / kWave] = prod;
        __syncthreads();
        if (threadIdx.x == 0)
            prods[tiles - 1 - blockIdx.x] = ((s_p[0] * s_p[1]) * s_p[2]) * s_p[3];
    }
}

// Kaplan-Meier G as the inclusive suffix product of the factors, and the
// competing-event weights.  Tile t scans from the end of the positions.
__global__ __launch_bounds__(SB) void k_km_weights(int64_t n, int64_t tiles, const double *fac,
                                                   const double *prods, const int8_t *st_s,
                                                   double *g_end, double *w_comp)
{
    __shared__ double s_w[SB / kWave];
    // thread t holds the items of run SB - 1 - t of the tile, last one first
    const int64_t k0 = (int64_t)blockIdx.x * ST + (int64_t)(SB - 1 - (int)threadIdx.x) * SI;
    double f[SI], it[SI];
    load_items<double, OpMul<double>>(fac, k0, n, f);
#pragma unroll
    for (int i = 0; i < SI; ++i) it[i] = f[SI - 1 - i];
    const double carry = tile_carry<double, OpMul<double>, true>(prods, tiles, s_w);
    block_scan<double, OpMul<double>>(it, carry, s_w);
    double g[SI], wt[SI];
#pragma unroll
    for (int i = 0; i < SI; ++i) {
        g[i] = it[SI - 1 - i];
        const int64_t k = k0 + i;
        wt[i] = k < n && st_s[k] == 2 ? 1.0 / g[i] : 0.0;
    }
    store_items<double>(g_end, k0, n, g);
    store_items<double>(w_comp, k0, n, wt);
}

int grid_1d(int64_t work, int cap = 8192)
{
    int64_t g = ceil_div(work, 256);
    if (g < 1) g = 1;
    if (g > cap) g = cap;
    return (int)g;
}

// ------------------------------------------------------------ workspace
struct PrepWs {
    uint64_t *keyA, *keyB;
    uint32_t *valA, *valB;
    uint32_t *hist;
    uint64_t *sums;       // scan spine (8-byte slots for any T)
    double *prods;
    int8_t *st_s;
    uint32_t *ev_bits;
    uint64_t *vary;       // then the error word and k_after_sort's
    void *design;
};

size_t layout(int64_t n, int64_t p, int64_t nnz, char *base, PrepWs *w)
{
    const int64_t nbr = ceil_div(n, RT);
    const int64_t hist_len = 256 * nbr;
    const int64_t scan_len = hist_len > n ? hist_len : n;
    const int64_t nbs = ceil_div(scan_len, ST) + 1;
    size_t off = 0;
    auto take = [&](size_t bytes) {
        char *p = base ? base + off : nullptr;
        off = align_up(off + bytes, 256);
        return p;
    };
    PrepWs t;
    t.ev_bits = (uint32_t *)take(4 * 2 * (size_t)ceil_div(n, kWave));
    t.vary = (uint64_t *)take(256);
    // the design's scratch takes the place of the ordering's, which is done
    t.design = base ? base + off : nullptr;
    const size_t design_end = off + design_ws_bytes(n, p, nnz);
    t.keyA = (uint64_t *)take(8 * (size_t)n);
    t.keyB = (uint64_t *)take(8 * (size_t)n);
    t.valA = (uint32_t *)take(4 * (size_t)n);
    t.valB = (uint32_t *)take(4 * (size_t)n);
    t.hist = (uint32_t *)take(4 * (size_t)hist_len);
    t.sums = (uint64_t *)take(8 * (size_t)nbs);
    t.prods = (double *)take(8 * (size_t)nbs);
    t.st_s = (int8_t *)take(align_up((size_t)n, SI));
    if (w) *w = t;
    return off > design_end ? off : design_end;
}

// Sorts (keyA, valA) by the key bits [low, high); result in the returned
// buffers.
int32_t radix_sort(int64_t m, int low, int high, PrepWs &w, uint64_t **keys_out,
                   uint32_t **vals_out, hipStream_t s)
{
    uint64_t *ka = w.keyA, *kb = w.keyB;
    uint32_t *va = w.valA, *vb = w.valB;
    const int64_t nb = ceil_div(m, RT);
    for (int shift = low; shift < high; shift += 8) {
        const dim3 grid((unsigned)nb);
        if (nb <= kOwnOffsets) {
            if (nb > 1) {
                hipLaunchKernelGGL(k_radix_hist<true>, grid, dim3(RB), 0, s, ka, m, shift, w.hist,
                                   nb);
                SS_LAUNCH_CHECK();
            }
            hipLaunchKernelGGL(k_radix_scatter<true>, grid, dim3(RB), 0, s, ka, va, m, shift,
                               w.hist, nb, kb, vb, (uint32_t *)(w.vary + 1));
        } else {
            hipLaunchKernelGGL(k_radix_hist<false>, grid, dim3(RB), 0, s, ka, m, shift, w.hist,
                               nb);
            SS_LAUNCH_CHECK();
            const int32_t rc = scan_add_u32_excl(w.hist, w.hist, 256 * nb, w.sums, s);
            if (rc) return rc;
            hipLaunchKernelGGL(k_radix_scatter<false>, grid, dim3(RB), 0, s, ka, va, m, shift,
                               w.hist, nb, kb, vb, (uint32_t *)(w.vary + 1));
        }
        SS_LAUNCH_CHECK();
        std::swap(ka, kb);
        std::swap(va, vb);
    }
    *keys_out = ka;
    *vals_out = va;
    return SS_OK;
}

}  // namespace

size_t prepare_ws_bytes(int64_t n, int64_t p, int64_t nnz)
{
    return layout(n, p, nnz, nullptr, nullptr);
}

int32_t run_prepare(int32_t model, int64_t n, int64_t p, int64_t nnz, const double *y,
                    const int8_t *status, const int64_t *col_ptr, const int32_t *rows,
                    const double *vals, int32_t *perm, int32_t *inv_perm, uint8_t *d8,
                    int32_t *d32, double *c, int32_t *rows_sorted, double *vals_sorted,
                    int32_t *chunk_ptr, double *w_comp, double *g_end, void *ws,
                    size_t ws_bytes, hipStream_t s)
{
    PrepWs w;
    if (layout(n, p, nnz, (char *)ws, &w) > ws_bytes) return SS_EWORKSPACE;
    const bool fg = model == SS_FINE_GRAY;
    int32_t rc;

    uint32_t *err = (uint32_t *)(w.vary + 1);
    const bool packed = n <= (int64_t)1 << kIdxBits;
    std::vector<int64_t> cp_host((size_t)p + 1);
    std::vector<int64_t> host_list;
    for (bool all_bits = false;; all_bits = true) {
        hipLaunchKernelGGL(k_fill_i32, dim3(1), dim3(64), 0, s, (int32_t *)w.vary, (int64_t)4, 0);
        SS_LAUNCH_CHECK();
        if (packed)
            hipLaunchKernelGGL(k_time_keys<true>, dim3(grid_1d(n, 1024)), dim3(256), 0, s, y,
                               status, n, w.keyA, w.valA, (unsigned long long *)w.vary, err);
        else
            hipLaunchKernelGGL(k_time_keys<false>, dim3(grid_1d(n, 1024)), dim3(256), 0, s, y,
                               status, n, w.keyA, w.valA, (unsigned long long *)w.vary, err);
        SS_LAUNCH_CHECK();
        // ---- on the host: the key bits that vary, and the column pointers,
        // which are checked here
        uint64_t vary = 0;
        SS_HIP_CHECK(hipMemcpyAsync(&vary, w.vary, sizeof(vary), hipMemcpyDeviceToHost, s));
        SS_HIP_CHECK(hipMemcpyAsync(cp_host.data(), col_ptr, sizeof(int64_t) * (size_t)(p + 1),
                                    hipMemcpyDeviceToHost, s));
        SS_HIP_CHECK(hipStreamSynchronize(s));
        if (cp_host[0] != 0 || cp_host[(size_t)p] != nnz) return SS_EINVAL;
        for (int64_t j = 0; j < p; ++j) {
            const int64_t a = cp_host[(size_t)j], b = cp_host[(size_t)j + 1];
            if (b < a || a < 0 || b > nnz) return SS_EINVAL;
        }

        // ---- ordering by decreasing time, stable in the subject index: the
        // upper 32 (n > kFewBits: 40) of the bits that vary, the rest within
        // the groups that agree in those, or, where one is not small, all
        const int high = vary ? 64 - __builtin_clzll(vary) : 0;
        const int bottom = vary ? __builtin_ctzll(vary) : 0;
        int low = bottom;
        const int bits = n <= kFewBits ? 32 : 40;
        if (!all_bits && high - bits > bottom) low = high - bits;
        uint64_t *ks;
        uint32_t *vs;
        rc = radix_sort(n, low, high, w, &ks, &vs, s);
        if (rc) return rc;
        uint64_t *key_s = ks == w.keyA ? w.keyB : w.keyA;
        const int check = low > bottom ? low : 0;
        if (packed)
            hipLaunchKernelGGL(k_after_sort<true>, dim3(grid_1d(n)), dim3(256), 0, s, n, check,
                               ks, vs, status, perm, inv_perm, key_s, w.st_s, err);
        else
            hipLaunchKernelGGL(k_after_sort<false>, dim3(grid_1d(n)), dim3(256), 0, s, n, check,
                               ks, vs, status, perm, inv_perm, key_s, w.st_s, err);
        SS_LAUNCH_CHECK();
        uint32_t found = 0;
        if (check) {
            SS_HIP_CHECK(hipMemcpyAsync(&found, err + 1, sizeof(found), hipMemcpyDeviceToHost, s));
            SS_HIP_CHECK(hipStreamSynchronize(s));
            if (found) continue;
        }

        // ---- tie runs and event counts; Fine-Gray: Kaplan-Meier G and the
        // weights
        const int64_t tiles = ceil_div(n, (int64_t)ST);
        const dim3 tg((unsigned)tiles);
        hipLaunchKernelGGL(k_runs_reduce, tg, dim3(SB), 0, s, n, (int)model, key_s, w.st_s,
                           w.sums, (uint8_t *)w.ev_bits);
        SS_LAUNCH_CHECK();
        if (tiles > ST) {
            hipLaunchKernelGGL((k_scan_spine<uint64_t, OpRun>), dim3(1), dim3(SB), 0, s, w.sums,
                               tiles);
            SS_LAUNCH_CHECK();
        }
        double *fac = (double *)ks;  // the sorted records have been read
        if (fg) {
            hipLaunchKernelGGL(k_runs_finish<true>, tg, dim3(SB), 0, s, n, (int)model, tiles,
                               key_s, w.st_s, w.sums, d8, d32, fac, w.prods);
            SS_LAUNCH_CHECK();
            if (tiles > ST) {
                hipLaunchKernelGGL((k_scan_spine<double, OpMul<double>>), dim3(1), dim3(SB), 0, s,
                                   w.prods, tiles);
                SS_LAUNCH_CHECK();
            }
            hipLaunchKernelGGL(k_km_weights, tg, dim3(SB), 0, s, n, tiles, fac, w.prods, w.st_s,
                               g_end, w_comp);
        } else {
            hipLaunchKernelGGL(k_runs_finish<false>, tg, dim3(SB), 0, s, n, (int)model, tiles,
                               key_s, w.st_s, w.sums, d8, d32, fac, w.prods);
        }
        SS_LAUNCH_CHECK();

        // ---- design: re-labelled to sorted positions, ascending inside columns
        host_list.clear();
        rc = run_design(n, p, nnz, cp_host.data(), col_ptr, rows, vals, inv_perm, w.ev_bits,
                        rows_sorted, vals_sorted, chunk_ptr, c, err, w.design, host_list, s);
        if (rc) return rc;

        // ---- data errors found on the device
        SS_HIP_CHECK(hipMemcpyAsync(&found, err, sizeof(found), hipMemcpyDeviceToHost, s));
        SS_HIP_CHECK(hipStreamSynchronize(s));
        return found ? SS_EINVAL : SS_OK;
    }
}

int32_t scan_add_u32_excl(const uint32_t *in, uint32_t *out, int64_t m, void *sums_raw,
                          hipStream_t s)
{
    if (m <= 0) return SS_OK;
    uint32_t *sums = (uint32_t *)sums_raw;
    const int64_t tiles = ceil_div(m, (int64_t)ST);
    hipLaunchKernelGGL(k_scan_reduce, dim3((unsigned)tiles), dim3(SB), 0, s, in, m, sums);
    SS_LAUNCH_CHECK();
    if (tiles > ST) {
        hipLaunchKernelGGL((k_scan_spine<uint32_t, OpAdd<uint32_t>>), dim3(1), dim3(SB), 0, s,
                           sums, tiles);
        SS_LAUNCH_CHECK();
    }
    hipLaunchKernelGGL(k_scan_down, dim3((unsigned)tiles), dim3(SB), 0, s, in, out, m, tiles, sums);
    SS_LAUNCH_CHECK();
    return SS_OK;
}

}  // namespace ss
