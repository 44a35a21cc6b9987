// All-to-all exchange between the workgroups of a cooperative launch: every
// workgroup publishes N values per round as tagged 16-byte words and reads
// everyone's (gathering in one workgroup and broadcasting back takes two
// round trips through the coherence point instead of one).  Slots alternate
// between two areas by round parity: a workgroup can be at most one round
// ahead of the slowest reader, as it needs everyone's publication of a round
// to go on.
#pragma once

#include "ss_device.h"

namespace ss {
namespace {

using namespace dev;

// One wave publishes t (the same in every lane) to COPIES slots, copy c at
// slot + c * copy_words: lane l stores word l mod NQ of copy l / NQ.
template <int N, int COPIES>
__device__ __forceinline__ void publish_slots(u32x4 *slot, int64_t copy_words,
                                              const double (&t)[N], uint64_t tag)
{
    constexpr int NQ = pub_words<N>();
    static_assert(NQ * COPIES <= kWave, "one wave stores every copy of a publication");
    const int lane = lane_id();
    u32x4 wd[NQ];
    pub_pack<N>(t, (uint32_t)tag, wd);
    const int word = lane % NQ;
    // (an empty asm statement per word: a select chain over the array
    // itself is folded into an indexed load from scratch)
    u32x4 x = wd[0];
#pragma unroll
    for (int c = 1; c < NQ; ++c) {
        u32x4 y = wd[c];
        asm volatile("" : "+v"(y));
        x = word == c ? y : x;
    }
    if (lane < NQ * COPIES) st_quad(slot + (int64_t)(lane / NQ) * copy_words + word, x);
}

// Thread t of `span` reads the publications t + k span (k < K; the last of
// G again past the end), STRIDE words apart in `area` of `words` words, until
// all carry the tag.  Returns false if the wait gave up or another
// workgroup's did.
template <int N, int STRIDE, int K>
__device__ __forceinline__ bool gather_slots(u32x4 *area, int words, WsHeader *hdr, int t,
                                             int span, int G, uint64_t tag, double (&v)[K][N])
{
    constexpr int NQ = pub_words<N>();
    static_assert(NQ <= STRIDE, "a slot holds a publication");
    const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(area, 0, words * 16, 0x00020000);
    int off[K];
#pragma unroll
    for (int k = 0; k < K; ++k) off[k] = min(t + k * span, G - 1) * (STRIDE * 16);
    uint32_t spins = 0;
    for (;;) {
        // agent-scope loads (sc1), read again on every pass
        u32x4 r[K][NQ];
#pragma unroll
        for (int k = 0; k < K; ++k)
#pragma unroll
            for (int c = 0; c < NQ; ++c)
                r[k][c] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, off[k] + 16 * c, 0, 16);
        asm volatile("" ::: "memory");
        bool ok = true;
#pragma unroll
        for (int k = 0; k < K; ++k) ok = ok && pub_tagged<NQ>(r[k], (uint32_t)tag);
        if (ok) {
#pragma unroll
            for (int k = 0; k < K; ++k) pub_unpack<N>(r[k], v[k]);
            return true;
        }
        if (((++spins & 31u) == 0 && ld_relaxed_u32(&hdr->error)) || spins > kSpinLimit) {
            __hip_atomic_store(&hdr->error, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            return false;
        }
        __builtin_amdgcn_s_sleep(1);
    }
}

// Sums over the publications in a fixed order, one wave's share into dst: of
// every value (mode[c] = 0), of those before segment b (1) or after it (2).
constexpr int kAll = 0, kBefore = 1, kAfter = 2;

template <int N, int STRIDE, int NS, int K>
__device__ __forceinline__ bool gather_sums(u32x4 *area, int words, WsHeader *hdr, int t,
                                            int span, int G, int64_t b, uint64_t tag,
                                            const int (&from)[NS], const int (&mode)[NS],
                                            double *dst)
{
    double s[NS];
#pragma unroll
    for (int c = 0; c < NS; ++c) s[c] = 0.0;
    bool ok = true;
    for (int t0 = t; ok && t0 - t < G; t0 += K * span) {  // K segments a thread at a time
        double v[K][N];
        ok = gather_slots<N, STRIDE, K>(area, words, hdr, t0, span, G, tag, v);
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const int64_t q = t0 + k * span;
#pragma unroll
            for (int c = 0; c < NS; ++c) {
                const bool in = ok && q < G &&
                                (mode[c] == kAll || (mode[c] == kBefore ? q < b : q > b));
                s[c] += in ? v[k][from[c]] : 0.0;
            }
        }
    }
    wave_sums_to<NS>(s, dst);
    return ok;
}

}  // namespace
}  // namespace ss
