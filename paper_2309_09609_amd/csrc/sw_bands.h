// One matrix of Eq. 1-3 swept by bands of query rows, a wave to a band, the
// bands running behind one another on as many waves as the GPU holds: the
// intra-task parallelism of Sec. II-B (processing elements share one matrix,
// Fig. 1) for a single long pair and for the traceback fills.
//
// Lane b of a wave owns R rows and at step t updates column t - b; the bottom
// row of lane b reaches lane b + 1 through a DPP shift, and lane 63's goes to
// the band below through global memory, 16 bytes a column: two 8-byte words
// {H, tag}, {F, tag}.  The tag is the number of the band that reads them, so a
// word says by itself whether it is there: the reader polls the words, and no
// fence, flag or launch orders the two.  (Words start out with tag 0; a band
// overwrites a column only after it has read it, and only the band below it
// looks for the new tag.)  Both sides use single 8-byte accesses at device
// scope, past the XCDs' own caches.
//
// Every wait ends: bands are taken from a counter in order, a band waits only
// for the band before it, and the first waits for none, so whichever waves
// happen to run, the lowest band taken always goes on.
//
// A reader takes 32 columns at a time (lane l: word l of the 64) and asks for
// the next 32 at step kAsk of these, so a band runs about 64 + 64 - kAsk + the
// time a word is on its way, some 130 steps, behind the band above.  Asking half
// way gains where few bands wait (sw_pair, 20,000 x 20,000: 2.90 ms from the
// start, 2.75 at step 8, 2.72 at 16, 2.68 at 24; 100,000: 15.1, 14.6, 14.4, 14.6);
// the traceback's many bands find their words late then (0.70 ms a call from the
// start, 0.71 at 16, 0.77 at 24).  A matrix of m
// rows and n columns takes n + m / (64 R) x 130 steps of a lone wave, where one
// launch per anti-diagonal of tiles (256 rows x 256 columns) took (m + n) / 256
// launches of 320 steps each.
//
// Bound by a lone wave's issue rate, one instruction in about 2 ns.
#pragma once

#include <hip/hip_runtime.h>

#include <stdint.h>

namespace sw {

constexpr int kBandBatch = 32;                   // columns per read of the band above, two words each: 64 lanes
constexpr int64_t kBandColBytes = 16;            // of the row between two bands, per column

// Steps of a band of n columns: the 64 lanes' skew, rounded up to whole batches.
__host__ __device__ constexpr int64_t band_steps(int64_t n) { return (n + 63 + kBandBatch - 1) / kBandBatch * kBandBatch; }

typedef __amdgpu_buffer_rsrc_t band_rsrc;

__device__ __forceinline__ band_rsrc band_buffer(void* base, uint32_t bytes) {
    const uint64_t p = (uint64_t)base;
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)p), hi = __builtin_amdgcn_readfirstlane((uint32_t)(p >> 32));
    return __builtin_amdgcn_make_buffer_rsrc((void*)(((uint64_t)hi << 32) | lo), (short)0,
                                             (int)__builtin_amdgcn_readfirstlane(bytes), 0x00020000);
}

// Lane b - 1's v; lane 0 takes `first`.
__device__ __forceinline__ int from_above(int v, int first) {
    return __builtin_amdgcn_update_dpp(first, v, 0x138, 0xf, 0xf, false);      // wave_shr:1
}

// One band of n columns.  rec: 32 records in LDS; prof: the band's profile in LDS, [image byte][lane] dwords of R
// scores (image byte 0: padding); tag: the band's number, 0 for the first; row: the words between bands; last: nothing
// reads the bottom row.  code(j) is the image byte of column j < n; cells(t, scores, htop, ftop, &hb, &fb) updates the
// lane's R rows at its column t - b (before column 0 and from n on, scores are padding's and the tops zero or the
// band's own) and hands back the bottom row.
template <int kAsk, class Code, class Cells>
__device__ __forceinline__ void sweep_band(uint4* rec, const uint32_t* prof, uint64_t* row, int n, uint32_t tag, bool last,
                                           int b, Code&& code, Cells&& cells) {
    const int col = b & (kBandBatch - 1), half = b / kBandBatch;
    const int nbatch = (int)(band_steps(n) / kBandBatch);
    auto words = [&](int c) -> uint64_t {
        const int j = kBandBatch * c + col;
        if (tag == 0 || j >= n) return (uint64_t)tag << 32;
        return __hip_atomic_load(row + 2 * (int64_t)j + half, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
    // offset of column j's scores in the profile
    auto at = [&](int j) -> int { return j < n ? (int)code(j) * 256 : 0; };
    const band_rsrc out = band_buffer(row, (uint32_t)(kBandColBytes * n));
    // lane 63's bottom row of step t is column t - 63's; every other offset lies past the row, where nothing is written
    uint32_t to = b == 63 && !last ? (uint32_t)(-63 * kBandColBytes) : 0x80000000u;
    const char* mine = reinterpret_cast<const char*>(prof + b);
    auto scores = [&](int o) { return *reinterpret_cast<const uint32_t*>(mine + o); };
    // residues run two columns ahead of the cells, their scores one: ro is the offset of column t + 1 - b's
    int ro = at(b == 0 ? 1 : 0);
    uint32_t pv = scores(b == 0 ? at(0) : 0);
    if (b > 1) ro = 0;
    uint32_t pn = scores(ro);
    uint64_t v = words(0);
    int next = half == 0 ? at(2 + col) : 0;
    int hb = 0, fb = 0;
    for (int c = 0; c < nbatch; ++c) {
        while (__ballot((uint32_t)(v >> 32) != tag)) {
            __builtin_amdgcn_s_sleep(1);
            v = words(c);
        }
        reinterpret_cast<uint32_t*>(rec)[4 * col + half] = (uint32_t)v;
        if (half == 0) reinterpret_cast<uint32_t*>(rec)[4 * col + 2] = (uint32_t)next;
        next = half == 0 ? at(kBandBatch * (c + 1) + 2 + col) : 0;
        __builtin_amdgcn_wave_barrier();
        uint4 r = rec[0];
#pragma unroll
        for (int u = 0; u < kBandBatch; ++u) {
            const uint4 rn = rec[u + 1 < kBandBatch ? u + 1 : u];
            if (u == kAsk) v = words(c + 1);
            ro = from_above(ro, (int)r.z);
            const uint32_t pnn = scores(ro);
            const int htop = from_above(hb, (int)r.x), ftop = from_above(fb, (int)r.y);
            cells(kBandBatch * c + u, pv, htop, ftop, hb, fb);
            typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
            const u32x4 w = {(uint32_t)hb, tag + 1, (uint32_t)fb, tag + 1};
            __builtin_amdgcn_raw_buffer_store_b128(w, out, to, 0, 16);         // (16: sc1, device scope)
            to += (uint32_t)kBandColBytes;
            pv = pn;
            pn = pnn;
            r = rn;
        }
        __builtin_amdgcn_wave_barrier();
    }
}

}  // namespace sw
