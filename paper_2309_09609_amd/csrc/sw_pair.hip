// One long pair (query x subject) scored by the whole GPU: the intra-task
// parallelism of Sec. II-B (processing elements share one matrix, Fig. 1) taken
// from one wave to many, as SW# does for one-to-one alignment of long sequences
// (Sec. III-A).
//
// Smith-Waterman with Gotoh gaps (Eq. 1-3) in int32 cells, E and F floored at
// 0 (H is unchanged by it, H >= 0 anyway), in bands of 256 rows (sw_bands.h).
// A step costs one column of the shorter sequence but a 64th part of 4 rows of
// the longer, so the longer one lies along the rows, whichever it is.  The
// profile of the band's rows sits in LDS as [residue][lane] dwords of four int8
// scores, so a step's lookup is conflict-free whatever the residues.  The best H
// of each band goes to the score with one atomic maximum.
//
// 20,001 x 19,500 residues: 10.6 -> 2.7 ms (143 GCUPS) against tiles of 256 x 256
// on one launch per anti-diagonal; 100,000 x 100,000: 54 -> 14.4 ms (693 GCUPS).
// 97 ns a step.  Against 2.9 and 15.0 ms then, 2 rows per lane measured 2.9 and
// 15.7 ms (500 x 40,000: 2.7 against 1.8), 16 columns per read of the band above
// 3.2 and 16.9 ms.
#include <hip/hip_runtime.h>

#include <stdint.h>

#include <algorithm>

#include "../../include/swsearch.h"
#include "sw_bands.h"
#include "sw_internal.h"

namespace sw {
sw_status report(sw_status s, const char* fmt, ...);
hipError_t launch_fill(int32_t* p, int64_t n, int32_t v, hipStream_t st);

constexpr int kPairRows = 4;                               // rows per lane
constexpr int kPairBand = 64 * kPairRows;                  // rows per band

struct PairArgs {
    const int8_t* rows;     // residue codes along the rows, m of them
    const int8_t* cols;     // along the columns, n
    const int8_t* sm;       // A x A substitution scores
    uint64_t* between;      // the row between two bands (sw_bands.h), all zeros
    int32_t* counter;       // bands taken, 0
    int32_t* best;          // the score
    int64_t m;
    int32_t n, nb;          // columns, bands
    int32_t A, go, ge;
    int32_t row_step, col_step;   // of a row's and a column's residue in sm
};

__global__ __launch_bounds__(64) void k_pair(PairArgs a) {
    __shared__ uint32_t prof[(kMaxAlphabet + 1) * 64];           // [residue code + 1][lane]; row 0 padding
    __shared__ uint4 rec[kBandBatch];
    __shared__ int8_t smat[kMaxAlphabet * kMaxAlphabet];
    const int b = threadIdx.x;
    for (int e = b; e < a.A * a.A; e += 64) smat[e] = a.sm[e];
    int S = 0;
    for (;;) {
        int band = 0;
        if (b == 0) band = atomicAdd(a.counter, 1);
        band = __builtin_amdgcn_readfirstlane(band);
        if (band >= a.nb) break;
        const int64_t r0 = (int64_t)band * kPairBand + kPairRows * b;          // this lane's first row
        __syncthreads();                                         // the matrix is in LDS, the last band's profile done with
        // profile: padding scores -128 on every row (a padded row or column never raises the score), rows past m too
        int at[kPairRows];
#pragma unroll
        for (int r = 0; r < kPairRows; ++r) at[r] = r0 + r < a.m ? a.rows[r0 + r] * a.row_step : -1;
        prof[b] = 0x80808080u;
        for (int c = 0; c < a.A; ++c) {
            uint32_t v = 0;
#pragma unroll
            for (int r = 0; r < kPairRows; ++r)
                v |= (uint32_t)(uint8_t)(at[r] >= 0 ? smat[at[r] + c * a.col_step] : (int8_t)-128) << (8 * r);
            prof[(c + 1) * 64 + b] = v;
        }
        __syncthreads();
        int H[kPairRows] = {}, E[kPairRows] = {}, diag = 0;
        sweep_band<16>(rec, prof, a.between, a.n, (uint32_t)band, band == a.nb - 1, b,
                   [&](int j) { return a.cols[j] + 1; },
                   [&](int, uint32_t pv, int htop, int ftop, int& hb, int& fb) {
                       int dg = diag, F = ftop;                  // ftop: F advanced to this lane's first row
#pragma unroll
                       for (int r = 0; r < kPairRows; ++r) {
                           const int hd = dg + (int)(int8_t)(pv >> (8 * r));
                           const int h = max(max(hd, E[r]), F);  // E, F >= 0: the local floor
                           S = max(S, h);
                           const int hgo = h - a.go;
                           E[r] = max(max(E[r] - a.ge, hgo), 0);
                           F = max(max(F - a.ge, hgo), 0);
                           dg = H[r];
                           H[r] = h;
                       }
                       diag = htop;
                       hb = H[kPairRows - 1];
                       fb = F;
                   });
        __syncthreads();                                         // every lane comes to the next pull with the others
    }
    for (int o = 32; o >= 1; o >>= 1) S = max(S, __shfl_xor(S, o, 64));
    if (b == 0 && S > 0) atomicMax(a.best, S);
}

}  // namespace sw

using namespace sw;

namespace {

struct PairLayout { int64_t counter, q, s, sm, fill_words, total; };

int64_t up256(int64_t x) { return (x + 255) / 256 * 256; }

// The row between bands and the counter first: one fill zeroes them.
PairLayout pair_layout(int64_t m, int64_t n) {
    PairLayout L{};
    L.counter = kBandColBytes * std::min(m, n);
    L.fill_words = (L.counter + 4) / 4;
    L.q = up256(L.counter + 4);
    L.s = up256(L.q + m);
    L.sm = up256(L.s + n);
    L.total = up256(L.sm + kMaxAlphabet * kMaxAlphabet);
    return L;
}

constexpr int kPairGrid = 1024;                   // waves: one on every SIMD of the GPU, more would only wait

}  // namespace

extern "C" {

sw_status sw_pair_workspace_bytes(int64_t qlen, int64_t slen, int64_t* bytes) {
    report(SW_OK, "");
    if (!bytes) return report(SW_E_INVALID, "bytes is NULL");
    if (qlen < 0 || slen < 0) return report(SW_E_INVALID, "lengths must be >= 0");
    if (qlen > ((int64_t)1 << 31) || slen > ((int64_t)1 << 31)) return report(SW_E_UNSUPPORTED, "longer than 2^31");
    *bytes = pair_layout(qlen, slen).total;
    return SW_OK;
}

sw_status sw_pair(const int8_t* h_query, int64_t qlen, const int8_t* h_subject, int64_t slen, int32_t alphabet,
                  const int8_t* h_subst, int32_t gap_open, int32_t gap_extend, int32_t* d_score, void* d_workspace,
                  int64_t ws_bytes, sw_stream stream) {
    report(SW_OK, "");
    if (!d_score) return report(SW_E_INVALID, "score is NULL");
    if (qlen < 0 || slen < 0) return report(SW_E_INVALID, "lengths must be >= 0");
    if ((qlen > 0 && !h_query) || (slen > 0 && !h_subject) || !h_subst) return report(SW_E_INVALID, "NULL input");
    if (qlen > ((int64_t)1 << 31) || slen > ((int64_t)1 << 31)) return report(SW_E_UNSUPPORTED, "longer than 2^31");
    const int A = alphabet > 0 ? alphabet : 20;
    if (A > kMaxAlphabet) return report(SW_E_INVALID, "alphabet must be 0 (= 20) or 1..%d", kMaxAlphabet);
    if (gap_open < 0 || gap_extend < 0) return report(SW_E_INVALID, "gap penalties must be >= 0");
    // int32 cells: the score is at most 127 x min(m, n)
    if (127 * std::min(qlen, slen) >= ((int64_t)1 << 31) - 1) return report(SW_E_UNSUPPORTED, "score may exceed int32");
    for (int64_t i = 0; i < qlen; ++i)
        if (h_query[i] < 0 || h_query[i] >= A) return report(SW_E_RESIDUE, "query residue at %lld outside 0..%d", (long long)i, A - 1);
    for (int64_t i = 0; i < slen; ++i)
        if (h_subject[i] < 0 || h_subject[i] >= A) return report(SW_E_RESIDUE, "subject residue at %lld outside 0..%d", (long long)i, A - 1);
    const PairLayout L = pair_layout(qlen, slen);
    if (qlen > 0 && slen > 0 && (!d_workspace || ws_bytes < L.total))
        return report(SW_E_SIZE, "workspace of %lld bytes < %lld needed", (long long)ws_bytes, (long long)L.total);
    if (d_workspace && (reinterpret_cast<uintptr_t>(d_workspace) & 255) != 0)
        return report(SW_E_INVALID, "workspace not 256-byte aligned");
    const hipStream_t st = static_cast<hipStream_t>(stream);
    hipError_t e = launch_fill(d_score, 1, 0, st);
    if (e != hipSuccess) return report(SW_E_HIP, "fill: %s", hipGetErrorString(e));
    if (qlen == 0 || slen == 0) return SW_OK;
    char* base = static_cast<char*>(d_workspace);
    const bool turn = qlen < slen;                    // the subject along the rows
    PairArgs a{};
    a.rows = reinterpret_cast<const int8_t*>(base + (turn ? L.s : L.q));
    a.cols = reinterpret_cast<const int8_t*>(base + (turn ? L.q : L.s));
    a.sm = reinterpret_cast<const int8_t*>(base + L.sm);
    a.between = reinterpret_cast<uint64_t*>(base);
    a.counter = reinterpret_cast<int32_t*>(base + L.counter);
    a.best = d_score;
    a.m = std::max(qlen, slen);
    a.n = (int32_t)std::min(qlen, slen);              // (below 2^24: the score fits 32 bits)
    a.nb = (int32_t)((a.m + kPairBand - 1) / kPairBand);
    a.A = A;
    a.go = gap_open;
    a.ge = gap_extend;
    a.row_step = turn ? 1 : A;
    a.col_step = turn ? A : 1;
    if ((e = hipMemcpyAsync(base + L.q, h_query, qlen, hipMemcpyHostToDevice, st)) != hipSuccess ||
        (e = hipMemcpyAsync(base + L.s, h_subject, slen, hipMemcpyHostToDevice, st)) != hipSuccess ||
        (e = hipMemcpyAsync(base + L.sm, h_subst, (size_t)A * A, hipMemcpyHostToDevice, st)) != hipSuccess ||
        (e = launch_fill(reinterpret_cast<int32_t*>(base), L.fill_words, 0, st)) != hipSuccess)
        return report(SW_E_HIP, "set-up: %s", hipGetErrorString(e));
    hipLaunchKernelGGL(k_pair, dim3(std::min(a.nb, kPairGrid)), dim3(64), 0, st, a);
    if ((e = hipGetLastError()) != hipSuccess) return report(SW_E_HIP, "pair launch: %s", hipGetErrorString(e));
    return SW_OK;
}

}  // extern "C"
