// gfx950 kernels of libswsearch: the alignment behind a score (traceback).
//
// Only the top-ranked subjects of a search need their alignment (Sec. II-B);
// it is recovered by tracing back from the cell that holds the highest H.
// On a GPU with hundreds of GB of HBM the direct way pays: one pass over the
// (query x subject) matrix of Eq. 1-3 in 32-bit cells stores one direction
// byte per cell, and one wave then walks the bits back from the end cell.
//
// Fill.  The query is cut into bands of 128 rows, each swept by one wave (2 rows
// per lane, sw_bands.h): the bands of every pair of a launch are independent but
// for the row each hands to the band below it.  Bands are taken first bands of
// all pairs first, so that a wave rarely waits.  The direction bits of a lane's
// two rows form one 16-bit word per step, and the 64 lanes write 128
// consecutive bytes: word (band p, step t, lane b) at
// (p * band_steps(n) + t) * 64 + b.  Every band notes its first end cell.
//
// Walk.  One wave per pair copies the 128-byte step records of up to 256
// steps of the current band into LDS and follows the path through them until
// it leaves the copied steps; every move keeps or lowers the step index, so
// each copy serves dozens of moves.  The wave takes a run of equal moves (a
// diagonal stretch, a gap) at once: each lane checks one cell of the run and
// a ballot finds where it ends.
//
// Direction bits of cell (i, j), five of a lane's word (the lower row's in bits
// 0-4, the upper row's in bits 5-9), each the sign of a difference:
//   bit 4     H = 0: an alignment starts after this cell;
//   bit 3     H is above the diagonal H[i-1][j-1] + SM;
//   bit 2     H is above E;
//   bit 1     E[i][j] is above H[i][j-1] - Go: the horizontal gap was open before;
//   bit 0     F[i][j] is above H[i-1][j] - Go: the vertical gap was open before.
// H comes from the first of 0, the diagonal, E and F that equals it.  End cell:
// the first cell with H = S in row-major order.  These choices fix one alignment
// among those that reach S.
#include <hip/hip_runtime.h>

#include <stdint.h>

#include <climits>

#include <algorithm>

#include "sw_bands.h"
#include "sw_internal.h"

namespace sw {

constexpr int kAlignRows = 2;                    // query rows per lane
constexpr int kAlignBand = 64 * kAlignRows;      // query rows per band
constexpr int kTraceSteps = 256;                 // steps per LDS copy of the walk
constexpr int kAlignGrid = 2048;                 // waves of a fill: two to a SIMD issue nearly all the time

// (score desc, row asc, column asc): true if (s, i, j) comes before (t, k, l)
__device__ __forceinline__ bool end_before(int s, int i, int j, int t, int k, int l) {
    return s > t || (s == t && (i < k || (i == k && j < l)));
}

// The first end cell of the wave's lanes (score 0: none), in every lane.
__device__ __forceinline__ void first_end(int& sc, int& ci, int& cj) {
    for (int o = 1; o < 64; o <<= 1) {
        const int s2 = __shfl_xor(sc, o, 64), i2 = __shfl_xor(ci, o, 64), j2 = __shfl_xor(cj, o, 64);
        if (s2 > 0 && (sc == 0 || end_before(s2, i2, j2, sc, ci, cj))) { sc = s2; ci = i2; cj = j2; }
    }
}

// Fills the bands of all pairs of a launch.  E and F are not floored (only positive values lie on an alignment's
// path); before a lane's first column and past the last, padding's scores keep H at or below what the cells before
// it hold, so those cells are never a first end cell.
//
// A lone wave's issue rate bounds it, 21 instructions a cell: 8 for the cell, 10 for its direction bits (a difference
// and the shift of its sign into the word, each) and 3 for the end cell.  2 rows per lane: fewer than the 4 of
// sw_pair's cells, whose step would take as long as two of these, since the rows of a query are few (a query of 2,600
// residues has 21 bands).  Ten hits of each of eight queries of 144 to 2,600
// residues: 1,390 -> 415 us against a workgroup per pair whose waves kept a barrier every 128 steps (4 rows per lane, a
// byte of direction a cell); the whole call 1.81 -> 0.69 ms.
__global__ __launch_bounds__(64) void k_align_fill(const AlignPair* pairs, const AlignBand* bands, int nbands,
                                                   int32_t* counter, const int8_t* subst, int A, int go, int ge,
                                                   uint8_t* dirs, uint64_t* between, int32_t* ends) {
    __shared__ uint32_t prof[(kMaxAlphabet + 1) * 64];           // [image byte][lane]: the scores of the lane's rows
    __shared__ uint4 rec[kBandBatch];
    __shared__ int8_t sm[kMaxAlphabet * kMaxAlphabet];
    const int b = threadIdx.x;
    for (int e = b; e < A * A; e += 64) sm[e] = subst[e];
    for (;;) {
        int x = 0;
        if (b == 0) x = atomicAdd(counter, 1);
        x = __builtin_amdgcn_readfirstlane(x);
        if (x >= nbands) break;
        const AlignBand J = bands[x];
        const AlignPair P = pairs[J.pair];
        const int m = P.m, n = P.n;
        const int row0 = J.band * kAlignBand + b * kAlignRows;   // 0-based first row of this lane
        __syncthreads();                                         // the matrix is in LDS, the last band's profile done with
        int qa[kAlignRows];                                      // matrix row offset of each query row, -1 past the query
#pragma unroll
        for (int r = 0; r < kAlignRows; ++r) qa[r] = row0 + r < m ? P.query[row0 + r] * A : -1;
        // padding -128 on every row; rows past the query score 0 (they never end an alignment)
        prof[b] = 0x80808080u;
        for (int d = 0; d < A; ++d) {
            uint32_t v = 0;
#pragma unroll
            for (int r = 0; r < kAlignRows; ++r)
                if (qa[r] >= 0) v |= (uint32_t)(uint8_t)sm[qa[r] + d] << (8 * r);
            prof[(d + 1) * 64 + b] = v;
        }
        __syncthreads();
        int H[kAlignRows], G[kAlignRows], E[kAlignRows], bs[kAlignRows], bj[kAlignRows];    // G = H - Go
#pragma unroll
        for (int r = 0; r < kAlignRows; ++r) {
            H[r] = E[r] = bj[r] = 0;
            G[r] = -go;
            bs[r] = qa[r] >= 0 ? 0 : INT_MAX;                    // rows past the query never become the best
        }
        int diag = 0;                                            // H of the row above this lane's block, previous column
        // (a global pointer: flat loads would hold up the reads of LDS behind them)
        const auto residues = (const __attribute__((address_space(1))) uint8_t*)P.residues;
        uint16_t* dir = reinterpret_cast<uint16_t*>(dirs + P.dir_off) + (int64_t)J.band * band_steps(n) * 64;
        sweep_band<0>(rec, prof, between + 2 * P.bnd_off, n, (uint32_t)J.band, row0 - b * kAlignRows + kAlignBand >= m, b,
                   [&](int j) { return residues[(int64_t)(j >> 2) * kChunkBytes + (j & 3)]; },
                   [&](int t, uint32_t sv, int htop, int ftop, int& hb, int& fb) {
                       int dg = diag, gu = htop - go, fu = ftop;
                       uint32_t word = 0;
#pragma unroll
                       for (int r = 0; r < kAlignRows; ++r) {
                           const int eo = G[r], ee = E[r] - ge;
                           const int e = max(eo, ee);                       // Eq. 2
                           const int fe = fu - ge;
                           const int f = max(gu, fe);                       // Eq. 3
                           const int hd = dg + (int)(int8_t)(sv >> (8 * r));
                           const int h = max(max(hd, e), max(f, 0));        // Eq. 1
                           auto sign = [&](int v) { word = __builtin_amdgcn_alignbit(word, (uint32_t)v, 31); };
                           sign(h - 1);
                           sign(hd - h);
                           sign(e - h);
                           sign(eo - ee);
                           sign(gu - fe);
                           if (h > bs[r]) { bs[r] = h; bj[r] = t - b + 1; }
                           dg = H[r];
                           H[r] = h;
                           G[r] = gu = h - go;
                           E[r] = e;
                           fu = f;
                       }
                       diag = htop;
                       hb = H[kAlignRows - 1];
                       fb = fu;
                       dir[(uint32_t)t * 64u + (uint32_t)b] = (uint16_t)word;
                   });
        // the band's first end cell
        int sc = 0, ci = 0, cj = 0;
#pragma unroll
        for (int r = 0; r < kAlignRows; ++r)
            if (qa[r] >= 0 && bs[r] > 0 && end_before(bs[r], row0 + r + 1, bj[r], sc, ci, cj)) {
                sc = bs[r];
                ci = row0 + r + 1;
                cj = bj[r];
            }
        first_end(sc, ci, cj);
        // (every lane writes: joined with the pull above, a store of lane 0's alone lets the other lanes go on without
        // it, to band 0 again)
        int32_t* o = ends + 3 * (int64_t)(P.ends + J.band);
        o[0] = sc;
        o[1] = ci;
        o[2] = cj;
        __syncthreads();
    }
}

// One wave per pair: find its first end cell and walk the direction bits back
// from it, through LDS copies of up to kTraceSteps step records of the band it
// is in, a run of equal moves at a time; the word of (row rb of the band,
// 0-based column c) sits at (c + rb / 2 - t0) * 64 + rb / 2 in a copy that
// starts at step t0.  Operations, last to first, collect in LDS and the wave writes
// them out after each copy, from the end of the pair's space down; begin positions and the count go to
// info[4 * pair] = (q_begin, s_begin, count, status).
constexpr int kTraceOps = 1024;                  // operations buffered in LDS per copy

__global__ __launch_bounds__(64) void k_align_trace(const AlignPair* pairs, const uint8_t* dirs, const int32_t* ends,
                                                    int32_t* best, char* ops, int64_t ops_stride, int64_t* info) {
    __shared__ __attribute__((aligned(16))) uint16_t tile[kTraceSteps * 64];
    __shared__ char obuf[kTraceOps];
    __shared__ int64_t walk[7];                 // i, j, len, state, done, status, buffered operations
    const int k = blockIdx.x;
    const int lane = threadIdx.x;
    const AlignPair P = pairs[k];
    const int n = P.n, m = P.m;
    const int64_t nsteps = band_steps(n);
    const uint8_t* dir = dirs + P.dir_off;
    char* out = ops + (int64_t)k * ops_stride;
    int sc = 0, i = 0, j = 0;
    const int nb = n > 0 ? (m + kAlignBand - 1) / kAlignBand : 0;
    for (int x = lane; x < nb; x += 64) {
        const int32_t* o = ends + 3 * (int64_t)(P.ends + x);
        if (o[0] > 0 && (sc == 0 || end_before(o[0], o[1], o[2], sc, i, j))) { sc = o[0]; i = o[1]; j = o[2]; }
    }
    first_end(sc, i, j);
    if (lane == 0) {
        best[3 * k] = sc;
        best[3 * k + 1] = i;
        best[3 * k + 2] = j;
    }
    int64_t len = 0;
    int state = 0;                              // 0: H, 1: E, 2: F
    int64_t status = 0;
    bool done = sc <= 0;
    if (done) {
        i = 0;
        j = 0;
    }
    while (!done) {                             // wave-uniform
        if (i < 1 || j < 1 || i > m || j > n || len >= ops_stride) {
            if (state != 0) status = 1;         // a gap cannot reach the border: inconsistent bytes
            break;
        }
        const int row = i - 1;
        const int p = row / kAlignBand;
        const int t = j - 1 + (row % kAlignBand) / kAlignRows;
        const int t0 = max(0, t - kTraceSteps + 1);
        // step records t0 .. t of band p: (t - t0 + 1) * 128 contiguous bytes
        const uint4* src = reinterpret_cast<const uint4*>(dir + (p * nsteps + t0) * 128);
        const int words = (t - t0 + 1) * 8;
        for (int x = lane; x < words; x += 64) reinterpret_cast<uint4*>(tile)[x] = src[x];
        __syncthreads();
        {
            // the wave follows runs of equal moves: lane k looks at the k-th cell of the run (down the
            // diagonal in H, along the row in E, up the column in F) and the first lane whose cell ends
            // the run, or lies outside the copy, the band, the matrix or the room left, decides
            int rb = row - p * kAlignBand;      // row within the band
            int c = j - 1;                      // 0-based column
            int cnt = 0;
            const int64_t room = ops_stride - len;
            const int cap = room < kTraceOps ? (int)room : kTraceOps;
            for (;;) {
                const int rk = state == 1 ? rb : rb - lane;
                const int ck = state == 2 ? c : c - lane;
                const int tk = ck + (rk >> 1);
                const bool ok = rk >= 0 && ck >= 0 && tk >= t0 && cnt + lane < cap;
                const uint32_t v = ok ? (uint32_t)tile[(tk - t0) * 64 + (rk >> 1)] >> (rk & 1 ? 0 : 5) : 0u;
                // a run ends where H does not come from the diagonal, or where the gap opens
                const bool stop = !ok || (state == 0 ? (v & 0x18u) != 0u : (v & (state == 1 ? 2u : 1u)) == 0u);
                const uint64_t mask = __ballot(stop);
                const int K = mask ? (int)__builtin_ctzll(mask) : 64;
                const bool okK = K < 64 && __shfl((int)ok, K, 64) != 0;
                const uint32_t vK = (uint32_t)__shfl((int)v, K < 64 ? K : 0, 64);
                if (state == 0) {
                    if (lane < K) obuf[cnt + lane] = 'M';
                    cnt += K;
                    rb -= K;
                    c -= K;
                    if (K == 64) continue;
                    if (!okK) break;                             // the outer loop decides
                    if (vK & 0x10u) { done = true; break; }
                    state = vK & 4u ? 2 : 1;
                } else {
                    const char op = state == 1 ? 'D' : 'I';
                    const int moves = okK ? K + 1 : K;           // the gap's opening cell is its last move
                    if (lane < moves) obuf[cnt + lane] = op;
                    cnt += moves;
                    if (state == 1) c -= moves; else rb -= moves;
                    if (okK) state = 0;
                    else if (K < 64) break;                      // the outer loop decides
                }
            }
            if (lane == 0) {
                walk[0] = rb + p * kAlignBand + 1;
                walk[1] = c + 1;
                walk[2] = len + cnt;
                walk[3] = state;
                walk[4] = done;
                walk[5] = status;
                walk[6] = cnt;
            }
        }
        __syncthreads();
        const int cnt = (int)walk[6];
        for (int x = lane; x < cnt; x += 64) out[ops_stride - 1 - len - x] = obuf[x];
        i = (int)walk[0];
        j = (int)walk[1];
        len = walk[2];
        state = (int)walk[3];
        done = walk[4] != 0;
        status = walk[5];
        __syncthreads();                        // everyone has read the state and the buffer before the next copy
    }
    if (lane == 0) {
        info[4 * k] = i;
        info[4 * k + 1] = j;
        info[4 * k + 2] = len;
        info[4 * k + 3] = status;
    }
}

// The fill of the pairs' bands; counter is 0 and every word of `between` too.
hipError_t launch_align_fill(const AlignPair* pairs, const AlignBand* bands, int nbands, int32_t* counter,
                             const int8_t* subst, int A, int go, int ge, uint8_t* dirs, uint64_t* between, int32_t* ends,
                             hipStream_t st) {
    if (nbands <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_align_fill, dim3(std::min(nbands, kAlignGrid)), dim3(64), 0, st, pairs, bands, nbands, counter,
                       subst, A, go, ge, dirs, between, ends);
    return hipGetLastError();
}

hipError_t launch_align_trace(const AlignPair* pairs, int npairs, const uint8_t* dirs, const int32_t* ends, int32_t* best,
                              char* ops, int64_t ops_stride, int64_t* info, hipStream_t st) {
    if (npairs <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_align_trace, dim3(npairs), dim3(64), 0, st, pairs, dirs, ends, best, ops, ops_stride, info);
    return hipGetLastError();
}

int align_bands(int m, int64_t n) { return n > 0 ? (m + kAlignBand - 1) / kAlignBand : 0; }

int64_t align_dir_bytes(int m, int64_t n) { return ((m + kAlignBand - 1) / kAlignBand) * band_steps(n) * 128; }

}  // namespace sw
