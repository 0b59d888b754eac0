// Host side of libswsearch: the C ABI declared in include/swsearch.h.
//
// sw_db_pack sorts subjects by length (descending, ties by index), cuts the
// sorted list into groups of 128 and interleaves each group so that one wave
// reads 4 columns of 128 subjects as 512 contiguous bytes (one dwordx2 per lane).
//
// A search is planned on the host: every group gets a lane-cooperation degree
// B (1 = one pair of subjects per lane, 64 = a whole wave on one pair) so that
// no work unit is large against a persistent wave's share of the search, units
// are bundled four to a workgroup and ordered longest first, and one persistent
// launch pulls them from an atomic counter.  Pairs that would outlast the
// search run on a workgroup each, or several, first.  Pairs whose 16-bit score
// saturates are appended to a list that a 32-bit launch consumes.  The launch
// sequence itself allocates nothing, so the batched form captures a batch
// shape that comes twice in a row as a HIP graph and replays it.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <map>
#include <mutex>
#include <numeric>
#include <string>
#include <vector>

#include "../../include/swsearch.h"
#include "sw_internal.h"

namespace sw {
hipError_t launch_sweep(int form, int R, const SweepArgs& a, int grid, hipStream_t st);
hipError_t sweep_occupancy(int form, int R, int* blocks_per_cu);
hipError_t launch_sweep_q2(int form, int R, const SweepArgs& a, int grid, hipStream_t st);
hipError_t sweep_occupancy_q2(int form, int R, int* blocks_per_cu);
hipError_t launch_sweep_mode(int mode, int R, const SweepArgs& a, int grid, hipStream_t st);
hipError_t launch_sweep_mode16(int mode, int R, const SweepArgs& a, int grid, hipStream_t st);
hipError_t launch_sweep_mode_off(int mode, int R, const SweepArgs& a, int grid, hipStream_t st);
hipError_t sweep_occupancy_mode16(int mode, int R, int* blocks_per_cu);
hipError_t launch_align_fill(const AlignPair* pairs, const AlignBand* bands, int nbands, int32_t* counter,
                             const int8_t* subst, int A, int go, int ge, uint8_t* dirs, uint64_t* between, int32_t* ends,
                             hipStream_t st);
hipError_t launch_align_trace(const AlignPair* pairs, int npairs, const uint8_t* dirs, const int32_t* ends, int32_t* best,
                              char* ops, int64_t ops_stride, int64_t* info, hipStream_t st);
int align_bands(int m, int64_t n);
int64_t align_dir_bytes(int m, int64_t n);
hipError_t launch_profile(const int8_t* stage, int A, const QDesc* qd, int nq, const int64_t* qoff, int16_t* prof,
                          int32_t* counters, int ncounters, uint32_t* bits, int64_t nbits_words, int max_mp,
                          hipStream_t st, int add, int pad);
hipError_t launch_interleave(const int8_t* res, const int64_t* soff, const int32_t* slen, int64_t n, int A,
                             const GroupRec* groups, const int64_t* gdw, int ngroups, uint32_t* image,
                             int64_t total_dw, int32_t* err, hipStream_t st);
hipError_t launch_topk_ws(const int32_t* scores, int64_t n, int64_t row_stride, int rows, int k, int32_t* top_s,
                          int64_t* top_i, void* ws, hipStream_t st);
int64_t topk_ws_bytes(int64_t n, int rows, int k);
hipError_t launch_topk(const int32_t* scores, int64_t n, int64_t row_stride, int rows, int k, int32_t* top_s,
                       int64_t* top_i, hipStream_t st);
hipError_t launch_fill(int32_t* p, int64_t n, int32_t v, hipStream_t st);
}  // namespace sw

using namespace sw;

namespace {

thread_local std::string g_err;

sw_status fail(sw_status s, const char* fmt, ...) {
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    g_err = buf;
    return s;
}

#define HIP_TRY(expr)                                                                          \
    do {                                                                                       \
        hipError_t e_ = (expr);                                                                \
        if (e_ != hipSuccess) return fail(SW_E_HIP, "%s: %s", #expr, hipGetErrorString(e_));   \
    } while (0)

// Device buffer that grows on demand (contents are not preserved).  Every
// reallocation bumps *gen, which invalidates captured graphs.
struct DevBuf {
    void* p = nullptr;
    size_t bytes = 0;
    hipError_t reserve(size_t want, uint64_t* gen = nullptr) {
        if (want <= bytes && p) return hipSuccess;
        if (p) { hipFree(p); p = nullptr; bytes = 0; }
        const size_t sz = std::max<size_t>(want, 256);
        hipError_t e = hipMalloc(&p, sz);
        if (e == hipSuccess) bytes = sz;
        if (gen) ++*gen;
        return e;
    }
    void release() { if (p) hipFree(p); p = nullptr; bytes = 0; }
    template <class T> T* as() const { return static_cast<T*>(p); }
};

constexpr int kStageRing = 4;         // pinned staging buffers per handle

// Pinned staging buffer; the event marks completion of the last copy out of it.
struct HostPinned {
    void* p = nullptr;
    size_t bytes = 0;
    hipEvent_t done = nullptr;
    bool pending = false;
    hipError_t reserve(size_t want) {
        if (pending) { hipEventSynchronize(done); pending = false; }
        if (want <= bytes && p) return hipSuccess;
        if (p) { hipHostFree(p); p = nullptr; bytes = 0; }
        const size_t sz = std::max<size_t>(want, 4096);
        hipError_t e = hipHostMalloc(&p, sz, hipHostMallocDefault);
        if (e == hipSuccess) bytes = sz;
        return e;
    }
    void release() {
        if (pending) hipEventSynchronize(done);
        if (p) hipHostFree(p);
        if (done) hipEventDestroy(done);
        p = nullptr; done = nullptr; bytes = 0; pending = false;
    }
};

constexpr double kUnitShare = 0.25;   // see plan_units

// Work items of one search, run by one launch: the chained pairs (a workgroup
// each) and the bulk on offset cells; on plain cells the bulk alone, long pairs
// among it.  Searches on the handle's own workspace read the items from device
// copies made once; searches on a caller's workspace upload them with the
// queries.  That workspace has room for the offset cells' plan (sw_batch_workspace_bytes
// does not know the scoring) and some more; should the plain cells' not fit, they
// run the offset cells' one, the chained pairs on a wave each (unchained) ahead of the bulk.
struct Plan {
    std::vector<WgItem> h_items;  // [chained..., bulk..., unchained...]
    std::vector<int2> h_pairs;    // query pairs (query a, query b or -1) when qpack
    int32_t n_chain = 0, n_main = 0, n_unchained = 0;
    int32_t n_small = 0, n_small_unchained = 0;   // of these at 4 rows per lane
    int R_main = 16;
    bool qpack = false;           // items index query pairs (two queries per lane)
    DevBuf items, qpairs;         // device copies (handle workspace only)
    bool on_device = false;
    void release() { items.release(); qpairs.release(); on_device = false; }
    void clear() {
        release();
        h_items.clear();
        n_chain = n_main = n_unchained = n_small = n_small_unchained = 0;
    }
};

// What a plan is made for: offset cells, whose chained pairs may be cut into windows of the subject and parts; the same
// planned alike, but without the parts (gaps that extend for nothing: an alignment may cover the whole subject, so that
// every part would sweep all columns before its own too, eight of them 4.5 times the pair's, and the last end no
// sooner); offset cells of whole subjects (global scores); plain cells.
enum PlanKind { kPlanCut, kPlanOnePart, kPlanWhole, kPlanPlain };
constexpr int kPlanKinds = 4;

// Device pointers of the staged queries (descriptors, offsets, matrix + residues).
struct Staged {
    const QDesc* qd = nullptr;
    const int64_t* qoff = nullptr;
    const int8_t* sm_q = nullptr;
    int nq = 0;
    int max_mp = 0;
};

// The 16-bit cells of one search: their form and what the kernels are told about it.
struct CellForm {
    int cell = kCellI16;          // kCellI16 or kCellOff
    int32_t mode = SW_LOCAL;      // end-to-end modes: offset cells here, the others through their own launches
    int32_t bias = 0;             // plain cells: minus the lowest substitution score, at least 0; end-to-end modes: what
                                  // every value carries
    int32_t pad = kPadScore;      // what the profile holds for padding
    int32_t off_k = 0;            // offset cells: steps between renormalisations
    int32_t add = 0;              // offset cells: the profile holds SM + add
    int32_t sat = kSat16;         // scores (as the cells hold them) from here on are recomputed
    bool operator==(const CellForm& o) const {
        return cell == o.cell && mode == o.mode && bias == o.bias && pad == o.pad && off_k == o.off_k && add == o.add && sat == o.sat;
    }
};

struct GraphEntry {
    std::vector<int> qlens;
    int32_t go = 0, ge = 0, k = 0;
    CellForm form;
    const void* scores = nullptr;
    const void* top_s = nullptr;
    const void* top_i = nullptr;
    hipStream_t stream = nullptr;
    uint64_t gen = 0;
    const void* ws = nullptr;         // workspace base the sequence was captured with
    hipGraph_t graph = nullptr;
    hipGraphExec_t exec = nullptr;
    hipEvent_t done = nullptr;        // recorded after every launch of exec
    bool launched = false;
    void clear() {
        if (exec && launched && done) hipEventSynchronize(done);   // the last launch may still run
        if (exec) hipGraphExecDestroy(exec);
        if (graph) hipGraphDestroy(graph);
        exec = nullptr;
        graph = nullptr;
        launched = false;
        qlens.clear();
    }
};

// The inputs that decide a batched launch sequence; a shape is captured into a graph the second time
// it comes in a row (one-off shapes, e.g. served batches, are enqueued directly and never wait).
struct BatchKey {
    std::vector<int> qlens;
    int32_t go = 0, ge = 0, k = 0;
    CellForm form;
    const void* scores = nullptr;
    const void* top_s = nullptr;
    const void* top_i = nullptr;
    hipStream_t stream = nullptr;
    uint64_t gen = 0;
    const void* ws = nullptr;
    bool operator==(const BatchKey& o) const {
        return qlens == o.qlens && go == o.go && ge == o.ge && k == o.k && form == o.form && scores == o.scores &&
               top_s == o.top_s && top_i == o.top_i && stream == o.stream && gen == o.gen && ws == o.ws;
    }
};

int64_t round_up(int64_t x, int64_t a) { return (x + a - 1) / a * a; }

// 64-bit hash of offsets[0..n]: every value through the splitmix64 finaliser, combined with its
// position, so a changed, moved or swapped boundary changes it.
uint64_t offsets_hash(const int64_t* offsets, int64_t n) {
    uint64_t h = 0x243F6A8885A308D3ull ^ (uint64_t)n;
    for (int64_t k = 0; k <= n; ++k) {
        uint64_t x = (uint64_t)offsets[k] + 0x9E3779B97F4A7C15ull * (uint64_t)(k + 1);
        x = (x ^ (x >> 30)) * 0xBF58476D1CE4E5B9ull;
        x = (x ^ (x >> 27)) * 0x94D049BB133111EBull;
        h = (h ^ (x ^ (x >> 31))) * 0x100000001B3ull;
    }
    return h;
}

}  // namespace

struct sw_db {
    int device = 0;
    int64_t n = 0;
    int64_t total_res = 0;
    int64_t off_first = 0, off_last = 0;
    uint64_t off_hash = 0;            // offsets_hash of the offsets the image was packed with
    int ngroups = 0;
    std::vector<int32_t> ncols;       // per group
    std::vector<int32_t> pcols;       // per pair: longest subject of the pair, rounded up to 4
    int32_t ncols_max = 0;
    // The packed image: one device allocation, the handle's own (image_own) or the caller's
    // (sw_db_pack_into), laid out by DbLayout.
    DevBuf image_own;
    bool caller_image = false;
    uint8_t* d_image = nullptr;       // interleaved residues
    GroupRec* d_groups = nullptr;
    int32_t* d_perm = nullptr;        // sorted slot -> original subject index, -1 for padding slots
    int32_t* d_pair_cols = nullptr;   // per pair: longest subject of the pair, rounded up to 4
    int32_t* d_slen = nullptr;        // subject length per sorted slot (end-to-end modes), 0 for padding
    int64_t image_bytes = 0;
    // per original subject: length and sorted slot; per group: byte offset in the image (alignments)
    std::vector<int32_t> lens, slot_of;
    std::vector<int64_t> gbase;
    DevBuf align_dirs, align_bnd, align_misc;              // traceback workspace
    HostPinned align_host;            // what goes to the device and comes back, up to kAlignPinned bytes
    int wg_mode = 0;                  // persistent workgroups of an end-to-end sweep
    Plan mode_plan;
    int mode_side_rows = 16;          // end-to-end modes: rows per lane of the long pairs' launch
    // launch geometry
    int cus = 0, wg16 = 0, wg32 = 0;  // scratch slots (workgroups) of the 16-bit sweeps; 32-bit grid
    int wgR[17] = {0};                // persistent workgroups per 16-bit instance, by R
    int wgQ[17] = {0};                // persistent workgroups per query-pair instance, by R
    int64_t slot_cap = 0;             // (column x pair) capacity of one wave's boundary slot
    hipStream_t side = nullptr;       // end-to-end modes on plain cells: the long pairs of short queries
    hipStream_t side2 = nullptr;      // and the 32-bit groups beside both 16-bit launches
    hipStream_t cap = nullptr;        // stream the batched sequence is captured on
    hipEvent_t ev_fork = nullptr, ev_join = nullptr, ev_join2 = nullptr;
    // workspace of searches without a caller workspace (laid out by WsLayout)
    uint64_t gen = 1;                 // bumped on every workspace reallocation
    DevBuf ws_own;
    // pinned staging of the queries (and, on a caller's workspace, the plan), a ring so that a call
    // reuses a buffer only once the copy of the call kStageRing before it has run
    HostPinned hstage[kStageRing];
    int hstage_next = 0;
    std::map<int64_t, Plan> plans;    // query length and kind -> plan of one query
    Plan batch_plan[kPlanKinds], multi_plan;
    std::vector<int> batch_qlens[kPlanKinds];
    GraphEntry graph;                 // batched form: last captured shape
    BatchKey last_eager;              // batched form: the last shape enqueued without a graph
    // tuning knobs and test hooks
    int force_lgB = -1;               // fixed lanes per pair
    int force_R = 0;                  // fixed rows per lane (4, 8, 16)
    double unit_share = kUnitShare;   // largest unit / one wave's share of a search
    bool fixed_share = false;         // it was set: no other is tried
    int32_t sat = kSat16;             // rerun threshold
    int64_t rerun_cap_hook = 0;       // test hook: list capacity of the recompute (0 = default)
    int poison = 0;                   // test hook: flagged pairs' 16-bit scores read kPoison
    int lane_pack = 1;                // 1: subject pairs per lane; 2: query pairs per lane (several queries)
    int alphabet = 20;                // residue codes 0..alphabet-1; matrices are alphabet x alphabet
    // statistics and timing
    int last_items = 0, last_rows = 16, last_grid = 0, last_side_items = 0, last_side_rows = 0;
    int64_t last_cap = 0;             // list capacity of the last search's recompute
    const int32_t* last_counters = nullptr;   // device counters of the last search (its workspace)
    bool timing = false;
    std::vector<std::pair<hipEvent_t, hipEvent_t>> ev_pool;
    std::vector<int> ev_used;         // indices into ev_pool, in launch order
    std::mutex mu;
};

namespace {

// [0] sweep counter, [1] flagged pairs, [2] recompute work counter, [3] and [4] counters of the launches beside
// (end-to-end modes on plain cells), [5] pairs recomputed
constexpr int kSplits = 6;     // from here on: the slots of chained pairs in parts
constexpr int kCounters = kSplits + 4 * kMaxSplits;
static_assert(kCounters <= 256, "one block clears them");
// Most entries of the recompute list; flagged pairs beyond it are found through their bits.
constexpr int64_t kRerunListMax = (int64_t)1 << 20;
constexpr int kRerunGrid = 64;
constexpr int kRerunRows = 8;  // rows per lane of the 32-bit recompute
constexpr int kMaxWgPerCu = 4; // persistent workgroups per CU (bounds the scratch slots)
const int kRowChoices[3] = {4, 8, 16};

struct DeviceGuard {
    int prev = -1;
    explicit DeviceGuard(int dev) {
        if (hipGetDevice(&prev) != hipSuccess) prev = -1;
        if (prev != dev) hipSetDevice(dev);
    }
    ~DeviceGuard() { if (prev >= 0) hipSetDevice(prev); }
};

sw_status apply_opts(sw_db* db, const sw_pack_opts* opts) {
    if (!opts) return SW_OK;
    const int fl = opts->force_lanes;
    if (fl < 0 || fl > 64 || (fl & (fl - 1))) return fail(SW_E_INVALID, "force_lanes must be 0 or a power of two <= 64");
    if (opts->rerun_threshold < 0) return fail(SW_E_INVALID, "rerun_threshold must be >= 0");
    const int rpl = opts->rows_per_lane;
    if (rpl != 0 && rpl != 4 && rpl != 8 && rpl != 16) return fail(SW_E_INVALID, "rows_per_lane must be 0, 4, 8 or 16");
    if (opts->lane_pack < 0 || opts->lane_pack > 2) return fail(SW_E_INVALID, "lane_pack must be 0, 1 or 2");
    if (opts->unit_share < 0 || opts->unit_share > 100000) return fail(SW_E_INVALID, "unit_share must be in 0..100000");
    if (opts->rerun_cap < 0) return fail(SW_E_INVALID, "rerun_cap must be >= 0");
    if (opts->poison != 0 && opts->poison != 1) return fail(SW_E_INVALID, "poison must be 0 or 1");
    if (opts->align_tiles < 0 || opts->align_tiles > 2) return fail(SW_E_INVALID, "align_tiles must be 0, 1 or 2");
    db->force_lgB = fl ? __builtin_ctz(fl) : -1;
    db->force_R = rpl;
    db->unit_share = opts->unit_share > 0 ? opts->unit_share / 1000.0 : kUnitShare;
    db->fixed_share = opts->unit_share > 0;
    db->sat = opts->rerun_threshold > 0 ? std::min<int32_t>(opts->rerun_threshold, kSat16) : kSat16;
    db->lane_pack = opts->lane_pack == 2 ? 2 : 1;
    db->rerun_cap_hook = opts->rerun_cap;
    db->poison = opts->poison;
    return SW_OK;
}

// ------------------------------------------------------------------ planning
// Issue slots of a step of R rows per lane in half instructions: 6.25 instructions per row of offset cells and 9.5 of
// plain ones, less the permutes where the lane holds two queries, plus loads, addressing and, with cooperating lanes,
// the hand-over of the bottom row.
int64_t step_cost(int cell, int R, bool coop, bool two_queries = false) {
    const int64_t rows = cell == kCellOff ? (two_queries ? 21 : 25) * R / 2 + 32 : (two_queries ? 17 : 19) * R + 30;
    return rows + (coop ? 8 : 0);
}

// Elapsed cost of a unit whose wave issues ahead of the others of its SIMD (long units run at raised priority), in
// the same units.  A lone wave's step takes 70 + 11 R ns on offset cells (measured at 4, 8 and 16 rows per lane), about
// 35 units more than it issues for; on plain cells 50 + 16 R, 16 units more; in the end-to-end modes on plain cells 120 +
// 19 R, 100 units more.  Other waves' instructions in flight hold up every one of its own (x 1.4).
constexpr int kLoneOff = 35, kLonePlain = 16, kLoneModes = 100;
int64_t elapsed(int64_t step, int lone, int64_t steps) { return (step + lone) * steps * 7 / 5; }

// The same for one pair on a workgroup (a chain item): its four waves at 4 rows per lane run side by side, 96
// steps apart, or on windows of the subject (whose overlap depends on the query; 4 m is typical), which global scores
// cannot be cut into.
int64_t chain_cost(int m, int ncols, bool cut, int parts = 1) {
    const int64_t passes = (m + 1023) / 1024;
    const int waves = passes > 1 ? 4 : (m + 255) / 256;
    const int64_t share = ncols / parts, lead = parts > 1 ? std::min(4 * m, ncols) : 0;
    int64_t cols = share + lead;
    for (int windows = cut ? 4 / waves : 1; windows > 1; --windows)
        if (4 * m + share / windows <= cols - cols / 4) { cols = share / windows + 4 * m; break; }
    return elapsed(25 * 4 / 2 + 55, kLoneOff, passes * (cols + 100 * waves));
}

// The parts to split a chained pair into, so that it ends within `busy`: the fewest that do, or as many as still
// shorten it by a tenth each, of at least kPartCols columns (2,000 subjects of at most 1,000 residues, split: 115
// instead of 110 us).  100,000 subjects, the longest of 35,000 residues, semi-global, a query of 331: unsplit 3.5
// ms, split 2.15.
constexpr int kPartCols = 1024;
int chain_parts(int m, int ncols, double busy) {
    int parts = 1;
    for (int64_t now = chain_cost(m, ncols, true);
         parts < kMaxParts && ncols / (parts + 1) >= kPartCols && (double)now > busy; ++parts) {
        const int64_t next = chain_cost(m, ncols, true, parts + 1);
        if (next > now - now / 10) break;
        now = next;
    }
    return parts;
}

// A unit of one wave (the widest lane cooperation) that may outlast the search: pair k of group g against query (or
// query pair) q.
struct LongUnit {
    int g, k, q;
    int64_t cost;                 // elapsed as a unit of one wave, at the rows per lane it would run with
    int64_t chain;                // elapsed as chain items: the longest one, and
    int64_t chain_sum;            // all of them (a query pair makes two)
    bool small;                   // the unit of one wave runs at 4 rows per lane
    int parts[2] = {1, 1};        // of the chain items
};

// What large units cost beyond what they issue, in times of the largest one's issue time: see plan_units.
constexpr double kLarge = 0.55;

// How many of the long units (sorted, longest first; `below` is the longest not among them) to run as chain items.
// A workgroup finishes a pair sooner than a wave but spends four waves' time on it, much of it waiting, so only the
// units that would outlast the search go: the first cut that leaves nothing outlasting the rest, or the one with the
// smallest estimated end of the search, which is the issue time of all work, the longest chain item, or the longest
// unit left to one wave.  (A chain item's four waves issue for about half of its elapsed time, a unit's wave for two
// thirds: `all` is the issue time of everything with no unit chained.)
constexpr double kLoneIssue = 0.67;
template <class Chain>                                   // chain(u, busy) fills in u.chain, u.chain_sum and u.parts
size_t chain_cut(const sw_db* db, std::vector<LongUnit>& units, double all, double below, double* end, Chain&& chain) {
    const double nsimd = 4.0 * std::max(db->cus, 1);
    double longest = 0, best = 0;
    size_t cut = 0;
    for (size_t k = 0;; ++k) {
        const double rest = k < units.size() ? (double)units[k].cost : below;
        const double busy = std::max(all / nsimd, longest);
        if (k == 0 || std::max(busy, rest) < best) { best = std::max(busy, rest); cut = k; }
        if (k == units.size() || rest <= busy) break;
        chain(units[k], all / nsimd);
        all += 2.0 * (double)units[k].chain_sum - kLoneIssue * (double)units[k].cost;
        longest = std::max(longest, (double)units[k].chain);
    }
    *end = std::max(*end, best);
    return cut;
}

struct PlanItem { WgItem it; int64_t cost; };

// Bundles units of one query (or query pair) into items of up to kWaves of one lane count, in the order they are added.
struct Bundle {
    std::vector<PlanItem>& out;
    WgItem cur;
    int64_t cost = 0, next = 0;      // next: position in the unit sequence that continues the item
    Bundle(std::vector<PlanItem>& o, int q, int nc) : out(o), cur{0, q, 0, -1, 0, nc} {}
    void flush() {
        if (cur.count > 0) out.push_back({cur, cost});
        cur.count = 0;
        cost = 0;
    }
    // unit k of the seq-th group, g, which has `units` of them
    void add(int g, int64_t seq, int units, int k, int lgB, int64_t c) {
        const int64_t at = seq * units + k;
        if (cur.count == 0 || cur.count == kWaves || cur.lgB != lgB || at != next) {
            flush();
            cur.g0 = g;
            cur.k0 = (int16_t)k;
            cur.lgB = (int8_t)lgB;
        }
        next = at + 1;
        cur.count++;
        cost = std::max(cost, c);
    }
};

// Items longest first.
void emit(std::vector<PlanItem>& v, std::vector<WgItem>& out) {
    // (mostly a few runs, each longest first)
    auto longer = [](const PlanItem& a, const PlanItem& b) { return a.cost > b.cost; };
    for (int runs = 0; runs < 16 && !std::is_sorted(v.begin(), v.end(), longer); ++runs) {
        const auto from = std::is_sorted_until(v.begin(), v.end(), longer);
        std::inplace_merge(v.begin(), from, std::is_sorted_until(from, v.end(), longer), longer);
    }
    if (!std::is_sorted(v.begin(), v.end(), longer)) std::stable_sort(v.begin(), v.end(), longer);
    out.reserve(out.size() + v.size());
    for (auto& t : v) out.push_back(t.it);
}

// The chain items of one pair, in at most the parts that slots are left for.
void push_chain(std::vector<PlanItem>& to, PlanKind kind, int g, int q, int k, int parts, int64_t cost, int& splits) {
    if (splits == kMaxSplits || kind != kPlanCut) parts = 1;
    for (int i = 0; i < parts; ++i)
        to.push_back({WgItem{g, q, (int16_t)k, kItemChain, 1, chain_split(parts > 1 ? splits : 0, parts, i)}, cost});
    splits += parts > 1;
}

// Units of one query by lanes per pair: what a unit of `cols` columns costs to issue (passes x steps x the step's
// cost), and elapsed where it runs alone.
struct CostTable {
    int lone_step;
    int64_t passes[7], step[7];
    int pad[7];
    CostTable(int m, int R, int cell, bool modes = false)
        : lone_step(cell == kCellOff ? kLoneOff : modes ? kLoneModes : kLonePlain) {
        for (int l = 0; l < 7; ++l) {
            passes[l] = (m + (R << l) - 1) / (R << l);
            step[l] = step_cost(cell, R, l > 0);
            pad[l] = (int)round_up((1 << l) - 1, 4);
        }
    }
    // (a unit's columns are a multiple of 4)
    int64_t steps(int cols, int l) const { return passes[l] * (cols + pad[l]); }
    int64_t unit(int cols, int l) const { return steps(cols, l) * step[l]; }
    int64_t lone(int cols, int l) const { return elapsed(step[l], lone_step, steps(cols, l)); }
};

// Work items for queries of lengths qlens (query index = position) against all
// groups.  Every group gets the smallest lanes-per-pair B whose units cost at
// most a set fraction of a persistent wave's share of the work (0.25 by
// default: smaller units force wide lane cooperation whose pass height exceeds
// short queries, larger ones lengthen the longest-first tail) and whose
// boundary row fits a scratch slot.  Units still above that share at B = 64
// are long pairs that a single wave sweeps column by column.  Those that would
// outlast the search are chained (chain_cut).  Where a unit's lanes x rows pad
// a short query, the group may run at 4 rows per lane instead of the launch's
// R: among the choices that keep its units within the share, the cheaper one is
// taken.  Items are ordered longest first.  The launch's R is the one with the
// smallest estimated end; the estimates sum costs alone, and items are made for
// the chosen R (a first search of six queries over 5,000 subjects spends 0.4 ms
// here instead of 2.4).
// Large units cost more than they issue (a last wave of them, and the rows
// between passes, of which few lanes per pair keep many): searches of 144 to
// 5,478 residues over 570,000 subjects at shares of 0.03 to 0.25 fit the issue
// time plus kLarge times the largest unit's.  More lanes pad a short query
// instead, so the chosen R is also sketched at half the share and the smaller
// estimate taken: 1,003 residues 22.3 -> 21.0 ms, 5,478 120 -> 115 ms; 144 (3.6
// against 4.5 ms) and 405 (10.4 against 10.8) keep the share.
// Overrides for sweeps other than the 16-bit ones: fixed R, their slot capacity and wave count, and
// whether the long pairs of a single short query may still go to the side list at a smaller R.
struct PlanLimits { int R; int64_t slot_cap; int64_t nwaves; bool side = false; };

// Groups [g_lo, g_hi) only (g_hi < 0: to the end).
// Offset cells: head_out takes the chained pairs and side_out the same as units of one wave.  Plain cells chain none;
// under limits (end-to-end modes) the long pairs of a single query may go to side_out at fewer rows per lane.
void plan_units(const sw_db* db, const std::vector<int>& qlens, PlanKind kind, Plan* plan, std::vector<WgItem>& main_out,
                std::vector<WgItem>& side_out, std::vector<WgItem>& head_out, const std::vector<int>* chunk = nullptr,
                int nchunks = 1, const PlanLimits* lim = nullptr, int g_lo = 0, int g_hi = -1,
                int* side_rows_out = nullptr) {
    const int cell = kind == kPlanPlain ? kCellI16 : kCellOff;
    if (g_hi < 0) g_hi = db->ngroups;
    const int64_t slot_cap = lim ? lim->slot_cap : db->slot_cap;
    const bool force_R = lim ? true : db->force_R != 0;
    // query qi covers groups chunk[qi], chunk[qi] + nchunks, ... (all groups when nchunks == 1) within [g_lo, g_hi)
    auto first_group = [&](size_t qi) { return chunk ? (*chunk)[qi] : 0; };
    auto start_group = [&](size_t qi) {
        const int f = first_group(qi);
        return f >= g_lo ? f : f + (int)round_up(g_lo - f, nchunks);
    };
    // How the launch at R rows per lane would run: lanes per pair of every (query, group), kItemSmall added where at 4
    // rows per lane, the largest cost of a unit, the chained units and the estimated end in cost units per wave.
    struct Sketch {
        int R = 0;
        std::vector<int8_t> lgB;
        int64_t cap = 0;
        std::vector<LongUnit> chained;
        double end = 0, share = 0;
    };
    auto side_rows = [&](int m, int R_main) {
        int r = R_main;
        if (qlens.size() == 1 && (!force_R || (lim && lim->side)))
            for (int R : kRowChoices)
                if (CostTable(m, R, cell, true).lone(db->ncols_max, 6) < CostTable(m, r, cell, true).lone(db->ncols_max, 6)) r = R;
        return r;
    };
    // The groups a sketch looks at: the longest ones each, of the rest of a large database every stride-th for its
    // neighbours too (groups are sorted by length); the chosen one is sketched in full.
    constexpr int kEach = 64;
    const int64_t ngroups = (g_hi - g_lo + nchunks - 1) / nchunks;
    const int stride = (int)std::max<int64_t>(1, ngroups / 512);
    auto walk = [&](size_t qi, bool full, auto&& visit) {
        const int g0 = start_group(qi);
        const int count = g0 < g_hi ? (g_hi - g0 + nchunks - 1) / nchunks : 0;
        for (int o = 0, w; o < count; o += w) {
            w = full || o < kEach ? 1 : std::min(stride, count - o);
            visit(g0 + o * nchunks, w);
        }
    };
    auto sketch = [&](int R_main, double share, bool full) {
        Sketch K;
        K.R = R_main;
        K.share = share;
        const int64_t nwaves = std::max<int64_t>(lim ? lim->nwaves : (int64_t)db->wgR[R_main] * kWaves, 1);
        std::vector<CostTable> big, small;
        int64_t total = 0;
        for (size_t qi = 0; qi < qlens.size(); ++qi) {
            big.emplace_back(std::max(qlens[qi], 1), R_main, cell);
            small.emplace_back(std::max(qlens[qi], 1), kSmallRows, cell);
            if (qlens[qi] <= 0) continue;
            walk(qi, full, [&](int g, int w) { total += w * big[qi].unit(db->ncols[g], 0); });
        }
        const double cap = share * (double)total / (double)nwaves;
        K.cap = (int64_t)std::min(cap, 9.0e18);
        const bool mix = !lim && R_main != kSmallRows && db->force_lgB < 0 && db->force_R == 0;
        int64_t sum = 0, biggest = 0;
        double lone_sum = 0, lone_end = 0;
        for (size_t qi = 0; qi < qlens.size(); ++qi) {
            const int m = qlens[qi];
            if (m <= 0) continue;
            const CostTable side(m, lim ? side_rows(m, R_main) : R_main, cell, lim != nullptr);
            walk(qi, full, [&](int g, int weight) {
                const int nc = db->ncols[g];
                // the fewest lanes per pair whose units stay within the share (6: perhaps none do)
                auto lanes = [&](const CostTable& t) {
                    int l = 0;
                    while (l < 6 && (t.unit(nc, l) > K.cap || (int64_t)nc * (kGroupPairs >> l) > slot_cap)) ++l;
                    return l;
                };
                int l = lanes(big[qi]);
                bool at4 = false;
                if (mix) {
                    const int l4 = lanes(small[qi]);
                    const int64_t c4 = small[qi].unit(nc, l4), c = big[qi].unit(nc, l);
                    // (units over the share are compared by what they take, the others by what the group takes)
                    at4 = std::min(c, c4) > K.cap ? c4 < c : c4 <= K.cap && ((c4 << l4) < (c << l) || c > K.cap);
                    if (at4) l = l4;
                }
                if (db->force_lgB >= 0) {
                    l = db->force_lgB;
                    while (l < 6 && (int64_t)nc * (kGroupPairs >> l) > slot_cap) ++l;
                }
                K.lgB.push_back((int8_t)(l + (at4 ? kItemSmall : 0)));
                const CostTable& t = at4 ? small[qi] : big[qi];
                // (a group's pairs are of about one length, longest first: sums take the mean of the ends)
                const int32_t* pc = db->pcols.data() + (size_t)g * kGroupPairs;
                int k = 0;                                   // units past the share, the first ones
                if (l == 6 && db->force_lgB < 0) {
                    if (t.unit(pc[kGroupPairs - 1], 6) > K.cap) k = kGroupPairs;
                    else while (t.unit(pc[k], 6) > K.cap) ++k;
                    if (k > 0) {
                        const CostTable& w = lim ? side : t;
                        const double e = (double)w.lone(pc[0], 6);
                        lone_sum += 0.5 * k * weight * (e + (double)w.lone(pc[k - 1], 6));
                        lone_end = std::max(lone_end, e);
                    }
                }
                const int units = (1 << l) - k;
                if (units > 0) {
                    const int64_t c = t.unit(pc[k], l);
                    biggest = std::max(biggest, c);
                    sum += weight * units * (c + t.unit(pc[kGroupPairs - 1], l)) / 2;
                }
            });
        }
        // issue time: the SIMDs share the total; a unit shares its SIMD with the other resident waves
        const double nsimd = 4.0 * db->cus, per_simd = (double)nwaves / nsimd;
        K.end = std::max((double)sum / nsimd, (double)biggest * per_simd);
        if (lim) {
            K.end = std::max(K.end, lone_end * per_simd);
            return K;
        }
        const double all = (double)sum + kLoneIssue * lone_sum;
        K.end = std::max(K.end, all / nsimd + kLarge * (double)biggest * per_simd);
        if (cell != kCellOff) {
            K.end = std::max(K.end, lone_end);
            return K;
        }
        // only units that take more than half of the search's issue time can outlast it
        std::vector<LongUnit> longs;
        double below = 0;
        size_t at = 0;
        for (size_t qi = 0; qi < qlens.size(); ++qi) {
            if (qlens[qi] <= 0) continue;
            bool on = true;                              // (shorter groups follow)
            walk(qi, full, [&](int g, int) {
                const int lg = K.lgB[at++];
                if (!on || (lg & (kItemSmall - 1)) != 6 || db->force_lgB >= 0) return;
                const bool at4 = lg >= kItemSmall;
                const CostTable& t = at4 ? small[qi] : big[qi];
                const int32_t* pc = db->pcols.data() + (size_t)g * kGroupPairs;
                for (int k = 0; k < kGroupPairs && t.unit(pc[k], 6) > K.cap; ++k) {
                    const int64_t e = t.lone(pc[k], 6);
                    if (2.0 * (double)e * nsimd <= all) {
                        below = std::max(below, (double)e);
                        on = k > 0;
                        break;
                    }
                    longs.push_back({g, k, (int)qi, e, 0, 0, at4});
                }
            });
        }
        std::stable_sort(longs.begin(), longs.end(), [](const LongUnit& a, const LongUnit& b) { return a.cost > b.cost; });
        longs.resize(chain_cut(db, longs, all, below, &K.end, [&](LongUnit& u, double busy) {
            const int uc = db->pcols[(size_t)u.g * kGroupPairs + u.k];
            u.parts[0] = kind != kPlanWhole ? chain_parts(qlens[u.q], uc, busy) : 1;
            u.chain = chain_cost(qlens[u.q], uc, kind != kPlanWhole, u.parts[0]);
            u.chain_sum = u.parts[0] * u.chain;
        }));
        K.chained.swap(longs);
        return K;
    };
    const bool one = force_R && (lim || db->fixed_share || db->force_lgB >= 0);           // nothing to choose
    Sketch K = sketch(lim ? lim->R : db->force_R ? db->force_R : 16, db->unit_share, one || stride == 1);
    if (!force_R) {
        // fewer rows per lane pay more per cell but pad less when lanes cooperate on a short query
        for (int R : {12, 8}) {
            if (R == 12 && cell != kCellOff) continue;       // (no kernel)
            Sketch other = sketch(R, db->unit_share, stride == 1);
            if (other.end < K.end) std::swap(K, other);
        }
    }
    if (!lim && !db->fixed_share && db->force_lgB < 0) {
        Sketch other = sketch(K.R, 0.5 * db->unit_share, stride == 1);
        if (other.end < K.end) std::swap(K, other);
    }
    if (!one && stride > 1) K = sketch(K.R, K.share, true);
    std::vector<PlanItem> main, side, head;
    std::vector<LongUnit> chained = K.chained;
    std::sort(chained.begin(), chained.end(), [](const LongUnit& a, const LongUnit& b) {
        return a.q != b.q ? a.q < b.q : a.g != b.g ? a.g < b.g : a.k < b.k;
    });
    size_t at = 0, ch = 0;
    int splits = 0;
    for (size_t qi = 0; qi < qlens.size(); ++qi) {
        const int m = qlens[qi];
        if (m <= 0) continue;
        const CostTable big(m, K.R, cell), small(m, kSmallRows, cell);
        // under limits a single query's long pairs go to the side list at fewer rows per lane where that is cheaper
        const int r_long = lim ? side_rows(m, K.R) : K.R;
        const CostTable lone(m, r_long, cell);
        Bundle bulk(main, (int)qi, nchunks), bulk4(main, (int)qi, nchunks);
        Bundle apart(side, (int)qi, nchunks), apart4(side, (int)qi, nchunks);
        int64_t seq = (start_group(qi) - first_group(qi)) / nchunks;
        for (int g = start_group(qi); g < g_hi; g += nchunks, ++at, ++seq) {
            const bool at4 = K.lgB[at] >= kItemSmall;
            const int l = K.lgB[at] & (kItemSmall - 1);
            const CostTable& t = at4 ? small : big;
            for (int k = 0; k < (1 << l); ++k) {
                const int uc = db->pcols[(size_t)g * kGroupPairs + (k << (6 - l))];
                const int64_t c = t.unit(uc, l);
                if (ch < chained.size() && chained[ch].q == (int)qi && chained[ch].g == g && chained[ch].k == k) {
                    push_chain(head, kind, g, (int)qi, k, chained[ch].parts[0], chained[ch].chain, splits);
                    (at4 ? apart4 : apart).add(g, seq, 1 << l, k, K.lgB[at], c);
                    ++ch;
                } else if (r_long != K.R && l == 6 && db->force_lgB < 0 && c > K.cap)
                    apart.add(g, seq, 1 << l, k, 6, lone.unit(uc, 6));
                else
                    (at4 ? bulk4 : bulk).add(g, seq, 1 << l, k, K.lgB[at], c);
            }
        }
        bulk.flush();
        bulk4.flush();
        apart.flush();
        apart4.flush();
    }
    emit(main, main_out);
    emit(side, side_out);
    emit(head, head_out);
    plan->R_main = K.R;
    if (side_rows_out) *side_rows_out = qlens.size() != 1 ? K.R : side_rows(qlens[0], K.R);
}

// Query-pair plan: queries on the same chunk are sorted by length and paired
// neighbour with neighbour, each pair sweeping max(m_a, m_b) rows: all of them,
// or those alone where that takes fewer passes than one query at a time at one lane
// per subject (a step takes two queries of a subject for less than two subjects
// of a query, since it needs no permutes, so a pair pays while the shorter
// query has about three quarters of the longer one's rows).  The others run two subjects
// per lane in the same launch (I.q the query, kItemSmall added to their lanes).
// The smaller estimated end decides: on a large database the passes count (16
// queries of 62 to 4,868 residues over 40,000 subjects, all paired 31.7 ms, by
// length 27.0), on a small one, whose units need many lanes, a pass of them
// takes a short query as well as a long one, and a pair saves half the units (on
// plain cells also a query without a partner: its step is the shorter one; 68 and
// 115 residues over 12,000 subjects of 300 residues: apart, a unit to an item, 1.67
// ms; paired, four to an item, 0.43).
// A pair's unit holds P = 64/B subjects and a group 2B units; B is capped at 32
// (the interleaved slice is twice as large).  Long subject pairs are chained as
// in plan_units (a chain item takes one query against the two subjects), the
// others of their length bundled with the rest, and half the share is tried.
void plan_units_q2(const sw_db* db, const std::vector<int>& qlens, PlanKind kind, Plan* plan, std::vector<WgItem>& out,
                   std::vector<WgItem>& side_out, std::vector<WgItem>& head_out, std::vector<int2>& pairs,
                   const std::vector<int>* chunk, int nchunks) {
    const int R = db->force_R == 8 ? 8 : 16;
    const int cell = kind == kPlanPlain ? kCellI16 : kCellOff;
    auto ch = [&](int q) { return chunk ? (*chunk)[q] : 0; };
    auto step2 = [&](int l) { return step_cost(cell, R, l > 0, true); };
    // One query, or a pair (x the longer one): what its units cost.
    struct Entry {
        int x, y, pair;            // pair < 0: one query, two subjects per lane
        CostTable t;
        int most() const { return pair < 0 ? 6 : 5; }          // log2 of the most lanes
        int units(int l) const { return pair < 0 ? 1 << l : 2 << l; }
        int first_pair(int k, int l) const { return pair < 0 ? k << (6 - l) : (k * (kGroupPairs >> l)) >> 1; }
    };
    std::vector<int> order;
    for (int q = 0; q < (int)qlens.size(); ++q)
        if (qlens[q] > 0) order.push_back(q);
    std::stable_sort(order.begin(), order.end(), [&](int a, int b) {
        return ch(a) != ch(b) ? ch(a) < ch(b) : qlens[a] > qlens[b];
    });
    auto entries_of = [&](bool all, std::vector<int2>& to) {
        std::vector<Entry> entries;
        for (size_t i = 0; i < order.size(); ++i) {
            Entry e{order[i], -1, -1, CostTable(qlens[order[i]], R, cell)};
            bool paired = all && cell != kCellOff;           // (half its lanes empty, if it has no partner)
            if (i + 1 < order.size() && ch(order[i]) == ch(order[i + 1])) {
                const CostTable next(qlens[order[i + 1]], R, cell);
                paired = all || 2 * e.t.passes[0] * step2(0) <= (e.t.passes[0] + next.passes[0]) * e.t.step[0];
                if (paired) e.y = order[++i];
            }
            if (paired) {
                e.pair = (int)to.size();
                for (int l = 0; l < 7; ++l) e.t.step[l] = step2(l);
                to.push_back(make_int2(e.x, e.y));
            }
            entries.push_back(e);
        }
        return entries;
    };
    const int64_t nwaves = std::max<int64_t>((int64_t)db->wgQ[R] * kWaves, 1);
    const double nsimd = 4.0 * std::max(db->cus, 1), per_simd = (double)nwaves / nsimd;
    // An estimate looks at the longest groups each and, of the rest, at every stride-th for its neighbours too.
    constexpr int kEach = 64;
    const int stride = std::max(1, db->ngroups / nchunks / 512);
    auto walk = [&](const Entry& e, auto&& visit) {
        const int count = (db->ngroups - ch(e.x) + nchunks - 1) / nchunks;
        for (int o = 0, w; o < count; o += w) {
            w = o < kEach ? 1 : std::min(stride, count - o);
            visit(ch(e.x) + o * nchunks, w);
        }
    };
    auto lanes = [&](const Entry& e, int nc, double cap) {
        int l = 0;
        while (l < e.most() && ((double)e.t.unit(nc, l) > cap || (int64_t)nc * (kGroupPairs >> l) > db->slot_cap)) ++l;
        if (db->force_lgB >= 0) {
            l = std::min(db->force_lgB, e.most());
            while (l < e.most() && (int64_t)nc * (kGroupPairs >> l) > db->slot_cap) ++l;
        }
        return l;
    };
    // units of the widest lane cooperation past the share run one pair each (unit k is pair k)
    auto is_long = [&](const Entry& e, int l, double c, double cap) { return l == e.most() && db->force_lgB < 0 && c > cap; };
    struct Sketch {
        std::vector<Entry> entries;
        std::vector<int2> pairs;
        std::vector<LongUnit> chained;
        double cap = 0, end = 0;
    };
    auto sketch = [&](bool all_pairs, double share) {
        Sketch K;
        K.entries = entries_of(all_pairs, K.pairs);
        double total = 0;
        for (const Entry& e : K.entries)
            walk(e, [&](int g, int w) { total += (double)w * e.units(0) * (double)e.t.unit(db->ncols[g], 0); });
        K.cap = share * total / (double)nwaves;
        double sum = 0, biggest = 0, lone_sum = 0;
        for (const Entry& e : K.entries)
            walk(e, [&](int g, int w) {
                const int l = lanes(e, db->ncols[g], K.cap), units = e.units(l);
                const int32_t* pc = db->pcols.data() + (size_t)g * kGroupPairs;
                auto cost = [&](int k) { return (double)e.t.unit(pc[e.first_pair(k, l)], l); };
                int k = 0;                                   // units past the share, the first ones
                if (is_long(e, l, cost(units - 1), K.cap)) k = units;
                else while (is_long(e, l, cost(k), K.cap)) ++k;
                // (pairs of a group are longest first and, but for the longest groups, of about one length: sums
                // take the mean of the ends there)
                auto mean = [&](int from, int to, auto&& of) {
                    double x = 0;
                    if (w > 1 && to > from) return 0.5 * w * (to - from) * (of(from) + of(to - 1));
                    for (int i = from; i < to; ++i) x += of(i);
                    return x;
                };
                lone_sum += mean(0, k, [&](int i) { return (double)e.t.lone(pc[i], l); });
                if (k < units) biggest = std::max(biggest, cost(k));
                sum += mean(k, units, cost);
            });
        // only units that take more than half of the search's issue time can outlast it
        double all = sum + kLoneIssue * lone_sum;
        std::vector<LongUnit> longs;
        double below = 0;
        for (size_t ei = 0; ei < K.entries.size(); ++ei) {
            const Entry& e = K.entries[ei];
            bool on = true;                                  // (shorter groups follow)
            for (int g = ch(e.x); on && g < db->ngroups; g += nchunks) {
                const int l = lanes(e, db->ncols[g], K.cap);
                const int32_t* pc = db->pcols.data() + (size_t)g * kGroupPairs;
                for (int k = 0; on && k < kGroupPairs; ++k) {
                    if (!is_long(e, l, (double)e.t.unit(pc[k], l), K.cap)) { on = false; break; }
                    const int64_t lone = e.t.lone(pc[k], l);
                    if (2.0 * (double)lone * nsimd <= all) {
                        below = std::max(below, (double)lone);
                        on = false;
                    } else
                        longs.push_back({g, k, (int)ei, lone, 0, 0, false});
                }
            }
        }
        if (cell != kCellOff) {
            for (const LongUnit& u : longs) below = std::max(below, (double)u.cost);
            K.end = std::max(below, all / nsimd + kLarge * biggest * per_simd);
            return K;
        }
        std::stable_sort(longs.begin(), longs.end(), [](const LongUnit& a, const LongUnit& b) { return a.cost > b.cost; });
        longs.resize(chain_cut(db, longs, all, below, &K.end, [&](LongUnit& u, double busy) {
            const int uc = db->pcols[(size_t)u.g * kGroupPairs + u.k];
            for (int i = 0; i < 2; ++i) {
                const int q = i == 0 ? K.entries[u.q].x : K.entries[u.q].y;
                if (q < 0) continue;
                u.parts[i] = chain_parts(qlens[q], uc, busy);
                const int64_t x = chain_cost(qlens[q], uc, true, u.parts[i]);
                u.chain = std::max(u.chain, x);
                u.chain_sum += u.parts[i] * x;
            }
        }));
        for (const LongUnit& u : longs) all += 2.0 * (double)u.chain_sum - kLoneIssue * (double)u.cost;
        K.end = std::max(K.end, all / nsimd + kLarge * biggest * per_simd);
        K.chained.swap(longs);
        return K;
    };
    Sketch K = sketch(false, db->unit_share);
    auto instead = [&](bool all_pairs, double share, double by) {
        Sketch other = sketch(all_pairs, share);
        const bool better = other.end < by * K.end;
        if (better) std::swap(K, other);
        return better;
    };
    // (all in pairs where that is clearly shorter on offset cells, whose estimates of chained pairs are rough: at 0.85 of
    // the estimate, 600 subjects of 3,000 to 12,000 residues against 77 and 203, it took 0.87 ms instead of 0.74)
    const bool all_pairs = 2 * K.pairs.size() < order.size() && instead(true, db->unit_share, cell == kCellOff ? 0.8 : 1.0);
    if (!db->fixed_share && db->force_lgB < 0) instead(all_pairs, 0.5 * db->unit_share, 1.0);
    std::vector<PlanItem> main, side, head;
    int splits = 0;
    for (const LongUnit& u : K.chained)                      // (the longest pairs get the slots for parts)
        for (int i = 0; i < 2; ++i) {
            const int q = i == 0 ? K.entries[u.q].x : K.entries[u.q].y;
            if (q >= 0) push_chain(head, kind, u.g, q, u.k, u.parts[i], u.chain, splits);
        }
    std::sort(K.chained.begin(), K.chained.end(), [](const LongUnit& a, const LongUnit& b) {
        return a.q != b.q ? a.q < b.q : a.g != b.g ? a.g < b.g : a.k < b.k;
    });
    size_t at = 0;
    for (size_t ei = 0; ei < K.entries.size(); ++ei) {
        const Entry& e = K.entries[ei];
        const int q = e.pair < 0 ? e.x : e.pair, flag = e.pair < 0 ? kItemSmall : 0;
        Bundle bulk(main, q, nchunks), apart(side, q, nchunks);
        int64_t seq = 0;
        for (int g = ch(e.x); g < db->ngroups; g += nchunks, ++seq) {
            const int l = lanes(e, db->ncols[g], K.cap);
            for (int k = 0; k < e.units(l); ++k) {
                const int64_t c = e.t.unit(db->pcols[(size_t)g * kGroupPairs + e.first_pair(k, l)], l);
                if (at < K.chained.size() && K.chained[at].q == (int)ei && K.chained[at].g == g && K.chained[at].k == k) {
                    apart.add(g, seq, e.units(l), k, l + flag, c);
                    ++at;
                } else
                    bulk.add(g, seq, e.units(l), k, l + flag, c);
            }
        }
        bulk.flush();
        apart.flush();
    }
    emit(main, out);
    emit(side, side_out);
    emit(head, head_out);
    pairs = K.pairs;
    plan->R_main = R;
}

sw_status build_plan(sw_db* db, const std::vector<int>& qlens, PlanKind kind, Plan* p,
                     const std::vector<int>* chunk = nullptr, int nchunks = 1) {
    std::vector<WgItem> mi, si, hi;
    std::vector<int2> pairs;
    int nonempty = 0;
    for (int m : qlens) nonempty += m > 0;
    p->qpack = db->lane_pack == 2 && nonempty >= 2;
    if (p->qpack)
        plan_units_q2(db, qlens, kind, p, mi, si, hi, pairs, chunk, nchunks);
    else
        plan_units(db, qlens, kind, p, mi, si, hi, chunk, nchunks);
    p->n_chain = (int32_t)hi.size();
    p->n_main = (int32_t)mi.size();
    p->n_unchained = (int32_t)si.size();
    auto small = [&](const std::vector<WgItem>& v) {
        if (p->qpack) return 0;
        return (int32_t)std::count_if(v.begin(), v.end(), [](const WgItem& it) { return it.lgB >= kItemSmall; });
    };
    p->n_small = small(mi);
    p->n_small_unchained = small(si);
    mi.insert(mi.begin(), hi.begin(), hi.end());
    mi.insert(mi.end(), si.begin(), si.end());
    p->h_items.swap(mi);
    p->h_pairs.swap(pairs);
    p->on_device = false;
    return SW_OK;
}

// Device copies of a plan's items and query pairs (searches on the handle's own workspace).
sw_status upload_plan(sw_db* db, Plan* p) {
    if (p->on_device) return SW_OK;
    HIP_TRY(p->items.reserve(std::max<size_t>(p->h_items.size(), 1) * sizeof(WgItem), &db->gen));
    if (!p->h_items.empty())
        HIP_TRY(hipMemcpy(p->items.p, p->h_items.data(), p->h_items.size() * sizeof(WgItem), hipMemcpyHostToDevice));
    if (p->qpack) {
        HIP_TRY(p->qpairs.reserve(std::max<size_t>(p->h_pairs.size(), 1) * sizeof(int2), &db->gen));
        if (!p->h_pairs.empty())
            HIP_TRY(hipMemcpy(p->qpairs.p, p->h_pairs.data(), p->h_pairs.size() * sizeof(int2), hipMemcpyHostToDevice));
    }
    p->on_device = true;
    return SW_OK;
}

sw_status get_plan(sw_db* db, int m, PlanKind kind, Plan** out) {
    const int64_t key = (int64_t)m * kPlanKinds + kind;
    auto it = db->plans.find(key);
    if (it != db->plans.end()) { *out = &it->second; return SW_OK; }
    if (db->plans.size() >= 64) {
        for (auto& kv : db->plans) kv.second.release();
        db->plans.clear();
    }
    Plan& p = db->plans[key];
    sw_status s = build_plan(db, std::vector<int>{m}, kind, &p);
    if (s != SW_OK) { p.release(); db->plans.erase(key); return s; }
    *out = &p;
    return SW_OK;
}

// Room for a plan in a caller's workspace: the offset cells' plan of the same queries and half as much again.
struct PlanRoom {
    size_t items = 0, pairs = 0;
    PlanRoom() = default;
    PlanRoom(const Plan& p, int nq) : items(p.h_items.size() + p.h_items.size() / 2 + 64), pairs(p.qpack ? (nq + 1) / 2 : 0) {}
    bool holds(const Plan& p) const { return p.h_items.size() <= items && p.h_pairs.size() <= pairs; }
};

void clear_caches(sw_db* db) {
    for (auto& kv : db->plans) kv.second.release();
    db->plans.clear();
    for (int k = 0; k < kPlanKinds; ++k) {
        db->batch_plan[k].clear();
        db->batch_qlens[k].clear();
    }
    db->multi_plan.clear();
    db->graph.clear();
    db->last_eager = BatchKey();
}

sw_status check_subst_gaps(const int8_t* subst, int32_t go, int32_t ge) {
    if (!subst) return fail(SW_E_INVALID, "substitution matrix pointer is NULL");
    if (go < 0 || ge < 0) return fail(SW_E_INVALID, "gap penalties must be >= 0 (got %d, %d)", go, ge);
    return SW_OK;
}

// Launch geometry (occupancy of every sweep instance, boundary-slot sizes), streams and events.
// Allocates no device memory.
sw_status ensure_geometry(sw_db* db) {
    if (db->wg16 == 0) {
        // a failure part way leaves wg16 at 0, so the next call sets up again (streams and events are
        // created once)
        struct Undo {
            sw_db* d;
            bool done = false;
            ~Undo() { if (!done) d->wg16 = 0; }
        } undo{db};
        hipDeviceProp_t prop;
        HIP_TRY(hipGetDeviceProperties(&prop, db->device));
        db->cus = prop.multiProcessorCount;
        int b32 = 0;
        db->wg16 = 0;
        for (int R : kRowChoices) {
            int b = 0, bo = 0;
            HIP_TRY(sweep_occupancy(kCellI16, R, &b));
            HIP_TRY(sweep_occupancy(kCellOff, R, &bo));
            if (b < 1 || bo < 1) return fail(SW_E_HIP, "16-bit sweep (R=%d) cannot be resident", R);
            db->wgR[R] = db->cus * std::min(std::max(b, bo), kMaxWgPerCu);
            db->wg16 = std::max(db->wg16, db->wgR[R]);
        }
        int b12 = 0;
        HIP_TRY(sweep_occupancy(kCellOff, 12, &b12));
        if (b12 < 1) return fail(SW_E_HIP, "16-bit sweep (R=12) cannot be resident");
        db->wgR[12] = db->cus * std::min(b12, kMaxWgPerCu);
        db->wg16 = std::max(db->wg16, db->wgR[12]);
        for (int R : {8, 16}) {
            int b = 0, bo = 0;
            HIP_TRY(sweep_occupancy_q2(kCellI16, R, &b));
            HIP_TRY(sweep_occupancy_q2(kCellOff, R, &bo));
            if (b < 1 || bo < 1) return fail(SW_E_HIP, "query-pair sweep (R=%d) cannot be resident", R);
            db->wgQ[R] = db->cus * std::min(std::max(b, bo), kMaxWgPerCu);
            db->wg16 = std::max(db->wg16, db->wgQ[R]);
        }
        HIP_TRY(sweep_occupancy(kCellI32, kRerunRows, &b32));
        if (b32 < 1) return fail(SW_E_HIP, "32-bit sweep cannot be resident");
        db->wg32 = kRerunGrid;
        // a unit's boundary row is (columns x subjects-or-pairs per wave); the widest
        // query-pair unit is 2 subjects of the longest subject's width
        db->slot_cap = std::max<int64_t>(65536, 2 * (int64_t)db->ncols_max);
        if (!db->side) HIP_TRY(hipStreamCreateWithFlags(&db->side, hipStreamNonBlocking));
        if (!db->side2) HIP_TRY(hipStreamCreateWithFlags(&db->side2, hipStreamNonBlocking));
        if (!db->cap) HIP_TRY(hipStreamCreateWithFlags(&db->cap, hipStreamNonBlocking));
        if (!db->ev_fork) HIP_TRY(hipEventCreateWithFlags(&db->ev_fork, hipEventDisableTiming));
        if (!db->ev_join) HIP_TRY(hipEventCreateWithFlags(&db->ev_join, hipEventDisableTiming));
        if (!db->ev_join2) HIP_TRY(hipEventCreateWithFlags(&db->ev_join2, hipEventDisableTiming));
        for (HostPinned& h : db->hstage)
            if (!h.done) HIP_TRY(hipEventCreateWithFlags(&h.done, hipEventDisableTiming));
        undo.done = true;
    }
    return SW_OK;
}

// Rows of a query's profile: whole passes at every B x R, of which 64 x 16 rows and 64 x 12 are the largest (the
// slices of a pass are read without a look at the query's end).
int prof_rows(int m) { return (int)std::max(round_up(std::max(m, 1), 1024), round_up(std::max(m, 1), 768)); }

// Layout of the staging buffer: [QDesc x nq][qoff x nq][subst, kMaxAlphabet^2 bytes][queries]
// [query pairs][plan items]; the plan parts only when the plan travels with the queries (a caller's
// workspace).
struct StageLayout { size_t off_qoff, off_sm, off_pairs, off_items, total; int64_t prof_elems; int max_mp; };

StageLayout stage_layout(const int64_t* h_qoffsets, int nq, const PlanRoom& room) {
    StageLayout L{};
    L.off_qoff = round_up(sizeof(QDesc) * nq, 64);
    L.off_sm = L.off_qoff + round_up(sizeof(int64_t) * nq, 64);
    L.off_pairs = round_up(L.off_sm + kMaxAlphabet * kMaxAlphabet + (h_qoffsets[nq] - h_qoffsets[0]), 64);
    L.off_items = round_up(L.off_pairs + room.pairs * sizeof(int2), 64);
    L.total = L.off_items + room.items * sizeof(WgItem);
    L.max_mp = prof_rows(1);
    for (int q = 0; q < nq; ++q) {
        const int m = (int)(h_qoffsets[q + 1] - h_qoffsets[q]);
        const int mp = prof_rows(m);
        L.prof_elems += (int64_t)kNRes * mp;
        L.max_mp = std::max(L.max_mp, mp);
    }
    return L;
}

// Capacity of the recompute list for nq queries: a flagged (query, subject
// pair) is appended once, so nq x pairs entries can never overflow; the list
// stops at kRerunListMax (or the test hook's capacity) and the pairs past it
// go through their flag bits.
int64_t rerun_capacity(const sw_db* db, int nq) {
    int64_t cap = std::min<int64_t>((int64_t)db->ngroups * kGroupPairs * std::max(nq, 1), kRerunListMax);
    if (db->rerun_cap_hook > 0) cap = std::min<int64_t>(cap, db->rerun_cap_hook);
    return std::max<int64_t>(cap, 1);
}

int64_t rerun_words(const sw_db* db, int nq) { return (int64_t)std::max(nq, 1) * db->ngroups * 2; }

// The device workspace of a launch sequence, one region laid out in this order:
// 16-bit boundary slots, 32-bit slots, counters, profiles, staging, recompute
// list, flag bits, top-k pieces, score rows (a batch that keeps only its top k).
struct WsLayout {
    StageLayout st;
    int64_t scratch16 = 0, scratch32 = 0, counters = 0, prof = 0, stage = 0, rerun = 0, bits = 0, topk = 0,
            scores = 0, total = 0;
    int64_t rerun_cap = 0, bits_words = 0;
};

WsLayout ws_layout(const sw_db* db, const int64_t* h_qoffsets, int nq, int k, bool with_scores, const PlanRoom& room) {
    WsLayout L;
    L.st = stage_layout(h_qoffsets, nq, room);
    L.rerun_cap = rerun_capacity(db, nq);
    L.bits_words = rerun_words(db, nq);
    int64_t o = 0;
    auto take = [&](int64_t bytes) { const int64_t at = o; o = round_up(o + std::max<int64_t>(bytes, 1), 256); return at; };
    L.scratch16 = take((int64_t)db->wg16 * kWaves * db->slot_cap * 2 * 4);
    L.scratch32 = take((int64_t)db->wg32 * kWaves * std::max<int64_t>(db->ncols_max, 4) * 4 * 4);
    L.counters = take(kCounters * sizeof(int32_t));
    L.prof = take(L.st.prof_elems * (int64_t)sizeof(int16_t));
    L.stage = take((int64_t)L.st.total);
    L.rerun = take(L.rerun_cap * (int64_t)sizeof(WgItem));
    L.bits = take(L.bits_words * (int64_t)sizeof(uint32_t));
    L.topk = take(k > 0 ? topk_ws_bytes(db->n, nq, k) : 0);
    L.scores = take(with_scores ? (int64_t)nq * std::max<int64_t>(db->n, 1) * (int64_t)sizeof(int32_t) : 0);
    L.total = o;
    return L;
}

// Device pointers of a workspace (the handle's own or a caller's) carved by a layout, and where the
// plan's items live.
struct Work {
    WsLayout L;
    uint32_t* scratch16 = nullptr;
    uint32_t* scratch32 = nullptr;
    int32_t* counters = nullptr;
    int16_t* prof = nullptr;
    char* stage = nullptr;
    WgItem* rerun = nullptr;
    uint32_t* bits = nullptr;
    void* topk = nullptr;
    int32_t* scores = nullptr;
    const WgItem* items = nullptr;
    const int2* qpairs = nullptr;
    HostPinned* host = nullptr;       // the pinned staging buffer of this call
};

Work carve(void* base, const WsLayout& L) {
    char* b = static_cast<char*>(base);
    Work W;
    W.L = L;
    W.scratch16 = reinterpret_cast<uint32_t*>(b + L.scratch16);
    W.scratch32 = reinterpret_cast<uint32_t*>(b + L.scratch32);
    W.counters = reinterpret_cast<int32_t*>(b + L.counters);
    W.prof = reinterpret_cast<int16_t*>(b + L.prof);
    W.stage = b + L.stage;
    W.rerun = reinterpret_cast<WgItem*>(b + L.rerun);
    W.bits = reinterpret_cast<uint32_t*>(b + L.bits);
    W.topk = b + L.topk;
    W.scores = reinterpret_cast<int32_t*>(b + L.scores);
    return W;
}

// The workspace of a launch sequence: the caller's (d_ws, checked against the layout) or the
// handle's own (grown as needed); plan items from the plan's device copy or, with a caller's
// workspace, from the staging area they are uploaded to.
sw_status get_work(sw_db* db, const int64_t* h_qoffsets, int nq, int k, bool with_scores, Plan* plan,
                   const PlanRoom& room, void* d_ws, int64_t ws_bytes, Work* out) {
    const bool caller = d_ws != nullptr;
    const WsLayout L = ws_layout(db, h_qoffsets, nq, k, with_scores, room);
    if (caller) {
        if (ws_bytes < L.total)
            return fail(SW_E_SIZE, "workspace of %lld bytes < %lld needed", (long long)ws_bytes, (long long)L.total);
        if ((reinterpret_cast<uintptr_t>(d_ws) & 255) != 0) return fail(SW_E_INVALID, "workspace not 256-byte aligned");
        *out = carve(d_ws, L);
    } else {
        HIP_TRY(db->ws_own.reserve((size_t)L.total, &db->gen));
        *out = carve(db->ws_own.p, L);
    }
    HostPinned& hs = db->hstage[db->hstage_next];
    db->hstage_next = (db->hstage_next + 1) % kStageRing;
    HIP_TRY(hs.reserve(L.st.total));
    out->host = &hs;
    if (plan) {
        if (caller) {
            out->items = reinterpret_cast<const WgItem*>(out->stage + L.st.off_items);
            out->qpairs = plan->qpack ? reinterpret_cast<const int2*>(out->stage + L.st.off_pairs) : nullptr;
        } else {
            sw_status s = upload_plan(db, plan);
            if (s != SW_OK) return s;
            out->items = plan->items.as<WgItem>();
            out->qpairs = plan->qpack ? plan->qpairs.as<int2>() : nullptr;
        }
    }
    return SW_OK;
}

// The recompute fields of a 16-bit sweep's arguments (flagged pairs are listed, then set as bits).
void set_rerun_args(sw_db* db, SweepArgs& a, const Work& W, int32_t* ctr) {
    a.rerun = W.rerun;
    a.rerun_count = ctr + 1;
    a.rerun_cap = (int32_t)W.L.rerun_cap;
    a.rerun_bits = W.bits;
    a.rerun_groups = db->ngroups;
    a.rerun_words = W.L.bits_words;
    a.recomputed = ctr + 5;
    a.poison = db->poison;
    db->last_cap = a.rerun_cap;
}

// Arguments of the 32-bit recompute that follows sweep arguments a: every listed pair, then (when the
// list overflowed) every pair whose flag bit is set; one unit per workgroup in the 32-bit slots.
SweepArgs recompute_args(const sw_db* db, const SweepArgs& a, const Work& W, int32_t* ctr) {
    SweepArgs r = a;
    r.items = W.rerun;
    r.n_items_dev = ctr + 1;
    r.n_items = a.rerun_cap;
    r.counter = ctr + 2;
    r.scratch = W.scratch32;
    r.slot_words = (int64_t)std::max<int32_t>(db->ncols_max, 4) * 4;
    r.slot_base = 0;
    r.rerun = nullptr;              // reads rerun_bits, appends nothing
    r.rerun_count = nullptr;
    r.unit_list = 1;
    r.poison = 0;
    return r;
}

// Sweep arguments shared by every launch of a search: image, profile, queries, gaps, 16-bit slots.
SweepArgs sweep_args(const sw_db* db, const Staged& S, const Work& W, int32_t go, int32_t ge, int32_t* scores) {
    SweepArgs a{};
    a.image = db->d_image;
    a.groups = db->d_groups;
    a.perm = db->d_perm;
    a.pair_cols = db->d_pair_cols;
    a.slen = db->d_slen;
    a.prof = W.prof;
    a.qd = S.qd;
    a.go = go;
    a.ge = ge;
    a.scratch = W.scratch16;
    a.slot_words = db->slot_cap * 2;
    a.slot_base = 0;
    a.scores = scores;
    return a;
}

// Most subject residues that a local alignment of a positive score covers, for a query of m residues whose best
// substitution scores add up to top: at most m are aligned, and d more in gaps cost at least Go + (d - 1) Ge
// (Ge <= Go), which must stay below top.
int32_t alignment_span(int64_t m, int64_t top, int32_t go, int32_t ge) {
    constexpr int64_t kWhole = (int64_t)1 << 28;              // beyond every subject
    if (top <= go) return (int32_t)std::min(m + 1, kWhole);
    if (ge <= 0 || ge > go) return (int32_t)kWhole;
    return (int32_t)std::min(m + (top - go) / ge + 1, kWhole);
}

// The same for a semi-global alignment that scores more than the query's own gap run, -(Go + (m - 1) Ge), which
// every subject's column 0 offers.
int32_t semiglobal_span(int64_t m, int64_t top, int32_t go, int32_t ge) {
    constexpr int64_t kWhole = (int64_t)1 << 28;
    if (ge <= 0 || ge > go) return (int32_t)kWhole;
    return (int32_t)std::min(m + (top + (m - 1) * ge) / ge + 1, kWhole);
}

// Copies the queries (host) into the staging buffer on the device.  No launch.
sw_status stage_queries(sw_db* db, const Work& W, const int8_t* h_queries, const int64_t* h_qoffsets, int nq,
                        const int8_t* subst, int32_t go, int32_t ge, int64_t score_row_stride, hipStream_t st, Staged* out,
                        int32_t* const* per_query_out = nullptr, const Plan* with_plan = nullptr,
                        int32_t mode = SW_LOCAL) {
    const StageLayout& L = W.L.st;
    char* h = static_cast<char*>(W.host->p);
    int64_t prof_off = 0;
    int best[kMaxAlphabet];
    for (int q = 0; q < db->alphabet; ++q) {
        best[q] = 0;
        for (int d = 0; d < db->alphabet; ++d) best[q] = std::max<int>(best[q], subst[q * db->alphabet + d]);
    }
    QDesc* qd = reinterpret_cast<QDesc*>(h);
    int64_t* qo = reinterpret_cast<int64_t*>(h + L.off_qoff);
    for (int q = 0; q < nq; ++q) {
        const int m = (int)(h_qoffsets[q + 1] - h_qoffsets[q]);
        const int mp = prof_rows(m);
        int64_t top = 0;
        for (int64_t i = h_qoffsets[q]; i < h_qoffsets[q + 1]; ++i) top += best[h_queries[i]];
        qd[q] = QDesc{prof_off, (int64_t)q * score_row_stride, per_query_out ? per_query_out[q] : nullptr, m, mp,
                      mode == SW_LOCAL ? alignment_span(m, top, go, ge) : semiglobal_span(m, top, go, ge), 0};
        prof_off += (int64_t)kNRes * mp;
        qo[q] = h_qoffsets[q] - h_qoffsets[0];
    }
    memcpy(h + L.off_sm, subst, (size_t)db->alphabet * db->alphabet);
    const int64_t qbytes = h_qoffsets[nq] - h_qoffsets[0];
    if (qbytes) memcpy(h + L.off_sm + kMaxAlphabet * kMaxAlphabet, h_queries + h_qoffsets[0], qbytes);
    if (with_plan) {
        if (!with_plan->h_items.empty())
            memcpy(h + L.off_items, with_plan->h_items.data(), with_plan->h_items.size() * sizeof(WgItem));
        if (with_plan->qpack && !with_plan->h_pairs.empty())
            memcpy(h + L.off_pairs, with_plan->h_pairs.data(), with_plan->h_pairs.size() * sizeof(int2));
    }
    const size_t used = L.off_items + (with_plan ? with_plan->h_items.size() * sizeof(WgItem) : 0);
    HIP_TRY(hipMemcpyAsync(W.stage, h, used, hipMemcpyHostToDevice, st));
    HIP_TRY(hipEventRecord(W.host->done, st));
    W.host->pending = true;
    const char* d = W.stage;
    out->qd = reinterpret_cast<const QDesc*>(d);
    out->qoff = reinterpret_cast<const int64_t*>(d + L.off_qoff);
    out->sm_q = reinterpret_cast<const int8_t*>(d + L.off_sm);
    out->nq = nq;
    out->max_mp = L.max_mp;
    return SW_OK;
}

// The cells of a local search of these queries.  Offset cells (sw_offset.h) need Ge <= Go (a gap opens at
// Go - Ge more), substitution bytes SM + Go + Ge in 0..255 and offsets that leave nearly the whole 16-bit
// range: they are lowered every K steps, with Ge K <= 128 (more would let a NaN pattern in S pass 0x7FFF),
// so Ge <= 32.  The usual protein scorings (10/2, 11/1, 14/2 with BLOSUM, PAM) all qualify.  Their exact
// range ends Go + Ge (K + 17) below the plain cells' 0x7C00, so a query whose best possible score lies
// between the two limits keeps plain cells, which hold every one of its scores without a recompute; from
// the plain limit on both forms recompute, and the offset cells are the faster ones.
CellForm choose_form(const sw_db* db, const int8_t* subst, int32_t go, int32_t ge, const int8_t* h_queries,
                     const int64_t* h_qoffsets, int nq) {
    const int A = db->alphabet;
    int lo = 0, hi = 0, best[kMaxAlphabet];
    for (int q = 0; q < A; ++q) {
        best[q] = 0;
        for (int d = 0; d < A; ++d) {
            lo = std::min<int>(lo, subst[q * A + d]);
            best[q] = std::max<int>(best[q], subst[q * A + d]);
        }
        hi = std::max(hi, best[q]);
    }
    CellForm f;
    f.bias = -lo;
    f.sat = std::min<int32_t>(db->sat + f.bias, kSat16);
    if (ge > go || ge > 32 || go > 255 || go + ge + lo < 0 || go + ge + hi > 255) return f;
    const int K = ge > 0 ? std::min(64, 4 * (32 / ge)) : 64;
    const int32_t limit = kSat16 - go - ge * (K + 17);
    for (int q = 0; q < nq; ++q) {
        int64_t top = 0;
        for (int64_t i = h_qoffsets[q]; i < h_qoffsets[q + 1]; ++i) top += best[h_queries[i]];
        if (top >= limit && top < kSat16 - f.bias) return f;
    }
    f.cell = kCellOff;
    f.bias = 0;
    f.off_k = K;
    f.add = go + ge;
    f.sat = std::min<int32_t>(db->sat, limit);
    return f;
}

// The cells of an end-to-end search: offset cells under the local form's conditions on gaps and bytes, as long as the
// lowest value a pair of this query can reach (the gap run down it, and what the cells themselves take off) leaves
// room above: half the range for semi-global scores, and for global ones, whose long similar subjects are lifted
// by their gap run as well, a fifth (queries up to about 3,100 residues at 10/2; beyond, plain cells run the longest
// subjects in 32 bits beside the others instead of recomputing high scorers one by one).  Anything else stays with
// the plain cells (cell = kCellI16 here).
CellForm choose_mode_form(const sw_db* db, int32_t mode, const int8_t* subst, int32_t go, int32_t ge, int32_t m) {
    int lo = 0, hi = 0;
    for (int i = 0; i < db->alphabet * db->alphabet; ++i) {
        lo = std::min<int>(lo, subst[i]);
        hi = std::max<int>(hi, subst[i]);
    }
    CellForm f;
    f.mode = mode;
    if (ge > go || ge > 32 || go > 255 || go + ge + lo < 0 || go + ge + hi > 255) return f;
    const int64_t run = (int64_t)go + (int64_t)(m - 1) * ge;          // the gap run down the query
    if (mode == SW_GLOBAL ? 5 * (128 + run) > 2 * (int64_t)kModeBias : kOffLo + run + 3 * (go - ge) > kModeBias) return f;
    f.cell = kCellOff;
    f.off_k = ge > 0 ? std::min(64, 4 * (32 / ge)) : 64;
    f.add = go + ge;
    f.bias = (int32_t)(kOffLo + run) + 3 * (go - ge);
    // padding neither gains nor loses: its diagonal step grows by what the offset does
    f.pad = mode == SW_GLOBAL ? go : go + ge;
    // (the range test reads G, Go - Ge below H)
    f.sat = (db->sat < kSat16 ? std::min<int32_t>(f.bias + db->sat, kSat16) : kSat16) - (go - ge);
    return f;
}

PlanKind plan_kind(const CellForm& f, int32_t ge) {
    return f.cell != kCellOff ? kPlanPlain : f.mode == SW_GLOBAL ? kPlanWhole : ge == 0 ? kPlanOnePart : kPlanCut;
}

// Timing events of the dominant launches (sw_profile_kernels): a ring of
// kTimerSlots start/stop pairs; the oldest is forgotten when it is full.
constexpr int kTimerSlots = 4096;

int record_timer_start(sw_db* db, hipStream_t st) {
    if (db->ev_used.size() >= (size_t)kTimerSlots) db->ev_used.erase(db->ev_used.begin());
    const int ev = (int)((db->ev_used.empty() ? -1 : db->ev_used.back()) + 1) % kTimerSlots;
    while ((int)db->ev_pool.size() <= ev) {
        hipEvent_t x, y;
        if (hipEventCreate(&x) != hipSuccess) return -1;
        if (hipEventCreate(&y) != hipSuccess) { hipEventDestroy(x); return -1; }
        db->ev_pool.push_back({x, y});
    }
    if (hipEventRecord(db->ev_pool[ev].first, st) != hipSuccess) return -1;
    return ev;
}

// The launch sequence of a search: profile (zeroes the counters), the 16-bit
// sweep, the 32-bit recompute, top-k.  Allocates nothing and never
// waits on the host, so it can be captured into a graph.
sw_status enqueue(sw_db* db, const Staged& S, const CellForm& form, const Plan& plan, const Work& W, int32_t go,
                  int32_t ge, int32_t* d_scores, int64_t n, int k, int32_t* top_s, int64_t* top_i, hipStream_t st,
                  bool time_sweep) {
    int32_t* ctr = W.counters;
    HIP_TRY(launch_profile(S.sm_q, db->alphabet, S.qd, S.nq, S.qoff, W.prof, ctr, kCounters, W.bits, W.L.bits_words,
                           S.max_mp, st, form.add, form.pad));
    SweepArgs a = sweep_args(db, S, W, go, ge, d_scores);
    // one launch: the chained pairs and then the bulk, or the unchained units and then the bulk
    const bool off = form.cell == kCellOff;
    a.items = W.items + (off ? 0 : plan.n_chain);
    a.n_items_dev = nullptr;
    a.n_items = plan.n_main + (off ? plan.n_chain : plan.n_unchained);
    a.first_item = off || plan.n_unchained == 0 ? 0 : plan.n_main;
    a.counter = ctr + 0;
    a.splits = ctr + kSplits;
    set_rerun_args(db, a, W, ctr);
    a.unit_list = 0;
    a.bias = form.bias;
    a.sat = form.sat;
    a.off_k = form.off_k;
    a.sm_shift = form.add;
    a.qpairs = plan.qpack ? W.qpairs : nullptr;
    // (a bulk wholly at 4 rows per lane takes the kernel of 4, which is smaller; plain cells have no kernel of 12
    // rows per lane: the units of such a plan run at 16)
    const int R = plan.n_main > 0 && plan.n_small == plan.n_main ? kSmallRows : !off && plan.R_main == 12 ? 16 : plan.R_main;
    const int grid = std::max(1, std::min(plan.qpack ? db->wgQ[R] : db->wgR[R], std::max(a.n_items, 1)));
    const int ev = time_sweep && db->timing ? record_timer_start(db, st) : -1;
    if (a.n_items > 0) {
        if (plan.qpack)
            HIP_TRY(launch_sweep_q2(form.cell, R, a, grid, st));
        else if (form.mode != SW_LOCAL)
            HIP_TRY(launch_sweep_mode_off(form.mode, R, a, grid, st));
        else
            HIP_TRY(launch_sweep(form.cell, R, a, grid, st));
    }
    if (ev >= 0) {
        HIP_TRY(hipEventRecord(db->ev_pool[ev].second, st));
        db->ev_used.push_back(ev);
    }
    // exact 32-bit recompute of saturated pairs; the count is read on the device
    SweepArgs r = recompute_args(db, a, W, ctr);
    if (form.mode != SW_LOCAL) {
        r.bias = 0;
        HIP_TRY(launch_sweep_mode(form.mode, kRerunRows, r, db->wg32, st));
    } else
        HIP_TRY(launch_sweep(kCellI32, kRerunRows, r, db->wg32, st));
    if (k > 0)
        HIP_TRY(launch_topk_ws(d_scores, n, n, S.nq, k, top_s, top_i, topk_ws_bytes(n, S.nq, k) > 0 ? W.topk : nullptr,
                               st));
    db->last_side_items = plan.n_small + (off ? plan.n_chain : plan.n_small_unchained);
    db->last_items = a.n_items - db->last_side_items;
    db->last_rows = R;
    db->last_side_rows = db->last_side_items > 0 ? kSmallRows : 0;
    db->last_grid = grid;
    db->last_counters = ctr;
    return SW_OK;
}

sw_status check_db_args(sw_db* db, const int64_t* h_offsets, int64_t n) {
    if (!db) return fail(SW_E_INVALID, "db is NULL");
    if (n != db->n) return fail(SW_E_INVALID, "n = %lld but the database holds %lld subjects", (long long)n, (long long)db->n);
    if (h_offsets && n > 0 &&
        (h_offsets[0] != db->off_first || h_offsets[n] != db->off_last || offsets_hash(h_offsets, n) != db->off_hash))
        return fail(SW_E_INVALID, "offsets do not match the packed database");
    return SW_OK;
}


}  // namespace

namespace {

// Host side of packing: the length order, the groups of 128 subjects and where each subject goes.
struct PackPlan {
    std::vector<int32_t> len;         // per original subject
    std::vector<int32_t> order;       // sorted slot -> original subject
    std::vector<GroupRec> groups;
    std::vector<int64_t> gdw;         // group base in dwords
    std::vector<int32_t> perm;        // [G * 128] sorted slot -> original subject, -1 for padding slots
    std::vector<int64_t> soff;        // sorted slot -> residue offset of the subject
    std::vector<int32_t> slen;        // [G * 128] sorted slot -> length, 0 for padding slots
    std::vector<int32_t> ncols;       // per group
    std::vector<int32_t> pcols;       // per pair
    int32_t ncols_max = 0;
    int64_t image_bytes = 0;
    int G = 0;
};

sw_status plan_pack(const int64_t* h_offsets, int64_t n, PackPlan* P) {
    if (n < 0) return fail(SW_E_INVALID, "n must be >= 0");
    if (n > ((int64_t)1 << 31) - 256) return fail(SW_E_UNSUPPORTED, "more than 2^31 subjects");
    if (n > 0 && !h_offsets) return fail(SW_E_INVALID, "NULL offsets");
    if (n > 0 && h_offsets[0] < 0) return fail(SW_E_INVALID, "offsets[0] < 0");
    P->len.resize(n);
    for (int64_t k = 0; k < n; ++k) {
        const int64_t l = h_offsets[k + 1] - h_offsets[k];
        if (l < 0) return fail(SW_E_INVALID, "offsets decrease at %lld", (long long)k);
        if (l > (1 << 24)) return fail(SW_E_UNSUPPORTED, "subject %lld longer than 2^24", (long long)k);
        P->len[k] = (int32_t)l;
    }
    P->order.resize(n);
    std::iota(P->order.begin(), P->order.end(), 0);
    std::stable_sort(P->order.begin(), P->order.end(), [&](int32_t a, int32_t b) { return P->len[a] > P->len[b]; });
    const int G = P->G = (int)((n + kGroupSubjects - 1) / kGroupSubjects);
    P->groups.resize(G);
    P->gdw.resize(G);
    P->ncols.resize(G);
    int64_t base = 0;
    for (int g = 0; g < G; ++g) {
        const int32_t nc = (int32_t)round_up(P->len[P->order[(size_t)g * kGroupSubjects]], kChunkCols);
        P->groups[g] = GroupRec{base, nc, g * kGroupSubjects};
        P->gdw[g] = base / 4;
        P->ncols[g] = nc;
        P->ncols_max = std::max(P->ncols_max, nc);
        base += (int64_t)nc * kGroupSubjects;
    }
    P->image_bytes = base;
    P->perm.assign((size_t)G * kGroupSubjects, -1);
    P->slen.assign((size_t)G * kGroupSubjects, 0);
    P->soff.resize(n);
    P->pcols.assign((size_t)G * kGroupPairs, 0);
    for (int64_t i = 0; i < n; ++i) {
        const int32_t o = P->order[i];
        P->pcols[(size_t)(i / 2)] = std::max<int32_t>(P->pcols[(size_t)(i / 2)], (int32_t)round_up(P->len[o], kChunkCols));
        P->perm[i] = o;
        P->soff[i] = h_offsets[o];
        P->slen[i] = P->len[o];
    }
    return SW_OK;
}

// Device layout of a packed image: interleaved residues, group table, permutation, pair widths,
// sorted lengths, then what packing alone uses (residue offsets per sorted slot, group bases, an
// error word), which may hold anything afterwards.
struct DbLayout { int64_t image, groups, perm, pair_cols, slen, soff, gdw, err, total; };

DbLayout db_layout(int64_t n, int G, int64_t image_bytes) {
    DbLayout L{};
    int64_t o = 0;
    auto take = [&](int64_t bytes) { const int64_t at = o; o = round_up(o + std::max<int64_t>(bytes, 1), 256); return at; };
    L.image = take(std::max<int64_t>(image_bytes, 4));
    L.groups = take((int64_t)sizeof(GroupRec) * G);
    L.perm = take(4 * (int64_t)G * kGroupSubjects);
    L.pair_cols = take(4 * (int64_t)G * kGroupPairs);
    L.slen = take(4 * (int64_t)G * kGroupSubjects);
    L.soff = take(8 * std::max<int64_t>(n, 1));
    L.gdw = take(8 * (int64_t)std::max(G, 1));
    L.err = take(4);
    L.total = o;
    return L;
}

// sw_db_pack (d_db NULL: the handle allocates the image) and sw_db_pack_into (the caller's buffer).
sw_status pack_db(const int8_t* d_residues, const int64_t* h_offsets, int64_t n, const sw_pack_opts* opts, void* d_db,
                  int64_t db_bytes, hipStream_t st, sw_db** out) {
    if (!out) return fail(SW_E_INVALID, "out is NULL");
    *out = nullptr;
    if (n > 0 && !d_residues) return fail(SW_E_INVALID, "NULL residues");
    PackPlan P;
    sw_status so = plan_pack(h_offsets, n, &P);
    if (so != SW_OK) return so;
    const DbLayout L = db_layout(n, P.G, P.image_bytes);
    if (d_db && db_bytes < L.total)
        return fail(SW_E_SIZE, "image buffer of %lld bytes < %lld needed", (long long)db_bytes, (long long)L.total);
    if (d_db && (reinterpret_cast<uintptr_t>(d_db) & 255) != 0) return fail(SW_E_INVALID, "image buffer not 256-byte aligned");
    sw_db* db = new (std::nothrow) sw_db();
    if (!db) return fail(SW_E_NOMEM, "host allocation failed");
    auto bail = [&](sw_status s) { sw_db_free(db); return s; };
    if (hipGetDevice(&db->device) != hipSuccess) return bail(fail(SW_E_HIP, "no current HIP device"));
    so = apply_opts(db, opts);
    if (so != SW_OK) return bail(so);
    if (opts && (opts->alphabet < 0 || opts->alphabet > kMaxAlphabet))
        return bail(fail(SW_E_INVALID, "alphabet must be 0 (= 20) or 1..%d", kMaxAlphabet));
    db->alphabet = (opts && opts->alphabet > 0) ? opts->alphabet : 20;
    db->n = n;
    db->off_first = n > 0 ? h_offsets[0] : 0;
    db->off_last = n > 0 ? h_offsets[n] : 0;
    db->off_hash = n > 0 ? offsets_hash(h_offsets, n) : 0;
    db->total_res = db->off_last - db->off_first;
    db->ngroups = P.G;
    db->ncols = P.ncols;
    db->pcols = P.pcols;
    db->ncols_max = P.ncols_max;
    db->image_bytes = P.image_bytes;
    db->lens = P.len;
    db->slot_of.assign(n, 0);
    for (int64_t i = 0; i < n; ++i) db->slot_of[P.order[i]] = (int32_t)i;
    db->gbase.resize(P.G);
    for (int g = 0; g < P.G; ++g) db->gbase[g] = P.groups[g].base;
    char* base = static_cast<char*>(d_db);
    if (!d_db) {
        const hipError_t e = db->image_own.reserve((size_t)L.total);
        if (e != hipSuccess)
            return bail(fail(e == hipErrorOutOfMemory ? SW_E_NOMEM : SW_E_HIP, "device allocation: %s", hipGetErrorString(e)));
        base = db->image_own.as<char>();
    }
    db->caller_image = d_db != nullptr;
    db->d_image = reinterpret_cast<uint8_t*>(base + L.image);
    db->d_groups = reinterpret_cast<GroupRec*>(base + L.groups);
    db->d_perm = reinterpret_cast<int32_t*>(base + L.perm);
    db->d_pair_cols = reinterpret_cast<int32_t*>(base + L.pair_cols);
    db->d_slen = reinterpret_cast<int32_t*>(base + L.slen);
    if (P.G > 0) {
        int64_t* d_soff = reinterpret_cast<int64_t*>(base + L.soff);
        int64_t* d_gdw = reinterpret_cast<int64_t*>(base + L.gdw);
        int32_t* d_err = reinterpret_cast<int32_t*>(base + L.err);
        int32_t zero = 0, herr = 0;
        hipError_t e = hipSuccess;
        auto step = [&](hipError_t x) { if (e == hipSuccess) e = x; };
        step(hipMemcpyAsync(db->d_groups, P.groups.data(), sizeof(GroupRec) * P.G, hipMemcpyHostToDevice, st));
        step(hipMemcpyAsync(db->d_perm, P.perm.data(), sizeof(int32_t) * P.perm.size(), hipMemcpyHostToDevice, st));
        step(hipMemcpyAsync(db->d_pair_cols, P.pcols.data(), sizeof(int32_t) * P.pcols.size(), hipMemcpyHostToDevice, st));
        step(hipMemcpyAsync(db->d_slen, P.slen.data(), sizeof(int32_t) * P.slen.size(), hipMemcpyHostToDevice, st));
        step(hipMemcpyAsync(d_soff, P.soff.data(), sizeof(int64_t) * n, hipMemcpyHostToDevice, st));
        step(hipMemcpyAsync(d_gdw, P.gdw.data(), sizeof(int64_t) * P.G, hipMemcpyHostToDevice, st));
        step(hipMemcpyAsync(d_err, &zero, 4, hipMemcpyHostToDevice, st));
        step(launch_interleave(d_residues, d_soff, db->d_slen, n, db->alphabet, db->d_groups, d_gdw, P.G,
                               reinterpret_cast<uint32_t*>(db->d_image), P.image_bytes / 4, d_err, st));
        step(hipMemcpyAsync(&herr, d_err, 4, hipMemcpyDeviceToHost, st));
        step(hipStreamSynchronize(st));
        if (e != hipSuccess) return bail(fail(SW_E_HIP, "packing: %s", hipGetErrorString(e)));
        if (herr) return bail(fail(SW_E_RESIDUE, "database residue code outside 0..%d", db->alphabet - 1));
    }
    *out = db;
    return SW_OK;
}

}  // namespace

namespace {

// sw_search and sw_search_ws: the plain form, on the handle's workspace (d_ws NULL) or the caller's.
sw_status search_one(const int8_t* h_query, int32_t qlen, sw_db* db, const int64_t* h_offsets, int64_t n,
                     const int8_t* h_subst, int32_t gap_open, int32_t gap_extend, int32_t* d_scores_out, void* d_ws,
                     int64_t ws_bytes, hipStream_t st) {
    sw_status s;
    if ((s = check_db_args(db, h_offsets, n)) != SW_OK) return s;
    if ((s = check_subst_gaps(h_subst, gap_open, gap_extend)) != SW_OK) return s;
    if (qlen < 0) return fail(SW_E_INVALID, "qlen must be >= 0");
    if (qlen > 0 && !h_query) return fail(SW_E_INVALID, "query is NULL");
    if (n > 0 && !d_scores_out) return fail(SW_E_INVALID, "scores_out is NULL");
    for (int32_t i = 0; i < qlen; ++i)
        if (h_query[i] < 0 || h_query[i] >= db->alphabet)
            return fail(SW_E_RESIDUE, "query residue %d at %d outside 0..%d", h_query[i], i, db->alphabet - 1);
    if (n == 0) return SW_OK;
    std::lock_guard<std::mutex> lk(db->mu);
    DeviceGuard dg(db->device);
    if (qlen == 0) { HIP_TRY(launch_fill(d_scores_out, n, 0, st)); return SW_OK; }
    if ((s = ensure_geometry(db)) != SW_OK) return s;
    const int64_t qo[2] = {0, qlen};
    const CellForm form = choose_form(db, h_subst, gap_open, gap_extend, h_query, qo, 1);
    PlanKind kind = plan_kind(form, gap_extend);
    PlanRoom room;
    Plan* plan = nullptr;
    if (d_ws) {
        if ((s = get_plan(db, qlen, kPlanCut, &plan)) != SW_OK) return s;
        room = PlanRoom(*plan, 1);
        if (kind != kPlanCut) {
            if ((s = get_plan(db, qlen, kind, &plan)) != SW_OK) return s;
            if (!room.holds(*plan)) kind = kPlanCut;
        }
    }
    if ((s = get_plan(db, qlen, kind, &plan)) != SW_OK) return s;
    Work W;
    if ((s = get_work(db, qo, 1, 0, false, plan, room, d_ws, ws_bytes, &W)) != SW_OK) return s;
    Staged S;
    if ((s = stage_queries(db, W, h_query, qo, 1, h_subst, gap_open, gap_extend, 0, st, &S, nullptr, d_ws ? plan : nullptr)) != SW_OK)
        return s;
    return enqueue(db, S, form, *plan, W, gap_open, gap_extend, d_scores_out, n, 0, nullptr, nullptr, st, true);
}

}  // namespace

namespace {

// The batch plan of a kind for these query lengths (kept while the lengths repeat).
sw_status plan_for(sw_db* db, const std::vector<int>& qlens, PlanKind kind, Plan** out) {
    Plan& p = db->batch_plan[kind];
    if (qlens != db->batch_qlens[kind]) {
        if (p.on_device) HIP_TRY(hipDeviceSynchronize());     // a batch in flight may read its items
        db->batch_qlens[kind].clear();
        p.release();
        sw_status s = build_plan(db, qlens, kind, &p);
        if (s != SW_OK) return s;
        db->batch_qlens[kind] = qlens;
    }
    *out = &p;
    return SW_OK;
}

// sw_search_batch and sw_search_batch_ws: the batched form, on the handle's workspace (d_ws NULL) or
// the caller's.
sw_status search_batch(const int8_t* h_queries, const int64_t* h_qoffsets, int32_t nq, sw_db* db,
                       const int8_t* h_subst, int32_t gap_open, int32_t gap_extend, int32_t k, int32_t* d_scores,
                       int32_t* d_top_scores, int64_t* d_top_index, void* d_ws, int64_t ws_bytes, hipStream_t st) {
    sw_status s;
    if (!db) return fail(SW_E_INVALID, "db is NULL");
    if ((s = check_subst_gaps(h_subst, gap_open, gap_extend)) != SW_OK) return s;
    if (nq < 0) return fail(SW_E_INVALID, "nq must be >= 0");
    if (nq > 0 && (!h_qoffsets || !h_queries)) return fail(SW_E_INVALID, "NULL queries or offsets");
    if (k < 0 || k > 1024) return fail(SW_E_UNSUPPORTED, "k must be in 0..1024 (got %d)", k);
    if (k > 0 && (!d_top_scores || !d_top_index)) return fail(SW_E_INVALID, "NULL top-k outputs");
    if (!d_scores && k == 0) return fail(SW_E_INVALID, "no output requested (scores NULL and k == 0)");
    for (int q = 0; q < nq; ++q) {
        if (h_qoffsets[q + 1] < h_qoffsets[q]) return fail(SW_E_INVALID, "query offsets decrease at %d", q);
        if (h_qoffsets[q + 1] - h_qoffsets[q] > (1 << 24)) return fail(SW_E_UNSUPPORTED, "query %d too long", q);
    }
    if (nq > 0)
        for (int64_t i = h_qoffsets[0]; i < h_qoffsets[nq]; ++i)
            if (h_queries[i] < 0 || h_queries[i] >= db->alphabet) return fail(SW_E_RESIDUE, "query residue outside 0..%d at %lld", db->alphabet - 1, (long long)i);
    if (nq == 0) return SW_OK;
    std::lock_guard<std::mutex> lk(db->mu);
    DeviceGuard dg(db->device);
    const int64_t n = db->n;
    if (n == 0) {
        if (k > 0) HIP_TRY(launch_topk(d_scores, 0, 0, nq, k, d_top_scores, d_top_index, st));
        return SW_OK;
    }
    if ((s = ensure_geometry(db)) != SW_OK) return s;
    std::vector<int> qlens(nq);
    for (int q = 0; q < nq; ++q) qlens[q] = (int)(h_qoffsets[q + 1] - h_qoffsets[q]);
    const CellForm form = choose_form(db, h_subst, gap_open, gap_extend, h_queries, h_qoffsets, nq);
    const PlanKind kind = plan_kind(form, gap_extend);
    // On the handle's workspace the plan's device copy may still be read by the previous batch; a caller's
    // workspace receives the plan with the queries, in stream order, so nothing waits.
    if (!d_ws && qlens != db->batch_qlens[kind]) HIP_TRY(hipStreamSynchronize(st));
    Plan* plan = nullptr;
    if ((s = plan_for(db, qlens, kind, &plan)) != SW_OK) return s;
    PlanRoom room;
    if (d_ws) {
        Plan* cut = plan;
        if (kind != kPlanCut && (s = plan_for(db, qlens, kPlanCut, &cut)) != SW_OK) return s;
        room = PlanRoom(*cut, nq);
        if (!room.holds(*plan)) plan = cut;
    }
    Work W;
    if ((s = get_work(db, h_qoffsets, nq, k, d_scores == nullptr, plan, room, d_ws, ws_bytes, &W)) != SW_OK) return s;
    int32_t* scores = d_scores ? d_scores : W.scores;
    // zero-length queries score 0 everywhere (outside the captured sequence)
    for (int q = 0; q < nq; ++q)
        if (qlens[q] == 0) HIP_TRY(launch_fill(scores + (int64_t)q * n, n, 0, st));
    Staged S;
    if ((s = stage_queries(db, W, h_queries, h_qoffsets, nq, h_subst, gap_open, gap_extend, n, st, &S, nullptr, d_ws ? plan : nullptr)) != SW_OK)
        return s;
    GraphEntry& G = db->graph;
    BatchKey key;
    key.qlens = qlens;
    key.go = gap_open;
    key.ge = gap_extend;
    key.k = k;
    key.form = form;
    key.scores = scores;
    key.top_s = d_top_scores;
    key.top_i = d_top_index;
    key.stream = st;
    key.gen = db->gen;
    key.ws = W.scratch16;
    const bool hit = G.exec && G.gen == db->gen && G.ws == W.scratch16 && G.qlens == qlens && G.go == gap_open &&
                     G.ge == gap_extend && G.form == form && G.k == k && G.scores == scores &&
                     G.top_s == d_top_scores && G.top_i == d_top_index && G.stream == st;
    if (!hit && !(key == db->last_eager)) {
        db->last_eager = key;
        const int ev = db->timing ? record_timer_start(db, st) : -1;
        s = enqueue(db, S, form, *plan, W, gap_open, gap_extend, scores, n, k, d_top_scores, d_top_index, st, false);
        if (s != SW_OK) return s;
        if (ev >= 0) {
            HIP_TRY(hipEventRecord(db->ev_pool[ev].second, st));
            db->ev_used.push_back(ev);
        }
        return SW_OK;
    }
    if (!hit) {
        // captured on the library's own stream (the caller's may be the legacy
        // default stream, which cannot be captured); launched on the caller's
        G.clear();
        HIP_TRY(hipStreamBeginCapture(db->cap, hipStreamCaptureModeThreadLocal));
        s = enqueue(db, S, form, *plan, W, gap_open, gap_extend, scores, n, k, d_top_scores, d_top_index, db->cap, false);
        hipGraph_t graph = nullptr;
        hipError_t e = hipStreamEndCapture(db->cap, &graph);
        if (s != SW_OK) { if (graph) hipGraphDestroy(graph); return s; }
        if (e != hipSuccess) return fail(SW_E_HIP, "graph capture: %s", hipGetErrorString(e));
        hipGraphExec_t exec = nullptr;
        e = hipGraphInstantiate(&exec, graph, nullptr, nullptr, 0);
        if (e != hipSuccess) { hipGraphDestroy(graph); return fail(SW_E_HIP, "graph instantiate: %s", hipGetErrorString(e)); }
        G.graph = graph;
        G.exec = exec;
        G.qlens = qlens;
        G.go = gap_open;
        G.ge = gap_extend;
        G.form = form;
        G.k = k;
        G.scores = scores;
        G.top_s = d_top_scores;
        G.top_i = d_top_index;
        G.stream = st;
        G.gen = db->gen;
        G.ws = W.scratch16;
        db->last_eager = BatchKey();
    }
    if (!G.done) HIP_TRY(hipEventCreateWithFlags(&G.done, hipEventDisableTiming));
    const int ev = db->timing ? record_timer_start(db, st) : -1;
    HIP_TRY(hipGraphLaunch(G.exec, st));
    HIP_TRY(hipEventRecord(G.done, st));
    G.launched = true;
    if (ev >= 0) {
        HIP_TRY(hipEventRecord(db->ev_pool[ev].second, st));
        db->ev_used.push_back(ev);
    }
    return SW_OK;
}


}  // namespace

namespace sw {
// Records an error for sw_last_error() from other files of the library and returns s.
sw_status report(sw_status s, const char* fmt, ...) {
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    g_err = buf;
    return s;
}
}  // namespace sw

// ====================================================================== C ABI
extern "C" {

const char* sw_status_str(sw_status s) {
    switch (s) {
        case SW_OK: return "SW_OK";
        case SW_E_INVALID: return "SW_E_INVALID";
        case SW_E_RESIDUE: return "SW_E_RESIDUE";
        case SW_E_NOMEM: return "SW_E_NOMEM";
        case SW_E_HIP: return "SW_E_HIP";
        case SW_E_UNSUPPORTED: return "SW_E_UNSUPPORTED";
        case SW_E_SIZE: return "SW_E_SIZE";
        default: return "SW_E_UNKNOWN";
    }
}

const char* sw_last_error(void) { return g_err.c_str(); }

sw_status sw_db_pack(const int8_t* d_residues, const int64_t* h_offsets, int64_t n, const sw_pack_opts* opts,
                     sw_stream stream, sw_db** out) {
    g_err.clear();
    return pack_db(d_residues, h_offsets, n, opts, nullptr, 0, static_cast<hipStream_t>(stream), out);
}

sw_status sw_db_pack_into(const int8_t* d_residues, const int64_t* h_offsets, int64_t n, const sw_pack_opts* opts,
                          void* d_db, int64_t db_bytes, sw_stream stream, sw_db** out) {
    g_err.clear();
    if (!d_db) return fail(SW_E_INVALID, "d_db is NULL");
    return pack_db(d_residues, h_offsets, n, opts, d_db, db_bytes, static_cast<hipStream_t>(stream), out);
}

sw_status sw_db_pack_bytes(const int64_t* h_offsets, int64_t n, const sw_pack_opts* opts, int64_t* bytes) {
    g_err.clear();
    (void)opts;                       // the image does not depend on the options
    if (!bytes) return fail(SW_E_INVALID, "bytes is NULL");
    PackPlan P;
    sw_status s = plan_pack(h_offsets, n, &P);
    if (s != SW_OK) return s;
    *bytes = db_layout(n, P.G, P.image_bytes).total;
    return SW_OK;
}

sw_status sw_db_tune(sw_db* db, const sw_pack_opts* opts) {
    g_err.clear();
    if (!db || !opts) return fail(SW_E_INVALID, "NULL argument");
    std::lock_guard<std::mutex> lk(db->mu);
    DeviceGuard dg(db->device);
    sw_db probe;
    sw_status s = apply_opts(&probe, opts);        // validate before touching the handle
    if (s != SW_OK) return s;
    HIP_TRY(hipDeviceSynchronize());               // no search of this handle may be in flight
    apply_opts(db, opts);
    clear_caches(db);
    return SW_OK;
}

void sw_db_free(sw_db* db) {
    if (!db) return;
    DeviceGuard dg(db->device);
    hipDeviceSynchronize();
    clear_caches(db);
    db->image_own.release();           // a caller's image stays the caller's
    db->align_dirs.release(); db->align_bnd.release(); db->align_misc.release(); db->align_host.release();
    db->mode_plan.release();
    db->ws_own.release();
    for (HostPinned& h : db->hstage) h.release();
    for (auto& e : db->ev_pool) { hipEventDestroy(e.first); hipEventDestroy(e.second); }
    if (db->side) hipStreamDestroy(db->side);
    if (db->side2) hipStreamDestroy(db->side2);
    if (db->cap) hipStreamDestroy(db->cap);
    if (db->graph.done) hipEventDestroy(db->graph.done);
    if (db->ev_fork) hipEventDestroy(db->ev_fork);
    if (db->ev_join) hipEventDestroy(db->ev_join);
    if (db->ev_join2) hipEventDestroy(db->ev_join2);
    delete db;
}

sw_status sw_db_info(const sw_db* db, int64_t* n, int64_t* residues, int64_t* device_bytes) {
    if (!db) return fail(SW_E_INVALID, "db is NULL");
    if (n) *n = db->n;
    if (residues) *residues = db->total_res;
    if (device_bytes) {
        // everything the handle itself allocated: its image, workspace, plan copies, alignment buffers
        size_t b = db->image_own.bytes + db->ws_own.bytes + db->align_dirs.bytes + db->align_bnd.bytes +
                   db->align_misc.bytes + db->mode_plan.items.bytes + db->multi_plan.items.bytes + db->multi_plan.qpairs.bytes;
        for (const auto& kv : db->plans) b += kv.second.items.bytes + kv.second.qpairs.bytes;
        for (const Plan& p : db->batch_plan) b += p.items.bytes + p.qpairs.bytes;
        *device_bytes = (int64_t)b;
    }
    return SW_OK;
}

sw_status sw_search(const int8_t* h_query, int32_t qlen, sw_db* db, const int64_t* h_offsets, int64_t n,
                    const int8_t* h_subst, int32_t gap_open, int32_t gap_extend, int32_t* d_scores_out,
                    sw_stream stream) {
    g_err.clear();
    return search_one(h_query, qlen, db, h_offsets, n, h_subst, gap_open, gap_extend, d_scores_out, nullptr, 0,
                      static_cast<hipStream_t>(stream));
}

sw_status sw_search_ws(const int8_t* h_query, int32_t qlen, sw_db* db, const int64_t* h_offsets, int64_t n,
                       const int8_t* h_subst, int32_t gap_open, int32_t gap_extend, int32_t* d_scores_out,
                       void* d_workspace, int64_t ws_bytes, sw_stream stream) {
    g_err.clear();
    if (!d_workspace) return fail(SW_E_INVALID, "workspace is NULL");
    return search_one(h_query, qlen, db, h_offsets, n, h_subst, gap_open, gap_extend, d_scores_out, d_workspace,
                      ws_bytes, static_cast<hipStream_t>(stream));
}

sw_status sw_topk(const int32_t* d_scores, int64_t n, int32_t k, int32_t* d_top_scores, int64_t* d_top_index,
                  sw_stream stream) {
    return sw_topk_ws(d_scores, n, k, d_top_scores, d_top_index, nullptr, 0, stream);
}

sw_status sw_topk_ws_bytes(int64_t n, int32_t k, int64_t* bytes) {
    g_err.clear();
    if (!bytes) return fail(SW_E_INVALID, "bytes is NULL");
    if (n < 0) return fail(SW_E_INVALID, "n must be >= 0");
    if (k < 1 || k > 1024) return fail(SW_E_UNSUPPORTED, "k must be in 1..1024 (got %d)", k);
    *bytes = topk_ws_bytes(n, 1, k);
    return SW_OK;
}

sw_status sw_topk_ws(const int32_t* d_scores, int64_t n, int32_t k, int32_t* d_top_scores, int64_t* d_top_index,
                     void* d_workspace, int64_t ws_bytes, sw_stream stream) {
    g_err.clear();
    if (n < 0) return fail(SW_E_INVALID, "n must be >= 0");
    if (k < 1 || k > 1024) return fail(SW_E_UNSUPPORTED, "k must be in 1..1024 (got %d)", k);
    if ((n > 0 && !d_scores) || !d_top_scores || !d_top_index) return fail(SW_E_INVALID, "NULL pointer");
    const hipStream_t st = static_cast<hipStream_t>(stream);
    const int64_t need = topk_ws_bytes(n, 1, k);
    if (d_workspace && need > 0 && ws_bytes < need) return fail(SW_E_SIZE, "workspace of %lld bytes < %lld", (long long)ws_bytes, (long long)need);
    HIP_TRY(launch_topk_ws(d_scores, n, n, 1, k, d_top_scores, d_top_index, need > 0 ? d_workspace : nullptr, st));
    return SW_OK;
}

sw_status sw_search_batch(const int8_t* h_queries, const int64_t* h_qoffsets, int32_t nq, sw_db* db,
                          const int8_t* h_subst, int32_t gap_open, int32_t gap_extend, int32_t k, int32_t* d_scores,
                          int32_t* d_top_scores, int64_t* d_top_index, sw_stream stream) {
    g_err.clear();
    return search_batch(h_queries, h_qoffsets, nq, db, h_subst, gap_open, gap_extend, k, d_scores, d_top_scores,
                        d_top_index, nullptr, 0, static_cast<hipStream_t>(stream));
}

sw_status sw_search_batch_ws(const int8_t* h_queries, const int64_t* h_qoffsets, int32_t nq, sw_db* db,
                             const int8_t* h_subst, int32_t gap_open, int32_t gap_extend, int32_t k, int32_t* d_scores,
                             int32_t* d_top_scores, int64_t* d_top_index, void* d_workspace, int64_t ws_bytes,
                             sw_stream stream) {
    g_err.clear();
    if (!d_workspace) return fail(SW_E_INVALID, "workspace is NULL");
    return search_batch(h_queries, h_qoffsets, nq, db, h_subst, gap_open, gap_extend, k, d_scores, d_top_scores,
                        d_top_index, d_workspace, ws_bytes, static_cast<hipStream_t>(stream));
}

sw_status sw_batch_workspace_bytes(sw_db* db, const int64_t* h_qoffsets, int32_t nq, int32_t k, int32_t scores_in_ws,
                                   int64_t* bytes) {
    g_err.clear();
    sw_status s;
    if (!db || !bytes) return fail(SW_E_INVALID, "NULL argument");
    if (nq < 0 || (nq > 0 && !h_qoffsets)) return fail(SW_E_INVALID, "bad query offsets");
    if (k < 0 || k > 1024) return fail(SW_E_UNSUPPORTED, "k must be in 0..1024 (got %d)", k);
    for (int q = 0; q < nq; ++q)
        if (h_qoffsets[q + 1] < h_qoffsets[q]) return fail(SW_E_INVALID, "query offsets decrease at %d", q);
    std::lock_guard<std::mutex> lk(db->mu);
    DeviceGuard dg(db->device);
    if ((s = ensure_geometry(db)) != SW_OK) return s;
    std::vector<int> qlens(nq);
    for (int q = 0; q < nq; ++q) qlens[q] = (int)(h_qoffsets[q + 1] - h_qoffsets[q]);
    Plan* plan = nullptr;
    if ((s = plan_for(db, qlens, kPlanCut, &plan)) != SW_OK) return s;
    const int64_t zero[1] = {0};
    *bytes = ws_layout(db, nq ? h_qoffsets : zero, nq, k, scores_in_ws != 0, PlanRoom(*plan, nq)).total;
    return SW_OK;
}

sw_status sw_search_multi(const int8_t* h_queries, const int64_t* h_qoffsets, int32_t nq, const int32_t* h_chunk,
                          int32_t nchunks, sw_db* db, const int8_t* h_subst, int32_t gap_open, int32_t gap_extend,
                          int32_t* const* h_d_scores, sw_stream stream) {
    g_err.clear();
    sw_status s;
    if (!db) return fail(SW_E_INVALID, "db is NULL");
    if ((s = check_subst_gaps(h_subst, gap_open, gap_extend)) != SW_OK) return s;
    if (nq < 0 || nchunks < 1) return fail(SW_E_INVALID, "nq must be >= 0 and nchunks >= 1");
    if (nq > 0 && (!h_qoffsets || !h_queries || !h_chunk || !h_d_scores)) return fail(SW_E_INVALID, "NULL argument");
    for (int q = 0; q < nq; ++q) {
        if (h_qoffsets[q + 1] < h_qoffsets[q]) return fail(SW_E_INVALID, "query offsets decrease at %d", q);
        if (h_qoffsets[q + 1] - h_qoffsets[q] > (1 << 24)) return fail(SW_E_UNSUPPORTED, "query %d too long", q);
        if (h_chunk[q] < 0 || h_chunk[q] >= nchunks) return fail(SW_E_INVALID, "chunk %d of query %d outside 0..%d", h_chunk[q], q, nchunks - 1);
        if (db->n > 0 && !h_d_scores[q]) return fail(SW_E_INVALID, "score vector of query %d is NULL", q);
    }
    if (nq > 0)
        for (int64_t i = h_qoffsets[0]; i < h_qoffsets[nq]; ++i)
            if (h_queries[i] < 0 || h_queries[i] >= db->alphabet) return fail(SW_E_RESIDUE, "query residue outside 0..%d at %lld", db->alphabet - 1, (long long)i);
    if (nq == 0 || db->n == 0) return SW_OK;
    std::lock_guard<std::mutex> lk(db->mu);
    DeviceGuard dg(db->device);
    hipStream_t st = static_cast<hipStream_t>(stream);
    if ((s = ensure_geometry(db)) != SW_OK) return s;
    std::vector<int> qlens(nq), chunk(h_chunk, h_chunk + nq);
    for (int q = 0; q < nq; ++q) qlens[q] = (int)(h_qoffsets[q + 1] - h_qoffsets[q]);
    // a zero-length query scores 0 on its chunk: fill its whole vector (other chunks are 0 as well)
    for (int q = 0; q < nq; ++q)
        if (qlens[q] == 0) HIP_TRY(launch_fill(h_d_scores[q], db->n, 0, st));
    HIP_TRY(hipStreamSynchronize(st));              // the previous call may still read the plan buffer
    const CellForm form = choose_form(db, h_subst, gap_open, gap_extend, h_queries, h_qoffsets, nq);
    if ((s = build_plan(db, qlens, plan_kind(form, gap_extend), &db->multi_plan, &chunk, nchunks)) != SW_OK) return s;
    if (db->multi_plan.h_items.empty()) return SW_OK;
    Work W;
    if ((s = get_work(db, h_qoffsets, nq, 0, false, &db->multi_plan, PlanRoom(), nullptr, 0, &W)) != SW_OK) return s;
    Staged S;
    if ((s = stage_queries(db, W, h_queries, h_qoffsets, nq, h_subst, gap_open, gap_extend, 0, st, &S, h_d_scores)) != SW_OK) return s;
    return enqueue(db, S, form, db->multi_plan, W, gap_open, gap_extend, nullptr, db->n, 0, nullptr, nullptr, st, true);
}

sw_status sw_profile_kernels(sw_db* db, int32_t enable) {
    if (!db) return fail(SW_E_INVALID, "db is NULL");
    std::lock_guard<std::mutex> lk(db->mu);
    db->timing = enable != 0;
    db->ev_used.clear();
    return SW_OK;
}

sw_status sw_kernel_times(sw_db* db, float* ms_out, int32_t cap, int32_t* count) {
    if (!db || !count || (cap > 0 && !ms_out)) return fail(SW_E_INVALID, "NULL argument");
    std::lock_guard<std::mutex> lk(db->mu);
    DeviceGuard dg(db->device);
    *count = 0;
    for (int i : db->ev_used) {
        HIP_TRY(hipEventSynchronize(db->ev_pool[i].second));
        float ms = 0.f;
        HIP_TRY(hipEventElapsedTime(&ms, db->ev_pool[i].first, db->ev_pool[i].second));
        if (*count < cap) ms_out[(*count)++] = ms;
    }
    db->ev_used.clear();
    return SW_OK;
}

sw_status sw_last_stats(sw_db* db, int64_t out[8]) {
    if (!db || !out) return fail(SW_E_INVALID, "NULL argument");
    DeviceGuard dg(db->device);
    int32_t c[kSplits] = {};
    if (db->last_counters) {
        HIP_TRY(hipDeviceSynchronize());
        HIP_TRY(hipMemcpy(c, db->last_counters, sizeof c, hipMemcpyDeviceToHost));
    }
    out[0] = db->last_items;
    out[1] = c[1];
    out[2] = db->last_rows;
    out[3] = (int64_t)db->last_grid * kWaves;
    out[4] = db->last_side_items;
    out[5] = db->last_side_rows;
    out[6] = c[5];
    out[7] = std::max<int64_t>(0, (int64_t)c[1] - db->last_cap);
    return SW_OK;
}

}  // extern "C"

// ------------------------------------------------------------------ alignments
namespace {
constexpr int64_t kAlignBudget = (int64_t)4 << 30;   // direction bytes per round of pairs
// Most pinned memory a handle keeps for alignments: what a call exchanges goes through it in one copy each way, or the
// operations that come back in pieces.  (Pinning takes a first call about 0.3 ms a MiB: 16 MiB at once made that of
// 5,000 alignments 10.3 ms, 7.1 without any.)
constexpr size_t kAlignPinned = (size_t)2 << 20;
}

sw_status sw_align_batch(const int8_t* h_queries, const int64_t* h_qoffsets, int32_t nq, sw_db* db,
                         const int64_t* h_subjects, const int64_t* h_soffsets, const int8_t* h_subst, int32_t gap_open,
                         int32_t gap_extend, sw_alignment* h_out, char* h_ops, int64_t ops_stride, sw_stream stream) {
    g_err.clear();
    sw_status s;
    if (!db) return fail(SW_E_INVALID, "db is NULL");
    if ((s = check_subst_gaps(h_subst, gap_open, gap_extend)) != SW_OK) return s;
    if (nq < 0) return fail(SW_E_INVALID, "nq must be >= 0");
    if (nq > 0 && (!h_qoffsets || !h_soffsets)) return fail(SW_E_INVALID, "NULL offsets");
    if (nq == 0) return SW_OK;
    if (h_soffsets[0] < 0) return fail(SW_E_INVALID, "subject offsets start below 0");
    for (int32_t q = 0; q < nq; ++q) {
        const int64_t m = h_qoffsets[q + 1] - h_qoffsets[q];
        if (m < 0) return fail(SW_E_INVALID, "query offsets decrease at %d", q);
        if (m > (1 << 20)) return fail(SW_E_UNSUPPORTED, "query %d longer than 2^20 residues", q);
        if (h_soffsets[q + 1] < h_soffsets[q]) return fail(SW_E_INVALID, "subject offsets decrease at %d", q);
        if (m > 0 && !h_queries) return fail(SW_E_INVALID, "queries is NULL");
        for (int64_t i = h_qoffsets[q]; i < h_qoffsets[q + 1]; ++i)
            if (h_queries[i] < 0 || h_queries[i] >= db->alphabet)
                return fail(SW_E_RESIDUE, "query %d residue %d at %lld outside 0..%d", q, h_queries[i],
                            (long long)(i - h_qoffsets[q]), db->alphabet - 1);
    }
    const int64_t s0 = h_soffsets[0], npairs = h_soffsets[nq] - s0;
    if (npairs > 0 && (!h_subjects || !h_out || !h_ops)) return fail(SW_E_INVALID, "NULL subjects or outputs");
    for (int32_t q = 0; q < nq; ++q) {
        const int64_t m = h_qoffsets[q + 1] - h_qoffsets[q];
        for (int64_t k = h_soffsets[q]; k < h_soffsets[q + 1]; ++k) {
            const int64_t sub = h_subjects[k - s0];
            if (sub < 0 || sub >= db->n) return fail(SW_E_INVALID, "subject index %lld outside 0..n-1", (long long)sub);
            if (ops_stride < m + db->lens[sub])
                return fail(SW_E_SIZE, "ops_stride %lld < query + subject (%lld) for query %d", (long long)ops_stride,
                            (long long)(m + db->lens[sub]), q);
            h_out[k - s0] = sw_alignment{0, 0, 0, sub, 0, 0, 0};
        }
    }
    // pairs with a non-empty query, longest first, so that the biggest fills start first
    struct Job { int64_t k; int32_t q; int32_t m; int32_t n; int64_t cost; };
    std::vector<Job> jobs;
    for (int32_t q = 0; q < nq; ++q) {
        const int32_t m = (int32_t)(h_qoffsets[q + 1] - h_qoffsets[q]);
        if (m == 0) continue;
        for (int64_t k = h_soffsets[q]; k < h_soffsets[q + 1]; ++k) {
            const int32_t n = db->lens[h_subjects[k - s0]];
            jobs.push_back({k - s0, q, m, n, align_dir_bytes(m, n)});
        }
    }
    if (jobs.empty()) return SW_OK;
    std::stable_sort(jobs.begin(), jobs.end(), [](const Job& a, const Job& b) { return a.cost > b.cost; });
    std::lock_guard<std::mutex> lk(db->mu);
    DeviceGuard dg(db->device);
    hipStream_t st = static_cast<hipStream_t>(stream);
    // penalties above every score (at most 127 x 2^20) all mean that no gap pays; capped, no difference overflows
    const int32_t go = std::min(gap_open, 1 << 28), ge = std::min(gap_extend, 1 << 28);
    size_t j0 = 0;
    while (j0 < jobs.size()) {
        // a round: pairs whose direction bytes fit the budget (at least one pair)
        size_t j1 = j0;
        int64_t dir_total = 0, columns = 0, stride = 1;
        int nbands = 0;
        std::vector<int32_t> qs_used;
        while (j1 < jobs.size()) {
            const Job& J = jobs[j1];
            if (j1 > j0 && dir_total + J.cost > kAlignBudget) break;
            dir_total += round_up(J.cost, 256);
            columns += J.n;
            nbands += align_bands(J.m, J.n);
            stride = std::max<int64_t>(stride, (int64_t)J.m + J.n + 1);
            qs_used.push_back(J.q);
            ++j1;
        }
        std::sort(qs_used.begin(), qs_used.end());
        qs_used.erase(std::unique(qs_used.begin(), qs_used.end()), qs_used.end());
        const int np = (int)(j1 - j0);
        // one buffer: what the host sends (pairs | bands | matrix | queries), the end cells of the bands, and what
        // comes back (best, 3 int32 a pair | info, 4 int64 a pair | operations)
        const size_t o_bands = round_up(sizeof(AlignPair) * np, 256);
        const size_t o_sm = o_bands + round_up(sizeof(AlignBand) * (size_t)nbands, 256);
        const size_t o_query = o_sm + 1024;
        std::vector<int64_t> qpos(nq, -1);
        size_t qbytes = 0;
        for (int32_t q : qs_used) {
            qpos[q] = (int64_t)qbytes;
            qbytes += (size_t)round_up(h_qoffsets[q + 1] - h_qoffsets[q], 256);
        }
        const size_t o_ends = o_query + qbytes;
        const size_t o_best = o_ends + round_up(12 * (int64_t)nbands, 256);
        const size_t o_info = o_best + round_up(12 * (size_t)np, 256);
        const size_t o_ops = o_info + round_up(32 * (size_t)np, 256);
        const size_t misc = o_ops + (size_t)np * stride;
        HIP_TRY(db->align_dirs.reserve((size_t)std::max<int64_t>(dir_total, 256)));
        // the bands' counter (256 bytes) and the rows between bands
        const int64_t bnd_bytes = 256 + 16 * columns;
        HIP_TRY(db->align_bnd.reserve((size_t)bnd_bytes));
        HIP_TRY(db->align_misc.reserve(misc));
        char* mb = db->align_misc.as<char>();
        HIP_TRY(db->align_host.reserve(std::min(misc, kAlignPinned)));
        char* const pinned = static_cast<char*>(db->align_host.p);
        std::vector<char> plain;
        if (o_ends > kAlignPinned) plain.resize(o_ends);
        char* hb = plain.empty() ? pinned : plain.data();
        AlignPair* pairs = reinterpret_cast<AlignPair*>(hb);
        int64_t dir_off = 0, bnd_off = 0;
        int32_t ends = 0;
        std::vector<int32_t> rest(np);
        for (int i = 0; i < np; ++i) {
            const Job& J = jobs[j0 + i];
            const int64_t sub = h_subjects[J.k];
            const int32_t slot = db->slot_of[sub];
            const int g = slot / kGroupSubjects, w = slot % kGroupSubjects;
            AlignPair& P = pairs[i];
            P.residues = db->d_image + db->gbase[g] + (int64_t)(w >> 1) * 8 + (w & 1) * 4;
            P.n = J.n;
            P.m = J.m;
            P.query = reinterpret_cast<const int8_t*>(mb + o_query + qpos[J.q]);
            P.dir_off = dir_off;
            P.bnd_off = bnd_off;
            P.ends = ends;
            dir_off += round_up(J.cost, 256);
            bnd_off += J.n;
            ends += align_bands(J.m, J.n);
            rest[i] = i;
        }
        // the first bands of all pairs, then the second ones, ...: a band comes after the one it waits for
        AlignBand* bands = reinterpret_cast<AlignBand*>(hb + o_bands);
        for (int32_t k = 0, at = 0; !rest.empty(); ++k) {
            rest.erase(std::remove_if(rest.begin(), rest.end(),
                                      [&](int32_t i) { return align_bands(pairs[i].m, pairs[i].n) <= k; }), rest.end());
            for (int32_t i : rest) bands[at++] = AlignBand{i, k};
        }
        memcpy(hb + o_sm, h_subst, (size_t)db->alphabet * db->alphabet);
        for (int32_t q : qs_used)
            memcpy(hb + o_query + qpos[q], h_queries + h_qoffsets[q], (size_t)(h_qoffsets[q + 1] - h_qoffsets[q]));
        HIP_TRY(hipMemcpyAsync(mb, hb, o_ends, hipMemcpyHostToDevice, st));
        HIP_TRY(launch_fill(db->align_bnd.as<int32_t>(), bnd_bytes / 4, 0, st));
        const AlignPair* d_pairs = reinterpret_cast<AlignPair*>(mb);
        int32_t* d_ends = reinterpret_cast<int32_t*>(mb + o_ends);
        HIP_TRY(launch_align_fill(d_pairs, reinterpret_cast<AlignBand*>(mb + o_bands), nbands, db->align_bnd.as<int32_t>(),
                                  reinterpret_cast<int8_t*>(mb + o_sm), db->alphabet, go, ge, db->align_dirs.as<uint8_t>(),
                                  reinterpret_cast<uint64_t*>(db->align_bnd.as<char>() + 256), d_ends, st));
        HIP_TRY(launch_align_trace(d_pairs, np, db->align_dirs.as<uint8_t>(), d_ends, reinterpret_cast<int32_t*>(mb + o_best),
                                   mb + o_ops, stride, reinterpret_cast<int64_t*>(mb + o_info), st));
        // the results of pairs [i0, i1), whose ends, begins and counts are at `head` and operations at `ops`
        auto take = [&](int i0, int i1, const char* head, const char* ops) -> sw_status {
            const int32_t* best = reinterpret_cast<const int32_t*>(head);
            const int64_t* info = reinterpret_cast<const int64_t*>(head + (o_info - o_best));
            for (int i = i0; i < i1; ++i) {
                const Job& J = jobs[j0 + i];
                if (info[4 * i + 3] != 0)
                    return fail(SW_E_HIP, "inconsistent traceback for subject %lld", (long long)h_subjects[J.k]);
                sw_alignment& A = h_out[J.k];
                const int64_t len = info[4 * i + 2];
                A.score = best[3 * i];
                A.q_begin = (int32_t)info[4 * i];
                A.q_end = best[3 * i + 1];
                A.s_begin = info[4 * i + 1];
                A.s_end = best[3 * i + 2];
                A.n_ops = len;
                memcpy(h_ops + J.k * ops_stride, ops + (size_t)(i - i0 + 1) * stride - len, (size_t)len);
            }
            return SW_OK;
        };
        if (misc <= kAlignPinned) {
            HIP_TRY(hipMemcpyAsync(pinned + o_best, mb + o_best, misc - o_best, hipMemcpyDeviceToHost, st));
            HIP_TRY(hipStreamSynchronize(st));
            if ((s = take(0, np, pinned + o_best, pinned + o_ops)) != SW_OK) return s;
        } else {
            std::vector<char> head(o_ops - o_best), one;
            const int some = (int)std::max<int64_t>(1, (int64_t)kAlignPinned / stride);
            if ((size_t)stride > kAlignPinned) one.resize((size_t)stride);
            char* const at = one.empty() ? pinned : one.data();
            HIP_TRY(hipMemcpyAsync(head.data(), mb + o_best, head.size(), hipMemcpyDeviceToHost, st));
            for (int i = 0; i < np; i += some) {
                const int n = std::min(some, np - i);
                HIP_TRY(hipMemcpyAsync(at, mb + o_ops + (size_t)i * stride, (size_t)n * stride, hipMemcpyDeviceToHost, st));
                HIP_TRY(hipStreamSynchronize(st));
                if ((s = take(i, i + n, head.data(), at)) != SW_OK) return s;
            }
        }
        j0 = j1;
    }
    return SW_OK;
}

sw_status sw_align(const int8_t* h_query, int32_t qlen, sw_db* db, const int64_t* h_subjects, int32_t nsub,
                   const int8_t* h_subst, int32_t gap_open, int32_t gap_extend, sw_alignment* h_out, char* h_ops,
                   int64_t ops_stride, sw_stream stream) {
    g_err.clear();
    if (!db) return fail(SW_E_INVALID, "db is NULL");
    if (qlen < 0 || nsub < 0) return fail(SW_E_INVALID, "qlen and nsub must be >= 0");
    if (qlen > 0 && !h_query) return fail(SW_E_INVALID, "query is NULL");
    const int64_t qo[2] = {0, qlen}, so[2] = {0, nsub};
    return sw_align_batch(h_query, qo, 1, db, h_subjects, so, h_subst, gap_open, gap_extend, h_out, h_ops, ops_stride,
                          stream);
}

// ------------------------------------------------------------------ end-to-end modes
namespace {
int64_t gap_run(int64_t k, int64_t go, int64_t ge) { return k <= 0 ? 0 : -(go + (k - 1) * std::min(go, ge)); }
}

sw_status sw_search_mode(int32_t mode, const int8_t* h_query, int32_t qlen, sw_db* db, const int64_t* h_offsets,
                         int64_t n, const int8_t* h_subst, int32_t gap_open, int32_t gap_extend, int32_t* d_scores_out,
                         sw_stream stream) {
    if (mode == SW_LOCAL)
        return sw_search(h_query, qlen, db, h_offsets, n, h_subst, gap_open, gap_extend, d_scores_out, stream);
    g_err.clear();
    if (mode != SW_GLOBAL && mode != SW_SEMIGLOBAL) return fail(SW_E_INVALID, "mode must be 0, 1 or 2 (got %d)", mode);
    sw_status s;
    if ((s = check_db_args(db, h_offsets, n)) != SW_OK) return s;
    if ((s = check_subst_gaps(h_subst, gap_open, gap_extend)) != SW_OK) return s;
    if (qlen < 0) return fail(SW_E_INVALID, "qlen must be >= 0");
    if (qlen > 0 && !h_query) return fail(SW_E_INVALID, "query is NULL");
    if (n > 0 && !d_scores_out) return fail(SW_E_INVALID, "scores_out is NULL");
    for (int32_t i = 0; i < qlen; ++i)
        if (h_query[i] < 0 || h_query[i] >= db->alphabet)
            return fail(SW_E_RESIDUE, "query residue %d at %d outside 0..%d", h_query[i], i, db->alphabet - 1);
    // every value of the recurrence stays within +-2^29: gap runs cost at most Go + (m + n) max(Go, Ge)
    const int64_t span = (int64_t)qlen + db->ncols_max + 1;
    if ((int64_t)gap_open + span * std::max(gap_open, gap_extend) >= ((int64_t)1 << 29) || span * 127 >= ((int64_t)1 << 29))
        return fail(SW_E_UNSUPPORTED, "gap penalties x lengths too large for 32-bit end-to-end scores");
    if (n == 0) return SW_OK;
    std::lock_guard<std::mutex> lk(db->mu);
    DeviceGuard dg(db->device);
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (qlen == 0) {
        // one gap run per subject (global) or nothing to align (semi-global)
        std::vector<int32_t> v((size_t)n);
        for (int64_t k = 0; k < n; ++k) v[k] = mode == SW_GLOBAL ? (int32_t)gap_run(db->lens[k], gap_open, gap_extend) : 0;
        HIP_TRY(hipMemcpyAsync(d_scores_out, v.data(), sizeof(int32_t) * n, hipMemcpyHostToDevice, st));
        HIP_TRY(hipStreamSynchronize(st));
        return SW_OK;
    }
    if ((s = ensure_geometry(db)) != SW_OK) return s;
    const int64_t qo[2] = {0, qlen};
    const CellForm form = choose_mode_form(db, mode, h_subst, gap_open, gap_extend, qlen);
    if (form.cell == kCellOff) {
        // one launch, planned as a local search's; not for a stream under capture, as with the plain cells below
        hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
        HIP_TRY(hipStreamIsCapturing(st, &cap));
        if (cap != hipStreamCaptureStatusNone) return fail(SW_E_HIP, "end-to-end search on a stream under capture");
        Plan* plan = nullptr;
        if ((s = get_plan(db, qlen, plan_kind(form, gap_extend), &plan)) != SW_OK) return s;
        Work W;
        if ((s = get_work(db, qo, 1, 0, false, plan, PlanRoom(), nullptr, 0, &W)) != SW_OK) return s;
        Staged S;
        if ((s = stage_queries(db, W, h_query, qo, 1, h_subst, gap_open, gap_extend, 0, st, &S, nullptr, nullptr, mode)) != SW_OK)
            return s;
        return enqueue(db, S, form, *plan, W, gap_open, gap_extend, d_scores_out, n, 0, nullptr, nullptr, st, true);
    }
    if (db->wg_mode == 0) {
        int b1 = 0, b2 = 0;
        int b3 = 0;
        HIP_TRY(sweep_occupancy_mode16(SW_GLOBAL, 16, &b1));
        HIP_TRY(sweep_occupancy_mode16(SW_SEMIGLOBAL, 16, &b2));
        HIP_TRY(sweep_occupancy_mode16(kModeGlobalOffset, 16, &b3));
        const int b = std::min(std::min(std::min(b1, b2), b3), kMaxWgPerCu);
        if (b < 1) return fail(SW_E_HIP, "16-bit end-to-end sweep cannot be resident");
        db->wg_mode = std::min(db->cus * b, db->wg16);     // within the 16-bit boundary slots
    }
    // Plain cells (gaps or substitution scores that offset cells cannot hold, or a query too long for them).
    // 16-bit cells hold values in [128 - bias, kModeTop - bias).  Semi-global H never falls below the
    // gap run down the query, g(m) = -(Go + (m - 1) Ge), so its bias is just large enough for that (at
    // most the middle of the range), which leaves the most room above for high scores.  Global mode with
    // Ge <= Go runs on column-offset cells H' = H - g(j) (g(j) the row-0 gap run to column j): every H'
    // is at least g(m) too, whatever the subject's length, so it takes the same bias; the profile then
    // carries SM + Ge, E extends for free and opens at Go - Ge, and a score is H'[m][n] + g(n).  Global
    // mode with Ge > Go keeps plain cells at the middle of the range, and so do long queries: their own
    // bias is high, and their long similar subjects are lifted by -g(n) as well, so high scorers leave
    // the range and go to the serial 32-bit recompute, where plain cells run the longest subjects in
    // 32 bits beside the 16-bit launch.  Offset cells are used while the query's bias stays within 2/5
    // of the middle one (queries up to about 3,100 residues at 10/2): there the 32-bit chain of a long
    // subject, which they remove, is the longer path (measured on the 570,000-subject workload).
    const int64_t offset_bias = 128 + (int64_t)gap_open + (int64_t)(qlen - 1) * gap_extend;
    const bool offset = mode == SW_GLOBAL && gap_extend <= gap_open && 5 * offset_bias <= 2 * (int64_t)kModeBias;
    int32_t bias = kModeBias;
    if (mode == SW_SEMIGLOBAL || offset)
        bias = (int32_t)std::min<int64_t>(kModeBias, 128 + (int64_t)gap_open + (int64_t)(qlen - 1) * gap_extend);
    // A query whose column-0 border (the gap run down its length) falls below the range runs wholly in
    // 32-bit cells; with plain global cells so do the longest subjects, whose row-0 border does (a prefix
    // of the length-sorted groups).
    const int64_t lowest = 128 - (int64_t)bias;
    int g_split = 0;                              // groups [0, g_split) run in 32-bit cells
    if (gap_run(qlen, gap_open, gap_extend) < lowest) g_split = db->ngroups;
    else if (mode == SW_GLOBAL && !offset)
        while (g_split < db->ngroups && gap_run(db->ncols[g_split], gap_open, gap_extend) < lowest) ++g_split;
    const bool use_offset = offset && g_split == 0;
    const int mode16 = use_offset ? kModeGlobalOffset : mode;      // the 16-bit kernels' form
    const int32_t sm_shift = use_offset ? gap_extend : 0;
    // 16-bit plan at 16 rows per lane; the long pairs of a short query go to a side list at 4 or 8 rows
    std::vector<WgItem> mi, si, m32, s32, none;
    if (g_split < db->ngroups) {
        PlanLimits lim{16, db->slot_cap, (int64_t)db->wg_mode * kWaves};
        lim.side = true;
        plan_units(db, std::vector<int>{qlen}, kPlanPlain, &db->mode_plan, mi, si, none, nullptr, 1, &lim, g_split, -1,
                   &db->mode_side_rows);
    }
    // (4 rows per lane measured no faster for the 32-bit chain of a short query, and slower for longer ones)
    constexpr int R32 = 8;
    if (g_split > 0) {
        // 32-bit units in the 32-bit boundary slots: one wave slot holds the widest subject's columns
        const PlanLimits lim32{R32, std::max<int64_t>(db->ncols_max, 4), (int64_t)db->wg32 * kWaves};
        Plan tmp;
        plan_units(db, std::vector<int>{qlen}, kPlanPlain, &tmp, m32, s32, none, nullptr, 1, &lim32, 0, g_split);
    }
    HIP_TRY(hipStreamSynchronize(st));            // the plan buffer may still be read by an earlier launch
    // device item list: [16-bit main..., 16-bit side..., 32-bit...]
    const size_t n16 = mi.size(), n16s = si.size(), n_items = n16 + n16s + m32.size();
    HIP_TRY(db->mode_plan.items.reserve(sizeof(WgItem) * std::max<size_t>(n_items, 1)));
    mi.insert(mi.end(), si.begin(), si.end());
    mi.insert(mi.end(), m32.begin(), m32.end());
    if (n_items) HIP_TRY(hipMemcpy(db->mode_plan.items.p, mi.data(), sizeof(WgItem) * n_items, hipMemcpyHostToDevice));
    Work W;
    if ((s = get_work(db, qo, 1, 0, false, nullptr, PlanRoom(), nullptr, 0, &W)) != SW_OK) return s;
    Staged S;
    if ((s = stage_queries(db, W, h_query, qo, 1, h_subst, gap_open, gap_extend, 0, st, &S)) != SW_OK) return s;
    int32_t* ctr = W.counters;
    HIP_TRY(launch_profile(S.sm_q, db->alphabet, S.qd, S.nq, S.qoff, W.prof, ctr, kCounters, W.bits, W.L.bits_words,
                           S.max_mp, st, sm_shift, kPadScore));
    SweepArgs a = sweep_args(db, S, W, gap_open, gap_extend, d_scores_out);
    a.sm_shift = sm_shift;
    a.items = db->mode_plan.items.as<WgItem>();
    a.n_items = (int32_t)n16;
    a.counter = ctr + 0;
    set_rerun_args(db, a, W, ctr);
    a.unit_list = 0;
    // every value carries the bias; a pair whose H leaves [128, sat) is recomputed
    a.bias = bias;
    a.sat = db->sat < kSat16 ? std::min<int32_t>(bias + db->sat, kModeTop) : kModeTop;
    // the 16-bit side launch takes the first slots; the 16-bit bulk launch fills the rest
    const int grid_side = n16s ? std::min<int>((int)n16s, std::max(1, db->wg_mode / 8)) : 0;
    const int grid = std::max(1, std::min<int>(db->wg_mode - grid_side, std::max<int>((int)n16, 1)));
    if (n16s || !m32.empty()) {
        HIP_TRY(hipEventRecord(db->ev_fork, st));
        if (n16s) HIP_TRY(hipStreamWaitEvent(db->side, db->ev_fork, 0));
        if (!m32.empty()) HIP_TRY(hipStreamWaitEvent(db->side2, db->ev_fork, 0));
    }
    if (n16s) {
        // long pairs of a short query at fewer rows per lane, concurrently on the side stream
        SweepArgs b = a;
        b.items = db->mode_plan.items.as<WgItem>() + n16;
        b.n_items = (int32_t)n16s;
        b.counter = ctr + 3;
        b.slot_base = grid;
        HIP_TRY(launch_sweep_mode16(mode16, db->mode_side_rows, b, grid_side, db->side));
        HIP_TRY(hipEventRecord(db->ev_join, db->side));
    }
    if (!m32.empty()) {
        // the longest subjects in 32-bit cells, concurrently on the second side stream
        SweepArgs b = a;
        b.items = db->mode_plan.items.as<WgItem>() + n16 + n16s;
        b.n_items = (int32_t)m32.size();
        b.counter = ctr + 4;
        b.scratch = W.scratch32;
        b.slot_words = (int64_t)std::max<int32_t>(db->ncols_max, 4) * 4;
        b.rerun = nullptr;
        b.rerun_count = nullptr;
        b.rerun_cap = 0;
        b.poison = 0;
        b.bias = 0;
        HIP_TRY(launch_sweep_mode(mode, R32, b, std::max(1, std::min<int>(db->wg32, (int)m32.size())), db->side2));
        HIP_TRY(hipEventRecord(db->ev_join2, db->side2));
    }
    const int ev = db->timing ? record_timer_start(db, st) : -1;
    if (n16 > 0) HIP_TRY(launch_sweep_mode16(mode16, 16, a, grid, st));
    // the recompute reads the side launches' rerun entries and reuses the 32-bit slots; the timed
    // region of the sweep ends when all three launches have
    if (n16s) HIP_TRY(hipStreamWaitEvent(st, db->ev_join, 0));
    if (!m32.empty()) HIP_TRY(hipStreamWaitEvent(st, db->ev_join2, 0));
    if (ev >= 0) {
        HIP_TRY(hipEventRecord(db->ev_pool[ev].second, st));
        db->ev_used.push_back(ev);
    }
    // exact 32-bit recompute of the pairs that left the range; the count is read on the device
    SweepArgs r = recompute_args(db, a, W, ctr);
    r.bias = 0;
    HIP_TRY(launch_sweep_mode(mode, kRerunRows, r, db->wg32, st));
    db->last_items = (int)n16;
    db->last_rows = 16;
    db->last_side_items = (int)(n16s + m32.size());
    db->last_side_rows = n16s ? db->mode_side_rows : m32.empty() ? 0 : R32;
    db->last_grid = grid + grid_side;
    db->last_counters = ctr;
    return SW_OK;
}
