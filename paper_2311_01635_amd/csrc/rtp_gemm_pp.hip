// Launcher of the tiled 16-bit GEMMs (rtp_gemm_pp.h, rtp_gemm_duo.h): shape rules, the choice of tiles for a
// launch (one GEMM or a group of independent ones) and the order of the group's problems.
#include "rtp_gemm_duo.h"

#include <string.h>

#include <algorithm>
#include <map>
#include <mutex>
#include <utility>

namespace rtp {

hipError_t launch_gemm_pp_nt_bf16(const PpGroup &g, hipStream_t s, hipEvent_t done);
hipError_t launch_gemm_pp_nn_bf16(const PpGroup &g, hipStream_t s, hipEvent_t done);
hipError_t launch_gemm_pp_tn_bf16(const PpGroup &g, hipStream_t s, hipEvent_t done);
hipError_t launch_gemm_pp_nt_f16(const PpGroup &g, hipStream_t s, hipEvent_t done);
hipError_t launch_gemm_pp_nn_f16(const PpGroup &g, hipStream_t s, hipEvent_t done);
hipError_t launch_gemm_pp_tn_f16(const PpGroup &g, hipStream_t s, hipEvent_t done);
hipError_t launch_gemm_pp_nn_tn_bf16(const PpGroup &g, hipStream_t s, hipEvent_t done);
hipError_t launch_gemm_pp_nn_tn_f16(const PpGroup &g, hipStream_t s, hipEvent_t done);
hipError_t launch_gemm_duo_nt_bf16(const PpGroup &g, hipStream_t s);
hipError_t launch_gemm_duo_nn_tn_bf16(const PpGroup &g, hipStream_t s);
hipError_t launch_gemm_duo_nt_f16(const PpGroup &g, hipStream_t s);
hipError_t launch_gemm_duo_nn_tn_f16(const PpGroup &g, hipStream_t s);

bool gemm_bf16_pp_supported(int layout, const GemmArgs &a)
{
    // a partial last sub-tile is read as zeros past K; fp16 layers are defined on whole sub-tiles only
    if (a.K <= 0 || (a.elem != ELEM_BF16 && (a.K & 31))) return false;
    if (layout == LAY_TN && a.M < 8) return false;
    if (layout != LAY_NT && a.N < 8) return false;
    // the kernel addresses each operand through a buffer descriptor with 32-bit byte offsets
    const bool a_kc = layout != LAY_TN, b_kc = layout == LAY_NT;
    const int64_t a_elems = (int64_t)((a_kc ? a.M : a.K) - 1) * a.lda + (a_kc ? a.K : a.M);
    const int64_t b_elems = (int64_t)((b_kc ? a.N : a.K) - 1) * a.ldb + (b_kc ? a.K : a.N);
    if (a_elems * 2 >= (int64_t)1 << 31 || b_elems * 2 >= (int64_t)1 << 31) return false;
    return true;
}

static int compute_units()
{
    static int cus = 0;
    if (cus == 0) {
        int dev = 0, n = 0;
        if (hipGetDevice(&dev) == hipSuccess &&
            hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && n > 0)
            cus = n;
        else
            cus = 256;
    }
    return cus;
}

// A tile is named by its height in gemm_pp_kernel (256, 192, 128: 256 wide; 64: 128 wide) or the code SMALL_128X128, by one of
// the codes DUO_* in gemm_duo_kernel.
static bool is_duo(int tile) { return tile >= DUO_128X128; }
static bool is_small(int tile) { return tile == 64 || tile == SMALL_128X128; } // rtp_gemm_small.h
static int tile_rows(int tile) { return tile == DUO_128X128 || tile == SMALL_128X128 ? 128 : is_duo(tile) ? 64 : tile; }
// output columns of a tile, and of each half for the paired epilogue
static int tile_cols(int tile) { return is_duo(tile) ? (tile == DUO_64X64 ? 64 : 128) : is_small(tile) ? pps::BN : pp::BN; }
static int tile_width(const GemmArgs &a, int tile) { return a.epi == EPI_SWIGLU_FWD ? tile_cols(tile) / 2 : tile_cols(tile); }
static int tile_bk(int tile, int lay) { return is_duo(tile) ? ppd::sub_tile(lay, tile_rows(tile)) : is_small(tile) ? pps::BK : pp::BK; }
static int tiles_n_of(const GemmArgs &a, int bm)
{
    const int ncols = a.epi == EPI_SWIGLU_FWD ? a.half : a.N, bn = tile_width(a, bm);
    return (ncols + bn - 1) / bn;
}
static int tiles_m_of(const GemmArgs &a, int bm) { return (a.M + tile_rows(bm) - 1) / tile_rows(bm); }
// K chunks that are not empty when the K loop of a tile of height bm is cut in `ksplit`; *each: sub-tiles of a chunk
static int k_chunks(const GemmArgs &a, int bm, int ksplit, int *each, int lay = LAY_NT)
{
    const int bk = tile_bk(bm, lay);
    const int kt = (a.K + bk - 1) / bk;
    *each = (kt + ksplit - 1) / ksplit;
    return (kt + *each - 1) / *each;
}

int gemm_bf16_pp_tiles_n(const GemmArgs &a) { return tiles_n_of(a, 128); } // (a producer never takes the small tile)

// ---- run-time estimate of a launch ------------------------------------------------------
// Unit: one K sub-tile (32) of a 256 x 256 tile.  A tile costs its K loop plus its epilogue,
// scaled by its height; the shorter tiles carry a small handicap because they move more
// operand bytes per flop.  The epilogue terms stand for the HBM traffic of the tile's results
// (fp32 read-modify-write of an accumulator is the heaviest) in units of main-loop steps.
static double epilogue_steps(int epi, int c_is_f32)
{
    switch (epi) {
    case EPI_ACC_ADD: return 30.0;
    case EPI_ACC_ATOMIC: return 40.0;
    case EPI_ACC_FIRST: return 16.0;
    case EPI_ACC_LAST: return 22.0;
    case EPI_SWIGLU_FWD: return 14.0;
    case EPI_GELU_ERF_FWD:
    case EPI_GELU_TANH_FWD: return 16.0;
    case EPI_SWIGLU_BWD: return 20.0;
    case EPI_GELU_ERF_BWD:
    case EPI_GELU_TANH_BWD: return 14.0;
    default: return c_is_f32 ? 16.0 : 8.0;
    }
}

// The 64 x 128 tile: a fixed part and a part per 64 K (the 128 x 128 one half a unit more and 1.45 times; beside another GEMM
// 1.6 times, with 1.45 a step of three 4864-wide shards on the streams took 2 % longer).  Launches alone (us, launch
// included): one round 512 x 2752 x 4096 21.0, two rounds 2048 x 1792 x 8192 75 and 992 x 4096 x 14336 139, three rounds 8192 x 768 x 2048 37.3 and
// 8192 x 768 x 384 16.6 (the 128-high tile: 50.4, 91, 168, 31.6, 11.6) give 1.5 and 0.44.  Beside another GEMM both are
// larger, as it fetches twice the bytes per flop: with 1.5 and 0.44 there too the ragged Llama-shaped step took 3.80 ms
// and the expert layer's 17.15, with 3.0 and 0.5 3.73 and 17.00.
struct SmallCost {
    double fixed, step;
};
constexpr SmallCost SMALL_ALONE = {1.5, 0.44}, SMALL_SHARED = {3.0, 0.5};

// frac: the share of the K loop's MFMA time an edge tile still needs (1 for an interior tile), area: the share
// of the tile that exists (scales the epilogue's traffic)
static double tile_cost(const GemmArgs &a, int bm, int ksplit, double frac = 1.0, double area = 1.0)
{
    int each;
    (void)k_chunks(a, bm, ksplit, &each);
    const SmallCost small = a.cu_share > 1 ? SMALL_SHARED : SMALL_ALONE;
    if (bm == SMALL_128X128)
        return small.fixed + 0.5 + (a.cu_share > 1 ? 1.6 : 1.45) * small.step * each + area * epilogue_steps(ksplit > 1 ? EPI_ACC_ATOMIC : a.epi, a.c_is_f32) / 4.0;
    if (bm == 64) // 64 x 128, sub-tiles of 64
        return small.fixed + small.step * each + area * epilogue_steps(ksplit > 1 ? EPI_ACC_ATOMIC : a.epi, a.c_is_f32) / 8.0;
    const double handicap = bm == 256 ? 1.0 : bm == 192 ? 1.04 : 1.12;
    // (an edge tile still fetches whole sub-tiles and passes every barrier: a floor under its loop time)
    const double loop = each * std::max(frac, 0.35);
    return handicap * (bm / 256.0) * (loop + area * epilogue_steps(ksplit > 1 ? EPI_ACC_ATOMIC : a.epi, a.c_is_f32));
}

// The kernel skips the fragments of an edge tile that lie wholly outside the matrix; the tile then runs as long
// as its busiest wave.  Waves split the tile's rows in two halves (BM / 64 fragment rows each) and hold two
// fragment columns 128 apart (gate / up halves of the paired epilogue: always both or none).
static void edge_shares(const GemmArgs &a, int bm, double *frac_m, double *area_m, double *frac_n, double *area_n)
{
    const int rows = tile_rows(bm), tm = (a.M + rows - 1) / rows, vr = a.M - (tm - 1) * rows; // valid rows of the last tile row
    const int fm = rows / 64;
    *frac_m = vr >= rows / 2 || is_small(bm) ? 1.0 : (double)((vr + 31) / 32) / fm; // (the small tile skips nothing)
    *area_m = (double)vr / rows;
    const bool paired = a.epi == EPI_SWIGLU_FWD;
    const int ncols = paired ? a.half : a.N, bn = tile_width(a, bm);
    const int tn = (ncols + bn - 1) / bn, vc = ncols - (tn - 1) * bn;
    *frac_n = paired || vc > 128 || is_small(bm) ? 1.0 : 0.5;
    *area_n = (double)vc / bn;
}

// A problem may have its K loop cut into chunks when its result is an fp32 sum onto an accumulator
// (the chunks' partial sums are added atomically) and it is short of tiles: the weight-gradient
// GEMM of a narrow shard contracts over all T tokens into an output of a few tiles.  The order of those adds is not
// fixed, so such a result does not repeat bit for bit.  Only whole sub-tiles and outputs of at least 64 x 64 are split:
// a batch of any other number of tokens, and a narrower shard, give the same gradients on every run.
static bool may_split_k(const GemmArgs &a)
{
    if (a.sync) return false; // the counters count whole tiles
    if ((a.K & 31) || a.M < 64 || a.N < 64) return false;
    return a.epi == EPI_ACC_ADD && a.c_is_f32 && a.C == (void *)a.ws && a.ldc == a.ldws;
}

// Greedy list schedule: each job goes to the server that is free first.  Servers free at one time are kept as one entry, so a
// run of equal jobs costs an entry a round, not a heap operation a job; the times are those of one job at a time.  (First
// plans on the host, mean of 1000 backward pairs: 165 -> 48 us; forward 89 -> 35.)
class Servers {
    static constexpr int MOST = 128;
    struct {
        double time;
        int count;
    } free_at[MOST]; // ascending times (no more entries than servers)
    int entries = 1;
public:
    explicit Servers(int count)
    {
        free_at[0].time = 0.0;
        free_at[0].count = std::min(count, MOST);
    }
    double next() const { return free_at[0].time; }
    // `jobs` jobs of `cost`; the time the last of them ends at, 0 for none
    double run(long jobs, double cost)
    {
        double last = 0.0;
        while (jobs > 0) {
            const int took = (int)std::min<long>(jobs, free_at[0].count);
            last = free_at[0].time + cost;
            jobs -= took;
            if ((free_at[0].count -= took) == 0) std::copy(free_at + 1, free_at + entries--, free_at);
            int at = entries;
            while (at > 0 && free_at[at - 1].time > last) --at;
            if (at > 0 && free_at[at - 1].time == last) {
                free_at[at - 1].count += took;
            } else {
                std::copy_backward(free_at + at, free_at + entries, free_at + entries + 1);
                ++entries;
                free_at[at].time = last;
                free_at[at].count = took;
            }
        }
        return last;
    }
};

// problems in descending order of cost, equal ones as they were
static void longest_first(int *order, const double *cost, int count)
{
    for (int i = 1; i < count; ++i)
        for (int k = i; k > 0 && cost[order[k]] > cost[order[k - 1]]; --k) std::swap(order[k], order[k - 1]);
}

// Schedule of one XCD's share (an eighth of each problem, rounded up) over its
// compute units, problems in the order given: the finishing time of the last tile.
static double makespan(const GemmArgs *a, const int *bm, const int *ks, const int *order, int count, int cus_per_xcd, bool whole_tile = true)
{
    Servers units(cus_per_xcd);
    double end = 0.0;
    for (int i = 0; i < count; ++i) {
        const int q = order[i];
        int each;
        const int chunks = k_chunks(a[q], bm[q], ks[q], &each);
        const long tm = tiles_m_of(a[q], bm[q]), tn = tiles_n_of(a[q], bm[q]);
        const long tiles = tm * tn * chunks;
        const long mine = (tiles + 7) / 8;
        // interior tiles, then the last tile column, the last tile row and the corner, each with its own cost
        double fm, am, fn, an;
        edge_shares(a[q], bm[q], &fm, &am, &fn, &an);
        const double cost[4] = {tile_cost(a[q], bm[q], ks[q]), tile_cost(a[q], bm[q], ks[q], fn, an),
                                tile_cost(a[q], bm[q], ks[q], fm, am), tile_cost(a[q], bm[q], ks[q], fm * fn, am * an)};
        const long cls[4] = {(tm - 1) * (tn - 1) * chunks, (tm - 1) * chunks, (tn - 1) * chunks, (long)chunks};
        // this XCD's share of each class: the edge classes rounded up, the interior takes the rest
        long cnt[4] = {0, 0, 0, 0}, left = mine;
        for (int c = 3; c >= 1; --c) {
            cnt[c] = std::min(left, (cls[c] * mine + tiles - 1) / tiles);
            left -= cnt[c];
        }
        cnt[0] = left;
        // No launch ends before one whole tile has: that share may leave out every class but the cheapest (a single tile
        // per XCD is always the corner), and the fragments an edge tile skips shorten a busy machine's work, not its own
        // K loop (768 x 2048 at height 192: 28 us for 8 rows as for 200).  Priced by the corner alone, those launches
        // went to tall tiles; the small tile takes 10.4 and 10.8 us.
        if (whole_tile) end = std::max(end, units.next() + cost[0]);
        // cheap tiles first: the grid hands tiles out in index order, not longest first, so the tile that starts a
        // further round is as likely a full one as not; an estimate that kept the cheap ones for last favoured plans
        // whose last round never comes out that short (a K split that spilled 8 tiles into a second round)
        for (int c = 3; c >= 0; --c) end = std::max(end, units.run(cnt[c], cost[c]));
    }
    return end;
}

// Heights, K splits and launch order (longest tiles first) of a group.  Every combination is tried
// (5 tiles, and up to 6 split factors for a problem that may be split and is short of tiles);
// the estimate above picks.  Plans are remembered per shape.
struct PlanKey {
    int layout, count, cu_share, square;
    int dims[PP_MAX_GROUP][6]; // M, N, K, epi, forced height, chunks it may be split in
    bool operator<(const PlanKey &o) const { return memcmp(this, &o, sizeof *this) < 0; }
};
struct Plan {
    int bm[PP_MAX_GROUP], ks[PP_MAX_GROUP], order[PP_MAX_GROUP];
};
// Plans by what they were made from.  An expert layer plans for each number of tokens that it meets: once full the store
// starts anew (a plan takes some ten us).
template <typename Key>
class PlanStore {
    static constexpr size_t MOST = 8192;
    std::map<Key, Plan> plans;
    std::mutex lock;
public:
    bool find(const Key &key, Plan *plan)
    {
        std::lock_guard<std::mutex> g(lock);
        const auto it = plans.find(key);
        if (it == plans.end()) return false;
        *plan = it->second;
        return true;
    }
    void keep(const Key &key, const Plan &plan)
    {
        std::lock_guard<std::mutex> g(lock);
        if (plans.size() >= MOST) plans.clear();
        plans[key] = plan;
    }
};

// whether a tile of gemm_duo_kernel takes the problem
static bool duo_takes(const GemmArgs &a, int tile)
{
    if (tile < DUO_128X128 || tile > DUO_64X64 || a.sync || !gemm_epilogue_vec_ok(a)) return false;
    return tile != DUO_64X64 || a.epi != EPI_SWIGLU_FWD; // (a wave of it holds one fragment column: no pairs)
}

// the height a caller asks for; 0 (pick) also for one that is not built, or that the problem's counters cannot take
static int forced_height(const GemmArgs &a, int asked)
{
    const bool built = asked == 256 || asked == 192 || asked == 128 || (is_small(asked) && !a.sync);
    return built ? asked : 0;
}

constexpr int MAX_SPLIT = 32;

// Where a sum's K loop is cut is part of its result: it decides the order of the additions, and whether they have one (one
// chunk repeats bit for bit, two do onto zeros).  The plan of the tall and the 64 x 128 tiles decides that; whatever tile then
// runs the problem cuts a sum of one chunk or two where that plan does, and one of more, which does not repeat, in two or
// more but not in more than that.  (Free to cut them anew, the other tiles took 1.5 % off the GPT-2-shaped step, 817 -> 804 us,
// with four chunks of a 384 x 768 sum over 8192 instead of two.)
static bool keeps_cuts(const GemmArgs &a, int ref_tile, int ref_ks, int tile, int ks, int lay)
{
    int ref_each, each;
    const int ref = k_chunks(a, ref_tile, ref_ks, &ref_each, lay), chunks = k_chunks(a, tile, ks, &each, lay);
    if (ref > 2) return chunks >= 2 && chunks <= ref;
    return chunks == ref && (chunks == 1 || each * tile_bk(tile, lay) == ref_each * tile_bk(ref_tile, lay));
}

// Whether 128 x 128 tiles would fill the machine more than one and a half times, where the estimate above prices them too low.
// Products alone, the other tiles -> these: at 1.8 to 2 fillings 0.83 to 1.1 times as fast, at 2.8 to 3 0.76 to 0.85 (3480 x
// 3448 x 5440 121 -> 150 us), at 4.1 to 4.3 0.81 to 0.95 (at just under four 1.1, given up); up to 1.3 0.98 to 1.6.  Units with such
// shards, us: training, 6488 tokens 2816 -> 7488 over 8 2825 -> 3129, 6096 tokens 1152 -> 3456 over 3 578 -> 676; at 1.34 to 1.5,
// forward, 992 tokens 6912 -> 21568 gated over 8 1748 -> 1561, 2008 tokens 3008 -> 5440 gated over 8 500 -> 442.
static bool crowded(const GemmArgs &a, int chunks)
{
    return 2L * tiles_m_of(a, SMALL_128X128) * tiles_n_of(a, SMALL_128X128) * chunks > 3L * compute_units();
}

// max_split (may be null): chunks of K each problem may be cut in; square: whether 128 x 128 tiles are considered
static Plan plan_group(int layout, const GemmArgs *given, int count, const int *bm_override, int cu_share, const int *max_split = nullptr,
                       bool square = true)
{
    static PlanStore<PlanKey> plans;
    GemmArgs a[PP_MAX_GROUP]; // priced for the share the plan is remembered under, not for what each problem says
    for (int q = 0; q < count; ++q) {
        a[q] = given[q];
        a[q].cu_share = cu_share;
    }
    PlanKey key;
    memset(&key, 0, sizeof key);
    key.layout = layout; key.count = count; key.cu_share = cu_share; key.square = square;
    int cap[PP_MAX_GROUP];
    for (int q = 0; q < count; ++q) {
        const int forced = bm_override ? forced_height(a[q], bm_override[q]) : 0;
        cap[q] = !may_split_k(a[q]) ? 1 : max_split ? max_split[q] : MAX_SPLIT;
        const int d[6] = {a[q].M, a[q].N, a[q].K, a[q].epi + (a[q].sync ? 64 : 0), forced, cap[q]};
        memcpy(key.dims[q], d, sizeof d);
    }
    Plan best_plan;
    if (plans.find(key, &best_plan)) return best_plan;
    Plan ref; // the plan without 128 x 128 tiles
    if (square) ref = plan_group(layout, given, count, bm_override, cu_share, max_split, false);
    const int heights[5] = {256, 192, 128, 64, SMALL_128X128};
    const int splits[6] = {1, 2, 4, 8, 16, MAX_SPLIT};
    const int cus = std::max(8, compute_units() / std::max(1, cu_share));
    const int cus_per_xcd = std::max(1, cus / 8);
    // A launch that shares the machine (cu_share > 1) seldom gets exactly its share: its partner on the other
    // stream may be a GEMM of a hundred tiles, or done already.  The estimate is the mean of the two ends, its
    // share of the compute units and all of them, which is what the in-situ sweeps of the tile heights favour
    // (a 96-tile GEMM planned for half the machine kept its 256-high tiles and left compute units idle).
    auto estimate = [&](const GemmArgs *p, const int *bm, const int *ks, const int *order, int n, bool whole_tile = true) {
        const double t = makespan(p, bm, ks, order, n, cus_per_xcd, whole_tile);
        return cu_share > 1 ? 0.5 * (t + makespan(p, bm, ks, order, n, std::max(1, compute_units() / 8), whole_tile)) : t;
    };
    // Whether a sum is split at all: only where a tall tile's split beats every tall tile, the unsplit ones priced by
    // one XCD's share alone.  That is cheap where an XCD gets a tile or two, and errs towards gradients that repeat.
    auto worth_splitting = [&](const GemmArgs &p) {
        const int heights[3] = {256, 192, 128}, splits[6] = {1, 2, 4, 8, 16, 32}, zero = 0;
        double best = 1e300;
        bool split = false;
        for (int h : heights)
            for (int k : splits) {
                if (k > 1 && p.K / 32 / k < 4) break;
                const double t = estimate(&p, &h, &k, &zero, 1, false);
                if (t < best - 1e-9) best = t, split = k > 1;
            }
        return split;
    };
    // options per problem
    int nopt[PP_MAX_GROUP], obm[PP_MAX_GROUP][30], oks[PP_MAX_GROUP][30];
    for (int q = 0; q < count; ++q) {
        nopt[q] = 0;
        const int forced = bm_override ? forced_height(a[q], bm_override[q]) : 0;
        const long tiles128 = (long)((a[q].M + 127) / 128) * tiles_n_of(a[q], 128);
        const bool split_ok = cap[q] > 1 && (square ? ref.ks[q] > 1 : tiles128 < cus && worth_splitting(a[q]));
        for (int h = 0; h < 5; ++h) {
            if (!square && forced == 0 && heights[h] == SMALL_128X128) continue;
            if (forced != 0 && forced != heights[h]) continue;
            if (is_small(heights[h]) && a[q].sync) continue; // the counters are the tall tiles'
            for (int k = 0; k < (split_ok ? 6 : 1); ++k) {
                if (splits[k] > cap[q]) break;
                if (splits[k] > 1 && (a[q].K + 31) / 32 / splits[k] < (is_small(heights[h]) ? 8 : 4)) break; // keep at least four sub-tiles per chunk
                if (forced == 0 && heights[h] == SMALL_128X128 && crowded(a[q], splits[k])) continue;
                if (square && !keeps_cuts(a[q], ref.bm[q], ref.ks[q], heights[h], splits[k], layout)) continue;
                obm[q][nopt[q]] = heights[h];
                oks[q][nopt[q]] = splits[k];
                ++nopt[q];
            }
        }
    }
    memset(&best_plan, 0, sizeof best_plan);
    double best = 1e300;
    if (square) best_plan = ref, best = estimate(a, ref.bm, ref.ks, ref.order, count);
    int idx[PP_MAX_GROUP] = {0, 0, 0, 0};
    for (;;) {
        int bm[PP_MAX_GROUP], ks[PP_MAX_GROUP], order[PP_MAX_GROUP];
        for (int q = 0; q < count; ++q) {
            bm[q] = obm[q][idx[q]];
            ks[q] = oks[q][idx[q]];
            order[q] = q;
        }
        bool ordered = false; // a producer / consumer pair keeps the order it was given in
        for (int q = 0; q < count; ++q) ordered = ordered || a[q].sync != nullptr;
        if (!ordered) {
            double cost[PP_MAX_GROUP];
            for (int q = 0; q < count; ++q) cost[q] = tile_cost(a[q], bm[q], ks[q]);
            longest_first(order, cost, count);
        }
        const double t = estimate(a, bm, ks, order, count);
        if (t < best - 1e-9) {
            best = t;
            for (int q = 0; q < count; ++q) {
                best_plan.bm[q] = bm[q];
                best_plan.ks[q] = ks[q];
                best_plan.order[q] = order[q];
            }
        }
        int q = 0;
        while (q < count && ++idx[q] == nopt[q]) idx[q++] = 0;
        if (q == count) break;
    }
    plans.keep(key, best_plan);
    return best_plan;
}

// ---- the kernel of a riding launch -------------------------------------------------------
// A launch that rides has the machine to itself and is priced in us for both kernels.  `once` a launch, and for each tile
// a compute unit works through `fixed` and `step` a sub-tile (of 32 K in tall tiles, else 64; `step_full` more where the
// machine is full of accumulators and its clock drops).  Fitted to the kernel times of 70 shapes drawn from the layers' ranges
// (16 to 8192 tokens, shards of 64 to 1536) and of 4096^3 products: within 7 (64 x 64) to 15 % (192 x 256).  A compute unit with
// one workgroup of the duo kernel waits for its operands between the sub-tiles of the two wider tiles (per_unit: tiles a
// unit).
// Passes, the tall and the 64 x 128 tile everywhere -> all of them where this estimate prefers them: 50 drawn units and layers
// 0.95 to 1.37 times as fast, geometric mean 1.09; 80 forward passes of 96 to 4096 tokens 1.17, 36 of 16 to 256 tokens
// with shards of 40 to 180 MB 1.06, one of them behind (68 tokens, 8192 -> 22272 over 3, 280 -> 304: 232 tiles of 64 x 64 that
// read 122 MB of weights leave the transfers no compute unit).
struct TileTime {
    double once, fixed, step, step_full;
};
static TileTime tile_time(int tile, int epi, int per_unit)
{
    const double pairs = epi == EPI_SWIGLU_FWD ? 1.08 : 1.0; // (such launches came out that much later than their estimate)
    switch (tile) {
    case 256: return {0.0, 9.1, 0.406, 0.27};
    case 192: return {0.0, 7.8, 0.380, 0.16};
    case 128: return {0.0, 6.7, 0.316, 0.14};
    case 64: return {1.4, 4.3, 0.208, 0.05};
    case SMALL_128X128: return {1.4, 5.5, 0.35, 0.11};
    case DUO_128X128: return {3.8, 1.9, pairs * (per_unit <= 1 ? 0.70 : per_unit == 2 ? 0.42 : 0.44), 0.0};
    case DUO_64X128: return {3.9, 1.7, pairs * (per_unit <= 1 ? 0.40 : per_unit == 2 ? 0.30 : 0.285), 0.0};
    default: return {3.4, 1.25, per_unit <= 1 ? 0.21 : 0.178, 0.0};
    }
}
// bytes the epilogue moves per element of the product
static double epilogue_bytes(int epi, int c_is_f32)
{
    switch (epi) {
    case EPI_ACC_ADD: return 8.0;
    case EPI_ACC_ATOMIC: return 16.0;
    case EPI_ACC_FIRST: return 4.0;
    case EPI_ACC_LAST: return c_is_f32 ? 8.0 : 6.0;
    case EPI_SWIGLU_FWD: return 3.0;
    case EPI_SWIGLU_BWD: return 8.0;
    case EPI_STORE: return c_is_f32 ? 4.0 : 2.0;
    default: return 4.0;
    }
}
// Schedule of one XCD's share over its compute units (the two workgroups a unit may hold of the duo kernel share
// its load path, so they count as one after the other).  The transfers have no part in it: priced beside the tiles, those of a
// prompt hid what the tiles cost, and gated units of 16 to 768 tokens went to the duo kernel, whose tiles for them take half
// as long again (us a forward pass, 320 tokens 3456 -> 13120 over 8: 349 on the tall tiles, 411, now 353; 160 tokens 2688 ->
// 8928 over 6: 218, 258, 215; without gates 200 tokens 4928 -> 18144 over 12: 536, 566, 497.  240 units and layers, against
// the transfers priced: 0.94 to 1.2 times as fast, the slower ones where the estimate had been off both ways, 536 -> 571 for 256
// tokens 5696 -> 15536 gated over 2).
static double launch_us(const GemmArgs *a, const int *tile, const int *ks, const int *order, int count)
{
    const int cus = compute_units(), servers = std::max(1, cus / 8);
    double area = 0.0, once = 0.0;
    long tiles = 0;
    for (int q = 0; q < count; ++q) {
        int each;
        const long n = (long)tiles_m_of(a[q], tile[q]) * tiles_n_of(a[q], tile[q]) * k_chunks(a[q], tile[q], ks[q], &each);
        tiles += n;
        area += (double)n * tile_rows(tile[q]) * tile_cols(tile[q]);
    }
    const double full = std::min(1.0, area / (cus * 65536.0));
    Servers units(servers);
    double end = 0.0, busy[PP_MAX_GROUP], loop[PP_MAX_GROUP], whole[PP_MAX_GROUP];
    long count_of[PP_MAX_GROUP];
    for (int i = 0; i < count; ++i) {
        const int q = order[i];
        int each;
        const int chunks = k_chunks(a[q], tile[q], ks[q], &each);
        const long n = ((long)tiles_m_of(a[q], tile[q]) * tiles_n_of(a[q], tile[q]) * chunks + 7) / 8;
        const TileTime t = tile_time(tile[q], a[q].epi, (int)std::min<long>(3, (tiles + cus - 1) / cus));
        once = std::max(once, t.once);
        const double cost = t.fixed + each * (t.step + full * t.step_full) +
                            full * tile_rows(tile[q]) * tile_cols(tile[q]) * epilogue_bytes(chunks > 1 ? EPI_ACC_ATOMIC : a[q].epi, a[q].c_is_f32) * cus / 10e6;
        busy[q] = each * t.step / cost;
        loop[q] = each * t.step;
        whole[q] = cost;
        count_of[q] = n;
        end = std::max(end, units.run(n, cost));
    }
    if (is_duo(tile[0]) && tiles > cus) { // a tile beside another all along: the slower, the longer that one multiplies
        double share = 0.0, sum = 0.0;
        for (int q = 0; q < count; ++q) share += busy[q] * whole[q] * count_of[q], sum += whole[q] * count_of[q];
        for (int q = 0; q < count; ++q) end = std::max(end, whole[q] + 1.2 * loop[q] * share / sum);
    }
    return end + once;
}

// The best plan of gemm_duo_kernel for the group that keeps the cuts of `ref`.  False if there is none.
static bool plan_duo(const int *layouts, const GemmArgs *a, int count, const Plan &ref, Plan *best_plan, double *best)
{
    const int splits[6] = {1, 2, 4, 8, 16, MAX_SPLIT};
    int nopt[PP_MAX_GROUP], otile[PP_MAX_GROUP][18], oks[PP_MAX_GROUP][18];
    for (int q = 0; q < count; ++q) {
        nopt[q] = 0;
        for (int tile = DUO_128X128; tile <= DUO_64X64; ++tile)
            for (int k : splits) {
                if (!duo_takes(a[q], tile) || (k > 1 && (ref.ks[q] == 1 || a[q].K / 32 / k < 8))) break;
                if (!keeps_cuts(a[q], ref.bm[q], ref.ks[q], tile, k, layouts[q])) continue;
                otile[q][nopt[q]] = tile;
                oks[q][nopt[q]++] = k;
            }
        if (nopt[q] == 0) return false;
    }
    *best = 1e300;
    int idx[PP_MAX_GROUP] = {0, 0, 0, 0};
    for (;;) {
        Plan p;
        memset(&p, 0, sizeof p);
        double cost[PP_MAX_GROUP];
        for (int q = 0; q < count; ++q) {
            p.bm[q] = otile[q][idx[q]];
            p.ks[q] = oks[q][idx[q]];
            p.order[q] = q;
            int each;
            (void)k_chunks(a[q], p.bm[q], p.ks[q], &each);
            cost[q] = each * tile_time(p.bm[q], a[q].epi, 3).step;
        }
        longest_first(p.order, cost, count);
        const double t = launch_us(a, p.bm, p.ks, p.order, count);
        if (t < *best - 1e-9) *best = t, *best_plan = p;
        int q = 0;
        while (q < count && ++idx[q] == nopt[q]) idx[q++] = 0;
        if (q == count) return true;
    }
}

void gemm_bf16_pp_plan(int layout, const GemmArgs *a, int count, const int *bm_override, int *bm_out, int *ksplit_out)
{
    if (count < 1 || count > PP_MAX_GROUP) return;
    const Plan pl = plan_group(layout, a, count, bm_override, count == 1 ? a[0].cu_share : 1);
    for (int q = 0; q < count; ++q) {
        if (bm_out) bm_out[q] = pl.bm[q];
        if (ksplit_out) ksplit_out[q] = pl.ks[q];
    }
}

// the group's tiles in the order of its plan, behind them the transfers that ride along (may be null)
static hipError_t launch_group(int layout, const int *layouts, const GemmArgs *a, int count, const Plan &pl, const Riders *riders,
                               hipStream_t s, hipEvent_t done)
{
    const int *bm = pl.bm, *order = pl.order;
    const bool duo = is_duo(bm[0]); // (a plan's tiles are of one kernel)
    PpGroup g;
    memset(&g, 0, sizeof g);
    g.count = count;
    unsigned per_xcd = 0;
    long tiles = 0;
    for (int i = 0; i < count; ++i) {
        const int q = order[i];
        PpProblem &p = g.p[i];
        p.a = a[q];
        p.lay = layouts ? layouts[q] : layout;
        p.bm = tile_rows(bm[q]);
        p.bn = tile_cols(bm[q]);
        p.tiles_m = tiles_m_of(a[q], bm[q]);
        p.tiles_n = tiles_n_of(a[q], bm[q]);
        p.vec_epilogue = gemm_epilogue_vec_ok(a[q]) ? 1 : 0;
        // as many chunks as are not empty
        int each;
        p.ksplit = k_chunks(a[q], bm[q], pl.ks[q], &each, p.lay);
        if (p.ksplit > 1) p.a.epi = EPI_ACC_ATOMIC;
        per_xcd += (unsigned)(((long)p.tiles_m * p.tiles_n * p.ksplit + 7) / 8);
        tiles += (long)p.tiles_m * p.tiles_n * p.ksplit;
    }
    g.tile_blocks = per_xcd * 8;
    if (riders) {
        if (riders->sums > 0 && !takes_sums(layout)) return hipErrorInvalidValue;
        const int slots = compute_units() * (duo ? 2 : 1);
        const hipError_t e = ride_list(*riders, std::max(64, slots - (int)std::min<long>(tiles, 1 << 20)), &g.ride);
        if (e != hipSuccess) return e;
        g.sum_blocks = (g.ride.sum_blocks + 7) / 8 * 8;
        for (int i = 0; i < riders->sums; ++i)
            if (riders->sum[i].elem != a[0].elem) return hipErrorInvalidValue;
    }
    const bool f16 = a[0].elem == ELEM_F16;
    if (duo) {
        if (done) return hipErrorInvalidValue;
        if (layout == LAY_NT) return f16 ? launch_gemm_duo_nt_f16(g, s) : launch_gemm_duo_nt_bf16(g, s);
        return f16 ? launch_gemm_duo_nn_tn_f16(g, s) : launch_gemm_duo_nn_tn_bf16(g, s);
    }
    switch (layout) {
    case LAY_NT: return f16 ? launch_gemm_pp_nt_f16(g, s, done) : launch_gemm_pp_nt_bf16(g, s, done);
    case LAY_NN: return f16 ? launch_gemm_pp_nn_f16(g, s, done) : launch_gemm_pp_nn_bf16(g, s, done);
    case LAY_TN: return f16 ? launch_gemm_pp_tn_f16(g, s, done) : launch_gemm_pp_tn_bf16(g, s, done);
    case LAY_NN_TN: return f16 ? launch_gemm_pp_nn_tn_f16(g, s, done) : launch_gemm_pp_nn_tn_bf16(g, s, done);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_gemm_bf16_pp_group(int layout, const GemmArgs *a_in, int count_in, const int *bm_override, hipStream_t s,
                                     hipEvent_t done)
{
    if (count_in < 0 || count_in > PP_MAX_GROUP) return hipErrorInvalidValue;
    GemmArgs a[PP_MAX_GROUP];
    int forced[PP_MAX_GROUP];
    int count = 0;
    for (int q = 0; q < count_in; ++q) {
        if (a_in[q].M <= 0 || a_in[q].N <= 0) continue; // nothing to compute
        if (!gemm_bf16_args_ok(layout, a_in[q]) || !gemm_bf16_pp_supported(layout, a_in[q])) return hipErrorInvalidValue;
        if (count > 0 && a_in[q].elem != a[0].elem) return hipErrorInvalidValue; // one element type per launch
        forced[count] = bm_override ? bm_override[q] : 0;
        a[count++] = a_in[q];
    }
    if (count == 0) return done ? hipEventRecord(done, s) : hipSuccess; // nothing to launch: the event still marks this point
    if (count == 1 && is_duo(forced[0])) {
        if (!duo_takes(a[0], forced[0])) return hipErrorInvalidValue;
        Plan pl;
        memset(&pl, 0, sizeof pl);
        pl.bm[0] = forced[0], pl.ks[0] = 1;
        return launch_group(layout, nullptr, a, 1, pl, nullptr, s, done);
    }
    const Plan pl = plan_group(layout, a, count, forced, count == 1 ? a[0].cu_share : 1);
    return launch_group(layout, nullptr, a, count, pl, nullptr, s, done);
}

// the layout code of a launch that holds problems of these layouts, -1 if no kernel does
static int common_layout(const int *layouts, int count)
{
    int lay = layouts[0];
    for (int q = 1; q < count; ++q)
        if (layouts[q] != lay) lay = lay == LAY_NT || layouts[q] == LAY_NT ? -1 : LAY_NN_TN;
    return lay;
}

// What a riding launch is planned from; cuts: the plan that decides the cuts, not the one that is launched
struct RidingKey {
    int layout, count, takes, cuts;
    int dims[PP_MAX_GROUP][6];
    bool operator<(const RidingKey &o) const { return memcmp(this, &o, sizeof *this) < 0; }
};
template <typename Make>
static Plan riding_plan(int layout, const GemmArgs *a, int count, bool cuts, Make make)
{
    static PlanStore<RidingKey> plans;
    RidingKey key;
    memset(&key, 0, sizeof key);
    key.layout = layout; key.count = count; key.cuts = cuts; key.takes = 1;
    for (int q = 0; q < count; ++q) {
        const int d[6] = {a[q].M, a[q].N, a[q].K, a[q].epi, a[q].c_is_f32 + 2 * may_split_k(a[q]), a[q].cu_share};
        memcpy(key.dims[q], d, sizeof d);
        key.takes = key.takes && duo_takes(a[q], DUO_128X128);
    }
    Plan plan;
    if (plans.find(key, &plan)) return plan;
    plan = make(key);
    plans.keep(key, plan);
    return plan;
}

// Chunks of K each problem of a riding launch, which has the machine to itself, may be cut in.  A sum repeats bit for bit if
// it is not split, and in two chunks it does onto zeros; it keeps that whichever way its pass runs: where the launch of its
// own that the streams would make (a[q].cu_share) has one chunk or two, it is cut in no more here.  Without that 8 % of
// shapes drawn from the layers' ranges were split that are not there, and 4 % in more than two chunks.  The fp16 unit with
// biases (384 x 768 over 1024, two chunks instead of four) 407 -> 399 us a step.
static void riding_caps(const int *layouts, const GemmArgs *a, int count, int *cap)
{
    for (int q = 0; q < count; ++q) {
        cap[q] = MAX_SPLIT;
        if (!may_split_k(a[q])) continue;
        const int alone = plan_group(layouts[q], &a[q], 1, nullptr, std::max(1, a[q].cu_share), nullptr, false).ks[0];
        if (alone <= 2) cap[q] = alone;
    }
}

// The plan of the tall and the 64 x 128 tiles, which decides where the launch cuts its sums (keeps_cuts)
static Plan riding_cuts(int layout, const int *layouts, const GemmArgs *a, int count)
{
    return riding_plan(layout, a, count, true, [&](const RidingKey &) {
        int cap[PP_MAX_GROUP];
        riding_caps(layouts, a, count, cap);
        return plan_group(layout, a, count, nullptr, 1, cap, false);
    });
}

static Plan plan_riding(int layout, const int *layouts, const GemmArgs *a, int count)
{
    return riding_plan(layout, a, count, false, [&](const RidingKey &key) {
        const Plan ref = riding_cuts(layout, layouts, a, count);
        Plan best = ref, duo;
        double tall = launch_us(a, best.bm, best.ks, best.order, count), us = 0.0;
        int cap[PP_MAX_GROUP];
        riding_caps(layouts, a, count, cap);
        const Plan square = plan_group(layout, a, count, nullptr, 1, cap);
        const double square_us = launch_us(a, square.bm, square.ks, square.order, count);
        const bool with_square = square_us < 0.95 * tall; // (a tie by the estimate came out 1-2 % slower)
        if (with_square) best = square, tall = square_us;
        if (key.takes && plan_duo(layouts, a, count, ref, &duo, &us)) {
            long tiles = 0;
            for (int q = 0; q < count; ++q) tiles += (long)tiles_m_of(a[q], duo.bm[q]) * tiles_n_of(a[q], duo.bm[q]) * duo.ks[q];
            // (short launches come out better than their estimate, 128 x 128 tiles one to a unit in them do not; long ones come out
            // later, but those of one to two tiles a unit)
            const bool pairs = tiles > compute_units() && tiles <= 2 * compute_units();
            if (us < tall * (tall < 40.0 ? (with_square ? 1.15 : 1.05) : pairs ? 1.05 : 0.90)) best = duo;
        }
        return best;
    });
}

void gemm_bf16_pp_riding_tiles(const int *layouts, const GemmArgs *a, int count, int *tiles_out, int *ksplit_out)
{
    if (count < 1 || count > PP_MAX_GROUP) return;
    const Plan pl = plan_riding(common_layout(layouts, count), layouts, a, count);
    for (int q = 0; q < count; ++q) {
        tiles_out[q] = pl.bm[q];
        if (ksplit_out) ksplit_out[q] = pl.ks[q];
    }
}

void gemm_bf16_pp_plan_riding(const int *layouts, const GemmArgs *a, int count, int *ksplit_out)
{
    if (count < 1 || count > PP_MAX_GROUP) return;
    const Plan pl = riding_cuts(common_layout(layouts, count), layouts, a, count);
    for (int q = 0; q < count; ++q) ksplit_out[q] = pl.ks[q];
}

hipError_t launch_gemm_bf16_pp_riding(const int *layouts_in, const GemmArgs *a_in, int count_in, const Riders &r, hipStream_t s)
{
    if (count_in < 0 || count_in > PP_MAX_GROUP) return hipErrorInvalidValue;
    GemmArgs a[PP_MAX_GROUP];
    int layouts[PP_MAX_GROUP], count = 0;
    for (int q = 0; q < count_in; ++q) {
        if (a_in[q].M <= 0 || a_in[q].N <= 0) continue;
        if (!gemm_bf16_args_ok(layouts_in[q], a_in[q]) || !gemm_bf16_pp_supported(layouts_in[q], a_in[q])) return hipErrorInvalidValue;
        if (count > 0 && a_in[q].elem != a[0].elem) return hipErrorInvalidValue;
        layouts[count] = layouts_in[q];
        a[count++] = a_in[q];
    }
    if (count == 0) return launch_riders(r, s);
    const int lay = common_layout(layouts, count);
    if (lay < 0) return hipErrorInvalidValue;
    const bool wide = std::all_of(r.sum, r.sum + r.sums, [](const RideSum &q) { return colsum_wide(q.Y, q.ld, q.cols); });
    const bool one_each = lay == LAY_NN_TN && !std::all_of(a, a + count, gemm_epilogue_vec_ok);
    if (!one_each && (r.sums == 0 || (wide && takes_sums(lay))))
        return launch_group(lay, layouts, a, count, plan_riding(lay, layouts, a, count), &r, s, nullptr);
    Riders moves = r, sums = r;
    moves.sums = sums.count = 0;
    if (!wide || !takes_sums(lay)) {
        const hipError_t e = launch_riders(sums, s);
        if (e != hipSuccess) return e;
        sums.sums = 0;
    }
    if (!one_each) return launch_group(lay, layouts, a, count, plan_riding(lay, layouts, a, count), &moves, s, nullptr);
    // one launch per layout, the transfers in the first and the sums in the second
    for (int one : {LAY_NN, LAY_TN}) {
        GemmArgs b[PP_MAX_GROUP];
        int lays[PP_MAX_GROUP], n = 0;
        for (int q = 0; q < count; ++q)
            if (layouts[q] == one) lays[n] = one, b[n++] = a[q];
        const hipError_t e = launch_group(one, nullptr, b, n, plan_riding(one, lays, b, n), one == LAY_NN ? &moves : &sums, s, nullptr);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_gemm_bf16_pp(int layout, const GemmArgs &a, int bm_override, hipStream_t s)
{
    return launch_gemm_bf16_pp_group(layout, &a, 1, &bm_override, s, nullptr);
}

} // namespace rtp
