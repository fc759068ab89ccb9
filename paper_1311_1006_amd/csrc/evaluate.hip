// evaluate.hip -- the FMM evaluation sequence (Sec. 2.1, Fig. 2.2) and the
// host-side work lists of a plan.
//
//   up      gather (strengths to tree order: the P2P sources, with the tree's
//           positions), P2M at the leaves, M2M (subtree.hip)
//   M2L     every box over its weak list (writes the box's local expansion)
//   P2P     leaves over their strong lists (near field, tree order)
//   down    L2L, and L2P at the leaves: far field + near field, scattered to
//           input order (subtree.hip)
// Problems of one or two levels have no M2M and no L2L: P2M and L2P at their
// leaves only (expansions.hip).
#include <algorithm>
#include <cstring>
#include <map>
#include <mutex>
#include <type_traits>

#include "fmm_internal.h"
#include "kernels_common.h"
#include "near_log.h"
#include "plan_extra.h"

namespace fmm {

template <class T>
void launch_p2m(const int32_t* leaves, int nleaf, const int32_t* bstart, const int32_t* bcount, int leaf_max,
                const double* geom, const double* X, const double* Y, const double* mt, int p, void* mp,
                hipStream_t s, const GatherOut* go);
template <class T>
void launch_l2p_field(const int32_t* leaves, int nleaf, const int32_t* bstart, const int32_t* bcount, int leaf_max,
                      const double* geom, const double* X, const double* Y, const void* loc, int p,
                      const double* near4, const int32_t* perm, double* phi, double* dphi, hipStream_t s);
template <class T>
void launch_l2p(const int32_t* leaves, int nleaf, const int32_t* bstart, const int32_t* bcount, int leaf_max,
                const double* geom, const double* X, const double* Y, const void* loc, int p,
                const double* nearf, const int32_t* perm, double* phi, double* phi_near, double* phi_far,
                hipStream_t s, const long long* guard);
template <class T>
void launch_m2l(int, const int2*, int, const int32_t*, const int32_t*, double*, bool,
                const int32_t*, const int32_t*, const int32_t*, const double*, const double*, int, const void*, void*,
                hipStream_t, int, const long long*);

template <class T>
void launch_up_leaves(const SubPlan& sp, const int32_t* bstart, const int32_t* bcount, const double* geom,
                      const double* X, const double* Y, const double* mt, int p, void* mp, const double* binom,
                      const GatherOut* go, hipStream_t s);
template <class T>
void launch_up_mid(const SubPlan& sp, const double* geom, int p, void* mp, const double* fact, hipStream_t s);
template <class T>
void launch_down_mid(const SubPlan& sp, const double* geom, int p, void* loc, const double* binom,
                     const long long* guard, hipStream_t s);
template <class T>
void launch_down_subtree(const SubPlan& sp, bool staged, const int32_t* bstart, const int32_t* bcount,
                         const double* geom, const double* X, const double* Y, void* loc, int p, const double* nearf,
                         const int32_t* perm, double* phi, double* phi_near, double* phi_far, double* dphi,
                         const long long* guard, const double* fact, hipStream_t s);

void launch_gather(int64_t n, const int32_t* perm, const double* m, double* mtree, hipStream_t s);

struct P2PItemH {
    int32_t leaf, t0, tn, pad;
};

// P2P launch shape for a leaf of nt targets: SUB lane subgroups, TG targets
// per lane (TG <= 8 in FP64, <= 16 in FP32, and 2 TG <= 64/SUB); a work item
// covers at most TG*SUB targets.  `knob` (> 0) fixes SUB, `tknob` (> 0) TG
// (with SUB then the most subgroups that TG allows unless knob fixes it).
static void p2p_shape(int nt, int knob, int tknob, bool mixed, int* tg, int* sub)
{
    if (tknob > 0) {
        *tg = tknob;
        *sub = knob > 0 ? knob : (tknob <= 4 ? 4 : 2);
        return;
    }
    int tgmax = mixed ? 16 : 8;
    int s = knob > 0 ? knob : 4;   // measured best for 15..61 targets per leaf, both precisions
    int need = (nt + s - 1) / s;
    int t = 1;
    while (t < need && t < tgmax) t <<= 1;
    int lo = s == 4 ? 1 : (s == 2 ? 2 : 4);
    int hi = s == 4 ? 4 : tgmax;
    t = t < lo ? lo : (t > hi ? hi : t);
    *tg = t;
    *sub = s;
}

// Above this many points per leaf a problem's P2M and L2P are launches of their own
// with 64 lanes per leaf, where the subtrees' kernels take 16: a lane's serial run
// over the leaf is four times as short, for two launches more.  Own / subtrees', us,
// phi and log: N = 20,000 on 4 levels (312 points per leaf) mixed p = 17 97 / 101 and
// 118 / 127, N = 30,000 on 4 (468) 129 / 138 and 169 / 184, FP64 p = 64 193 / 205 and 339 /
// 360, N = 1e5 on 5 (390) mixed p = 17 253 / 262 and 372 / 383 (but FP64 p = 64 389 / 378
// and 762 / 778), N = 1e6 on 6 (976) 4446 / 4460 and 6760 / 6790.  Below the line they
// are even or the launches cost more: N = 40,000 on 5 (156) mixed p = 17 107 / 107 and
// 145 / 147, FP64 p = 64 156 / 140, N = 1e5 on 6 (97) mixed p = 40 137 / 120.
constexpr int kFatLeaf = 256;

// the subtree launches of every pass: for a problem with levels 0 .. L-1, L >=
// 3, the roots are the boxes of level L-3; upward steps go from there to level
// 1, downward ones from level 1 to level L-4
static void prepare_subtrees(const TreeSchedule& sc, SubPlan& sp, UploadPack& up)
{
    sp.uniform = sc.L[0] >= 3;
    sp.L = sc.L[0];
    std::vector<int32_t> shallow, fat;
    std::vector<char> is_fat(sc.nprob, 0);
    int nfat = 0;
    for (int b = 0; b < sc.nprob; ++b) {
        sp.uniform = sp.uniform && sc.L[b] == sc.L[0];
        const int64_t base = sc.pbox[b] + level_base(sc.L[b] - 1), n = int64_t(1) << (2 * (sc.L[b] - 1));
        is_fat[b] = sc.L[b] >= 3 && sc.off[b + 1] - sc.off[b] > kFatLeaf * n;
        nfat += is_fat[b];
        if (sc.L[b] >= 3 && !is_fat[b]) continue;
        LeafSet& set = is_fat[b] ? sp.fat : sp.shallow;
        for (int64_t j = 0; j < n; ++j) {
            (is_fat[b] ? fat : shallow).push_back((int32_t)(base + j));
            set.max = std::max(set.max, (int)sc.box_count[base + j]);
        }
    }
    sp.shallow.n = (int)shallow.size();
    sp.fat.n = (int)fat.size();
    sp.all_fat = nfat == sc.nprob;
    sp.listed = !sp.uniform || (nfat > 0 && !sp.all_fat);
    std::vector<int4> list;
    // one launch: for every problem the boxes of level lev(L), D(L) levels (D = 0: none)
    auto step = [&](auto lev, auto D, bool roots = false) {
        SubStep st{(int64_t)list.size(), 0, lev(sp.L), D(sp.L) + (roots && sp.all_fat ? kSubFat : 0)};
        for (int b = 0; b < sc.nprob; ++b) {
            const int l = lev(sc.L[b]), d = D(sc.L[b]);
            if (d == 0) continue;
            const int64_t n = int64_t(1) << (2 * l);
            st.n += n;
            if (sp.listed)
                for (int64_t j = 0; j < n; ++j)
                    list.push_back(make_int4((int)sc.pbox[b], l, (int)j, d + (roots && is_fat[b] ? kSubFat : 0)));
        }
        return st;
    };
    sp.roots = step([](int L) { return L - 3; }, [](int L) { return L >= 3 ? 3 : 0; }, true);
    for (int h = 0; h < 2; ++h) {
        const int m = h ? kSubLevelsHigh : kSubLevels;
        for (int k = 0; m * k < sc.max_levels - 4; ++k) {
            auto D = [m, k](int L) { return std::max(0, std::min(m, L - 4 - m * k)); };
            sp.up[h].push_back(step([=](int L) { return std::max(0, L - 3 - m * k - D(L)); }, D));
        }
        for (int k = 0; 1 + m * k < sc.max_levels - 4; ++k)
            sp.down[h].push_back(step([m, k](int) { return 1 + m * k; },
                                      [m, k](int L) { return std::max(0, std::min(m, L - 4 - (1 + m * k))); }));
    }
    up.add(sp.shallow.ids, shallow);
    up.add(sp.fat.ids, fat);
    up.add(sp.list, list);
}

// The tables that depend on nothing but the mathematics: binomials,
// factorials and the logarithm's.  One block per device, made by the first plan
// there and kept (70 KB); with tables of its own the first plan of every layout took
// about 20 us longer (N = 60,000, N_levels 6: 165 us against 145).
static const double* constant_tables(int device, hipStream_t s)
{
    static std::mutex mu;
    static std::map<int, double*> blocks;
    std::lock_guard<std::mutex> lk(mu);
    auto it = blocks.find(device);
    if (it != blocks.end()) return it->second;
    std::vector<double> h(kBinomRows * kBinomStride + 2 * kMaxP + 2 * kLogTab, 0.0);
    // C(n, k), n < kBinomRows, k < kBinomStride (Pascal's rule)
    double* bin = h.data();
    for (int n = 0; n < kBinomRows; ++n) {
        bin[n * kBinomStride] = 1.0;
        for (int k = 1; k <= n && k < kBinomStride; ++k)
            bin[n * kBinomStride + k] = bin[(n - 1) * kBinomStride + k - 1] + (k < n ? bin[(n - 1) * kBinomStride + k] : 0.0);
    }
    // factorials and their reciprocals, each rounded once from extended precision
    double* fact = bin + kBinomRows * kBinomStride;
    long double f = 1.0L;
    for (int k = 0; k < kMaxP; ++k) {
        if (k > 0) f *= k;
        fact[k] = (double)f;
        fact[kMaxP + k] = (double)(1.0L / f);
    }
    log_table(reinterpret_cast<double2*>(fact + 2 * kMaxP));
    DBuf<double> block;
    block.alloc(h.size(), s);
    FMM_HIP(hipMemcpyAsync(block.p, h.data(), h.size() * sizeof(double), hipMemcpyHostToDevice, s));
    FMM_HIP(hipStreamSynchronize(s));
    const double* p = blocks[device] = block.p;
    block.p = nullptr;          // kept
    return p;
}

void prepare_plan_host(Plan& pl, PlanExtra& ex, hipStream_t s)
{
    TreeSchedule& sc = *pl.tree->sched;
    UploadPack up;
    int ml = sc.max_levels;
    ex.level_boxes.assign(ml, {});
    std::vector<int32_t> leaves, child0(sc.nbox, -1);
    for (int b = 0; b < sc.nprob; ++b) {
        for (int l = 0; l < sc.L[b]; ++l) {
            int64_t base = sc.pbox[b] + level_base(l);
            for (int64_t j = 0; j < (int64_t(1) << (2 * l)); ++j) {
                int32_t id = (int32_t)(base + j);
                ex.level_boxes[l].push_back(id);
                if (l + 1 < sc.L[b]) {
                    child0[id] = (int32_t)(sc.pbox[b] + level_base(l + 1) + 4 * j);
                } else {
                    leaves.push_back(id);
                    ex.leaf_max = std::max(ex.leaf_max, (int)sc.box_count[id]);
                }
            }
        }
    }
    std::vector<int32_t> all;
    ex.level_boxes_off.assign(ml + 1, 0);
    for (int l = 0; l < ml; ++l) {
        ex.level_boxes_off[l] = (int64_t)all.size();
        all.insert(all.end(), ex.level_boxes[l].begin(), ex.level_boxes[l].end());
    }
    ex.level_boxes_off[ml] = (int64_t)all.size();
    up.add(ex.d_level_boxes, all);
    up.add(ex.leaves, leaves);
    up.add(ex.child0, child0);
    // P2P work items grouped by launch shape
    const bool mixed = pl.precision == FMM_MIXED;
    std::map<std::pair<int, int>, std::vector<P2PItemH>> cls;
    for (int32_t g : leaves) {
        int nt = sc.box_count[g];
        int tg, sub;
        p2p_shape(nt, pl.tune.p2p_split, pl.tune.p2p_targets, mixed, &tg, &sub);
        int chunk = tg * sub;
        for (int t0 = 0; t0 < nt; t0 += chunk)
            cls[{tg, sub}].push_back(P2PItemH{g, t0, std::min(chunk, nt - t0), 0});
    }
    std::vector<P2PItemH> items;
    ex.p2p_class.clear();
    for (auto& kv : cls) {
        ex.p2p_class.push_back({kv.first.first, kv.first.second, (int64_t)items.size(), (int64_t)kv.second.size()});
        items.insert(items.end(), kv.second.begin(), kv.second.end());
    }
    up.add(ex.p2p_items, reinterpret_cast<const char*>(items.data()), items.size() * sizeof(P2PItemH));
    prepare_adjoint_items(pl, ex, leaves, up);
    prepare_subtrees(sc, ex.sub, up);
    const double* tab = constant_tables(pl.tree->device, s);
    auto view = [&](DView<double>& d, size_t n) {
        d.p = const_cast<double*>(tab);
        d.n = n;
        tab += n;
    };
    view(ex.binom, kBinomRows * kBinomStride);
    view(ex.fact, 2 * kMaxP);
    view(ex.logtab, 2 * kLogTab);
    up.upload(ex.block, s);
}

void alloc_eval_buffers(Plan& pl, hipStream_t s)
{
    TreeSchedule& sc = *pl.tree->sched;
    int64_t n = sc.n;
    bool mixed = pl.precision == FMM_MIXED;
    size_t cs = mixed ? sizeof(float) : sizeof(double);
    pl.mtree.alloc(2 * n, s);
    pl.near.alloc(2 * n, s);
    pl.mpole.alloc(2 * cs * sc.nbox * coef_ld(pl.p, 2 * cs), s);
    pl.local.alloc(2 * cs * sc.nbox * coef_ld(pl.p, 2 * cs), s);
}

// Whether the subtrees' downward pass is staged (every box's complete
// expansion formed from its parent's and stored, rounded to the storage type):
// when it is asked for (`all`: the expansions of every level are read
// afterwards; FMM_FLAG_LEVELWISE), for problems of unlike depth (a problem's
// result is then the one it has alone with that flag, to the bit), and for
// more than 32 terms in mixed precision.  Otherwise the direct form, one
// launch.
static bool staged_down(const Plan& pl, const PlanExtra& ex, bool all)
{
    return all || !ex.sub.uniform || (pl.tune.flags & FMM_FLAG_LEVELWISE) ||
           (pl.precision == FMM_MIXED && pl.p > 32);
}

// The upward pass of the strengths m (input order), with their gather into tree
// order, into the multipoles mp; or, without m, of the strengths mt (tree
// order).  `after_gather` (optional) is recorded once the strengths are in
// tree order: work that needs only them (the near field) may start.  `keep`
// false: the strengths in tree order are written by a gather of their own.
template <class T>
static void run_up(Plan& pl, const double* m, const double* mt, void* mp, hipStream_t s,
                   hipEvent_t after_gather = nullptr, bool keep = true)
{
    Tree& t = *pl.tree;
    TreeSchedule& sc = *t.sched;
    PlanExtra& ex = *extra(pl);
    const GatherOut go{t.perm.p, (const double2*)m, keep ? (double2*)pl.mtree.p : nullptr};
    for (const LeafSet* set : {&ex.sub.fat, &ex.sub.shallow})
        launch_p2m<T>(set->ids.p, set->n, sc.d_box_start.p, sc.d_box_count.p, set->max, t.geom.p, t.x.p, t.y.p, mt,
                      pl.p, mp, s, m ? &go : nullptr);
    const bool gathered = ex.sub.all_fat;           // by P2M alone
    if (after_gather && gathered) FMM_HIP(hipEventRecord(after_gather, s));
    launch_up_leaves<T>(ex.sub, sc.d_box_start.p, sc.d_box_count.p, t.geom.p, t.x.p, t.y.p, mt, pl.p, mp, ex.fact.p,
                        m ? &go : nullptr, s);
    if (after_gather && !gathered) FMM_HIP(hipEventRecord(after_gather, s));
    launch_up_mid<T>(ex.sub, t.geom.p, pl.p, mp, ex.fact.p, s);
}

// The leaves of the downward pass: their complete expansions in loc, evaluated
// at the points when an output is given
template <class T>
static void run_down_leaves(Plan& pl, bool staged, void* loc, double* phi, double* phi_near, double* phi_far,
                            const long long* guard, hipStream_t s, double* dphi = nullptr)
{
    Tree& t = *pl.tree;
    TreeSchedule& sc = *t.sched;
    PlanExtra& ex = *extra(pl);
    launch_down_subtree<T>(ex.sub, staged, sc.d_box_start.p, sc.d_box_count.p, t.geom.p, t.x.p, t.y.p, loc, pl.p,
                           dphi ? pl.near4.p : pl.near.p, t.perm.p, phi, phi_near, phi_far, dphi, guard, ex.fact.p, s);
    for (const LeafSet* set : {&ex.sub.fat, &ex.sub.shallow}) {
        if (dphi)
            launch_l2p_field<T>(set->ids.p, set->n, sc.d_box_start.p, sc.d_box_count.p, set->max, t.geom.p, t.x.p,
                                t.y.p, loc, pl.p, pl.near4.p, t.perm.p, phi, dphi, s);
        else if (phi || phi_near || phi_far)
            launch_l2p<T>(set->ids.p, set->n, sc.d_box_start.p, sc.d_box_count.p, set->max, t.geom.p, t.x.p, t.y.p,
                          loc, pl.p, pl.near.p, t.perm.p, phi, phi_near, phi_far, s, guard);
    }
}

struct PhaseTimer {
    static constexpr int kEvents = 6;
    bool on;
    hipStream_t s;
    hipEvent_t ev[kEvents];
    int k = 0;
    PhaseTimer(bool o, hipStream_t st) : on(o), s(st)
    {
        if (on)
            for (auto& e : ev) FMM_HIP(hipEventCreate(&e));
    }
    void mark()
    {
        if (on) FMM_HIP(hipEventRecord(ev[k++], s));
    }
    float between(int a, int b)
    {
        float ms = 0;
        FMM_HIP(hipEventElapsedTime(&ms, ev[a], ev[b]));
        return ms * 1000.0f;
    }
    ~PhaseTimer()
    {
        if (on)
            for (auto& e : ev) (void)hipEventDestroy(e);
    }
};

// M2L into loc, and the staged downward pass's levels above the subtrees'
// roots (the direct form takes every ancestor in its only launch); with `all`
// the roots' subtrees too, so that the expansions of every level are complete.
template <class T>
static void run_far_down(Plan& pl, PlanExtra& ex, const void* mp, void* loc, hipStream_t s, PhaseTimer& tm,
                         const long long* guard, bool all = false)
{
    Tree& t = *pl.tree;
    TreeSchedule& sc = *t.sched;
    const Plan::Balance& b = pl.bal_m2l;
    launch_m2l<T>((int)sc.nbox, b.xitems.p, (int)b.total, b.icnt.p, b.ioff.p, b.partial.p,
                  b.total > sc.nbox, pl.w_beg.p, pl.w_cnt.p, pl.w_ids.p, t.geom.p, ex.binom.p, pl.p, mp, loc, s,
                  pl.tune.m2l_batch, guard);
    tm.mark();
    if (staged_down(pl, ex, all)) launch_down_mid<T>(ex.sub, t.geom.p, pl.p, loc, ex.fact.p, guard, s);
    if (all) run_down_leaves<T>(pl, true, loc, nullptr, nullptr, nullptr, guard, s);
}

void combine_chunks(const Plan::Balance& b, const double* partial, int vals, const void* items, int n,
                    const int32_t* bstart, double* out, hipStream_t s);

bool field_one_pass(const Plan& pl)
{
    for (auto& c : pl.ex->p2p_class)
        if (c.sub != 4) return false;
    return true;
}

// the near field: into pl.near, or with `field` (and the derivative's sums) pl.near4
static void run_p2p(Plan& pl, PlanExtra& ex, hipStream_t s, const long long* guard, bool log_kernel = false,
                    bool field = false)
{
    Tree& t = *pl.tree;
    TreeSchedule& sc = *t.sched;
    bool mixed = pl.precision == FMM_MIXED;
    const Plan::Balance& b = pl.bal;
    int nitems = 0;
    double* out = field ? pl.near4.p : pl.near.p;
    double* partial = field ? b.partial4.p : b.partial.p;
    for (size_t c = 0; c < ex.p2p_class.size(); ++c) {
        const P2PClass& k = ex.p2p_class[c];
        nitems = std::max<int>(nitems, (int)(k.off + k.n));
        const int64_t x0 = b.cls[c], x1 = b.cls[c + 1];
        launch_p2p(mixed, k.tg, k.sub, ex.p2p_items.p, (int)x0, b.xitems.p ? b.xitems.p + x0 : nullptr,
                   (int)(x1 - x0), b.icnt.p, b.ioff.p,
                   partial, sc.d_box_start.p, sc.d_box_count.p, pl.s_beg.p, pl.s_cnt.p, pl.s_ids.p,
                   t.x.p, t.y.p, (const double2*)pl.mtree.p, out, s, guard,
                   pl.tune.smooth_delta > 0.0 ? 1.0 / (pl.tune.smooth_delta * pl.tune.smooth_delta) : 0.0,
                   log_kernel ? ex.logtab.p : nullptr, Targets{}, pl.tune.p2p_src_tile, field);
    }
    combine_chunks(b, partial, field ? 4 : 2, ex.p2p_items.p, nitems, sc.d_box_start.p, out, s);
}

// Side streams per device (the near field; the list build), shared by all
// plans and kept until the process ends (creating a stream per plan costs
// more than a whole step).  Plans that share one are ordered by their own
// events.
hipStream_t side_stream(int device, int which)
{
    static std::mutex mu;
    static std::map<std::pair<int, int>, hipStream_t> streams;
    std::lock_guard<std::mutex> lk(mu);
    auto it = streams.find({device, which});
    if (it != streams.end()) return it->second;
    hipStream_t st = nullptr;
    FMM_HIP(hipStreamCreateWithFlags(&st, hipStreamNonBlocking));
    streams[{device, which}] = st;
    return st;
}

// Whether the near field runs on a second stream beside the far field instead
// of after M2L on the evaluation's own.  Where both fill the chip they are
// bound by VALU issue and take beside each other the time they take in turn,
// while the fork and the join cost the critical path about 10 us each: one
// stream for N = 1000 29 us against 49, N = 16,000 36 against 57, N = 1e6 mixed
// 249 against 252.  Two streams pay where one of them leaves part of the chip
// idle: lists split into work chunks (a tail of long items: batch of 128 problems
// 1252 us against 1325, clustered step 1512-1551 against 1533), and more than 32
// terms (few wavefronts of many registers: N = 1e5, p = 39 140 us against 150);
// not where the problem is so small that the streams' overhead is most of the time
// (one stream / two, FP64: split lists N = 3000 on 3 levels 64 / 74-82, N = 30,000
// on 5 levels 82 / 87; p = 39 N = 300 31 / 61, N = 1000 49-52 / 56-62, N = 3000
// on 3 levels 89 / 82).
static bool near_beside(const Plan& pl)
{
    const int64_t n = pl.tree->sched->n;
    return pl.p > 32 ? n > 2048 : n > 16384 && (pl.split_p2p || pl.split_m2l);
}

// Whether the second stream gathers the strengths itself, so that the near field
// does not wait for P2M (which does the gather otherwise).  P2M takes the longer
// the more points a leaf has and the more terms, while the extra gather reads every
// strength twice: P2M's / its own, us: p = 39 FP64 N = 3000 on 3 levels (187
// points per leaf) 98 / 82, N = 10,000 on 4 (156) 105 / 92,
// N = 10,000 on 5 (39) 72 / 68 (mixed 64 / 67), N = 150,000 on 7 (36) mixed 138 / 150, N =
// 1e5 on 7 (24) 139 / 144; p = 16 split lists N = 1e5 on 5 (390) 374 / 349, 1e6
// clustered on 9 (15) mixed 667 / 687, batch of 128 problems (16) 1281 / 1334.
constexpr int kGatherApart = 64;     // points per leaf

// The second stream and its events, where they are used, made when the plan is
// made (more than 32 terms) or its lists are final (split lists): the
// evaluations then create nothing, in a capture least of all.  Evaluations at
// many points make them in their first call.
void second_stream(Plan& pl)
{
    if (!pl.nstream) {
        pl.nstream = side_stream(pl.tree->device, kNearStream);
        FMM_HIP(hipEventCreateWithFlags(&pl.ev_fork, hipEventDisableTiming));
        FMM_HIP(hipEventCreateWithFlags(&pl.ev_join, hipEventDisableTiming));
    }
}
void plan_events(Plan& pl)
{
    if (near_beside(pl)) second_stream(pl);
}

// The part of an evaluation that needs no lists: gather and the upward
// pass.  evaluate_device then continues from there on the same stream (the
// near field is forked there, after the plan's remaining kernels).
void evaluate_upward(Plan& pl, const double* m, hipStream_t s)
{
    Tree& t = *pl.tree;
    TreeSchedule& sc = *t.sched;
    PlanExtra& ex = *extra(pl);
    const bool mixed = pl.precision == FMM_MIXED;
    if (mixed) run_up<float>(pl, m, nullptr, pl.mpole.p, s);
    else run_up<double>(pl, m, nullptr, pl.mpole.p, s);
    pl.upward_done = true;
}

// The far field of every box and nothing at the sources: the upward pass (with
// the gather of the strengths; needs no lists), then the M2L / L2L sweep over
// every level, so that the multipole expansion and the complete local expansion
// of every box are in the plan's buffers (evaluation at points apart from the
// sources).
void far_field_up(Plan& pl, const double* m, hipStream_t s)
{
    pl.upward_done = false;
    // the plan's buffers will hold the far field of m, not a forward evaluation
    pl.have_forward = false;
    if (pl.precision == FMM_MIXED) run_up<float>(pl, m, nullptr, pl.mpole.p, s);
    else run_up<double>(pl, m, nullptr, pl.mpole.p, s);
}
void far_field_down(Plan& pl, hipStream_t s)
{
    PhaseTimer tm(false, s);
    PlanExtra& ex = *extra(pl);
    if (pl.precision == FMM_MIXED) run_far_down<float>(pl, ex, pl.mpole.p, pl.local.p, s, tm, nullptr, true);
    else run_far_down<double>(pl, ex, pl.mpole.p, pl.local.p, s, tm, nullptr, true);
}

void transposed_far(Plan& pl, const double* w, hipStream_t s)
{
    Tree& t = *pl.tree;
    TreeSchedule& sc = *t.sched;
    PlanExtra& ex = *extra(pl);
    PhaseTimer tm(false, s);
    auto far = [&](auto tag) {
        using T = decltype(tag);
        run_up<T>(pl, nullptr, w, pl.amp.p, s);
        // mixed: every level rounded to the storage type
        const bool all = std::is_same<T, float>::value;
        run_far_down<T>(pl, ex, pl.amp.p, pl.aloc.p, s, tm, nullptr, all);
        if (!all) run_down_leaves<T>(pl, staged_down(pl, ex, false), pl.aloc.p, nullptr, nullptr, nullptr, nullptr, s);
    };
    if (pl.precision == FMM_MIXED) far(float());
    else far(double());
}

void launch_real_to_complex(int64_t n, const double* q, double* m, hipStream_t s);
template <class T>
void launch_log_constants(int nbox, const int32_t* w_beg, const int32_t* w_cnt, const int32_t* w_ids,
                          const int32_t* parent, const double* geom, const void* mp, const void* loc, int p,
                          double* c0, hipStream_t s);
template <class T>
void launch_l2p_log(const int32_t* leaves, int nleaf, int64_t n, const int32_t* bstart, const int32_t* bcount,
                    const int32_t* parent, const double* geom, const double* X, const double* Y, const void* loc,
                    int p, const double* c0, const double* near, const int32_t* perm, double* u, hipStream_t s);

// The logarithmic potential (see log.hip): the harmonic upward pass and far
// field of the strengths q as complex numbers, the constant terms of the local
// expansions, the near field with the logarithmic kernel, and L2P of the
// integrated series.
void evaluate_log_device(Plan& pl, const double* q, double* u, hipStream_t s, double* mlog, double* c0)
{
    Tree& t = *pl.tree;
    TreeSchedule& sc = *t.sched;
    PlanExtra& ex = *extra(pl);
    const bool mixed = pl.precision == FMM_MIXED;
    if (!mlog) {
        pl.mlog.alloc(2 * sc.n, s);
        pl.c0.alloc(sc.nbox, s);
        mlog = pl.mlog.p;
        c0 = pl.c0.p;
    }
    launch_real_to_complex(sc.n, q, mlog, s);
    PhaseTimer tm(false, s);
    if (mixed) run_up<float>(pl, mlog, nullptr, pl.mpole.p, s);
    else run_up<double>(pl, mlog, nullptr, pl.mpole.p, s);
    if (mixed) run_far_down<float>(pl, ex, pl.mpole.p, pl.local.p, s, tm, nullptr, true);
    else run_far_down<double>(pl, ex, pl.mpole.p, pl.local.p, s, tm, nullptr, true);
    auto constants = mixed ? launch_log_constants<float> : launch_log_constants<double>;
    constants((int)sc.nbox, pl.w_beg.p, pl.w_cnt.p, pl.w_ids.p, sc.d_box_parent.p, t.geom.p, pl.mpole.p, pl.local.p,
              pl.p, c0, s);
    run_p2p(pl, ex, s, nullptr, true);
    auto l2p = mixed ? launch_l2p_log<float> : launch_l2p_log<double>;
    l2p(ex.leaves.p, (int)sc.nleaf, sc.n, sc.d_box_start.p, sc.d_box_count.p, sc.d_box_parent.p, t.geom.p, t.x.p, t.y.p,
        pl.local.p, pl.p, c0, pl.near.p, t.perm.p, u, s);
    // the harmonic state of the plan now holds these strengths: no adjoint of it
    pl.have_forward = false;
}

static void evaluate_any(Plan& pl, const double* m, double* phi, double* phi_near, double* phi_far, hipStream_t s,
                         hipEvent_t lists_ev, const long long* guard, double* dphi)
{
    PlanExtra& ex = *extra(pl);
    bool mixed = pl.precision == FMM_MIXED;
    PhaseTimer tm((pl.tune.flags & FMM_FLAG_PHASE_TIMING) != 0, s);
    // Phase timing keeps the phases one after another on `s`.
    if (lists_ev && tm.on) throw Error(FMM_EINVAL, "an evaluation ahead of its lists has no phase timing");
    const bool beside = !tm.on && near_beside(pl);
    tm.mark();
    const bool up = pl.upward_done && !tm.on;   // gather and upward pass enqueued by evaluate_upward
    pl.upward_done = false;
    // on its own stream the near field forks as soon as the strengths are in
    // tree order, beside the upper levels' M2M, or gathers them itself
    const bool early_fork = beside && !up;
    const TreeSchedule& sc = *pl.tree->sched;
    const bool apart = early_fork && sc.n > kGatherApart * sc.nleaf;
    if (apart) FMM_HIP(hipEventRecord(pl.ev_fork, s));
    if (!up) {
        hipEvent_t ev = early_fork && !apart ? pl.ev_fork : nullptr;
        if (mixed) run_up<float>(pl, m, nullptr, pl.mpole.p, s, ev, !apart);
        else run_up<double>(pl, m, nullptr, pl.mpole.p, s, ev, !apart);
    }
    if (beside) {
        // it starts after everything enqueued on `s` so far: the gather (with
        // P2M), and the list and work-chunk kernels of the plan (which follow
        // the upward pass when evaluate_upward ran first); or after the gather
        // (the event recorded there), or before it
        if (!early_fork) FMM_HIP(hipEventRecord(pl.ev_fork, s));
        FMM_HIP(hipStreamWaitEvent(pl.nstream, pl.ev_fork, 0));
        if (apart) launch_gather(sc.n, pl.tree->perm.p, m, pl.mtree.p, pl.nstream);
        if (lists_ev) FMM_HIP(hipStreamWaitEvent(pl.nstream, lists_ev, 0));
        run_p2p(pl, ex, pl.nstream, guard, false, dphi != nullptr);
        FMM_HIP(hipEventRecord(pl.ev_join, pl.nstream));
    }
    tm.mark();
    if (lists_ev) FMM_HIP(hipStreamWaitEvent(s, lists_ev, 0));
    if (mixed) run_far_down<float>(pl, ex, pl.mpole.p, pl.local.p, s, tm, guard);
    else run_far_down<double>(pl, ex, pl.mpole.p, pl.local.p, s, tm, guard);
    tm.mark();
    if (beside) FMM_HIP(hipStreamWaitEvent(s, pl.ev_join, 0));
    else run_p2p(pl, ex, s, guard, false, dphi != nullptr);
    tm.mark();
    (mixed ? run_down_leaves<float> : run_down_leaves<double>)(pl, staged_down(pl, ex, false), pl.local.p, phi,
                                                               phi_near, phi_far, guard, s, dphi);
    tm.mark();
    if (tm.on) {
        FMM_HIP(hipEventSynchronize(tm.ev[5]));
        pl.t_up = tm.between(0, 1);
        pl.t_m2l = tm.between(1, 2);
        pl.t_l2l = tm.between(2, 3);
        pl.t_p2p = tm.between(3, 4);
        pl.t_down = tm.between(4, 5);
        pl.t_total = tm.between(0, 5);
    }
    pl.have_forward = true;
}

void evaluate_device(Plan& pl, const double* m, double* phi, double* phi_near, double* phi_far, hipStream_t s,
                     hipEvent_t lists_ev, const long long* guard)
{
    evaluate_any(pl, m, phi, phi_near, phi_far, s, lists_ev, guard, nullptr);
}
void evaluate_derivative_device(Plan& pl, const double* m, double* phi, double* dphi, hipStream_t s)
{
    evaluate_any(pl, m, phi, nullptr, nullptr, s, nullptr, nullptr, dphi);
}

}  // namespace fmm
