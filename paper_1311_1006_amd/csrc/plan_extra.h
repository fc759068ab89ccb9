// plan_extra.h -- per-plan launch lists (host + device), internal.
#pragma once
#include <map>

#include "fmm_internal.h"

namespace fmm {

struct P2PClass {
    int tg, sub;        // targets per lane, lane subgroups
    int64_t off, n;     // range in the item array
};

// Subtree launches of the far field's upward and downward passes (subtree.hip).
struct SubStep {
    int64_t off, n;     // the launch's workgroups: entries off .. off + n - 1 of the list (or n computed ones)
    int lev, D;         // trees of one depth: the level of the subtrees' roots, and their levels
};
constexpr int kSubLevels = 3, kSubLevelsHigh = 2;   // levels per launch above the roots, p <= 32 and more
// Leaves whose P2M and L2P are launches of their own (expansions.hip, up to 64 lanes
// per leaf) instead of parts of the subtrees' (16 lanes per leaf)
struct LeafSet {
    DView<int32_t> ids;
    int n = 0, max = 0;         // their number, and the largest one's points
};
constexpr int kSubFat = 256;    // added to D in the list: the leaves are in `fat`
struct SubPlan {
    bool uniform = false;       // every problem has the same depth L >= 3
    bool listed = false;        // the launches read the list (problems of unlike depth, or fat and thin ones)
    bool all_fat = false;       // not listed: every problem's leaves are in `fat`
    int L = 0;
    DView<int4> list;            // (root box of the problem, level, box of the level, levels D) per workgroup
    SubStep roots{};            // the boxes of level L-3 (problems of fewer levels: see shallow)
    // [0] for p <= 32, [1] for more terms (fewer levels per launch):
    std::vector<SubStep> up[2];    // levels L-4 .. 1, bottom up
    std::vector<SubStep> down[2];  // levels 2 .. L-4 from level 1, top down
    LeafSet shallow;            // the leaves of the problems of one or two levels (no shifts between levels)
    LeafSet fat;                // those of deeper problems with many points per leaf (kFatLeaf)
};
// the same as a kernel argument
struct SubWork {
    const int4* list;
    int lev, D, nper;           // without a list: every problem has NB boxes and nper subtrees of D levels
    int64_t NB;                 // rooted at level lev (D as in the list)
};

struct PlanExtra {
    std::vector<std::vector<int32_t>> level_boxes;  // global ids per level (all problems)
    std::vector<int64_t> level_boxes_off;
    DView<int32_t> d_level_boxes;                    // concatenated per level
    DView<int32_t> leaves;                           // global ids of all leaves
    int leaf_max = 0;                               // largest leaf population
    SubPlan sub;
    int cap_strong = 0, cap_weak = 0;               // per-box list capacities of the one-pass build
    bool levelwise_only = false;                    // a frontier overflowed on this layout
    int64_t pool_strong = 0, pool_weak = 0;        // id pool sizes for the next compact build
    bool compact_only = false;                      // fixed capacities would need too much memory
    DView<double> fact;                              // k! for k < 64, then 1/k! (these three: one block per device)
    DView<double> logtab;                            // table of the near field's FP64 logarithm
    DView<double> binom;                             // binomial table C(n, k), n, k < 64
    DView<int32_t> child0;                           // first child of every box, -1: a leaf
    DView<char> p2p_items;
    std::vector<P2PClass> p2p_class;
    DView<char> adj_items;                           // adjoint P2P work items
    std::vector<P2PClass> adj_class;
    DBuf<char> block;                               // the memory of the arrays above
};

inline PlanExtra* extra(Plan& pl) { return pl.ex; }

void prepare_plan_host(Plan& pl, PlanExtra& ex, hipStream_t s);
void alloc_eval_buffers(Plan& pl, hipStream_t s);
void prepare_adjoint_items(Plan& pl, PlanExtra& ex, const std::vector<int32_t>& leaves, UploadPack& up);

}  // namespace fmm
