// points.hip -- the field of the sources at evaluation points apart from them
// (eq. 2.2), from a plan over the sources' tree (Sec. 2.1, 2.2).
//
// A point y goes down the tree from the root, at every level into the child
// whose disc (centre c, radius r: the disc around the tight bounding box that
// the theta-criterion (2.3) is stated for) holds it with the smallest
// |y - c| / r, as deep as it can: box B.  The complete local expansion of B
// (after the M2L and L2L sweep over every level) holds the field of every
// source outside the boxes of B's strong list -- at every level the strong
// and weak lists of a box and of its ancestors partition the sources -- and
// it converges at y with the bound of the sources' own evaluation, because y
// lies in the disc of B and of each of its ancestors, the discs whose radii
// entered the theta-criterion of those M2L shifts.  The discs overlap and
// cover the gaps between the tight boxes, so nearly every point among the
// sources reaches a leaf.
//
// When B is a leaf, the sources of its strong list (leaves) are summed
// directly, as for the sources of B, so the point's value has the accuracy
// of theirs.  Otherwise (a point outside the discs of B's children) every box
// of B's strong list is descended: a box well separated from the point
// contributes its multipole expansion at y, a leaf that is not contributes
// its points directly, any other box is opened.
// "Well separated" is the criterion (2.3) between the box and a box of the
// same radius r around the point, r (1 + theta) <= theta d (squared, every
// operation rounded alone as in the list build), so that these expansions
// are used at the distances the M2L shifts of the plan use them.  The root
// is always opened (no list needs its multipole expansion, so the upward
// pass stops at level 1): a point outside every disc of level 1 gets its
// whole field from the descent of the root.  A source at y's position is
// left out, as (2.2) says.  The points join neither the tree nor the lists,
// so they change nothing of the sources' own evaluation.
//
// Expansions are the scaled ones of expansions.hip (a_k = sum m_j w_j^k,
// w_j = (z_j - c)/rs; phi(z) = sum b_l ((z - c)/rs)^l), so with u = rs/(y - c)
//     multipole at y:  (u/rs) sum_k a_k u^k,
//     its derivative:  -(u/rs)^2 sum_k (k+1) a_k u^k.
// Coefficients are read in their storage type and used in FP64; the direct
// sums of the mixed path are FP32 with the double-float difference of the
// near-field kernel.
//
// The points are sorted by B (a counting sort: count, scan, scatter).  The
// near field of the points in leaves is the near-field kernel of the sources
// (p2p.hip) with the points as its targets: sources of the leaf's strong list
// staged in LDS, a lane subgroup per few points; with the derivative a kernel
// of its own (k_pts_near_der; where the points are few, or few per leaf, and in
// leaves with long lists they descend instead).  The descents of the other
// points run a wavefront per point, lanes over the boxes of a frontier.  The far
// field is one lane per point.  Locating, sorting and the descents wait for memory most
// of the time, so they run on a second stream beside the sources' far field.
#include <algorithm>
#include <cfloat>
#include <type_traits>

#include "fmm_internal.h"
#include "kernels_common.h"

namespace fmm {

void far_field_up(Plan& pl, const double* m, hipStream_t s);
void far_field_down(Plan& pl, hipStream_t s);

// near-field work items over the points: at most kPtsItem points of one box
// each, for the (4 targets per lane, 4 subgroups) shape
constexpr int kPtsItem = 16;
constexpr int64_t kTwoStreamPoints = 50000, kDescendPoints = 8192;   // see evaluate_points_device
// of split layouts: strong lists longer than this are descended, for many points
// and for few (at most kFewPoints and kFewPerLeaf per leaf; likewise)
constexpr int kLongList = 512, kLongListFew = 64;
constexpr int64_t kFewPoints = 131072, kFewPerLeaf = 32;
// the lists of uniform sources hold less than kUniformList / theta^2 boxes
constexpr double kUniformList = 3.0;
static int long_list(int64_t M, int64_t nleaf, double theta)
{
    if (M > std::min(kFewPoints, kFewPerLeaf * nleaf)) return kLongList;
    return (int)std::min<double>(kLongList, std::max<double>(kLongListFew, kUniformList / (theta * theta)));
}
struct PtsItem {
    int32_t leaf, t0, tn, pad;
};

__global__ void k_pts_clear(int32_t* a, int64_t n)
{
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i < n) a[i] = 0;
}

// the deepest box whose disc (centre c, radius r: the disc of the
// theta-criterion, around the tight bounding box) holds each point, going
// down from the root into the child that holds it with the smallest
// |y - c| / r, the points per box and each point's rank among its box's
// points (the order the counter gave them).  The geometry of levels 1 ..
// kLocTop is read from a copy in LDS (the first kLocTop of a point's
// dependent loads), deeper levels from the tree.
constexpr int kLocTop = 4;
constexpr int kLocTopBoxes = 340;   // boxes of levels 1 .. kLocTop
__device__ __forceinline__ void locate_child(const double2 q, const double* g, int k, int& best, double& bq)
{
    const double dx = q.x - g[0], dy = q.y - g[1];
    const double d2 = dx * dx + dy * dy, r2 = g[2] * g[2];
    if (!(d2 <= r2)) return;                                // outside (a zero-radius disc holds its centre)
    const double qk = r2 > 0.0 ? d2 / r2 : 0.0;
    if (qk < bq) {
        bq = qk;
        best = k;
    }
}
__global__ void __launch_bounds__(256)
k_pts_locate(const double2* __restrict__ y, int64_t M, int L, const double* __restrict__ geom, int32_t* box,
             int32_t* cnt, int32_t* rank)
{
    static_assert(kLocTopBoxes == ((4 << (2 * kLocTop)) - 1) / 3 - 1, "levels 1 .. kLocTop");
    __shared__ double sg[kLocTopBoxes][3];
    const int top = L - 1 < kLocTop ? L - 1 : kLocTop;     // levels cached
    const int ntop = (int)(level_base(top + 1) - 1);
    for (int t = threadIdx.x; t < ntop; t += blockDim.x) {
        const double* g = geom + 4 * (int64_t)(t + 1);
        sg[t][0] = g[0];
        sg[t][1] = g[1];
        sg[t][2] = g[2];
    }
    __syncthreads();
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= M) return;
    const double2 q = y[i];
    int64_t b = 0, j = 0;
    for (int l = 0; l + 1 < L; ++l) {
        const int64_t c0 = level_base(l + 1) + 4 * j;
        int best = -1;
        double bq = 2.0;     // the smallest (|y - c| / r)^2 so far; at most 1 inside a disc
        if (l + 1 <= top) {
            for (int k = 0; k < 4; ++k) locate_child(q, sg[c0 + k - 1], k, best, bq);
        } else {
            for (int k = 0; k < 4; ++k) locate_child(q, geom + 4 * (c0 + k), k, best, bq);
        }
        if (best < 0) break;
        b = c0 + best;
        j = 4 * j + best;
    }
    box[i] = (int32_t)b;
    rank[i] = atomicAdd(&cnt[b], 1);
}

// The boxes' points and the leaves' near-field items (the points of a leaf in
// groups of kPtsItem) as offsets: one exclusive scan of both, and the items
// written from it.  Two passes over blocks of 1024 boxes (sums per block, then
// every block adds those before it); a tree of at most kScanOne boxes takes the
// second alone, one block walking the boxes.  Both sums, the items and the
// spare items (no target) in one kernel: ten launches that sorted the points
// and made the items are four or five (N = M = 1000 on one stream: 74 -> 53 us).
constexpr int kScanOne = 8192;
__device__ __forceinline__ int2 pts_counts(const int32_t* __restrict__ cnt, int b, int nb, int lb)
{
    const int c = b < nb ? cnt[b] : 0;
    return make_int2(c, b >= lb ? (c + kPtsItem - 1) / kPtsItem : 0);
}
// exclusive scan over the workgroup's 1024 threads; tot receives its sums
__device__ __forceinline__ int2 scan2_1024(int2 v, int2 (*sh)[16], int2& tot)
{
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int2 x = make_int2(wave_incl_scan(v.x), wave_incl_scan(v.y));
    __syncthreads();                       // the sums of an earlier call are read
    if (lane == 63) (*sh)[w] = x;
    __syncthreads();
    int2 before = make_int2(0, 0);
    tot = make_int2(0, 0);
    for (int k = 0; k < 16; ++k) {
        const int2 s = (*sh)[k];
        if (k < w) { before.x += s.x; before.y += s.y; }
        tot.x += s.x;
        tot.y += s.y;
    }
    return make_int2(before.x + x.x - v.x, before.y + x.y - v.y);
}
__global__ void __launch_bounds__(1024)
k_pts_scan_sums(const int32_t* __restrict__ cnt, int nb, int lb, int2* bsum)
{
    __shared__ int2 sh[16];
    int2 tot;
    scan2_1024(pts_counts(cnt, blockIdx.x * 1024 + threadIdx.x, nb, lb), &sh, tot);
    if (threadIdx.x == 0) bsum[blockIdx.x] = tot;
}
__global__ void __launch_bounds__(1024)
k_pts_scan(const int32_t* __restrict__ cnt, int nb, int lb, const int2* __restrict__ bsum, int32_t* off,
           PtsItem* items, int nx)
{
    __shared__ int2 sh[16];
    int2 base = make_int2(0, 0), all = make_int2(0, 0), tot;
    if (bsum) {                            // the sums of the blocks before this one, and of all
        for (int b0 = 0; b0 < (int)gridDim.x; b0 += 1024) {
            const int b = b0 + threadIdx.x;
            const int2 v = b < (int)gridDim.x ? bsum[b] : make_int2(0, 0);
            const bool pre = b < (int)blockIdx.x;
            scan2_1024(v, &sh, tot);
            all.x += tot.x;
            all.y += tot.y;
            scan2_1024(pre ? v : make_int2(0, 0), &sh, tot);
            base.x += tot.x;
            base.y += tot.y;
        }
    }
    const int first = bsum ? blockIdx.x * 1024 : 0, last = bsum ? min(first + 1024, nb) : nb;
    for (int b0 = first; b0 < last; b0 += 1024) {
        const int b = b0 + threadIdx.x;
        const int2 v = pts_counts(cnt, b, nb, lb), e = scan2_1024(v, &sh, tot);
        if (b < nb) {
            off[b] = base.x + e.x;
            if (b == nb - 1) off[nb] = base.x + e.x + v.x;
            for (int t = 0; t < v.y; ++t)
                items[base.y + e.y + t] = PtsItem{b, t * kPtsItem, min(kPtsItem, v.x - t * kPtsItem), 0};
        }
        base.x += tot.x;
        base.y += tot.y;
    }
    if (!bsum) all = base;
    for (int k = all.y + blockIdx.x * 1024 + threadIdx.x; k < nx; k += gridDim.x * 1024)
        items[k] = PtsItem{0, 0, 0, 0};
}

// sorted position of every point: its box's offset plus its rank in the box
// (the order inside a box is immaterial: each point's value depends on its
// own position only), and its position in box order, as the near-field kernel
// reads its targets
__global__ void k_pts_scatter(const double2* __restrict__ y, const int32_t* __restrict__ box, int64_t M,
                              const int32_t* __restrict__ off, const int32_t* __restrict__ rank, int32_t* order,
                              double* rx, double* ry)
{
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= M) return;
    const double2 v = y[i];
    const int q = off[box[i]] + rank[i];
    order[q] = (int32_t)i;
    rx[q] = v.x;
    ry[q] = v.y;
}

// point criterion: a box of radius r at squared distance d2 is well separated
// from a point when r^2 <= t^2 d2 (d2 > 0), t = theta / (1 + theta)
__device__ __forceinline__ bool point_separated(double r, double dx, double dy, double theta)
{
#pragma clang fp contract(off)     // every product and sum rounded alone, as in the list build
    const double d2 = ((dx * dx) + (dy * dy));
    const double rr = (r * r);
    return (d2 > 0.0) && (rr <= ((theta * theta) * d2));
}

template <class T>
__device__ __forceinline__ double2 coef(const T* c, int k)
{
    return make_double2((double)c[2 * k], (double)c[2 * k + 1]);
}

// multipole expansion of a box at the point: phi += (u/rs) sum a_k u^k and
// dphi -= (u/rs)^2 sum (k+1) a_k u^k, u = rs/(y - c)
template <class T, bool DER>
__device__ __forceinline__ void m2p(const T* a, int p, double rs, double dx, double dy, double2& phi, double2& dphi)
{
    const double id = 1.0 / (dx * dx + dy * dy);
    const double2 inv = make_double2(dx * id, -dy * id);       // 1 / (y - c)
    const double2 u = make_double2(rs * inv.x, rs * inv.y);
    double2 s = coef(a, p - 1), t = make_double2((double)p * s.x, (double)p * s.y);
    for (int k = p - 2; k >= 0; --k) {
        const double2 ak = coef(a, k);
        s = cmul(s, u);
        s.x += ak.x;
        s.y += ak.y;
        if (DER) {
            t = cmul(t, u);
            t.x += (double)(k + 1) * ak.x;
            t.y += (double)(k + 1) * ak.y;
        }
    }
    const double2 f = cmul(s, inv);
    phi.x += f.x;
    phi.y += f.y;
    if (DER) {
        const double2 g = cmul(t, cmul(inv, inv));
        dphi.x -= g.x;
        dphi.y -= g.y;
    }
}

// 1/x by v_rcp_f64 and two Newton steps (a division takes three times the instructions)
__device__ __forceinline__ double rcp_full(double x)
{
    double y = __builtin_amdgcn_rcp(x);
    y = fma(y, fma(-x, y, 1.0), y);
    return fma(y, fma(-x, y, 1.0), y);
}

// the points of one leaf, directly: phi += m/(y - x), dphi -= m/(y - x)^2
template <bool DER>
__device__ __forceinline__ void direct64(const double* __restrict__ X, const double* __restrict__ Y,
                                         const double2* __restrict__ mt, int st, int n, double yx, double yy,
                                         double2& phi, double2& dphi)
{
#pragma unroll 8
    for (int q = 0; q < n; ++q) {         // unrolled: eight loads in flight
        const double2 m = mt[st + q];
        const double4 sv = make_double4(X[st + q], Y[st + q], m.x, m.y);   // x, y, Re m, Im m
        const double dx = yx - sv.x, dy = yy - sv.y;
        const double r2 = dx * dx + (dy * dy + DBL_MIN);     // 0/DBL_MIN: a coincident source adds 0
        const double id = rcp_full(r2);
        const double a = sv.z * dx + sv.w * dy, b = sv.w * dx - sv.z * dy;   // m conj(y - x)
        phi.x += a * id;
        phi.y += b * id;
        if (DER) {
            // m conj(y - x)^2 / |y - x|^4, as (c id) id: a coincident source
            // (c = d = 0) adds 0, not 0 * inf
            const double c = a * dx + b * dy, d = b * dx - a * dy;
            dphi.x -= (c * id) * id;
            dphi.y -= (d * id) * id;
        }
    }
}

// (the difference in FP64 rounded once to FP32, the strengths rounded to
// FP32, as in the near-field kernel)
template <bool DER>
__device__ __forceinline__ void direct32(const double* __restrict__ X, const double* __restrict__ Y,
                                         const double2* __restrict__ mt, int st, int n, double yx, double yy,
                                         float2& phi, float2& dphi)
{
    // unrolled by four: with eight sources' loads in flight the descent kernel
    // held 129 vector registers (3 wavefronts per SIMD) and ran 1.6x longer
#pragma unroll 4
    for (int q = 0; q < n; ++q) {
        const double2 m = mt[st + q];
        const float mr = (float)m.x, mi = (float)m.y;
        const float dx = (float)(yx - X[st + q]);
        const float dy = (float)(yy - Y[st + q]);
        const float r2 = fmaf(dx, dx, fmaf(dy, dy, FLT_MIN));
        const float id = __builtin_amdgcn_rcpf(r2);
        const float a = fmaf(mr, dx, mi * dy), b = fmaf(mi, dx, -(mr * dy));
        phi.x = fmaf(a, id, phi.x);
        phi.y = fmaf(b, id, phi.y);
        if (DER) {
            // (c id) id: a coincident source (c = d = 0) adds 0, not 0 * inf
            const float c = fmaf(a, dx, b * dy), d = fmaf(b, dx, -(a * dy));
            dphi.x = fmaf(-(c * id), id, dphi.x);
            dphi.y = fmaf(-(d * id), id, dphi.y);
        }
    }
}

// What a box adds to a point's near field: its multipole expansion when it
// is well separated from the point (never the root, which has none), its
// points when it is a leaf; returns false (nothing added) when the box must
// be opened.  The mixed direct sums go to FP32 accumulators (nf, nd).
template <class T, bool DER>
struct Visit {
    double2 y;
    int L, p;
    double theta;
    const int8_t* level;
    const double* geom;
    const int32_t *bstart, *bcount;
    const T* mpole;
    const double *X, *Y;            // the sources: positions and strengths in tree order
    const double2* mt;

    __device__ __forceinline__ bool operator()(int32_t bx, int lv, double2& phi, double2& dphi, float2& nf,
                                               float2& nd, bool direct = false) const
    {
        const double* g = geom + 4 * (int64_t)bx;
        const double dx = y.x - g[0], dy = y.y - g[1];
        if (!direct && lv > 0 && point_separated(g[2], dx, dy, theta)) {
            m2p<T, DER>(mpole + 2 * (int64_t)bx * coef_ld<T>(p), p, g[3], dx, dy, phi, dphi);
            return true;
        }
        if (lv != L - 1) return false;
        if constexpr (std::is_same<T, float>::value) direct32<DER>(X, Y, mt, bstart[bx], bcount[bx], y.x, y.y, nf, nd);
        else direct64<DER>(X, Y, mt, bstart[bx], bcount[bx], y.x, y.y, phi, dphi);
        return true;
    }

    // the whole subtree of box S, one box after the other (no stack: the
    // next box is the next sibling, or that of the nearest ancestor that has
    // one; done when back at S)
    __device__ void subtree(int32_t S, double2& phi, double2& dphi, float2& nf, float2& nd) const
    {
        int32_t cur = S;
        int lv = level[S];
        while (true) {
            if (!(*this)(cur, lv, phi, dphi, nf, nd)) {
                cur = (int32_t)(level_base(lv + 1) + 4 * ((int64_t)cur - level_base(lv)));   // first child
                ++lv;
                continue;
            }
            bool done = false;
            while (true) {
                if (cur == S) { done = true; break; }
                const int64_t j = (int64_t)cur - level_base(lv);
                if ((j & 3) != 3) { ++cur; break; }
                cur = (int32_t)(level_base(lv - 1) + (j >> 2));
                --lv;
            }
            if (done) return;
        }
    }
};

// The near field with the derivative of the points in leaves: a wavefront per
// work item (at most 16 points of one leaf), lane (g, t) = point t, every fourth
// box of the leaf's strong list from g on, its sources one after the other (the
// 16 lanes of a row read the same source, four boxes are in flight); the four
// rows' sums are added by two row exchanges.  In mixed precision a box's FP32
// sums start at zero (boxes 64 entries apart share one: the order of the
// descents' lanes) and are added in FP64.  N = M = 1e5, L = 7: 212 us as descents
// of a wavefront per point, 12 of its 64 lanes with a box to sum, now 57 us.
template <class T, bool PART>
__global__ void __launch_bounds__(256)
k_pts_near_der(const PtsItem* __restrict__ items, int nx, const int32_t* __restrict__ off,
               const double* __restrict__ rx, const double* __restrict__ ry, const int32_t* __restrict__ bstart,
               const int32_t* __restrict__ bcount, const int32_t* __restrict__ s_beg,
               const int32_t* __restrict__ s_cnt, const int32_t* __restrict__ s_ids, const double* __restrict__ X,
               const double* __restrict__ Y, const double2* __restrict__ mt, int longest, double2* tnear,
               double2* tdnear)
{
    const int i = __builtin_amdgcn_readfirstlane(xcd_block() * 4 + (threadIdx.x >> 6));
    if (i >= nx) return;
    const PtsItem it = items[i];
    if (it.tn == 0) return;                       // a spare item
    const int g = (threadIdx.x >> 4) & 3, t = threadIdx.x & 15;
    const int64_t q = (int64_t)off[it.leaf] + it.t0 + (t < it.tn ? t : 0);
    const double yx = rx[q], yy = ry[q];
    const int e0 = s_beg[it.leaf], n = s_cnt[it.leaf];
    if (PART && n > longest) return;              // its points are descended
    double2 phi = make_double2(0.0, 0.0), dphi = make_double2(0.0, 0.0);
    // the first 64 boxes' ranges, a box per lane, loaded together
    const int lane = threadIdx.x & 63;
    int st0 = 0, n0 = 0;
    if (lane < n) {
        const int32_t S = s_ids[e0 + lane];
        st0 = bstart[S];
        n0 = bcount[S];
    }
    const int rows = (min(n, 64) + 3) >> 2;        // uniform: every lane takes part in the exchanges
    for (int k = 0; k < rows; ++k) {
        const int r = g + 4 * k;
        int st = __shfl(st0, r, 64), ns = __shfl(n0, r, 64);   // (no box: no sources)
        float2 nf = make_float2(0.f, 0.f), nd = make_float2(0.f, 0.f);
        for (int e = r; e < n; e += 64) {
            if (e != r) {
                const int32_t S = s_ids[e0 + e];
                st = bstart[S];
                ns = bcount[S];
            }
            if constexpr (std::is_same<T, float>::value) direct32<true>(X, Y, mt, st, ns, yx, yy, nf, nd);
            else direct64<true>(X, Y, mt, st, ns, yx, yy, phi, dphi);
        }
        phi.x += (double)nf.x;
        phi.y += (double)nf.y;
        dphi.x += (double)nd.x;
        dphi.y += (double)nd.y;
    }
    auto sum4 = [](double v) {
        v += partner<16>(v);
        return v + partner<32>(v);
    };
    phi = make_double2(sum4(phi.x), sum4(phi.y));
    dphi = make_double2(sum4(dphi.x), sum4(dphi.y));
    if (g == 0 && t < it.tn) {
        tnear[q] = phi;
        tdnear[q] = dphi;
    }
}

constexpr int kFront = 512;   // frontier boxes per wavefront (LDS)

// The near field of the points at box-order positions q < nq (PART: those in leaves
// whose strong list has at most `skip` boxes left out) by descents of
// their box's strong list: one wavefront per point, breadth first, lanes over
// the frontier (the first frontier is the strong list itself, read from the
// pool; later ones are in LDS).  A lane's box adds its expansion or its
// points, or puts its four children in the next frontier; a box whose
// children no longer fit is descended by its lane alone.  The lanes' sums
// are added by a fixed butterfly, so the result does not depend on timing.
// Results go to tnear (and tdnear) in box order.  A descent is a chain of
// dependent loads, so wavefronts in flight set its rate: the mixed kernel
// without the derivative is held to 80 registers (six wavefronts per SIMD,
// no spills); the others need 97-120 and would spill below that.
template <class T, bool DER, bool PART>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(sizeof(T) == 4 && !DER ? 6 : 1)))
k_pts_descend(const double2* __restrict__ y, const int32_t* __restrict__ order, const int32_t* __restrict__ box,
              const int32_t* __restrict__ nq_dev, int skip, int L, const int8_t* __restrict__ level,
              const double* __restrict__ geom, const int32_t* __restrict__ bstart, const int32_t* __restrict__ bcount,
              const int32_t* __restrict__ s_beg, const int32_t* __restrict__ s_cnt, const int32_t* __restrict__ s_ids,
              const T* __restrict__ mpole, int p, double theta, const double* __restrict__ X,
              const double* __restrict__ Y, const double2* __restrict__ mt, double2* tnear, double2* tdnear)
{
    __shared__ int32_t front[4][2][kFront];
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const unsigned long long below = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    const int nq = *nq_dev;
    const int nw = (int)gridDim.x * 4;
    auto descend = [&](int q) {      // uniform in the wavefront
        const int32_t i = order[q];
        Visit<T, DER> vis;
        vis.y = y[i];
        vis.L = L; vis.p = p; vis.theta = theta; vis.level = level; vis.geom = geom;
        vis.bstart = bstart; vis.bcount = bcount; vis.mpole = mpole;
        vis.X = X; vis.Y = Y; vis.mt = mt;
        const int32_t B = box[i];
        double2 phi = make_double2(0.0, 0.0), dphi = make_double2(0.0, 0.0);
        float2 nf = make_float2(0.f, 0.f), nd = make_float2(0.f, 0.f);
        int32_t* cur = front[w][0];
        int32_t* nxt = front[w][1];
        const int e0 = s_beg[B];
        int n = s_cnt[B];
        bool first = true;
        // a point in a leaf sums the leaves of its strong list directly, as
        // the sources of that leaf do
        const bool in_leaf = level[B] == L - 1;
        while (n > 0) {
            int nn = 0;
            for (int c0 = 0; c0 < n; c0 += 64) {
                const int k = c0 + lane;
                int32_t bx = -1;
                if (k < n) bx = first ? s_ids[e0 + k] : cur[k];
                bool open = false;
                int lv = 0;
                if (bx >= 0) {
                    lv = level[bx];
                    open = !vis(bx, lv, phi, dphi, nf, nd, first && in_leaf);
                }
                const unsigned long long om = __ballot(open);
                if (open) {
                    const int pos = nn + 4 * __popcll(om & below);
                    if (pos + 4 <= kFront) {
                        const int32_t c = (int32_t)(level_base(lv + 1) + 4 * ((int64_t)bx - level_base(lv)));
                        for (int t = 0; t < 4; ++t) nxt[pos + t] = c + t;
                    } else {
                        vis.subtree(bx, phi, dphi, nf, nd);
                    }
                }
                nn = min(nn + 4 * __popcll(om), kFront);
            }
            wave_sync();
            int32_t* t = cur;
            cur = nxt;
            nxt = t;
            n = nn;
            first = false;
        }
        phi.x += (double)nf.x;
        phi.y += (double)nf.y;
        dphi.x += (double)nd.x;
        dphi.y += (double)nd.y;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            phi.x += __shfl_xor(phi.x, o, 64);
            phi.y += __shfl_xor(phi.y, o, 64);
            if (DER) {
                dphi.x += __shfl_xor(dphi.x, o, 64);
                dphi.y += __shfl_xor(dphi.y, o, 64);
            }
        }
        if (lane == 0) {
            tnear[q] = phi;
            if (DER) tdnear[q] = dphi;
        }
        wave_sync();
    };
    // a wavefront's points are every nw-th
    if constexpr (!PART) {
        for (int q = (int)blockIdx.x * 4 + w; q < nq; q += nw) descend(q);
    } else {
        // 64 of them are looked at together
        for (int64_t q0 = (int)blockIdx.x * 4 + w; q0 < nq; q0 += (int64_t)64 * nw) {
            const int64_t ql = q0 + (int64_t)lane * nw;
            bool mine = ql < nq;
            if (mine) {
                const int32_t B = box[order[ql]];
                mine = level[B] != L - 1 || s_cnt[B] > skip;
            }
            for (unsigned long long todo = __ballot(mine); todo; todo &= todo - 1)
                descend((int)(q0 + (int64_t)__builtin_ctzll(todo) * nw));
        }
    }
}

// the far field of every point (B's local expansion; the root has none) plus
// its near field (tnear, box order), into the outputs in input order
template <class T, bool DER>
__global__ void __launch_bounds__(256)
k_pts_far(const double2* __restrict__ y, int64_t M, const int32_t* __restrict__ order, const int32_t* __restrict__ box,
          const int8_t* __restrict__ level, const double* __restrict__ geom, const T* __restrict__ local, int p,
          const double2* __restrict__ tnear, const double2* __restrict__ tdnear, double2* __restrict__ phi_out,
          double2* __restrict__ dphi_out)
{
    const int64_t qi = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (qi >= M) return;
    const int32_t i = order[qi];
    const double2 yv = y[i];
    const int32_t B = box[i];
    double2 phi = tnear[qi], dphi = DER ? tdnear[qi] : make_double2(0.0, 0.0);
    if (level[B] > 0) {
        const double* g = geom + 4 * (int64_t)B;
        const double irs = 1.0 / g[3];
        const double2 w = make_double2((yv.x - g[0]) * irs, (yv.y - g[1]) * irs);
        const T* b = local + 2 * (int64_t)B * coef_ld<T>(p);
        double2 s = coef(b, p - 1), t = make_double2((double)(p - 1) * s.x, (double)(p - 1) * s.y);
        for (int l = p - 2; l >= 0; --l) {
            const double2 bl = coef(b, l);
            s = cmul(s, w);
            s.x += bl.x;
            s.y += bl.y;
            if (DER && l >= 1) {
                t = cmul(t, w);
                t.x += (double)l * bl.x;
                t.y += (double)l * bl.y;
            }
        }
        phi.x += s.x;
        phi.y += s.y;
        if (DER && p > 1) {
            dphi.x += t.x * irs;
            dphi.y += t.y * irs;
        }
    }
    phi_out[i] = phi;
    if (DER) dphi_out[i] = dphi;
}

void evaluate_points_device(Plan& pl, const double* m, const double* y, int64_t M, double* phi, double* dphi,
                            hipStream_t s)
{
    Tree& t = *pl.tree;
    TreeSchedule& sc = *t.sched;
    if (sc.nprob != 1) throw Error(FMM_EINVAL, "evaluation points need a plan over a single problem");
    if (M < 0 || M >= INT32_MAX) throw Error(FMM_EINVAL, "the number of evaluation points must be in [0, 2^31 - 1)");
    if (M == 0) return;
    const bool mixed = pl.precision == FMM_MIXED, der = dphi != nullptr;
    const int L = sc.L[0];
    // the near field of a point in a leaf is the direct sum over the sources
    // of the leaf's strong list (the near-field kernel); a point stopped
    // higher up (outside the discs of the leaves, a few per cent of points
    // among the sources) descends its box's strong list instead, a wavefront
    // per point
    const int ld = L - 1;
    const int64_t nb = sc.nbox, lb = level_base(ld);
    const int nleaf = (int)(nb - lb);
    // a point takes a box's multipole expansion when the box would be well
    // separated from a box of its own radius around the point: r (1 + theta)
    // <= theta d, i.e. r <= theta' d with theta' = theta / (1 + theta); the
    // ratio r/d of every such expansion is then that of the M2L shifts of the
    // plan, and so is its truncation
    const double theta_pt = pl.theta / (1.0 + pl.theta);
    // item list: at most M / kPtsItem + nleaf items (spares have no target)
    const int64_t nx = M / kPtsItem + nleaf + 1;
    if (nx >= INT32_MAX / 4) throw Error(FMM_EINVAL, "too many evaluation points");
    DBuf<int32_t> box, rank, order, cnt, off;
    DBuf<int2> bsum;
    DBuf<double> rx, ry, tnear, tdnear;
    DBuf<PtsItem> items;
    box.alloc(M, s);
    rank.alloc(M, s);
    order.alloc(M, s);
    cnt.alloc(nb, s);
    off.alloc(nb + 1, s);
    bsum.alloc((nb + 1023) / 1024, s);
    items.alloc(nx, s);
    rx.alloc(M, s);
    ry.alloc(M, s);
    tnear.alloc(2 * M, s);
    if (der) tdnear.alloc(2 * M, s);
    // the points on the second stream, the sources' far field on the caller's;
    // what needs no lists is enqueued first, so that the device works while the
    // host waits for the lists' flags of a new plan
    // two streams from 50,000 points on: the fork and the joins cost more than
    // the overlap hides below (one stream / two, N = M: 30,000 91 / 123 us
    // mixed, 118 / 126 us FP64 with the derivative; 100,000 153 / 127 and
    // 195 / 163 us FP64)
    const bool two = M >= kTwoStreamPoints;
    plan_start(pl, s);
    hipStream_t ps = s;
    if (two) {
        second_stream(pl);
        ps = pl.nstream;
        FMM_HIP(hipEventRecord(pl.ev_fork, s));
        FMM_HIP(hipStreamWaitEvent(ps, pl.ev_fork, 0));
    }
    // the second stream's work is joined into `s` before the buffers above go
    // back to the pool, also when a call below fails
    struct Join {
        Plan& pl;
        hipStream_t s;
        bool done;
        void now()
        {
            if (done) return;
            done = true;
            FMM_HIP(hipEventRecord(pl.ev_join, pl.nstream));
            FMM_HIP(hipStreamWaitEvent(s, pl.ev_join, 0));
        }
        ~Join()
        {
            if (done) return;
            (void)hipEventRecord(pl.ev_join, pl.nstream);
            (void)hipStreamWaitEvent(s, pl.ev_join, 0);
        }
    } join{pl, s, !two};
    far_field_up(pl, m, s);
    const unsigned gb = (unsigned)((nb + 255) / 256), gm = (unsigned)((M + 255) / 256);
    k_pts_clear<<<gb, 256, 0, ps>>>(cnt.p, nb);
    k_pts_locate<<<gm, 256, 0, ps>>>((const double2*)y, M, L, t.geom.p, box.p, cnt.p, rank.p);
    if (nb <= kScanOne) {
        k_pts_scan<<<1, 1024, 0, ps>>>(cnt.p, (int)nb, (int)lb, nullptr, off.p, items.p, (int)nx);
    } else {
        const unsigned gs = (unsigned)((nb + 1023) / 1024);
        k_pts_scan_sums<<<gs, 1024, 0, ps>>>(cnt.p, (int)nb, (int)lb, bsum.p);
        k_pts_scan<<<gs, 1024, 0, ps>>>(cnt.p, (int)nb, (int)lb, bsum.p, off.p, items.p, (int)nx);
    }
    k_pts_scatter<<<gm, 256, 0, ps>>>((const double2*)y, box.p, M, off.p, rank.p, order.p, rx.p, ry.p);
    check_launch("point order");
    if (two) FMM_HIP(hipEventRecord(pl.ev_join, ps));     // the items, for the near field
    // the descents read the multipoles and the lists: after the upward pass
    plan_finalize(pl);
    plan_join(pl, s);
    if (two) {
        FMM_HIP(hipEventRecord(pl.ev_fork, s));
        FMM_HIP(hipStreamWaitEvent(ps, pl.ev_fork, 0));
    }
    far_field_down(pl, s);
    if (two) FMM_HIP(hipStreamWaitEvent(s, pl.ev_join, 0));
    // descents: the points that stopped above the leaves (box-order positions
    // before the first leaf).  Workgroups: four times those the occupancy holds at
    // once (six wavefronts per SIMD for the mixed kernel without the derivative,
    // four for the others), so that the last ones even out what the near field
    // beside them and long lists make uneven (once / four times, us, FP64 phi and
    // with the derivative: 100,000 points beside 3000 sources on a line, nearly
    // all descended 1237 / 1149 and 1172 / 1167; beside 300,000 clustered sources
    // 2057 / 2048 and 1845 / 1769; 1e6 beside 1e6 846 / 833 and 1298 / 1300)
    const unsigned gd = (unsigned)std::min<int64_t>((M + 3) / 4, 4 * (mixed && !der ? 1536 : 1024));
    // with the derivative every near field is a descent where the points are few,
    // or few per leaf: the own kernel's wavefront takes the points of one leaf
    // and sums three boxes in turn, whether it holds one point or sixteen.
    // Descents / own kernel, us, by points per leaf, FP64 (mixed):
    //   N = 1e5, 7 levels  2: 107 / 132 (99 / 117)   3: 112 / 134 (107 / 119)   8: 155 / 145 (145 / 128)
    //   N = 1e6, 8 levels  1: 216 / 435 (199 / 379)  3: 383 / 462 (355 / 405)   5: 537 / 460 (492 / 400)
    //   N = 1e6, 9 levels  1: 407 / 656 (337 / 470)  2: 563 / 695 (547 / 504)   3: 720 / 737 (760 / 538)
    // and on small trees N = 30,000 with M = 8192, 8 per leaf, 84 / 100 (80 / 90).
    const bool all_descend = der && M <= std::max<int64_t>(kDescendPoints, (int64_t)nleaf * (mixed ? 2 : 3));
    // Where some strong list is split into work chunks, the points of leaves with
    // longer lists than a line are descended too: the own kernel walks every fourth
    // box in turn, a descent every 64th.  100,000 points beside the sources, all
    // descents / above 512 boxes / own kernel alone, us: 300,000 sources of which 5
    // lie far off (one list of 16,384 boxes) 2500 / 2440 / 10,760, 300,000 in clusters
    // 3320 / 3040 / 4720, 30,000 in clusters (lists of up to 244 boxes) 860 / 790 /
    // 790, 100,000 in clusters 1270 / 1310 / 1530.  Few points leave the chip to the
    // long lists, hence a lower line.  Clustered sources, uniform points, FP64, lines
    // at 64 / 128 / 512 boxes: N = 20,000 on 7 levels M = 20,000 150 / 178 / 262, M =
    // 100,000 269 / 281 / 328; on 6 levels M = 20,000 182 / 206 / 242, 40,000 (39 per
    // leaf) 281 / 268 / 261; N = 30,000 on 6 levels M = 20,000 254 / 293 / 343; N = 1e5 on
    // 7 levels M = 100,000 766 / 736 / 812; N = 300,000 on 8 levels M = 98,304 1428 / 1394
    // / 1693, 262,144 3400 / 3399 / 3237; N = 1e6 on 8 levels M = 98,304 6830 / 6756 /
    // 6522, 262,144 18,091 / 18,377 / 14,361; N = 60,000 on 7 levels M = 300,000 1785 /
    // 1586 / 1086.  Not for what every list of uniform sources holds at small theta: N
    // = 1e5 on 6 levels, theta = 0.15, M = 30,720, mixed 1007 / 605 / 605, at 0.2 442 /
    // 416 / 417.
    const bool part_descend = der && !all_descend && pl.split_p2p;
    const int32_t* nq_dev = off.p + (all_descend || part_descend ? nb : lb);
    const int line = long_list(M, nleaf, pl.theta);
    const int skip = part_descend ? line : 0, longest = part_descend ? line : INT32_MAX;
#define DESC_ARGS                                                                                             \
    (const double2*)y, order.p, box.p, nq_dev, skip, L, sc.d_box_level.p, t.geom.p, sc.d_box_start.p,         \
        sc.d_box_count.p, pl.s_beg.p, pl.s_cnt.p, pl.s_ids.p
#define FAR_ARGS (const double2*)y, M, order.p, box.p, sc.d_box_level.p, t.geom.p
#define SRC_ARGS t.x.p, t.y.p, (const double2*)pl.mtree.p
    double2* tn = (double2*)tnear.p;
    double2* td = der ? (double2*)tdnear.p : nullptr;
    auto run = [&](auto tag, auto dtag) {
        using T = decltype(tag);
        constexpr bool DER = decltype(dtag)::value;
        const T* mp = (const T*)pl.mpole.p;
        if (DER && part_descend)
            k_pts_descend<T, DER, DER><<<gd, 256, 0, ps>>>(DESC_ARGS, mp, pl.p, theta_pt, SRC_ARGS, tn, td);
        else
            k_pts_descend<T, DER, false><<<gd, 256, 0, ps>>>(DESC_ARGS, mp, pl.p, theta_pt, SRC_ARGS, tn, td);
        // the near field of the points in leaves, over the sources of the
        // leaf's strong list
        if constexpr (DER) {
            if (!all_descend) {
                auto near_der = part_descend ? k_pts_near_der<T, true> : k_pts_near_der<T, false>;
                near_der<<<(unsigned)((nx + 3) / 4), 256, 0, s>>>(
                    items.p, (int)nx, off.p, rx.p, ry.p, sc.d_box_start.p, sc.d_box_count.p, pl.s_beg.p, pl.s_cnt.p,
                    pl.s_ids.p, SRC_ARGS, longest, tn, td);
            }
        } else {
            Targets tgt;
            tgt.x = rx.p;
            tgt.y = ry.p;
            tgt.start = off.p;
            launch_p2p(mixed, 4, 4, items.p, 0, nullptr, (int)nx, nullptr, nullptr, nullptr, sc.d_box_start.p,
                       sc.d_box_count.p, pl.s_beg.p, pl.s_cnt.p, pl.s_ids.p, SRC_ARGS, tnear.p, s, nullptr, 0.0,
                       nullptr, tgt, pl.tune.p2p_src_tile);
        }
        join.now();
        k_pts_far<T, DER><<<gm, 256, 0, s>>>(FAR_ARGS, (const T*)pl.local.p, pl.p, tn, td, (double2*)phi,
                                             (double2*)dphi);
    };
    if (mixed) der ? run(float{}, std::true_type{}) : run(float{}, std::false_type{});
    else der ? run(double{}, std::true_type{}) : run(double{}, std::false_type{});
#undef DESC_ARGS
#undef FAR_ARGS
#undef SRC_ARGS
    check_launch("points");
}

}  // namespace fmm
