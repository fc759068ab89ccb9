// expansions.hip -- P2M and L2P of shallow problems (one or two levels: no
// shift between levels) and of leaves with many points (others: subtree.hip), and
// the point gathers (Sec. 2.1, Fig. 2.2) on gfx950.
//
// Expansions are stored scaled by the box's scaling radius rs (its radius,
// or the nearest ancestor's radius when it is 0):
//     multipole  a_k = sum_j m_j ((z_j - c)/rs)^k        (k < p)
//     local      phi(z) = sum_l b_l ((z - c)/rs)^l
// so that every stored coefficient and every power is bounded by the data
// (|z - c| <= r <= rs inside the box).  In these variables the shifts are
//     M2M  a^P_k = sum_{l<=k} C(k,l) rho^l tau^(k-l) a^C_l
//     L2L  b^C_l = sum_{k>=l} C(k,l) rho^l tau^(k-l) b^P_k
// with rho = rs_C / rs_P and tau = (c_C - c_P) / rs_P (both exact re-centrings
// of the truncated series; subtree.hip).  All four operators compute in FP64; T is the
// storage type of the coefficients (double for the FP64 path, float for the
// mixed path).
#include "fmm_internal.h"
#include "kernels_common.h"

namespace fmm {

// strengths into tree order (with the tree's positions, the near field's
// sources)
__global__ void k_gather(int64_t n, const int32_t* __restrict__ perm, const double2* __restrict__ m, double2* mtree)
{
    int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= n) return;
    mtree[i] = m[perm[i]];
}

// P2M at the leaves.  G lanes per leaf (64/G leaves per wavefront, four
// wavefronts per workgroup): each lane takes the points j = lane, lane + G,
// ... of its leaf and accumulates the P terms m_j w_j^k, k = k0 .. k0+P-1
// (w_j = (z_j - c)/rs) in FP64 registers; a transposing butterfly then sums
// them over the G lanes.  P = 16 or 32; p > 32 takes two launches (k0 = 0
// and 32).
__device__ __forceinline__ double2 cpow(double2 b, int e)
{
    double2 r = make_double2(1.0, 0.0);
    while (e) {
        if (e & 1) r = cmul(r, b);
        b = cmul(b, b);
        e >>= 1;
    }
    return r;
}
template <class T, int G, int P, bool GATHER>
__global__ void __launch_bounds__(256)
k_p2m(const int32_t* __restrict__ leaves, int nleaf, const int32_t* __restrict__ bstart,
      const int32_t* __restrict__ bcount, const double* __restrict__ geom, const double* __restrict__ X,
      const double* __restrict__ Y, const double2* __restrict__ mt, int p, int k0, T* mp, GatherOut go)
{
    constexpr int V = 2 * P;
    const int lane = threadIdx.x & 63;
    const int li = (blockIdx.x * 4 + (threadIdx.x >> 6)) * (64 / G) + lane / G;
    const int sl = lane % G;
    const bool valid = li < nleaf;
    int g = 0, st = 0, n = 0;
    double cx = 0.0, cy = 0.0, inv = 0.0;
    if (valid) {
        g = leaves[li];
        st = bstart[g];
        n = bcount[g];
        cx = geom[4 * (int64_t)g];
        cy = geom[4 * (int64_t)g + 1];
        inv = 1.0 / geom[4 * (int64_t)g + 3];
    }
    double v[V];
#pragma unroll
    for (int i = 0; i < V; ++i) v[i] = 0.0;
    for (int j = sl; j < n; j += G) {
        const int i = st + j;
        double2 w, t;
        if constexpr (GATHER) {
            // the gather's output for this point, as k_gather writes it
            const double2 mm = go.m[go.perm[i]];
            const double x = X[i], y = Y[i];
            if (go.mtree) go.mtree[i] = mm;
            w = make_double2((x - cx) * inv, (y - cy) * inv);
            t = mm;
        } else {
            w = make_double2((X[i] - cx) * inv, (Y[i] - cy) * inv);
            t = mt[i];
        }
        if (k0 != 0) t = cmul(t, cpow(w, k0));   // the block of terms from k0 on
#pragma unroll
        for (int k = 0; k < P; ++k) {
            v[2 * k] += t.x;
            v[2 * k + 1] += t.y;
            if (k + 1 < P) t = cmul(t, w);
        }
    }
    treduce<V, G>(v, lane);
    const int base = treduce_base<V, G>(sl);
    constexpr int NV = V >= G ? V / G : 1;
    const bool writer = V >= G || (sl & (G / V - 1)) == 0;
    if (valid && writer) {
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            const int idx = base + i, k = k0 + (idx >> 1);
            if (k < p) mp[2 * ((int64_t)g * coef_ld<T>(p) + k) + (idx & 1)] = (T)v[i];
        }
    }
}

// L2P at the leaves, plus the near field, scattered to input order.  G
// lanes per leaf as in P2M; every lane holds the leaf's P coefficients (FP64)
// and evaluates the series by Horner's rule at its points.
template <class T, int G, int P>
__global__ void __launch_bounds__(256)
k_l2p(const int32_t* __restrict__ leaves, int nleaf, const int32_t* __restrict__ bstart,
      const int32_t* __restrict__ bcount, const double* __restrict__ geom, const double* __restrict__ X,
      const double* __restrict__ Y, const T* __restrict__ loc, int p, const double2* __restrict__ nearf,
      const int32_t* __restrict__ perm, double2* phi, double2* phi_near, double2* phi_far,
      const long long* __restrict__ guard)
{
    if (guard != nullptr && *guard != 0) return;   // lists flagged: this launch is void
    using T2 = typename Vec2<T>::type;
    // P = 64: the coefficients stay in LDS (64 complex FP64 values would
    // take every register of a lane); below that they go to registers
    constexpr bool kLdsCoef = P > 32;
    __shared__ double2 sco[kLdsCoef ? 256 / G : 1][kLdsCoef ? P : 1];
    const int lane = threadIdx.x & 63;
    const int li = (blockIdx.x * 4 + (threadIdx.x >> 6)) * (64 / G) + lane / G;
    const int sl = lane % G;
    if (li >= nleaf) return;
    const int g = leaves[li];
    const int st = bstart[g], n = bcount[g];
    const double cx = geom[4 * (int64_t)g], cy = geom[4 * (int64_t)g + 1], inv = 1.0 / geom[4 * (int64_t)g + 3];
    const T2* b = reinterpret_cast<const T2*>(loc) + (int64_t)g * coef_ld<T>(p);
    double2 bl[kLdsCoef ? 1 : P];
    double2* co = sco[kLdsCoef ? threadIdx.x / G : 0];
    if constexpr (kLdsCoef) {
        for (int k = sl; k < P; k += G) {
            if (k < p) { const T2 v = b[k]; co[k] = make_double2((double)v.x, (double)v.y); }
            else co[k] = make_double2(0.0, 0.0);
        }
        wave_sync();   // the group lies in one wavefront
    } else {
#pragma unroll
        for (int k = 0; k < P; ++k) {
            if (k < p) { const T2 v = b[k]; bl[k] = make_double2((double)v.x, (double)v.y); }
            else bl[k] = make_double2(0.0, 0.0);
        }
    }
    for (int j = sl; j < n; j += G) {
        const int i = st + j;
        const double2 w = make_double2((X[i] - cx) * inv, (Y[i] - cy) * inv);
        double2 acc;
        if constexpr (kLdsCoef) {
            acc = co[P - 1];
            for (int l = P - 2; l >= 0; --l) {
                acc = cmul(acc, w);
                acc.x += co[l].x;
                acc.y += co[l].y;
            }
        } else {
            acc = bl[P - 1];
#pragma unroll
            for (int l = P - 2; l >= 0; --l) {
                acc = cmul(acc, w);
                acc.x += bl[l].x;
                acc.y += bl[l].y;
            }
        }
        const double2 nf = nearf[i];
        const int o = perm[i];
        if (phi) phi[o] = make_double2(acc.x + nf.x, acc.y + nf.y);
        if (phi_near) phi_near[o] = nf;
        if (phi_far) phi_far[o] = acc;
    }
}

// ------------------------------------------------------------ launchers

void launch_gather(int64_t n, const int32_t* perm, const double* m, double* mtree, hipStream_t s)
{
    k_gather<<<(unsigned)((n + 255) / 256), 256, 0, s>>>(n, perm, (const double2*)m, (double2*)mtree);
    check_launch("gather");
}

// lanes per leaf: the smallest of 16, 32, 64 not below the largest leaf
static int leaf_lanes(int leaf_max) { return leaf_max <= 16 ? 16 : (leaf_max <= 32 ? 32 : 64); }

template <class T>
void launch_p2m(const int32_t* leaves, int nleaf, const int32_t* bstart, const int32_t* bcount, int leaf_max,
                const double* geom, const double* X, const double* Y, const double* mt, int p, void* mp,
                hipStream_t s, const GatherOut* go)
{
    const GatherOut none{};
    const GatherOut& gg = go ? *go : none;
    if (nleaf == 0) return;
    const int G = leaf_lanes(leaf_max);
    const int PB = p <= 16 ? 16 : 32;
    const unsigned grid = (unsigned)((nleaf + 4 * (64 / G) - 1) / (4 * (64 / G)));
    // blocks of PB terms: the first one does the gather, the second (p > 32)
    // reads the strengths it put into tree order, if it did
    for (int k0 = 0; k0 < p; k0 += PB) {
        const bool gat = go && (k0 == 0 || !go->mtree);
        const double2* mtk = (const double2*)(k0 == 0 ? mt : (go ? (const double*)go->mtree : mt));
#define P2M_CASE(G_, P_)                                                                                   \
    if (G == G_ && PB == P_) {                                                                            \
        if (gat)                                                                                          \
            k_p2m<T, G_, P_, true><<<grid, 256, 0, s>>>(leaves, nleaf, bstart, bcount, geom, X, Y, mtk, p, \
                                                        k0, (T*)mp, gg);                                  \
        else                                                                                              \
            k_p2m<T, G_, P_, false><<<grid, 256, 0, s>>>(leaves, nleaf, bstart, bcount, geom, X, Y, mtk, p, \
                                                         k0, (T*)mp, gg);                                 \
        check_launch("p2m");                                                                              \
        continue;                                                                                         \
    }
        P2M_CASE(16, 16) P2M_CASE(32, 16) P2M_CASE(64, 16) P2M_CASE(16, 32) P2M_CASE(32, 32) P2M_CASE(64, 32)
#undef P2M_CASE
        throw Error(FMM_EINVAL, "unsupported P2M configuration");
    }
}

template <class T>
void launch_l2p(const int32_t* leaves, int nleaf, const int32_t* bstart, const int32_t* bcount, int leaf_max,
                const double* geom, const double* X, const double* Y, const void* loc, int p,
                const double* nearf, const int32_t* perm, double* phi, double* phi_near, double* phi_far,
                hipStream_t s, const long long* guard)
{
    if (nleaf == 0) return;
    const int G = leaf_lanes(leaf_max);
    const unsigned grid = (unsigned)((nleaf + 4 * (64 / G) - 1) / (4 * (64 / G)));
#define L2P_CASE(G_, P_)                                                                                   \
    if (G == G_ && (p <= 16 ? 16 : (p <= 32 ? 32 : 64)) == P_) {                                          \
        k_l2p<T, G_, P_><<<grid, 256, 0, s>>>(leaves, nleaf, bstart, bcount, geom, X, Y, (const T*)loc, p, \
                                              (const double2*)nearf, perm, (double2*)phi,                 \
                                              (double2*)phi_near, (double2*)phi_far, guard);              \
        check_launch("l2p");                                                                              \
        return;                                                                                           \
    }
    L2P_CASE(16, 16) L2P_CASE(32, 16) L2P_CASE(64, 16) L2P_CASE(16, 32) L2P_CASE(32, 32) L2P_CASE(64, 32)
    L2P_CASE(16, 64) L2P_CASE(32, 64) L2P_CASE(64, 64)
#undef L2P_CASE
    throw Error(FMM_EINVAL, "unsupported L2P configuration");
}

#define INST(T)                                                                                          \
    template void launch_p2m<T>(const int32_t*, int, const int32_t*, const int32_t*, int, const double*, \
                                const double*, const double*, const double*, int, void*, hipStream_t,    \
                                const GatherOut*);                                                       \
    template void launch_l2p<T>(const int32_t*, int, const int32_t*, const int32_t*, int, const double*, \
                                const double*, const double*, const void*, int, const double*,           \
                                const int32_t*, double*, double*, double*, hipStream_t,                  \
                                const long long*);
INST(double)
INST(float)
#undef INST

}  // namespace fmm
