// log.hip -- the logarithmic potential (the paper's second kernel, Sec. 3.3;
// its multipole expansion a_0 log(z - z0) + sum_k a_k / (z - z0)^k, Sec. 2.1).
//
// For real strengths q the potential is u(z) = sum_j q_j log|z - z_j| =
// Re F(z), F(z) = sum_j q_j log(z - z_j), and F' is the harmonic field
// f(z) = sum_j q_j / (z - z_j) that the rest of the library expands.  So the
// far field reuses the harmonic expansions and adds one number per box:
//   multipole of S (harmonic coefficients A_k = sum q_j (z_j - c_S)^k):
//       F_S(z) = A_0 log(z - c_S) - sum_{k>=1} A_k / (k (z - c_S)^k);
//   local expansion of T: F(z) = c0_T + sum_{l>=1} (B_{l-1} / l) (z - c_T)^l,
//       B_l the harmonic local coefficients, c0_T the constant term;
//   M2L adds Re F_S(c_T) over the weak list of T to c0_T;
//   L2L adds the parent's whole Re F_P(c_T) (with its own constant);
//   L2P evaluates Re F at the points.
// Stored coefficients are scaled (multipole a_k = A_k / rs^k, local
// b_l = B_l rs^l), so with d = c_T - c_S and x_k = a_k (rs_S / d)^k:
//   Re F_S(c_T) = Re(A_0) log|d| - Re sum_{k>=1} x_k / k,
//   Re F_T(z)   = c0_T + rs_T Re sum_{l>=0} b_l w^(l+1) / (l + 1),  w = (z - c_T) / rs_T.
// The constants are formed in FP64 from the stored coefficients of either
// precision.
#include "fmm_internal.h"
#include "kernels_common.h"

namespace fmm {

__global__ void k_real_to_complex(int64_t n, const double* __restrict__ q, double2* __restrict__ m)
{
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i < n) m[i] = make_double2(q[i], 0.0);
}

// 1/k for the series of the constant terms (a multiplication in place of an
// FP64 division per term)
struct InvK {
    double v[kMaxP];
};
constexpr InvK make_inv_k()
{
    InvK t{};
    for (int k = 1; k < kMaxP; ++k) t.v[k] = 1.0 / k;
    return t;
}
__constant__ InvK kInvK = make_inv_k();

// The constant term of every box without its ancestors' part: M2L over its weak
// list, plus the parent's local series (complete: M2L and L2L done) at the box's
// centre.  The whole constant of a leaf is the sum over it and its ancestors
// (k_l2p_log).
//
// 32 lanes per box, lane e takes pairs e, e + 32, ... (on uniform inputs at
// theta = 0.5 most lists are shorter than 64, so one or two passes; clustered
// inputs reach lists of a few hundred entries, which take more passes of the
// same lanes); then lane l takes term l of the parent's series; the lanes' sums
// are added by a butterfly (a fixed order, so the result is reproducible).
// Bound by the gathers of the sources' coefficients: kLogRun of them are in
// flight per lane, so that a line is used while it is in the cache (one at a
// time: 45.6 us for 500,000 points on 8 levels, and 35.8 us of one launch per
// level for the parents' part; now 33.2 us for both).
constexpr int kLogRun = 8;

template <class T>
__global__ void __launch_bounds__(256)
k_log_constants(int nbox, const int32_t* __restrict__ w_beg, const int32_t* __restrict__ w_cnt,
                const int32_t* __restrict__ w_ids, const int32_t* __restrict__ parent,
                const double* __restrict__ geom, const T* __restrict__ mp, const T* __restrict__ loc, int p,
                double* __restrict__ c0)
{
    struct alignas(2 * sizeof(T)) C { T x, y; };
    const int g = blockIdx.x * 8 + (threadIdx.x >> 5), lane = threadIdx.x & 31;
    const bool live = g < nbox;   // every lane stays for the butterfly
    const int b = live ? w_beg[g] : 0, n = live ? w_cnt[g] : 0;
    const double cx = live ? geom[4 * (int64_t)g] : 0.0, cy = live ? geom[4 * (int64_t)g + 1] : 0.0;
    double acc = 0.0;
    for (int e = lane; e < n; e += 32) {
        const int S = w_ids[b + e];
        const double dx = cx - geom[4 * (int64_t)S], dy = cy - geom[4 * (int64_t)S + 1];
        const double rs = geom[4 * (int64_t)S + 3];
        const double r2 = dx * dx + dy * dy;   // > 0: weak pairs are well separated
        const C* a = (const C*)(mp + 2 * (int64_t)S * coef_ld<T>(p));
        const double a0 = (double)a[0].x;
        const double2 u = make_double2(rs * dx / r2, -rs * dy / r2);   // rs_S / d
        double2 pw = u;
        for (int k0 = 1; k0 < p; k0 += kLogRun) {
            C c[kLogRun];
#pragma unroll
            for (int q = 0; q < kLogRun; ++q) c[q] = a[min(k0 + q, p - 1)];
#pragma unroll
            for (int q = 0; q < kLogRun; ++q) {
                if (k0 + q < p) {
                    const double2 x = cmul(pw, make_double2((double)c[q].x, (double)c[q].y));
                    acc -= x.x * kInvK.v[k0 + q];
                    pw = cmul(pw, u);
                }
            }
        }
        acc += a0 * 0.5 * log(r2);
    }
    const int P = live ? parent[g] : -1;
    if (P >= 0) {
        const double rs = geom[4 * (int64_t)P + 3];
        if (rs > 0.0) {
            const double2 tau = make_double2((cx - geom[4 * (int64_t)P]) / rs, (cy - geom[4 * (int64_t)P + 1]) / rs);
            const C* bl = (const C*)(loc + 2 * (int64_t)P * coef_ld<T>(p));
            for (int l = lane; l < p; l += 32) {
                const C c = bl[l];
                // tau^(l+1) by squaring
                double2 pw = make_double2(1.0, 0.0), t = tau;
                for (int e = l + 1; e; e >>= 1) {
                    if (e & 1) pw = cmul(pw, t);
                    t = cmul(t, t);
                }
                acc += rs * cmul(make_double2((double)c.x, (double)c.y), pw).x / (double)(l + 1);
            }
        }
    }
#pragma unroll
    for (int o = 16; o > 0; o >>= 1) acc += __shfl_xor(acc, o, 32);
    if (live && lane == 0) c0[g] = acc;
}

// L2P of the logarithmic series at the points of every leaf, plus the near field,
// scattered to input order.  The constant term is summed over the leaf and its
// ancestors, root last.  G = 32 lanes per leaf, eight leaves per workgroup (leaves
// hold about 30 points), or above kLogWide points per leaf a workgroup per leaf:
// 32 lanes / 256, whole evaluation, us, mixed, p = 17: N = 150,000 on 5 levels (585
// points per leaf) 733 / 714, 20,000 on 4 (312) 136 / 128, 20,000 on 5 (78) 90 / 88,
// one leaf of 1000 at p = 40 108 / 75.
constexpr int kLogWide = 64;
template <class T, int G>
__global__ void __launch_bounds__(256)
k_l2p_log(const int32_t* __restrict__ leaves, int nleaf, const int32_t* __restrict__ bstart,
          const int32_t* __restrict__ bcount, const int32_t* __restrict__ parent, const double* __restrict__ geom,
          const double* __restrict__ X, const double* __restrict__ Y, const T* __restrict__ loc, int p,
          const double* __restrict__ c0, const double* __restrict__ near, const int32_t* __restrict__ perm,
          double* __restrict__ u)
{
    __shared__ double2 scf[256 / G][kMaxP];
    const int lane = threadIdx.x & (G - 1);
    const int li = blockIdx.x * (256 / G) + threadIdx.x / G;
    if (li >= nleaf) return;   // (a workgroup barrier below only where every workgroup has a leaf)
    double2* cf = scf[threadIdx.x / G];
    const int g = leaves[li];
    const int st = bstart[g], n = bcount[g];
    const double cx = geom[4 * (int64_t)g], cy = geom[4 * (int64_t)g + 1], rs = geom[4 * (int64_t)g + 3];
    const T* b = loc + 2 * (int64_t)g * coef_ld<T>(p);
    for (int l = lane; l < p; l += G)
        cf[l] = make_double2((double)b[2 * l] / (l + 1), (double)b[2 * l + 1] / (l + 1));
    double base = 0.0;
    for (int a = g; a >= 0; a = parent[a]) base += c0[a];
    if constexpr (G > 64) __syncthreads();
    else wave_sync();
    for (int i = lane; i < n; i += G) {
        const int pos = st + i;
        double v = base;
        if (rs > 0.0) {
            const double2 w = make_double2((X[pos] - cx) / rs, (Y[pos] - cy) / rs);
            double2 acc = make_double2(0.0, 0.0);
            for (int l = p - 1; l >= 0; --l) {
                acc = cmul(acc, w);
                acc.x += cf[l].x;
                acc.y += cf[l].y;
            }
            v += rs * cmul(acc, w).x;
        }
        u[perm[pos]] = v + near[2 * (int64_t)pos];
    }
}

void launch_real_to_complex(int64_t n, const double* q, double* m, hipStream_t s)
{
    if (n == 0) return;
    k_real_to_complex<<<(unsigned)((n + 255) / 256), 256, 0, s>>>(n, q, (double2*)m);
    check_launch("log strengths");
}

template <class T>
void launch_log_constants(int nbox, const int32_t* w_beg, const int32_t* w_cnt, const int32_t* w_ids,
                          const int32_t* parent, const double* geom, const void* mp, const void* loc, int p,
                          double* c0, hipStream_t s)
{
    if (nbox == 0) return;
    k_log_constants<T><<<(unsigned)((nbox + 7) / 8), 256, 0, s>>>(nbox, w_beg, w_cnt, w_ids, parent, geom,
                                                                  (const T*)mp, (const T*)loc, p, c0);
    check_launch("log constants");
}

template <class T>
void launch_l2p_log(const int32_t* leaves, int nleaf, int64_t n, const int32_t* bstart, const int32_t* bcount,
                    const int32_t* parent, const double* geom, const double* X, const double* Y, const void* loc,
                    int p, const double* c0, const double* near, const int32_t* perm, double* u, hipStream_t s)
{
    if (nleaf == 0) return;
    const bool wide = n > kLogWide * (int64_t)nleaf;
    auto l2p = wide ? k_l2p_log<T, 256> : k_l2p_log<T, 32>;
    l2p<<<(unsigned)(wide ? nleaf : (nleaf + 7) / 8), 256, 0, s>>>(leaves, nleaf, bstart, bcount, parent, geom, X, Y,
                                                                   (const T*)loc, p, c0, near, perm, u);
    check_launch("log l2p");
}

#define LOG_INSTANCE(T)                                                                                            \
    template void launch_log_constants<T>(int, const int32_t*, const int32_t*, const int32_t*, const int32_t*,     \
                                          const double*, const void*, const void*, int, double*, hipStream_t);     \
    template void launch_l2p_log<T>(const int32_t*, int, int64_t, const int32_t*, const int32_t*, const int32_t*,  \
                                    const double*, const double*, const double*, const void*, int, const double*,  \
                                    const double*, const int32_t*, double*, hipStream_t);
LOG_INSTANCE(float)
LOG_INSTANCE(double)
#undef LOG_INSTANCE

}  // namespace fmm
