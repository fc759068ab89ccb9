// subtree.hip -- the upward and downward passes of the far field (Sec. 2.1,
// Fig. 2.2) by subtrees, for trees whose problems have at least three levels.
// L is a problem's number of levels; problems of one tree may differ in it.
//
// Expansions are the scaled ones of expansions.hip (multipole a_k and local
// b_l in powers of (z - c)/rs); the shifts are the same exact re-centrings:
//     M2M  a^P_k = k! sum_{l<=k} (a^C_l rho^l / l!) (tau^(k-l) / (k-l)!)
//     L2L  b^C_l = (rho^l / l!) sum_{k>=l} (k! b^P_k) (tau^(k-l) / (k-l)!)
// with rho = rs_C / rs_P and tau = (c_C - c_P) / rs_P, computed in FP64 (the
// storage type T of the coefficients is float for mixed precision).  With the
// binomial coefficients written as factorials the inner sums are plain
// convolutions of two vectors in LDS: four FMAs and two 16-byte LDS reads per
// term, where the sums with a binomial table took six FP64 operations and
// three reads.  The tables tau^j / j! carry zeros in front, so that a block
// of 16 terms that crosses the triangle's edge needs no test.
//
// Upward: one workgroup per box R of level L-3 forms the multipoles of its 16
// leaves (P2M, with the gather of the strengths into tree order, which the near
// field reads; leaves with many points have it done before, LeafSet::fat), of its 4
// children and of R itself, all from LDS; then one workgroup per box of level a
// forms the levels a+D-1 .. a above the level a+D that the previous launch wrote,
// until level 1 (nothing reads the root's multipole).  Three launches at L = 9
// instead of one per level.
//
// Downward, direct form: the local expansion of a box is its own M2L sum plus
// the L2L image of its parent's complete expansion, hence plus the images,
// shifted directly into the box, of the M2L sums of all its ancestors (the
// shifts are exact, so the two forms agree up to rounding).  One workgroup per
// box R of level L-3 shifts the M2L sums of R's ancestors (levels 0 .. L-4)
// into R, one 16-lane group per ancestor, adds them to R's own, hands the
// result down to R's 4 children and 16 leaves in LDS, stores every leaf's
// complete expansion and evaluates it at the leaf's points (L2P), adding the
// near field and scattering to input order.  There is no L2L launch.
//
// Downward, staged form: every box's complete expansion is stored, rounded to
// the storage type level by level.  One workgroup per box A of level a hands
// A's complete expansion down D <= 3 levels (k_down_mid; from level 1 to level
// L-4), then the kernel above takes R's parent as its only
// ancestor and stores R and its children too.  It serves the evaluations that
// read the expansions of every level (points apart from the sources, the
// logarithmic constants), and the mixed-precision forms whose sums were always
// rounded at every level (problems of unlike depth, more than 32 terms).
#include <type_traits>

#include "fmm_internal.h"
#include "kernels_common.h"
#include "plan_extra.h"

namespace fmm {

// b^e, 0 <= e < 2^BITS, by repeated squaring, without branches
template <int BITS>
__device__ __forceinline__ double2 sub_cpow(double2 b, int e)
{
    double2 r = make_double2(1.0, 0.0);
#pragma unroll
    for (int i = 0; i < BITS; ++i) {
        const double2 v = cmul(r, b);
        r.x = (e >> i) & 1 ? v.x : r.x;
        r.y = (e >> i) & 1 ? v.y : r.y;
        if (i + 1 < BITS) b = cmul(b, b);
    }
    return r;
}
template <int BITS>
__device__ __forceinline__ double sub_rpow(double b, int e)
{
    double r = 1.0;
#pragma unroll
    for (int i = 0; i < BITS; ++i) {
        r = (e >> i) & 1 ? r * b : r;
        if (i + 1 < BITS) b *= b;
    }
    return r;
}
template <int P>
constexpr int kBits = P <= 16 ? 4 : P <= 32 ? 5 : 6;   // of an exponent below P

// id of box j of level l of the problem whose root is box pb
__device__ __forceinline__ int sub_box(int pb, int l, int64_t j) { return (int)(pb + level_base(l) + j); }

// the subtree of this workgroup: box j of level `lev` of the problem whose root
// is box pb, D levels; from the launch's list, or, when every problem has the
// same depth, computed (one dependent load less)
struct SubAt {
    int pb, lev, D;
    int64_t j;
    bool fat;            // P2M and L2P of its leaves are done elsewhere
};
__device__ __forceinline__ SubAt sub_at(const SubWork& w)
{
    if (w.list) {
        const int4 v = w.list[blockIdx.x];
        return SubAt{v.x, v.y, v.w & (kSubFat - 1), v.z, (v.w & kSubFat) != 0};
    }
    const int b = blockIdx.x / w.nper;
    return SubAt{(int)((int64_t)b * w.NB), w.lev, w.D & (kSubFat - 1), (int64_t)(blockIdx.x % w.nper),
                 (w.D & kSubFat) != 0};
}

// centre and scaling radius of a box
struct SubGeo {
    double x, y, rs;
};
__device__ __forceinline__ SubGeo sub_geo(const double* __restrict__ geom, int64_t box)
{
    return SubGeo{geom[4 * box], geom[4 * box + 1], geom[4 * box + 3]};
}
// tau and rho of the shift between a child and its parent
__device__ __forceinline__ double2 sub_tau(const SubGeo& par, const SubGeo& ch)
{
    const double inv = 1.0 / par.rs;
    return make_double2((ch.x - par.x) * inv, (ch.y - par.y) * inv);
}

// Factorials in the kernels' argument `fact`: fact[k] = k!, fact[64 + k] = 1/k!.
constexpr int kInvFact = 64;

// The table t_j = tau^j / j! of a shift, by a 16-lane group: t[16 + j], j < P
// (zero for j >= p), zeros in t[0 .. 15]
template <int P>
__device__ __forceinline__ void shift_table(double2* t, double2 tau, int p, int sl, const double (&ifac)[P / 16])
{
    t[sl] = make_double2(0.0, 0.0);
#pragma unroll
    for (int q = 0; q < P / 16; ++q) {
        const int j = sl + 16 * q;
        const double2 v = sub_cpow<kBits<P>>(tau, j);
        const double f = j < p ? ifac[q] : 0.0;
        t[16 + j] = make_double2(v.x * f, v.y * f);
    }
}

// acc += a b over real accumulators (xx - yy is the real part, xy + yx the imaginary)
struct CAcc {
    double xx = 0.0, yy = 0.0, xy = 0.0, yx = 0.0;
    __device__ __forceinline__ void add(double2 a, double2 b)
    {
        xx = fma(a.x, b.x, xx);
        yy = fma(a.y, b.y, yy);
        xy = fma(a.x, b.y, xy);
        yx = fma(a.y, b.x, yx);
    }
    __device__ __forceinline__ double2 value() const { return make_double2(xx - yy, xy + yx); }
};

// sum_{l <= k} a[l] t_(k-l), k = j + 16 q (blocks of 16 terms; the last one
// crosses l = k, where the table's zeros end the sum)
template <int P, int Q>
__device__ __forceinline__ double2 m2m_conv(const double2* a, const double2* t, int j)
{
    CAcc s;
#pragma unroll
    for (int l = 0; l < 16 * (Q + 1); ++l) s.add(a[l], t[16 + 16 * Q + j - l]);
    return s.value();
}
// sum_{k >= l} b[k] t_(k-l), l = j + 16 q (the first block crosses k = l); with
// STEP = 4 only the terms k = first mod 4 (a quarter of the sum per lane row)
template <int P, int Q, int STEP>
__device__ __forceinline__ double2 l2l_conv(const double2* b, const double2* t, int j, int first)
{
    CAcc s;
#pragma unroll
    for (int k = 16 * Q; k < P; k += STEP) s.add(b[k + first], t[16 + k + first - (j + 16 * Q)]);
    return s.value();
}
// f(q, integral constant q) for q = 0 .. N-1, unrolled
template <int N, class F>
__device__ __forceinline__ void for_q(F&& f)
{
    f(std::integral_constant<int, 0>{});
    if constexpr (N > 1) f(std::integral_constant<int, 1>{});
    if constexpr (N > 2) f(std::integral_constant<int, 2>{});
    if constexpr (N > 3) f(std::integral_constant<int, 3>{});
}

// store a coefficient in the storage type; the value as stored
template <class T>
__device__ __forceinline__ double2 store_coef(T* dst, int64_t box, int p, int k, double2 v)
{
    const T tx = (T)v.x, ty = (T)v.y;
    dst[2 * (box * coef_ld<T>(p) + k)] = tx;
    dst[2 * (box * coef_ld<T>(p) + k) + 1] = ty;
    return make_double2((double)tx, (double)ty);
}

// M2M into one parent by one wavefront: lane (c, j), c = lane/16 the child,
// forms child c's contribution to the coefficients k = j + 16 q of the parent
// from a[c][l] = a^C_l rho^l / l! and the table t[c]; the four contributions
// are added by two row exchanges.  Coefficient k is stored (row q of the
// lanes stores the block q); with `next`, scaled by f(k), also to LDS.
template <class T, int P, class F>
__device__ __forceinline__ void m2m_wave(int p, const double2 (*a)[P], const double2 (*t)[P + 16],
                                         const double (&fac)[P / 16], T* mp, int64_t par, double2* next, F&& f)
{
    const int lane = threadIdx.x & 63, c = lane >> 4, j = lane & 15;
    for_q<P / 16>([&](auto qc) {
        constexpr int q = decltype(qc)::value;
        const int k = j + 16 * q;
        double2 v = m2m_conv<P, q>(a[c], t[c], j);
        v.x += partner<16>(v.x);
        v.y += partner<16>(v.y);
        v.x += partner<32>(v.x);
        v.y += partner<32>(v.y);
        if (c == q) {
            double2 r = make_double2(0.0, 0.0);
            if (k < p) {
                r = store_coef<T>(mp, par, p, k, make_double2(fac[q] * v.x, fac[q] * v.y));
                if (next) {
                    const double s = f(k, q);
                    r.x *= s;
                    r.y *= s;
                }
            }
            if (next) next[k] = r;
        }
    });
}

// ------------------------------------------------------------------ upward

// One workgroup per box R of level L-3: P2M of its 16 leaves (16 lanes per
// leaf, a transposing butterfly), M2M into its 4 children (one wavefront each,
// from the wavefront's own four leaves) and into R (wavefront 0).  N = 2e5,
// L = 7, p = 16: 10 us (12.5 us with a binomial table); p = 39, N = 1e5: 14 us,
// where two P2M and two M2M launches took 40 us.  GATHER: the strengths come in tree
// order (None), or through the permutation, and are put into tree order here (Store)
// or elsewhere (Read).
constexpr int kGatherNone = 0, kGatherStore = 1, kGatherRead = 2;
template <class T, int P, int GATHER>
__global__ void __launch_bounds__(256)
k_up_leaf(SubWork work, const int32_t* __restrict__ bstart, const int32_t* __restrict__ bcount,
          const double* __restrict__ geom, const double* __restrict__ X, const double* __restrict__ Y,
          const double2* __restrict__ mt, int p, T* mp, const double* __restrict__ fact, GatherOut go)
{
    constexpr int V = 2 * P, KP = P / 16;
    __shared__ double2 sco[16][P];        // the leaves' coefficients (as stored) times rho^l / l!
    __shared__ double2 st_[16][P + 16];   // their shift tables
    __shared__ double2 spar[4][P];        // the same of the children of R
    __shared__ double2 stp[4][P + 16];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int gl = threadIdx.x >> 4, sl = threadIdx.x & 15;
    const SubAt at = sub_at(work);
    const int R = sub_box(at.pb, at.lev, at.j);
    const int leaf = sub_box(at.pb, at.lev + 2, 16 * at.j + gl);
    const int cw = sub_box(at.pb, at.lev + 1, 4 * at.j + w);
    const int st = bstart[leaf], n = bcount[leaf];
    const SubGeo gf = sub_geo(geom, leaf), gc = sub_geo(geom, cw), gR = sub_geo(geom, R);
    const int base = treduce_base<V, 16>(sl) >> 1;   // the coefficients base .. base + KP - 1 end in this lane
    double fac[KP], ifac[KP], ifb[KP];
#pragma unroll
    for (int q = 0; q < KP; ++q) {
        fac[q] = fact[sl + 16 * q];
        ifac[q] = fact[kInvFact + sl + 16 * q];
        ifb[q] = fact[kInvFact + base + q];
    }
    const double inv = 1.0 / gf.rs;
    double v[V];
#pragma unroll
    for (int i = 0; i < V; ++i) v[i] = 0.0;
    for (int j = at.fat ? n : sl; j < n; j += 16) {
        const int i = st + j;
        double2 z, t;
        if constexpr (GATHER != kGatherNone) {
            const double2 mm = go.m[go.perm[i]];
            const double x = X[i], y = Y[i];
            if constexpr (GATHER == kGatherStore) go.mtree[i] = mm;
            z = make_double2((x - gf.x) * inv, (y - gf.y) * inv);
            t = mm;
        } else {
            z = make_double2((X[i] - gf.x) * inv, (Y[i] - gf.y) * inv);
            t = mt[i];
        }
#pragma unroll
        for (int k = 0; k < P; ++k) {
            v[2 * k] += t.x;
            v[2 * k + 1] += t.y;
            if (k + 1 < P) t = cmul(t, z);
        }
    }
    treduce<V, 16>(v, lane);
    const double rl = gf.rs / gc.rs;
#pragma unroll
    for (int i = 0; i < KP; ++i) {
        const int k = base + i;
        double2 c = make_double2(0.0, 0.0);
        if (k < p) {
            if (at.fat) {
                const T* a = mp + 2 * ((int64_t)leaf * coef_ld<T>(p) + k);
                c = make_double2((double)a[0], (double)a[1]);
            } else {
                c = store_coef<T>(mp, leaf, p, k, make_double2(v[2 * i], v[2 * i + 1]));
            }
            const double s = sub_rpow<kBits<P>>(rl, k) * ifb[i];
            c.x *= s;
            c.y *= s;
        }
        sco[gl][k] = c;
    }
    shift_table<P>(st_[gl], sub_tau(gc, gf), p, sl, ifac);
    if ((lane >> 4) == 0) shift_table<P>(stp[w], sub_tau(gR, gc), p, sl, ifac);
    wave_sync();   // the four leaves of a wavefront are its own lanes'
    // the children of R: wavefront w forms child w from leaves 4w .. 4w+3
    const double rc = gc.rs / gR.rs;
    m2m_wave<T, P>(p, sco + 4 * w, st_ + 4 * w, fac, mp, cw, spar[w],
                   [&](int k, int q) { return sub_rpow<kBits<P>>(rc, k) * ifac[q]; });
    __syncthreads();
    if (w == 0) m2m_wave<T, P>(p, spar, stp, fac, mp, R, nullptr, [](int, int) { return 0.0; });
}

// The geometry and the shift tables of the boxes under A, levels a .. a+D
// (slot s = (4^d - 1)/3 + i holds box i of level a+d; slots 1 .. are the
// children), by NT threads: every geometry record loaded once, the tables by
// 16-lane groups.
template <int NS>
struct SubBoxes {
    double g[NS][3];
};
template <int NT, int NS>
__device__ __forceinline__ void sub_boxes(SubBoxes<NS>& sg, const SubAt& at, const double* __restrict__ geom, int ngeo)
{
    const int s = threadIdx.x;
    if (s < ngeo) {
        int d = 0, base = 0;
        while (s >= base + (1 << (2 * d))) {
            base += 1 << (2 * d);
            ++d;
        }
        const SubGeo g = sub_geo(geom, sub_box(at.pb, at.lev + d, (at.j << (2 * d)) + (s - base)));
        sg.g[s][0] = g.x;
        sg.g[s][1] = g.y;
        sg.g[s][2] = g.rs;
    }
}
template <int NS>
__device__ __forceinline__ SubGeo sub_slot(const SubBoxes<NS>& sg, int s)
{
    return SubGeo{sg.g[s][0], sg.g[s][1], sg.g[s][2]};
}

// Levels of a subtree launch and its workgroup: up to three levels and 16
// wavefronts (a wavefront per parent of the widest step) for p <= 32, two
// levels and four wavefronts for more terms (their tables take the LDS).
template <int P>
constexpr int kSubD = P <= 32 ? kSubLevels : kSubLevelsHigh;
template <int P>
constexpr int kSubThreads = P <= 32 ? 1024 : 256;
template <int P>
constexpr int kSubSlots = ((4 << (2 * kSubD<P>)) - 1) / 3;      // boxes under A, A itself first

// One workgroup per box A of level a: the multipoles of levels a+D-1 .. a of
// A's subtree from those of level a+D.  A chain of D dependent steps on few
// workgroups (64 at L = 9): latency is all of it, so the geometry, the shift
// tables and the scale factors of every box are formed first, all at once,
// and a step is a convolution, two row exchanges and a store; 16 wavefronts
// take the 16 parents of the widest step together.  Both launches at N = 1e5,
// L = 7, p = 16: 7 us (21 us with four wavefronts, and powers and divisions
// formed in every step); p = 39: 34 us beside the near field (63 us).
template <class T, int P>
__global__ void __launch_bounds__(kSubThreads<P>)
k_up_mid(SubWork work, const double* __restrict__ geom, int p, T* mp, const double* __restrict__ fact)
{
    constexpr int NT = kSubThreads<P>, NS = kSubSlots<P>, KP = P / 16, NG = NT / 16;
    constexpr int NIN = 1 << (2 * kSubD<P>);
    __shared__ SubBoxes<NS> sg;
    __shared__ double2 tab[NS][P + 16];
    __shared__ double sf[NS][P];          // rho^k / k! of every child slot
    __shared__ double2 sc0[NIN][P], sc1[NIN / 4][P];
    const int w = threadIdx.x >> 6, gl = threadIdx.x >> 4, sl = threadIdx.x & 15;
    const SubAt at = sub_at(work);
    const int a = at.lev, D = at.D;
    const int ngeo = ((4 << (2 * D)) - 1) / 3, nin = 1 << (2 * D);
    double fac[KP], ifac[KP];
#pragma unroll
    for (int q = 0; q < KP; ++q) {
        fac[q] = fact[sl + 16 * q];
        ifac[q] = fact[kInvFact + sl + 16 * q];
    }
    // level a+D, a 16-lane group per box, all loads in flight before the first use
    constexpr int R = (NIN + NG - 1) / NG;
    double2 v[R][KP];
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int q = 0; q < KP; ++q) {
            const int64_t box = sub_box(at.pb, a + D, (at.j << (2 * D)) + min(gl + NG * r, nin - 1));
            const int k = min(sl + 16 * q, p - 1);
            v[r][q] = make_double2((double)mp[2 * (box * coef_ld<T>(p) + k)], (double)mp[2 * (box * coef_ld<T>(p) + k) + 1]);
        }
    sub_boxes<NT>(sg, at, geom, ngeo);
    __syncthreads();
    for (int s = 1 + gl; s < ngeo; s += NG) {
        const SubGeo gc = sub_slot(sg, s), gp = sub_slot(sg, (s - 1) >> 2);
        shift_table<P>(tab[s], sub_tau(gp, gc), p, sl, ifac);
        const double rho = gc.rs / gp.rs;
#pragma unroll
        for (int q = 0; q < KP; ++q) sf[s][sl + 16 * q] = sub_rpow<kBits<P>>(rho, sl + 16 * q) * ifac[q];
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int q = 0; q < KP; ++q) {
            const int c = gl + NG * r, k = sl + 16 * q;
            if (c < nin) {
                const double s = k < p ? sf[ngeo - nin + c][k] : 0.0;
                sc0[c][k] = make_double2(s * v[r][q].x, s * v[r][q].y);
            }
        }
    __syncthreads();
    double2 (*cur)[P] = sc0;
    double2 (*nxt)[P] = sc1;
    for (int d = D - 1; d >= 0; --d) {
        const int np = 1 << (2 * d), s0 = ((1 << (2 * d)) - 1) / 3;   // parents at level a+d, the first one's slot
        for (int q = w; q < np; q += NT / 64) {
            const int par = sub_box(at.pb, a + d, (at.j << (2 * d)) + q);
            const double* f = sf[s0 + q];
            m2m_wave<T, P>(p, cur + 4 * q, tab + (4 * (s0 + q) + 1), fac, mp, par, d > 0 ? nxt[q] : nullptr,
                           [&](int k, int) { return f[k]; });
        }
        __syncthreads();
        double2 (*tmp)[P] = cur;
        cur = nxt;
        nxt = tmp;
    }
}

// ---------------------------------------------------------------- downward

// One workgroup per box A of level a, whose complete expansion is stored: the
// complete expansions of the D levels below A, every one its own M2L sum plus
// its parent's image, rounded to T as it is stored.  Latency is all of it, as
// in k_up_mid: loads and tables first, then a 16-lane group per child.  One
// launch of 5 us at L = 7, p = 16, where a launch per level took 24 us.
template <class T, int P>
__global__ void __launch_bounds__(kSubThreads<P>)
k_down_mid(SubWork work, const double* __restrict__ geom, int p, T* loc, const double* __restrict__ fact,
           const long long* __restrict__ guard)
{
    if (guard != nullptr && *guard != 0) return;   // lists flagged: this launch is void
    using T2 = typename Vec2<T>::type;
    constexpr int NT = kSubThreads<P>, NS = kSubSlots<P>, KP = P / 16, NG = NT / 16, DM = kSubD<P>;
    __shared__ SubBoxes<NS> sg;
    __shared__ double2 tab[NS][P + 16];
    __shared__ double2 sp[2][1 << (2 * (DM - 1))][P];   // k! b_k of the parents of a step, in turn
    const int gl = threadIdx.x >> 4, sl = threadIdx.x & 15;
    const SubAt at = sub_at(work);
    const int a = at.lev, D = at.D;
    const T2* lo = reinterpret_cast<const T2*>(loc);
    const int ngeo = ((4 << (2 * D)) - 1) / 3;
    double fac[KP], ifac[KP];
#pragma unroll
    for (int q = 0; q < KP; ++q) {
        fac[q] = fact[sl + 16 * q];
        ifac[q] = fact[kInvFact + sl + 16 * q];
    }
    // A's expansion, and the M2L sums of the child this group takes in every
    // step (indices clamped into the subtree)
    T2 ca[KP], cs[DM][KP];
#pragma unroll
    for (int q = 0; q < KP; ++q) {
        const int k = min(sl + 16 * q, p - 1);
        ca[q] = lo[(int64_t)sub_box(at.pb, a, at.j) * coef_ld<T>(p) + k];
#pragma unroll
        for (int d = 1; d <= DM; ++d) {
            const int dd = min(d, D);
            cs[d - 1][q] = lo[(int64_t)sub_box(at.pb, a + dd, (at.j << (2 * dd)) + min(gl, (1 << (2 * dd)) - 1)) * coef_ld<T>(p) + k];
        }
    }
    sub_boxes<NT>(sg, at, geom, ngeo);
    __syncthreads();
    for (int s = 1 + gl; s < ngeo; s += NG)
        shift_table<P>(tab[s], sub_tau(sub_slot(sg, (s - 1) >> 2), sub_slot(sg, s)), p, sl, ifac);
    if (gl == 0)
#pragma unroll
        for (int q = 0; q < KP; ++q) {
            const double f = sl + 16 * q < p ? fac[q] : 0.0;
            sp[0][0][sl + 16 * q] = make_double2(f * (double)ca[q].x, f * (double)ca[q].y);
        }
    __syncthreads();
    static_assert((1 << (2 * DM)) <= NG, "a group per child of the widest step");
#pragma unroll
    for (int d = 1; d <= DM; ++d) {
        if (d > D) break;               // uniform
        if (gl < 1 << (2 * d)) {
            const int s = ((1 << (2 * d)) - 1) / 3 + gl;
            const double rho = sg.g[s][2] / sg.g[(s - 1) >> 2][2];
            const int64_t box = sub_box(at.pb, a + d, (at.j << (2 * d)) + gl);
            for_q<KP>([&](auto qc) {
                constexpr int q = decltype(qc)::value;
                const int l = sl + 16 * q;
                const double2 v = l2l_conv<P, q, 1>(sp[(d - 1) & 1][gl >> 2], tab[s], sl, 0);
                double2 r = make_double2(0.0, 0.0);
                if (l < p) {
                    const double f = sub_rpow<kBits<P>>(rho, l) * ifac[q];
                    r = store_coef<T>(loc, box, p, l, make_double2(fma(f, v.x, (double)cs[d - 1][q].x),
                                                                  fma(f, v.y, (double)cs[d - 1][q].y)));
                }
                if (d < DM) sp[d & 1][gl][l] = make_double2(fac[q] * r.x, fac[q] * r.y);
            });
        }
        __syncthreads();
    }
}

// One workgroup per box R of level L-3.  See the file header.  N = 1e6, L = 9,
// p = 13: 35 us (38 us with a binomial table), HBM and latency: 80 MB in 35 us;
// N = 1e5, L = 7, p = 39: 13 us, where four L2L launches and L2P took 83 us.
// Every global load that does not depend on a computed value (the geometry
// and the M2L sums of R, of its ancestors, of its children and of the leaf
// of each 16-lane group, the leaf's first 32 points with their near field)
// is issued at the start, so the workgroup waits for memory twice (the
// points' loads need the leaf's start) instead of once per phase.
// STAGED: the only ancestor is R's parent, whose complete expansion is stored;
// R and its children are stored complete as well, every level rounded to T.
// EVAL: L2P at the points; EVAL 2: with the derivative (d/dz = (1/rs) d/dw,
// Horner in w), the near field's four sums per point in nearf.
template <class T, int P, bool STAGED, int EVAL>
__global__ void __launch_bounds__(256)
k_down_leaf(SubWork work, const int32_t* __restrict__ bstart, const int32_t* __restrict__ bcount,
            const double* __restrict__ geom, const double* __restrict__ X, const double* __restrict__ Y, T* loc,
            int p, const double2* __restrict__ nearf, const int32_t* __restrict__ perm, double2* phi,
            double2* phi_near, double2* phi_far, double2* dphi, const long long* __restrict__ guard,
            const double* __restrict__ fact)
{
    if (guard != nullptr && *guard != 0) return;   // lists flagged: this launch is void
    using T2 = typename Vec2<T>::type;
    constexpr int KP = P / 16;          // coefficients per lane of a 16-lane group
    constexpr int NPT = 2;              // points per lane loaded ahead (a leaf's first 32)
    __shared__ double2 sanc[16][P];     // k! b_k of the ancestors' M2L sums, then the leaves' expansions
    __shared__ double2 stab[16][P + 16];   // a shift table per 16-lane group
    __shared__ double2 spart[16][P];    // the ancestors' images in R
    __shared__ double2 sR[P];           // k! times R's complete expansion
    __shared__ double2 sC[4][P];        // the same of the children
    const int gl = threadIdx.x >> 4, sl = threadIdx.x & 15, w = threadIdx.x >> 6;
    const SubAt at = sub_at(work);
    const int64_t jR = at.j;
    const int lR = at.lev;
    const int R = sub_box(at.pb, lR, jR);
    const int leaf = sub_box(at.pb, lR + 2, 16 * jR + gl);
    const T2* lo = reinterpret_cast<const T2*>(loc);
    // ---- loads: every one unconditional, at an index clamped into range (a
    // load under a branch would be waited for where the branch ends); the
    // lanes that have no use for a value never read it
    const int st = EVAL ? bstart[leaf] : 0, n = EVAL ? bcount[leaf] : 0;
    const SubGeo gf = sub_geo(geom, leaf), gR = sub_geo(geom, R);
    // group gl < nanc: the ancestor of level gl (staged: the parent; the root
    // hands nothing down, it has no weak list)
    const int nanc = STAGED ? (lR >= 2 ? 1 : 0) : lR;
    const bool anc = gl < nanc;
    const int lA = STAGED ? lR - 1 : gl;
    const int A = anc ? sub_box(at.pb, lA, jR >> (2 * (lR - lA))) : R;
    const SubGeo ga = sub_geo(geom, A);
    // wavefront w: child w of R, the parent of its four leaves
    const int Cw = sub_box(at.pb, lR + 1, 4 * jR + w);
    const SubGeo gc = sub_geo(geom, Cw);
    T2 ca[KP], cR, cc[KP], cl[KP];
    double fac[KP], ifac[KP];
#pragma unroll
    for (int q = 0; q < KP; ++q) {
        const int k = min(sl + 16 * q, p - 1);
        ca[q] = lo[(int64_t)A * coef_ld<T>(p) + k];
        cc[q] = lo[(int64_t)Cw * coef_ld<T>(p) + k];
        cl[q] = lo[(int64_t)leaf * coef_ld<T>(p) + k];
        fac[q] = fact[sl + 16 * q];
        ifac[q] = fact[kInvFact + sl + 16 * q];
    }
    // thread l < P: R's own sum
    cR = lo[(int64_t)R * coef_ld<T>(p) + min((int)threadIdx.x, p - 1)];
    const double facR = fact[threadIdx.x & 63];
    // the leaf's first points (a lane past the leaf's end reads point 0)
    double px[NPT], py[NPT];
    double2 pn[NPT], pd[NPT];
    int po[NPT];
    if constexpr (EVAL != 0) {
#pragma unroll
        for (int q = 0; q < NPT; ++q) {
            const int j = sl + 16 * q;
            const int i = j < n ? st + j : 0;
            px[q] = X[i];
            py[q] = Y[i];
            pn[q] = nearf[EVAL == 2 ? 2 * (int64_t)i : i];
            if constexpr (EVAL == 2) pd[q] = nearf[2 * (int64_t)i + 1];
            po[q] = perm[i];
        }
    }
    // ---- the ancestors into R: group gl takes one
    if (anc) {
#pragma unroll
        for (int q = 0; q < KP; ++q) {
            const double f = sl + 16 * q < p ? fac[q] : 0.0;
            sanc[gl][sl + 16 * q] = make_double2(f * (double)ca[q].x, f * (double)ca[q].y);
        }
        shift_table<P>(stab[gl], sub_tau(ga, gR), p, sl, ifac);
        wave_sync();
        const double rho = gR.rs / ga.rs;
        for_q<KP>([&](auto qc) {
            constexpr int q = decltype(qc)::value;
            const double2 v = l2l_conv<P, q, 1>(sanc[gl], stab[gl], sl, 0);
            const double f = sub_rpow<kBits<P>>(rho, sl + 16 * q) * ifac[q];
            spart[gl][sl + 16 * q] = make_double2(f * v.x, f * v.y);
        });
    }
    __syncthreads();
    // R's complete expansion: its own M2L sum, then the ancestors top-down
    if ((int)threadIdx.x < P) {
        const int l = threadIdx.x;
        double2 acc = make_double2(0.0, 0.0);
        if (l < p) {
            acc = make_double2((double)cR.x, (double)cR.y);
            for (int a = 0; a < nanc; ++a) {
                acc.x += spart[a][l].x;
                acc.y += spart[a][l].y;
            }
            if constexpr (STAGED) acc = store_coef<T>(loc, R, p, l, acc);
        }
        sR[l] = make_double2(facR * acc.x, facR * acc.y);
    }
    // ---- R into its child w, by wavefront w: row r of the lanes takes the
    // terms k = r mod 4
    const int row = gl & 3;
    if (row == 0) shift_table<P>(stab[gl], sub_tau(gR, gc), p, sl, ifac);
    __syncthreads();
    {
        const double rho = gc.rs / gR.rs;
        for_q<KP>([&](auto qc) {
            constexpr int q = decltype(qc)::value;
            const int l = sl + 16 * q;
            double2 v = l2l_conv<P, q, 4>(sR, stab[4 * w], sl, row);
            v.x += partner<16>(v.x);
            v.y += partner<16>(v.y);
            v.x += partner<32>(v.x);
            v.y += partner<32>(v.y);
            if (row == q) {
                double2 r = make_double2(0.0, 0.0);
                if (l < p) {
                    const double f = sub_rpow<kBits<P>>(rho, l) * ifac[q];
                    r = make_double2(fma(f, v.x, (double)cc[q].x), fma(f, v.y, (double)cc[q].y));
                    if constexpr (STAGED) r = store_coef<T>(loc, Cw, p, l, r);
                }
                sC[w][l] = make_double2(fac[q] * r.x, fac[q] * r.y);
            }
        });
    }
    wave_sync();
    // ---- child w into its four leaves (wavefront w, group gl = leaf 4w + m):
    // the leaf's complete expansion, stored (the storage type) and kept for L2P
    shift_table<P>(stab[gl], sub_tau(gc, gf), p, sl, ifac);
    wave_sync();
    {
        const double rho = gf.rs / gc.rs;
        for_q<KP>([&](auto qc) {
            constexpr int q = decltype(qc)::value;
            const int l = sl + 16 * q;
            const double2 v = l2l_conv<P, q, 1>(sC[w], stab[gl], sl, 0);
            double2 r = make_double2(0.0, 0.0);
            if (l < p) {
                const double f = sub_rpow<kBits<P>>(rho, l) * ifac[q];
                r = store_coef<T>(loc, leaf, p, l, make_double2(fma(f, v.x, (double)cl[q].x),
                                                               fma(f, v.y, (double)cl[q].y)));
            }
            sanc[gl][l] = r;
        });
    }
    if (EVAL == 0 || at.fat) return;
    wave_sync();
    // ---- L2P at the leaf's points (Horner), plus the near field, to input order
    const double inv = 1.0 / gf.rs;
    const double2* co = sanc[gl];
    for (int j = sl, q = 0; j < n; j += 16, ++q) {
        const int i = st + j;
        double x, y, nfx, nfy, ndx = 0.0, ndy = 0.0;
        int o;
        if (q < NPT) {
            // (a run-time index into the arrays would move them to scratch)
            x = q == 0 ? px[0] : px[NPT - 1];
            y = q == 0 ? py[0] : py[NPT - 1];
            nfx = q == 0 ? pn[0].x : pn[NPT - 1].x;
            nfy = q == 0 ? pn[0].y : pn[NPT - 1].y;
            o = q == 0 ? po[0] : po[NPT - 1];
            if constexpr (EVAL == 2) {
                ndx = q == 0 ? pd[0].x : pd[NPT - 1].x;
                ndy = q == 0 ? pd[0].y : pd[NPT - 1].y;
            }
        } else {
            x = X[i]; y = Y[i];
            const double2 nf = nearf[EVAL == 2 ? 2 * (int64_t)i : i];
            nfx = nf.x; nfy = nf.y;
            if constexpr (EVAL == 2) {
                const double2 nd = nearf[2 * (int64_t)i + 1];
                ndx = nd.x; ndy = nd.y;
            }
            o = perm[i];
        }
        const double2 z = make_double2((x - gf.x) * inv, (y - gf.y) * inv);
        double2 acc = co[P - 1], der = make_double2(0.0, 0.0);
#pragma unroll
        for (int l = P - 2; l >= 0; --l) {
            if constexpr (EVAL == 2) {
                der = cmul(der, z);
                der.x += acc.x;
                der.y += acc.y;
            }
            acc = cmul(acc, z);
            acc.x += co[l].x;
            acc.y += co[l].y;
        }
        if (phi) phi[o] = make_double2(acc.x + nfx, acc.y + nfy);
        if constexpr (EVAL == 2) {
            dphi[o] = make_double2(der.x * inv - ndx, der.y * inv - ndy);
        } else {
            if (phi_near) phi_near[o] = make_double2(nfx, nfy);
            if (phi_far) phi_far[o] = acc;
        }
    }
}

// ---------------------------------------------------------------- launchers

static SubWork sub_work(const SubPlan& sp, const SubStep& st)
{
    if (sp.listed) return SubWork{sp.list.p + st.off, 0, 0, 0, 0};
    return SubWork{nullptr, st.lev, st.D, 1 << (2 * st.lev), nbox_levels(sp.L)};
}

#define SUB_BY_ORDER(CASE)                                                   \
    if (p <= 16) { CASE(16) }                                                \
    else if (p <= 32) { CASE(32) }                                           \
    else if (p <= 48) { CASE(48) }                                           \
    else if (p <= 64) { CASE(64) }                                           \
    else throw Error(FMM_EINVAL, "subtree passes need p <= 64");

template <class T>
void launch_up_leaves(const SubPlan& sp, const int32_t* bstart, const int32_t* bcount, const double* geom,
                      const double* X, const double* Y, const double* mt, int p, void* mp, const double* fact,
                      const GatherOut* go, hipStream_t s)
{
    if (sp.roots.n == 0) return;
    const GatherOut none{};
    const GatherOut& gg = go ? *go : none;
    const SubWork w = sub_work(sp, sp.roots);
    const unsigned grid = (unsigned)sp.roots.n;
#define UP_CASE(P_)                                                                                        \
    auto up = !go ? k_up_leaf<T, P_, kGatherNone>                                                          \
                  : go->mtree ? k_up_leaf<T, P_, kGatherStore> : k_up_leaf<T, P_, kGatherRead>;            \
    up<<<grid, 256, 0, s>>>(w, bstart, bcount, geom, X, Y, (const double2*)mt, p, (T*)mp, fact, gg);
    SUB_BY_ORDER(UP_CASE)
#undef UP_CASE
    check_launch("upward leaves");
}

// levels L-4 .. 1
template <class T>
void launch_up_mid(const SubPlan& sp, const double* geom, int p, void* mp, const double* fact, hipStream_t s)
{
    for (const SubStep& st : sp.up[p > 32]) {
        const SubWork w = sub_work(sp, st);
        const unsigned grid = (unsigned)st.n;
#define MID_CASE(P_) k_up_mid<T, P_><<<grid, kSubThreads<P_>, 0, s>>>(w, geom, p, (T*)mp, fact);
        SUB_BY_ORDER(MID_CASE)
#undef MID_CASE
        check_launch("upward subtrees");
    }
}

// the staged form's levels 2 .. L-4
template <class T>
void launch_down_mid(const SubPlan& sp, const double* geom, int p, void* loc, const double* fact,
                     const long long* guard, hipStream_t s)
{
    for (const SubStep& st : sp.down[p > 32]) {
        const SubWork w = sub_work(sp, st);
        const unsigned grid = (unsigned)st.n;
#define DMID_CASE(P_) k_down_mid<T, P_><<<grid, kSubThreads<P_>, 0, s>>>(w, geom, p, (T*)loc, fact, guard);
        SUB_BY_ORDER(DMID_CASE)
#undef DMID_CASE
        check_launch("downward subtrees");
    }
}

template <class T>
void launch_down_subtree(const SubPlan& sp, bool staged, const int32_t* bstart, const int32_t* bcount,
                         const double* geom, const double* X, const double* Y, void* loc, int p, const double* nearf,
                         const int32_t* perm, double* phi, double* phi_near, double* phi_far, double* dphi,
                         const long long* guard, const double* fact, hipStream_t s)
{
    if (sp.roots.n == 0) return;
    const SubWork w = sub_work(sp, sp.roots);
    const unsigned grid = (unsigned)sp.roots.n;
    const bool own = sp.all_fat && !sp.listed;      // L2P elsewhere for all
    const bool eval = !own && (phi != nullptr || phi_near != nullptr || phi_far != nullptr);
    if (own) dphi = nullptr;
#define DOWN_ARGS w, bstart, bcount, geom, X, Y, (T*)loc, p, (const double2*)nearf, perm, (double2*)phi, \
                  (double2*)phi_near, (double2*)phi_far, (double2*)dphi, guard, fact
#define DOWN_CASE(P_)                                                                    \
    if (staged && dphi) k_down_leaf<T, P_, true, 2><<<grid, 256, 0, s>>>(DOWN_ARGS);     \
    else if (dphi) k_down_leaf<T, P_, false, 2><<<grid, 256, 0, s>>>(DOWN_ARGS);         \
    else if (staged && eval) k_down_leaf<T, P_, true, 1><<<grid, 256, 0, s>>>(DOWN_ARGS); \
    else if (staged) k_down_leaf<T, P_, true, 0><<<grid, 256, 0, s>>>(DOWN_ARGS);        \
    else if (eval) k_down_leaf<T, P_, false, 1><<<grid, 256, 0, s>>>(DOWN_ARGS);         \
    else k_down_leaf<T, P_, false, 0><<<grid, 256, 0, s>>>(DOWN_ARGS);
    SUB_BY_ORDER(DOWN_CASE)
#undef DOWN_CASE
#undef DOWN_ARGS
    check_launch("downward leaves");
}

#define INST(T)                                                                                           \
    template void launch_up_leaves<T>(const SubPlan&, const int32_t*, const int32_t*, const double*,      \
                                      const double*, const double*, const double*, int, void*,            \
                                      const double*, const GatherOut*, hipStream_t);                      \
    template void launch_up_mid<T>(const SubPlan&, const double*, int, void*, const double*, hipStream_t); \
    template void launch_down_mid<T>(const SubPlan&, const double*, int, void*, const double*,            \
                                     const long long*, hipStream_t);                                      \
    template void launch_down_subtree<T>(const SubPlan&, bool, const int32_t*, const int32_t*,            \
                                         const double*, const double*, const double*, void*, int,         \
                                         const double*, const int32_t*, double*, double*, double*,        \
                                         double*, const long long*, const double*, hipStream_t);
INST(double)
INST(float)
#undef INST

}  // namespace fmm
