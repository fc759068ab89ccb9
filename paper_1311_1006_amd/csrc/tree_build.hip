// tree_build.hip -- balanced median-split tree (Sec. 2.2) on gfx950.
//
// Every box is split in four by two successive binary splits.  A binary
// split cuts the longer side of the tight bounding box of the points being
// split (x when equal) and sends the floor(n/2) points smallest in
// (coordinate, input index) to the first half.  Because every split halves a
// count exactly, the size and position of every segment depend on N only;
// the host precomputes them and the device only decides membership.
//
// Device pipeline for one build (all problems of a batch at once):
//   init        copy positions into SoA buffers, bounding box of each root,
//               finiteness check (problems without a global stage: done by
//               the lds split itself);
//   per global stage s (segments larger than one workgroup's LDS):
//     hist1     256-bucket histogram of the split coordinate per segment
//               (buckets are equal-width in value over a range that holds
//               the segment, hence monotone in the coordinate): at stage 0
//               a kernel of its own over the root's bounding box; at later
//               stages the parent stage's partition has already counted its
//               children on both axes over the parent's bounding box;
//     hist2     if the bucket holding the median rank has too many points,
//               a second 2048-bucket histogram inside that bucket;
//     collect   each tile counts its points below the median's bucket and
//               appends the points of that bucket to a candidate list (an
//               exact single-workgroup radix select is the fallback for
//               pathological ties);
//     partition every tile takes the exact median (coordinate, index) from
//               the sorted candidates and its output offset, then does a
//               stable two-way partition into the next buffer, with the
//               bounding boxes of both halves (atomic min/max on
//               order-preserving integer images of the doubles) and the
//               children's histograms for the next stage;
//   lds split   each remaining segment (<= 4096 points) is finished by one
//               workgroup: the points are sorted once by (x, index) and once
//               by (y, index); every later split keeps both lists sorted by
//               a stable partition of the list of the other axis; the boxes of
//               the global stages are shared out over its workgroups;
//   geometry    box centre (bbox midpoint) and radius (half diagonal),
//               computed with explicitly rounded operations so that they are
//               bit-identical to a plain IEEE evaluation, and the scaling
//               radius (r, or the nearest ancestor's r when r = 0).
// The point order inside a segment after a stable partition is a function of
// the input order only, and the final order inside a leaf is sorted by
// (x, index), so the whole build is deterministic.
#include <algorithm>
#include <cstring>

#include "fmm_internal.h"
#include "kernels_common.h"
#include "lds_bucket.h"

// Box geometry, split axes and the theta-criterion must round every product
// and sum on its own (no fused multiply-add), like a plain IEEE evaluation.
#pragma clang fp contract(off)

namespace fmm {

// ------------------------------------------------------------------ schedule

static void seg_range(int64_t off, int64_t n, int s, int64_t j, int64_t* start, int64_t* cnt)
{
    int64_t st = off, c = n;
    for (int t = s - 1; t >= 0; --t) {
        int64_t h = c / 2;
        if ((j >> t) & 1) { st += h; c -= h; } else c = h;
    }
    *start = st; *cnt = c;
}

TreeSchedule* make_schedule(const std::vector<int64_t>& off, const std::vector<int>& L)
{
    auto* sc = new TreeSchedule();
    int nprob = (int)L.size();
    sc->nprob = nprob;
    sc->off = off;
    sc->L = L;
    sc->n = off[nprob];
    sc->pbox.resize(nprob);
    int64_t nb = 0, nl = 0;
    std::vector<int> g(nprob), S(nprob);
    std::vector<char> lds(nprob);
    int nstage = 0;
    for (int b = 0; b < nprob; ++b) {
        sc->pbox[b] = nb;
        nb += nbox_levels(L[b]);
        nl += int64_t(1) << (2 * (L[b] - 1));
        sc->max_levels = std::max(sc->max_levels, L[b]);
        int64_t n = off[b + 1] - off[b];
        S[b] = 2 * (L[b] - 1);
        int gb = 0;
        while (gb < S[b] && ((n + (int64_t(1) << gb) - 1) >> gb) > kLdsCap) ++gb;
        g[b] = gb;
        lds[b] = ((n + (int64_t(1) << gb) - 1) >> gb) <= kLdsCap;
        nstage = std::max(nstage, gb);
    }
    sc->nbox = nb;
    sc->nleaf = nl;
    sc->nstage = nstage;
    // key segments of stage s: problems with s <= g_b
    sc->nkeys.assign(nstage + 1, 0);
    sc->keys_off.assign(nstage + 2, 0);
    std::vector<std::vector<int64_t>> kbase(nstage + 1, std::vector<int64_t>(nprob, -1));
    for (int s = 0; s <= nstage; ++s) {
        int64_t c = 0;
        for (int b = 0; b < nprob; ++b)
            if (s <= g[b]) { kbase[s][b] = c; c += int64_t(1) << s; }
        sc->nkeys[s] = (int)c;
        sc->keys_off[s + 1] = sc->keys_off[s] + c;
    }
    sc->total_keys = sc->keys_off[nstage + 1];
    sc->segs.assign(sc->total_keys, SegInfo{});
    sc->tile_off.assign(nstage + 1, 0);
    sc->ntile.assign(nstage, 0);
    for (int s = 0; s <= nstage; ++s) {
        for (int b = 0; b < nprob; ++b) {
            if (s > g[b]) continue;
            int64_t n = off[b + 1] - off[b];
            for (int64_t j = 0; j < (int64_t(1) << s); ++j) {
                int64_t st, cnt;
                seg_range(off[b], n, s, j, &st, &cnt);
                int64_t gi = sc->keys_off[s] + kbase[s][b] + j;
                SegInfo& si = sc->segs[gi];
                si.start = (int32_t)st;
                si.count = (int32_t)cnt;
                si.box = (s % 2 == 0) ? (int32_t)(sc->pbox[b] + level_base(s / 2) + j) : -1;
                si.child = -1;
                si.tile0 = 0;
                si.ntile = 0;
                if (s < g[b]) {
                    si.child = (int32_t)(sc->keys_off[s + 1] + kbase[s + 1][b] + 2 * j);
                    si.tile0 = (int32_t)sc->tiles.size();
                    int32_t nt = (int32_t)((cnt + kTile - 1) / kTile);
                    si.ntile = nt;
                    for (int32_t t = 0; t < nt; ++t) {
                        TileInfo ti;
                        ti.seg = (int32_t)gi;
                        ti.start = (int32_t)(st + int64_t(t) * kTile);
                        ti.count = (int32_t)std::min<int64_t>(kTile, cnt - int64_t(t) * kTile);
                        ti.rank = t;
                        ti.seg_start = si.start;
                        ti.seg_count = si.count;
                        ti.tile0 = si.tile0;
                        ti.child = si.child;
                        ti.range = s == 0 ? (int32_t)gi : (int32_t)(sc->keys_off[s - 1] + kbase[s - 1][b] + (j >> 1));
                        ti.flags = (s + 1 < g[b]) ? 1 : 0;
                        sc->tiles.push_back(ti);
                    }
                }
            }
        }
        if (s < nstage) {
            sc->tile_off[s + 1] = (int64_t)sc->tiles.size();
            sc->ntile[s] = (int)(sc->tile_off[s + 1] - sc->tile_off[s]);
        }
    }
    sc->total_tile = (int64_t)sc->tiles.size();
    // init tiles: every problem's root (stage-0 key segment b' = kbase[0][b])
    sc->copy_tiles.clear();
    // geometry jobs from global-stage keys, lds work, copy tiles
    std::vector<std::vector<int64_t>> jbase(nstage + 1, std::vector<int64_t>(nprob, -1));
    for (int s = 0; s <= nstage; s += 2) {
        for (int b = 0; b < nprob; ++b) {
            bool from_keys = (s < g[b]) || (!lds[b] && s == g[b]);
            if (!from_keys) continue;
            jbase[s][b] = (int64_t)sc->geom.size();
            for (int64_t j = 0; j < (int64_t(1) << s); ++j) {
                GeomJob gj;
                gj.box = (int32_t)(sc->pbox[b] + level_base(s / 2) + j);
                gj.seg = (int32_t)(sc->keys_off[s] + kbase[s][b] + j);
                gj.parent = s ? (int32_t)(jbase[s - 2][b] + (j >> 2)) : -1;
                sc->geom.push_back(gj);
            }
        }
    }
    for (int b = 0; b < nprob; ++b) {
        int64_t n = off[b + 1] - off[b];
        if (lds[b]) {
            for (int64_t j = 0; j < (int64_t(1) << g[b]); ++j) {
                int64_t st, cnt;
                seg_range(off[b], n, g[b], j, &st, &cnt);
                LdsWork w;
                w.start = (int32_t)st; w.count = (int32_t)cnt;
                w.stages = S[b] - g[b]; w.stage0 = g[b]; w.j0 = (int32_t)j;
                w.boxbase = (int32_t)sc->pbox[b];
                const int up = (g[b] - 1) & ~1;   // the nearest box above: an even stage before g
                w.up = g[b] ? (int32_t)(jbase[up][b] + (j >> (g[b] - up))) : -1;
                w.pad = 0;
                sc->lds_max = std::max(sc->lds_max, w.count);
                sc->lds_stages = std::min(sc->lds_stages, w.stages);
                sc->lds.push_back(w);
            }
        } else {
            for (int64_t st = off[b]; st < off[b + 1]; st += kTile) {
                TileInfo ti;
                ti.seg = g[b] % 2;      // ping-pong buffer holding the final stage
                ti.start = (int32_t)st;
                ti.count = (int32_t)std::min<int64_t>(kTile, off[b + 1] - st);
                ti.rank = 0;
                ti.seg_start = ti.seg_count = ti.tile0 = ti.child = ti.range = ti.flags = 0;
                sc->copy_tiles.push_back(ti);
            }
        }
    }
    // per-box ranges, parents, levels, problems
    sc->box_start.assign(nb, 0); sc->box_count.assign(nb, 0);
    sc->box_parent.assign(nb, -1); sc->box_level.assign(nb, 0); sc->box_prob.assign(nb, 0);
    for (int b = 0; b < nprob; ++b) {
        int64_t n = off[b + 1] - off[b];
        for (int l = 0; l < L[b]; ++l) {
            for (int64_t j = 0; j < (int64_t(1) << (2 * l)); ++j) {
                int64_t st, cnt;
                seg_range(off[b], n, 2 * l, j, &st, &cnt);
                int64_t id = sc->pbox[b] + level_base(l) + j;
                sc->box_start[id] = (int32_t)st;
                sc->box_count[id] = (int32_t)cnt;
                sc->box_parent[id] = l ? (int32_t)(sc->pbox[b] + level_base(l - 1) + (j >> 2)) : -1;
                sc->box_level[id] = (int8_t)l;
                sc->box_prob[id] = b;
            }
        }
    }
    return sc;
}

void upload_schedule(TreeSchedule& sc, hipStream_t s)
{
    UploadPack u;
    u.add(sc.d_segs, sc.segs);
    u.add(sc.d_tiles, sc.tiles);
    u.add(sc.d_copy, sc.copy_tiles);
    u.add(sc.d_lds, sc.lds);
    u.add(sc.d_geom, sc.geom);
    u.add(sc.d_box_start, sc.box_start);
    u.add(sc.d_box_count, sc.box_count);
    u.add(sc.d_box_parent, sc.box_parent);
    u.add(sc.d_box_level, sc.box_level);
    u.add(sc.d_box_prob, sc.box_prob);
    u.add(sc.d_off, sc.off);
    u.add(sc.d_pbox, sc.pbox);
    u.upload(sc.block, s);
}

// ------------------------------------------------------------ device helpers

// order-preserving unsigned image of a double (+0 and -0 map to the same key)
__device__ __forceinline__ uint64_t okey(double x)
{
    x = x + 0.0;
    uint64_t u = (uint64_t)__double_as_longlong(x);
    return (u >> 63) ? ~u : (u | 0x8000000000000000ull);
}
__device__ __forceinline__ double okey_inv(uint64_t k)
{
    uint64_t u = (k >> 63) ? (k & 0x7fffffffffffffffull) : ~k;
    return __longlong_as_double((long long)u);
}

// geometry of a box from its bounding box, every operation rounded alone
__device__ __forceinline__ void box_geometry(double x0, double x1, double y0, double y1,
                                             double* bb, double* gm)
{
    bb[0] = x0; bb[1] = x1; bb[2] = y0; bb[3] = y1;
    gm[0] = (0.5 * (x0 + x1));
    gm[1] = (0.5 * (y0 + y1));
    double dx = (x1 - x0), dy = (y1 - y0);
    gm[2] = 0.5 * __dsqrt_rn((dx * dx) + (dy * dy));
}

// Every segment's bounding box is kept as kKeyCopies copies of four order
// keys (xmin, xmax, ymin, ymax) so that the workgroups updating it with
// atomics spread over several addresses; readers combine the copies.
constexpr int kKeyCopies = 32;
constexpr int kKeyWords = 4 * kKeyCopies;

__device__ __forceinline__ void read_keys(const uint64_t* k, double* bb)
{
    uint64_t a = k[0], b = k[1], c = k[2], d = k[3];
#pragma unroll
    for (int i = 1; i < kKeyCopies; ++i) {
        a = min(a, k[4 * i]); b = max(b, k[4 * i + 1]); c = min(c, k[4 * i + 2]); d = max(d, k[4 * i + 3]);
    }
    bb[0] = okey_inv(a); bb[1] = okey_inv(b); bb[2] = okey_inv(c); bb[3] = okey_inv(d);
}

// read_keys for a whole workgroup: lane c of wave 0 reads copy c and the
// wave combines them; every thread receives the result (one barrier)
static_assert(kKeyCopies == 32, "one key copy per lane of a half wavefront");
__device__ __forceinline__ void block_read_keys(const uint64_t* k, double* bb)
{
    // the copies as doubles (an untouched copy decodes to NaN, which the
    // minimum and maximum ignore, as the integer order placed it last)
    __shared__ double sk[4];
    if (threadIdx.x < 64) {
        const int c = threadIdx.x & (kKeyCopies - 1);
        const double a = half_wave_min(okey_inv(k[4 * c])), b = half_wave_max(okey_inv(k[4 * c + 1]));
        const double d = half_wave_min(okey_inv(k[4 * c + 2])), e = half_wave_max(okey_inv(k[4 * c + 3]));
        if (threadIdx.x == 0) { sk[0] = a; sk[1] = b; sk[2] = d; sk[3] = e; }
    }
    __syncthreads();
    bb[0] = sk[0]; bb[1] = sk[1]; bb[2] = sk[2]; bb[3] = sk[3];
}

// Two levels of bucket selection: the first histogram of a segment has
// kBuckets1 buckets over its extent, the second kBuckets2 buckets inside the
// first-level bucket that holds the median (when that bucket is large).
constexpr int kBuckets1 = 256;
constexpr int kBuckets2 = kBuckets;
// Every first-level histogram is kept as kHistCopies copies, updated by
// workgroups of different block index, so that the atomics of the many
// tiles of a large segment spread over several addresses; readers add them.
// Layout: ((segment * 2 + axis) * kHistCopies + copy) * kBuckets1 + bucket.
constexpr int kHistCopies = 8;
static_assert(kBuckets1 == kTileThreads, "one first-level bucket per thread");

template <class W>
__device__ __forceinline__ W* hist1_at(W* h, int64_t seg, int axis, int copy)
{
    return h + ((seg * 2 + axis) * kHistCopies + copy) * kBuckets1;
}

struct Bucketer {
    double lo, scale;
    int axis;
};

// first-level buckets of one axis over the bounding box bb (x0 x1 y0 y1)
__device__ __forceinline__ Bucketer axis_bucketer(const double* bb, int axis)
{
    Bucketer b;
    b.axis = axis;
    b.lo = axis ? bb[2] : bb[0];
    const double ext = axis ? (bb[3] - bb[2]) : (bb[1] - bb[0]);
    const double sc = ext > 0.0 ? (double)kBuckets1 / ext : 0.0;
    b.scale = (sc < 1e300) ? sc : 0.0;
    return b;
}

// read_keys of two segments for a whole workgroup (one barrier)
__device__ __forceinline__ void block_read_keys2(const uint64_t* k0, const uint64_t* k1, double* b0, double* b1)
{
    __shared__ double sk[8];
    if (threadIdx.x < 64) {
        const uint64_t* k = threadIdx.x < 32 ? k0 : k1;   // one segment per half wavefront
        const int c = threadIdx.x & (kKeyCopies - 1);
        const double a = half_wave_min(okey_inv(k[4 * c])), b = half_wave_max(okey_inv(k[4 * c + 1]));
        const double d = half_wave_min(okey_inv(k[4 * c + 2])), e = half_wave_max(okey_inv(k[4 * c + 3]));
        if ((threadIdx.x & 31) == 0) {
            const int o = threadIdx.x >> 3;   // 0 or 4
            sk[o] = a; sk[o + 1] = b; sk[o + 2] = d; sk[o + 3] = e;
        }
    }
    __syncthreads();
    for (int i = 0; i < 4; ++i) { b0[i] = sk[i]; b1[i] = sk[4 + i]; }
}

// The bucketer of a segment, computed by the whole workgroup (every thread
// of the block calls it, once per kernel): the split axis from the
// segment's own bounding box (the longer side), the bucket range from the
// bounding box of segment `range` along that axis (the parent, whose
// partition histograms the segment before its own box is complete).
__device__ __forceinline__ Bucketer make_bucketer(const uint64_t* keys, const uint64_t* range_keys,
                                                  double* own_bb = nullptr)
{
    double bb[4], rb[4];
    block_read_keys2(keys, range_keys, bb, rb);
    if (own_bb)
        for (int i = 0; i < 4; ++i) own_bb[i] = bb[i];
    const double w = (bb[1] - bb[0]), h = (bb[3] - bb[2]);
    return axis_bucketer(rb, (w >= h) ? 0 : 1);
}

__device__ __forceinline__ int bucket_of(const Bucketer& b, double c)
{
    double v = ((c - b.lo) * b.scale);
    int k = (int)fmin(fmax(v, 0.0), (double)(kBuckets1 - 1));
    return k;
}

__device__ __forceinline__ bool key_less(double c, int32_t i, double sc, int32_t si)
{
    return (c < sc) || (c == sc && i < si);
}

// block-wide exclusive scan of one value per thread (256 threads); returns
// the exclusive prefix, *total receives the block sum
template <int NT>
__device__ __forceinline__ int block_excl_scan(int v, int* sh, int* total)
{
    int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    const int x = wave_incl_scan(v);
    if (lane == 63) sh[wid] = x;
    __syncthreads();
    int base = 0, tot = 0;
#pragma unroll
    for (int w = 0; w < NT / 64; ++w) {
        int s = sh[w];
        if (w < wid) base += s;
        tot += s;
    }
    __syncthreads();
    *total = tot;
    return base + x - v;
}

// ------------------------------------------------------------------ kernels

// start of a build: the counter words zeroed; the bounding-box keys (every
// copy: kxmin kxmax kymin kymax) set to the empty box; the tree's error word
// cleared
__global__ void k_fill_start(uint32_t* words, int64_t nwords, uint64_t* k, int64_t nkeywords, uint32_t* err)
{
    if (blockIdx.x == 0 && threadIdx.x == 0) *err = 0u;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < nwords; i += stride) words[i] = 0u;
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < nkeywords; i += stride)
        k[i] = (i & 1) ? 0ull : ~0ull;
}

__device__ __forceinline__ void block_minmax_atomic(double x0, double x1, double y0, double y1,
                                                    uint64_t* keys, bool any)
{
    __shared__ double red[4][kTileThreads / 64];
    // over the wavefront as doubles (a thread without a point contributes
    // +-infinity), turned into order keys once per workgroup
    double a = wave_min(any ? x0 : INFINITY), b = wave_max(any ? x1 : -INFINITY);
    double c = wave_min(any ? y0 : INFINITY), d = wave_max(any ? y1 : -INFINITY);
    int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    if (lane == 0) { red[0][w] = a; red[1][w] = b; red[2][w] = c; red[3][w] = d; }
    __syncthreads();
    if (threadIdx.x == 0) {
        keys += 4 * (blockIdx.x & (kKeyCopies - 1));
        for (int i = 1; i < kTileThreads / 64; ++i) {
            a = fmin(a, red[0][i]); b = fmax(b, red[1][i]);
            c = fmin(c, red[2][i]); d = fmax(d, red[3][i]);
        }
        if (isfinite(a)) {
            atomicMin((unsigned long long*)&keys[0], (unsigned long long)okey(a));
            atomicMax((unsigned long long*)&keys[1], (unsigned long long)okey(b));
            atomicMin((unsigned long long*)&keys[2], (unsigned long long)okey(c));
            atomicMax((unsigned long long*)&keys[3], (unsigned long long)okey(d));
        }
    }
    __syncthreads();
}

// positions into SoA buffers, input order; root bounding boxes; finiteness
__global__ void __launch_bounds__(kTileThreads)
k_init(const double* __restrict__ z, const int64_t* __restrict__ poff, int nprob,
       double* X, double* Y, int32_t* I, uint64_t* keys0, uint32_t* err)
{
    constexpr int R = kTile / kTileThreads;
    int b = blockIdx.y;
    int64_t s0 = poff[b], s1 = poff[b + 1];
    int64_t t0 = s0 + (int64_t)blockIdx.x * kTile;
    if (t0 >= s1) return;   // uniform per block
    const int cnt = (int)min(s1 - t0, (int64_t)kTile);
    // every load of the tile issued before the first use
    double2 v[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int i = r * kTileThreads + threadIdx.x;
        v[r] = reinterpret_cast<const double2*>(z)[t0 + (i < cnt ? i : 0)];
    }
    double x0 = 1e308, x1 = -1e308, y0 = 1e308, y1 = -1e308;
    bool any = false, bad = false;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int i = r * kTileThreads + threadIdx.x;
        if (i < cnt) {
            // a non-finite position is flagged and built as (0, 0): the tree
            // stays a valid permutation, whatever runs before the flag is read
            if (!(isfinite(v[r].x) && isfinite(v[r].y))) {
                bad = true;
                v[r] = make_double2(0.0, 0.0);
            }
            X[t0 + i] = v[r].x; Y[t0 + i] = v[r].y; I[t0 + i] = (int32_t)(t0 + i);
            x0 = fmin(x0, v[r].x); x1 = fmax(x1, v[r].x); y0 = fmin(y0, v[r].y); y1 = fmax(y1, v[r].y);
            any = true;
        }
    }
    if (bad) atomicOr(err, 1u);
    // any is false only for threads without points; min/max skip them
    block_minmax_atomic(x0, x1, y0, y1, keys0 + kKeyWords * b, any);
}

// the split coordinate of the tile's points (element r * kTileThreads + tid)
// into registers, every load issued before the first use
template <int R>
__device__ __forceinline__ void load_tile(const double* __restrict__ C, const TileInfo& t, double (&v)[R])
{
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int i = r * kTileThreads + threadIdx.x;
        v[r] = C[t.start + (i < t.count ? i : 0)];
    }
}

__global__ void __launch_bounds__(kTileThreads)
k_hist1(const TileInfo* __restrict__ tiles, const double* __restrict__ X,
        const double* __restrict__ Y, const uint64_t* __restrict__ keys, uint32_t* hist1)
{
    constexpr int R = kTile / kTileThreads;
    __shared__ uint32_t h[kBuckets1];
    TileInfo t = tiles[blockIdx.x];
    Bucketer bk = make_bucketer(keys + kKeyWords * (int64_t)t.seg, keys + kKeyWords * (int64_t)t.range);
    double v[R];
    load_tile(bk.axis ? Y : X, t, v);
    for (int i = threadIdx.x; i < kBuckets1; i += kTileThreads) h[i] = 0;
    __syncthreads();
#pragma unroll
    for (int r = 0; r < R; ++r)
        if (r * kTileThreads + (int)threadIdx.x < t.count) atomicAdd(&h[bucket_of(bk, v[r])], 1u);
    __syncthreads();
    uint32_t* g = hist1_at(hist1, t.seg, bk.axis, blockIdx.x & (kHistCopies - 1));
    for (int i = threadIdx.x; i < kBuckets1; i += kTileThreads)
        if (h[i]) atomicAdd(&g[i], h[i]);
}

// find the bucket holding rank k among NB buckets: returns bucket, writes the
// rank inside it and the bucket's count.  hist in global memory, 256 threads.
// (find_bucket_loc: thread i holds the counts loc of buckets PER i .. PER i + PER - 1)
template <int PER>
__device__ int find_bucket_loc(const int (&loc)[PER], int k, int* rank_in, int* cnt_in, int* sh)
{
    int s = 0;
#pragma unroll
    for (int i = 0; i < PER; ++i) s += loc[i];
    int tot;
    int base = block_excl_scan<kTileThreads>(s, sh, &tot);
    // the thread whose range holds rank k writes the answer
    __shared__ int ans[3];
    int c = base;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        if (loc[i] > 0 && c <= k && k < c + loc[i]) {
            ans[0] = threadIdx.x * PER + i; ans[1] = k - c; ans[2] = loc[i];
        }
        c += loc[i];
    }
    __syncthreads();
    int b = ans[0];
    *rank_in = ans[1];
    *cnt_in = ans[2];
    __syncthreads();
    return b;
}
template <int NB>
__device__ int find_bucket(const uint32_t* hist, int k, int* rank_in, int* cnt_in, int* sh)
{
    static_assert(NB % kTileThreads == 0, "whole buckets per thread");
    constexpr int PER = NB / kTileThreads;
    int loc[PER];
#pragma unroll
    for (int i = 0; i < PER; ++i) loc[i] = (int)hist[threadIdx.x * PER + i];
    return find_bucket_loc<PER>(loc, k, rank_in, cnt_in, sh);
}

// a median bucket with more points than this is refined by a second histogram
// (a second pass over the segment's coordinates costs less than ranking a
// longer candidate list in every partition tile)
constexpr int kSubThreshold = 16;

struct SubBucketer {
    double lo, scale;
};
__device__ __forceinline__ SubBucketer make_sub(const Bucketer& bk, int b1)
{
    SubBucketer s;
    s.lo = bk.lo + (double)b1 / bk.scale;
    s.scale = (bk.scale * (double)kBuckets2);
    return s;
}
__device__ __forceinline__ int sub_of(const SubBucketer& s, double c)
{
    double v = ((c - s.lo) * s.scale);
    return (int)fmin(fmax(v, 0.0), (double)(kBuckets2 - 1));
}

// the first-level bucket of a segment's median (its rank inside the bucket
// and the bucket's population) and the segment's bucketer, found by hist2
// and read by collect (which then needs no bounding box of its own)
struct Level1 {
    int32_t b1, r1, c1, axis;
    double lo, scale;
    double bb[4];     // the segment's bounding box, for its partition
};

__global__ void __launch_bounds__(kTileThreads)
k_hist2(const TileInfo* __restrict__ tiles, const SegInfo* __restrict__ segs,
        const double* __restrict__ X, const double* __restrict__ Y,
        const uint64_t* __restrict__ keys, const uint32_t* __restrict__ hist1, uint32_t* hist2, Level1* lvl1)
{
    __shared__ uint32_t h[kBuckets2];
    __shared__ int sh[kTileThreads / 64];
    TileInfo t = tiles[blockIdx.x];
    // this thread's first-level bucket on both axes (the copies added),
    // loaded while the bounding boxes are read
    int hx = 0, hy = 0;
#pragma unroll
    for (int c = 0; c < kHistCopies; ++c) {
        hx += (int)hist1_at(hist1, t.seg, 0, c)[threadIdx.x];
        hy += (int)hist1_at(hist1, t.seg, 1, c)[threadIdx.x];
    }
    double bb[4];
    Bucketer bk = make_bucketer(keys + kKeyWords * (int64_t)t.seg, keys + kKeyWords * (int64_t)t.range, bb);
    int r1, c1;
    const int loc[1] = {bk.axis ? hy : hx};
    int b1 = find_bucket_loc<1>(loc, t.seg_count / 2, &r1, &c1, sh);
    if (t.rank == 0 && threadIdx.x == 0) {
        Level1 v;
        v.b1 = b1; v.r1 = r1; v.c1 = c1; v.axis = bk.axis;
        v.lo = bk.lo; v.scale = bk.scale;
        for (int i = 0; i < 4; ++i) v.bb[i] = bb[i];
        lvl1[t.seg] = v;
    }
    if (c1 <= kSubThreshold) return;   // uniform per block
    if (bk.scale == 0.0) return;  // all points in one bucket: the exact fallback handles it
    SubBucketer sb = make_sub(bk, b1);
    constexpr int R = kTile / kTileThreads;
    double v[R];
    load_tile(bk.axis ? Y : X, t, v);
    for (int i = threadIdx.x; i < kBuckets2; i += kTileThreads) h[i] = 0;
    __syncthreads();
#pragma unroll
    for (int r = 0; r < R; ++r)
        if (r * kTileThreads + (int)threadIdx.x < t.count && bucket_of(bk, v[r]) == b1)
            atomicAdd(&h[sub_of(sb, v[r])], 1u);
    __syncthreads();
    uint32_t* g = hist2 + (int64_t)t.seg * kBuckets2;
    for (int i = threadIdx.x; i < kBuckets2; i += kTileThreads)
        if (h[i]) atomicAdd(&g[i], h[i]);
}

struct Cand {
    double c;
    int32_t idx;
    int32_t tile;
};
struct Splitter {
    double c;
    int32_t idx;
    int32_t pad;
};
// the median's class of a segment as collect found it, for the partition
struct ClassInfo {
    int32_t rank;     // rank of the median within the class
    int32_t count;    // points in the class (the candidates, when <= kCandCap)
    int32_t axis;     // split axis: 0 x, 1 y
    int32_t pad;
};

// candidate class of a point: -1 below, 0 inside, 1 above
struct ClassRule {
    Bucketer bk;
    SubBucketer sb;
    int b1, b2;     // b2 < 0: one level
};
__device__ __forceinline__ int class_of(const ClassRule& r, double c)
{
    int b = bucket_of(r.bk, c);
    if (b != r.b1) return b < r.b1 ? -1 : 1;
    if (r.b2 < 0) return 0;
    int s = sub_of(r.sb, c);
    return s == r.b2 ? 0 : (s < r.b2 ? -1 : 1);
}

// exact selection of the k-th smallest (coordinate, index) of a segment by a
// most-significant-digit radix select over the 96-bit key, by one workgroup.
__device__ void exact_select(const double* C, const int32_t* I, int start, int count, int k,
                             Splitter* out)
{
    __shared__ uint32_t h[256];
    __shared__ int sh[kTileThreads / 64];
    __shared__ uint64_t pre_hi;
    __shared__ uint32_t pre_lo;
    __shared__ int rk;
    if (threadIdx.x == 0) { pre_hi = 0; pre_lo = 0; rk = k; }
    __syncthreads();
    for (int d = 0; d < 12; ++d) {
        for (int i = threadIdx.x; i < 256; i += kTileThreads) h[i] = 0;
        __syncthreads();
        uint64_t ph = pre_hi;
        uint32_t pl = pre_lo;
        for (int i = threadIdx.x; i < count; i += kTileThreads) {
            uint64_t kh = okey(C[start + i]);
            uint32_t kl = (uint32_t)I[start + i];
            bool match;
            int digit;
            if (d < 8) {
                int sh_ = 8 * (8 - d);   // bits above the current digit
                match = (sh_ >= 64) ? true : ((kh >> sh_) == (ph >> sh_));
                digit = (int)((kh >> (8 * (7 - d))) & 0xff);
            } else {
                int dd = d - 8;
                int sh_ = 8 * (4 - dd);
                match = (kh == ph) && ((sh_ >= 32) ? true : ((kl >> sh_) == (pl >> sh_)));
                digit = (int)((kl >> (8 * (3 - dd))) & 0xff);
            }
            if (match) atomicAdd(&h[digit], 1u);
        }
        __syncthreads();
        int v = (int)h[threadIdx.x];
        int tot;
        int base = block_excl_scan<kTileThreads>(v, sh, &tot);
        int r = rk;
        __syncthreads();
        if (v > 0 && base <= r && r < base + v) {
            if (d < 8) pre_hi |= (uint64_t)threadIdx.x << (8 * (7 - d));
            else pre_lo |= (uint32_t)threadIdx.x << (8 * (3 - (d - 8)));
            rk = r - base;
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) { out->c = okey_inv(pre_hi); out->idx = (int32_t)pre_lo; out->pad = 0; }
    __syncthreads();
}

// the candidate class (one or two histogram levels) of a segment's median,
// from the first-level bucket and the bucketer that hist2 recorded
__device__ __forceinline__ ClassRule median_class(const Level1* lvl1, const uint32_t* hist2, int seg, int* rank,
                                                  int* ccount, int* sh)
{
    ClassRule rule;
    const Level1 L1 = lvl1[seg];
    rule.bk.axis = L1.axis;
    rule.bk.lo = L1.lo;
    rule.bk.scale = L1.scale;
    const int r1 = L1.r1, c1 = L1.c1;
    rule.b1 = L1.b1;
    rule.b2 = -1;
    *rank = r1;
    *ccount = c1;
    if (c1 > kSubThreshold && rule.bk.scale != 0.0) {
        rule.sb = make_sub(rule.bk, rule.b1);
        int r2, c2;
        rule.b2 = find_bucket<kBuckets2>(hist2 + (int64_t)seg * kBuckets2, r1, &r2, &c2, sh);
        *rank = r2;
        *ccount = c2;
    }
    return rule;
}

// Segments whose median class holds more than kCandCap points (heavy ties):
// one workgroup finds the exact median (coordinate, index) of the segment
// by a radix select, and the output offset of every tile's lower half.
__device__ void pick_exact(int seg, const SegInfo& sg, const TileInfo* __restrict__ all_tiles,
                           const double* __restrict__ C, const int32_t* __restrict__ I, uint32_t* tile_below,
                           uint32_t* lo_base, Splitter* split, int* sh)
{
    __shared__ Splitter sp;
    const int k = sg.count / 2;
    exact_select(C, I, sg.start, sg.count, k, &sp);
    for (int tt = 0; tt < sg.ntile; ++tt) {
        TileInfo ti = all_tiles[sg.tile0 + tt];
        int cnt = 0;
        for (int i = threadIdx.x; i < ti.count; i += kTileThreads)
            cnt += key_less(C[ti.start + i], I[ti.start + i], sp.c, sp.idx);
        int tot2;
        block_excl_scan<kTileThreads>(cnt, sh, &tot2);
        if (threadIdx.x == 0) tile_below[sg.tile0 + tt] = (uint32_t)tot2;
    }
    __syncthreads();
    // exclusive scan of the per-tile lower counts into output offsets
    int run = 0;
    for (int c0 = 0; c0 < sg.ntile; c0 += kTileThreads) {
        int i = c0 + threadIdx.x;
        int v = (i < sg.ntile) ? (int)tile_below[sg.tile0 + i] : 0;
        int tot3;
        int ex = block_excl_scan<kTileThreads>(v, sh, &tot3);
        if (i < sg.ntile) lo_base[sg.tile0 + i] = (uint32_t)(run + ex);
        run += tot3;
    }
    if (threadIdx.x == 0) split[seg] = sp;
}

// every tile: count of points below the median's class, and the points of
// that class appended to the segment's candidate list.  When the class
// overflowed, the last tile of the segment to finish (per-segment counter
// seg_done) runs the exact selection for the whole segment; the partition
// tiles of other segments find the median themselves.
__global__ void __launch_bounds__(kTileThreads)
k_collect(const TileInfo* __restrict__ tiles, const TileInfo* __restrict__ all_tiles, const SegInfo* __restrict__ segs,
          const double* __restrict__ X, const double* __restrict__ Y, const int32_t* __restrict__ I,
          const Level1* __restrict__ lvl1, const uint32_t* __restrict__ hist2, Cand* cand, uint32_t* cand_cnt,
          uint32_t* tile_below, uint32_t* seg_done, ClassInfo* cinfo, uint32_t* lo_base, Splitter* split)
{
    __shared__ int sh[kTileThreads / 64];
    TileInfo t = tiles[blockIdx.x];
    constexpr int R = kTile / kTileThreads;
    int rank, ccount;
    ClassRule rule = median_class(lvl1, hist2, t.seg, &rank, &ccount, sh);
    const bool overflow = ccount > kCandCap;
    if (t.rank == 0 && threadIdx.x == 0) {
        ClassInfo ci;
        ci.rank = rank; ci.count = ccount; ci.axis = rule.bk.axis; ci.pad = 0;
        cinfo[t.seg] = ci;
    }
    double v[R];
    load_tile(rule.bk.axis ? Y : X, t, v);
    int below = 0;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int i = r * kTileThreads + threadIdx.x;
        if (i >= t.count) continue;
        int cl = class_of(rule, v[r]);
        below += (cl < 0);
        if (cl == 0 && !overflow) {
            uint32_t pos = atomicAdd(&cand_cnt[t.seg], 1u);
            if (pos < (uint32_t)kCandCap) {
                Cand cd; cd.c = v[r]; cd.idx = I[t.start + i]; cd.tile = t.rank;
                cand[(int64_t)t.seg * kCandCap + pos] = cd;
            }
        }
    }
    int tot;
    block_excl_scan<kTileThreads>(below, sh, &tot);
    if (threadIdx.x == 0) tile_below[t.tile0 + t.rank] = (uint32_t)tot;
    if (overflow) {   // uniform per block
        __shared__ bool last;
        __threadfence();   // this tile's count is visible before the tile is counted done
        __syncthreads();
        if (threadIdx.x == 0) last = atomicAdd(&seg_done[t.seg], 1u) + 1u == (uint32_t)segs[t.seg].ntile;
        __syncthreads();
        if (last) {   // every tile of the segment has written its count: overwrite them all
            __threadfence();
            pick_exact(t.seg, segs[t.seg], all_tiles, rule.bk.axis ? Y : X, I, tile_below, lo_base, split, sh);
        }
    }
}

// bounding boxes of both halves of a tile into the next stage's keys (one
// barrier for the two)
__device__ __forceinline__ void block_minmax2_atomic(const double (&l)[4], const double (&u)[4], bool anyl,
                                                     bool anyu, uint64_t* keys_lo, uint64_t* keys_hi)
{
    __shared__ double red[8][kTileThreads / 64];
    // minima and maxima over the wavefront as doubles (a lane without a
    // point contributes +-infinity), turned into order keys once per
    // workgroup
    double k[8];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const double inf = (q & 1) ? -INFINITY : INFINITY;
        k[q] = anyl ? l[q] : inf;
        k[4 + q] = anyu ? u[q] : inf;
    }
#pragma unroll
    for (int q = 0; q < 8; ++q) k[q] = (q & 1) ? wave_max(k[q]) : wave_min(k[q]);
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    if (lane == 0)
#pragma unroll
        for (int q = 0; q < 8; ++q) red[q][w] = k[q];
    __syncthreads();
    // thread q < 8 combines value q over the waves and updates one key
    if (threadIdx.x < 8) {
        const int q = threadIdx.x;
        double v = red[q][0];
        for (int i = 1; i < kTileThreads / 64; ++i) v = (q & 1) ? fmax(v, red[q][i]) : fmin(v, red[q][i]);
        uint64_t* kk = (q < 4 ? keys_lo : keys_hi) + 4 * (blockIdx.x & (kKeyCopies - 1)) + (q & 3);
        const bool empty = !isfinite(v);
        const uint64_t a = empty ? 0ull : okey(v);
        if (!empty) {
            if (q & 1) atomicMax((unsigned long long*)kk, (unsigned long long)a);
            else atomicMin((unsigned long long*)kk, (unsigned long long)a);
        }
    }
}

// The median (coordinate, index) of a segment from its candidate list (the
// points of the median's class), and the lower points of the tiles before
// tile `rank_t`: below-class counts of those tiles plus their candidates
// ranked below the median.  Every tile of the segment computes the same
// median.  Up to one candidate per thread, a candidate's rank is its count
// of smaller candidates; longer lists are sorted (bitonic, in LDS).
__device__ void tile_median(const Cand* __restrict__ cs, int n, int rank, const uint32_t* __restrict__ below,
                            int rank_t, Splitter* sp, int* lob, int* sh)
{
    __shared__ uint64_t skey[kCandCap];
    __shared__ uint32_t sidx[kCandCap];
    __shared__ uint32_t stile[kCandCap];
    __shared__ Splitter ssp;
    int P = n;
    if (n > kTileThreads) {
        P = 1;
        while (P < n) P <<= 1;
    }
    for (int i = threadIdx.x; i < P; i += kTileThreads) {
        if (i < n) {
            const Cand cd = cs[i];
            skey[i] = okey(cd.c);
            sidx[i] = (uint32_t)cd.idx;
            stile[i] = (uint32_t)cd.tile;
        } else {
            skey[i] = ~0ull; sidx[i] = 0xffffffffu; stile[i] = 0xffffffffu;
        }
    }
    int v = 0;
    for (int i = threadIdx.x; i < rank_t; i += kTileThreads) v += (int)below[i];
    __syncthreads();
    if (n <= kTileThreads) {
        const int i = threadIdx.x;
        if (i < n) {
            const uint64_t ki = skey[i];
            const uint32_t ii = sidx[i];
            int ri = 0;
            for (int j = 0; j < n; ++j) ri += (skey[j] < ki) | ((skey[j] == ki) & (sidx[j] < ii));
            if (ri == rank) { ssp.c = okey_inv(ki); ssp.idx = (int32_t)ii; ssp.pad = 0; }
            v += (ri < rank) & ((int)stile[i] < rank_t);
        }
    } else {
        for (int kk = 2; kk <= P; kk <<= 1)
            for (int j = kk >> 1; j > 0; j >>= 1) {
                for (int i = threadIdx.x; i < P / 2; i += kTileThreads) {
                    const int lo = ((i & ~(j - 1)) << 1) | (i & (j - 1));
                    const int hi = lo + j;
                    const bool asc = (lo & kk) == 0;
                    const bool less_hl = (skey[hi] < skey[lo]) || (skey[hi] == skey[lo] && sidx[hi] < sidx[lo]);
                    if (less_hl == asc) {
                        const uint64_t a = skey[lo]; skey[lo] = skey[hi]; skey[hi] = a;
                        const uint32_t b = sidx[lo]; sidx[lo] = sidx[hi]; sidx[hi] = b;
                        const uint32_t c = stile[lo]; stile[lo] = stile[hi]; stile[hi] = c;
                    }
                }
                __syncthreads();
            }
        if (threadIdx.x == 0) { ssp.c = okey_inv(skey[rank]); ssp.idx = (int32_t)sidx[rank]; ssp.pad = 0; }
        for (int i = threadIdx.x; i < rank; i += kTileThreads) v += ((int)stile[i] < rank_t);
    }
    int tot;
    block_excl_scan<kTileThreads>(v, sh, &tot);   // its barriers also publish ssp
    *lob = tot;
    *sp = ssp;
}

// Stable two-way partition of one tile.  Element i = r * kTileThreads + tid
// is lower if (coordinate, index) < splitter; its rank among the lower
// (upper) elements of the tile comes from per-wave ballots of every row,
// combined with one barrier.  The splitter and the tile's output offset come
// from tile_median, or from the exact selection (pick_exact, run by the last
// collect tile) for a segment whose class overflowed.
__global__ void __launch_bounds__(kTileThreads)
k_partition(const TileInfo* __restrict__ tiles, const SegInfo* __restrict__ segs,
            const double* __restrict__ X, const double* __restrict__ Y, const int32_t* __restrict__ I,
            double* X2, double* Y2, int32_t* I2, uint64_t* keys_next, const ClassInfo* __restrict__ cinfo,
            const Cand* __restrict__ cand, const uint32_t* __restrict__ tile_below,
            const Splitter* __restrict__ split, const uint32_t* __restrict__ lo_base, uint32_t* hist1,
            const Level1* __restrict__ lvl1)
{
    constexpr int R = kTile / kTileThreads;
    constexpr int NW = kTileThreads / 64;
    __shared__ int wcnt[R][NW];
    __shared__ int sh[NW];
    __shared__ uint32_t chist[4 * kBuckets1];   // the children's first-level histograms, (child, axis)
    const TileInfo t = tiles[blockIdx.x];
    const bool hist_children = (t.flags & 1) != 0;   // uniform per block
    const int k = t.seg_count / 2;
    const int toff = t.start - t.seg_start;
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    // the tile's points first: their loads overlap the median search
    double x[R], y[R];
    int32_t id[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int i = r * kTileThreads + threadIdx.x;
        const int ii = t.start + (i < t.count ? i : 0);
        x[r] = X[ii]; y[r] = Y[ii]; id[r] = I[ii];
    }
    // a child split by a later global stage is histogrammed here, on both
    // axes over this segment's bounding box (its split axis is not known yet)
    Bucketer cb[2];
    if (hist_children) {
        double bb[4];   // this segment's bounding box, as hist2 read it
        for (int i = 0; i < 4; ++i) bb[i] = lvl1[t.seg].bb[i];
        cb[0] = axis_bucketer(bb, 0);
        cb[1] = axis_bucketer(bb, 1);
        for (int i = threadIdx.x; i < 4 * kBuckets1; i += kTileThreads) chist[i] = 0u;
    }
    const ClassInfo ci = cinfo[t.seg];
    Splitter sp;
    int lob;
    if (ci.count > kCandCap) {
        sp = split[t.seg];
        lob = (int)lo_base[t.tile0 + t.rank];
    } else {
        tile_median(cand + (int64_t)t.seg * kCandCap, ci.count, ci.rank, tile_below + t.tile0, t.rank, &sp, &lob, sh);
    }
    const unsigned long long lt = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    int inwave[R];
    bool lower[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int i = r * kTileThreads + threadIdx.x;
        lower[r] = i < t.count && key_less(ci.axis ? y[r] : x[r], id[r], sp.c, sp.idx);
        const unsigned long long m = __ballot(lower[r]);
        inwave[r] = __popcll(m & lt);
        if (lane == 0) wcnt[r][wid] = __popcll(m);
    }
    __syncthreads();
    double l[4] = {1e308, -1e308, 1e308, -1e308}, u[4] = {1e308, -1e308, 1e308, -1e308};
    bool anyl = false, anyu = false;
    int before = 0;   // lower elements of the tile in earlier rows
#pragma unroll
    for (int r = 0; r < R; ++r) {
        int rowtot = 0, prev = 0;
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            const int c = wcnt[r][w];
            prev += (w < wid) ? c : 0;
            rowtot += c;
        }
        const int i = r * kTileThreads + threadIdx.x;
        if (i < t.count) {
            const int lb = before + prev + inwave[r];   // lower elements before i in the tile
            int dst;
            if (lower[r]) {
                dst = t.seg_start + lob + lb;
                l[0] = fmin(l[0], x[r]); l[1] = fmax(l[1], x[r]); l[2] = fmin(l[2], y[r]); l[3] = fmax(l[3], y[r]);
                anyl = true;
            } else {
                dst = t.seg_start + k + (toff - lob) + (i - lb);
                u[0] = fmin(u[0], x[r]); u[1] = fmax(u[1], x[r]); u[2] = fmin(u[2], y[r]); u[3] = fmax(u[3], y[r]);
                anyu = true;
            }
            if (dst >= t.seg_start && dst < t.seg_start + t.seg_count) { X2[dst] = x[r]; Y2[dst] = y[r]; I2[dst] = id[r]; }
            if (hist_children) {
                const int c = lower[r] ? 0 : 2;   // (child, axis) slot of axis 0
                atomicAdd(&chist[c * kBuckets1 + bucket_of(cb[0], x[r])], 1u);
                atomicAdd(&chist[(c + 1) * kBuckets1 + bucket_of(cb[1], y[r])], 1u);
            }
        }
        before += rowtot;
    }
    // its barrier also completes the histogram updates above
    block_minmax2_atomic(l, u, anyl, anyu, keys_next + kKeyWords * (int64_t)t.child,
                         keys_next + kKeyWords * ((int64_t)t.child + 1));
    if (hist_children) {   // slot c * 2 + axis: child t.child + c, one bucket per thread
        const int copy = blockIdx.x & (kHistCopies - 1);
#pragma unroll
        for (int sl = 0; sl < 4; ++sl) {
            const uint32_t v = chist[sl * kBuckets1 + threadIdx.x];
            if (v) atomicAdd(&hist1_at(hist1, (int64_t)t.child + (sl >> 1), sl & 1, copy)[threadIdx.x], v);
        }
    }
}

// The scaling radius that a box without extent takes over: r of the nearest
// ancestor that has one, 1 without; `job` is the nearest ancestor's
__device__ double ancestor_radius(const GeomJob* __restrict__ jobs, int job, const uint64_t* __restrict__ keys)
{
    while (job >= 0) {
        double kb[4], bb[4], gm[3];
        read_keys(keys + kKeyWords * (int64_t)jobs[job].seg, kb);
        box_geometry(kb[0], kb[1], kb[2], kb[3], bb, gm);
        if (gm[2] > 0.0) return gm[2];
        job = jobs[job].parent;
    }
    return 1.0;
}

// Geometry of the boxes [first, end) whose bounding box came from a global
// stage, by the calling workgroup: a half wavefront per box, one lane per copy
// of its keys.
__device__ void geom_from_keys(const GeomJob* __restrict__ jobs, int first, int end,
                               const uint64_t* __restrict__ keys, double* bbox, double* geom)
{
    const int half = (threadIdx.x >> 5) & 1, c = threadIdx.x & (kKeyCopies - 1);
    for (int j0 = first + 2 * (threadIdx.x >> 6); j0 < end; j0 += 2 * (blockDim.x >> 6)) {
        const GeomJob j = jobs[min(j0 + half, end - 1)];
        const uint64_t* k = keys + kKeyWords * (int64_t)j.seg;
        const double x0 = half_wave_min(okey_inv(k[4 * c])), x1 = half_wave_max(okey_inv(k[4 * c + 1]));
        const double y0 = half_wave_min(okey_inv(k[4 * c + 2])), y1 = half_wave_max(okey_inv(k[4 * c + 3]));
        if (c == 0 && j0 + half < end) {
            double bb[4], gm[3];
            box_geometry(x0, x1, y0, y1, bb, gm);
            for (int q = 0; q < 4; ++q) bbox[4 * (int64_t)j.box + q] = bb[q];
            for (int q = 0; q < 3; ++q) geom[4 * (int64_t)j.box + q] = gm[q];
            geom[4 * (int64_t)j.box + 3] = gm[2] > 0.0 ? gm[2] : ancestor_radius(jobs, j.parent, keys);
        }
    }
}

// of a layout without in-LDS work
__global__ void __launch_bounds__(256)
k_geom_keys(const GeomJob* __restrict__ jobs, int n, const uint64_t* __restrict__ keys, double* bbox, double* geom)
{
    const int first = 8 * blockIdx.x;
    geom_from_keys(jobs, first, min(n, first + 8), keys, bbox, geom);
}

__global__ void k_copy_final(const TileInfo* __restrict__ tiles, const double* XA, const double* YA,
                             const int32_t* IA, const double* XB, const double* YB, const int32_t* IB,
                             double* X, double* Y, int32_t* I)
{
    TileInfo t = tiles[blockIdx.x];
    const double* xs = t.seg ? XB : XA;
    const double* ys = t.seg ? YB : YA;
    const int32_t* is = t.seg ? IB : IA;
    for (int i = threadIdx.x; i < t.count; i += blockDim.x) {
        X[t.start + i] = xs[t.start + i]; Y[t.start + i] = ys[t.start + i]; I[t.start + i] = is[t.start + i];
    }
}

// ------------------------------------------------- in-LDS completion kernel
// Sorted lists LX (by x, index) and LY (by y, index) of local point ids; a
// split along an axis keeps that axis' list as is (its first floor(n/2)
// entries are the lower half) and stably partitions the other list.  Both
// lists hold every sub-segment at the same positions, so a thread owns
// positions [PER*tid, PER*tid + PER) of both and keeps the sub-segment of
// each of them (start, count, box) in registers.  posX/posY invert the
// lists: an element is in the lower half of its sub-segment iff its
// position in the split axis' list is below start + count/2.
constexpr int kLdsThreads = 1024;
constexpr int kLdsWaves = kLdsThreads / 64;

// PER positions (and buckets) per thread
template <int PER>
struct LdsSort {
    uint64_t key[PER * kLdsThreads];
    uint16_t id[PER * kLdsThreads];
};
template <int PER>
struct LdsPos {
    uint16_t posX[PER * kLdsThreads];
    uint16_t posY[PER * kLdsThreads];
};
template <int PER>
struct LdsBucket {
    uint32_t cnt[PER * kLdsThreads];      // bucket populations, then bucket ends
    uint64_t key[PER * kLdsThreads];      // order keys in bucket order
    uint16_t id[PER * kLdsThreads];       // local ids in bucket order (any order inside a bucket)
};
template <int PER>
union LdsUnion {
    LdsSort<PER> s;
    LdsPos<PER> q;
    LdsBucket<PER> b;
};

// (key, input index) order of two entries of the sort buffer; padding entries
// (key ~0, which no finite coordinate has) come last, in any order
__device__ __forceinline__ bool lds_less(uint64_t ka, uint16_t ia, uint64_t kb, uint16_t ib, const uint32_t* idxs)
{
    if (ka != kb) return ka < kb;
    return ka != ~0ull && idxs[ia] < idxs[ib];
}

// Sort of the entries of S (n of them, padding behind) by (key, input index): a
// merge sort, thread t owning positions PER t .. PER t + PER - 1.  The thread's
// entries are sorted in registers; then the runs are merged pairwise, each
// thread finding by a binary search along its diagonal where its PER outputs
// start in the two runs (merge path) and merging them in registers.  Up to
// runs of a wavefront's 64 PER positions a round needs no workgroup barrier; the
// last four rounds take two each.  The bitonic network it replaced had 78
// dependent steps, each a pass over LDS with a barrier: the in-LDS stage took
// 148 us for the clustered million points with it and 92 us with this.
template <int PER>
__device__ void lds_sort(LdsSort<PER>& S, const uint32_t* idxs, int n)
{
    const int p0 = PER * (int)threadIdx.x;
    uint64_t k[PER];
    uint16_t id[PER];
#pragma unroll
    for (int u = 0; u < PER; ++u) { k[u] = S.key[p0 + u]; id[u] = S.id[p0 + u]; }
    auto order = [&](int a, int b) {
        if (lds_less(k[b], id[b], k[a], id[a], idxs)) {
            const uint64_t t = k[a]; k[a] = k[b]; k[b] = t;
            const uint16_t v = id[a]; id[a] = id[b]; id[b] = v;
        }
    };
    static_assert(PER == 1 || PER == 2 || PER == 4, "sorting network of the thread's entries");
    if constexpr (PER >= 2) order(0, 1);
    if constexpr (PER == 4) { order(2, 3); order(0, 2); order(1, 3); order(1, 2); }
#pragma unroll
    for (int u = 0; u < PER; ++u) { S.key[p0 + u] = k[u]; S.id[p0 + u] = id[u]; }
    for (int w = PER; w < n; w <<= 1) {
        const bool block = 2 * w > 64 * PER;     // the merged run spans wavefronts
        if (block) __syncthreads();
        else wave_sync();
        const int base = p0 & ~(2 * w - 1), d = p0 - base;   // the pair of runs, this thread's diagonal
        const uint64_t* A = S.key + base;
        const uint64_t* B = A + w;
        const uint16_t* Ai = S.id + base;
        const uint16_t* Bi = Ai + w;
        int lo = max(0, d - w), hi = min(d, w);
        while (lo < hi) {                          // entries of A before the diagonal
            const int mid = (lo + hi) >> 1, q = d - 1 - mid;
            if (lds_less(B[q], Bi[q], A[mid], Ai[mid], idxs)) hi = mid;
            else lo = mid + 1;
        }
        int a = lo, b = d - lo;
        uint64_t ka = a < w ? A[a] : ~0ull, kb = b < w ? B[b] : ~0ull;
        uint16_t ia = a < w ? Ai[a] : 0, ib = b < w ? Bi[b] : 0;
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            const bool tb = a >= w || (b < w && lds_less(kb, ib, ka, ia, idxs));
            k[u] = tb ? kb : ka;
            id[u] = tb ? ib : ia;
            if (u + 1 < PER) {
                if (tb) {
                    ++b;
                    if (b < w) { kb = B[b]; ib = Bi[b]; }
                } else {
                    ++a;
                    if (a < w) { ka = A[a]; ia = Ai[a]; }
                }
            }
        }
        if (block) __syncthreads();
        else wave_sync();
#pragma unroll
        for (int u = 0; u < PER; ++u) { S.key[p0 + u] = k[u]; S.id[p0 + u] = id[u]; }
    }
    __syncthreads();
}

// Local ids 0..n-1 of the segment ordered by (coordinate, input index) into
// out.  Bucket sort: 1024 PER equal-width buckets between the segment's
// minimum and maximum coordinate (a monotone map), an exclusive scan of the
// populations, a scatter, and the place of every element inside its bucket
// from the count of the bucket's elements that precede it.  When a bucket
// holds more than kBucketMax points (ties, tight clusters, rows of a grid) a
// merge sort runs instead.
// The line between the two: ranking costs VALU time in proportion to the
// largest bucket, 15 us per axis at 64 points and full segments against 20 us
// for the merge sort; at 16 points the sheet's columns (28 points, one bucket
// each) took the sort, 90 us for the stage instead of 75.
// Before that, where a bucket holds more than kRefine points, every bucket is
// divided once more in proportion to its population (3 us per axis): a smooth but
// uneven density then has a few points per bucket.  The sheet's y order took 36 us
// by the merge sort and takes 19; its columns are ties that no division
// separates.  Uniform points have up to 9 in one of their 4096 buckets, and no
// second pass.  More passes than one gave the clustered points nothing (34 us
// of merge sort became 38).
constexpr int kBucketMax = 64;
constexpr int kRefine = 12;

template <int PER>
__device__ void lds_order(LdsUnion<PER>& U, const double* __restrict__ c, const uint32_t* idxs, int n, uint16_t* out,
                          int* sh, double* red)
{
    constexpr int NB = PER * kLdsThreads;
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    // range of the coordinate
    double lo = 1e308, hi = -1e308;
    double cv[PER];
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        const int i = tid + u * kLdsThreads;
        cv[u] = i < n ? c[i] : 0.0;
        if (i < n) { lo = fmin(lo, cv[u]); hi = fmax(hi, cv[u]); }
    }
    lo = wave_min(lo);
    hi = wave_max(hi);
    if (lane == 0) { red[wid] = lo; red[kLdsWaves + wid] = hi; }
    for (int b = tid; b < NB; b += kLdsThreads) U.b.cnt[b] = 0;
    __syncthreads();
    lo = red[0]; hi = red[kLdsWaves];
    for (int w = 1; w < kLdsWaves; ++w) { lo = fmin(lo, red[w]); hi = fmax(hi, red[kLdsWaves + w]); }
    const double ext = hi - lo;
    double scale = ext > 0.0 ? (double)NB / ext : 0.0;
    scale = scale < 1e300 ? scale : 0.0;
    int bk[PER];
    double fr[PER];   // the place inside the bucket, 0 .. 1
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        const LdsPlace at = lds_place(cv[u], lo, scale, NB);
        bk[u] = at.bucket;
        fr[u] = at.place;
    }
    int mx;
    for (int level = 0;; ++level) {
#pragma unroll
        for (int u = 0; u < PER; ++u)
            if (tid + u * kLdsThreads < n) atomicAdd(&U.b.cnt[bk[u]], 1u);
        __syncthreads();
        // exclusive scan of the populations (thread t owns buckets PER t .. PER t + PER - 1) and
        // the largest population
        uint32_t q[PER];
        int loc = 0;
        mx = 0;
#pragma unroll
        for (int v = 0; v < PER; ++v) {
            q[v] = U.b.cnt[PER * tid + v];
            loc += (int)q[v];
            mx = max(mx, (int)q[v]);
        }
        mx = wave_max_i32(mx);
        int tot;
        int run = block_excl_scan<kLdsThreads>(loc, sh, &tot);
        if (lane == 0) sh[kLdsWaves + wid] = mx;
#pragma unroll
        for (int v = 0; v < PER; ++v) {
            U.b.cnt[PER * tid + v] = (uint32_t)run;
            run += (int)q[v];
        }
        __syncthreads();
        mx = 0;
        for (int w = 0; w < kLdsWaves; ++w) mx = max(mx, sh[kLdsWaves + w]);
        if (level == 1 || mx <= kRefine) break;
        // the second level: a bucket of c points becomes c buckets of equal
        // width, in the places that its points take
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            if (tid + u * kLdsThreads < n) {
                const int b0 = (int)U.b.cnt[bk[u]], b1 = bk[u] + 1 < NB ? (int)U.b.cnt[bk[u] + 1] : n;
                bk[u] = lds_finer(fr[u], b0, b1);
            }
        }
        __syncthreads();
        for (int b = tid; b < NB; b += kLdsThreads) U.b.cnt[b] = 0;
        __syncthreads();
    }
    __syncthreads();
    if (mx > kBucketMax) {
        // merge sort instead (uniform branch)
        for (int i = tid; i < NB; i += kLdsThreads) {
            U.s.key[i] = i < n ? okey(c[i]) : ~0ull;
            U.s.id[i] = i < n ? (uint16_t)i : 0xffff;
        }
        __syncthreads();
        lds_sort<PER>(U.s, idxs, n);
        for (int i = tid; i < n; i += kLdsThreads) out[i] = U.s.id[i];
        __syncthreads();
        return;
    }
    // scatter into bucket order; cnt becomes the end of every bucket
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        const int i = tid + u * kLdsThreads;
        if (i < n) {
            const uint32_t pos = atomicAdd(&U.b.cnt[bk[u]], 1u);
            U.b.key[pos] = okey(cv[u]);
            U.b.id[pos] = (uint16_t)i;
        }
    }
    __syncthreads();
    // the place of every element inside its bucket (at most kBucketMax
    // elements): the count of the bucket's elements smaller in (key, input
    // index); the reads of the bucket are independent, so they are issued
    // together
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        const int i = tid + u * kLdsThreads;
        if (i < n) {
            const int b = bk[u];
            const int e = (int)U.b.cnt[b], s0 = b == 0 ? 0 : (int)U.b.cnt[b - 1];
            const uint64_t km = okey(cv[u]);
            const uint32_t xm = idxs[i];
            // the first kRankFirst keys of the bucket are read unconditionally
            // (indices clamped into the bucket, which holds this element);
            // the input index only for an exact tie; larger buckets go on
            constexpr int kRankFirst = 8;
            uint64_t kk[kRankFirst];
#pragma unroll
            for (int t = 0; t < kRankFirst; ++t) kk[t] = U.b.key[min(s0 + t, e - 1)];
            int r = 0;
#pragma unroll
            for (int t = 0; t < kRankFirst; ++t) {
                if (s0 + t < e) {
                    r += kk[t] < km;
                    if (kk[t] == km) r += idxs[U.b.id[s0 + t]] < xm;
                }
            }
            for (int q = s0 + kRankFirst; q < e; ++q) {
                const uint64_t kq = U.b.key[q];
                r += kq < km;
                if (kq == km) r += idxs[U.b.id[q]] < xm;
            }
            out[s0 + r] = (uint16_t)i;
        }
    }
    __syncthreads();
}

// One stage (d of `stages`) of the splits of the positions that a thread owns, p0 ..
// p0 + PER - 1 (those below `end`): st, cn and sid are the start, the count and
// the index at stage t of their sub-segments.
template <int PER, class POS, class ANC>
__device__ __forceinline__ void lds_stage(int t, int d, bool last, int p0, int end, const LdsWork& w,
                                          const double* xs, const double* ys, uint16_t* LX, uint16_t* LY, POS& q,
                                          int* sh, int (&st)[PER], int (&cn)[PER], int (&sid)[PER], ANC above,
                                          double* bbox, double* geom)
{
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    // split axis of the sub-segment of every owned position, from the
    // ends of both lists; the head position (the sub-segment's first)
    // writes the box geometry at even stages
    int ax[PER];
    bool valid[PER];
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        const int i = p0 + u;
        valid[u] = i < end;
        ax[u] = 0;
        if (!valid[u]) continue;
        if (u > 0 && valid[u > 0 ? u - 1 : 0] && st[u] == st[u > 0 ? u - 1 : 0]) {
            ax[u] = ax[u > 0 ? u - 1 : 0];
            continue;
        }
        const int e1 = st[u] + cn[u] - 1;
        const double x0 = xs[LX[st[u]]], x1 = xs[LX[e1]];
        const double y0 = ys[LY[st[u]]], y1 = ys[LY[e1]];
        ax[u] = ((x1 - x0) >= (y1 - y0)) ? 0 : 1;
        if (i == st[u] && (t & 1) == 0) {
            const int64_t j = ((int64_t)w.j0 << d) + sid[u], box = (int64_t)w.boxbase + level_base(t / 2) + j;
            double bb[4], gm[3];
            box_geometry(x0, x1, y0, y1, bb, gm);
            for (int c = 0; c < 4; ++c) bbox[4 * box + c] = bb[c];
            for (int c = 0; c < 3; ++c) geom[4 * box + c] = gm[c];
            // no extent: the nearest ancestor's radius, of the boxes that this
            // workgroup has written or of those above
            double rs = gm[2];
            for (int b = 2; !(rs > 0.0) && b <= d; b += 2)
                rs = geom[4 * ((int64_t)w.boxbase + level_base((t - b) / 2) + (j >> b)) + 2];
            geom[4 * box + 3] = rs > 0.0 ? rs : above();
        }
    }
    if (last) return;
    // element of the other list at every owned position and whether it
    // lies in the lower half along the split axis
    uint16_t e[PER];
    int f[PER], lb[PER];
    bool tail[PER];   // no head at or before this position within the thread
    int run = 0;
    bool seen = false;
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        const int i = p0 + u;
        f[u] = 0;
        e[u] = 0;
        if (valid[u]) {
            e[u] = ax[u] ? LX[i] : LY[i];
            const int pa = ax[u] ? (int)q.posY[e[u]] : (int)q.posX[e[u]];
            f[u] = (pa - st[u]) < (cn[u] >> 1);
            if (i == st[u]) { run = 0; seen = true; }
        }
        tail[u] = !seen;
        lb[u] = run;
        run += f[u];
    }
    // segmented exclusive scan of the lower flags over the positions
    // (restarting at every sub-segment head): within the wavefront by
    // lane permutations, across wavefronts through one barrier
    int v = run, hf = seen ? 1 : 0, ev, eh;
    wave_seg_scan(hf, v, eh, ev);
    if (lane == 63) { sh[wid] = v; sh[kLdsWaves + wid] = hf; }
    __syncthreads();
    // (a scan of the wavefronts' totals by lanes 0 .. 15 of each wavefront)
    int wv = sh[lane & (kLdsWaves - 1)], wh = sh[kLdsWaves + (lane & (kLdsWaves - 1))];
    row_seg_scan(wh, wv);
    const int wu = __builtin_amdgcn_readfirstlane(wid);
    const int carry = wu ? __builtin_amdgcn_readlane(wv, wu - 1) : 0;
    const int cin = eh ? ev : carry + ev;
    // scatter the other list's elements in place (every read of the
    // lists and positions of this stage came before the barrier) and
    // step every owned position into its child
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        if (!valid[u]) continue;
        const int i = p0 + u;
        const int before = lb[u] + (tail[u] ? cin : 0);   // lower elements in [st, i)
        const int kq = cn[u] >> 1, rel = i - st[u];
        const int dst = f[u] ? st[u] + before : st[u] + kq + (rel - before);
        if (ax[u]) { LX[dst] = e[u]; q.posX[e[u]] = (uint16_t)dst; }
        else { LY[dst] = e[u]; q.posY[e[u]] = (uint16_t)dst; }
        if (rel < kq) { cn[u] = kq; sid[u] = 2 * sid[u]; }
        else { st[u] += kq; cn[u] -= kq; sid[u] = 2 * sid[u] + 1; }
    }
    __syncthreads();
}

// Where the segments of k_lds_split come from: the global stages' buffers, or
// (z set: no problem has a global stage) the caller's positions, checked here
struct LdsInput {
    const double *XA, *YA, *XB, *YB;
    const int32_t *IA, *IB;
    const double* z;
    uint32_t* err;      // with z: non-finite positions
    int err_store;      // 1: the only segment, err is written; 0: err was cleared
};
// The boxes of the global stages, shared out over the workgroups
struct LdsGeom {
    const GeomJob* jobs;
    int n;
    const uint64_t* keys;
};

// A segment of at most 1024 PER points per workgroup; with QUARTERS four
// workgroups per segment: each sorts it and does the first two splits, then
// goes on with one of the four sub-segments alone.
// Bound by LDS accesses and the chain of barriers of the sort and the stages.
// PER from the largest segment: with 4 positions per thread a segment of 1024
// points keeps 4 of the 16 wavefronts busy.  QUARTERS where the chip has room
// for four times the workgroups: past the second split a thread owns one
// position instead of PER (1.2 us a stage instead of 2.6).  Measured: N = 1000,
// one segment, 25.5 us (and 10 us of three launches around it, now part of this
// one) to 19.8; 16,000 points of a sheet, four segments, 74.7 to 56.6 (and 9 us
// of two launches); 1e6 points, 256 segments, 50 to 53 (and 10 us of two
// launches), of which the loads take 3, either sort 10, the stages 24.
template <int PER, bool QUARTERS>
__global__ void __launch_bounds__(kLdsThreads)
k_lds_split(const LdsWork* __restrict__ work, const LdsInput in, const LdsGeom gk, double* Xo, double* Yo,
            int32_t* Io, double* bbox, double* geom)
{
    constexpr int CAP = PER * kLdsThreads;
    __shared__ LdsUnion<PER> U;
    __shared__ uint32_t idxs[CAP];
    __shared__ uint16_t LX[CAP], LY[CAP];
    __shared__ int sh[2 * kLdsWaves];
    __shared__ double red[2 * kLdsWaves];
    __shared__ double xs[CAP], ys[CAP];   // coordinates by local id
    const int quarter = QUARTERS ? blockIdx.x & 3 : 0;
    const LdsWork w = work[QUARTERS ? blockIdx.x >> 2 : blockIdx.x];
    const int n = w.count;
    {
        // every load of the segment in flight before the first LDS store
        uint32_t li[PER];
        double lx[PER], ly[PER];
        if (in.z) {
            bool bad = false;
#pragma unroll
            for (int u = 0; u < PER; ++u) {
                const int i = threadIdx.x + u * kLdsThreads;
                const int ic = w.start + (i < n ? i : 0);
                const double2 v = reinterpret_cast<const double2*>(in.z)[ic];
                // a non-finite position is flagged and built as (0, 0)
                const bool ok = isfinite(v.x) && isfinite(v.y);
                bad |= !ok;
                li[u] = (uint32_t)ic;
                lx[u] = ok ? v.x : 0.0;
                ly[u] = ok ? v.y : 0.0;
            }
            const int any = __syncthreads_or(bad);
            if (threadIdx.x == 0 && quarter == 0) {
                if (in.err_store) *in.err = any ? 1u : 0u;
                else if (any) atomicOr(in.err, 1u);
            }
        } else {
            const double* xg = ((w.stage0 & 1) ? in.XB : in.XA) + w.start;
            const double* yg = ((w.stage0 & 1) ? in.YB : in.YA) + w.start;
            const int32_t* is = ((w.stage0 & 1) ? in.IB : in.IA) + w.start;
#pragma unroll
            for (int u = 0; u < PER; ++u) {
                const int i = threadIdx.x + u * kLdsThreads;
                const int ic = i < n ? i : 0;
                li[u] = (uint32_t)is[ic];
                lx[u] = xg[ic];
                ly[u] = yg[ic];
            }
        }
        const int64_t nb = gridDim.x;
        geom_from_keys(gk.jobs, (int)(gk.n * (int64_t)blockIdx.x / nb), (int)(gk.n * ((int64_t)blockIdx.x + 1) / nb),
                       gk.keys, bbox, geom);
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            const int i = threadIdx.x + u * kLdsThreads;
            if (i < n) {
                idxs[i] = li[u];
                xs[i] = lx[u];
                ys[i] = ly[u];
            }
        }
    }
    __syncthreads();
    lds_order<PER>(U, xs, idxs, n, LX, sh, red);
    lds_order<PER>(U, ys, idxs, n, LY, sh, red);
    for (int i = threadIdx.x; i < n; i += kLdsThreads) {
        U.q.posX[LX[i]] = (uint16_t)i;
        U.q.posY[LY[i]] = (uint16_t)i;
    }
    __syncthreads();
    auto above = [&] { return ancestor_radius(gk.jobs, w.up, gk.keys); };
    const int p0 = PER * (int)threadIdx.x;
    int st[PER], cn[PER], sid[PER];
#pragma unroll
    for (int u = 0; u < PER; ++u) { st[u] = 0; cn[u] = n; sid[u] = 0; }
    const int shared = QUARTERS ? 2 : w.stages + 1;    // stages of the whole segment
    for (int d = 0; d < shared; ++d)
        lds_stage<PER>(w.stage0 + d, d, d == w.stages, p0, n, w, xs, ys, LX, LY, U.q, sh, st, cn, sid, above, bbox,
                       geom);
    int first = 0, count = n;
    if constexpr (QUARTERS) {
        // (the boxes of the first two splits are written by all four, alike)
        for (int b = 1; b >= 0; --b) {
            const int h = count >> 1;
            if ((quarter >> b) & 1) { first += h; count -= h; }
            else count = h;
        }
        int s1[1] = {first}, c1[1] = {count}, i1[1] = {quarter};
        for (int d = 2; d <= w.stages; ++d)
            lds_stage<1>(w.stage0 + d, d, d == w.stages, first + (int)threadIdx.x, first + count, w, xs, ys, LX, LY, U.q,
                         sh, s1, c1, i1, above, bbox, geom);
    }
    // final order: sorted by (x, index) inside every leaf
#pragma unroll
    for (int u = 0; u < (QUARTERS ? 1 : PER); ++u) {
        const int i = threadIdx.x + u * kLdsThreads;
        if (i < count) {
            const int id = LX[first + i], o = w.start + first + i;
            Xo[o] = xs[id]; Yo[o] = ys[id]; Io[o] = (int32_t)idxs[id];
        }
    }
}

__global__ void k_update_positions(const double* __restrict__ z, const int32_t* __restrict__ perm,
                                   int64_t n, double* X, double* Y)
{
    int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= n) return;
    double2 v = reinterpret_cast<const double2*>(z)[perm[i]];
    X[i] = v.x; Y[i] = v.y;
}

// ------------------------------------------------------------------- driver

static int grid_for(int64_t n, int bs) { return (int)std::min<int64_t>((n + bs - 1) / bs, 65535 * 4); }

// Four workgroups per segment while that is at most one per compute unit and
// every segment has more than two splits; not for segments of at most 1024
// points, whose threads own one position anyway.
constexpr int kQuarterBlocks = 256;

static void run_lds_split(Tree& t, const LdsInput& in, const uint64_t* keys, hipStream_t s)
{
    TreeSchedule& sc = *t.sched;
    const int per = (sc.lds_max + kLdsThreads - 1) / kLdsThreads;
    const unsigned nw = (unsigned)sc.lds.size();
    const bool quarters = per > 1 && 4 * nw <= kQuarterBlocks && sc.lds_stages > 2;
    const LdsGeom gk{sc.d_geom.p, keys ? (int)sc.geom.size() : 0, keys};
#define LDS_SPLIT(PER, Q)                                                                                        \
    k_lds_split<PER, Q><<<(Q ? 4 : 1) * nw, kLdsThreads, 0, s>>>(sc.d_lds.p, in, gk, t.x.p, t.y.p, t.perm.p,     \
                                                                 t.bbox.p, t.geom.p)
    if (per <= 1) LDS_SPLIT(1, false);
    else if (per == 2 && quarters) LDS_SPLIT(2, true);
    else if (per == 2) LDS_SPLIT(2, false);
    else if (quarters) LDS_SPLIT(4, true);
    else LDS_SPLIT(4, false);
#undef LDS_SPLIT
    check_launch("lds split");
}

static void build_tree_select(Tree& t, const double* z, hipStream_t s)
{
    TreeSchedule& sc = *t.sched;
    int64_t n = sc.n;
    // no global stage: the in-LDS kernel reads the positions and does the rest
    if (sc.nstage == 0 && sc.copy_tiles.empty()) {
        const bool one = sc.lds.size() == 1;
        if (!one) {
            k_fill_start<<<1, 64, 0, s>>>(nullptr, 0, nullptr, 0, t.err.p);
            check_launch("fill");
        }
        run_lds_split(t, LdsInput{nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, z, t.err.p, one}, nullptr, s);
        return;
    }
    // workspace
    DBuf<double> XA, YA, XB, YB;
    DBuf<int32_t> IA, IB;
    XA.alloc(n, s); YA.alloc(n, s); IA.alloc(n, s);
    if (sc.nstage > 0) { XB.alloc(n, s); YB.alloc(n, s); IB.alloc(n, s); }
    int64_t nkeys = sc.total_keys;
    DBuf<uint64_t> keys; keys.alloc(kKeyWords * nkeys, s);
    int64_t nseg_split = sc.nstage > 0 ? sc.keys_off[sc.nstage] : 0;   // segments of split stages
    DBuf<uint32_t> words;   // hist1 | hist2 | cand_cnt | tiles done per segment | tile_below | lo_base
    int64_t nt = sc.total_tile;
    int64_t o_h1 = 0, o_h2 = nseg_split * 2 * kHistCopies * kBuckets1, o_cc = o_h2 + nseg_split * kBuckets2;
    int64_t o_sd = o_cc + nseg_split, o_tb = o_sd + nseg_split;
    int64_t o_lb = o_tb + nt, nwords = o_lb + nt;
    words.alloc(nwords, s);
    DBuf<Cand> cand; cand.alloc(std::max<int64_t>(nseg_split, 1) * kCandCap, s);
    DBuf<Splitter> split; split.alloc(std::max<int64_t>(nseg_split, 1), s);
    DBuf<ClassInfo> cinfo; cinfo.alloc(std::max<int64_t>(nseg_split, 1), s);
    DBuf<Level1> lvl1; lvl1.alloc(std::max<int64_t>(nseg_split, 1), s);

    k_fill_start<<<grid_for(std::max<int64_t>(nwords, kKeyWords * nkeys), 256), 256, 0, s>>>(
        words.p, nwords, keys.p, kKeyWords * nkeys, t.err.p);
    check_launch("fill");
    uint32_t* W = words.p;
    // init: every problem's root segment is stage-0 key segment b
    int64_t maxn = 0;
    for (int b = 0; b < sc.nprob; ++b) maxn = std::max(maxn, sc.off[b + 1] - sc.off[b]);
    dim3 gi((unsigned)((maxn + kTile - 1) / kTile), (unsigned)sc.nprob);
    k_init<<<gi, kTileThreads, 0, s>>>(z, sc.d_off.p, sc.nprob, XA.p, YA.p, IA.p, keys.p, t.err.p);
    check_launch("init");
    double* Xb[2] = {XA.p, XB.p};
    double* Yb[2] = {YA.p, YB.p};
    int32_t* Ib[2] = {IA.p, IB.p};
    for (int st = 0; st < sc.nstage; ++st) {
        int ntl = sc.ntile[st];
        if (ntl == 0) continue;
        const TileInfo* tl = sc.d_tiles.p + sc.tile_off[st];
        int a = st & 1;
        // later stages' first-level histograms come from the previous partition
        if (st == 0) k_hist1<<<ntl, kTileThreads, 0, s>>>(tl, Xb[a], Yb[a], keys.p, W + o_h1);
        k_hist2<<<ntl, kTileThreads, 0, s>>>(tl, sc.d_segs.p, Xb[a], Yb[a], keys.p, W + o_h1, W + o_h2, lvl1.p);
        k_collect<<<ntl, kTileThreads, 0, s>>>(tl, sc.d_tiles.p, sc.d_segs.p, Xb[a], Yb[a], Ib[a], lvl1.p, W + o_h2,
                                              cand.p, W + o_cc, W + o_tb, W + o_sd, cinfo.p, W + o_lb, split.p);
        k_partition<<<ntl, kTileThreads, 0, s>>>(tl, sc.d_segs.p, Xb[a], Yb[a], Ib[a], Xb[a ^ 1], Yb[a ^ 1],
                                                Ib[a ^ 1], keys.p, cinfo.p, cand.p, W + o_tb, split.p, W + o_lb,
                                                W + o_h1, lvl1.p);
        check_launch("split stage");
    }
    if (!sc.copy_tiles.empty()) {
        k_copy_final<<<(unsigned)sc.copy_tiles.size(), 256, 0, s>>>(sc.d_copy.p, XA.p, YA.p, IA.p, XB.p, YB.p,
                                                                    IB.p, t.x.p, t.y.p, t.perm.p);
        check_launch("copy final");
    }
    if (!sc.lds.empty()) {
        run_lds_split(t, LdsInput{XA.p, YA.p, XB.p, YB.p, IA.p, IB.p, nullptr, nullptr, 0}, keys.p, s);
    } else if (!sc.geom.empty()) {
        const int ng = (int)sc.geom.size();
        k_geom_keys<<<(unsigned)((ng + 7) / 8), 256, 0, s>>>(sc.d_geom.p, ng, keys.p, t.bbox.p, t.geom.p);
        check_launch("geom");
    }
    // non-finite positions: t.err, read at the next synchronising call on the tree
}

void build_tree_device(Tree& t, const double* z, hipStream_t s)
{
    TreeSchedule& sc = *t.sched;
    const int64_t n = sc.n;
    t.x.alloc(n, s); t.y.alloc(n, s); t.perm.alloc(n, s);
    t.bbox.alloc(4 * sc.nbox, s); t.geom.alloc(4 * sc.nbox, s);
    t.err.alloc(1, s);
    build_tree_select(t, z, s);
}

void update_positions_device(Tree& t, const double* z, hipStream_t s)
{
    int64_t n = t.sched->n;
    k_update_positions<<<(unsigned)((n + 255) / 256), 256, 0, s>>>(z, t.perm.p, n, t.x.p, t.y.p);
    check_launch("update positions");
}

}  // namespace fmm
