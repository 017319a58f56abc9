// HIP kernels of the semantic TSDF integrator (gfx950, wave64).
//
// One frame runs as five kernels on the map's stream:
//   1. ray_walk       one lane per point: pose application, ray, band, voxel
//                     walk (Sec. III-A), truncation gate.  The leaves the
//                     block's rays touch are collected in an LDS table, so each
//                     (block, leaf) makes one staging insert and one bucket
//                     reservation; the walk is recorded, some 50 bytes a ray.
//   2. leaf_plan      one lane per touched leaf: find it in the map (or number
//                     it as new), number record pages for newly touched 8x8
//                     slabs, allocate its pair bucket.
//   3. ray_emit       one lane per point: the recorded walk again, every kept
//                     (voxel, point) observation written to its leaf's bucket.
//   4. leaf_acc       geometry and int32 labels (K <= 32): one workgroup per
//                     touched leaf (or one wave per small leaf) adds every pair
//                     into its voxel's LDS accumulators with integer atomics --
//                     observation counts, class counts, fixed-point distance
//                     sums -- and one lane per touched voxel applies them, Eq.
//                     (1)-(2) for D and W and Eq. (6) for the class counts.
//      leaf_fuse      probability or logit rows, the open set, the most-recent
//                     modes: counting sort of the bucket by voxel offset in LDS,
//                     then by point index inside each voxel, and the combine of
//                     every touched voxel in point order (the open set's Eqs.
//                     (11)-(14) with lambda = 2 nu = W in k_voxel_combine).
//   5. frame_commit   one workgroup: counters, status, frame reset.
// Kernels 1-3 only read the map, and kernel 4 writes it only if the frame's new
// leaves and record pages fit (decided from totals that kernel 2 completed), so
// a frame that does not fit changes nothing.  No floating-point atomics are
// used: integer sums are exact in any order and every floating-point sum runs
// in point order, so results are bitwise repeatable and independent of launch
// shapes.
//
// The geometric decision path (pose, ray, walk, gate) is a fixed sequence of
// binary32 operations; build with -ffp-contract=off so that only the fmaf()
// calls written here fuse, and with correctly rounded division and sqrt.

#include <hip/hip_runtime.h>

#include <algorithm>
#include <mutex>
#include <utility>

#include "slim_internal.h"
#include "slimvdb.h"

namespace slim {

// ---------------------------------------------------------------------------
// small device helpers
// ---------------------------------------------------------------------------

__device__ __forceinline__ uint32_t leaf_hash(unsigned long long k, uint32_t mask)
{
    k ^= k >> 33;
    k *= 0xff51afd7ed558ccdull;
    k ^= k >> 33;
    k *= 0xc4ceb9fe1a85ec53ull;
    k ^= k >> 33;
    return (uint32_t)k & mask;
}

// Slot of a leaf in the map's table, or -1.
__device__ int32_t map_find(const MapDev &md, unsigned long long key)
{
    uint32_t h = leaf_hash(key, md.hmask);
    for (uint32_t probe = 0; probe <= md.hmask; ++probe) {
        const uint4 e = *(const uint4 *)&md.htab[h];
        const unsigned long long k = ((unsigned long long)e.y << 32) | e.x;
        if (k == key) return (int32_t)e.z;
        if (k == kEmptyKey) return -1;
        h = (h + 1) & md.hmask;
    }
    return -1;
}

// Inserts a leaf known to be absent, in two steps so that the first probe's
// round trip can overlap other loads: map_insert_start claims the leaf's home
// slot if it is free (one compare-and-swap) and map_insert_finish, given that
// result, probes on if it was taken and stores the slot.  The table is at
// most half full.
__device__ __forceinline__ unsigned long long map_insert_start(const MapDev &md, unsigned long long key,
                                                               uint32_t *h)
{
    *h = leaf_hash(key, md.hmask);
    return atomicCAS(&md.htab[*h].key, kEmptyKey, key);
}

__device__ void map_insert_finish(const MapDev &md, unsigned long long key, int32_t slot, uint32_t h,
                                  unsigned long long prev)
{
    for (uint32_t probe = 0; probe <= md.hmask; ++probe) {
        if (prev == kEmptyKey) {
            md.htab[h].val = slot;
            return;
        }
        h = (h + 1) & md.hmask;
        prev = atomicCAS(&md.htab[h].key, kEmptyKey, key);
    }
}

__device__ __forceinline__ int lane_id() { return (int)(threadIdx.x & 63); }

__device__ __forceinline__ uint32_t wave_incl_scan(uint32_t v)
{
    const int lane = lane_id();
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        uint32_t t = __shfl_up(v, d, 64);
        if (lane >= d) v += t;
    }
    return v;
}

// ---------------------------------------------------------------------------
// geometry (binary32, fixed operation order)
// ---------------------------------------------------------------------------

struct Ray {
    float p[3];   // point relative to the anchor corner
    float u[3];   // unit direction
    float t0, t1; // band
};

__device__ __forceinline__ bool make_ray(const FrameParams &fp, float x, float y, float z, Ray &ry)
{
    if (!(isfinite(x) && isfinite(y) && isfinite(z))) return false;
#pragma unroll
    for (int a = 0; a < 3; ++a)
        ry.p[a] = fmaf(fp.R[3 * a + 0], x, fmaf(fp.R[3 * a + 1], y, fmaf(fp.R[3 * a + 2], z, fp.t[a])));
    const float d0 = ry.p[0] - fp.t[0], d1 = ry.p[1] - fp.t[1], d2 = ry.p[2] - fp.t[2];
    const float r = sqrtf(fmaf(d2, d2, fmaf(d1, d1, d0 * d0)));
    if (!(r > 0.0f) || !isfinite(r) || r < fp.rmin || r > fp.rmax) return false;
    ry.u[0] = d0 / r;
    ry.u[1] = d1 / r;
    ry.u[2] = d2 / r;
    ry.t0 = fmaxf(r - fp.tau, 0.0f);
    ry.t1 = r + fp.tau;
    return true;
}

// Sensor-frame point i: given directly, as range * unit direction (one
// binary32 product per component), or back-projected from pixel i of a depth
// image, ((u - cx) / fx) d, ((v - cy) / fy) d, d, rounded in that order (a
// depth that is not finite and positive gives a rejected point).
__device__ __forceinline__ void load_point(const FrameParams &fp, int i, float &x, float &y, float &z)
{
    if (fp.pts) {
        x = fp.pts[3 * i + 0];
        y = fp.pts[3 * i + 1];
        z = fp.pts[3 * i + 2];
    } else if (fp.depth) {
        const int v = i / fp.width, u = i - v * fp.width;
        const float d = fp.depth[i];
        if (!(d > 0.0f) || !isfinite(d)) {
            x = y = z = NAN;
            return;
        }
        x = (((float)u - fp.cx) / fp.fx) * d;
        y = (((float)v - fp.cy) / fp.fy) * d;
        z = d;
    } else {
        const float r = fp.ranges[i];
        x = r * fp.dirs[3 * i + 0];
        y = r * fp.dirs[3 * i + 1];
        z = r * fp.dirs[3 * i + 2];
    }
}

// Amanatides-Woo walk over the band of the ray from the sensor origin
// (fp.t).  Calls visit(cx, cy, cz) per cell (anchor-relative).  Ties between
// axes step the lowest axis first, one axis per step; the walk stops when the
// next boundary lies beyond t1, or after maxsteps cells.
// Start of the walk: first cell c, step direction, first boundary crossing
// tm and crossing interval td per axis (tm = td = inf on an axis the ray does
// not move along).
struct WalkState {
    int c[3], stp[3];
    float tm[3], td[3];
};

// Returns false when a start cell lies 2^30 or more cells from the anchor: its
// key is then outside |k| < 2^20 whatever the anchor, so the point is rejected
// (and the cell index never overflows an int while the walk steps on).
constexpr float kCellLimit = 1073741824.0f;  // 2^30

__device__ __forceinline__ bool walk_start(const FrameParams &fp, const Ray &ry, WalkState &w)
{
    const float vs = fp.vs, t0 = ry.t0;
    bool ok = true;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const float s = fmaf(t0, ry.u[a], fp.t[a]);
        const float fc = floorf(s / vs);
        ok = ok && fabsf(fc) < kCellLimit;
        w.c[a] = fabsf(fc) < kCellLimit ? (int)fc : 0;
        if (ry.u[a] > 0.0f) {
            w.stp[a] = 1;
            w.tm[a] = t0 + fmaf((float)(w.c[a] + 1), vs, -s) / ry.u[a];
            w.td[a] = vs / ry.u[a];
        } else if (ry.u[a] < 0.0f) {
            w.stp[a] = -1;
            w.tm[a] = t0 + fmaf((float)w.c[a], vs, -s) / ry.u[a];
            w.td[a] = -vs / ry.u[a];
        } else {
            w.stp[a] = 0;
            w.tm[a] = INFINITY;
            w.td[a] = INFINITY;
        }
    }
    return ok;
}

// Axis of the next step (ties step the lowest axis) and the ray parameter of
// the boundary it crosses.
__device__ __forceinline__ int walk_axis(const WalkState &w, float &tnext)
{
    const bool xy = w.tm[0] <= w.tm[1];
    const int ax = xy ? (w.tm[0] <= w.tm[2] ? 0 : 2) : (w.tm[1] <= w.tm[2] ? 1 : 2);
    tnext = ax == 0 ? w.tm[0] : (ax == 1 ? w.tm[1] : w.tm[2]);
    return ax;
}

// One step along axis ax, written as selects (no branch per axis).
__device__ __forceinline__ void walk_step(WalkState &w, int ax)
{
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const bool on = ax == a;
        w.c[a] += on ? w.stp[a] : 0;
        const float nt = w.tm[a] + w.td[a];
        w.tm[a] = on ? nt : w.tm[a];
    }
}

// Amanatides-Woo walk over the band of the ray from the sensor origin
// (fp.t).  Calls visit(cx, cy, cz) per cell (anchor-relative).  Ties between
// axes step the lowest axis first, one axis per step; the walk stops when the
// next boundary lies beyond t1, or after maxsteps cells.
template <class Visit>
__device__ __forceinline__ bool band_walk(const FrameParams &fp, const Ray &ry, Visit &&visit)
{
    WalkState w;
    if (!walk_start(fp, ry, w)) return false;
    for (int it = 0; it < fp.maxsteps; ++it) {
        visit(w.c[0], w.c[1], w.c[2]);
        float tnext;
        const int ax = walk_axis(w, tnext);
        if (tnext > ry.t1) break;
        walk_step(w, ax);
    }
    return true;
}

// Signed distance (binary32) of a cell centre to the point along the ray;
// positive in front of the surface.
__device__ __forceinline__ float cell_sdf(const FrameParams &fp, const Ray &ry, int cx, int cy, int cz)
{
    const float h = 0.5f * fp.vs;
    const float qx = fmaf(-(float)cx, fp.vs, ry.p[0]) - h;
    const float qy = fmaf(-(float)cy, fp.vs, ry.p[1]) - h;
    const float qz = fmaf(-(float)cz, fp.vs, ry.p[2]) - h;
    return fmaf(qz, ry.u[2], fmaf(qy, ry.u[1], qx * ry.u[0]));
}

// The same for a cell held as binary32 coordinates (integers below 2^24).
__device__ __forceinline__ float ray_sdf(float vs, const Ray &ry, float cx, float cy, float cz)
{
    const float h = 0.5f * vs;
    const float qx = fmaf(-cx, vs, ry.p[0]) - h;
    const float qy = fmaf(-cy, vs, ry.p[1]) - h;
    const float qz = fmaf(-cz, vs, ry.p[2]) - h;
    return fmaf(qz, ry.u[2], fmaf(qy, ry.u[1], qx * ry.u[0]));
}

__device__ __forceinline__ bool key_ok(int k) { return k > -kKeyLimit && k < kKeyLimit; }

// ---------------------------------------------------------------------------
// block-wide helpers (blockDim.x a multiple of 64, at most 256)
// ---------------------------------------------------------------------------

// Exclusive prefix sum over the block of one value per thread; *total gets
// the block sum.  Uses wsum[4] of LDS.
__device__ __forceinline__ uint32_t block_excl_scan(uint32_t v, uint32_t *wsum, uint32_t *total)
{
    const int lane = lane_id(), w = threadIdx.x >> 6;
    const uint32_t incl = wave_incl_scan(v);
    if (lane == 63) wsum[w] = incl;
    __syncthreads();
    uint32_t before = 0, tot = 0;
    const int nw = (int)(blockDim.x >> 6);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        if (q < w) before += wsum[q];
        if (q < nw) tot += wsum[q];
    }
    __syncthreads();
    *total = tot;
    return before + incl - v;
}

// Exclusive prefix sum of 512 LDS counters by 256 threads.
__device__ void block_scan512(const uint32_t *in, uint32_t *out, uint32_t *wsum)
{
    const int t = threadIdx.x;
    const uint32_t a = in[2 * t], b = in[2 * t + 1];
    uint32_t total;
    const uint32_t ex = block_excl_scan(a + b, wsum, &total);
    out[2 * t] = ex;
    out[2 * t + 1] = ex + a;
    __syncthreads();
}

// ---------------------------------------------------------------------------
// 1. ray walk
// ---------------------------------------------------------------------------

constexpr int kWaveItemPairs = 256;  // leaves with at most this many pairs are one wave's work
static_assert(kWalkTable >= kWalkThreads * kMaxRuns, "the walk table must hold every run of a block");

__device__ __forceinline__ uint32_t lds_hash(unsigned long long k)
{
    return (uint32_t)((k * 0x9E3779B97F4A7C15ull) >> 40) & (kWalkTable - 1);
}

// Staging-table position of a leaf for the walk: one compare-and-swap per
// probe (an empty slot is claimed, a slot holding the key is found), so the
// common case is one round trip.  *fresh is true for the claiming caller.
__device__ __forceinline__ uint32_t stage_leaf_cas(const MapDev &md, unsigned long long key, bool *fresh)
{
    *fresh = false;
    uint32_t h = leaf_hash(key, md.hmask);
    for (uint32_t probe = 0; probe <= md.hmask; ++probe) {
        const unsigned long long prev = atomicCAS(&md.skeys[h], kEmptyKey, key);
        if (prev == kEmptyKey) {
            *fresh = true;
            return h;
        }
        if (prev == key) return h;
        h = (h + 1) & md.hmask;
    }
    return kNoPos;
}

// A cell's place in its leaf as 5-bit fields (place + 8), x highest: bit 3 of every
// field is set while the cell is inside.
constexpr uint32_t kPlaceInside = (8u << 10) | (8u << 5) | 8u;

// Block-local table of the leaves a walk block's rays touch.
// Kept small enough for three workgroups per CU: slab masks are 8-bit fields,
// four to a word, and entry lists 16-bit.
static_assert(kWalkTable <= 65536, "walk-table entries are listed as 16-bit indices");
struct WalkShared {
    unsigned long long t_key[kWalkTable];
    uint32_t t_cnt[kWalkTable];       // pairs of this block in the leaf, then their first bucket rank
    uint32_t t_pos[kWalkTable];       // staging position
    uint32_t t_slab[kWalkTable / 4];  // x-slabs of the leaf this block touches (8 bits per entry)
    uint16_t t_list[kWalkTable];      // occupied entries
    uint16_t t_fresh[kWalkTable];     // entries whose staging insert this block made
    uint32_t s_n, s_nfresh, s_pairs;
};

// One block of the walk: rays blk * blockDim.x + [0, blockDim.x) of a frame, whose
// records are rblk * blockDim.x + [0, blockDim.x).  A ray's record is what
// ray_emit_block needs to write its pairs where they belong once the leaves'
// buckets are laid out: which cells it kept and how it steps (bits), and for each
// leaf it visits the staging position and the first of its ranks in the leaf's
// bucket.
__device__ __forceinline__ void walk_block(const FrameParams &fp, const MapDev &md, int blk, int rblk, WalkShared &ws)
{
    unsigned long long *t_key = ws.t_key;
    uint32_t *t_cnt = ws.t_cnt, *t_pos = ws.t_pos, *t_slab = ws.t_slab;
    uint16_t *t_list = ws.t_list, *t_fresh = ws.t_fresh;
    uint32_t &s_n = ws.s_n, &s_nfresh = ws.s_nfresh, &s_pairs = ws.s_pairs;

    const int tid = threadIdx.x;
    const int i = blk * blockDim.x + tid;
    // the point is loaded first: its latency overlaps the table clear
    Ray ry;
    bool valid = false;
    if (i < fp.n) {
        float x, y, z;
        load_point(fp, i, x, y, z);
        valid = make_ray(fp, x, y, z, ry);
        if (valid && fp.sem_kind == SLIM_IN_LABEL_I32) {
            const int lab = ((const int32_t *)fp.sem)[i];
            valid = lab >= 0 && lab < fp.K;
        }
    }
    for (int e = tid; e < kWalkTable; e += blockDim.x) {
        t_key[e] = kEmptyKey;
        t_cnt[e] = 0;
    }
    for (int e = tid; e < kWalkTable / 4; e += blockDim.x) t_slab[e] = 0;
    if (tid == 0) {
        s_n = 0;
        s_nfresh = 0;
        s_pairs = 0;
    }
    __syncthreads();

    // the walk, with few instructions a step (a frame of a few thousand
    // points is one wave per SIMD, whose time is the length of this loop's chain).
    // The cell is held as binary32 coordinates, which the distance is formed from
    // (exact: an accepted cell is within 2^21 of the anchor), and as its place in
    // its leaf, a word of three 5-bit fields (place + 8: bit 3 of a field clears
    // when the cell leaves the leaf on that axis).  Recorded: which steps went along
    // x and y, and which cells passed the gate.  Of each leaf the ray visits: its kept cells and their x-slabs (16 bits a visit)
    // and the axis on which the ray leaves it.  Coordinates are monotone along the
    // ray, so the first and the last cell decide the key range.  (Per-cell leaf keys,
    // key-range tests and run arrays before: 20.5 -> 16.7 us for 20,011 points,
    // 23 -> 19.4 for 65,536.)
    uint32_t cnt = 0;
    int nvis = 0, visit = 0;
    unsigned long long stepx = 0ull, stepy = 0ull, kept = 0ull, info[2] = {0ull, 0ull};
    uint32_t exits = 0, at0 = 0;
    unsigned long long key0 = kEmptyKey;
    float cf0[3] = {0.0f, 0.0f, 0.0f}, sf[3] = {0.0f, 0.0f, 0.0f};
    uint32_t st[3] = {0u, 0u, 0u};
    if (valid) {
        WalkState w;
        const bool started = walk_start(fp, ry, w);
        int k0[3];
        float cf[3];
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            k0[a] = fp.a[a] + w.c[a];
            cf0[a] = cf[a] = (float)w.c[a];
            sf[a] = (float)w.stp[a];
            at0 |= (uint32_t)((k0[a] & 7) + 8) << (10 - 5 * a);
            st[a] = (uint32_t)w.stp[a] << (10 - 5 * a);
        }
        key0 = pack_leaf(k0[0] >> 3, k0[1] >> 3, k0[2] >> 3);
        uint32_t at = at0, len = 0, slab = 0;
        auto leave = [&]() {
            const unsigned long long f = (unsigned long long)((len << 8) | slab) << (16 * (visit & 3));
            info[0] |= visit < 4 ? f : 0ull;
            info[1] |= visit < 4 ? 0ull : f;
        };
        const int limit = started ? fp.maxsteps : 0;
        for (int it = 0; it < limit; ++it) {
            nvis = it + 1;
            const bool in = ray_sdf(fp.vs, ry, cf[0], cf[1], cf[2]) > -fp.tau;
            kept |= in ? 1ull << it : 0ull;
            len += in ? 1u : 0u;
            slab |= in ? 1u << ((at >> 10) & 7u) : 0u;
            const bool xy = w.tm[0] <= w.tm[1];
            const float txy = xy ? w.tm[0] : w.tm[1];
            const bool iz = !(txy <= w.tm[2]), ix = xy && !iz, iy = !xy && !iz;
            if ((iz ? w.tm[2] : txy) > ry.t1) break;
            stepx |= ix ? 1ull << it : 0ull;
            stepy |= iy ? 1ull << it : 0ull;
            w.tm[0] = ix ? w.tm[0] + w.td[0] : w.tm[0];
            w.tm[1] = iy ? w.tm[1] + w.td[1] : w.tm[1];
            w.tm[2] = iz ? w.tm[2] + w.td[2] : w.tm[2];
            cf[0] += ix ? sf[0] : 0.0f;
            cf[1] += iy ? sf[1] : 0.0f;
            cf[2] += iz ? sf[2] : 0.0f;
            const uint32_t s1 = ix ? st[0] : 0u, s2 = iy ? st[1] : 0u, s3 = iz ? st[2] : 0u;
            at += s1 + s2 + s3;
            if ((at & kPlaceInside) != kPlaceInside) {
                leave();
                at -= 8u * (s1 + s2 + s3);
                exits |= (ix ? 0u : (iy ? 1u : 2u)) << (2 * (visit & 7));
                ++visit;
                len = slab = 0;
            }
        }
        leave();
        cnt = (uint32_t)__popcll(kept);
        // steps along each axis to the last cell
        const int nx = __popcll(stepx), ny = __popcll(stepy), nz = nvis - 1 - nx - ny;
        valid = started && visit < kMaxRuns && key_ok(k0[0]) && key_ok(k0[1]) && key_ok(k0[2]) &&
                key_ok(k0[0] + nx * w.stp[0]) && key_ok(k0[1] + ny * w.stp[1]) && key_ok(k0[2] + nz * w.stp[2]);
    }
    if (!valid) {
        cnt = 0;
        kept = 0ull;
        info[0] = info[1] = 0ull;
        visit = 0;
    }

    // the visited leaves' runs of kept cells into the block table: local rank of
    // each run inside its leaf
    uint32_t rent[kMaxRuns], rloc[kMaxRuns];
    unsigned long long key = key0;
#pragma unroll
    for (int q = 0; q < kMaxRuns; ++q) {
        rent[q] = kWalkTable;
        rloc[q] = 0;
        if (q <= visit) {
            const uint32_t run = (uint32_t)(info[q >> 2] >> (16 * (q & 3))) & 0xFFFFu;
            if (run) {
                // distinct keys <= runs of the block <= table size, so a free or
                // matching entry always exists; the probe bound is a safeguard
                uint32_t h = lds_hash(key);
                bool found = false;
                for (int probe = 0; probe < kWalkTable && !found; ++probe) {
                    unsigned long long k = t_key[h];
                    if (k == kEmptyKey) {
                        k = atomicCAS(&t_key[h], kEmptyKey, key);
                        if (k == kEmptyKey) {
                            t_list[atomicAdd(&s_n, 1u)] = (uint16_t)h;
                            k = key;
                        }
                    }
                    if (k == key) found = true;
                    else h = (h + 1) & (kWalkTable - 1);
                }
                if (found) {
                    rent[q] = h;
                    rloc[q] = atomicAdd(&t_cnt[h], run >> 8);
                    atomicOr(&t_slab[h >> 2], (run & 0xFFu) << (8u * (h & 3u)));
                } else {
                    atomicOr(&md.fs->frame_err.v, 1u);  // pairs of this run are dropped, frame rejected
                }
            }
            // the leaf that the ray enters next
            const uint32_t ax = (exits >> (2 * q)) & 3u;
            const unsigned long long one = ax == 0 ? 1ull << 36 : (ax == 1 ? 1ull << 18 : 1ull);
            const bool up = (ax == 0 ? sf[0] : (ax == 1 ? sf[1] : sf[2])) > 0.0f;
            key += up ? one : 0ull - one;
        }
    }
    const size_t r = (size_t)rblk * blockDim.x + tid, rcap = md.ray_cap;
    md.ray_bits[r] = kept | ((unsigned long long)visit << kVisitShift);
    if (cnt) {
        md.ray_bits[rcap + r] = stepx;
        md.ray_bits[2 * rcap + r] = stepy;
    }
    uint32_t wcnt = cnt;
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) wcnt += __shfl_xor(wcnt, d, 64);
    if (lane_id() == 0 && wcnt) atomicAdd(&s_pairs, wcnt);
    const uint32_t rejected_block = __syncthreads_count((i < fp.n) && !valid);
    if (tid == 0) {
        if (s_pairs) atomicAdd(&md.fs->pairs.v, s_pairs);
        if (rejected_block) atomicAdd(&md.fs->rejected.v, rejected_block);
    }
    // one staging lookup, one bucket reservation and one slab update per leaf of the block
    const uint32_t nloc = s_n;
    for (uint32_t e = tid; e < nloc; e += blockDim.x) {
        const uint32_t h = t_list[e];
        bool fresh;
        const uint32_t pos = stage_leaf_cas(md, t_key[h], &fresh);
        t_pos[h] = pos;
        if (pos != kNoPos) {
            t_cnt[h] = atomicAdd(&md.pos_count[pos], t_cnt[h]);
            atomicOr(&md.pos_slab[pos], (t_slab[h >> 2] >> (8u * (h & 3u))) & 0xFFu);
            if (fresh) t_fresh[atomicAdd(&s_nfresh, 1u)] = (uint16_t)h;
        } else {
            atomicOr(&md.fs->frame_err.v, 1u);
        }
    }
    __syncthreads();
    // wave 0 reserves the block's touched-list range now and writes it after
    // its own runs, so that the reservation's latency overlaps them
    const uint32_t nfresh = s_nfresh;
    uint32_t fresh_base = 0;
    if (tid == 0 && nfresh) fresh_base = atomicAdd(&md.fs->n_touched.v, nfresh);

    if (cnt) {
#pragma unroll
        for (int q = 0; q < kMaxRuns; ++q) {
            if (q > visit) continue;
            const uint32_t e = rent[q];
            md.ray_run[q * rcap + r] = e < (uint32_t)kWalkTable ? make_uint2(t_pos[e], t_cnt[e] + rloc[q])
                                                                : make_uint2(kNoPos, 0u);
        }
    }
    if (tid < 64 && nfresh) {
        const uint32_t base = __shfl(fresh_base, 0, 64);
        for (uint32_t e = tid; e < nfresh; e += 64) {
            const uint32_t h = t_fresh[e];
            md.touched[base + e] = t_pos[h];
            md.touched_key[base + e] = t_key[h];
        }
    }
}

__global__ __launch_bounds__(kWalkThreads) void k_ray_walk(FrameParams fp, MapDev md)
{
    __shared__ WalkShared ws;
    walk_block(fp, md, blockIdx.x, blockIdx.x, ws);
}

// Map of a block of a batched launch (frame of a multi-frame pass): the last i
// with start[i] <= blk.
__device__ __forceinline__ int batch_map(const int *start, int nmaps, int blk)
{
    int lo = 0, hi = nmaps;
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (start[mid] <= blk) lo = mid;
        else hi = mid;
    }
    return lo;
}

__global__ __launch_bounds__(kWalkThreads) void k_ray_walk_batch(MapBatch mb)
{
    __shared__ WalkShared ws;
    const int i = batch_map(mb.walk_start, mb.nmaps, blockIdx.x);
    const int blk = blockIdx.x - mb.walk_start[i];
    walk_block(mb.fps[i], mb.mds[i], blk, blk, ws);
}

// The rays of every frame of a multi-frame pass into one staging buffer.
__global__ __launch_bounds__(kWalkThreads) void k_ray_walk_pass(PassWalk pw, MapDev md)
{
    __shared__ WalkShared ws;
    const int f = batch_map(pw.blk_start, pw.nframes, blockIdx.x);
    walk_block(pw.fp[f], md, blockIdx.x - pw.blk_start[f], blockIdx.x, ws);
}

// Frame (within a multi-frame pass) of sort-key point index p.
__device__ __forceinline__ int pass_frame(const FrameParams &fp, uint32_t p)
{
    int f = 0;
#pragma unroll
    for (int q = 1; q < kPassFrames; ++q) f += (q < fp.nsub && p >= fp.sub_start[q]) ? 1 : 0;
    return f;
}

// ---------------------------------------------------------------------------
// 2. leaf planning
// ---------------------------------------------------------------------------

__device__ __forceinline__ void leaf_plan_range(const FrameParams &fp, const MapDev &md, uint32_t blk, uint32_t nblk)
{
    // work lists: the sorting leaf kernel splits a leaf with more pairs than
    // LDS holds into x-slab items and gives a wave leaves of up to
    // kWaveItemPairs pairs; the accumulating one takes every leaf whole
    const bool acc = accum_path(fp);
    const uint32_t slab_cap = (uint32_t)kLeafLdsPairs, wave_cap = acc ? (uint32_t)kAccWavePairs : (uint32_t)kWaveItemPairs;
    const uint32_t big_lim = acc ? 0xFFFFFFFFu : (md.slab_pairs > 0 ? min((uint32_t)md.slab_pairs, slab_cap) : slab_cap);
    const uint32_t small_lim = md.wave_pairs > 0 ? min((uint32_t)md.wave_pairs, wave_cap) : wave_cap;
    const uint32_t nt = md.fs->n_touched.v;
    const unsigned long long pused = md.st->pages_used;
    const uint32_t stride = nblk * blockDim.x;
    for (uint32_t jb = blk * blockDim.x; jb < nt; jb += stride) {
        const uint32_t j = jb + threadIdx.x;
        const bool act = j < nt;
        int32_t slot = -1;
        uint32_t npairs = 0, pos = 0, need = 0;
        unsigned long long key = kEmptyKey;
        uint4 occ[4] = {make_uint4(0u, 0u, 0u, 0u), make_uint4(0u, 0u, 0u, 0u), make_uint4(0u, 0u, 0u, 0u),
                        make_uint4(0u, 0u, 0u, 0u)};
        int pg[kLeafPages];
#pragma unroll
        for (int q = 0; q < kLeafPages; ++q) pg[q] = -1;
        if (act) {
            pos = md.touched[j];
            key = md.touched_key[j];
            slot = map_find(md, key);
            npairs = md.pos_count[pos];
            uint32_t have = 0;
            if (slot >= 0) {
                const int4 p0 = ((const int4 *)md.leaf_page)[2 * slot], p1 = ((const int4 *)md.leaf_page)[2 * slot + 1];
                pg[0] = p0.x; pg[1] = p0.y; pg[2] = p0.z; pg[3] = p0.w;
                pg[4] = p1.x; pg[5] = p1.y; pg[6] = p1.z; pg[7] = p1.w;
#pragma unroll
                for (int q = 0; q < 4; ++q) occ[q] = ((const uint4 *)md.leaf_occ)[(size_t)slot * 4 + q];
#pragma unroll
                for (int q = 0; q < kLeafPages; ++q) have |= (pg[q] >= 0 ? 1u : 0u) << q;
            }
            need = md.pos_slab[pos] & ~have & 0xFFu;
        }
        // a leaf with more pairs than the leaf kernel holds in LDS becomes one
        // work item per touched x-slab, or per range of its binned pairs
        const uint32_t tslabs = act ? md.pos_slab[pos] & 0xFFu : 0u;
        const bool big = act && npairs > big_lim;
        // the other leaves: one workgroup each, or one wave each if small
        const bool small = act && npairs <= small_lim;
        const bool med = act && !big && !small;
        // the larger workgroup and wave leaves are listed from the front of
        // their arrays, the smaller ones from the back
        const bool medf = med && npairs > min(big_lim, slab_cap) / 2, medb = med && !medf;
        const bool smallf = small && npairs > small_lim / 4, smallb = small && !smallf;
        const uint32_t nparts = !big ? 0u
                                : md.binned ? (npairs + (uint32_t)kRangePairs - 1u) / (uint32_t)kRangePairs
                                            : (uint32_t)__popc(tslabs);
        // eight reservations with six atomics in flight together (two list
        // counters share each 64-bit word)
        const uint32_t want[4] = {(act && slot < 0) ? 1u : 0u, (uint32_t)__popc(need), npairs,
                                  nparts};
        uint32_t incl[4], total[4], base[4] = {0u, 0u, 0u, 0u};
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            incl[q] = wave_incl_scan(want[q]);
            total[q] = __shfl(incl[q], 63, 64);
        }
        const uint32_t mincl = wave_incl_scan(medf ? 1u : 0u), sincl = wave_incl_scan(smallf ? 1u : 0u);
        const uint32_t mincb = wave_incl_scan(medb ? 1u : 0u), sincb = wave_incl_scan(smallb ? 1u : 0u);
        const unsigned long long lt = ((unsigned long long)__shfl(sincl, 63, 64) << 32) | __shfl(mincl, 63, 64);
        const unsigned long long ltb = ((unsigned long long)__shfl(sincb, 63, 64) << 32) | __shfl(mincb, 63, 64);
        unsigned long long lbase = 0, lbaseb = 0;
        if (lane_id() == 63) {
            if (total[0]) base[0] = atomicAdd(&md.fs->new_leaves.v, total[0]);
            if (total[1]) base[1] = atomicAdd(&md.fs->new_pages.v, total[1]);
            if (total[2]) base[2] = atomicAdd(&md.fs->pair_cursor.v, total[2]);
            if (total[3]) base[3] = atomicAdd(&md.fs->work_big.v, total[3]);
            if (lt) lbase = atomicAdd((unsigned long long *)&md.fs->n_lists, lt);
            if (ltb) lbaseb = atomicAdd((unsigned long long *)&md.fs->n_lists_tail, ltb);
        }
        uint32_t got[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) got[q] = __shfl(base[q], 63, 64) + incl[q] - want[q];
        const unsigned long long lb = __shfl(lbase, 63, 64), lbb = __shfl(lbaseb, 63, 64);
        const uint32_t newleaf = got[0], pbase = got[1], bstart = got[2], ibase = got[3];
        const uint32_t last = md.hmask;  // the item arrays of the lists hold hmask + 1 entries
        LeafItem *dst = nullptr;
        if (medf) dst = &md.items[(uint32_t)lb + mincl - 1u];
        if (smallf) dst = &md.items_small[(uint32_t)(lb >> 32) + sincl - 1u];
        if (medb) dst = &md.items[last - ((uint32_t)lbb + mincb - 1u)];
        if (smallb) dst = &md.items_small[last - ((uint32_t)(lbb >> 32) + sincb - 1u)];
        if (big) {
            // the leaf's work items sit at ibase .. ibase + nparts - 1, its item at
            // ibase; every work entry below work_cap is written, so the leaf
            // kernel never reads an unwritten one (a frame that overflows the
            // work list is not applied)
            if (ibase < md.work_cap) dst = &md.items_big[ibase];
            uint32_t left = tslabs;
            for (uint32_t r = 0; r < nparts; ++r) {
                const int part = md.binned ? (int)r : __ffs(left) - 1;
                left &= left - 1u;
                if (ibase + r < md.work_cap) md.work[ibase + r] = make_int2((int)ibase, part);
                else atomicOr(&md.fs->frame_err.v, 1u);
            }
        }
        if (act) {
            uint32_t r = 0;
#pragma unroll
            for (int q = 0; q < kLeafPages; ++q)
                if ((need >> q) & 1u) pg[q] = (int)(pused + pbase + r++);
            md.pos_pages[2 * pos] = make_int4(pg[0], pg[1], pg[2], pg[3]);
            md.pos_pages[2 * pos + 1] = make_int4(pg[4], pg[5], pg[6], pg[7]);
            md.pos_plan[pos] = make_int4(slot, slot < 0 ? (int)newleaf : -1, (int)bstart, 0);
        }
        if (dst) {
            // the leaf kernel's item: header, pages, occupancy before this frame
            uint4 *it = (uint4 *)dst;
            it[0] = make_uint4(pos, npairs, bstart, (uint32_t)(slot >= 0 ? slot : -1 - (int)newleaf));
            it[1] = make_uint4(tslabs, 0u, (uint32_t)key, (uint32_t)(key >> 32));
            it[2] = make_uint4((uint32_t)pg[0], (uint32_t)pg[1], (uint32_t)pg[2], (uint32_t)pg[3]);
            it[3] = make_uint4((uint32_t)pg[4], (uint32_t)pg[5], (uint32_t)pg[6], (uint32_t)pg[7]);
#pragma unroll
            for (int q = 0; q < 4; ++q) it[4 + q] = occ[q];
        }
    }
}

__global__ __launch_bounds__(256) void k_leaf_plan(FrameParams fp, MapDev md)
{
    leaf_plan_range(fp, md, blockIdx.x, gridDim.x);
}

__global__ __launch_bounds__(256) void k_leaf_plan_batch(MapBatch mb)
{
    const int i = batch_map(mb.plan_first, mb.nmaps, blockIdx.x);
    leaf_plan_range(mb.fps[i], mb.mds[i], blockIdx.x - mb.plan_first[i], mb.plan_first[i + 1] - mb.plan_first[i]);
}

// ---------------------------------------------------------------------------
// 3. pairs into the leaves' buckets
// ---------------------------------------------------------------------------

// Softmax of every point's logits (max-subtracted), one lane per point, into rows
// of soft_stride(K) floats (padded with zeros) in the wave combine's descriptor
// buffer, which frames of class rows do not use (16 bytes x at least 10 cells per
// point hold 32 classes).  Formed here once per point, an observation costs the
// combine one row of additions; formed there, once per observation (9 per point),
// its exponentials and divisions bound the leaf kernel.  65,536 rays, 20 classes:
// leaf kernel 96 -> 43 us (vector rows included) for 4 us more in this stage; 131,071
// rays: 200 -> 65 us for 7.
__host__ __device__ inline int soft_stride(int K) { return (K + 3) & ~3; }

__host__ __device__ inline bool soft_rows(const FrameParams &fp)
{
    return fp.sem_kind == SLIM_IN_LOGIT_F32 && !fp.last && fp.K <= 32;
}

__device__ __forceinline__ void softmax_rows_range(const FrameParams &fp, const MapDev &md, uint32_t blk, uint32_t nblk)
{
    constexpr int KMAX = 32;
    const int K = fp.K, stride = soft_stride(K);
    for (uint32_t i = blk * blockDim.x + threadIdx.x; i < (uint32_t)fp.n; i += nblk * blockDim.x) {
        const float *row = (const float *)fp.sem + (size_t)i * K;
        float4 *out = (float4 *)((float *)md.vox_list + (size_t)i * stride);
        float x[KMAX];
#pragma unroll
        for (int k = 0; k < KMAX; ++k) x[k] = k < K ? row[k] : 0.0f;
        float mx = x[0];
#pragma unroll
        for (int k = 1; k < KMAX; ++k)
            if (k < K) mx = fmaxf(mx, x[k]);
        float den = 0.0f;
#pragma unroll
        for (int k = 0; k < KMAX; ++k)
            if (k < K) {
                x[k] = expf(x[k] - mx);
                den += x[k];
            }
#pragma unroll
        for (int v = 0; v < KMAX / 4; ++v)
            if (4 * v < K) out[v] = make_float4(x[4 * v] / den, x[4 * v + 1] / den, x[4 * v + 2] / den, x[4 * v + 3] / den);
    }
}

// Writes the pairs of rays blk * blockDim.x + [0, blockDim.x) of a frame to their
// leaves' buckets, one lane per ray: the recorded walk again, each kept cell's key
// and distance (and the ray's label) at the bucket's start + rank.  All of a ray's
// runs and bucket starts are read before the walk, side by side.  Written straight
// to the buckets, the pairs pass through memory once; as 16-byte records in walk
// order, bucketed by a launch of their own, an 8-sweep pass took 94 us for the walk
// and 56 for the bucketing, now 70 and 52; 16 maps 103 and 33, now 52 and 38.
__device__ __forceinline__ void ray_emit_block(const FrameParams &fp, const MapDev &md, int blk, int rblk)
{
    const int i = blk * blockDim.x + threadIdx.x;
    if (i >= fp.n) return;
    const size_t r = (size_t)rblk * blockDim.x + threadIdx.x, rcap = md.ray_cap;
    const bool labels = fp.K > 0 && accum_path(fp);  // (the sorting leaf kernels read labels by point index)
    // everything that does not depend on another read is requested first: the bits,
    // the point, the label and the runs of the first three leaves (few rays visit
    // more; a run that the walk did not write is not used)
    constexpr int kFirst = 3;
    const unsigned long long bits = md.ray_bits[r], stepx = md.ray_bits[rcap + r], stepy = md.ray_bits[2 * rcap + r];
    uint2 run[kMaxRuns];
#pragma unroll
    for (int q = 0; q < kFirst; ++q) run[q] = md.ray_run[q * rcap + r];
    const int32_t lab = labels ? ((const int32_t *)fp.sem)[i] : 0;
    float x, y, z;
    load_point(fp, i, x, y, z);
    const unsigned long long kept = bits & ((1ull << kVisitShift) - 1ull);
    if (!kept) return;
    const int last = (int)(bits >> kVisitShift);
    uint32_t dst[kMaxRuns];
#pragma unroll
    for (int q = 0; q < kMaxRuns; ++q) {
        if (q >= kFirst) run[q] = q <= last ? md.ray_run[q * rcap + r] : make_uint2(kNoPos, 0u);
        dst[q] = q <= last && run[q].x != kNoPos ? (uint32_t)md.pos_plan[run[q].x].z + run[q].y : kNoPos;
    }
    Ray ry;
    make_ray(fp, x, y, z, ry);
    float cf[3], sf[3];
    uint32_t at = 0, st[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const float s = fmaf(ry.t0, ry.u[a], fp.t[a]);  // as walk_start
        const int c = (int)floorf(s / fp.vs), up = ry.u[a] > 0.0f ? 1 : (ry.u[a] < 0.0f ? -1 : 0);
        cf[a] = (float)c;
        sf[a] = (float)up;
        at |= (uint32_t)(((fp.a[a] + c) & 7) + 8) << (10 - 5 * a);
        st[a] = (uint32_t)up << (10 - 5 * a);
    }
    const uint32_t pid = fp.pid_base + (uint32_t)i;
    // (the batched forms read the frame and the map from memory, which the stores below
    // may alias as far as the compiler knows: read before the loop, not at every cell.
    // 8 maps of 3,000 points 25 -> 21 us, with no more workgroups than rays fill 10.5)
    const float vs = fp.vs, tau = fp.tau;
    uint2 *const kv = md.srt_kv;
    int32_t *const labs = md.srt_lab;
    uint32_t d = dst[0];
    int visit = 0;
    for (int vi = 0; (kept >> vi) != 0ull; ++vi) {
        if (((kept >> vi) & 1ull) && d != kNoPos) {
            const float sd = ray_sdf(vs, ry, cf[0], cf[1], cf[2]);
            const uint32_t voff = ((at >> 4) & 0x1C0u) | ((at >> 2) & 0x38u) | (at & 7u);
            kv[d] = make_uint2((voff << kPidBits) | pid, __float_as_uint(fminf(sd, tau)));
            if (labels) labs[d] = lab;
            ++d;
        }
        const bool ix = (stepx >> vi) & 1ull, iy = (stepy >> vi) & 1ull, iz = !ix && !iy;
        cf[0] += ix ? sf[0] : 0.0f;
        cf[1] += iy ? sf[1] : 0.0f;
        cf[2] += iz ? sf[2] : 0.0f;
        const uint32_t step = ix ? st[0] : (iy ? st[1] : st[2]);
        at += step;
        if ((at & kPlaceInside) != kPlaceInside) {
            at -= 8u * step;
            ++visit;
            d = kNoPos;
#pragma unroll
            for (int q = 1; q < kMaxRuns; ++q) d = q == visit ? dst[q] : d;
        }
    }
}

// SOFT: frames of logit rows (apart, so that the others keep their registers)
template <bool SOFT>
__global__ __launch_bounds__(kWalkThreads) void k_ray_emit(FrameParams fp, MapDev md)
{
    if constexpr (SOFT) softmax_rows_range(fp, md, blockIdx.x, gridDim.x);
    const int n = (fp.n + kWalkThreads - 1) / kWalkThreads;
    for (int b = blockIdx.x; b < n; b += gridDim.x) ray_emit_block(fp, md, b, b);
}

__global__ __launch_bounds__(kWalkThreads) void k_ray_emit_pass(PassWalk pw, MapDev md)
{
    const int f = batch_map(pw.blk_start, pw.nframes, blockIdx.x);
    ray_emit_block(pw.fp[f], md, blockIdx.x - pw.blk_start[f], blockIdx.x);
}

// Blocks blk, blk + nblk, ... of a map's rays.
__device__ __forceinline__ void ray_emit_range(const FrameParams &fp, const MapDev &md, uint32_t blk, uint32_t nblk)
{
    if (soft_rows(fp)) softmax_rows_range(fp, md, blk, nblk);
    const uint32_t n = ((uint32_t)fp.n + kWalkThreads - 1) / kWalkThreads;
    for (uint32_t b = blk; b < n; b += nblk) ray_emit_block(fp, md, (int)b, (int)b);
}

__global__ __launch_bounds__(kWalkThreads) void k_ray_emit_batch(MapBatch mb)
{
    const int i = batch_map(mb.bucket_first, mb.nmaps, blockIdx.x);
    ray_emit_range(mb.fps[i], mb.mds[i], blockIdx.x - mb.bucket_first[i], mb.bucket_first[i + 1] - mb.bucket_first[i]);
}

// ---------------------------------------------------------------------------
// 3'. binning of large leaves
// ---------------------------------------------------------------------------
//
// A leaf with more pairs than the sorting leaf kernel holds in LDS is shared by
// several workgroups.  Without binning each of them takes an x-slab and reads
// every pair of the leaf to find its own, twice when they are many: at 640x480
// pixels and 2 cm voxels the 206 leaves touched hold up to 61,000 pairs, and
// those reads were most of the leaf kernel's time.  These two kernels group the
// pairs by voxel offset first, a workgroup per range of kRangePairs of a bucket's
// pairs: k_leaf_count counts each range's offsets, k_leaf_bin forms the leaf's
// bin starts from its ranges' counts (no atomics between workgroups) and moves
// the range's pairs to their bins.  The leaf kernel's items are then ranges of
// whole bins of about that many pairs, each reading its own pairs once.
// Bound by the pairs' bytes (8 read twice, 8 written); the order inside a bin is
// arbitrary, as it is without binning.  That frame: leaf kernel 532 -> 65 us, these
// two kernels 9 and 18 us.

// 16-bit counts of range u's offsets, two to a word, in the sorted keys' buffer
// (free until the leaf kernel).  A large leaf has more than 512 pairs, so the
// ranges are at most pairs / 1536 + pairs / 512 and their 1 KB rows fit.
constexpr int kRangeBatch = kRangePairs / 256;
__device__ __forceinline__ uint32_t *range_counts(const MapDev &md, uint32_t u) { return md.pair_key + (size_t)u * 256; }

__global__ __launch_bounds__(256) void k_leaf_count(MapDev md)
{
    __shared__ uint32_t hist[kLeafVoxels];
    const uint32_t nbig = min(md.fs->work_big.v, md.work_cap), tid = threadIdx.x;
    for (uint32_t u = blockIdx.x; u < nbig; u += gridDim.x) {
        const int2 it = md.work[u];
        const LeafItem &item = md.items_big[it.x];
        const uint32_t t0 = (uint32_t)it.y * kRangePairs, n = min(item.n - t0, (uint32_t)kRangePairs);
        const uint2 *kv = md.srt_kv + item.bstart + t0;
        hist[tid] = 0u;
        hist[tid + 256] = 0u;
        uint32_t key[kRangeBatch];
#pragma unroll
        for (int q = 0; q < kRangeBatch; ++q) key[q] = q * 256 + tid < n ? kv[q * 256 + tid].x : 0u;
        __syncthreads();
#pragma unroll
        for (int q = 0; q < kRangeBatch; ++q)
            if (q * 256 + tid < n) atomicAdd(&hist[key[q] >> kPidBits], 1u);
        __syncthreads();
        range_counts(md, u)[tid] = hist[2 * tid] | (hist[2 * tid + 1] << 16);
        __syncthreads();
    }
}

__global__ __launch_bounds__(256) void k_leaf_bin(MapDev md)
{
    __shared__ uint32_t cur[kLeafVoxels], wsum[4];
    const uint32_t nbig = min(md.fs->work_big.v, md.work_cap), tid = threadIdx.x;
    for (uint32_t u = blockIdx.x; u < nbig; u += gridDim.x) {
        const int2 it = md.work[u];
        const LeafItem &item = md.items_big[it.x];
        const uint32_t c = (uint32_t)it.y, t0 = c * kRangePairs, n = min(item.n - t0, (uint32_t)kRangePairs);
        const uint32_t nranges = (item.n + kRangePairs - 1) / kRangePairs;
        const uint2 *kv = md.srt_kv + item.bstart + t0;
        uint2 e[kRangeBatch];
#pragma unroll
        for (int q = 0; q < kRangeBatch; ++q) e[q] = q * 256 + tid < n ? kv[q * 256 + tid] : make_uint2(0u, 0u);
        // offsets 2 tid and 2 tid + 1: their pairs in the leaf, and in the ranges before this one
        uint32_t a = 0, b = 0, a0 = 0, b0 = 0;
#pragma unroll 8
        for (uint32_t r = 0; r < nranges; ++r) {
            const uint32_t w = range_counts(md, (uint32_t)it.x + r)[tid];
            if (r == c) {
                a0 = a;
                b0 = b;
            }
            a += w & 0xFFFFu;
            b += w >> 16;
        }
        uint32_t total;
        const uint32_t start = block_excl_scan(a + b, wsum, &total);
        if (c == 0) ((uint2 *)(md.srt_lab + item.bstart + (item.bstart & 1u)))[tid] = make_uint2(start, start + a);
        cur[2 * tid] = start + a0;
        cur[2 * tid + 1] = start + a + b0;
        __syncthreads();
#pragma unroll
        for (int q = 0; q < kRangeBatch; ++q)
            if (q * 256 + tid < n) {
                const uint32_t p = item.bstart + atomicAdd(&cur[e[q].x >> kPidBits], 1u);
                md.tmp_key[p] = e[q].x;
                md.tmp_tsdf[p] = __uint_as_float(e[q].y);
            }
        __syncthreads();
    }
}

// ---------------------------------------------------------------------------
// 4. per-leaf sort, reduce and conjugate combine
// ---------------------------------------------------------------------------

struct LeafShared {
    uint32_t a_key[kLeafLdsPairs], b_key[kLeafLdsPairs];  // sorted / binned pairs
    float a_val[kLeafLdsPairs], b_val[kLeafLdsPairs];
    uint32_t hist[kLeafVoxels], bin0[kLeafVoxels], cur[kLeafVoxels];
    uint32_t touch[kMaskWords], occ0[kMaskWords], wsum[4];
    int pages[kLeafPages];
    uint32_t chunk_end, uold, unew;
    uint32_t stash_n;         // pairs of an x-slab item's own offsets (kept in a_key/a_val while they fit)
    uint32_t item[32];        // the current block item
};

__device__ __forceinline__ float load_emb(const FrameParams &fp, uint32_t pid, int comp)
{
    const size_t idx = (size_t)pid * fp.L + comp;
    return fp.sem_kind == SLIM_IN_EMB_BF16 ? __uint_as_float((uint32_t)((const uint16_t *)fp.sem)[idx] << 16)
                                           : ((const float *)fp.sem)[idx];
}

__device__ __forceinline__ float wave_max(float v)
{
    for (int d = 32; d > 0; d >>= 1) v = fmaxf(v, __shfl_xor(v, d, 64));
    return v;
}

__device__ __forceinline__ float wave_sum(float v)
{
    for (int d = 32; d > 0; d >>= 1) v += __shfl_xor(v, d, 64);
    return v;
}

// Orders the wave's LDS accesses before the barrier ahead of those after it
// (lanes of one wave exchanging data through LDS).
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Eq. (1)-(2) with unit weights.  Each truncated distance is taken as the
// fixed-point integer q = rint(tsdf 2^k), where 2^k is the largest power of two
// with tau 2^k <= 2^40, and a frame's q are summed in 64-bit integers: the sum
// is exact, so it does not depend on the order of the observations, and it
// differs from the real sum of the distances by at most n 2^-(k+1) (n
// observations: 2^-42 tau each), far inside the tolerance.  The running mean
// is formed in binary64 and rounded once to the stored binary32.
struct FixScale {
    float s;     // 2^k
    double inv;  // 2^-k
};

__device__ __forceinline__ FixScale fix_scale(const FrameParams &fp)
{
    int e;
    (void)frexpf(fp.tau, &e);  // tau < 2^e
    return {ldexpf(1.0f, 40 - e), ldexp(1.0, e - 40)};
}

__device__ __forceinline__ long long fix_q(float tsdf, float s) { return __float2ll_rn(tsdf * s); }

__device__ __forceinline__ long long tsdf_sum(const float *vals, uint32_t n, float s)
{
    long long sum = 0;
    for (uint32_t q = 0; q < n; ++q) sum += fix_q(vals[q], s);
    return sum;
}

__device__ __forceinline__ float tsdf_mean(float D0, float W0, float W1, long long sum, double inv)
{
    return (float)(((double)W0 * (double)D0 + (double)sum * inv) / (double)W1);
}

// One voxel, one lane: its n observations sit at keys[0..n) / vals[0..n) in
// point order.  Closed set with probability rows (or the softmax of logit rows,
// formed once per point by softmax_rows_range) and K <= KMAX classes in
// registers.  Rows (16-byte aligned ones) and the record move as 16-byte
// vectors.
template <int KMAX>
__device__ __forceinline__ void combine_lane(const FrameParams &fp, const MapDev &md, const uint32_t *keys,
                                             const float *vals, uint32_t n, long long rec, bool existed)
{
    static_assert(KMAX > 0 && KMAX % 4 == 0, "rows of at least one class, in whole vectors");
    constexpr int NV = (2 + KMAX + 3) / 4;
    const int nv = md.rec_stride / 4, K = fp.K;
    const bool soft = fp.sem_kind == SLIM_IN_LOGIT_F32;
    const float *rows = soft ? (const float *)md.vox_list : (const float *)fp.sem;
    const int stride = soft ? soft_stride(K) : K;
    const bool vec = (stride & 3) == 0 && ((uintptr_t)rows & 15u) == 0;
    // up to 16 classes the record is requested first, so its round trip
    // overlaps the rows (more would spill registers)
    constexpr bool early = KMAX <= 16;
    float4 *R = (float4 *)(md.vox + (size_t)rec * md.rec_stride);
    float r[4 * NV];
    auto load_record = [&]() {
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            const float4 x = (existed && v < nv) ? R[v] : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            r[4 * v + 0] = x.x;
            r[4 * v + 1] = x.y;
            r[4 * v + 2] = x.z;
            r[4 * v + 3] = x.w;
        }
    };
    if constexpr (early) load_record();
    float acc[KMAX];
#pragma unroll
    for (int k = 0; k < KMAX; ++k) acc[k] = 0.0f;
    // one row per lane at a time, added in point order: four workgroups per CU hide
    // more than two rows and three workgroups do (131,071 rays, 20 classes: 56 and
    // 65 us)
    for (uint32_t q = 0; q < n; ++q) {
        const float *row = rows + (size_t)(keys[q] & kPidMask) * stride;
        float x[KMAX];
        if (vec) {
#pragma unroll
            for (int v = 0; v < KMAX / 4; ++v) {
                const float4 f = 4 * v < K ? ((const float4 *)row)[v] : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
                x[4 * v + 0] = f.x;
                x[4 * v + 1] = f.y;
                x[4 * v + 2] = f.z;
                x[4 * v + 3] = f.w;
            }
        } else {
#pragma unroll
            for (int k = 0; k < KMAX; ++k) x[k] = k < K ? row[k] : 0.0f;
        }
#pragma unroll
        for (int k = 0; k < KMAX; ++k) acc[k] += x[k];
    }
    if constexpr (!early) load_record();
    // Eq. (1)-(2) with unit weights
    const float nf = (float)n, W0 = r[1], W1 = W0 + nf;
    const FixScale fx = fix_scale(fp);
    r[0] = tsdf_mean(r[0], W0, W1, tsdf_sum(vals, n, fx.s), fx.inv);
    r[1] = W1;
    // Eq. (6): concentrations grow by the expected class counts
#pragma unroll
    for (int k = 0; k < KMAX; ++k)
        if (k < K) r[2 + k] += acc[k];
#pragma unroll
    for (int v = 0; v < NV; ++v)
        if (v < nv) R[v] = make_float4(r[4 * v + 0], r[4 * v + 1], r[4 * v + 2], r[4 * v + 3]);
}

// Raw words of one lane's share of an open-set row: V / 2 words of bf16
// pairs, or V floats.
template <int V, bool BF>
struct RowWords {
    static constexpr int W = BF ? V / 2 : V;
    uint32_t w[W];
};

template <int V, bool BF>
__device__ __forceinline__ void load_row_words(const FrameParams &fp, uint32_t pid, int lane, RowWords<V, BF> &r)
{
    constexpr int W = RowWords<V, BF>::W;
    const uint32_t *row = (const uint32_t *)fp.sem + (size_t)pid * (64 * W) + lane * W;
    if constexpr (W % 4 == 0) {
#pragma unroll
        for (int c = 0; c < W / 4; ++c) {
            const uint4 u = ((const uint4 *)row)[c];
            r.w[4 * c] = u.x;
            r.w[4 * c + 1] = u.y;
            r.w[4 * c + 2] = u.z;
            r.w[4 * c + 3] = u.w;
        }
    } else if constexpr (W == 2) {
        const uint2 u = *(const uint2 *)row;
        r.w[0] = u.x;
        r.w[1] = u.y;
    } else {
#pragma unroll
        for (int c = 0; c < W; ++c) r.w[c] = row[c];
    }
}

template <int V, bool BF>
__device__ __forceinline__ void unpack_row(const RowWords<V, BF> &r, float (&z)[V])
{
    if constexpr (BF) {
#pragma unroll
        for (int e = 0; e < V / 2; ++e) {
            z[2 * e] = __uint_as_float(r.w[e] << 16);
            z[2 * e + 1] = __uint_as_float(r.w[e] & 0xFFFF0000u);
        }
    } else {
#pragma unroll
        for (int e = 0; e < V; ++e) z[e] = __uint_as_float(r.w[e]);
    }
}

// Sum over the wave of one 64-bit integer per lane (every lane gets the sum).
__device__ __forceinline__ long long wave_sum_i64(long long x)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const int lo = __shfl_xor((int)(unsigned long long)x, o, 64);
        const int hi = __shfl_xor((int)((unsigned long long)x >> 32), o, 64);
        x += (long long)(((unsigned long long)(uint32_t)hi << 32) | (uint32_t)lo);
    }
    return x;
}

// Open set with L = 64 V, one wave per voxel: lane l owns components l V ..
// l V + V - 1, so one observation's row is one or two wide loads per lane and
// many observations are in flight at once.  Sums as in combine_wave: the
// shifted sums in observation order, the distance sum as exact integers.  The
// point index of each row is read from its lane as a wave-uniform value, and
// a batch's rows are all requested before any is unpacked (a batch's slots
// past the last observation load that observation's row again and add
// nothing).
// kl0, vl0: point index and distance of observation `lane` (lanes below
// min(n, 64)), 0 elsewhere; the caller may have requested them ahead.
// V consecutive floats of a record (8-byte aligned for even V), read or
// written as pairs.  A record is read and written once per frame while the
// rows of the voxel's observations are read again by the neighbouring voxels:
// the record accesses are marked streaming (non-temporal), so that they do not
// push the rows out of L2.
typedef float f32x2_t __attribute__((ext_vector_type(2)));

template <int V>
__device__ __forceinline__ void rec_load(const float *p, float (&o)[V])
{
    if constexpr (V % 2 == 0) {
#pragma unroll
        for (int c = 0; c < V / 2; ++c) {
            const f32x2_t f = __builtin_nontemporal_load((const f32x2_t *)p + c);
            o[2 * c] = f.x;
            o[2 * c + 1] = f.y;
        }
    } else {
#pragma unroll
        for (int i = 0; i < V; ++i) o[i] = __builtin_nontemporal_load(p + i);
    }
}

template <int V>
__device__ __forceinline__ void rec_store(float *p, const float (&o)[V])
{
    if constexpr (V % 2 == 0) {
#pragma unroll
        for (int c = 0; c < V / 2; ++c) {
            f32x2_t f;
            f.x = o[2 * c];
            f.y = o[2 * c + 1];
            __builtin_nontemporal_store(f, (f32x2_t *)p + c);
        }
    } else {
#pragma unroll
        for (int i = 0; i < V; ++i) __builtin_nontemporal_store(o[i], p + i);
    }
}

template <int V, bool BF>
__device__ __forceinline__ void combine_wave_vec_t(const FrameParams &fp, const MapDev &md, const uint32_t *keys,
                                                   const float *vals, uint32_t n, long long rec, bool existed,
                                                   uint32_t kl0, float vl0)
{
    // observations per batch of rows: fewer for L = 256 (few observations per
    // voxel), whose kernel runs more waves instead; a batch never crosses a
    // group of 64 observations (the lanes' point indices are reloaded there)
    constexpr int B = V >= 16 || V == 4 ? 4 : 8;
    static_assert(64 % B == 0, "batches tile the 64-observation groups");
    const int lane = lane_id();
    float *R = md.vox + (size_t)rec * md.rec_stride;
    // (up to 8 components per lane) the voxel's record is requested with the rows
    constexpr bool early = V <= 8;
    uint32_t kl = kl0;
    float vl = vl0;
    float *M = R + 2 + lane * V, *Bt = R + 2 + 64 * V + lane * V;
    float m0[early ? V : 1], b0[early ? V : 1];
    float W0 = 0.0f, D0 = 0.0f;
    if constexpr (early) {
        W0 = existed ? R[1] : 0.0f;
        D0 = existed ? R[0] : 0.0f;
        if (existed) {
            rec_load<V>(M, m0);
            rec_load<V>(Bt, b0);
        } else {
#pragma unroll
            for (int i = 0; i < V; ++i) {
                m0[i] = 0.0f;
                b0[i] = 0.0f;
            }
        }
    }
    float z0[V], s1[V], s2[V];
    {
        RowWords<V, BF> r0;
        load_row_words<V, BF>(fp, (uint32_t)__builtin_amdgcn_readlane((int)kl, 0), lane, r0);
        unpack_row<V, BF>(r0, z0);
    }
#pragma unroll
    for (int i = 0; i < V; ++i) {
        s1[i] = 0.0f;
        s2[i] = 0.0f;
    }
    // fixed-point distance sum (Eq. (1)-(2)): each lane converts its own
    // observations, one wave-wide sum at the end
    const FixScale fx = fix_scale(fp);
    long long sum_t = 0;
    // batches of B observations from observation 0 (whose difference is 0);
    // a batch never crosses a group of 64 observations
    for (uint32_t q = 0; q < n; q += B) {
        if ((q & 63u) == 0) {
            if (q > 0) {
                kl = q + (uint32_t)lane < n ? keys[q + lane] & kPidMask : 0u;
                vl = q + (uint32_t)lane < n ? vals[q + lane] : 0.0f;
            }
            if (q + (uint32_t)lane < n) sum_t += fix_q(vl, fx.s);
        }
        RowWords<V, BF> raw[B];
#pragma unroll
        for (int b = 0; b < B; ++b) {
            const uint32_t t = min(q + (uint32_t)b, n - 1u);
            load_row_words<V, BF>(fp, (uint32_t)__builtin_amdgcn_readlane((int)kl, (int)(t & 63u)), lane, raw[b]);
        }
#pragma unroll
        for (int b = 0; b < B; ++b)
            if (q + b > 0 && q + b < n) {
                float z[V];
                unpack_row<V, BF>(raw[b], z);
#pragma unroll
                for (int i = 0; i < V; ++i) {
                    const float d = z[i] - z0[i];
                    s1[i] += d;
                    s2[i] += d * d;
                }
            }
    }
    sum_t = wave_sum_i64(sum_t);
    // Eqs. (11)-(14) with lambda = W, nu = W / 2
    const float nf = (float)n;
    if constexpr (!early) {
        W0 = existed ? R[1] : 0.0f;
        D0 = existed ? R[0] : 0.0f;
    }
    const float W1 = W0 + nf;
    const float inv_n = 1.0f / nf, inv_w1 = 1.0f / W1;
    const float cross = W0 * nf * inv_w1;
    float mo[V], bo[V];
#pragma unroll
    for (int i = 0; i < V; ++i) {
        const float zbar = z0[i] + s1[i] * inv_n;
        const float scat = fmaxf(s2[i] - s1[i] * s1[i] * inv_n, 0.0f);
        float mi, bi;
        if constexpr (early) {
            mi = m0[i];
            bi = b0[i];
        } else {
            mi = existed ? M[i] : 0.0f;
            bi = existed ? Bt[i] : 0.0f;
        }
        const float dm = zbar - mi;
        bo[i] = bi + 0.5f * scat + cross * dm * dm * 0.5f;
        mo[i] = (W0 * mi + nf * zbar) * inv_w1;
    }
    rec_store<V>(Bt, bo);
    rec_store<V>(M, mo);
    if (lane == 0) {
        R[0] = tsdf_mean(D0, W0, W1, sum_t, fx.inv);
        R[1] = W1;
    }
}

template <int V>
__device__ __forceinline__ void combine_wave_vec(const FrameParams &fp, const MapDev &md, const uint32_t *keys,
                                                 const float *vals, uint32_t n, long long rec, bool existed,
                                                 uint32_t kl0, float vl0)
{
    if constexpr (V >= 2) {
        if (fp.sem_kind == SLIM_IN_EMB_BF16) {
            combine_wave_vec_t<V, true>(fp, md, keys, vals, n, rec, existed, kl0, vl0);
            return;
        }
    }
    combine_wave_vec_t<V, false>(fp, md, keys, vals, n, rec, existed, kl0, vl0);
}

template <int V>
__device__ __forceinline__ void combine_wave_vec(const FrameParams &fp, const MapDev &md, const uint32_t *keys,
                                                 const float *vals, uint32_t n, long long rec, bool existed)
{
    const uint32_t lane = (uint32_t)lane_id();
    combine_wave_vec<V>(fp, md, keys, vals, n, rec, existed, lane < n ? keys[lane] & kPidMask : 0u,
                        lane < n ? vals[lane] : 0.0f);
}

// Components per lane of the general wave combine (a row of up to 64 J
// components), and observations whose rows are in flight at once.
constexpr int kWaveComps = 16;
constexpr int wave_batch(int j) { return j <= 2 ? 8 : 4; }

// One voxel, one wave: lane l owns components l, l + 64, ... of the open-set
// statistics (L <= 64 J) or of the class counts (K <= 64 J).  The rows of
// kWaveBatch observations are loaded before any is used; up to two components per
// lane the record is requested before the rows.  Open set: one pass
// over the observations with sums shifted by the first one, s1 = sum (z - z_0),
// s2 = sum (z - z_0)^2, so the batch mean is z_0 + s1 / n and the scatter
// s2 - s1^2 / n (the shift keeps the subtraction well conditioned).
template <int J>
__device__ __forceinline__ void combine_wave(const FrameParams &fp, const MapDev &md, const uint32_t *keys,
                                             const float *vals, uint32_t n, long long rec, bool existed)
{
    constexpr int kWaveBatch = wave_batch(J);
    constexpr bool early = J <= 2;
    const int lane = lane_id();
    const bool open = fp.L > 0;
    const int C = open ? fp.L : fp.K;
    float *R = md.vox + (size_t)rec * md.rec_stride;
    float s1[J], s2[J];
#pragma unroll
    for (int j = 0; j < J; ++j) {
        s1[j] = 0.0f;
        s2[j] = 0.0f;
    }
    // the point indices of 64 observations at a time, one per lane; a batch's
    // indices come from the lanes, so its rows do not wait on a load of them
    // (batches start at multiples of their size and never cross a window)
    uint32_t kl = (uint32_t)lane < n ? keys[lane] & kPidMask : 0u;
    const float vl = (uint32_t)lane < n ? vals[lane] : 0.0f;
    const float W0 = existed ? R[1] : 0.0f, D0 = existed ? R[0] : 0.0f;
    float m0[early ? J : 1], b0[early ? J : 1];
    if constexpr (early) {
#pragma unroll
        for (int j = 0; j < J; ++j) {
            const int comp = lane + 64 * j;
            m0[j] = existed && comp < C ? R[2 + comp] : 0.0f;
            b0[j] = open && existed && comp < C ? R[2 + C + comp] : 0.0f;
        }
    }
    auto window = [&](uint32_t q) {
        if (q > 0 && (q & 63u) == 0) kl = q + (uint32_t)lane < n ? keys[q + lane] & kPidMask : 0u;
    };
    auto pid_at = [&](uint32_t t) { return (uint32_t)__shfl((int)kl, (int)(t & 63u), 64); };
    if (open) {
        float z0[J];
        const uint32_t p0 = pid_at(0);
#pragma unroll
        for (int j = 0; j < J; ++j) z0[j] = (lane + 64 * j < C) ? load_emb(fp, p0, lane + 64 * j) : 0.0f;
        // observation 0 enters as its own difference, 0
        for (uint32_t q = 0; q < n; q += kWaveBatch) {
            window(q);
            float z[kWaveBatch][J];
#pragma unroll
            for (int b = 0; b < kWaveBatch; ++b) {
                const bool has = q + b < n && q + b > 0;
                const uint32_t pid = pid_at(q + b);
#pragma unroll
                for (int j = 0; j < J; ++j)
                    z[b][j] = (has && lane + 64 * j < C) ? load_emb(fp, pid, lane + 64 * j) : z0[j];
            }
#pragma unroll
            for (int b = 0; b < kWaveBatch; ++b)
#pragma unroll
                for (int j = 0; j < J; ++j) {
                    const float d = z[b][j] - z0[j];
                    s1[j] += d;
                    s2[j] += d * d;
                }
        }
        // Eqs. (11)-(14) with lambda = W, nu = W / 2
        const float nf = (float)n;
        const float W1 = W0 + nf;
        const float inv_n = 1.0f / nf, inv_w1 = 1.0f / W1;
        const float cross = W0 * nf * inv_w1;
        float *M = R + 2, *B = R + 2 + fp.L;
#pragma unroll
        for (int j = 0; j < J; ++j) {
            const int comp = lane + 64 * j;
            if (comp < C) {
                const float zbar = z0[j] + s1[j] * inv_n;
                const float scat = fmaxf(s2[j] - s1[j] * s1[j] * inv_n, 0.0f);
                float mi, bi;
                if constexpr (early) {
                    mi = m0[j];
                    bi = b0[j];
                } else {
                    mi = existed ? M[comp] : 0.0f;
                    bi = existed ? B[comp] : 0.0f;
                }
                const float dm = zbar - mi;
                B[comp] = bi + 0.5f * scat + cross * dm * dm * 0.5f;
                M[comp] = (W0 * mi + nf * zbar) * inv_w1;
            }
        }
    } else if (fp.sem_kind == SLIM_IN_LABEL_I32) {
        for (uint32_t q = 0; q < n; q += 2 * kWaveBatch) {
            window(q);
            int lab[2 * kWaveBatch];
#pragma unroll
            for (int b = 0; b < 2 * kWaveBatch; ++b) {
                const uint32_t pid = pid_at(q + b);
                lab[b] = q + b < n ? ((const int32_t *)fp.sem)[pid] : -1;
            }
#pragma unroll
            for (int b = 0; b < 2 * kWaveBatch; ++b)
#pragma unroll
                for (int j = 0; j < J; ++j) s1[j] += (lab[b] == lane + 64 * j) ? 1.0f : 0.0f;
        }
    } else if (fp.sem_kind == SLIM_IN_PROB_F32) {
        for (uint32_t q = 0; q < n; q += kWaveBatch) {
            window(q);
            float x[kWaveBatch][J];
#pragma unroll
            for (int b = 0; b < kWaveBatch; ++b) {
                const bool has = q + b < n;
                const uint32_t pid = pid_at(q + b);
                const size_t row = has ? (size_t)pid * C : 0;
#pragma unroll
                for (int j = 0; j < J; ++j)
                    x[b][j] = (has && lane + 64 * j < C) ? ((const float *)fp.sem)[row + lane + 64 * j] : 0.0f;
            }
#pragma unroll
            for (int b = 0; b < kWaveBatch; ++b)
#pragma unroll
                for (int j = 0; j < J; ++j) s1[j] += x[b][j];
        }
    } else {
        // logits, K <= 64: softmax across the wave
        for (uint32_t q = 0; q < n; q += kWaveBatch) {
            window(q);
            float l[kWaveBatch];
#pragma unroll
            for (int b = 0; b < kWaveBatch; ++b) {
                const uint32_t pid = pid_at(q + b);
                l[b] = (q + b < n && lane < C) ? ((const float *)fp.sem)[(size_t)pid * C + lane] : -INFINITY;
            }
#pragma unroll
            for (int b = 0; b < kWaveBatch; ++b) {
                if (q + b >= n) break;
                const float mx = wave_max(l[b]);
                const float e = lane < C ? expf(l[b] - mx) : 0.0f;
                s1[0] += e / wave_sum(e);
            }
        }
    }
    const float nf = (float)n;
    const float W1 = W0 + nf;
    if (!open) {
#pragma unroll
        for (int j = 0; j < J; ++j) {
            const int comp = lane + 64 * j;
            if (comp < C) {
                float c0;
                if constexpr (early) c0 = m0[j];
                else c0 = existed ? R[2 + comp] : 0.0f;
                R[2 + comp] = c0 + s1[j];
            }
        }
    }
    // fixed-point distance sum, 64 distances loaded at a time, one per lane
    const FixScale fx = fix_scale(fp);
    long long sum_t = (uint32_t)lane < n ? fix_q(vl, fx.s) : 0ll;
    for (uint32_t w0 = 64; w0 < n; w0 += 64)
        sum_t += w0 + (uint32_t)lane < n ? fix_q(vals[w0 + lane], fx.s) : 0ll;
    for (int d = 32; d > 0; d >>= 1) sum_t += __shfl_xor(sum_t, d, 64);
    if (lane == 0) {
        R[0] = tsdf_mean(D0, W0, W1, sum_t, fx.inv);
        R[1] = W1;
    }
}

// Non-Bayesian mode (SLIM-VDB*, Sec. IV): D and W as Eq. (1)-(2); the voxel's
// semantics become those of its most recent measurement, the last pair in point
// order (a ray visits a voxel at most once, so point indices are distinct).
// Closed set, one lane per voxel: the class the measurement names -- its label,
// or the first index of the largest probability or logit of its row.
__device__ __forceinline__ void combine_last_lane(const FrameParams &fp, const MapDev &md, const uint32_t *keys,
                                                  const float *vals, uint32_t n, long long rec, bool existed)
{
    const uint32_t pid = keys[n - 1] & kPidMask;
    int cls;
    if (fp.sem_kind == SLIM_IN_LABEL_I32) {
        cls = ((const int32_t *)fp.sem)[pid];
    } else {
        const float *row = (const float *)fp.sem + (size_t)pid * fp.K;
        float best = row[0];
        cls = 0;
        for (int k = 1; k < fp.K; ++k) {
            const float x = row[k];
            if (x > best) {
                best = x;
                cls = k;
            }
        }
    }
    float4 *R = (float4 *)(md.vox + (size_t)rec * md.rec_stride);
    const float4 r = existed ? R[0] : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    const float nf = (float)n, W1 = r.y + nf;
    const FixScale fx = fix_scale(fp);
    R[0] = make_float4(tsdf_mean(r.x, r.y, W1, tsdf_sum(vals, n, fx.s), fx.inv), W1, (float)cls, 0.0f);
}

// Open set, one wave per voxel: lane l copies components l, l + 64, ... of the
// measurement's embedding.
__device__ __forceinline__ void combine_last_wave(const FrameParams &fp, const MapDev &md, const uint32_t *keys,
                                                  const float *vals, uint32_t n, long long rec, bool existed)
{
    const uint32_t pid = keys[n - 1] & kPidMask;
    float *R = md.vox + (size_t)rec * md.rec_stride;
    for (int comp = lane_id(); comp < fp.L; comp += 64) R[2 + comp] = load_emb(fp, pid, comp);
    if (lane_id() == 0) {
        const float W0 = existed ? R[1] : 0.0f, D0 = existed ? R[0] : 0.0f, W1 = W0 + (float)n;
        const FixScale fx = fix_scale(fp);
        R[0] = tsdf_mean(D0, W0, W1, tsdf_sum(vals, n, fx.s), fx.inv);
        R[1] = W1;
    }
}

// Combines every touched voxel with offset in [o0, o1); the sorted pairs of
// bin o sit at keys[bin0[o] - base] / vals[bin0[o] - base] (LDS or global).
// Bits of touched-mask word w that fall in offsets [o0, o1).
__device__ __forceinline__ uint32_t range_bits(uint32_t bits, uint32_t w, uint32_t o0, uint32_t o1)
{
    if ((w << 5) < o0) bits &= ~0u << (o0 & 31);
    if (((w + 1) << 5) > o1) bits &= (o1 & 31) ? ((1u << (o1 & 31)) - 1u) : ~0u;
    return bits;
}

// Position of the k-th set bit (from 0) of x, which has more than k set bits.
__device__ __forceinline__ uint32_t select_bit(uint32_t x, uint32_t k)
{
    uint32_t pos = 0;
#pragma unroll
    for (int s = 16; s > 0; s >>= 1) {
        const uint32_t low = x & ((1u << s) - 1u), c = (uint32_t)__popc(low);
        if (k >= c) {
            k -= c;
            x >>= s;
            pos += (uint32_t)s;
        } else {
            x = low;
        }
    }
    return pos;
}

template <int KMAX, bool WAVE, bool ROWS>
__device__ void combine_range(const FrameParams &fp, const MapDev &md, LeafShared &sh, const uint32_t *keys,
                              const float *vals, uint32_t o0, uint32_t o1, uint32_t base)
{
    if constexpr (!WAVE) {
        // thread t takes the touched offsets of rank t, t + blockDim.x, ... in
        // [o0, o1), so a leaf with at most blockDim.x touched voxels loads its
        // records in one round
        const uint32_t w0 = o0 >> 5, w1 = (o1 - 1) >> 5;
        uint32_t cnt = 0;
        for (uint32_t w = w0; w <= w1; ++w) cnt += __popc(range_bits(sh.touch[w], w, o0, o1));
        for (uint32_t r = threadIdx.x; r < cnt; r += blockDim.x) {
            uint32_t w = w0, before = 0, bits = 0;
            for (; w <= w1; ++w) {
                bits = range_bits(sh.touch[w], w, o0, o1);
                const uint32_t c = __popc(bits);
                if (r < before + c) break;
                before += c;
            }
            const uint32_t o = (w << 5) + select_bit(bits, r - before);
            const uint32_t n = sh.hist[o];
            const long long rec = (long long)sh.pages[o >> 6] * kPageVoxels + (o & (kPageVoxels - 1));
            const bool existed = (sh.occ0[o >> 5] >> (o & 31)) & 1u;
            if constexpr (KMAX < 0)
                combine_last_lane(fp, md, keys + (sh.bin0[o] - base), vals + (sh.bin0[o] - base), n, rec, existed);
            else
                combine_lane<KMAX>(fp, md, keys + (sh.bin0[o] - base), vals + (sh.bin0[o] - base), n, rec, existed);
        }
    } else {
        const uint32_t wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
        for (uint32_t o = o0 + wave; o < o1; o += nw) {
            const uint32_t n = sh.hist[o];
            if (!n) continue;
            const long long rec = (long long)sh.pages[o >> 6] * kPageVoxels + (o & (kPageVoxels - 1));
            const bool existed = (sh.occ0[o >> 5] >> (o & 31)) & 1u;
            if (KMAX < 0)
                combine_last_wave(fp, md, keys + (sh.bin0[o] - base), vals + (sh.bin0[o] - base), n, rec, existed);
            else if (KMAX > 0)  // wave kernels: KMAX is the components per lane of a word-aligned embedding
                combine_wave_vec<(KMAX > 0 ? KMAX : 1)>(fp, md, keys + (sh.bin0[o] - base), vals + (sh.bin0[o] - base),
                                                        n, rec, existed);
            else
                combine_wave<kWaveComps>(fp, md, keys + (sh.bin0[o] - base), vals + (sh.bin0[o] - base), n, rec, existed);
        }
    }
}

// Orders the pairs of bins [o0, o1) (binned in `bk`/`bv`, at bucket indices
// starting at `lo`) by point index inside each bin: a pair's position is the
// number of smaller keys in its bin.  Writes sh.a_*.
template <class KP, class VP>
__device__ __forceinline__ void rank_bins(LeafShared &sh, KP bk, VP bv, uint32_t lo, uint32_t hi)
{
    for (uint32_t t = lo + threadIdx.x; t < hi; t += blockDim.x) {
        const uint32_t k = bk[t - lo];
        const uint32_t o = k >> kPidBits, blo = sh.bin0[o], bhi = blo + sh.hist[o];
        uint32_t r = 0;
#pragma unroll 8
        for (uint32_t u = blo; u < bhi; ++u) r += bk[u - lo] < k;
        sh.a_key[blo + r - lo] = k;
        sh.a_val[blo + r - lo] = bv[t - lo];
    }
}

// One work item of the leaf kernel: the touched leaf of item *itp, all
// of it (part < 0) or, for a leaf with more pairs than LDS holds, one part of
// it, so that the parts of a large leaf run in different workgroups.  The part
// is an x-slab (offsets 64 part .. 64 part + 63): the item then reads every
// pair of the leaf for the offset histogram (which fixes the bucket position of
// every voxel) and keeps those of its offsets, reading the leaf once when they
// fit LDS and a second time otherwise.  In a binned frame the part is the
// voxels whose bins start in pairs kRangePairs part + [0, kRangePairs): bin
// starts and binned pairs are there already.  The item orders its pairs by point
// index inside each voxel and combines the voxels.
template <int KMAX, bool WAVE, bool ROWS>
__device__ __forceinline__ void fuse_item(const FrameParams &fp, const MapDev &md, LeafShared &sh, LeafItem *itp,
                                          int part, unsigned long long lused, bool ok)
{
    const int tid = threadIdx.x;
    if (tid < 32) sh.item[tid] = ((const uint32_t *)itp)[tid];
    for (int o = tid; o < kLeafVoxels; o += blockDim.x) sh.hist[o] = 0;
    if (tid == 0) sh.stash_n = 0;
    __syncthreads();
    const uint32_t pos = sh.item[0], n = sh.item[1], bstart = sh.item[2];
    const int islot = (int)sh.item[3];
    const int slot = islot >= 0 ? islot : (int)(lused + (unsigned long long)(-1 - islot));
    const bool binned = part >= 0 && md.binned;
    uint32_t ob = part < 0 ? 0u : 64u * (uint32_t)part, oe = part < 0 ? (uint32_t)kLeafVoxels : ob + 64u;
    // a new leaf is inserted by its whole-leaf item, the item of its lowest
    // touched slab or of its first range; the first probe goes out with the pair loads
    const bool lead = part < 0 || part == (binned ? 0 : __ffs(sh.item[4] & 0xFFu) - 1);
    const bool inserts = ok && lead && islot < 0 && tid == 0;
    const unsigned long long lkey = ((unsigned long long)sh.item[7] << 32) | sh.item[6];
    uint32_t ih = 0;
    unsigned long long iprev = 0;
    if (inserts) iprev = map_insert_start(md, lkey, &ih);
    if (tid < kMaskWords) sh.occ0[tid] = sh.item[16 + tid];
    if (tid < kLeafPages) sh.pages[tid] = (int)sh.item[8 + tid];

    const uint2 *gkv = md.srt_kv + bstart;
    uint32_t *tk = md.tmp_key + bstart;
    float *tv = md.tmp_tsdf + bstart;
    const bool whole_small = part < 0 && n <= (uint32_t)kLeafLdsPairs;

    // histogram of the voxel offsets of every pair of the leaf; kLeafBatch loads
    // in flight per thread, and a whole leaf that fits LDS stays in registers
    uint32_t rk[kLeafBatch];
    float rv[kLeafBatch];
    if (binned) {
        const uint2 s2 = ((const uint2 *)(md.srt_lab + bstart + (bstart & 1u)))[tid];
        sh.bin0[2 * tid] = s2.x;
        sh.bin0[2 * tid + 1] = s2.y;
        __syncthreads();
        sh.hist[2 * tid] = s2.y - s2.x;
        sh.hist[2 * tid + 1] = (tid < 255 ? sh.bin0[2 * tid + 2] : n) - s2.y;
        // first offsets whose bins start at or after the range's ends
        auto first = [&](uint32_t lim) {
            uint32_t lo = 0, hi = kLeafVoxels;
            while (lo < hi) {
                const uint32_t mid = (lo + hi) >> 1;
                if (sh.bin0[mid] < lim) lo = mid + 1;
                else hi = mid;
            }
            return lo;
        };
        ob = first((uint32_t)part * kRangePairs);
        oe = first(((uint32_t)part + 1u) * kRangePairs);
    } else if (whole_small) {
#pragma unroll
        for (int u = 0; u < kLeafBatch; ++u) {
            const uint32_t t = u * kLeafThreads + tid;
            const uint2 e = t < n ? gkv[t] : make_uint2(0u, 0u);
            rk[u] = e.x;
            rv[u] = __uint_as_float(e.y);
        }
#pragma unroll
        for (int u = 0; u < kLeafBatch; ++u)
            if ((uint32_t)(u * kLeafThreads + tid) < n) atomicAdd(&sh.hist[rk[u] >> kPidBits], 1u);
    } else {
        // every pair into the histogram; the pairs of the item's own offsets
        // into a_key/a_val in arrival order, as long as they fit (one slot
        // reservation per wave and batch)
        for (uint32_t t0 = 0; t0 < n; t0 += kLeafLdsPairs) {
#pragma unroll
            for (int u = 0; u < kLeafBatch; ++u) {
                const uint32_t t = t0 + u * kLeafThreads + tid;
                const uint2 e = t < n ? gkv[t] : make_uint2(0u, 0u);
                rk[u] = e.x;
                rv[u] = __uint_as_float(e.y);
            }
            uint32_t mine = 0;
#pragma unroll
            for (int u = 0; u < kLeafBatch; ++u) {
                const uint32_t o = rk[u] >> kPidBits;
                if (t0 + u * kLeafThreads + tid < n) {
                    atomicAdd(&sh.hist[o], 1u);
                    mine += (o >= ob && o < oe) ? 1u : 0u;
                }
            }
            const uint32_t incl = wave_incl_scan(mine);
            uint32_t wbase = 0;
            if (lane_id() == 63 && incl) wbase = atomicAdd(&sh.stash_n, incl);
            uint32_t q = __shfl(wbase, 63, 64) + incl - mine;
#pragma unroll
            for (int u = 0; u < kLeafBatch; ++u) {
                const uint32_t o = rk[u] >> kPidBits;
                if (t0 + u * kLeafThreads + tid < n && o >= ob && o < oe) {
                    if (q < (uint32_t)kLeafLdsPairs) {
                        sh.a_key[q] = rk[u];
                        sh.a_val[q] = rv[u];
                    }
                    q++;
                }
            }
        }
    }
    __syncthreads();
    if (!binned) {
        block_scan512(sh.hist, sh.bin0, sh.wsum);
        for (int o = tid; o < kLeafVoxels; o += blockDim.x) sh.cur[o] = sh.bin0[o];
    }
    {
        // touched offsets: wave w covers bins 64w + [0, 64) and 256 + 64w + [0, 64)
        const int w = tid >> 6;
        const unsigned long long b0 = __ballot(sh.hist[tid] != 0u);
        const unsigned long long b1 = __ballot(sh.hist[tid + 256] != 0u);
        if (lane_id() == 0) {
            sh.touch[2 * w] = (uint32_t)b0;
            sh.touch[2 * w + 1] = (uint32_t)(b0 >> 32);
            sh.touch[8 + 2 * w] = (uint32_t)b1;
            sh.touch[9 + 2 * w] = (uint32_t)(b1 >> 32);
        }
    }
    __syncthreads();
    if (WAVE && ok && lead) {
        // the leaf's item that inserts it also lists all its touched voxels for
        // the wave combine, in offset order at consecutive entries, so that the
        // voxels of one leaf (which share observations) are combined at the
        // same time; every item of the leaf has its histogram, so the voxel's
        // sorted pairs start at bucket position bin0[o] whichever item sorts them
        if (tid == 0) {
            uint32_t t = 0;
            for (int q = 0; q < kMaskWords; ++q) t += __popc(sh.touch[q]);
            sh.chunk_end = atomicAdd(&md.fs->n_vox.v, t);  // (free until the runs below)
        }
        __syncthreads();
        const uint32_t vbase = sh.chunk_end;
        for (uint32_t o = tid; o < (uint32_t)kLeafVoxels; o += blockDim.x) {
            const uint32_t n_o = sh.hist[o];
            if (!n_o) continue;
            // rank of o among the leaf's touched offsets
            uint32_t r = __popc(sh.touch[o >> 5] & ((1u << (o & 31)) - 1u));
            for (uint32_t w32 = 0; w32 < (o >> 5); ++w32) r += __popc(sh.touch[w32]);
            const uint32_t rec = (uint32_t)sh.pages[o >> 6] * kPageVoxels + (o & (kPageVoxels - 1));
            const uint32_t existed = (sh.occ0[o >> 5] >> (o & 31)) & 1u;
            md.vox_list[vbase + r] = make_uint4(rec, n_o | (existed << 31), bstart + sh.bin0[o], 0u);
        }
    }
    const uint32_t lo_all = ob < (uint32_t)kLeafVoxels ? sh.bin0[ob] : n;
    const uint32_t hi_all = oe < (uint32_t)kLeafVoxels ? sh.bin0[oe] : n;
    const bool small = whole_small || (part >= 0 && hi_all - lo_all <= (uint32_t)kLeafLdsPairs);
    if (tid == 0) {
        uint32_t uo = 0, un = 0;
        for (uint32_t w = ob >> 5; w < (oe + 31u) >> 5; ++w) {
            const uint32_t mine = range_bits(sh.touch[w], w, ob, oe);
            uo += __popc(mine & sh.occ0[w]);
            un += __popc(mine & ~sh.occ0[w]);
        }
        sh.uold += uo;
        sh.unew += un;
    }

    // bin by offset (order inside a bin arbitrary): in LDS if the item fits,
    // else in the scratch buffer.  An x-slab item that fits bins from the
    // pairs it kept (exactly those of its offsets: their count is the width
    // of its range of the histogram)
    if (whole_small) {
#pragma unroll
        for (int u = 0; u < kLeafBatch; ++u)
            if ((uint32_t)(u * kLeafThreads + tid) < n) {
                const uint32_t p = atomicAdd(&sh.cur[rk[u] >> kPidBits], 1u);
                sh.b_key[p] = rk[u];
                sh.b_val[p] = rv[u];
            }
    } else if (binned) {
        if (small)
            for (uint32_t t = tid; t < hi_all - lo_all; t += blockDim.x) {
                sh.b_key[t] = tk[lo_all + t];
                sh.b_val[t] = tv[lo_all + t];
            }
    } else if (small) {
        const uint32_t m = hi_all - lo_all;
        for (uint32_t t = tid; t < m; t += blockDim.x) {
            const uint32_t k = sh.a_key[t];
            const uint32_t p = atomicAdd(&sh.cur[k >> kPidBits], 1u);
            sh.b_key[p - lo_all] = k;
            sh.b_val[p - lo_all] = sh.a_val[t];
        }
    } else {
        for (uint32_t t0 = 0; t0 < n; t0 += kLeafLdsPairs) {
#pragma unroll
            for (int u = 0; u < kLeafBatch; ++u) {
                const uint32_t t = t0 + u * kLeafThreads + tid;
                const uint2 e = t < n ? gkv[t] : make_uint2(0u, 0u);
                rk[u] = e.x;
                rv[u] = __uint_as_float(e.y);
            }
#pragma unroll
            for (int u = 0; u < kLeafBatch; ++u) {
                const uint32_t o = rk[u] >> kPidBits;
                if (t0 + u * kLeafThreads + tid < n && o >= ob && o < oe) {
                    const uint32_t p = atomicAdd(&sh.cur[o], 1u);
                    tk[p] = rk[u];
                    tv[p] = rv[u];
                }
            }
        }
    }
    __syncthreads();

    // runs of whole bins that fit LDS: order each bin by point index, then
    // combine its voxels (a small item is one run, already in LDS)
    uint32_t o0 = ob;
    while (o0 < oe) {
        uint32_t o1 = oe;
        if (!small) {
            if (tid == 0) {
                // bin ends are non-decreasing: first o1 > o0 whose end passes
                // bin0[o0] + capacity (at least o0 + 1)
                const uint32_t lim = sh.bin0[o0] + (uint32_t)kLeafLdsPairs;
                uint32_t lo = o0 + 1, hi = oe;
                while (lo < hi) {
                    const uint32_t mid = (lo + hi) >> 1;
                    if (sh.bin0[mid] + sh.hist[mid] <= lim) lo = mid + 1;
                    else hi = mid;
                }
                sh.chunk_end = lo;
            }
            __syncthreads();
            o1 = sh.chunk_end;
        }
        const uint32_t lo = sh.bin0[o0], hi = (o1 < (uint32_t)kLeafVoxels) ? sh.bin0[o1] : n;
        const bool fits = hi - lo <= (uint32_t)kLeafLdsPairs;
        if (fits) {
            if (!small) {
                for (uint32_t t = lo + tid; t < hi; t += blockDim.x) {
                    sh.b_key[t - lo] = tk[t];
                    sh.b_val[t - lo] = tv[t];
                }
                __syncthreads();
            }
            rank_bins(sh, sh.b_key, sh.b_val, lo, hi);
        } else {
            // one bin larger than LDS: order it into the sorted pairs' buffers, at
            // the bin's own range of the leaf's bucket, which no other item touches
            uint32_t *bk = md.pair_key + bstart;
            float *bv = md.pair_tsdf + bstart;
            for (uint32_t t = lo + tid; t < hi; t += blockDim.x) {
                const uint32_t k = tk[t];
                uint32_t r = 0;
                for (uint32_t u = lo; u < hi; ++u) r += tk[u] < k;
                bk[lo + r] = k;
                bv[lo + r] = tv[t];
            }
        }
        __syncthreads();
        if (ok && WAVE) {
            // wave combines run in their own kernel over every voxel of the frame:
            // the sorted pairs go to the pair buffers at their bucket positions
            if (fits)
                for (uint32_t t = tid; t < hi - lo; t += blockDim.x) {
                    md.pair_key[bstart + lo + t] = sh.a_key[t];
                    md.pair_tsdf[bstart + lo + t] = sh.a_val[t];
                }
        } else if (ok) {
            // sorted pairs of bin o sit at keys[bin0[o] - base]
            const uint32_t *ck = fits ? sh.a_key : md.pair_key + bstart;
            const float *cv = fits ? sh.a_val : md.pair_tsdf + bstart;
            combine_range<KMAX, WAVE, ROWS>(fp, md, sh, ck, cv, o0, o1, fits ? lo : 0u);
        }
        __syncthreads();
        o0 = o1;
    }

    // leaf bookkeeping: an x-slab item owns the page entry and the occupancy
    // words of its offsets; the item of the leaf's lowest touched slab also
    // inserts a new leaf and writes the entries of untouched slabs.  The
    // whole-leaf item, or the item of the first range (every item of a binned
    // leaf has the whole leaf's counts), does all of it
    if (ok) {
        const uint32_t tslabs = sh.item[4] & 0xFFu;
        if (inserts) {
            map_insert_finish(md, lkey, slot, ih, iprev);
            md.leaf_key[slot] = lkey;
        }
        if (tid < kLeafPages) {
            const bool mine = part < 0 || binned ? lead : tid == part || (lead && !((tslabs >> tid) & 1u));
            if (mine) md.leaf_page[(size_t)slot * kLeafPages + tid] = sh.pages[tid];
        }
        if (tid < kMaskWords) {
            const int sl = tid >> 1;
            const bool mine = part < 0 || binned ? lead : sl == part || (lead && !((tslabs >> sl) & 1u));
            if (mine) md.leaf_occ[(size_t)slot * kMaskWords + tid] = sh.occ0[tid] | sh.touch[tid];
        }
    }
    __syncthreads();
    if (tid == 0) {
        // the staging entry is clean for the next frame once the leaf's last
        // item is done (a whole-leaf item is the only one; the parts of a large
        // leaf count themselves in the item's spare word, which the plan kernel zeroes)
        const uint32_t nparts = binned ? (n + (uint32_t)kRangePairs - 1u) / (uint32_t)kRangePairs
                                       : (uint32_t)__popc(sh.item[4] & 0xFFu);
        const bool last = part < 0 || atomicAdd(&itp->pad, 1u) + 1u == nparts;
        if (last) {
            md.skeys[pos] = kEmptyKey;
            md.pos_count[pos] = 0u;
            md.pos_slab[pos] = 0u;
        }
    }
}

// A touched leaf with at most kWaveItemPairs pairs is the work of one wave:
// its pairs are ordered in the wave's quarter of the block's LDS by the full
// key (offset, point index), which groups them by voxel in point order; lanes
// then take one voxel each.  Waves run such leaves independently (no block
// barrier), four per block.
constexpr int kWaveLds = kLeafLdsPairs / 4;  // LDS pairs per wave
static_assert(kWaveItemPairs <= kWaveLds, "a wave item must fit its LDS quarter");

template <int KMAX, bool WAVE, bool ROWS>
__device__ __forceinline__ void fuse_wave_item(const FrameParams &fp, const MapDev &md, LeafShared &sh,
                                               const LeafItem *itp, unsigned long long lused, bool ok)
{
    const int lane = lane_id(), w = threadIdx.x >> 6;
    uint32_t *wk = sh.a_key + w * kWaveLds;
    float *wv = sh.a_val + w * kWaveLds;
    uint32_t *seg = sh.b_key + w * kWaveLds;     // voxel segment starts
    uint32_t *wt = sh.hist + w * 16;             // touched-offset mask (16 words)
    uint32_t *wo = sh.bin0 + w * 16;             // occupancy words of the leaf before this frame
    int *wp = (int *)sh.cur + w * 8;             // record pages of the leaf's slabs
    uint32_t *wi = sh.cur + 64 + w * 32;         // the leaf's item
    if (lane < 32) wi[lane] = ((const uint32_t *)itp)[lane];
    wave_sync();
    const uint32_t pos = wi[0], n = wi[1], bstart = wi[2];
    const int islot = (int)wi[3];
    const int slot = islot >= 0 ? islot : (int)(lused + (unsigned long long)(-1 - islot));
    // a new leaf's first insertion probe goes out with the pair loads
    const bool inserts = ok && islot < 0 && lane == 0;
    const unsigned long long lkey = ((unsigned long long)wi[7] << 32) | wi[6];
    uint32_t ih = 0;
    unsigned long long iprev = 0;
    if (inserts) iprev = map_insert_start(md, lkey, &ih);
    // the pairs in registers (four per lane), their keys also in LDS; keys are
    // distinct (a ray visits a voxel once), so a pair's rank is the number of
    // smaller keys, and writing each pair at its rank sorts them by (offset,
    // point index)
    uint32_t *uk = sh.b_key + w * kWaveLds;  // unsorted keys, padded to a multiple of 4
    uint32_t kq[4];
    float vq[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const uint32_t i = lane + 64 * q;
        const bool has = i < n;
        const uint2 e = has ? md.srt_kv[bstart + i] : make_uint2(0xFFFFFFFFu, 0u);
        kq[q] = e.x;
        vq[q] = __uint_as_float(e.y);
        if (i < ((n + 3u) & ~3u)) uk[i] = kq[q];
    }
    const uint32_t occ = lane < kMaskWords ? wi[16 + lane] : 0u;
    const int page = lane < kLeafPages ? (int)wi[8 + lane] : -1;
    if (lane < 16) {
        wt[lane] = 0u;
        wo[lane] = occ;
    }
    if (lane < kLeafPages) wp[lane] = page;
    wave_sync();
    uint32_t rq[4] = {0u, 0u, 0u, 0u};
    for (uint32_t s4 = 0; s4 < n; s4 += 4) {
        const uint4 c = *(const uint4 *)(uk + s4);
#pragma unroll
        for (int q = 0; q < 4; ++q)
            rq[q] += (uint32_t)(c.x < kq[q]) + (uint32_t)(c.y < kq[q]) + (uint32_t)(c.z < kq[q]) +
                     (uint32_t)(c.w < kq[q]);
    }
#pragma unroll
    for (int q = 0; q < 4; ++q)
        if (lane + 64 * q < n) {
            wk[rq[q]] = kq[q];
            wv[rq[q]] = vq[q];
        }
    wave_sync();
    // voxel segments: starts where the offset changes
    uint32_t nseg = 0;
    const uint32_t per = (n + 63u) >> 6;
    for (uint32_t q = 0; q < per; ++q) {
        const uint32_t i = lane + 64 * q;
        const bool start = i < n && (i == 0 || (wk[i] >> kPidBits) != (wk[i - 1] >> kPidBits));
        const unsigned long long b = __ballot(start);
        if (start) seg[nseg + __popcll(b & ((1ull << lane) - 1ull))] = i;
        nseg += (uint32_t)__popcll(b);
    }
    wave_sync();
    for (uint32_t sgi = lane; sgi < nseg; sgi += 64) {
        const uint32_t o = wk[seg[sgi]] >> kPidBits;
        atomicOr(&wt[o >> 5], 1u << (o & 31));
    }
    wave_sync();
    if (ok) {
        for (uint32_t sgi = lane; sgi < nseg; sgi += 64) {
            const uint32_t b0 = seg[sgi], b1 = sgi + 1 < nseg ? seg[sgi + 1] : n;
            const uint32_t o = wk[b0] >> kPidBits;
            const int pg = wp[o >> 6];
            const uint32_t ow = wo[o >> 5];
            const long long rec = (long long)pg * kPageVoxels + (o & (kPageVoxels - 1));
            const bool existed = (ow >> (o & 31)) & 1u;
            if constexpr (KMAX < 0)
                combine_last_lane(fp, md, wk + b0, wv + b0, b1 - b0, rec, existed);
            else
                combine_lane<KMAX>(fp, md, wk + b0, wv + b0, b1 - b0, rec, existed);
        }
    }
    // statistics and leaf bookkeeping
    const uint32_t tw = lane < kMaskWords ? wt[lane] : 0u;
    uint32_t uo = __popc(tw & occ), un = __popc(tw & ~occ);
    for (int d = 32; d > 0; d >>= 1) {
        uo += __shfl_xor(uo, d, 64);
        un += __shfl_xor(un, d, 64);
    }
    if (lane == 0) {
        atomicAdd(&sh.uold, uo);
        atomicAdd(&sh.unew, un);
    }
    if (ok) {
        if (inserts) {
            map_insert_finish(md, lkey, slot, ih, iprev);
            md.leaf_key[slot] = lkey;
        }
        if (lane < kLeafPages) md.leaf_page[(size_t)slot * kLeafPages + lane] = page;
        if (lane < kMaskWords) md.leaf_occ[(size_t)slot * kMaskWords + lane] = occ | tw;
    }
    if (lane == 0) {
        md.skeys[pos] = kEmptyKey;
        md.pos_count[pos] = 0u;
        md.pos_slab[pos] = 0u;
    }
    wave_sync();
}

// The leaf kernel's work of one map's frame for blocks blk, blk + nblk, ...:
// first the slab items of large leaves (the longest work, started first), then
// every other touched leaf whole.  Its statistics are added to the frame's.
template <int KMAX, bool WAVE, bool ROWS>
__device__ __forceinline__ void leaf_fuse_range(const FrameParams &fp, const MapDev &md, LeafShared &sh,
                                                uint32_t blk, uint32_t nblk)
{
    const DevState *st = md.st;
    const uint32_t nbig = min(md.fs->work_big.v, md.work_cap);
    const unsigned long long lused = st->leaves_used;
    const bool ok = md.fs->frame_err.v == 0 && st->pass_failed == 0 &&
                    lused + md.fs->new_leaves.v <= (unsigned long long)md.max_leaves &&
                    st->pages_used + md.fs->new_pages.v <= (unsigned long long)md.max_pages;
    if (threadIdx.x == 0) {
        sh.uold = 0;
        sh.unew = 0;
    }
    __syncthreads();
    // units of work, one per block at a time: the slab items of large leaves,
    // then the leaves done by a workgroup, then groups of four small leaves
    // (one per wave; the wave kernels take the small leaves one per workgroup)
    // each list: its larger leaves from the front of the array, then its
    // smaller ones from the back
    const uint32_t medf = (uint32_t)md.fs->n_lists, smallf = (uint32_t)(md.fs->n_lists >> 32);
    const uint32_t nmed = medf + (uint32_t)md.fs->n_lists_tail;
    const uint32_t nsmall = smallf + (uint32_t)(md.fs->n_lists_tail >> 32);
    const uint32_t last = md.hmask;
    auto med_at = [&](uint32_t m) { return &md.items[m < medf ? m : last - (m - medf)]; };
    auto small_at = [&](uint32_t k) { return &md.items_small[k < smallf ? k : last - (k - smallf)]; };
    const uint32_t nw = blockDim.x >> 6, w = threadIdx.x >> 6;
    const uint32_t ngroups = WAVE ? nsmall : (nsmall + nw - 1) / nw;
    const uint32_t nunits = nbig + nmed + ngroups;
    for (uint32_t u = blk; u < nunits; u += nblk) {
        if (u < nbig) {
            const int2 it = md.work[u];
            fuse_item<KMAX, WAVE, ROWS>(fp, md, sh, &md.items_big[it.x], it.y, lused, ok);
        } else if (u < nbig + nmed) {
            fuse_item<KMAX, WAVE, ROWS>(fp, md, sh, med_at(u - nbig), -1, lused, ok);
        } else if constexpr (WAVE) {
            fuse_item<KMAX, WAVE, ROWS>(fp, md, sh, small_at(u - nbig - nmed), -1, lused, ok);
        } else {
            const uint32_t k = (u - nbig - nmed) * nw + w;
            if (k < nsmall) fuse_wave_item<KMAX, WAVE, ROWS>(fp, md, sh, small_at(k), lused, ok);
            __syncthreads();
        }
    }
    __syncthreads();
    if (threadIdx.x == 0 && (sh.uold | sh.unew))
        atomicAdd(&md.fs->stat[blk & 63u].v, ((unsigned long long)sh.unew << 32) | sh.uold);
    __syncthreads();
}

// Row kernels at four workgroups per CU hold 128 registers and spill a few (4, 11 and
// 18 with 16, 24 and 32 classes in registers; none with 8).  With three, which do not,
// a frame of probability rows with 5, 12, 20 and 28 classes takes 48.5, 49.3, 51.2 and
// 52.8 us at 4,096 rays (with four 48.0, 49.7, 52.0 and 54.3), 62.7, 71.6, 76.2 and
// 81.8 us at 65,536 (63.3, 65.9, 71.2 and 78.1), 97, 112, 119 and 127 us at 131,071
// (98, 102, 110 and 118); with voxels twice as large, 20 classes, 66,000 rays 115 us
// (121).
template <int KMAX, bool WAVE, bool ROWS>
__global__ __launch_bounds__(kLeafThreads, WAVE ? 1 : 4) void k_leaf_fuse(FrameParams fp, MapDev md)
{
    __shared__ LeafShared sh;
    leaf_fuse_range<KMAX, WAVE, ROWS>(fp, md, sh, blockIdx.x, gridDim.x);
}

// The maps mb.subset[0 .. nsubset) of a batch, all of this kernel's kind, each
// on its share of the grid.  Row kernels at four workgroups per CU up to 24 classes (16
// maps of 30,000 rays with 5, 12 and 20 classes 347, 387 and 464 us; at three 386, 417
// and 477), at three above (28 classes: at four 56 registers spill, 546 us, at three
// none, 501).
template <int KMAX, bool WAVE, bool ROWS>
__global__ __launch_bounds__(kLeafThreads, WAVE ? 1 : (KMAX > 24 ? 3 : 4)) void k_leaf_fuse_batch(MapBatch mb)
{
    __shared__ LeafShared sh;
    const int q = batch_map(mb.part_first, mb.nsubset, blockIdx.x), i = mb.subset[q];
    leaf_fuse_range<KMAX, WAVE, ROWS>(mb.fps[i], mb.mds[i], sh, blockIdx.x - mb.part_first[q],
                                      mb.part_first[q + 1] - mb.part_first[q]);
}


// ---------------------------------------------------------------------------
// 4'. per-leaf accumulation: geometry, or int32 labels with K <= 32 (Bayesian)
// ---------------------------------------------------------------------------
//
// Everything such a frame adds to a voxel is an integer: its observation count
// (W grows by it, Eq. (1)-(2)), its class counts (Eq. (6)) and its fixed-point
// distance sum.  Integer sums do not depend on the order of their terms, so a
// leaf's pairs are not sorted at all: each pair adds into its voxel's LDS
// accumulators with integer atomics (one set per frame of a multi-frame pass),
// then one lane per touched voxel applies them to the record, frame after
// frame.  The record is bitwise the same whatever order the pairs arrive in.

template <int KMAX, int FR>
struct AccShared {
    static constexpr int KW = KMAX > 0 ? (KMAX + 1) / 2 : 1;  // class counts as 16-bit fields, two to a word
    union {
        struct {  // one leaf per workgroup, indexed by voxel offset
            unsigned long long sum[FR][kLeafVoxels];
            uint32_t cnt[FR][kLeafVoxels];
            uint32_t lab[kLeafVoxels][KW];
        } b;
        struct {  // one leaf per wave, indexed by rank among the leaf's touched voxels
            unsigned long long sum[FR][kAccWavePairs];
            uint32_t cnt[FR][kAccWavePairs];
            uint32_t lab[kAccWavePairs][KW];
        } w[4];
    };
    uint32_t touch[4][kMaskWords];  // touched offsets of the workgroup's leaf, or of each wave's
    uint32_t pre[4][kMaskWords];    // touched offsets below each mask word (wave leaves)
    uint32_t item[4][32];           // the leaf item of the workgroup, or of each wave
    uint32_t uold, unew;
};

// Class counts of a voxel with more than 65535 observations in a unit (whose
// 16-bit counts may have wrapped), counted again from the unit's pairs, one
// class at a time, and added to its record.  Slow, and only for such voxels.
__device__ __noinline__ void acc_recount(const FrameParams &fp, const MapDev &md, long long rec, const uint2 *gkv,
                                         const int32_t *glab, uint32_t npairs, uint32_t o)
{
    float *R = md.vox + (size_t)rec * md.rec_stride;
    for (int k = 0; k < fp.K; ++k) {
        uint32_t c = 0;
        for (uint32_t t = 0; t < npairs; ++t) c += ((gkv[t].x >> kPidBits) == o && glab[t] == k) ? 1u : 0u;
        R[2 + k] += (float)c;
    }
}

// Applies one voxel's accumulators to its record: Eq. (1)-(2) frame after frame
// (each frame's run exactly as that frame alone), then Eq. (6).  sum and cnt
// point at frame 0's entry, the frames fstride apart; lab holds the 16-bit
// class counts.  A voxel with more than 65535 observations in the unit may have
// wrapped a 16-bit count: its labels are then counted again from the unit's
// pairs (gkv, glab, npairs), which only a workgroup unit passes.
template <int KMAX, int FR>
__device__ __forceinline__ void acc_apply(const FrameParams &fp, const MapDev &md, long long rec, bool existed,
                                          const unsigned long long *sum, const uint32_t *cnt, int fstride,
                                          const uint32_t *lab, int nf, const FixScale &fx, const uint2 *gkv,
                                          const int32_t *glab, uint32_t npairs, uint32_t o)
{
    constexpr int NV = (2 + KMAX + 3) / 4;
    const int nv = md.rec_stride / 4, K = fp.K;
    float4 *R = (float4 *)(md.vox + (size_t)rec * md.rec_stride);
    float r[4 * NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) {
        const float4 x = (existed && v < nv) ? R[v] : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        r[4 * v + 0] = x.x;
        r[4 * v + 1] = x.y;
        r[4 * v + 2] = x.z;
        r[4 * v + 3] = x.w;
    }
    uint32_t ntot = 0;
#pragma unroll
    for (int f = 0; f < FR; ++f) {
        const uint32_t c = f < nf ? cnt[f * fstride] : 0u;
        if (c) {
            const float W0 = r[1], W1 = W0 + (float)c;
            r[0] = tsdf_mean(r[0], W0, W1, (long long)sum[f * fstride], fx.inv);
            r[1] = W1;
            ntot += c;
        }
    }
    const bool wrapped = ntot > 0xFFFFu;
    if constexpr (KMAX > 0) {
        if (!wrapped) {
#pragma unroll
            for (int k = 0; k < KMAX; ++k)
                if (k < K) r[2 + k] += (float)((lab[k >> 1] >> ((k & 1) << 4)) & 0xFFFFu);
        }
    }
#pragma unroll
    for (int v = 0; v < NV; ++v)
        if (v < nv) R[v] = make_float4(r[4 * v + 0], r[4 * v + 1], r[4 * v + 2], r[4 * v + 3]);
    if (KMAX > 0 && wrapped) acc_recount(fp, md, rec, gkv, glab, npairs, o);
}

// A leaf with more than kAccWavePairs pairs, whole, by one workgroup of
// kLeafThreads threads: its pairs stream through registers (kLeafBatch loads in
// flight per thread) into accumulators indexed by voxel offset.
template <int KMAX, int FR>
__device__ __forceinline__ void acc_block_unit(const FrameParams &fp, const MapDev &md, AccShared<KMAX, FR> &sh,
                                               const LeafItem *itp, unsigned long long lused, bool ok,
                                               const FixScale &fx, int nf)
{
    const int tid = threadIdx.x;
    if (tid < 32) sh.item[0][tid] = ((const uint32_t *)itp)[tid];
    {
        uint4 *p = (uint4 *)&sh.b;
        constexpr int nvec = (int)(sizeof(sh.b) / 16);
        for (int i = tid; i < nvec; i += blockDim.x) p[i] = make_uint4(0u, 0u, 0u, 0u);
    }
    __syncthreads();
    const uint32_t *it = sh.item[0];
    const uint32_t pos = it[0], n = it[1], bstart = it[2];
    const int islot = (int)it[3];
    const int slot = islot >= 0 ? islot : (int)(lused + (unsigned long long)(-1 - islot));
    // a new leaf's first insertion probe goes out with the pair loads
    const bool inserts = ok && islot < 0 && tid == 0;
    const unsigned long long lkey = ((unsigned long long)it[7] << 32) | it[6];
    uint32_t ih = 0;
    unsigned long long iprev = 0;
    if (inserts) iprev = map_insert_start(md, lkey, &ih);
    const uint2 *gkv = md.srt_kv + bstart;
    const int32_t *glab = md.srt_lab + bstart;
    for (uint32_t t0 = 0; t0 < n; t0 += kLeafBatch * blockDim.x) {
        uint32_t rk[kLeafBatch];
        float rv[kLeafBatch];
        int32_t rl[kLeafBatch];
#pragma unroll
        for (int u = 0; u < kLeafBatch; ++u) {
            const uint32_t t = t0 + u * blockDim.x + tid;
            const uint2 e = t < n ? gkv[t] : make_uint2(0u, 0u);
            rk[u] = e.x;
            rv[u] = __uint_as_float(e.y);
            rl[u] = (KMAX > 0 && t < n) ? glab[t] : 0;
        }
#pragma unroll
        for (int u = 0; u < kLeafBatch; ++u)
            if (t0 + u * blockDim.x + tid < n) {
                const uint32_t o = rk[u] >> kPidBits;
                const int f = FR > 1 ? pass_frame(fp, rk[u] & kPidMask) : 0;
                atomicAdd(&sh.b.cnt[f][o], 1u);
                atomicAdd(&sh.b.sum[f][o], (unsigned long long)fix_q(rv[u], fx.s));
                if constexpr (KMAX > 0) atomicAdd(&sh.b.lab[o][rl[u] >> 1], 1u << ((rl[u] & 1) << 4));
            }
    }
    __syncthreads();
    {
        // touched offsets: wave w covers offsets 64 w + [0, 64) and 256 + 64 w + [0, 64)
        uint32_t c0 = 0, c1 = 0;
#pragma unroll
        for (int f = 0; f < FR; ++f)
            if (f < nf) {
                c0 += sh.b.cnt[f][tid];
                c1 += sh.b.cnt[f][tid + 256];
            }
        const unsigned long long b0 = __ballot(c0 != 0u), b1 = __ballot(c1 != 0u);
        const int w = tid >> 6;
        if (lane_id() == 0) {
            sh.touch[0][2 * w] = (uint32_t)b0;
            sh.touch[0][2 * w + 1] = (uint32_t)(b0 >> 32);
            sh.touch[0][8 + 2 * w] = (uint32_t)b1;
            sh.touch[0][9 + 2 * w] = (uint32_t)(b1 >> 32);
        }
    }
    __syncthreads();
    // thread t takes the touched offsets of rank t, t + blockDim.x, ...
    uint32_t ntouch = 0;
#pragma unroll
    for (int w = 0; w < kMaskWords; ++w) ntouch += __popc(sh.touch[0][w]);
    if (ok) {
        for (uint32_t r = tid; r < ntouch; r += blockDim.x) {
            uint32_t w = 0, before = 0, bits = 0;
            for (; w < (uint32_t)kMaskWords; ++w) {
                bits = sh.touch[0][w];
                const uint32_t c = __popc(bits);
                if (r < before + c) break;
                before += c;
            }
            const uint32_t o = (w << 5) + select_bit(bits, r - before);
            const long long rec = (long long)(int)it[8 + (o >> 6)] * kPageVoxels + (o & (kPageVoxels - 1));
            const bool existed = (it[16 + (o >> 5)] >> (o & 31)) & 1u;
            acc_apply<KMAX, FR>(fp, md, rec, existed, &sh.b.sum[0][o], &sh.b.cnt[0][o], kLeafVoxels, sh.b.lab[o], nf,
                                fx, gkv, glab, n, o);
        }
    }
    if (tid == 0) {
        uint32_t uo = 0, un = 0;
        for (int w = 0; w < kMaskWords; ++w) {
            uo += __popc(sh.touch[0][w] & it[16 + w]);
            un += __popc(sh.touch[0][w] & ~it[16 + w]);
        }
        sh.uold += uo;
        sh.unew += un;
    }
    // leaf bookkeeping: the unit owns the whole leaf
    if (ok) {
        if (inserts) {
            map_insert_finish(md, lkey, slot, ih, iprev);
            md.leaf_key[slot] = lkey;
        }
        if (tid < kLeafPages) md.leaf_page[(size_t)slot * kLeafPages + tid] = (int)it[8 + tid];
        if (tid < kMaskWords) md.leaf_occ[(size_t)slot * kMaskWords + tid] = it[16 + tid] | sh.touch[0][tid];
    }
    if (tid == 0) {
        md.skeys[pos] = kEmptyKey;
        md.pos_count[pos] = 0u;
        md.pos_slab[pos] = 0u;
    }
    __syncthreads();
}

// A leaf with at most kAccWavePairs pairs, by one wave (two pairs per lane):
// accumulators indexed by the rank of the voxel among the leaf's touched
// voxels.  Waves run such leaves independently, four per workgroup.
template <int KMAX, int FR>
__device__ __forceinline__ void acc_wave_unit(const FrameParams &fp, const MapDev &md, AccShared<KMAX, FR> &sh,
                                              const LeafItem *itp, unsigned long long lused, bool ok,
                                              const FixScale &fx, int nf)
{
    const int lane = lane_id(), w = threadIdx.x >> 6;
    auto &A = sh.w[w];
    uint32_t *wi = sh.item[w], *wt = sh.touch[w], *wp = sh.pre[w];
    if (lane < 32) wi[lane] = ((const uint32_t *)itp)[lane];
    if (lane < kMaskWords) wt[lane] = 0u;
    {
        uint4 *p = (uint4 *)&A;
        constexpr int nvec = (int)(sizeof(A) / 16);
        for (int i = lane; i < nvec; i += 64) p[i] = make_uint4(0u, 0u, 0u, 0u);
    }
    wave_sync();
    const uint32_t pos = wi[0], n = wi[1], bstart = wi[2];
    const int islot = (int)wi[3];
    const int slot = islot >= 0 ? islot : (int)(lused + (unsigned long long)(-1 - islot));
    const bool inserts = ok && islot < 0 && lane == 0;
    const unsigned long long lkey = ((unsigned long long)wi[7] << 32) | wi[6];
    uint32_t ih = 0;
    unsigned long long iprev = 0;
    if (inserts) iprev = map_insert_start(md, lkey, &ih);
    uint32_t kq[2];
    float vq[2];
    int32_t lq[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const uint32_t i = lane + 64 * q;
        const bool has = i < n;
        const uint2 e = has ? md.srt_kv[bstart + i] : make_uint2(0u, 0u);
        kq[q] = e.x;
        vq[q] = __uint_as_float(e.y);
        lq[q] = (KMAX > 0 && has) ? md.srt_lab[bstart + i] : 0;
    }
#pragma unroll
    for (int q = 0; q < 2; ++q)
        if (lane + 64 * q < n) {
            const uint32_t o = kq[q] >> kPidBits;
            atomicOr(&wt[o >> 5], 1u << (o & 31));
        }
    wave_sync();
    // rank of a touched offset: the touched offsets below its mask word, plus
    // those below it in the word
    const uint32_t pc = lane < kMaskWords ? (uint32_t)__popc(wt[lane]) : 0u;
    const uint32_t incl = wave_incl_scan(pc);
    if (lane < kMaskWords) wp[lane] = incl - pc;
    const uint32_t nvox = (uint32_t)__shfl((int)incl, kMaskWords - 1, 64);
    wave_sync();
#pragma unroll
    for (int q = 0; q < 2; ++q)
        if (lane + 64 * q < n) {
            const uint32_t o = kq[q] >> kPidBits;
            const uint32_t ci = wp[o >> 5] + (uint32_t)__popc(wt[o >> 5] & ((1u << (o & 31)) - 1u));
            const int f = FR > 1 ? pass_frame(fp, kq[q] & kPidMask) : 0;
            atomicAdd(&A.cnt[f][ci], 1u);
            atomicAdd(&A.sum[f][ci], (unsigned long long)fix_q(vq[q], fx.s));
            if constexpr (KMAX > 0) atomicAdd(&A.lab[ci][lq[q] >> 1], 1u << ((lq[q] & 1) << 4));
        }
    wave_sync();
    if (ok) {
        for (uint32_t ci = lane; ci < nvox; ci += 64) {
            // offset of rank ci: its mask word, then its bit there
            uint32_t wd = 0;
            while (wd + 1 < (uint32_t)kMaskWords && wp[wd + 1] <= ci) ++wd;
            const uint32_t o = (wd << 5) + select_bit(wt[wd], ci - wp[wd]);
            const long long rec = (long long)(int)wi[8 + (o >> 6)] * kPageVoxels + (o & (kPageVoxels - 1));
            const bool existed = (wi[16 + (o >> 5)] >> (o & 31)) & 1u;
            acc_apply<KMAX, FR>(fp, md, rec, existed, &A.sum[0][ci], &A.cnt[0][ci], kAccWavePairs, A.lab[ci], nf, fx,
                                nullptr, nullptr, 0u, o);
        }
    }
    // statistics and leaf bookkeeping
    const uint32_t tw = lane < kMaskWords ? wt[lane] : 0u;
    const uint32_t occ = lane < kMaskWords ? wi[16 + lane] : 0u;
    uint32_t uo = __popc(tw & occ), un = __popc(tw & ~occ);
    for (int d = 32; d > 0; d >>= 1) {
        uo += __shfl_xor(uo, d, 64);
        un += __shfl_xor(un, d, 64);
    }
    if (lane == 0) {
        atomicAdd(&sh.uold, uo);
        atomicAdd(&sh.unew, un);
    }
    if (ok) {
        if (inserts) {
            map_insert_finish(md, lkey, slot, ih, iprev);
            md.leaf_key[slot] = lkey;
        }
        if (lane < kLeafPages) md.leaf_page[(size_t)slot * kLeafPages + lane] = (int)wi[8 + lane];
        if (lane < kMaskWords) md.leaf_occ[(size_t)slot * kMaskWords + lane] = occ | tw;
    }
    if (lane == 0) {
        md.skeys[pos] = kEmptyKey;
        md.pos_count[pos] = 0u;
        md.pos_slab[pos] = 0u;
    }
    wave_sync();
}

// The accumulation kernel's work of one map's frame for blocks blk, blk + nblk,
// ...: the leaves done by a workgroup (the larger ones first), then groups of
// four small leaves, one per wave.  Its statistics are added to the frame's.
template <int KMAX, int FR>
__device__ __forceinline__ void leaf_acc_range(const FrameParams &fp, const MapDev &md, AccShared<KMAX, FR> &sh,
                                               uint32_t blk, uint32_t nblk)
{
    const DevState *st = md.st;
    const unsigned long long lused = st->leaves_used;
    const bool ok = md.fs->frame_err.v == 0 && st->pass_failed == 0 &&
                    lused + md.fs->new_leaves.v <= (unsigned long long)md.max_leaves &&
                    st->pages_used + md.fs->new_pages.v <= (unsigned long long)md.max_pages;
    if (threadIdx.x == 0) {
        sh.uold = 0;
        sh.unew = 0;
    }
    __syncthreads();
    const uint32_t medf = (uint32_t)md.fs->n_lists, smallf = (uint32_t)(md.fs->n_lists >> 32);
    const uint32_t nmed = medf + (uint32_t)md.fs->n_lists_tail;
    const uint32_t nsmall = smallf + (uint32_t)(md.fs->n_lists_tail >> 32);
    const uint32_t last = md.hmask;
    const uint32_t nw = blockDim.x >> 6, w = threadIdx.x >> 6;
    const uint32_t nunits = nmed + (nsmall + nw - 1) / nw;
    const FixScale fx = fix_scale(fp);
    const int nf = fp.nsub > 1 ? fp.nsub : 1;
    for (uint32_t u = blk; u < nunits; u += nblk) {
        if (u < nmed) {
            acc_block_unit<KMAX, FR>(fp, md, sh, &md.items[u < medf ? u : last - (u - medf)], lused, ok, fx, nf);
        } else {
            const uint32_t k = (u - nmed) * nw + w;
            if (k < nsmall)
                acc_wave_unit<KMAX, FR>(fp, md, sh, &md.items_small[k < smallf ? k : last - (k - smallf)], lused, ok,
                                        fx, nf);
            __syncthreads();
        }
    }
    __syncthreads();
    if (threadIdx.x == 0 && (sh.uold | sh.unew))
        atomicAdd(&md.fs->stat[blk & 63u].v, ((unsigned long long)sh.unew << 32) | sh.uold);
    __syncthreads();
}

template <int KMAX, int FR>
__global__ __launch_bounds__(kLeafThreads, 3) void k_leaf_acc(FrameParams fp, MapDev md)
{
    __shared__ AccShared<KMAX, FR> sh;
    leaf_acc_range<KMAX, FR>(fp, md, sh, blockIdx.x, gridDim.x);
}

// The maps mb.subset[0 .. nsubset) of a batch (one frame each), all of this
// kernel's kind, each on its share of the grid.
template <int KMAX>
__global__ __launch_bounds__(kLeafThreads, 3) void k_leaf_acc_batch(MapBatch mb)
{
    __shared__ AccShared<KMAX, 1> sh;
    const int q = batch_map(mb.part_first, mb.nsubset, blockIdx.x), i = mb.subset[q];
    leaf_acc_range<KMAX, 1>(mb.fps[i], mb.mds[i], sh, blockIdx.x - mb.part_first[q],
                            mb.part_first[q + 1] - mb.part_first[q]);
}

// One wave per voxel descriptor of the frame (open set, wide class counts,
// most-recent open set): the combine of the wave-per-voxel leaf kernels, run
// over all voxels of the frame at once so that the heavy voxels spread over the
// whole GPU.  Consecutive descriptors (neighbouring voxels, which share
// observations) go to workgroups on the same XCD.
template <int KMAX, int J = kWaveComps>
__device__ __forceinline__ void voxel_combine_range(const FrameParams &fp, const MapDev &md, uint32_t blk,
                                                    uint32_t nblk)
{
    const uint32_t nv = md.fs->n_vox.v;
    const uint32_t nw = blockDim.x >> 6, w = threadIdx.x >> 6;
    // blocks are dealt to the 8 XCDs round robin: give each XCD a contiguous
    // share (XCD r holds the nblk / 8 blocks, plus one if r < nblk % 8, whose
    // index is r modulo 8; a one-to-one map of [0, nblk) for any nblk)
    const uint32_t r = blk % 8, q = nblk / 8, m = nblk % 8;
    const uint32_t vb = r * q + min(r, m) + blk / 8;
    const uint32_t step = nblk * nw;
    if constexpr (KMAX >= 8) {
        // L >= 512: a wave's voxels one after another, each one's descriptor requested
        // two voxels ahead and its observations' point indices and distances
        // one voxel ahead, so that only the rows and the record are waited
        // for (indices past the end read the wave's first voxel again)
        const uint32_t lane = (uint32_t)lane_id();
        const uint32_t v0 = vb * nw + w;
        if (v0 >= nv) return;
        uint4 d = md.vox_list[v0];
        uint32_t kl = lane < (d.y & 0x7FFFFFFFu) ? md.pair_key[d.z + lane] & kPidMask : 0u;
        float vl = lane < (d.y & 0x7FFFFFFFu) ? md.pair_tsdf[d.z + lane] : 0.0f;
        uint32_t vn = v0 + step;
        uint4 dn = md.vox_list[vn < nv ? vn : v0];
        for (;;) {
            const bool more = vn < nv;
            const uint32_t nn = more ? dn.y & 0x7FFFFFFFu : 0u;
            const uint32_t kn = lane < nn ? md.pair_key[dn.z + lane] & kPidMask : 0u;
            const float vln = lane < nn ? md.pair_tsdf[dn.z + lane] : 0.0f;
            const uint32_t vnn = vn + step;
            const uint4 dnn = md.vox_list[vnn < nv ? vnn : v0];
            combine_wave_vec<(KMAX > 0 ? KMAX : 1)>(fp, md, md.pair_key + d.z, md.pair_tsdf + d.z,
                                                    d.y & 0x7FFFFFFFu, (long long)d.x, (d.y >> 31) != 0u, kl, vl);
            if (!more) break;
            d = dn;
            kl = kn;
            vl = vln;
            vn = vnn;
            dn = dnn;
        }
    } else {
        // the other kinds one voxel at a time: for L <= 256 (few observations
        // per voxel) requesting ahead gains nothing and costs the registers
        // of more waves
        for (uint32_t v = vb * nw + w; v < nv; v += step) {
            const uint4 d = md.vox_list[v];
            const uint32_t n = d.y & 0x7FFFFFFFu;
            const bool existed = (d.y >> 31) != 0u;
            const uint32_t *keys = md.pair_key + d.z;
            const float *vals = md.pair_tsdf + d.z;
            if constexpr (KMAX > 0)
                combine_wave_vec<(KMAX > 0 ? KMAX : 1)>(fp, md, keys, vals, n, (long long)d.x, existed);
            else if constexpr (KMAX < 0)
                combine_last_wave(fp, md, keys, vals, n, (long long)d.x, existed);
            else
                combine_wave<J>(fp, md, keys, vals, n, (long long)d.x, existed);
        }
    }
}

// The wave combine of the maps mb.subset[0 .. nsubset) of a batch in one
// launch: their voxel lists are taken as one list, map after map, and the
// whole grid strides over it as voxel_combine_range does over one map's, so
// that the work spreads evenly whatever the maps' sizes.
constexpr int kMaxBatchMaps = 1024;
template <int KMAX>
__device__ __forceinline__ void voxel_combine_maps(const MapBatch &mb, uint32_t blk, uint32_t nblk)
{
    __shared__ uint32_t pre[kMaxBatchMaps + 1];  // first voxel of each map in the joint list, then the total
    __shared__ uint32_t wsum[4];
    const int ns = min(mb.nsubset, kMaxBatchMaps), tid = threadIdx.x;
    uint32_t c[4], t = 0;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int q = tid * 4 + u;
        c[u] = q < ns ? mb.mds[mb.subset[q]].fs->n_vox.v : 0u;
        t += c[u];
    }
    const uint32_t incl = wave_incl_scan(t);
    if (lane_id() == 63) wsum[tid >> 6] = incl;
    __syncthreads();
    uint32_t run = incl - t;
    for (int w = 0; w < (tid >> 6); ++w) run += wsum[w];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int q = tid * 4 + u;
        if (q < ns) pre[q] = run;
        run += c[u];
    }
    if (tid == 0) pre[ns] = wsum[0] + wsum[1] + wsum[2] + wsum[3];
    __syncthreads();
    const uint32_t nv = pre[ns];
    const uint32_t nw = blockDim.x >> 6, w = tid >> 6;
    // the XCD deal of voxel_combine_range
    const uint32_t r = blk % 8, qb = nblk / 8, m = nblk % 8;
    const uint32_t vb = r * qb + min(r, m) + blk / 8;
    const uint32_t step = nblk * nw;
    int q = 0;
    for (uint32_t v = vb * nw + w; v < nv; v += step) {
        while (pre[q + 1] <= v) ++q;  // the map of joint voxel v (pre[ns] = nv > v)
        const int i = mb.subset[q];
        const MapDev &md = mb.mds[i];
        const FrameParams &fp = mb.fps[i];
        const uint4 d = md.vox_list[v - pre[q]];
        const uint32_t n = d.y & 0x7FFFFFFFu;
        const bool existed = (d.y >> 31) != 0u;
        const uint32_t *keys = md.pair_key + d.z;
        const float *vals = md.pair_tsdf + d.z;
        if constexpr (KMAX > 0)
            combine_wave_vec<(KMAX > 0 ? KMAX : 1)>(fp, md, keys, vals, n, (long long)d.x, existed);
        else if constexpr (KMAX < 0)
            combine_last_wave(fp, md, keys, vals, n, (long long)d.x, existed);
        else
            combine_wave<kWaveComps>(fp, md, keys, vals, n, (long long)d.x, existed);
    }
}

// Workgroups per CU the combine kernels are built for: the vectorised kinds are
// bound by the latency of their row and record accesses, so they keep enough
// waves in flight (register budgets 72, 100, 72, 168 for L = 64, 128, 256, 512).
__host__ __device__ constexpr int combine_min_blocks(int kmax)
{
    return kmax == 1 ? 7 : (kmax == 2 ? 5 : (kmax == 4 ? 7 : (kmax == 8 ? 3 : 1)));
}

// and the general one with J components per lane
__host__ __device__ constexpr int general_min_blocks(int j) { return j == 1 ? 7 : (j == 2 ? 6 : (j == 4 ? 4 : 1)); }

template <int KMAX, int J = kWaveComps>
__global__ __launch_bounds__(256, KMAX == 0 ? general_min_blocks(J) : combine_min_blocks(KMAX)) void k_voxel_combine(
    FrameParams fp, MapDev md)
{
    voxel_combine_range<KMAX, J>(fp, md, blockIdx.x, gridDim.x);
}

template <int KMAX>
__global__ __launch_bounds__(256, combine_min_blocks(KMAX)) void k_voxel_combine_batch(MapBatch mb)
{
    voxel_combine_maps<KMAX>(mb, blockIdx.x, gridDim.x);
}

// ---------------------------------------------------------------------------
// 5. commit (one workgroup)
// ---------------------------------------------------------------------------

// By the first wave.  Its time is one round trip for all counters, then the
// stores: the leaf kernel's statistics are 64 words, one a lane (4,096 workgroups
// left a word each before, summed by 256 threads with a barrier per halving: 6.3 us
// a frame, now 4.3).
__device__ __forceinline__ void frame_commit_block(const FrameParams &fp, const MapDev &md)
{
    if (threadIdx.x >= 64) return;
    DevState *st = md.st;
    const unsigned long long stat = md.fs->stat[threadIdx.x].v;
    md.fs->stat[threadIdx.x].v = 0ull;
    unsigned long long nl = 0, np = 0, lu = 0, pu = 0, vu = 0;
    uint32_t ferr = 0, nrej = 0, npairs = 0, ntouch = 0;
    int failed = 0, status = 0;
    if (threadIdx.x == 0) {
        nl = md.fs->new_leaves.v;
        np = md.fs->new_pages.v;
        ferr = md.fs->frame_err.v;
        nrej = md.fs->rejected.v;
        npairs = md.fs->pairs.v;
        ntouch = md.fs->n_touched.v;
        failed = st->pass_failed;
        status = st->status;
        lu = st->leaves_used;
        pu = st->pages_used;
        vu = st->voxels_used;
    }
    const unsigned long long uo = (unsigned long long)wave_sum_i64((long long)(stat & 0xFFFFFFFFull));
    const unsigned long long un = (unsigned long long)wave_sum_i64((long long)(stat >> 32));
    if (threadIdx.x == 0) {
        // after a multi-frame pass that could not be applied, the frames that
        // follow it in the same sequence call are skipped too: the host
        // integrates them again one by one
        const bool skipped = failed != 0;
        const bool ok = !skipped && ferr == 0 && lu + nl <= (unsigned long long)md.max_leaves &&
                        pu + np <= (unsigned long long)md.max_pages;
        if (ok) {
            st->leaves_used = lu + nl;
            st->pages_used = pu + np;
            st->voxels_used = vu + un;
        } else if (!skipped && fp.nsub > 1) {
            st->pass_failed = 1 + fp.pass_first;
        } else if (!skipped && status == SLIM_OK) {
            st->status = SLIM_ERR_CAPACITY;
        }
        if (!skipped && (ok || fp.nsub <= 1)) {
            st->last_points = fp.n;
            st->last_rejected = nrej;
            st->last_pairs = npairs;
            st->last_touched = ntouch;
            st->last_new_leaves = nl;
            st->last_u_old = (long long)uo;
            st->last_u_new = (long long)un;
            st->last_status = ok ? SLIM_OK : SLIM_ERR_CAPACITY;
        }
        md.fs->n_touched.v = 0;
        md.fs->pairs.v = 0;
        md.fs->rejected.v = 0;
        md.fs->new_leaves.v = 0;
        md.fs->new_pages.v = 0;
        md.fs->pair_cursor.v = 0;
        md.fs->work_big.v = 0;
        md.fs->n_lists = 0;
        md.fs->n_lists_tail = 0;
        md.fs->n_vox.v = 0;
        md.fs->frame_err.v = 0;
    }
}

__global__ __launch_bounds__(64) void k_frame_commit(FrameParams fp, MapDev md)
{
    frame_commit_block(fp, md);
}

__global__ __launch_bounds__(64) void k_frame_commit_batch(MapBatch mb)
{
    frame_commit_block(mb.fps[blockIdx.x], mb.mds[blockIdx.x]);
}

// ---------------------------------------------------------------------------
// 6. the persistent batched launch
// ---------------------------------------------------------------------------
//
// One launch integrates one frame into each of many maps.  Its workgroups stay
// resident and take work items from an integer queue in order: the ray-chunk
// items of every map's walk, then every map's planning, emitting, leaf-tile,
// voxel-combine and commit items.  An item of a stage starts once all items of
// the previous stage of the same map have finished (a per-map, per-stage
// counter), so the stages of different maps overlap and a large frame does
// not hold up a small one.  Items are taken in queue order and an item only
// waits for items earlier in the queue, which are held by running workgroups:
// the queue always drains, whatever the number of workgroups.  Every item runs
// the same code as the per-stage kernels, so the maps are bitwise the same as
// after the per-stage launches (and the per-map calls).

// Leaf-kernel variants whose voxels are combined by k_voxel_combine (one wave
// per voxel), with that kernel's template argument; -2: combined in the leaf kernel.
__host__ __device__ int voxel_combine_arg(int kind)
{
    switch (kind) {
    case 8: return 0;
    case 10: return -1;
    case 11: return 1;
    case 12: return 2;
    case 13: return 4;
    case 14: return 8;
    case 15: return 16;
    default: return -2;
    }
}

static_assert(kWalkThreads == 256 && kLeafThreads == 256, "persistent items assume 256-thread workgroups");

union PersistShared {
    WalkShared walk;
    LeafShared leaf;
    AccShared<0, 1> acc0;
    AccShared<8, 1> acc8;
    AccShared<16, 1> acc16;
    AccShared<24, 1> acc24;
    AccShared<32, 1> acc32;
};
// The launch's LDS, one copy per workgroup, named directly by the stage
// functions below (a reference passed to a called function would lose its
// address space).
static __shared__ PersistShared g_ps;

template <int KMAX>
__device__ __forceinline__ AccShared<KMAX, 1> &persist_acc_lds()
{
    if constexpr (KMAX == 0) return g_ps.acc0;
    else if constexpr (KMAX == 8) return g_ps.acc8;
    else if constexpr (KMAX == 16) return g_ps.acc16;
    else if constexpr (KMAX == 24) return g_ps.acc24;
    else return g_ps.acc32;
}

// A waiting workgroup gives up after this many polls (seconds), raises the
// launch's abort flag and marks its map failed: every later item is then
// skipped, so the launch always ends.  The queue order makes this unreachable
// in a correct launch; it is a guard against a broken item list.
constexpr uint32_t kPersistSpinLimit = 1u << 22;

// Arguments of a called stage function arrive in vector registers; the
// workgroup's item is the same in every lane, so they are taken back as
// wave-uniform values on entry.
__device__ __forceinline__ uint32_t uni(uint32_t v) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)v); }

template <class T>
__device__ __forceinline__ const T &uni_ref(const T &r)
{
    const unsigned long long p = (unsigned long long)&r;
    return *(const T *)(((unsigned long long)uni((uint32_t)(p >> 32)) << 32) | uni((uint32_t)p));
}

// Each stage variant is a function of its own (called, not inlined), so it is
// register-allocated alone, as in its own kernel.
__device__ __noinline__ void persist_walk(const FrameParams &fpa, const MapDev &mda, uint32_t b0a, uint32_t nba)
{
    const FrameParams &fp = uni_ref(fpa);
    const MapDev &md = uni_ref(mda);
    const uint32_t b0 = uni(b0a), b1 = b0 + uni(nba);
    for (uint32_t b = b0; b < b1; ++b) {
        walk_block(fp, md, (int)b, (int)b, g_ps.walk);
        __syncthreads();
    }
}

__device__ __noinline__ void persist_plan(const FrameParams &fp, const MapDev &md, uint32_t j, uint32_t cnt)
{
    leaf_plan_range(uni_ref(fp), uni_ref(md), uni(j), uni(cnt));
}

__device__ __noinline__ void persist_bucket(const FrameParams &fp, const MapDev &md, uint32_t j, uint32_t cnt)
{
    ray_emit_range(uni_ref(fp), uni_ref(md), uni(j), uni(cnt));
}

template <int KMAX>
__device__ __noinline__ void persist_acc(const FrameParams &fp, const MapDev &md, uint32_t j, uint32_t cnt)
{
    leaf_acc_range<KMAX, 1>(uni_ref(fp), uni_ref(md), persist_acc_lds<KMAX>(), uni(j), uni(cnt));
}

template <int KMAX, bool WAVE, bool ROWS>
__device__ __noinline__ void persist_fuse(const FrameParams &fp, const MapDev &md, uint32_t j, uint32_t cnt)
{
    leaf_fuse_range<KMAX, WAVE, ROWS>(uni_ref(fp), uni_ref(md), g_ps.leaf, uni(j), uni(cnt));
}

template <int KMAX>
__device__ __noinline__ void persist_comb(const FrameParams &fp, const MapDev &md, uint32_t j, uint32_t cnt)
{
    voxel_combine_range<KMAX>(uni_ref(fp), uni_ref(md), uni(j), uni(cnt));
}

__device__ __noinline__ void persist_commit(const FrameParams &fp, const MapDev &md)
{
    frame_commit_block(uni_ref(fp), uni_ref(md));
}

__device__ __forceinline__ void persist_leaf(int kind, const FrameParams &fp, const MapDev &md, uint32_t j,
                                             uint32_t cnt)
{
    switch (kind) {
    case 0: persist_acc<0>(fp, md, j, cnt); break;
    case 1: persist_acc<8>(fp, md, j, cnt); break;
    case 2: persist_acc<16>(fp, md, j, cnt); break;
    case 3: persist_acc<24>(fp, md, j, cnt); break;
    case 4: persist_acc<32>(fp, md, j, cnt); break;
    case 5: persist_fuse<8, false, true>(fp, md, j, cnt); break;
    case 6: persist_fuse<16, false, true>(fp, md, j, cnt); break;
    case 7: persist_fuse<32, false, true>(fp, md, j, cnt); break;
    case 16: persist_fuse<24, false, true>(fp, md, j, cnt); break;
    case 9: persist_fuse<-1, false, false>(fp, md, j, cnt); break;
    case 10: persist_fuse<-1, true, false>(fp, md, j, cnt); break;
    case 11: persist_fuse<1, true, false>(fp, md, j, cnt); break;
    case 12: persist_fuse<2, true, false>(fp, md, j, cnt); break;
    case 13: persist_fuse<4, true, false>(fp, md, j, cnt); break;
    case 14: persist_fuse<8, true, false>(fp, md, j, cnt); break;
    case 15: persist_fuse<16, true, false>(fp, md, j, cnt); break;
    default: persist_fuse<0, true, false>(fp, md, j, cnt); break;
    }
}

__device__ __forceinline__ void persist_combine(int kind, const FrameParams &fp, const MapDev &md, uint32_t j,
                                                uint32_t cnt)
{
    switch (voxel_combine_arg(kind)) {
    case 0: persist_comb<0>(fp, md, j, cnt); break;
    case -1: persist_comb<-1>(fp, md, j, cnt); break;
    case 1: persist_comb<1>(fp, md, j, cnt); break;
    case 2: persist_comb<2>(fp, md, j, cnt); break;
    case 4: persist_comb<4>(fp, md, j, cnt); break;
    case 8: persist_comb<8>(fp, md, j, cnt); break;
    case 16: persist_comb<16>(fp, md, j, cnt); break;
    default: break;
    }
}

__global__ __launch_bounds__(256, 3) void k_batch_persistent(PersistArgs a)
{
    __shared__ uint4 s_item;
    __shared__ uint32_t s_skip;
    // Thread 0 alone talks to the queue, in one place per round: it counts the
    // item the workgroup has just finished (after the release below), takes
    // the next one and waits for its dependency.  Keeping that one guarded
    // region per round, and the item wave-uniform, keeps every barrier of the
    // loop in uniform control flow.
    uint32_t finished = kPersistEnd;  // counter of the item the workgroup finished last
    for (;;) {
        if (threadIdx.x == 0) {
            if (finished != kPersistEnd) atomicAdd(&a.ctl[kPersistCtlDone + finished], 1u);
            const uint32_t it = atomicAdd(&a.ctl[0], 1u);
            uint4 item = make_uint4(kPersistEnd, 0u, 0u, 0u);
            uint32_t skip = 0;
            if (it < a.nitems) {
                item = a.items[it];
                if (item.w != kPersistNoDep) {
                    // wait for every item of the map's previous stage
                    const uint32_t *done = &a.ctl[kPersistCtlDone + (item.w & 0xFFFFu)];
                    const uint32_t need = item.w >> 16;
                    uint32_t polls = 0;
                    while (__hip_atomic_load(done, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < need) {
                        if (++polls > kPersistSpinLimit) {
                            atomicOr(&a.ctl[kPersistCtlAbort], 1u);
                            break;
                        }
                        __builtin_amdgcn_s_sleep(2);
                    }
                }
                skip = __hip_atomic_load(&a.ctl[kPersistCtlAbort], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                __threadfence();
                // after an abort the map's remaining items are skipped and the map is marked failed
                const DevState *st = a.mds[item.x & 0xFFFFu].st;
                if (skip && st->status == SLIM_OK) ((DevState *)st)->status = SLIM_ERR_DEVICE;
            }
            s_item = item;
            s_skip = skip;
        }
        __syncthreads();
        // every thread reads the same item: taken as wave-uniform values, so
        // the loop and its exit stay uniform
        const uint4 item = make_uint4(__builtin_amdgcn_readfirstlane(s_item.x), __builtin_amdgcn_readfirstlane(s_item.y),
                                      __builtin_amdgcn_readfirstlane(s_item.z), __builtin_amdgcn_readfirstlane(s_item.w));
        const uint32_t skip = __builtin_amdgcn_readfirstlane(s_skip);
        if (item.x == kPersistEnd) break;
        // acquire (every wave): what the previous stage wrote on other XCDs is visible
        __threadfence();
        const uint32_t i = item.x & 0xFFFFu, stage = (item.x >> 16) & 0xFFu;
        const int kind = (int)(item.x >> 24);
        const FrameParams &fp = a.fps[i];
        const MapDev &md = a.mds[i];
        if (!skip) {
            switch (stage) {
            case 0: persist_walk(fp, md, item.y, item.z); break;
            case 1: persist_plan(fp, md, item.y, item.z); break;
            case 2: persist_bucket(fp, md, item.y, item.z); break;
            case 3: persist_leaf(kind, fp, md, item.y, item.z); break;
            case 4: persist_combine(kind, fp, md, item.y, item.z); break;
            default: persist_commit(fp, md); break;
            }
        }
        // release: this item's writes reach the device level before thread 0
        // counts it, at the top of the next round
        __threadfence();
        __syncthreads();
        finished = i * kPersistStages + stage;
    }
}

int persistent_blocks_per_cu()
{
    int nb = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, k_batch_persistent, 256, 0) != hipSuccess) return 1;
    return nb > 0 ? nb : 1;
}

hipError_t launch_integrate_persistent(const PersistArgs &a, int blocks, hipStream_t s)
{
    hipLaunchKernelGGL(k_batch_persistent, dim3(blocks > 0 ? blocks : 1), dim3(256), 0, s, a);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------

// Variant of the leaf kernel a frame needs: 0 geometry; 1..4 labels with
// 8/16/24/32 classes in registers; 5..7 probability or logit rows with 8/16/32 (17..24 classes: 16);
// 8 one wave per voxel (open set, or more than 32 classes); 9 and 10 the
// most-recent-measurement modes (closed: lane per voxel; open: wave per voxel);
// 11..15 the open set with L = 64, 128, 256, 512, 1024 read as whole words;
// 16 probability or logit rows with 24 classes in registers.
int leaf_kernel_kind(const FrameParams &fp)
{
    if (fp.last) return fp.L > 0 ? 10 : 9;
    if (fp.L > 0 && (fp.L & 63) == 0 && ((uintptr_t)fp.sem & 15u) == 0) {
        // embeddings whose rows split into whole 4- to 16-byte words per lane
        const int v = fp.L >> 6;
        const bool bf = fp.sem_kind == SLIM_IN_EMB_BF16;
        if (v == 1 && !bf) return 11;
        if (v == 2) return 12;
        if (v == 4) return 13;
        if (v == 8) return 14;
        if (v == 16) return 15;
    }
    if (fp.L > 0 || fp.K > 32) return 8;
    if (fp.K == 0) return 0;
    const bool rows = fp.sem_kind == SLIM_IN_PROB_F32 || fp.sem_kind == SLIM_IN_LOGIT_F32;
    if (rows) return fp.K > 24 ? 7 : (fp.K > 16 ? 16 : (fp.K > 8 ? 6 : 5));
    return fp.K > 24 ? 4 : (fp.K > 16 ? 3 : (fp.K > 8 ? 2 : 1));
}

// Grid of the wave combine.  Its blocks take equal static shares of the
// voxels, so the kinds built for 3 or 7 workgroups per CU (L = 512, 256 as
// whole words) run two rounds of what the CUs hold at once, the others the leaf
// kernel's grid.
int combine_blocks(int kind, const LaunchShape &shape)
{
    const int k = voxel_combine_arg(kind);
    return (k == 4 || k == 8) ? 2 * combine_min_blocks(k) * shape.cus : shape.leaf_blocks;
}

static void launch_voxel_combine(int kind, const FrameParams &fp, const MapDev &md, int blocks, hipStream_t s)
{
    const dim3 gl(blocks), bl(256);
    switch (voxel_combine_arg(kind)) {
    case 0: {
        // as many components per lane as the rows need: with 16 for every length,
        // rows of 100 components (2 per lane) went through 8 times the instructions
        // in 4 waves per CU; 18,600 voxels with 216,000 such rows 247 -> 43 us
        const int c = fp.L > 0 ? fp.L : fp.K;
        if (c <= 64) hipLaunchKernelGGL((k_voxel_combine<0, 1>), gl, bl, 0, s, fp, md);
        else if (c <= 128) hipLaunchKernelGGL((k_voxel_combine<0, 2>), gl, bl, 0, s, fp, md);
        else if (c <= 256) hipLaunchKernelGGL((k_voxel_combine<0, 4>), gl, bl, 0, s, fp, md);
        else hipLaunchKernelGGL((k_voxel_combine<0, 16>), gl, bl, 0, s, fp, md);
        break;
    }
    case -1: hipLaunchKernelGGL((k_voxel_combine<-1>), gl, bl, 0, s, fp, md); break;
    case 1: hipLaunchKernelGGL((k_voxel_combine<1>), gl, bl, 0, s, fp, md); break;
    case 2: hipLaunchKernelGGL((k_voxel_combine<2>), gl, bl, 0, s, fp, md); break;
    case 4: hipLaunchKernelGGL((k_voxel_combine<4>), gl, bl, 0, s, fp, md); break;
    case 8: hipLaunchKernelGGL((k_voxel_combine<8>), gl, bl, 0, s, fp, md); break;
    case 16: hipLaunchKernelGGL((k_voxel_combine<16>), gl, bl, 0, s, fp, md); break;
    default: break;
    }
}

static void launch_voxel_combine_batch(int kind, const MapBatch &mb, int blocks, hipStream_t s)
{
    const dim3 gl(blocks), bl(256);
    switch (voxel_combine_arg(kind)) {
    case 0: hipLaunchKernelGGL((k_voxel_combine_batch<0>), gl, bl, 0, s, mb); break;
    case -1: hipLaunchKernelGGL((k_voxel_combine_batch<-1>), gl, bl, 0, s, mb); break;
    case 1: hipLaunchKernelGGL((k_voxel_combine_batch<1>), gl, bl, 0, s, mb); break;
    case 2: hipLaunchKernelGGL((k_voxel_combine_batch<2>), gl, bl, 0, s, mb); break;
    case 4: hipLaunchKernelGGL((k_voxel_combine_batch<4>), gl, bl, 0, s, mb); break;
    case 8: hipLaunchKernelGGL((k_voxel_combine_batch<8>), gl, bl, 0, s, mb); break;
    case 16: hipLaunchKernelGGL((k_voxel_combine_batch<16>), gl, bl, 0, s, mb); break;
    default: break;
    }
}

static void launch_leaf(int kind, const FrameParams &fp, const MapDev &md, int blocks, hipStream_t s)
{
    const dim3 gl(blocks), bl(kLeafThreads);
    if (kind <= 4) {
        // accumulating kernel with one set of accumulators per frame of the pass
        const int fr = fp.nsub <= 1 ? 1 : (fp.nsub == 2 ? 2 : (fp.nsub <= 4 ? 4 : 8));
        const int kmax = kind * 8;
#define SLIM_ACC(K, F) \
    if (kmax == K && fr == F) hipLaunchKernelGGL((k_leaf_acc<K, F>), gl, bl, 0, s, fp, md);
        SLIM_ACC(0, 1) SLIM_ACC(0, 2) SLIM_ACC(0, 4) SLIM_ACC(8, 1) SLIM_ACC(8, 2) SLIM_ACC(8, 4)
        SLIM_ACC(16, 1) SLIM_ACC(16, 2) SLIM_ACC(16, 4) SLIM_ACC(24, 1) SLIM_ACC(24, 2) SLIM_ACC(24, 4)
        SLIM_ACC(32, 1) SLIM_ACC(32, 2) SLIM_ACC(32, 4) SLIM_ACC(0, 8) SLIM_ACC(8, 8) SLIM_ACC(16, 8)
        SLIM_ACC(24, 8) SLIM_ACC(32, 8)
#undef SLIM_ACC
        return;
    }
    switch (kind) {
    case 5: hipLaunchKernelGGL((k_leaf_fuse<8, false, true>), gl, bl, 0, s, fp, md); break;
    case 6: hipLaunchKernelGGL((k_leaf_fuse<16, false, true>), gl, bl, 0, s, fp, md); break;
    case 7: hipLaunchKernelGGL((k_leaf_fuse<32, false, true>), gl, bl, 0, s, fp, md); break;
    case 16: hipLaunchKernelGGL((k_leaf_fuse<24, false, true>), gl, bl, 0, s, fp, md); break;
    case 9: hipLaunchKernelGGL((k_leaf_fuse<-1, false, false>), gl, bl, 0, s, fp, md); break;
    case 10: hipLaunchKernelGGL((k_leaf_fuse<-1, true, false>), gl, bl, 0, s, fp, md); break;
    case 11: hipLaunchKernelGGL((k_leaf_fuse<1, true, false>), gl, bl, 0, s, fp, md); break;
    case 12: hipLaunchKernelGGL((k_leaf_fuse<2, true, false>), gl, bl, 0, s, fp, md); break;
    case 13: hipLaunchKernelGGL((k_leaf_fuse<4, true, false>), gl, bl, 0, s, fp, md); break;
    case 14: hipLaunchKernelGGL((k_leaf_fuse<8, true, false>), gl, bl, 0, s, fp, md); break;
    case 15: hipLaunchKernelGGL((k_leaf_fuse<16, true, false>), gl, bl, 0, s, fp, md); break;
    default: hipLaunchKernelGGL((k_leaf_fuse<0, true, false>), gl, bl, 0, s, fp, md); break;
    }
}

static void launch_leaf_batch(int kind, const MapBatch &mb, int blocks, hipStream_t s)
{
    const dim3 gl(blocks), bl(kLeafThreads);
    switch (kind) {
    case 0: hipLaunchKernelGGL((k_leaf_acc_batch<0>), gl, bl, 0, s, mb); break;
    case 1: hipLaunchKernelGGL((k_leaf_acc_batch<8>), gl, bl, 0, s, mb); break;
    case 2: hipLaunchKernelGGL((k_leaf_acc_batch<16>), gl, bl, 0, s, mb); break;
    case 3: hipLaunchKernelGGL((k_leaf_acc_batch<24>), gl, bl, 0, s, mb); break;
    case 4: hipLaunchKernelGGL((k_leaf_acc_batch<32>), gl, bl, 0, s, mb); break;
    case 5: hipLaunchKernelGGL((k_leaf_fuse_batch<8, false, true>), gl, bl, 0, s, mb); break;
    case 6: hipLaunchKernelGGL((k_leaf_fuse_batch<16, false, true>), gl, bl, 0, s, mb); break;
    case 7: hipLaunchKernelGGL((k_leaf_fuse_batch<32, false, true>), gl, bl, 0, s, mb); break;
    case 16: hipLaunchKernelGGL((k_leaf_fuse_batch<24, false, true>), gl, bl, 0, s, mb); break;
    case 9: hipLaunchKernelGGL((k_leaf_fuse_batch<-1, false, false>), gl, bl, 0, s, mb); break;
    case 10: hipLaunchKernelGGL((k_leaf_fuse_batch<-1, true, false>), gl, bl, 0, s, mb); break;
    case 11: hipLaunchKernelGGL((k_leaf_fuse_batch<1, true, false>), gl, bl, 0, s, mb); break;
    case 12: hipLaunchKernelGGL((k_leaf_fuse_batch<2, true, false>), gl, bl, 0, s, mb); break;
    case 13: hipLaunchKernelGGL((k_leaf_fuse_batch<4, true, false>), gl, bl, 0, s, mb); break;
    case 14: hipLaunchKernelGGL((k_leaf_fuse_batch<8, true, false>), gl, bl, 0, s, mb); break;
    case 15: hipLaunchKernelGGL((k_leaf_fuse_batch<16, true, false>), gl, bl, 0, s, mb); break;
    default: hipLaunchKernelGGL((k_leaf_fuse_batch<0, true, false>), gl, bl, 0, s, mb); break;
    }
}

// Frames whose large leaves are binned.  The two launches cost about 10 us and
// save what the x-slab items read more than once, which grows with the square of
// the points per leaf.  The points of the frame stand for those of a leaf, which the
// host does not know.  A frame with slabs and binned: LiDAR rays with 20-class rows,
// voxel 0.1 m, 66,000 rays 73 and 79 us, 80,000 81 and 85, 100,000 94 and 92, 131,071
// 120 and 110; voxel 0.2 m, 66,000 rays 186 and 121, 131,071 498 and 197; depth images
// at 2 cm, 100-d embeddings, 19,200 pixels 75 and 86, 33,338 101 and 93, 62,208 141 and
// 110, 76,800 165 and 123, 512-d, 307,200 pixels 544 and 104 in the leaf stage alone.
// The line keeps sweeps of up to 65,536 rays with the slabs; dense images would gain
// from half of it on.  Batched and persistent calls always have the slabs: they have no
// stages for the binning.
constexpr int kBinPoints = 65536;

static bool bins_large_leaves(const FrameParams &fp) { return !accum_path(fp) && fp.n > kBinPoints; }

static void launch_emit(const FrameParams &fp, const MapDev &md, const LaunchShape &shape, const PassWalk *pw,
                        hipStream_t s)
{
    if (pw) {
        const int nb = pw->blk_start[pw->nframes];
        hipLaunchKernelGGL(k_ray_emit_pass, dim3(nb > 0 ? nb : 1), dim3(kWalkThreads), 0, s, *pw, md);
    } else {
        const int bw = (fp.n + kWalkThreads - 1) / kWalkThreads;
        const dim3 grid(std::max(1, std::min(bw, shape.bucket_blocks)));
        if (soft_rows(fp)) hipLaunchKernelGGL(k_ray_emit<true>, grid, dim3(kWalkThreads), 0, s, fp, md);
        else hipLaunchKernelGGL(k_ray_emit<false>, grid, dim3(kWalkThreads), 0, s, fp, md);
    }
    if (md.binned) {
        hipLaunchKernelGGL(k_leaf_count, dim3(4 * shape.cus), dim3(256), 0, s, md);
        hipLaunchKernelGGL(k_leaf_bin, dim3(4 * shape.cus), dim3(256), 0, s, md);
    }
}

hipError_t launch_integrate(const FrameParams &fp, const MapDev &md_in, const LaunchShape &shape, hipStream_t s,
                            hipEvent_t *ev, const PassWalk *pw)
{
    MapDev md = md_in;
    md.binned = bins_large_leaves(fp) ? 1 : 0;
    md.wave_pairs = shape.wave_pairs;
    md.slab_pairs = shape.slab_pairs;
    const int bw = (fp.n + kWalkThreads - 1) / kWalkThreads;
    auto rec = [&](int e) {
        if (ev) (void)hipEventRecord(ev[e], s);
    };
    rec(0);
    if (pw) {
        const int nb = pw->blk_start[pw->nframes];
        hipLaunchKernelGGL(k_ray_walk_pass, dim3(nb > 0 ? nb : 1), dim3(kWalkThreads), 0, s, *pw, md);
    } else {
        hipLaunchKernelGGL(k_ray_walk, dim3(bw > 0 ? bw : 1), dim3(kWalkThreads), 0, s, fp, md);
    }
    rec(1);
    rec(2);
    hipLaunchKernelGGL(k_leaf_plan, dim3(shape.plan_blocks), dim3(256), 0, s, fp, md);
    rec(3);
    rec(4);
    launch_emit(fp, md, shape, pw, s);
    rec(5);
    rec(6);
    const int kind = leaf_kernel_kind(fp);
    launch_leaf(kind, fp, md, shape.leaf_blocks, s);
    rec(7);
    rec(8);
    launch_voxel_combine(kind, fp, md, combine_blocks(kind, shape), s);
    rec(9);
    rec(10);
    hipLaunchKernelGGL(k_frame_commit, dim3(1), dim3(64), 0, s, fp, md);
    rec(11);
    return hipGetLastError();
}

hipError_t launch_walk(const FrameParams &fp, const MapDev &md, hipStream_t s, const PassWalk *pw)
{
    if (pw) {
        const int nb = pw->blk_start[pw->nframes];
        hipLaunchKernelGGL(k_ray_walk_pass, dim3(nb > 0 ? nb : 1), dim3(kWalkThreads), 0, s, *pw, md);
        return hipGetLastError();
    }
    const int bw = (fp.n + kWalkThreads - 1) / kWalkThreads;
    hipLaunchKernelGGL(k_ray_walk, dim3(bw > 0 ? bw : 1), dim3(kWalkThreads), 0, s, fp, md);
    return hipGetLastError();
}

hipError_t launch_after_walk(const FrameParams &fp, const MapDev &md_in, const LaunchShape &shape, hipStream_t s,
                             const PassWalk *pw)
{
    MapDev md = md_in;
    md.binned = bins_large_leaves(fp) ? 1 : 0;
    md.wave_pairs = shape.wave_pairs;
    md.slab_pairs = shape.slab_pairs;
    hipLaunchKernelGGL(k_leaf_plan, dim3(shape.plan_blocks), dim3(256), 0, s, fp, md);
    launch_emit(fp, md, shape, pw, s);
    const int kind = leaf_kernel_kind(fp);
    launch_leaf(kind, fp, md, shape.leaf_blocks, s);
    launch_voxel_combine(kind, fp, md, combine_blocks(kind, shape), s);
    hipLaunchKernelGGL(k_frame_commit, dim3(1), dim3(64), 0, s, fp, md);
    return hipGetLastError();
}

hipError_t launch_integrate_batched(const MapBatch &mb, const BatchPlan &plan, const LaunchShape &shape,
                                    hipStream_t s)
{
    hipLaunchKernelGGL(k_ray_walk_batch, dim3(std::max(plan.walk_blocks, 1)), dim3(kWalkThreads), 0, s, mb);
    hipLaunchKernelGGL(k_leaf_plan_batch, dim3(plan.plan_blocks), dim3(256), 0, s, mb);
    hipLaunchKernelGGL(k_ray_emit_batch, dim3(plan.bucket_blocks), dim3(kWalkThreads), 0, s, mb);
    for (int g = 0; g < plan.ngroups; ++g) {
        MapBatch sub = mb;
        sub.subset = mb.subset + plan.group_begin[g];
        sub.nsubset = plan.group_size[g];
        sub.part_first = mb.part_first + plan.leaf_part[g];
        launch_leaf_batch(plan.group_kind[g], sub, plan.leaf_blocks[g], s);
        sub.part_first = mb.part_first + plan.comb_part[g];
        if (plan.comb_blocks[g] > 0) launch_voxel_combine_batch(plan.group_kind[g], sub, plan.comb_blocks[g], s);
    }
    hipLaunchKernelGGL(k_frame_commit_batch, dim3(plan.nmaps), dim3(64), 0, s, mb);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// map loss and backward (differentiation workload)
// ---------------------------------------------------------------------------

// Record of the voxel with integer key (kx, ky, kz), or -1 if it has W = 0.
__device__ __forceinline__ long long voxel_record(const MapDev &md, int kx, int ky, int kz)
{
    const int slot = map_find(md, pack_leaf(kx >> 3, ky >> 3, kz >> 3));
    if (slot < 0) return -1;
    const int off = ((kx & 7) << 6) | ((ky & 7) << 3) | (kz & 7);
    if (!((md.leaf_occ[(size_t)slot * kMaskWords + (off >> 5)] >> (off & 31)) & 1u)) return -1;
    return (long long)md.leaf_page[(size_t)slot * kLeafPages + (off >> 6)] * kPageVoxels + (off & (kPageVoxels - 1));
}

// Record of the voxel holding world point (x, y, z): floor(x / vs), binary32.
__device__ __forceinline__ long long point_record(const MapDev &md, float vs, float x, float y, float z)
{
    if (!(isfinite(x) && isfinite(y) && isfinite(z))) return -1;
    const float fx = floorf(x / vs), fy = floorf(y / vs), fz = floorf(z / vs);
    const float lim = (float)kKeyLimit;
    if (!(fabsf(fx) < lim && fabsf(fy) < lim && fabsf(fz) < lim)) return -1;
    return voxel_record(md, (int)fx, (int)fy, (int)fz);
}

// Block sum of one float per thread in a fixed tree order (blockDim.x = 256).
__device__ __forceinline__ float block_sum(float v, float *red)
{
    red[threadIdx.x] = v;
    __syncthreads();
    for (int d = kLossThreads / 2; d > 0; d >>= 1) {
        if (threadIdx.x < (unsigned)d) red[threadIdx.x] += red[threadIdx.x + d];
        __syncthreads();
    }
    const float r = red[0];
    __syncthreads();
    return r;
}

// A record's bytes of adj_flag: nonzero once its dL/dD (x) and its dL/dc (y) have been
// written.  Only these and the sample counts are cleared (6 bytes a record instead of
// a row): what has not been written carries zero adjoints into the backward.  Two bytes,
// each only ever set: a voxel listed twice, once without a class, keeps its dL/dc
// whichever comes first.
__global__ __launch_bounds__(256) void k_loss_clear(MapDev md, LossParams lp)
{
    // (records come in pages of 64)
    const size_t pages = (size_t)md.st->pages_used, stride = (size_t)gridDim.x * blockDim.x;
    const size_t t = blockIdx.x * (size_t)blockDim.x + threadIdx.x;
    const int4 zero = make_int4(0, 0, 0, 0);
    for (size_t i = t; i < pages * (kPageVoxels / 4); i += stride) ((int4 *)lp.adj_cnt)[i] = zero;
    for (size_t i = t; i < pages * (kPageVoxels / 8); i += stride) ((int4 *)lp.adj_flag)[i] = zero;
}

// Surface samples: per voxel count (integer, so order-free) and block partials
// of |D| and of the number of samples that land in the map.
__global__ __launch_bounds__(kLossThreads) void k_loss_samples(FrameParams fp, MapDev md, LossParams lp)
{
    __shared__ float red[kLossThreads];
    const long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x;
    float a = 0.0f, c = 0.0f;
    if (i < lp.s) {
        const long long rec = point_record(md, fp.vs, lp.samples[3 * i], lp.samples[3 * i + 1], lp.samples[3 * i + 2]);
        if (rec >= 0) {
            atomicAdd(&lp.adj_cnt[rec], 1);
            a = fabsf(md.vox[(size_t)rec * md.rec_stride]);
            c = 1.0f;
        }
    }
    a = block_sum(a, red);
    c = block_sum(c, red);
    if (threadIdx.x == 0) {
        lp.part[blockIdx.x] = a;
        lp.part_cnt[blockIdx.x] = (int)c;
    }
}

// Voxels: cross-entropy of the Dirichlet predictive (Eq. (7)) at the true class,
// adjoints dL/dc and dL/dD, block partials of the cross-entropy.  Bound by the
// records read and the rows written, both as 16-byte vectors; the number of
// samples in the map is summed by the whole workgroup (one thread did it before:
// 591,000 voxels and 40 blocks of samples 220 -> 51 us).
__global__ __launch_bounds__(kLossThreads) void k_loss_voxels(FrameParams fp, MapDev md, LossParams lp, int nsb)
{
    __shared__ float red[kLossThreads];
    __shared__ int s_mp;
    if (threadIdx.x == 0) s_mp = 0;
    const long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x;
    long long rec = -1;
    int y = -1;
    if (i < lp.m) {
        rec = voxel_record(md, lp.keys[3 * i], lp.keys[3 * i + 1], lp.keys[3 * i + 2]);
        y = lp.labels[i];
    }
    int mp = 0;
    for (int b = threadIdx.x; b < nsb; b += kLossThreads) mp += lp.part_cnt[b];
    __syncthreads();
    if (mp) atomicAdd(&s_mp, mp);
    __syncthreads();
    const float inv_m = 1.0f / (float)lp.m, inv_mp = s_mp > 0 ? 1.0f / (float)s_mp : 0.0f;
    const int K = fp.K;
    float ce = 0.0f;
    if (rec >= 0) {
        const float4 *R = (const float4 *)(md.vox + (size_t)rec * md.rec_stride);
        float4 *A = (float4 *)(lp.adj + (size_t)rec * lp.adj_stride);
        // a label outside [0, K) adds no cross-entropy term (dL/dc = 0);
        // the voxel's surface samples still count
        const bool term = y >= 0 && y < K;
        float tot = (float)K * lp.alpha0, cy = 0.0f, D = 0.0f;
#pragma unroll 4
        for (int v = 0; v < md.rec_stride / 4; ++v) {
            const float4 q = R[v];
            const float x[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int k = 4 * v + e - 2;
                if (k == -2) D = x[e];
                if (k >= 0 && k < K) {
                    tot += x[e];
                    cy = k == y ? x[e] : cy;
                }
            }
        }
        const float ay = lp.alpha0 + cy;
        const float sg = D > 0.0f ? 1.0f : (D < 0.0f ? -1.0f : 0.0f);
        const float ad = sg * (float)lp.adj_cnt[rec] * inv_mp;
        if (term) {
            const float g = inv_m / tot, gy = g - inv_m / ay;
            ce = -logf(ay / tot);
            for (int v = 0; v < lp.adj_stride / 4; ++v) {
                float x[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int k = 4 * v + e;
                    x[e] = k < K ? (k == y ? gy : g) : (k == K ? ad : 0.0f);
                }
                A[v] = make_float4(x[0], x[1], x[2], x[3]);
            }
            lp.adj_flag[rec].y = 1;
        } else {
            ((float *)A)[K] = ad;
        }
        lp.adj_flag[rec].x = 1;
    }
    ce = block_sum(ce, red);
    if (threadIdx.x == 0) lp.part[nsb + blockIdx.x] = ce;
}

// Sums of the block partials, by one workgroup: each thread strides over them,
// then a fixed tree, in binary64 (2,310 partials one after the other took 95 us,
// this 5 us).
__global__ __launch_bounds__(kLossThreads) void k_loss_final(LossParams lp, int nsb, int nvb)
{
    __shared__ double s_l1[kLossThreads], s_ce[kLossThreads];
    __shared__ int s_mp[kLossThreads];
    const int t = threadIdx.x;
    double l1 = 0.0, ce = 0.0;
    int mp = 0;
    for (int b = t; b < nsb; b += kLossThreads) {
        l1 += (double)lp.part[b];
        mp += lp.part_cnt[b];
    }
    for (int b = t; b < nvb; b += kLossThreads) ce += (double)lp.part[nsb + b];
    s_l1[t] = l1;
    s_ce[t] = ce;
    s_mp[t] = mp;
    __syncthreads();
    for (int d = kLossThreads / 2; d > 0; d >>= 1) {
        if (t < d) {
            s_l1[t] += s_l1[t + d];
            s_ce[t] += s_ce[t + d];
            s_mp[t] += s_mp[t + d];
        }
        __syncthreads();
    }
    if (t != 0) return;
    const double t_ce = s_ce[0] / (double)lp.m, t_l1 = s_mp[0] > 0 ? s_l1[0] / (double)s_mp[0] : 0.0;
    lp.loss[0] = (float)(t_ce + t_l1);
    lp.loss[1] = (float)t_ce;
    lp.loss[2] = (float)t_l1;
}

hipError_t launch_loss(const FrameParams &fp, const MapDev &md, const LossParams &lp, hipStream_t s)
{
    const int nsb = (int)((lp.s + kLossThreads - 1) / kLossThreads);
    const int nvb = (int)((lp.m + kLossThreads - 1) / kLossThreads);
    hipLaunchKernelGGL(k_loss_clear, dim3(1024), dim3(256), 0, s, md, lp);
    if (nsb > 0) hipLaunchKernelGGL(k_loss_samples, dim3(nsb), dim3(kLossThreads), 0, s, fp, md, lp);
    if (nvb > 0) hipLaunchKernelGGL(k_loss_voxels, dim3(nvb), dim3(kLossThreads), 0, s, fp, md, lp, nsb);
    hipLaunchKernelGGL(k_loss_final, dim3(1), dim3(kLossThreads), 0, s, lp, nsb, nvb);
    return hipGetLastError();
}

// Four lanes per ray: recompute the band walk, gather the adjoints of the voxels
// it observed, and chain them through the softmax and the clamp.  Bound by the
// latency of the gathers, so they are taken apart from the walk: the walk (all
// four lanes, registers only) lists the ray's leaves and cells in LDS; the lanes
// then look up the leaves side by side, then the cells' records, and then each
// adds its 16-byte vectors of the rows, four cells in flight.  (One lane per
// ray, which waited for the lookup, the page and the row of every cell in turn,
// took 62 us for 65,536 rays and 20 classes; this takes 25 us.)
// NVL: vectors of a row per lane; row vector v belongs to lane v mod 4.
constexpr int kBackRays = 64;               // rays per workgroup
constexpr int kBackCells = kMaxCells | 1;    // cells of a ray, odd row stride

template <int NVL>
__global__ __launch_bounds__(4 * kBackRays) void k_backward_rays(FrameParams fp, MapDev md, LossParams lp,
                                                                 const float *grad_scale, float *grad_logits,
                                                                 float *grad_ranges)
{
    __shared__ unsigned long long s_key[kBackRays][kMaxRuns];
    __shared__ int s_slot[kBackRays][kMaxRuns], s_cell[kBackRays][kBackCells];
    const int sub = threadIdx.x & 3, ray = threadIdx.x >> 2;
    const int i = blockIdx.x * kBackRays + ray;
    const int K = fp.K;
    bool valid = false;
    int ncell = 0, nrun = 0;
    unsigned long long inner = 0ull;  // cells in front of the clamp
    if (i < fp.n) {
        Ray ry;
        float x, y, z;
        load_point(fp, i, x, y, z);
        if (make_ray(fp, x, y, z, ry)) {
            bool inrange = true;
            unsigned long long cur = kEmptyKey;
            const bool started = band_walk(fp, ry, [&](int cx, int cy, int cz) {
                const int kx = fp.a[0] + cx, ky = fp.a[1] + cy, kz = fp.a[2] + cz;
                if (!(key_ok(kx) && key_ok(ky) && key_ok(kz))) {
                    inrange = false;
                    return;
                }
                const float sdf = cell_sdf(fp, ry, cx, cy, cz);
                if (!(sdf > -fp.tau) || !inrange) return;
                const unsigned long long lk = pack_leaf(kx >> 3, ky >> 3, kz >> 3);
                if (lk != cur) {
                    cur = lk;
                    if (sub == 0 && nrun < kMaxRuns) s_key[ray][nrun] = lk;
                    nrun++;
                }
                if (sub == 0 && ncell < kBackCells)
                    s_cell[ray][ncell] = ((nrun - 1) << 9) | ((kx & 7) << 6) | ((ky & 7) << 3) | (kz & 7);
                if (sdf < fp.tau) inner |= 1ull << ncell;
                ncell++;
            });
            // (a ray within the limits has at most kMaxRuns leaf runs and kMaxCells cells)
            valid = started && inrange && nrun <= kMaxRuns && ncell <= kBackCells;
        }
    }
    if (!valid) ncell = nrun = 0;
    wave_sync();
    for (int q = sub; q < nrun; q += 4) s_slot[ray][q] = map_find(md, s_key[ray][q]);
    wave_sync();
    for (int j = sub; j < ncell; j += 4) {
        const int c = s_cell[ray][j], off = c & 511, slot = s_slot[ray][c >> 9];
        // (a leaf or page that is not there: the inputs differ from the integrated ones)
        const int page = slot >= 0 ? md.leaf_page[(size_t)slot * kLeafPages + (off >> 6)] : -1;
        s_cell[ray][j] = page >= 0 ? page * kPageVoxels + (off & (kPageVoxels - 1)) : -1;
    }
    wave_sync();
    const int nv = lp.adj_stride / 4;
    float G[NVL][4];
#pragma unroll
    for (int v = 0; v < NVL; ++v)
#pragma unroll
        for (int e = 0; e < 4; ++e) G[v][e] = 0.0f;
    float gr = 0.0f;
    constexpr int U = 4;
    for (int j0 = 0; j0 < ncell; j0 += U) {
        float4 a[U][NVL];
        int rec[U];
        uchar2 flag[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            rec[u] = j0 + u < ncell ? s_cell[ray][j0 + u] : -1;
            const size_t r = (size_t)(rec[u] >= 0 ? rec[u] : 0);
            flag[u] = lp.adj_flag[r];
#pragma unroll
            for (int v = 0; v < NVL; ++v) {
                const int q = sub + 4 * v;
                a[u][v] = ((const float4 *)(lp.adj + r * lp.adj_stride))[q < nv ? q : 0];
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            // a voxel that is not listed (or an unobserved record of an observed slab)
            // has zero adjoints, one without a class zero dL/dc
            if (rec[u] < 0 || !flag[u].x) continue;
#pragma unroll
            for (int v = 0; v < NVL; ++v) {
                const float x[4] = {a[u][v].x, a[u][v].y, a[u][v].z, a[u][v].w};
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int k = 4 * (sub + 4 * v) + e;
                    if (k < K && flag[u].y) G[v][e] += x[e];
                    if (k == K && ((inner >> (j0 + u)) & 1ull) && x[e] != 0.0f)
                        gr += x[e] / md.vox[(size_t)rec[u] * md.rec_stride + 1];
                }
            }
        }
    }
    if (i >= fp.n) return;
    const float sc = grad_scale ? grad_scale[0] : 1.0f;
    const float *row = (const float *)fp.sem + (size_t)i * K;
    float *out = grad_logits + (size_t)i * K;
    const bool vec = (K & 3) == 0 && (((uintptr_t)fp.sem | (uintptr_t)grad_logits) & 15u) == 0;
    float l[NVL][4];
    float mx = -INFINITY;
#pragma unroll
    for (int v = 0; v < NVL; ++v) {
        const int k0 = 4 * (sub + 4 * v);
        if (vec) {
            const float4 q = k0 < K ? *(const float4 *)(row + k0) : make_float4(-INFINITY, -INFINITY, -INFINITY, -INFINITY);
            l[v][0] = q.x;
            l[v][1] = q.y;
            l[v][2] = q.z;
            l[v][3] = q.w;
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) l[v][e] = k0 + e < K ? row[k0 + e] : -INFINITY;
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) mx = fmaxf(mx, l[v][e]);
    }
    // sums over the ray's four lanes
    auto quad = [](float x) {
        x += __shfl_xor(x, 1, 64);
        return x + __shfl_xor(x, 2, 64);
    };
    mx = fmaxf(mx, __shfl_xor(mx, 1, 64));
    mx = fmaxf(mx, __shfl_xor(mx, 2, 64));
    float den = 0.0f;
#pragma unroll
    for (int v = 0; v < NVL; ++v)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            l[v][e] = 4 * (sub + 4 * v) + e < K ? expf(l[v][e] - mx) : 0.0f;
            den += l[v][e];
        }
    den = quad(den);
    float pg = 0.0f;
#pragma unroll
    for (int v = 0; v < NVL; ++v)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            l[v][e] /= den;
            pg += l[v][e] * G[v][e];
        }
    pg = quad(pg);
#pragma unroll
    for (int v = 0; v < NVL; ++v) {
        const int k0 = 4 * (sub + 4 * v);
        float x[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) x[e] = valid ? sc * l[v][e] * (G[v][e] - pg) : 0.0f;
        if (vec) {
            if (k0 < K) *(float4 *)(out + k0) = make_float4(x[0], x[1], x[2], x[3]);
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (k0 + e < K) out[k0 + e] = x[e];
        }
    }
    gr = quad(gr);  // (only the lane that holds dL/dD has a term)
    if (sub == 0) grad_ranges[i] = valid ? sc * gr : 0.0f;
}

hipError_t launch_backward(const FrameParams &fp, const MapDev &md, const LossParams &lp, const float *grad_scale,
                           float *grad_logits, float *grad_ranges, hipStream_t s)
{
    const int b = (fp.n + kBackRays - 1) / kBackRays;
    if (b == 0) return hipGetLastError();
    const dim3 grid(b), block(4 * kBackRays);
    // a row holds K + 1 adjoints, 16 to each vector of the four lanes
    if (fp.K > 31) hipLaunchKernelGGL(k_backward_rays<3>, grid, block, 0, s, fp, md, lp, grad_scale, grad_logits, grad_ranges);
    else if (fp.K > 15) hipLaunchKernelGGL(k_backward_rays<2>, grid, block, 0, s, fp, md, lp, grad_scale, grad_logits, grad_ranges);
    else hipLaunchKernelGGL(k_backward_rays<1>, grid, block, 0, s, fp, md, lp, grad_scale, grad_logits, grad_ranges);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// reset, extract, query
// ---------------------------------------------------------------------------

// Empties a map (or, without `map`, a second staging buffer) in one launch: the
// tables in 16-byte stores (free slots: key kEmptyKey; slot and padding all
// ones, never read), the counters word by word by the first block.  Five
// launches, the last of which cleared the counters from one thread's stack,
// took 53 us for a table of 2^19 slots, this one 5 us.
__global__ __launch_bounds__(256) void k_reset(const MapDev md, int map)
{
    const size_t cap = (size_t)md.hmask + 1, stride = (size_t)gridDim.x * blockDim.x;
    const size_t t = blockIdx.x * (size_t)blockDim.x + threadIdx.x;
    const uint4 ones = make_uint4(~0u, ~0u, ~0u, ~0u), zero = make_uint4(0u, 0u, 0u, 0u);
    if (map)
        for (size_t i = t; i < cap; i += stride) ((uint4 *)md.htab)[i] = ones;
    for (size_t i = t; i < cap / 2; i += stride) ((uint4 *)md.skeys)[i] = ones;
    for (size_t i = t; i < cap / 4; i += stride) ((uint4 *)md.pos_count)[i] = zero;
    for (size_t i = t; i < cap / 4; i += stride) ((uint4 *)md.pos_slab)[i] = zero;
    if (blockIdx.x == 0) {
        for (size_t i = threadIdx.x; i < sizeof(FrameState) / 4; i += blockDim.x) ((uint32_t *)md.fs)[i] = 0u;
        if (map)
            for (size_t i = threadIdx.x; i < kFilterWords / 4; i += blockDim.x) ((uint4 *)md.filter)[i] = zero;
        if (map)
            for (size_t i = threadIdx.x; i < sizeof(DevState) / 4; i += blockDim.x) ((uint32_t *)md.st)[i] = 0u;
    }
}

static hipError_t reset(const MapDev &md, int map, hipStream_t s)
{
    // capacities are powers of two from 1024 on; four slots per thread, at most 16 blocks per CU's worth
    const size_t cap = (size_t)md.hmask + 1;
    const int blocks = (int)std::min<size_t>(cap / 1024, 4096);
    hipLaunchKernelGGL(k_reset, dim3(blocks), dim3(256), 0, s, md, map);
    return hipGetLastError();
}

hipError_t launch_reset(const MapDev &md, hipStream_t s) { return reset(md, 1, s); }

// Clears a second staging buffer (its table, counts and frame counters).
hipError_t launch_reset_staging(const MapDev &md, hipStream_t s) { return reset(md, 0, s); }

__device__ __forceinline__ uint32_t bits_below(const uint32_t *mask, uint32_t o)
{
    uint32_t r = 0;
    for (uint32_t w = 0; w < (o >> 5); ++w) r += __popc(mask[w]);
    return r + __popc(mask[o >> 5] & ((1u << (o & 31)) - 1u));
}

// Rows of semantic state, record to caller: one wave copies the rows of n
// records (lane q < n holds record index q, or -1 for a row of zeros) to n
// consecutive rows at out.  The n x nsem floats are dealt to the lanes as one
// run of W-float words, so stores are contiguous and loads follow each record's
// own run; eight loads per lane are issued before the first store.  per = nsem
// / W words make a row; div = floor(2^32 / per) + 1 (0: per = 1) divides a word's
// index by per exactly (index x per stays below 2^32: at most 64 rows of 2048
// floats).  W = 2 needs an even nsem and an 8-byte aligned out (records hold
// their semantics at an 8-byte boundary).
constexpr int kCopyBatch = 8;

template <int W>
__device__ __forceinline__ void copy_rows_wave(const MapDev &md, int rec, uint32_t n, uint32_t per, uint32_t div,
                                               float *out)
{
    const uint32_t total = n * per;
    for (uint32_t e0 = 0; e0 < total; e0 += 64 * kCopyBatch) {
        float v[kCopyBatch][W];
#pragma unroll
        for (int u = 0; u < kCopyBatch; ++u) {
            const uint32_t e = e0 + 64 * u + (uint32_t)lane_id();
            const uint32_t q = div ? __umulhi(e, div) : e;
            const int r = __shfl(rec, (int)(q & 63u), 64);
            const bool has = e < total && r >= 0;
            const float *src = md.vox + (size_t)(has ? r : 0) * md.rec_stride + 2 + W * (has ? e - q * per : 0u);
            if constexpr (W == 2) {
                const float2 f = has ? *(const float2 *)src : make_float2(0.0f, 0.0f);
                v[u][0] = f.x;
                v[u][1] = f.y;
            } else {
                v[u][0] = has ? *src : 0.0f;
            }
        }
#pragma unroll
        for (int u = 0; u < kCopyBatch; ++u) {
            const uint32_t e = e0 + 64 * u + (uint32_t)lane_id();
            if (e >= total) continue;
            if constexpr (W == 2) ((float2 *)out)[e] = make_float2(v[u][0], v[u][1]);
            else out[e] = v[u][0];
        }
    }
}

// Division constant of copy_rows_wave.
static uint32_t row_div(uint32_t per) { return per > 1 ? (uint32_t)((1ull << 32) / per) + 1u : 0u; }

// The leaves in key order: runs of kSortRun leaves sorted in LDS (a bitonic
// network, two leaves per thread), then merged kMergeRuns runs at a time by rank:
// a leaf's place is its place in its own run plus, for each other run, the number
// of smaller keys there, found by binary searches that advance together (keys are
// distinct).  Only keys are moved: the last of these launches finds each leaf's slot in
// the leaf table and counts its voxels (the slots moved beside the keys took 28 bytes of
// scratch a leaf instead of 16, and the same time).  11,500 leaves: two launches of 26
// and 17 us instead of 105 compare-exchange launches of 2.4 us each.
constexpr int kSortRun = 2048, kMergeRuns = 8;

// A leaf's slot and its number of voxels.
__device__ __forceinline__ uint2 leaf_entry(const MapDev &md, unsigned long long key)
{
    const int slot = map_find(md, key);
    if (slot < 0) return make_uint2(0u, 0u);  // (every leaf of the map is in its table)
    uint32_t c = 0;
#pragma unroll
    for (int w = 0; w < kMaskWords / 4; ++w) {
        const uint4 o = ((const uint4 *)md.leaf_occ)[(size_t)slot * (kMaskWords / 4) + w];
        c += __popc(o.x) + __popc(o.y) + __popc(o.z) + __popc(o.w);
    }
    return make_uint2((uint32_t)slot, c);
}

// leaves: the entries in key order where one run is all (or null)
__global__ __launch_bounds__(kSortRun / 2) void k_leaf_sort(const MapDev md, long long nleaves, unsigned long long *keys,
                                                            uint2 *leaves)
{
    __shared__ unsigned long long k[kSortRun];
    const long long base = (long long)blockIdx.x * kSortRun;
    const int t = threadIdx.x;
#pragma unroll
    for (int q = t; q < kSortRun; q += kSortRun / 2)
        k[q] = base + q < nleaves ? md.leaf_key[base + q] : kEmptyKey;  // (above every key)
    // a step over spans of at most 128 places stays inside the 128 that a wave's
    // lanes compare, so only the wider steps (10 of 66) need the whole workgroup
    int before = kSortRun;
    for (int n = 2; n <= kSortRun; n <<= 1)
        for (int d = n >> 1; d > 0; d >>= 1) {
            const int span = 2 * d;
            if (max(span, before) > 128) __syncthreads();
            else wave_sync();
            before = span;
            // the first step of a stage compares mirrored places, so every run sorts upwards
            const int a = (t / d) * 2 * d + (t & (d - 1));
            const int b = d == n >> 1 ? (a & ~(n - 1)) + (n - 1) - (a & (n - 1)) : a + d;
            const unsigned long long ka = k[a], kb = k[b];
            if (kb < ka) {
                k[a] = kb;
                k[b] = ka;
            }
        }
    __syncthreads();
#pragma unroll
    for (int q = t; q < kSortRun; q += kSortRun / 2)
        if (base + q < nleaves) {
            if (leaves) leaves[base + q] = leaf_entry(md, k[q]);
            else keys[base + q] = k[q];
        }
}

// leaves: the entries in key order from the last merge (or null)
__global__ __launch_bounds__(256) void k_leaf_merge(const MapDev md, long long nleaves, long long run,
                                                    const unsigned long long *keys, unsigned long long *keys_out,
                                                    uint2 *leaves)
{
    const long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x;
    if (i >= nleaves) return;
    const unsigned long long key = keys[i];
    const long long group = i / (run * kMergeRuns) * (run * kMergeRuns), own = (i - group) / run;
    const unsigned long long *base[kMergeRuns];
    uint32_t len[kMergeRuns], pos[kMergeRuns];
#pragma unroll
    for (int q = 0; q < kMergeRuns; ++q) {
        const long long start = group + q * run;
        base[q] = keys + start;
        len[q] = q == own || start >= nleaves ? 0u : (uint32_t)min(run, nleaves - start);
        pos[q] = 0;
    }
    for (uint32_t step = (uint32_t)run; step > 0; step >>= 1) {
        bool less[kMergeRuns];
#pragma unroll
        for (int q = 0; q < kMergeRuns; ++q)
            less[q] = pos[q] + step <= len[q] && base[q][pos[q] + step - 1] < key;
#pragma unroll
        for (int q = 0; q < kMergeRuns; ++q) pos[q] += less[q] ? step : 0u;
    }
    long long out = i - own * run;  // group + place in the own run
#pragma unroll
    for (int q = 0; q < kMergeRuns; ++q) out += pos[q];
    if (leaves) leaves[out] = leaf_entry(md, key);
    else keys_out[out] = key;
}

// Exclusive prefix sum of the leaves' voxel counts, in place, by one workgroup
// (16 counts per thread and round: 11,500 leaves are one round).
__global__ __launch_bounds__(1024) void k_leaf_offsets(long long nleaves, uint2 *leaves)
{
    __shared__ uint32_t wsum[16];
    constexpr int U = 16;
    uint32_t carry = 0;
    for (long long b = 0; b < nleaves; b += 1024 * U) {
        const long long i = b + (long long)threadIdx.x * U;
        uint32_t c[U], t = 0;
#pragma unroll
        for (int q = 0; q < U; ++q) {
            c[q] = i + q < nleaves ? leaves[i + q].y : 0u;
            t += c[q];
        }
        const uint32_t incl = wave_incl_scan(t);
        if (lane_id() == 63) wsum[threadIdx.x >> 6] = incl;
        __syncthreads();
        uint32_t run = carry + incl - t, total = 0;
#pragma unroll
        for (int w = 0; w < 16; ++w) {
            if (w < (int)(threadIdx.x >> 6)) run += wsum[w];
            total += wsum[w];
        }
#pragma unroll
        for (int q = 0; q < U; ++q) {
            if (i + q < nleaves) leaves[i + q].y = run;
            run += c[q];
        }
        carry += total;
        __syncthreads();
    }
}

// Export of the sorted leaves, a workgroup per leaf: keys, D and W by one thread
// per voxel, then the rows of the leaf's voxels, which are consecutive in the
// output, as one run of W-float words (as copy_rows_wave).  Bound by the rows'
// bytes: 912,588 voxels of 20 classes 188 -> 58 us (168 MB; one thread per
// voxel copied its row alone before).
template <int W>
__global__ __launch_bounds__(256) void k_extract(const MapDev md, long long nleaves, uint32_t nsem, uint32_t div,
                                                 const uint2 *leaves, int32_t *keys, float *d, float *w, float *sem)
{
    __shared__ uint32_t occ[kMaskWords];
    __shared__ int pages[kLeafPages];
    __shared__ int recs[kLeafVoxels];
    const int tid = threadIdx.x;
    for (long long j = blockIdx.x; j < nleaves; j += gridDim.x) {
        const uint2 leaf = leaves[j];
        const int slot = (int)leaf.x;
        const unsigned long long lk = md.leaf_key[slot];
        const size_t first = leaf.y;
        if (tid < kMaskWords) occ[tid] = md.leaf_occ[(size_t)slot * kMaskWords + tid];
        if (tid < kLeafPages) pages[tid] = md.leaf_page[(size_t)slot * kLeafPages + tid];
        __syncthreads();
        const int lx = (int)((lk >> 36) & 0x3FFFF) - kLeafBias;
        const int ly = (int)((lk >> 18) & 0x3FFFF) - kLeafBias;
        const int lz = (int)(lk & 0x3FFFF) - kLeafBias;
        uint32_t cnt = 0;
#pragma unroll
        for (int q = 0; q < kMaskWords; ++q) cnt += __popc(occ[q]);
#pragma unroll
        for (int t = tid; t < kLeafVoxels; t += 256) {
            if (!((occ[t >> 5] >> (t & 31)) & 1u)) continue;
            const uint32_t r = bits_below(occ, (uint32_t)t);
            const size_t o = first + r;
            const int rec = pages[t >> 6] * kPageVoxels + (t & (kPageVoxels - 1));
            const float *R = md.vox + (size_t)rec * md.rec_stride;
            keys[3 * o + 0] = lx * 8 + (t >> 6);
            keys[3 * o + 1] = ly * 8 + ((t >> 3) & 7);
            keys[3 * o + 2] = lz * 8 + (t & 7);
            d[o] = R[0];
            w[o] = R[1];
            recs[r] = rec;
        }
        __syncthreads();
        if constexpr (W > 0) {
            const uint32_t per = nsem / W, total = cnt * per;
            float *out = sem + first * nsem;
            constexpr int U = 4;
            for (uint32_t e0 = tid; e0 < total; e0 += 256 * U) {
                float v[U][W];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const uint32_t e = min(e0 + 256 * u, total - 1u), q = div ? (uint32_t)(((unsigned long long)e * div) >> 32) : e;
                    const float *src = md.vox + (size_t)recs[q] * md.rec_stride + 2 + W * (e - q * per);
                    if constexpr (W == 2) {
                        const float2 f = *(const float2 *)src;
                        v[u][0] = f.x;
                        v[u][1] = f.y;
                    } else {
                        v[u][0] = *src;
                    }
                }
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const uint32_t e = e0 + 256 * u;
                    if (e >= total) continue;
                    if constexpr (W == 2) ((float2 *)out)[e] = make_float2(v[u][0], v[u][1]);
                    else out[e] = v[u][0];
                }
            }
        }
        __syncthreads();
    }
}

hipError_t launch_extract(const MapDev &md, int nsem, long long nleaves, const ExtractScratch &x, int32_t *keys,
                          float *d, float *w, float *sem, hipStream_t s)
{
    if (nleaves <= 0) return hipGetLastError();
    unsigned long long *ka = x.keys, *kb = x.keys2;
    uint2 *leaves = nleaves <= kSortRun ? (uint2 *)ka : nullptr;
    hipLaunchKernelGGL(k_leaf_sort, dim3((unsigned)((nleaves + kSortRun - 1) / kSortRun)), dim3(kSortRun / 2), 0, s, md,
                       nleaves, ka, leaves);
    for (long long run = kSortRun; run < nleaves; run *= kMergeRuns) {
        if (run * kMergeRuns >= nleaves) leaves = (uint2 *)kb;
        hipLaunchKernelGGL(k_leaf_merge, dim3((unsigned)((nleaves + 255) / 256)), dim3(256), 0, s, md, nleaves, run, ka,
                           kb, leaves);
        std::swap(ka, kb);
    }
    hipLaunchKernelGGL(k_leaf_offsets, dim3(1), dim3(1024), 0, s, nleaves, leaves);
    const uint32_t n = sem ? (uint32_t)nsem : 0u;
    const bool pair = n % 2 == 0 && ((uintptr_t)sem & 7u) == 0;
    const dim3 grid((unsigned)std::min<long long>(nleaves, 16384)), block(256);
    if (n == 0) hipLaunchKernelGGL(k_extract<0>, grid, block, 0, s, md, nleaves, n, 0u, leaves, keys, d, w, sem);
    else if (pair) hipLaunchKernelGGL(k_extract<2>, grid, block, 0, s, md, nleaves, n, row_div(n / 2), leaves, keys, d, w, sem);
    else hipLaunchKernelGGL(k_extract<1>, grid, block, 0, s, md, nleaves, n, row_div(n), leaves, keys, d, w, sem);
    return hipGetLastError();
}

// Scratch of the allocation-free extract (slim_extract_noalloc): two arrays of
// leaf keys (a merge reads one and writes the other), for at most
// kNoAllocMaxLeaves leaves.  Each GPU the library runs on holds its own copy
// until the process ends.  In host code `scratch` names a host-side stand-in:
// kernels get the device address that noalloc_scratch_setup resolved.
static __device__ __align__(256) unsigned char scratch[kNoAllocMaxLeaves * 16];

namespace {
std::mutex g_scratch_mu;
void *g_scratch_ptr[kNoAllocMaxDevices];
}  // namespace

hipError_t noalloc_scratch_setup(int device)
{
    if (device < 0 || device >= kNoAllocMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (g_scratch_ptr[device]) return hipSuccess;
    void *ptr = nullptr;
    const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!ptr) return hipErrorInvalidSymbol;
    g_scratch_ptr[device] = ptr;
    return hipSuccess;
}

void *noalloc_scratch(int device)
{
    if (device < 0 || device >= kNoAllocMaxDevices) return nullptr;
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    return g_scratch_ptr[device];
}

// Record of the voxel holding world point (x, y, z), floor(x / vs) in binary32;
// -1 if unobserved, non-finite or out of the key range.
__device__ __forceinline__ long long lookup_point(const MapDev &md, float vs, float x, float y, float z)
{
    if (!(isfinite(x) && isfinite(y) && isfinite(z))) return -1;
    const float fx = floorf(x / vs), fy = floorf(y / vs), fz = floorf(z / vs);
    const float lim = (float)kKeyLimit;
    if (!(fabsf(fx) < lim && fabsf(fy) < lim && fabsf(fz) < lim)) return -1;
    const int kx = (int)fx, ky = (int)fy, kz = (int)fz;
    const int slot = map_find(md, pack_leaf(kx >> 3, ky >> 3, kz >> 3));
    if (slot < 0) return -1;
    const int off = ((kx & 7) << 6) | ((ky & 7) << 3) | (kz & 7);
    if (!((md.leaf_occ[(size_t)slot * kMaskWords + (off >> 5)] >> (off & 31)) & 1u)) return -1;
    return (long long)md.leaf_page[(size_t)slot * kLeafPages + (off >> 6)] * kPageVoxels + (off & (kPageVoxels - 1));
}

// State at world points: a wave takes g consecutive points at a time, one lane
// each for the lookup (hash probe, occupancy, page, record: four dependent
// reads) and D and W, then all lanes for the rows (W = 0: no rows).  Bound by
// the rows' bytes when they are long, by the lookup's latency when short.
// Against one thread per point that copied its row alone: 38,400 points with
// rows of 4 KB 509 -> 54 us, 414,000 points of 16 maps (half with rows of 2 KB)
// 2409 -> 155 us, 65,536 points with 20 classes 13.8 -> 7 us.
template <int W>
__global__ __launch_bounds__(256) void k_query(const MapDev md, uint32_t nsem, uint32_t div, int g, float vs,
                                               const float *xyz, long long m, float *d, float *w, float *sem)
{
    const int lane = lane_id();
    const long long nwaves = (long long)gridDim.x * (blockDim.x >> 6);
    for (long long q0 = (blockIdx.x * (long long)(blockDim.x >> 6) + (threadIdx.x >> 6)) * g; q0 < m;
         q0 += nwaves * g) {
        const long long i = q0 + lane;
        int rec = -1;
        if (lane < g && i < m) {
            rec = (int)lookup_point(md, vs, xyz[3 * i], xyz[3 * i + 1], xyz[3 * i + 2]);
            const float *R = md.vox + (size_t)(rec >= 0 ? rec : 0) * md.rec_stride;
            d[i] = rec >= 0 ? R[0] : 0.0f;
            w[i] = rec >= 0 ? R[1] : 0.0f;
        }
        if constexpr (W > 0)
            copy_rows_wave<W>(md, rec, (uint32_t)min((long long)g, m - q0), nsem / W, div, sem + (size_t)q0 * nsem);
    }
}

hipError_t launch_query(const MapDev &md, int nsem, float vs, const float *xyz, long long m, float *d, float *w,
                        float *sem, hipStream_t s)
{
    if (m <= 0) return hipGetLastError();
    const uint32_t n = sem ? (uint32_t)nsem : 0u;
    const bool pair = n % 2 == 0 && ((uintptr_t)sem & 7u) == 0;
    // points per wave: 16 short rows keep four waves per 64 points in flight;
    // from 128 floats on (open-set records of 0.5 KB and more) 4 rows fill a
    // wave's loads, and more would leave the chip short of waves
    const int g = n == 0 ? 64 : (n < 128 ? 16 : 4);
    const int blocks = (int)std::min<long long>((m + 4 * g - 1) / (4 * g), 16384);
    if (n == 0) hipLaunchKernelGGL(k_query<0>, dim3(blocks), dim3(256), 0, s, md, n, 0u, g, vs, xyz, m, d, w, sem);
    else if (pair) hipLaunchKernelGGL(k_query<2>, dim3(blocks), dim3(256), 0, s, md, n, row_div(n / 2), g, vs, xyz, m, d, w, sem);
    else hipLaunchKernelGGL(k_query<1>, dim3(blocks), dim3(256), 0, s, md, n, row_div(n), g, vs, xyz, m, d, w, sem);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// semantic read-out: Eq. (7), Eq. (15), prototype softmax and threshold
// ---------------------------------------------------------------------------

// First index of the largest value across the wave: (v, i) pairs, larger v
// wins, equal v the smaller i.
__device__ __forceinline__ void wave_argmax(float &v, int &i)
{
    for (int d = 32; d > 0; d >>= 1) {
        const float ov = __shfl_xor(v, d, 64);
        const int oi = __shfl_xor(i, d, 64);
        if (ov > v || (ov == v && oi < i)) {
            v = ov;
            i = oi;
        }
    }
}

// Closed set, one wave per query point.
__global__ __launch_bounds__(256) void k_predict(const MapDev md, const PredictParams pp, const float *xyz,
                                                 long long m, float *prob, int32_t *label)
{
    const int lane = lane_id(), wv = threadIdx.x >> 6;
    const long long nwaves = (long long)gridDim.x * (blockDim.x >> 6);
    for (long long q = blockIdx.x * (long long)(blockDim.x >> 6) + wv; q < m; q += nwaves) {
        const long long rec = lookup_point(md, pp.vs, xyz[3 * q], xyz[3 * q + 1], xyz[3 * q + 2]);
        const float *R = rec >= 0 ? md.vox + (size_t)rec * md.rec_stride : nullptr;
        float best = -INFINITY;
        int arg = 0x7FFFFFFF;
        if (pp.mode == SLIM_SEM_CLOSED) {
            // Eq. (7): the Dirichlet predictive
            float part = 0.0f;
            for (int k = lane; k < pp.K; k += 64) part += R ? R[2 + k] : 0.0f;
            const float den = (float)pp.K * pp.alpha0 + wave_sum(part);
            for (int k = lane; k < pp.K; k += 64) {
                const float p = (pp.alpha0 + (R ? R[2 + k] : 0.0f)) / den;
                if (prob) prob[q * pp.K + k] = p;
                if (p > best) {
                    best = p;
                    arg = k;
                }
            }
        } else {
            const int cls = R ? (int)R[2] : -1;
            for (int k = lane; k < pp.K; k += 64) {
                const float p = k == cls ? 1.0f : 0.0f;
                if (prob) prob[q * pp.K + k] = p;
                if (p > best) {
                    best = p;
                    arg = k;
                }
            }
        }
        wave_argmax(best, arg);
        if (label && lane == 0) label[q] = (R && best >= pp.threshold) ? arg : -1;
    }
}

// Open set: a workgroup takes 16 points.  Their means against the prototypes
// are a contraction (m x L by L x P), done on the matrix cores in binary32: each
// of the four waves takes every fourth run of 16 components of all rows, 16 x 16
// products at a time (v_mfma_f32_16x16x4f32), CT tiles of 16 prototypes at a time.
// A lane loads four consecutive components of one row (lane mod 16) for the four
// steps of a run, so the fragments come straight from the records and from the
// prototypes, which stay in L2: no staging.  Norms are formed from the same
// registers.  One wave per point then does the softmax, the threshold and the
// variances.
// A sum is formed in three levels, so that no chain of roundings is long: a run's 16
// products in two chains of 8 added together, a wave's L / 64 runs one after the
// other, and the waves' four sums in binary64, as the norms' reciprocals and the
// similarity until it is rounded once.  Root-mean-square relative error of a probability at temperature
// 0.02, 56 prototypes, 512 components: 2.8e-7 with components of mean 0 and 1.6e-6
// with mean 5; with one chain of L / 4 products a wave 6.1e-7 and 4.8e-6, with one
// wave a point 3.7e-7 and 2.7e-6.
// Bound by the records' bytes (mean and beta once) and the outputs, and by the waves
// in flight: five workgroups a CU need 96 registers, which the scheduling barrier
// after every second tile keeps to (without it four, and 130 us; six spill 15, 122 us).
// 50,000 points x 56 prototypes x 512 components take 114 us; one wave a point, which forms every dot
// product and every prototype norm by itself, 960 us.  With 32 points a workgroup,
// half the prototype traffic but a third fewer waves, 180 us.
// Where none of the 16 points has a record nothing is contracted (2,000 such points,
// 1,024 prototypes of 512 components: 121 us if it is).
// CT = 1 (at most 16 prototypes): no work for tiles that are not there, and four
// runs' loads in flight.  2,000 points, 2 prototypes of 1,024 components: 20 -> 15 us
// (one wave a point 14), 16,384 points 38 -> 25 us (49).
// FAST: L a multiple of 16 and 16-byte aligned prototypes, no edge in a load.
typedef float f32x4_t __attribute__((ext_vector_type(4)));

template <int PMAX, int CT, bool FAST>
__global__ __launch_bounds__(256, PMAX == 1024 ? 1 : 5) void k_predict_open(const MapDev md, const PredictParams pp,
                                                                           const float *xyz, long long m, float *prob,
                                                                           int32_t *label, float *var)
{
    constexpr int TQ = 16, PC = 16 * CT, U = 4 / CT;
    __shared__ float sims[TQ][PMAX];
    __shared__ float part[4][TQ][PC + 4];
    __shared__ float n2s[4][TQ], q2s[4][PC];
    const int tid = threadIdx.x, lane = lane_id(), w = tid >> 6, g = lane >> 4, c = lane & 15;
    const int L = pp.L, P = pp.P;
    for (long long q0 = blockIdx.x * (long long)TQ; q0 < m; q0 += gridDim.x * (long long)TQ) {
        // lane c of every 16 holds the record of point c
        const long long qc = q0 + c;
        const int rec = qc < m ? (int)lookup_point(md, pp.vs, xyz[3 * qc], xyz[3 * qc + 1], xyz[3 * qc + 2]) : -1;
        const float *A = md.vox + (size_t)(rec >= 0 ? rec : 0) * md.rec_stride + 2;
        // (every wave holds all 16 records: the branch is the workgroup's)
        const int P1 = __ballot(rec >= 0) != 0ull ? P : 0;
        for (int p0 = 0; p0 < P1; p0 += PC) {
            f32x4_t acc[CT];
            float n2 = 0.0f, q2[CT];
#pragma unroll
            for (int u = 0; u < CT; ++u) {
                q2[u] = 0.0f;
                acc[u] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
            }
            uint32_t row[CT];  // (32-bit offsets into the prototypes: at most 2^20 floats)
#pragma unroll
            for (int u = 0; u < CT; ++u) row[u] = p0 + 16 * u + c < P ? (uint32_t)(p0 + 16 * u + c) * (uint32_t)L : 0u;
            for (int s = w; 16 * s < L; s += 4 * U) {
                float a[U][4], b[U][CT][4];
#pragma unroll
                for (int v = 0; v < U; ++v) {
                    const int k = 16 * (s + 4 * v) + 4 * g;
                    if constexpr (FAST) {
                        const bool has = rec >= 0 && k < L;
                        const float2 x = has ? *(const float2 *)(A + k) : make_float2(0.0f, 0.0f);
                        const float2 y = has ? *(const float2 *)(A + k + 2) : make_float2(0.0f, 0.0f);
                        a[v][0] = x.x; a[v][1] = x.y; a[v][2] = y.x; a[v][3] = y.y;
                    } else {
#pragma unroll
                        for (int j = 0; j < 4; ++j) a[v][j] = rec >= 0 && k + j < L ? A[k + j] : 0.0f;
                    }
#pragma unroll
                    for (int u = 0; u < CT; ++u) {
                        const int p = p0 + 16 * u + c;
                        const float *B = pp.protos + (row[u] + (uint32_t)k);
                        if constexpr (FAST) {
                            const float4 x = p < P && k < L ? *(const float4 *)B : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
                            b[v][u][0] = x.x; b[v][u][1] = x.y; b[v][u][2] = x.z; b[v][u][3] = x.w;
                        } else {
#pragma unroll
                            for (int j = 0; j < 4; ++j) b[v][u][j] = p < P && k + j < L ? B[j] : 0.0f;
                        }
                    }
                }
#pragma unroll
                for (int v = 0; v < U; ++v) {
                    n2 += fmaf(a[v][3], a[v][3], fmaf(a[v][2], a[v][2], fmaf(a[v][1], a[v][1], a[v][0] * a[v][0])));
#pragma unroll
                    for (int u = 0; u < CT; ++u) {
                        const float *y = b[v][u];
                        const f32x4_t zero = {0.0f, 0.0f, 0.0f, 0.0f};
                        f32x4_t z0 = __builtin_amdgcn_mfma_f32_16x16x4f32(a[v][0], y[0], zero, 0, 0, 0);
                        f32x4_t z1 = __builtin_amdgcn_mfma_f32_16x16x4f32(a[v][2], y[2], zero, 0, 0, 0);
                        z0 = __builtin_amdgcn_mfma_f32_16x16x4f32(a[v][1], y[1], z0, 0, 0, 0);
                        z1 = __builtin_amdgcn_mfma_f32_16x16x4f32(a[v][3], y[3], z1, 0, 0, 0);
                        acc[u] += z0 + z1;
                        if (CT == 1 || (u & 1)) __builtin_amdgcn_sched_barrier(0);
                        q2[u] += fmaf(y[3], y[3], fmaf(y[2], y[2], fmaf(y[1], y[1], y[0] * y[0])));
                    }
                }
            }
            n2 += __shfl_xor(n2, 16, 64);
            n2 += __shfl_xor(n2, 32, 64);
            if (g == 0) n2s[w][c] = n2;
#pragma unroll
            for (int u = 0; u < CT; ++u)
#pragma unroll
                for (int r = 0; r < 4; ++r) part[w][4 * g + r][16 * u + c] = acc[u][r];
#pragma unroll
            for (int u = 0; u < CT; ++u) {
                q2[u] += __shfl_xor(q2[u], 16, 64);
                q2[u] += __shfl_xor(q2[u], 32, 64);
                if (g == 0) q2s[w][16 * u + c] = q2[u];
            }
            __syncthreads();
            // cosine similarity of the predictive mean with every prototype
            // (the reciprocals of the norms take the place of two of the partial sums)
            if (tid < TQ + PC) {
                const bool row = tid < TQ;
                float *q = row ? &n2s[0][tid] : &q2s[0][tid - TQ];
                const int st = row ? TQ : PC;
                const double x = (row ? 1.0 : (double)pp.inv_temp) /
                                 sqrt(((double)q[0] + q[st]) + ((double)q[2 * st] + q[3 * st]));
                q[0] = __int_as_float(__double2loint(x));
                q[st] = __int_as_float(__double2hiint(x));
            }
            __syncthreads();
            for (int e = tid; e < TQ * PC; e += 256) {
                const int i = e / PC, j = e % PC;
                if (p0 + j >= P) continue;
                const double dot = ((double)part[0][i][j] + part[1][i][j]) + ((double)part[2][i][j] + part[3][i][j]);
                const double rn = __hiloint2double(__float_as_int(n2s[1][i]), __float_as_int(n2s[0][i]));
                const double rq = __hiloint2double(__float_as_int(q2s[1][j]), __float_as_int(q2s[0][j]));
                sims[i][p0 + j] = (float)(dot * rn * rq);
            }
            __syncthreads();
        }
        // wave w's points: w, w + 4, w + 8, w + 12
        if (var && pp.mode == SLIM_SEM_OPEN) {
            // Eq. (15) with lambda = 2 nu = W: variance 2 beta (W + 1) / (W (W - 2)) for W > 2
            float W[4];
            const float *B[4];
            float *out[4];
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const int i = w + 4 * t, r = __shfl(rec, i, 64);
                const float *R = md.vox + (size_t)(r >= 0 ? r : 0) * md.rec_stride;
                W[t] = r >= 0 ? R[1] : 0.0f;
                B[t] = R + 2 + L;
                out[t] = q0 + i < m ? var + (size_t)(q0 + i) * L : nullptr;
            }
#pragma unroll 2
            for (int d = lane; d < L; d += 64) {
                float x[4];
#pragma unroll
                for (int t = 0; t < 4; ++t) x[t] = W[t] > 2.0f ? B[t][d] : 0.0f;
#pragma unroll
                for (int t = 0; t < 4; ++t)
                    if (out[t]) out[t][d] = W[t] > 2.0f ? 2.0f * x[t] * (W[t] + 1.0f) / (W[t] * (W[t] - 2.0f)) : NAN;
            }
        }
        for (int i = w; i < TQ && q0 + i < m; i += 4) {
            const long long q = q0 + i;
            const float *S = sims[i];
            const bool has = __shfl(rec, i, 64) >= 0;
            float best = -INFINITY;
            int arg = 0x7FFFFFFF;
            if (has) {
                float mx = -INFINITY;
                for (int j = lane; j < P; j += 64) mx = fmaxf(mx, S[j]);
                mx = wave_max(mx);
                float es = 0.0f;
                for (int j = lane; j < P; j += 64) es += expf(S[j] - mx);
                const float den = wave_sum(es);
                for (int j = lane; j < P; j += 64) {
                    const float p = expf(S[j] - mx) / den;
                    if (prob) prob[q * P + j] = p;
                    if (p > best) {
                        best = p;
                        arg = j;
                    }
                }
            } else if (prob) {
                for (int j = lane; j < P; j += 64) prob[q * P + j] = 0.0f;
            }
            wave_argmax(best, arg);
            if (label && lane == 0) label[q] = (has && best >= pp.threshold) ? arg : -1;
        }
        __syncthreads();
    }
}

hipError_t launch_predict(const MapDev &md, const PredictParams &pp, const float *xyz, long long m, float *prob,
                          int32_t *label, float *var, hipStream_t s)
{
    if (m <= 0) return hipGetLastError();
    if (pp.mode != SLIM_SEM_OPEN && pp.mode != SLIM_SEM_OPEN_LAST) {
        const int blocks = (int)std::min<long long>((m + 3) / 4, 65536);
        hipLaunchKernelGGL(k_predict, dim3(blocks), dim3(256), 0, s, md, pp, xyz, m, prob, label);
        return hipGetLastError();
    }
    const bool fast = pp.L % 16 == 0 && ((uintptr_t)pp.protos & 15u) == 0;
    // (a launch holds fewer than 2^32 threads: beyond 2^22 points the workgroups stride)
    const dim3 grid((unsigned)std::min<long long>((m + 15) / 16, 1 << 18)), block(256);
#define SLIM_PREDICT(PMAX, CT, FAST) \
    hipLaunchKernelGGL((k_predict_open<PMAX, CT, FAST>), grid, block, 0, s, md, pp, xyz, m, prob, label, var)
    // the similarities sit in LDS: up to 128 prototypes five workgroups fit a CU
    if (pp.P <= 16 && fast) SLIM_PREDICT(16, 1, true);
    else if (pp.P <= 16) SLIM_PREDICT(16, 1, false);
    else if (pp.P <= 128 && fast) SLIM_PREDICT(128, 4, true);
    else if (pp.P <= 128) SLIM_PREDICT(128, 4, false);
    else if (fast) SLIM_PREDICT(1024, 4, true);
    else SLIM_PREDICT(1024, 4, false);
#undef SLIM_PREDICT
    return hipGetLastError();
}


// ---------------------------------------------------------------------------
// render: first surface per pixel (the map-viewing role of Sec. III-E)
// ---------------------------------------------------------------------------

// Filters of the render: a bit per leaf, and per block of 8 x 8 x 8 leaves, taken
// at their coordinates modulo 64 leaves and 32 blocks, set for every leaf of the
// map, so that a clear bit means that nothing is there.  A ray through empty space
// then reads LDS instead of the leaf table.  A render sets the bits of the leaves
// beyond DevState::filtered, which the render kernel moves on once they are set; none
// is cleared before the map is (leaves leave a map only then), so renders of one map
// on several streams find theirs set.  (x, y, z: voxel keys.)
__device__ __forceinline__ uint32_t leaf_bit(int x, int y, int z)
{
    return (((uint32_t)x >> 3) & 63u) | ((((uint32_t)y >> 3) & 63u) << 6) | ((((uint32_t)z >> 3) & 63u) << 12);
}

__device__ __forceinline__ uint32_t block_bit(int x, int y, int z)
{
    return (1u << kFilterLog2) +
           ((((uint32_t)x >> 6) & 31u) | ((((uint32_t)y >> 6) & 31u) << 5) | ((((uint32_t)z >> 6) & 31u) << 10));
}
static_assert(kFilterLog2 == 18 && kFilterBlockLog2 == 15, "6 bits of each leaf coordinate, 5 of each block's");

// Bound by the atomics on one word: the leaves of a surface share few blocks, and
// those a workgroup holds are gathered in LDS first (8,200 new leaves: 24 -> 7 us).
// (With the bits of all leaves set by every render, one of a single cell took 37 us
// over 630,000 leaves; without the filters of any kind it takes 12.)
__global__ __launch_bounds__(256) void k_render_filter(const MapDev md)
{
    __shared__ uint32_t s_block[(1 << kFilterBlockLog2) / 32];
    const unsigned long long n = md.st->leaves_used;
    const unsigned long long first = md.st->filtered + blockIdx.x * (unsigned long long)blockDim.x;
    if (first >= n) return;
    constexpr int kWords = (1 << kFilterBlockLog2) / 32, kBase = (1 << kFilterLog2) / 32;
    for (int w = threadIdx.x; w < kWords; w += 256) s_block[w] = 0u;
    __syncthreads();
    for (unsigned long long i = first + threadIdx.x; i < n; i += (unsigned long long)gridDim.x * blockDim.x) {
        const unsigned long long k = md.leaf_key[i];
        const int x = ((int)((k >> 36) & 0x3FFFF) - kLeafBias) * 8, y = ((int)((k >> 18) & 0x3FFFF) - kLeafBias) * 8;
        const int z = ((int)(k & 0x3FFFF) - kLeafBias) * 8;
        const uint32_t b = leaf_bit(x, y, z), c = block_bit(x, y, z);
        atomicOr(&md.filter[b >> 5], 1u << (b & 31));
        atomicOr(&s_block[(c >> 5) - kBase], 1u << (c & 31));
    }
    __syncthreads();
    for (int w = threadIdx.x; w < kWords; w += 256)
        if (s_block[w]) atomicOr(&md.filter[kBase + w], s_block[w]);
}

// One step of a render's walk (ties step the lowest axis): tm advances by td along
// the axis of the next crossing, the cell's place by that axis' step.
__device__ __forceinline__ void render_step(float &tx, float &ty, float &tz, uint32_t &at, float &tnext, bool &ix,
                                            float tdx, float tdy, float tdz, uint32_t stx, uint32_t sty, uint32_t stz)
{
    const bool xy = tx <= ty;
    const float txy = xy ? tx : ty;
    const uint32_t sxy = xy ? stx : sty;
    const bool iz = !(txy <= tz), iy = !xy && !iz;
    ix = xy && !iz;
    tnext = iz ? tz : txy;
    at += iz ? stz : sxy;
    tx = ix ? tx + tdx : tx;
    ty = iy ? ty + tdy : ty;
    tz = iz ? tz + tdz : tz;
}

// One thread per pixel, a wave per 8 x 8 pixels (neighbouring rays cross the same
// leaves).  The ray is formed as a sensor point at unit depth is (same binary32
// operations), walked with the integration walk's stepping rule over [t0, t1], and
// stops at the first pair of consecutive observed cells with D > 0 then D <= 0; the
// depth interpolates the cell centres' projections onto the ray linearly in D.
// Bound by the instructions of a step, of which a ray takes up to a thousand, most
// of them in empty space.  The cell's place in its block of 64 cells a side is one
// word of three 8-bit fields (place + 64), and a step through an empty block or leaf
// is the choice of the axis, three conditional additions, one to the fields and one
// test of their upper bits; lookups and the test for the ray's end wait for the way
// out.  In a leaf of the map 8 cells are stepped through before their occupancy, then
// their D, are read side by side.  1209 x 448 pixels over 8,200 leaves 675 -> 402 us with
// the filters' launch (with the filters cleared and built by two launches 420, then 474
// with one cell's reads at a time, 468 with 4 cells and 8 waves per SIMD).  (Jumping to the way out of
// an empty block in closed form, exact while tm stays in a binade, took 1,143 us: too
// many rays are at a binade's end somewhere in the wave.)
constexpr int kRenderThreads = 256, kRenderCells = 8;

template <bool FILTER>
__global__ __launch_bounds__(kRenderThreads) void k_render(const MapDev md, const RenderParams rp,
                                                           float *depth, int32_t *key, int32_t *label)
{
    __shared__ uint32_t s_filter[FILTER ? kFilterWords : 4];
    if constexpr (FILTER) {
        if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) md.st->filtered = md.st->leaves_used;
        for (int i = threadIdx.x; i < kFilterWords / 4; i += kRenderThreads)
            ((uint4 *)s_filter)[i] = ((const uint4 *)md.filter)[i];
        __syncthreads();
    }
    // 4 waves of 8 x 8 pixels
    const int lane = lane_id(), wv = threadIdx.x >> 6;
    const int px = blockIdx.x * 32 + wv * 8 + (lane & 7), py = blockIdx.y * 8 + (lane >> 3);
    if (px >= rp.width || py >= rp.height) return;
    const long long i = (long long)py * rp.width + px;
    float out_d = NAN;
    int ok[3] = {0, 0, 0}, out_l = -1;
    const float dc0 = ((float)px - rp.cx) / rp.fx, dc1 = ((float)py - rp.cy) / rp.fy, dc2 = 1.0f;
    float p[3], u[3];
#pragma unroll
    for (int a = 0; a < 3; ++a)
        p[a] = fmaf(rp.R[3 * a + 0], dc0, fmaf(rp.R[3 * a + 1], dc1, fmaf(rp.R[3 * a + 2], dc2, rp.t[a])));
    const float d0 = p[0] - rp.t[0], d1 = p[1] - rp.t[1], d2 = p[2] - rp.t[2];
    const float r = sqrtf(fmaf(d2, d2, fmaf(d1, d1, d0 * d0)));
    if (r > 0.0f && isfinite(r)) {
        u[0] = d0 / r;
        u[1] = d1 / r;
        u[2] = d2 / r;
        const float vs = rp.vs, t0 = rp.t0, h = 0.5f * vs;
        int k[3], stp[3];
        float tm[3], td[3];
        bool go = true;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            const float s = fmaf(t0, u[a], rp.t[a]);
            const float fc = floorf(s / vs);
            go = go && fabsf(fc) < kCellLimit;
            const int c = fabsf(fc) < kCellLimit ? (int)fc : 0;
            if (u[a] > 0.0f) {
                stp[a] = 1;
                tm[a] = t0 + fmaf((float)(c + 1), vs, -s) / u[a];
                td[a] = vs / u[a];
            } else if (u[a] < 0.0f) {
                stp[a] = -1;
                tm[a] = t0 + fmaf((float)c, vs, -s) / u[a];
                td[a] = -vs / u[a];
            } else {
                stp[a] = 0;
                tm[a] = INFINITY;
                td[a] = INFINITY;
            }
            k[a] = rp.a[a] + c;
            go = go && key_ok(k[a]);
        }
        bool have_prev = false;
        float Dp = 0.0f, sp = 0.0f;
        const uint32_t stx = (uint32_t)stp[0] << 16, sty = (uint32_t)stp[1] << 8, stz = (uint32_t)stp[2];
        const float tdx = td[0], tdy = td[1], tdz = td[2];
        float tx = tm[0], ty = tm[1], tz = tm[2];
        uint32_t at = 0;
        constexpr uint32_t kBias = (64u << 16) | (64u << 8) | 64u;
        constexpr uint32_t kBlockBits = (0xC0u << 16) | (0xC0u << 8) | 0xC0u;  // change on the way out of a block
        constexpr uint32_t kLeafBits = (0xF8u << 16) | (0xF8u << 8) | 0xF8u;   // or of a leaf
        int it = 0;
        // one round per empty block or leaf, or leaf of the map
        while (go && it < rp.maxsteps) {
            // (past the key range no cell is observed, and a ray does not come back)
            if (((uint32_t)(k[0] + kKeyLimit) | (uint32_t)(k[1] + kKeyLimit) | (uint32_t)(k[2] + kKeyLimit)) >= 2u * kKeyLimit)
                break;
            uint32_t bits = kLeafBits;
            bool look = true;
            if constexpr (FILTER) {
                const uint32_t bb = block_bit(k[0], k[1], k[2]), lb = leaf_bit(k[0], k[1], k[2]);
                const uint32_t bw = s_filter[bb >> 5], lw = s_filter[lb >> 5];
                const bool block = (bw >> (bb & 31)) & 1u;
                bits = block ? kLeafBits : kBlockBits;
                look = block && ((lw >> (lb & 31)) & 1u);
            }
            int slot = -1;
            if (look) slot = map_find(md, pack_leaf(k[0] >> 3, k[1] >> 3, k[2] >> 3));
            const int l[3] = {k[0] >> 3, k[1] >> 3, k[2] >> 3};
            at = kBias + (((uint32_t)k[0] & 63u) << 16) + (((uint32_t)k[1] & 63u) << 8) + ((uint32_t)k[2] & 63u);
            const uint32_t at0 = at, home = at & bits;
            if (slot < 0) {
                have_prev = false;
                float tnext = 0.0f;
                bool ix;
                int n = 0;
                // (a way out takes at most 3 x 63 + 1 steps)
                do {
                    render_step(tx, ty, tz, at, tnext, ix, tdx, tdy, tdz, stx, sty, stz);
                    ++n;
                } while ((at & bits) == home && n < 192);
                it += n;
                // crossings come in order: one past the end on the way makes the last one so
                if (tnext > rp.t1) break;
            } else {
                // kRenderCells cells at a time: stepped through first, then their occupancy
                // and pages read side by side, then their D, then looked at in order
                bool inside = true;
                while (inside && it < rp.maxsteps) {
                    uint32_t cell[kRenderCells], word[kRenderCells];
                    int page[kRenderCells];
                    float D[kRenderCells];
                    int n = 0;
#pragma unroll
                    for (int c = 0; c < kRenderCells; ++c) {
                        cell[c] = at;
                        if (inside) {
                            float tnext;
                            bool ix;
                            render_step(tx, ty, tz, at, tnext, ix, tdx, tdy, tdz, stx, sty, stz);
                            ++n;
                            go = !(tnext > rp.t1);
                            inside = go && (at & kLeafBits) == home;
                        }
                    }
#pragma unroll
                    for (int c = 0; c < kRenderCells; ++c) {
                        const uint32_t x = (cell[c] >> 16) & 7u;
                        word[c] = c < n ? md.leaf_occ[(size_t)slot * kMaskWords + 2 * x + ((cell[c] >> 10) & 1u)] : 0u;
                        page[c] = c < n ? md.leaf_page[(size_t)slot * kLeafPages + x] : 0;
                    }
#pragma unroll
                    for (int c = 0; c < kRenderCells; ++c) {
                        const bool on = (word[c] >> (((cell[c] >> 5) & 24u) | (cell[c] & 7u))) & 1u;
                        const uint32_t off = ((cell[c] >> 5) & 56u) | (cell[c] & 7u);
                        D[c] = on ? md.vox[((size_t)page[c] * kPageVoxels + off) * md.rec_stride] : NAN;
                        word[c] = on ? 1u : 0u;
                    }
                    int hit = -1;
#pragma unroll
                    for (int c = 0; c < kRenderCells; ++c) {
                        if (c >= n || hit >= 0) continue;
                        if (!word[c]) {
                            have_prev = false;
                            continue;
                        }
                        const int kx = l[0] * 8 + (int)((cell[c] >> 16) & 7u), ky = l[1] * 8 + (int)((cell[c] >> 8) & 7u);
                        const int kz = l[2] * 8 + (int)(cell[c] & 7u);
                        const float qx = fmaf((float)(kx - rp.a[0]), vs, h) - rp.t[0];
                        const float qy = fmaf((float)(ky - rp.a[1]), vs, h) - rp.t[1];
                        const float qz = fmaf((float)(kz - rp.a[2]), vs, h) - rp.t[2];
                        const float sk = fmaf(qz, u[2], fmaf(qy, u[1], qx * u[0]));
                        if (have_prev && Dp > 0.0f && D[c] <= 0.0f) {
                            out_d = sp + (sk - sp) * (Dp / (Dp - D[c]));
                            ok[0] = kx;
                            ok[1] = ky;
                            ok[2] = kz;
                            hit = page[c];
                        }
                        have_prev = true;
                        Dp = D[c];
                        sp = sk;
                    }
                    it += n;
                    if (hit >= 0) {
                        const uint32_t off = (uint32_t)(((ok[0] & 7) << 3 | (ok[1] & 7)) << 3 | (ok[2] & 7)) & (kPageVoxels - 1);
                        const float *R = md.vox + ((size_t)hit * kPageVoxels + off) * md.rec_stride;
                        if (rp.mode == SLIM_SEM_CLOSED) {
                            float best = R[2];
                            out_l = 0;
                            for (int c = 1; c < rp.K; ++c)
                                if (R[2 + c] > best) {
                                    best = R[2 + c];
                                    out_l = c;
                                }
                        } else if (rp.mode == SLIM_SEM_CLOSED_LAST) {
                            out_l = (int)R[2];
                        }
                        go = inside = false;
                    }
                }
            }
            k[0] += (int)((at >> 16) & 255u) - (int)((at0 >> 16) & 255u);
            k[1] += (int)((at >> 8) & 255u) - (int)((at0 >> 8) & 255u);
            k[2] += (int)(at & 255u) - (int)(at0 & 255u);
        }
    }
    depth[i] = out_d;
    if (key) {
        key[3 * i + 0] = ok[0];
        key[3 * i + 1] = ok[1];
        key[3 * i + 2] = ok[2];
    }
    if (label) label[i] = out_l;
}

// Rays of at most this many cells are walked without the filters (every leaf on the
// way is looked up): the filters' launch and their copy to LDS take 3 to 7 us, more
// than a short walk saves.  Images of 64x48 over 63,000 scattered leaves, without and
// with: 1 cell 11 and 19 us, 32 cells 15 and 19, 48 cells 22 and 19, 100 cells 44 and
// 33; over the 8,200 leaves of a street 11 and 16, 30 and 33, 50 and 54, 95 and 99.
constexpr float kNearCells = 48.0f;

hipError_t launch_render(const MapDev &md, const RenderParams &rp, float *depth, int32_t *key, int32_t *label,
                         hipStream_t s)
{
    if (rp.width <= 0 || rp.height <= 0) return hipGetLastError();
    const dim3 grid((rp.width + 31) / 32, (rp.height + 7) / 8);
    if (rp.t1 - rp.t0 <= kNearCells * rp.vs) {
        hipLaunchKernelGGL(k_render<false>, grid, dim3(kRenderThreads), 0, s, md, rp, depth, key, label);
    } else {
        hipLaunchKernelGGL(k_render_filter, dim3(256), dim3(256), 0, s, md);
        hipLaunchKernelGGL(k_render<true>, grid, dim3(kRenderThreads), 0, s, md, rp, depth, key, label);
    }
    return hipGetLastError();
}

}  // namespace slim
