// Near field (Section 2.2, last step: the contributions of points in the near
// zone), written sorted as a float4 per point; the leaf-evaluation kernel adds
// it to the far field and writes the caller-order outputs.
//
// Work items of at most 64 targets of one leaf, heaviest first (a few in leaf
// order), taken off a counter by the blocks of a persistent grid.  An item with
// 16 or more targets gives each of its four waves a quarter of the targets and
// all of the sources; a smaller item gives every wave all of its targets and
// every fourth group of sources.  Inside a wave a target has
// S = floor(64 / targets of the wave) consecutive lanes that split the
// sources, so at least 60 of the 64 lanes work; the lane partial sums are
// combined by a shuffle tree inside the group of S lanes and, for a small
// item, over the waves, both in a fixed order.
// The source points are streamed through LDS as float4 (x, y, z, q) in global
// FP32 coordinates, so every pair difference is a correctly rounded FP32
// subtraction of the input coordinates.  Pairs at distance exactly zero (the
// self pair, coincident points) are skipped: the leaf's own points, the last of
// its sources, are tested pair by pair; between leaves two points meet only where their FP32
// coordinates round to one face, so those pairs run untested and an item whose
// sum comes out infinite or NaN is done again with every pair tested.
// The kernels are bound by VALU issue (14 instructions per untested pair
// forward, 16 tested; about 3 cycles each) once the reads are out of the way:
// a wave copies 64 staged positions at a time out of the runs of contiguous
// points that the tree build leaves, and the next batch is read while one is
// summed.  Reading box by box between barriers left the waves waiting for 58 %
// of their time (1M clustered points, alone: 0.84 ms forward and 1.36 ms
// backward with eight blocks per CU; now 0.75 and 1.07 with six, and 0.80 and
// 1.16 with the four it takes: 31 TFLOP/s forward at 20 FLOP per pair: 3 sub, 5
// for r^2, rsqrt, 4 for q/r and q/r^3, 7 for the four sums).
#include <float.h>
#include <math.h>

#include <algorithm>
#include <atomic>
#include <type_traits>

#include "common.h"

namespace kifmm {

namespace {

// source points staged per batch: kernels with one and with two arrays per
// source, and with two arrays and clump keys (at 512 these need 91 registers,
// and four blocks of them leave a CU no room for the M2L's: 200,000 pebbles,
// forces and gradients, 857 us against 802)
constexpr int NF_ONE = 512, NF_GRAD = 768, NF_TWO = 512, NF_KEYS = 256;

// near-field blocks wanted before the items of a small system are no longer divided
constexpr int kNearFill = 1024;

// Near-field blocks per CU.  Far-field kernels run beside it: with the CUs
// full of near-field blocks (eight) a far-field block waits until the near
// field's last blocks start, with four it starts at once and the far field's
// matrix products run beside the near field's vector instructions (524,288
// uniform points, evaluation and adjoint: 2.48 ms with four, 2.58 with three,
// 2.63 with six, 2.65 uncapped; 262,147 with field gradient 0.77 against 0.77,
// 0.97 and 1.01 ms).  Leaves of many points make no exception (evaluations with
// four and with six, ms: 330,000 uniform points, 81 a leaf, 0.48 and 0.55;
// 500,000 Plummer points, p = 8, 72 a leaf, 1.25 and 1.61; 1M clustered, 93 a
// leaf, 1.93 and 2.03); where the near field is nearly all the work six gain a
// little (1M clustered, p = 4, 93 a leaf, 1.62 and 1.52; 8.4M Plummer points
// 16.98 and 16.88).
constexpr int kNearBlocks = 4;

// Units of fewer than so many pairs (estimated from the mean near list) are taken
// four at a time (see near_units), or as many as a block has on average where
// that is fewer: 4,093 units over 1,024 blocks (100,000 points in a sheet, 24 a
// leaf, p = 4) took 189 us an evaluation one at a time, since each round of the
// blocks is then as long as the counter serves them (11 us), and 169 three at a
// time; half as many is no better at any size measured.  us an evaluation and an adjoint, one and
// four at a time: 3,800 pairs a unit (400,000 uniform points, 64 a leaf) 1407 +
// 1437 and 1221 + 1321, 11,600 (700,000, 128 a leaf) 1394 + 1494 and 1310 + 1481,
// 14,000 (1M clustered, 96 a leaf) 2140 + 2500 and 2090 + 2510, 31,800 (524,288
// uniform) 1156 + 1457 and 1160 + 1556.
constexpr int kNearChunk = 4;
constexpr double kNearLight = 16384;

// Blocks per CU the kernels are compiled for (at most 80 registers), none of
// them with scratch memory: bounds of seven and eight made six of the eight
// forms spill, and more registers leave the M2L no room beside four blocks.
constexpr int kNearBound = 6;

// The gathers precede everything else of a call on the caller's stream and
// zero its words: the near field's counter and the maximum of the right-hand
// side they set.
__global__ void k_gather(int64_t N, const float4* __restrict__ xs, const int* __restrict__ perm,
                         const float* __restrict__ q, float4* __restrict__ pts, int* __restrict__ words) {
    int64_t i = blockIdx.x * int64_t(256) + threadIdx.x;
    if (i == 0) words[0] = words[1] = 0;
    if (i >= N) return;
    float4 x = xs[i];
    x.w = q ? q[perm[i]] : 0.f;
    pts[i] = x;
}

__global__ void k_gather_adj(int64_t N, const int* __restrict__ perm, const float* __restrict__ gu,
                             const float* __restrict__ ge, float4* __restrict__ src2, int* __restrict__ words) {
    int64_t i = blockIdx.x * int64_t(256) + threadIdx.x;
    if (i == 0) words[0] = words[2] = 0;
    if (i >= N) return;
    int j = perm[i];
    src2[i] = make_float4(gu ? gu[j] : 0.f, ge ? ge[3 * size_t(j)] : 0.f, ge ? ge[3 * size_t(j) + 1] : 0.f,
                          ge ? ge[3 * size_t(j) + 2] : 0.f);
}

// 1/sqrt(r2); with CHK zero at r2 = 0, otherwise infinite there
template <bool CHK>
__device__ inline float rsq(float r2) {
    const float ri = __frsqrt_rn(r2);
    return CHK ? (r2 > 0.f ? ri : 0.f) : ri;
}

// Lane map of a work item (first target `first`, nt targets, 1 <= nt <= 64).
struct NearMap {
    int S;         // lanes per target in this wave (4 .. 64)
    float inv;     // 1 / dj
    int slice;     // this lane's place among them
    int i;         // target (sorted index)
    int j0, dj;    // staged sources lo + j0, lo + j0 + dj, ... of a range [lo, hi)
    bool act;      // the lane serves a target
    bool split;    // the waves split the sources (small item): sum over waves
};

__device__ inline NearMap near_map(int first, int nt) {
    NearMap m;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    m.split = nt < 16;
    const int per = m.split ? nt : (nt + 3) / 4;   // targets per wave
    const int t0 = m.split ? 0 : w * per;
    const int ntw = min(per, nt - t0);              // >= 1: nt - 3 ceil(nt/4) > 0 for nt >= 16
    // quotients of small integers through FP32: (k + 1/2) / n is never within
    // rounding of an integer, so its floor is exact
    m.S = int(64.5f / float(ntw));
    const int tl = int((float(lane) + 0.5f) / float(m.S));
    m.slice = lane - tl * m.S;
    m.act = tl < ntw;
    m.i = first + t0 + tl;
    m.j0 = m.split ? w * m.S + m.slice : m.slice;
    m.dj = m.split ? 4 * m.S : m.S;
    m.inv = 1.f / float(m.dj);
    return m;
}

// Calls f(j) for this lane's staged sources j = lo + j0, lo + j0 + dj, ...
// below hi.  Every lane of the wave has T = ceil((hi - lo) / dj) or T - 1 of
// them (j0 < dj), and its first T - 1 are below hi: those steps run without a
// bounds check and with a wave-uniform trip count, only the last one is checked.
template <int UNROLL, class F>
__device__ inline void for_sources(const NearMap& nm, int lo, int hi, F f) {
    const int T = __builtin_amdgcn_readfirstlane(int((float(hi - lo + nm.dj) - 0.5f) * nm.inv));
    int j = lo + nm.j0;
#pragma unroll UNROLL
    for (int st = 0; st < T - 1; ++st, j += nm.dj) f(j);
    if (T > 0 && j < hi) f(j);
}

// Sum over the S lanes of a target (lanes [g S, g S + S) of the wave); the
// first lane of the group ends with the total.
__device__ inline float group_sum(float v, int slice, int S) {
    for (int off = 1; off < S; off <<= 1) {
        const float t = __shfl_down(v, off, 64);
        if (slice + off < S) v += t;
    }
    return v;
}

// What the near-field kernels read beside the points.
struct NearArgs {
    const int4* items;   // two words an item, see k_item_fill
    int units, parts;    // units of work: every item in `parts` equal parts of its targets
    const int4* runs;    // runs of contiguous source points, see k_item_fill
    int* taken;          // units taken beyond the grid's first round, ...
    int chunk;           // ... so many at a time
    float cell;          // periodic cell side (image shifts)
};

// LDS of a near-field block; the wave reduction reuses the staging.
template <int CAP, bool TWO, bool KEY, int NV>
struct NearShared {
    union {
        struct {
            float4 p[CAP];
            float4 p2[TWO ? CAP : 1];
        };
        float red[4][NV][64];
    };
    int key[KEY ? CAP : 1];
    int next[2];   // the block's next unit, in turns
};

typedef float nv4 __attribute__((ext_vector_type(4)));

// The source points a thread copies of one batch.  (p2 as native vectors: an
// array of float4 structures stayed in scratch memory, stored and read back
// every batch.)
template <int CAP, bool TWO, bool KEY>
struct Staged {
    float4 p[CAP / 256];
    nv4 p2[TWO ? CAP / 256 : 1];
    int key[KEY ? CAP / 256 : 1];

    // Read the points at positions [b0, b0 + m) of the runs; a wave takes 64
    // consecutive positions at a time.  d, dn: this lane's run of the first 64
    // and the position behind it.  A periodic image is moved by its shift
    // times the cell side.
    __device__ inline void read(const int4* __restrict__ run, int nr, int4 d, int dn, int b0, int m, float cell,
                                const float4* __restrict__ pts, const float4* __restrict__ src2,
                                const int* __restrict__ ckey) {
        const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
#pragma unroll
        for (int c = 0; c < CAP / 256; ++c) {
            const int lo = b0 + c * 256 + w * 64;   // first position of the wave
            if (lo >= b0 + m) continue;
            const int pos = lo + lane, hi = min(lo + 64, b0 + m);
            int from = 0, code = 0;   // of the run that holds pos: index of the point - position, image
            for (int r0 = 0; r0 < nr; r0 += 64) {
                int4 e = d;
                int en = dn;
                if (r0) {   // more than 64 runs
                    const int r = min(r0 + lane, nr);
                    e = run[r];
                    en = run[min(r + 1, nr)].y;
                }
                // the runs that meet [lo, hi): lane k holds one when it starts before hi and ends after lo
                uint64_t meet = __ballot(r0 + lane < nr && e.y < hi && en > lo);
                while (meet) {
                    const int k = __builtin_ctzll(meet);
                    meet &= meet - 1;
                    // lane k need not be one of the lanes behind dst: all three reads with every lane on
                    const int src = __builtin_amdgcn_readlane(e.x, k), dst = __builtin_amdgcn_readlane(e.y, k),
                              img = __builtin_amdgcn_readlane(e.z, k);
                    const bool in = pos >= dst;
                    from = in ? src - dst : from;
                    code = in ? img : code;
                }
            }
            if (pos < hi) {
                const size_t at = size_t(from + pos);
                p[c] = pts[at];
                if (TWO) p2[c] = reinterpret_cast<const nv4*>(src2)[at];
                if (KEY) key[c] = ckey[at];
                if (code) {
                    int sx, sy, sz;
                    img_shift(code << kShiftBits, sx, sy, sz);
                    p[c].x += sx * cell;
                    p[c].y += sy * cell;
                    p[c].z += sz * cell;
                }
            }
        }
    }

    template <class Sh>
    __device__ inline void write(Sh& sh, int m) const {
#pragma unroll
        for (int c = 0; c < CAP / 256; ++c) {
            const int at = c * 256 + int(threadIdx.x);
            if (at < m) {
                sh.p[at] = p[c];
                if (TWO) reinterpret_cast<nv4*>(sh.p2)[at] = p2[c];
                if (KEY) sh.key[at] = key[c];
            }
        }
    }
};

// Sum NV per-lane values over the four waves in a fixed order (wave 0 ends
// with the totals).
template <int NV>
__device__ inline void wave_reduce(float (&v)[NV], float (*red)[NV][64]) {
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    __syncthreads();
#pragma unroll
    for (int q = 0; q < NV; ++q) red[w][q][lane] = v[q];
    __syncthreads();
    if (w == 0)
#pragma unroll
        for (int q = 0; q < NV; ++q) v[q] = ((red[0][q][lane] + red[1][q][lane]) + red[2][q][lane]) + red[3][q][lane];
}

// Totals of an item's lane partials; true on the lane that writes them.
// Block-uniform (m.split depends on the item only).
template <int NV>
__device__ inline bool near_finish(float (&v)[NV], const NearMap& m, float (*red)[NV][64]) {
#pragma unroll
    for (int q = 0; q < NV; ++q) v[q] = group_sum(v[q], m.slice, m.S);
    if (!m.split) return m.act && m.slice == 0;
    wave_reduce<NV>(v, red);
    return (threadIdx.x >> 6) == 0 && m.act && m.slice == 0;
}

// The units of a near-field block.  load(i, act) reads target i, pair(chk, j, v)
// adds staged source j to the sums v, store(i, v) writes the totals.
// The next batch of sources is read into registers while the present one is
// summed.  Blocks take their later units from a counter, so that a grid smaller
// than the work keeps its balance, several neighbouring ones at a time where
// there are many: the counter serves one block in 11 ns, which is longer than
// small leaves take (100,000 points in a sheet, 6 a leaf, 17,000 units: 188 us
// one at a time, 90 four at a time).  A unit's arithmetic does not depend on the
// block that does it.
template <int CAP, bool TWO, bool KEY, int NV, int UNROLL, class Load, class Pair, class Store>
__device__ inline void near_units(const NearArgs& a, const float4* __restrict__ pts, const float4* __restrict__ src2,
                                  const int* __restrict__ ckey, NearShared<CAP, TWO, KEY, NV>& sh, Load load,
                                  Pair pair, Store store) {
    const int lane = threadIdx.x & 63;
    int unit = blockIdx.x, end = unit + 1;   // end: behind the units taken (thread 0)
    int4 i0 = a.items[2 * size_t(unit / a.parts)], i1 = a.items[2 * size_t(unit / a.parts) + 1];
    for (int turn = 0; unit < a.units; turn ^= 1) {
        const int per = (i0.y + a.parts - 1) / a.parts, t0 = (unit % a.parts) * per, nt = min(per, i0.y - t0);
        const int4* run = a.runs + i0.z;
        const int nr = i0.w, own = KEY ? 0 : i1.x, total = nt > 0 ? i1.y : 0;
        const int4 d = run[min(lane, nr)];
        const int dn = run[min(lane + 1, nr)].y;
        int next = a.units;
        if (threadIdx.x == 0 && gridDim.x < unsigned(a.units)) {
            if (unit + 1 < end) {
                next = unit + 1;
            } else {
                next = int(gridDim.x) + atomicAdd(a.taken, a.chunk);
                end = next + a.chunk;
            }
        }
        const NearMap nm = near_map(i0.x + t0, max(nt, 1));
        load(nm.i, nm.act && nt > 0);
        float v[NV];
        // first with only the leaf's own points tested for distance zero (with
        // keys, none: they tell the self pair), then, if a sum is not finite, all
        for (int pass = 0; pass < 2; ++pass) {
#pragma unroll
            for (int q = 0; q < NV; ++q) v[q] = 0.f;
            Staged<CAP, TWO, KEY> st;
            st.read(run, nr, d, dn, 0, min(CAP, total), a.cell, pts, src2, ckey);
            for (int b0 = 0; b0 < total; b0 += CAP) {
                const int m = min(CAP, total - b0);
                const int untested = pass ? 0 : min(max(total - own - b0, 0), m);   // the leaf's own points come last
                __syncthreads();
                st.write(sh, m);
                __syncthreads();
                if (b0 + CAP < total)
                    st.read(run, nr, d, dn, b0 + CAP, min(CAP, total - b0 - CAP), a.cell, pts, src2, ckey);
                for_sources<UNROLL>(nm, 0, untested, [&](int j) { pair(std::false_type{}, j, v); });
                for_sources<UNROLL>(nm, untested, m, [&](int j) { pair(std::true_type{}, j, v); });
            }
            // every sum of v[0] has 1/r as a factor, and any number times
            // infinity is not finite
            if (threadIdx.x == 0) sh.next[turn] = next;
            if (!__syncthreads_or(pass == 0 && nm.act && !(fabsf(v[0]) <= FLT_MAX))) break;
        }
        unit = sh.next[turn];
        if (unit < a.units) {   // read ahead of the reduction
            i0 = a.items[2 * size_t(unit / a.parts)];
            i1 = a.items[2 * size_t(unit / a.parts) + 1];
        }
        if (near_finish<NV>(v, nm, sh.red) && nt > 0) store(nm.i, v);
    }
}

// EXCL: pairs whose clump keys (ckey, sorted) are equal are left out, which
// drops the pairs of pebbles of one clump and the self pair.
template <bool EXCL>
__global__ __launch_bounds__(256, kNearBound) void k_p2p(NearArgs a, const float4* __restrict__ pts, float cst,
                                             float4* __restrict__ nearv, const int* __restrict__ ckey) {
    __shared__ NearShared<NF_ONE, false, EXCL, 4> sh;
    float4 x;
    int ck = 0;
    near_units<NF_ONE, false, EXCL, 4, 4>(
        a, pts, nullptr, ckey, sh,
        [&](int i, bool act) {
            x = act ? pts[i] : make_float4(0, 0, 0, 0);
            if (EXCL) ck = act ? ckey[i] : 0;
        },
        [&](auto chk, int j, float(&v)[4]) {   // v: u, ex, ey, ez
            const float4 y = sh.p[j];
            const float dx = x.x - y.x, dy = x.y - y.y, dz = x.z - y.z;
            float ri = rsq<decltype(chk)::value>(dx * dx + dy * dy + dz * dz);
            if (EXCL) ri = sh.key[j] != ck ? ri : 0.f;
            const float qr = y.w * ri;
            const float qr3 = qr * ri * ri;
            v[0] += qr;
            v[1] += qr3 * dx;
            v[2] += qr3 * dy;
            v[3] += qr3 * dz;
        },
        [&](int i, const float(&v)[4]) { nearv[i] = make_float4(cst * v[0], cst * v[1], cst * v[2], cst * v[3]); });
}

// Near field of monopoles q_j and dipoles m_j (src2 = (q, m) sorted):
//   u += q_j/r - m_j.r/r^3,  E = -grad u += r (q_j/r^3 - 3 m_j.r/r^5) + m_j/r^3.
__global__ __launch_bounds__(256, kNearBound) void k_p2p_dip(NearArgs a, const float4* __restrict__ pts,
                                                 const float4* __restrict__ src2, float cst,
                                                 float4* __restrict__ nearv) {
    __shared__ NearShared<NF_TWO, true, false, 4> sh;
    float4 x;
    near_units<NF_TWO, true, false, 4, 2>(
        a, pts, src2, nullptr, sh, [&](int i, bool act) { x = act ? pts[i] : make_float4(0, 0, 0, 0); },
        [&](auto chk, int j, float(&v)[4]) {   // v: u, ex, ey, ez
            const float4 y = sh.p[j];
            const float4 bj = sh.p2[j];
            const float dx = x.x - y.x, dy = x.y - y.y, dz = x.z - y.z;
            const float ri = rsq<decltype(chk)::value>(dx * dx + dy * dy + dz * dz);
            const float ri2 = ri * ri;
            const float ri3 = ri2 * ri;
            // with c = m.r/r^2: u term (q - c)/r, radial field (q - 3c)/r^3
            const float c = (dx * bj.y + dy * bj.z + dz * bj.w) * ri2;
            v[0] += ri * (bj.x - c);
            const float gh = ri3 * (bj.x - 3.f * c);
            v[1] += gh * dx + bj.y * ri3;
            v[2] += gh * dy + bj.z * ri3;
            v[3] += gh * dz + bj.w * ri3;
        },
        [&](int i, const float(&v)[4]) { nearv[i] = make_float4(cst * v[0], cst * v[1], cst * v[2], cst * v[3]); });
}

// Near field with the field gradient, of monopoles (src2.x, or pts.w without
// src2) and dipoles (src2.yzw): u, E and dE_a/dx_b = -Hess u, the dipole
// part of the Hessian being 3 (m_a r_b + m_b r_a + (m.r) delta_ab)/r^5
// - 15 (m.r) r_a r_b / r^7.  (u, E) go to nearv, dE/dx (xx yy zz xy xz yz)
// to nearg.
template <bool DIP>
__global__ __launch_bounds__(256, kNearBound) void k_p2p_grad(NearArgs a, const float4* __restrict__ pts,
                                                  const float4* __restrict__ src2, float cst,
                                                  float4* __restrict__ nearv, float* __restrict__ nearg) {
    constexpr int CAP = DIP ? NF_TWO : NF_GRAD;
    __shared__ NearShared<CAP, DIP, false, 10> sh;
    float4 x;
    near_units<CAP, DIP, false, 10, DIP ? 2 : 4>(
        a, pts, src2, nullptr, sh, [&](int i, bool act) { x = act ? pts[i] : make_float4(0, 0, 0, 0); },
        [&](auto chk, int j, float(&v)[10]) {   // v: u, E xyz, dE/dx xx yy zz xy xz yz
            const float4 y = sh.p[j];
            const float d0 = x.x - y.x, d1 = x.y - y.y, d2 = x.z - y.z;
            const float ri = rsq<decltype(chk)::value>(d0 * d0 + d1 * d1 + d2 * d2);
            const float ri2 = ri * ri;
            const float ri3 = ri2 * ri;
            if constexpr (!DIP) {
                // charge q: u = q/r, E = g d, dE_a/dx_c = g delta_ac - 3 g d_a d_c / r^2, g = q/r^3
                const float g = y.w * ri3;
                const float c = -3.f * g * ri2;
                v[0] += y.w * ri;
                v[1] += g * d0;
                v[2] += g * d1;
                v[3] += g * d2;
                const float e0 = c * d0, e1 = c * d1, e2 = c * d2;
                v[4] += e0 * d0 + g;
                v[5] += e1 * d1 + g;
                v[6] += e2 * d2 + g;
                v[7] += e0 * d1;
                v[8] += e0 * d2;
                v[9] += e1 * d2;
            } else {
                // charge q and dipole m (u += q/r - m.d/r^3): with t = 3 (m.d)/r^5,
                // E = gh d + m/r^3, gh = q/r^3 - t, and
                // dE_a/dx_c = coef d_a d_c - p_a d_c - p_c d_a + gh delta_ac,
                // coef = 5 t/r^2 - 3 q/r^5, p = 3 m/r^5
                const float4 bj = sh.p2[j];
                const float ri5 = ri3 * ri2;
                const float mr = d0 * bj.y + d1 * bj.z + d2 * bj.w;
                const float t = 3.f * mr * ri5;
                const float gh = bj.x * ri3 - t;
                v[0] += bj.x * ri - mr * ri3;
                v[1] += gh * d0 + bj.y * ri3;
                v[2] += gh * d1 + bj.z * ri3;
                v[3] += gh * d2 + bj.w * ri3;
                const float coef = 5.f * t * ri2 - 3.f * bj.x * ri5;
                const float p0 = 3.f * ri5 * bj.y, p1 = 3.f * ri5 * bj.z, p2 = 3.f * ri5 * bj.w;
                // e_a = coef d_a - p_a, so that dE_a/dx_c = e_a d_c - p_c d_a (+ gh on the diagonal)
                const float e0 = coef * d0 - p0, e1 = coef * d1 - p1, e2 = coef * d2 - p2;
                v[4] += (e0 - p0) * d0 + gh;
                v[5] += (e1 - p1) * d1 + gh;
                v[6] += (e2 - p2) * d2 + gh;
                v[7] += e0 * d1 - p1 * d0;
                v[8] += e0 * d2 - p2 * d0;
                v[9] += e1 * d2 - p2 * d1;
            }
        },
        [&](int i, const float(&v)[10]) {
            nearv[i] = make_float4(cst * v[0], cst * v[1], cst * v[2], cst * v[3]);
#pragma unroll
            for (int k = 0; k < 6; ++k) nearg[6 * size_t(i) + k] = cst * v[4 + k];
        });
}

// Backward near field, summed directly as the near part of the combination
//   qbar_k = psi_k,  xbar_k = -ubar_k E_k - H_k Ebar_k - q_k E_psi,k
// where E, H come from the charges q and psi, E_psi from monopoles ubar and
// dipoles Ebar (psi = sum ubar K - Ebar . G).
template <bool EXCL>
__global__ __launch_bounds__(256, kNearBound) void k_p2p_bwd(NearArgs na, const float4* __restrict__ pts,
                                                    const float4* __restrict__ src2, float cst,
                                                    float4* __restrict__ nearv, const int* __restrict__ ckey) {
    constexpr int CAP = EXCL ? NF_KEYS : NF_TWO;
    __shared__ NearShared<CAP, true, EXCL, 9> sh;
    // The adjoint combination xbar_k = -ubar_k E_k - H_k Ebar_k - q_k E_psi,k
    // is summed pair by pair (r = x_k - y_j, c applied at the end):
    //   xbar += r [-(ubar_k q_j + q_k ubar_j)/r^3 - 3 (q_j r.Ebar_k - q_k r.Ebar_j)/r^5]
    //           + (q_j Ebar_k - q_k Ebar_j)/r^3,
    // with the target's Ebar_k taken out of the sum: v = (S, X xyz, T xyz, psi)
    // and xbar = X + S Ebar_k - q_k T;  qbar = psi = sum ubar_j/r - r.Ebar_j/r^3.
    // psi is kept as its two sums (v[7] ubar_j / r, v[8] r.Ebar_j / r^3)
    float4 x, a;
    int ck = 0;
    near_units<CAP, true, EXCL, 9, 1>(
        na, pts, src2, ckey, sh,
        [&](int i, bool act) {
            x = act ? pts[i] : make_float4(0, 0, 0, 0);
            a = act ? src2[i] : make_float4(0, 0, 0, 0);
            if (EXCL) ck = act ? ckey[i] : 0;
        },
        [&](auto chk, int j, float(&v)[9]) {
            const float uk = a.x, qk = x.w;
            const float4 y = sh.p[j];
            const float4 bj = sh.p2[j];
            const float dx = x.x - y.x, dy = x.y - y.y, dz = x.z - y.z;
            float ri = rsq<decltype(chk)::value>(dx * dx + dy * dy + dz * dz);
            if (EXCL) ri = sh.key[j] != ck ? ri : 0.f;
            const float ri2 = ri * ri;
            const float ri3 = ri2 * ri;
            const float rk = dx * a.y + dy * a.z + dz * a.w;
            const float rj = dx * bj.y + dy * bj.z + dz * bj.w;
            const float t1 = uk * y.w + qk * bj.x;
            const float t2 = y.w * rk - qk * rj;
            // -(t1 / r^3 + 3 t2 / r^5)
            const float coef = -ri3 * (t1 + 3.f * (ri2 * t2));
            v[1] += coef * dx;
            v[2] += coef * dy;
            v[3] += coef * dz;
            v[0] += y.w * ri3;
            v[4] += bj.y * ri3;
            v[5] += bj.z * ri3;
            v[6] += bj.w * ri3;
            v[7] += bj.x * ri;
            v[8] += rj * ri3;
        },
        [&](int i, const float(&v)[9]) {
            const float qk = x.w;
            nearv[i] = make_float4(cst * (v[1] + v[0] * a.y - qk * v[4]), cst * (v[2] + v[0] * a.z - qk * v[5]),
                                   cst * (v[3] + v[0] * a.w - qk * v[6]), cst * (v[7] - v[8]));
        });
}

// Stokeslet sources: pass 0 sets pts.w = f_x, src2 = (f_y, 0, 0, 0) and the
// sorted forces stk = (f_x, f_y, f_z, 0); pass 1 sets pts.w = f_z.  The
// fourth harmonic charge, (x - c) . f about each box's centre c, is formed
// from stk where a box's sources are summed.
__global__ void k_gather_stokes(int64_t N, const float4* __restrict__ xs, const int* __restrict__ perm,
                                const float* __restrict__ f, int pass, float4* __restrict__ pts,
                                float4* __restrict__ src2, float4* __restrict__ stk, int* __restrict__ words) {
    int64_t i = blockIdx.x * int64_t(256) + threadIdx.x;
    if (pass == 0 && i == 0) words[0] = 0;   // the near field of pass 0 may still run in pass 1
    if (i >= N) return;
    const size_t j = size_t(perm[i]);
    const float fx = f[3 * j], fy = f[3 * j + 1], fz = f[3 * j + 2];
    float4 x = xs[i];
    if (pass == 0) {
        x.w = fx;
        src2[i] = make_float4(fy, 0.f, 0.f, 0.f);
        stk[i] = make_float4(fx, fy, fz, 0.f);
    } else {
        x.w = fz;
    }
    pts[i] = x;
}

// Near field of point forces (the Stokeslet): u += f/r + (r.f) r/r^3 over
// the near lists, pairs at distance zero skipped; positions from xs, forces
// from stk (sorted); written as cst * u to out (sorted), with the unscaled sum
// of (r.f)/r^3 (the near part of the pressure, times 4 pi) in the fourth
// component.
__global__ __launch_bounds__(256, kNearBound) void k_p2p_stokes(NearArgs a, const float4* __restrict__ xs,
                                                    const float4* __restrict__ stk, float cst,
                                                    float4* __restrict__ out) {
    __shared__ NearShared<NF_TWO, true, false, 4> sh;
    float4 x;
    near_units<NF_TWO, true, false, 4, 1>(
        a, xs, stk, nullptr, sh, [&](int i, bool act) { x = act ? xs[i] : make_float4(0, 0, 0, 0); },
        [&](auto chk, int j, float(&v)[4]) {
            const float4 y = sh.p[j];
            const float4 fj = sh.p2[j];
            const float dx = x.x - y.x, dy = x.y - y.y, dz = x.z - y.z;
            const float ri = rsq<decltype(chk)::value>(dx * dx + dy * dy + dz * dz);
            const float t = (dx * fj.x + dy * fj.y + dz * fj.z) * ri * ri * ri;
            v[0] += fj.x * ri + t * dx;
            v[1] += fj.y * ri + t * dy;
            v[2] += fj.z * ri + t * dz;
            v[3] += t;
        },
        [&](int i, const float(&v)[4]) { out[i] = make_float4(cst * v[0], cst * v[1], cst * v[2], v[3]); });
}

// Arguments and grid of a near-field launch.
struct NearLaunch {
    NearArgs args;
    dim3 grid;
};

int device_cus() {
    static std::atomic<int> cus[kMaxDevices];
    int dev = 0;
    KIFMM_HIP(hipGetDevice(&dev));
    const bool kept = dev >= 0 && dev < kMaxDevices;
    int n = kept ? cus[dev].load(std::memory_order_relaxed) : 0;
    if (n == 0) {
        KIFMM_HIP(hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev));
        if (kept) cus[dev].store(n, std::memory_order_relaxed);
    }
    return n;
}

NearLaunch near_launch(kifmm_plan* P, bool images = true) {
    // few items: in parts, until the chip has work for half a round of eight
    // blocks per CU
    int parts = 1;
    while (parts < 8 && P->n_items * parts < kNearFill) parts *= 2;
    const int units = int(P->n_items) * parts;
    const int blocks = std::min(units, device_cus() * kNearBlocks);
    const double leaf = double(P->N) / double(P->nleaves), lists = double(P->near_entries) / double(P->nleaves);
    const bool light = std::min(64.0, leaf) * lists * leaf < kNearLight;
    return NearLaunch{NearArgs{P->items_near.as<int4>(), units, parts, P->runs, P->words.as<int>(),
                               light ? std::max(1, std::min(kNearChunk, units / blocks)) : 1, images ? float(P->side) : 0.f},
                      dim3(unsigned(blocks))};
}

}  // namespace

void launch_gather(kifmm_plan* P, const float* charges, const float* gpot, const float* gfield, bool adjoint,
                   hipStream_t s, bool points) {
    const int64_t N = P->N;
    int* words = static_cast<int*>(P->words.ensure(3 * sizeof(int)));
    if (charges || points) {
        P->pts.ensure(size_t(N) * 16);
        hipLaunchKernelGGL(k_gather, dim3(unsigned((N + 255) / 256)), dim3(256), 0, s, N, P->xs.as<float4>(),
                           P->perm.as<int>(), charges, P->pts.as<float4>(), words);
    }
    if (adjoint) {
        P->src2.ensure(size_t(N) * 16);
        hipLaunchKernelGGL(k_gather_adj, dim3(unsigned((N + 255) / 256)), dim3(256), 0, s, N, P->perm.as<int>(), gpot,
                           gfield, P->src2.as<float4>(), words);
    }
}

void launch_gather_stokes(kifmm_plan* P, const float* forces, int pass, hipStream_t s) {
    const int64_t N = P->N;
    P->pts.ensure(size_t(N) * 16);
    P->src2.ensure(size_t(N) * 16);
    P->stk.ensure(size_t(N) * 16);
    hipLaunchKernelGGL(k_gather_stokes, dim3(unsigned((N + 255) / 256)), dim3(256), 0, s, N, P->xs.as<float4>(),
                       P->perm.as<int>(), forces, pass, P->pts.as<float4>(), P->src2.as<float4>(),
                       P->stk.as<float4>(), static_cast<int*>(P->words.ensure(3 * sizeof(int))));
}

void launch_p2p_forward(kifmm_plan* P, hipStream_t s, bool excl) {
    const NearLaunch l = near_launch(P);
    if (excl)
        hipLaunchKernelGGL(k_p2p<true>, l.grid, dim3(256), 0, s, l.args, P->pts.as<float4>(), float(P->c),
                           P->nearv.as<float4>(), (const int*)P->cid_s.as<int>());
    else
        hipLaunchKernelGGL(k_p2p<false>, l.grid, dim3(256), 0, s, l.args, P->pts.as<float4>(), float(P->c),
                           P->nearv.as<float4>(), (const int*)nullptr);
}

void launch_p2p_stokes(kifmm_plan* P, double viscosity, hipStream_t s) {
    P->stk_near.ensure(size_t(P->N) * 16);
    // the Stokes cell is not periodic: no image shifts in the lists
    const NearLaunch l = near_launch(P, false);
    hipLaunchKernelGGL(k_p2p_stokes, l.grid, dim3(256), 0, s, l.args, P->xs.as<float4>(), P->stk.as<float4>(),
                       float(1.0 / (8.0 * M_PI * viscosity)), P->stk_near.as<float4>());
}

void launch_p2p_dipoles(kifmm_plan* P, hipStream_t s) {
    const NearLaunch l = near_launch(P);
    hipLaunchKernelGGL(k_p2p_dip, l.grid, dim3(256), 0, s, l.args, P->pts.as<float4>(), P->src2.as<float4>(),
                       float(P->c), P->nearv.as<float4>());
}

void launch_p2p_gradient(kifmm_plan* P, bool dipoles, hipStream_t s) {
    P->nearg.ensure(size_t(P->N) * 24);
    const NearLaunch l = near_launch(P);
    if (dipoles)
        hipLaunchKernelGGL(k_p2p_grad<true>, l.grid, dim3(256), 0, s, l.args, P->pts.as<float4>(),
                           P->src2.as<float4>(), float(P->c), P->nearv.as<float4>(), P->nearg.as<float>());
    else
        hipLaunchKernelGGL(k_p2p_grad<false>, l.grid, dim3(256), 0, s, l.args, P->pts.as<float4>(),
                           (const float4*)nullptr, float(P->c), P->nearv.as<float4>(), P->nearg.as<float>());
}

void launch_p2p_backward(kifmm_plan* P, hipStream_t s, bool excl) {
    const NearLaunch l = near_launch(P);
    if (excl)
        hipLaunchKernelGGL(k_p2p_bwd<true>, l.grid, dim3(256), 0, s, l.args, P->pts.as<float4>(),
                           P->src2.as<float4>(), float(P->c), P->nearv.as<float4>(), (const int*)P->cid_s.as<int>());
    else
        hipLaunchKernelGGL(k_p2p_bwd<false>, l.grid, dim3(256), 0, s, l.args, P->pts.as<float4>(),
                           P->src2.as<float4>(), float(P->c), P->nearv.as<float4>(), (const int*)nullptr);
}

}  // namespace kifmm
