// HIP kernels (gfx950 / CDNA4) of the charge-transport hot path of
// Avalos & Sofo Haro, arXiv 2203.11043:
//   field_tiles_matrix, field_tiles -- Eq. (6), softened all-pairs Coulomb field
//                    (the O(N^2) part)
//   near_matrix, near_waves -- the near part of the closure's split of Eq. (6)
//   step_update   -- Eqs. (1)-(4) and the z check of Sec. III.B, fused per carrier
//   drift_steps   -- the same for several steps at once, without repulsion
//   load_prepare  -- a load's positions taken in, with its boundary handling
//   make_keys, count_active, gather_tiles -- the spatially sorted carrier list
//   image_bin     -- 2D histogram of collected holes (Sec. V.A)
// Several independent events (clouds) can share one launch; every kernel
// keeps them apart through the per-event slot offsets.
#include "gccd.h"
#include "gccd_fp64.h"
#include "gccd_internal.h"
#include "gccd_sort_dev.h"

#include <math.h>
#include <type_traits>

namespace gccd {

// ---------------------------------------------------------------------------
// Keys.  A hole's 0.25 um cell (12 bits per axis, wrapping every 1024 um) is
// mapped to its 36-bit index along a 3D Hilbert curve, which visits
// face-adjacent cells one after the other: a run of consecutive keys is a
// compact region with no jumps, so source tiles and target blocks have small
// bounding boxes.  The index follows Skilling's transposition (J. Skilling,
// "Programming the Hilbert curve", AIP Conf. Proc. 707, 381 (2004)): undo
// the excess work axis by axis from the top bit down, Gray-encode, and
// interleave the bits of the transposed coordinates (x first in each triple).
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint32_t cell12(double v) {
    if (!isfinite(v)) return 0u;
    return (uint32_t)(int64_t)floor(v * kCellPerUm) & 0xFFFu;
}

__device__ __forceinline__ uint64_t hilbert36(uint32_t cx, uint32_t cy, uint32_t cz) {
    uint32_t X[3] = {cx, cy, cz};
#pragma unroll
    for (uint32_t Q = 1u << 11; Q > 1u; Q >>= 1) {
        const uint32_t P = Q - 1u;
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            const bool set = (X[i] & Q) != 0u;
            const uint32_t t = set ? 0u : ((X[0] ^ X[i]) & P);  // exchange low bits
            X[0] ^= (set ? P : 0u) ^ t;                          // or invert them
            X[i] ^= t;
        }
    }
    X[1] ^= X[0];
    X[2] ^= X[1];
    uint32_t t = 0u;
#pragma unroll
    for (uint32_t Q = 1u << 11; Q > 1u; Q >>= 1)
        if (X[2] & Q) t ^= Q - 1u;
    X[0] ^= t;
    X[1] ^= t;
    X[2] ^= t;
    uint64_t key = 0;
#pragma unroll
    for (int j = 11; j >= 0; --j) {
#pragma unroll
        for (int i = 0; i < 3; ++i) key = (key << 1) | (uint64_t)((X[i] >> j) & 1u);
    }
    return key;
}

__device__ __forceinline__ uint64_t make_key(uint32_t event, bool collected, double x, double y,
                                             double z, uint32_t local, KeyLayout kl) {
    uint64_t k = (uint64_t)local;
    k |= hilbert36(cell12(x), cell12(y), cell12(z)) << kl.lbits;
    if (collected) k |= 1ull << (kl.lbits + kCurveBits);
    k |= (uint64_t)event << (kl.lbits + kCurveBits + 1);
    return k;
}

__device__ __forceinline__ uint32_t key_local(uint64_t k, KeyLayout kl) {
    return (uint32_t)(k & ((1ull << kl.lbits) - 1ull));
}

__device__ __forceinline__ uint32_t key_event(uint64_t k, KeyLayout kl) {
    return (uint32_t)(k >> (kl.lbits + kCurveBits + 1));
}

__device__ __forceinline__ bool key_collected(uint64_t k, KeyLayout kl) {
    return ((k >> (kl.lbits + kCurveBits)) & 1ull) != 0ull;
}

// event of carrier i: the last e with ev_off[e] <= i (binary search)
__device__ __forceinline__ uint32_t event_of(const uint32_t* ev_off, uint32_t n_events,
                                             uint32_t i) {
    uint32_t lo = 0, hi = n_events;  // invariant: ev_off[lo] <= i < ev_off[hi]
    while (hi - lo > 1) {
        const uint32_t mid = (lo + hi) >> 1;
        if (ev_off[mid] <= i)
            lo = mid;
        else
            hi = mid;
    }
    return lo;
}

// A value every lane of the wave holds identically, moved to scalar
// registers (the compiler cannot prove uniformity after a shuffle reduction).
__device__ __forceinline__ double uniform(double v) {
    const uint64_t b = (uint64_t)__double_as_longlong(v);
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)b);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(b >> 32));
    return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}

__device__ __forceinline__ float uniform(float v) {
    return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(v)));
}

typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// Brackets a run of transcendental instructions (see diff_group).
__device__ __forceinline__ void transcendental_begin() {
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_setprio(3);
}
__device__ __forceinline__ void transcendental_end() {
    __builtin_amdgcn_s_setprio(0);
    __builtin_amdgcn_sched_barrier(0);
}

// f as three bf16 values h, m, l, each the rest rounded to nearest: 8 + 8 + 8
// bits hold the 24 of an FP32 value exactly.  Pairs as a matrix operand takes
// them (first in the low half).
struct Bf16x3 {
    uint32_t hh, hm, ml;
};
__device__ __forceinline__ uint32_t pack_bf16(float a, float b) {
    return __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2{a, b}), bf16x2));
}
__device__ __forceinline__ Bf16x3 split_bf16(float f) {
    Bf16x3 p;
    p.hh = pack_bf16(f, f);
    const float r = f - __uint_as_float(p.hh & 0xFFFF0000u);
    p.hm = pack_bf16(f, r);
    p.ml = pack_bf16(r, r - __uint_as_float(p.hm & 0xFFFF0000u));
    return p;
}

__device__ __forceinline__ double wave_min(double v) {
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) v = fmin(v, __shfl_xor(v, m));
    return v;
}

__device__ __forceinline__ double wave_max(double v) {
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) v = fmax(v, __shfl_xor(v, m));
    return v;
}

// Pairs closer than kExactRadius softening lengths are summed exactly.  The
// pair loop only records them (exact_push: the target's index in the item's
// block and the source's slot in its event, in an LDS list of the work item)
// and drops their FP32 terms; at the end of the item exact_flush forms each
// recorded term in FP64 from the FP64 positions, as Eq. (6) defines it, and
// adds it in fixed point to the target's slot of the close sums.  Integer
// addition is associative, so the sums do not depend on the order in which
// work items finish.  Keeping the FP64 work out of the pair loop keeps its
// registers (and the kernel's occupancy) as they are.  A pair that finds the
// list full keeps its FP32 term.
constexpr int kExactCap = 512;

struct ExactList {
    uint32_t n;
    uint32_t tgt[kExactCap];
    uint32_t src[kExactCap];
};

__device__ __forceinline__ bool exact_push(ExactList& L, uint32_t tgt, uint32_t src) {
    const uint32_t i = atomicAdd(&L.n, 1u);
    if (i >= (uint32_t)kExactCap) return false;
    L.tgt[i] = tgt;
    L.src[i] = src;
    return true;
}

// The term of source slot s at target slot t, in FP64, to the close sums.
__device__ __forceinline__ void exact_add(const FieldArgs& a, uint32_t t, uint32_t s) {
    const double dx = a.px[t] - a.px[s], dy = a.py[t] - a.py[s], dz = a.pz[t] - a.pz[s];
    double q = fma(dx, dx, a.eps2d);
    q = fma(dy, dy, q);
    q = fma(dz, dz, q);
    const double w = a.acc_scale / (q * sqrt(q));
    unsigned long long* c = a.close + t;
    atomicAdd(c, (unsigned long long)__double2ll_rn(dx * w));
    atomicAdd(c + a.pstride, (unsigned long long)__double2ll_rn(dy * w));
    atomicAdd(c + 2 * (size_t)a.pstride, (unsigned long long)__double2ll_rn(dz * w));
}

// The matrix kernel keeps one list per wave, filled without atomics: the
// wave counts its entries in a scalar register and each lane finds its place
// from the ballot.  (In the dense core of a cloud two of five turns of the
// near loop record a pair, and the atomic's round trip through LDS stalled
// the wave each time.)  The four lists hold as many pairs as ExactList.  Lists that
// fill (a large softening: its radius holds many pairs) cost their FP64 terms and
// atomics: 10,007 holes at a softening of 0.1 um 136 us per step with 128 entries,
// 177 with 256, 268 with 512 (173 with the one ExactList per workgroup that the
// kernel before had); 1e5 holes 4.55, 4.62, 4.89 ms (4.73).  At 1 nm no list fills
// outside clumps far denser than a fresh cloud.
constexpr int kWaveCap = kExactCap / (kFieldThreads / 64);

struct WaveList {
    uint32_t src[kWaveCap];
    uint8_t tgt[kWaveCap];  // target's index in the item's block
};

// Called by every lane of the workgroup after the item's last barrier;
// targets of the item are slots off + tbase + tgt, sources slots off + src.
// Leaves the list empty for the next item (whose first barrier orders the
// clearing before any push).
__device__ __forceinline__ void exact_flush(const FieldArgs& a, ExactList& L, uint32_t off,
                                            uint32_t tbase) {
    const uint32_t cnt = min(L.n, (uint32_t)kExactCap);
    if (cnt == 0) return;  // uniform: every lane reads L.n after the same barrier
    for (uint32_t i = threadIdx.x; i < cnt; i += blockDim.x)
        exact_add(a, off + tbase + L.tgt[i], off + L.src[i]);
    __syncthreads();
    if (threadIdx.x == 0) L.n = 0;
}

// ---------------------------------------------------------------------------
// Eq. (6):  E_j = K sum_i r_ij / (|r_ij|^2 + eps^2)^{3/2},  r_ij = r_j - r_i,
// summed over the sources of the target's own event.
//
// One workgroup takes one work item: kFieldThreads*TPT consecutive target
// slots of one event's spatially sorted segment (a compact region of the
// cloud) and one chunk of that event's source tiles, dealt round-robin
// (first, first + S, ... below the item's end).  Sources are staged
// through LDS in tiles of kTile (double buffered: the next tile's global
// loads are in flight while the current one is consumed); every lane of
// every wave reads the same LDS words, so the reads are bank-conflict-free
// broadcasts.  Each lane keeps TPT targets in registers.
//
// Precision.  The workgroup takes the centre o of its targets' bounding box
// (half-diagonal rho) as origin and holds every coordinate, targets and
// staged sources alike, as the FP32 pair hi = fl32(x - o), lo = fl32(x - o -
// hi).  A pair difference d is first formed from the hi parts alone; its
// error is at most 2u (rho + |d|), and since the Jacobian of d/|d|^3 has norm
// 2/|d|^3 the term's relative error is at most 4u (1 + |t - o|/|d|) <= 4u (1 +
// rho/|d|).  Pairs closer than a quarter of the target's distance |t - o|
// from the origin -- rare, found with one compare per pair, or ruled out for
// a whole source tile whose bounding box is rho/4 or more from the targets'
// box -- are recomputed with the lo parts added, which makes their
// difference accurate to about u |d|.
// Every term therefore carries at most 20u (1.2e-6) relative error from the
// coordinates, plus about 8u from r^2, the hardware reciprocal square root
// (cubed for r^-3) and the products, so each carrier's field is within about
// 2e-6 of the sum of its term magnitudes plus the FP32 summation error.
// Each tile's contributions are summed separately and then added to the
// running sum (blocked summation).
//
// Pairs closer than kExactRadius eps (64 nm at eps = 1 nm) are the one case
// where that relative bound is not enough: their terms reach 0.385 / eps^2,
// tens to hundreds of times the rms field of a cloud, and an FP32 term and the
// FP32 additions that follow it would carry about 10u of that into the
// target's field.  They are summed exactly instead (exact_push): the close-pair
// radius is at least that distance, so these pairs always take the checked
// path, and tiles that can hold them are never summed unchecked.
//
// The other GCCD_PRECISION_* modes change the origin (one per event, or
// none: absolute coordinates) or the difference formation (hi parts only,
// or hi and lo for every pair); they exist to measure those choices.
// ---------------------------------------------------------------------------
// How the difference of a pair is formed from the FP32 parts hi, lo of the
// origin-relative coordinates.
enum : int {
    kDiffHi = 0,    // hi parts only
    kDiffNear = 1,  // hi parts; pairs closer than rc recomputed with the lo parts added
    kDiffAll = 2    // hi and lo parts for every pair (double-single differences)
};

// The terms of G sources (k .. k + G - 1 of the staged tile; their parts in
// elements u .. u + G - 1 of h and l) with the lane's TPT targets.  The reciprocal square roots of the G * TPT pairs stand together at
// raised wave priority: a compute unit issues the full-rate FP32 instructions
// of two waves at once only while neither has a transcendental next, so single
// ones spread through the stream cost every wave that pairing (measured per
// wave and source, plain differences: 45 cycles spread, 41 grouped by four).
// The sums keep the order of the sources.
//
// CUT: the term counts only when r^2 + eps^2 < cut2 (the near part of a
// near/far split); 2 more VALU per pair.  EXACT (with kDiffNear): pairs with
// r^2 + eps^2 below ap->acc2 are recorded in *xl (target t of the lane is
// tgt0 + t * kFieldThreads of the item's block, source k is src0 + k of the
// event).
template <int TPT, int DIFF, bool CUT, bool EXACT, int G>
__device__ __forceinline__ void pair_terms(
    const f32x4 (&h)[3], const f32x4 (&l)[3], int u, const float* __restrict__ lxp,
    const float* __restrict__ lyp, const float* __restrict__ lzp, uint32_t k,
    const float (&thx)[TPT], const float (&thy)[TPT], const float (&thz)[TPT],
    const float (&tlx)[TPT], const float (&tly)[TPT], const float (&tlz)[TPT], float eps2,
    const float (&rc2)[TPT], float (&ax)[TPT], float (&ay)[TPT], float (&az)[TPT], float cut2,
    const FieldArgs* ap, ExactList* xl, uint32_t tgt0, uint32_t src0) {
    float dx[G][TPT], dy[G][TPT], dz[G][TPT], r2[G][TPT], inv[G][TPT];
#pragma unroll
    for (int g = 0; g < G; ++g) {
        const float shx = h[0][u + g], shy = h[1][u + g], shz = h[2][u + g];
        bool near = false;
#pragma unroll
        for (int t = 0; t < TPT; ++t) {
            dx[g][t] = thx[t] - shx;
            dy[g][t] = thy[t] - shy;
            dz[g][t] = thz[t] - shz;
            if (DIFF == kDiffAll) {
                dx[g][t] += tlx[t] - l[0][u + g];
                dy[g][t] += tly[t] - l[1][u + g];
                dz[g][t] += tlz[t] - l[2][u + g];
            }
            r2[g][t] = __builtin_fmaf(dx[g][t], dx[g][t], eps2);
            r2[g][t] = __builtin_fmaf(dy[g][t], dy[g][t], r2[g][t]);
            r2[g][t] = __builtin_fmaf(dz[g][t], dz[g][t], r2[g][t]);
            if (DIFF == kDiffNear) near |= r2[g][t] < rc2[t];
        }
        if (DIFF == kDiffNear && __builtin_expect(__ballot(near) != 0ull, 0)) {
            // wave-uniform branch, taken only when some lane of the wave has a
            // close pair: add the lo parts to the differences of those pairs
            const float nlx = lxp[k + g], nly = lyp[k + g], nlz = lzp[k + g];
#pragma unroll
            for (int t = 0; t < TPT; ++t) {
                if (r2[g][t] < rc2[t]) {
                    dx[g][t] += tlx[t] - nlx;
                    dy[g][t] += tly[t] - nly;
                    dz[g][t] += tlz[t] - nlz;
                    r2[g][t] = __builtin_fmaf(dx[g][t], dx[g][t], eps2);
                    r2[g][t] = __builtin_fmaf(dy[g][t], dy[g][t], r2[g][t]);
                    r2[g][t] = __builtin_fmaf(dz[g][t], dz[g][t], r2[g][t]);
                }
            }
            if (EXACT) {
                // rc2 is at least acc2 for a target and 0 for a padding slot; a
                // pair at distance 0 has a zero term and stays in the FP32 sum
#pragma unroll
                for (int t = 0; t < TPT; ++t) {
                    if (r2[g][t] < fminf(ap->acc2, rc2[t]) && r2[g][t] > eps2 &&
                        exact_push(*xl, tgt0 + (uint32_t)(t * kFieldThreads), src0 + k + g))
                        dx[g][t] = dy[g][t] = dz[g][t] = 0.0f;
                }
            }
        }
    }
    transcendental_begin();
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
        for (int t = 0; t < TPT; ++t) inv[g][t] = __builtin_amdgcn_rsqf(r2[g][t]);
    transcendental_end();
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
        for (int t = 0; t < TPT; ++t) {
            // r^-3 as rsq^3: one transcendental and two multiplies measured
            // faster on gfx950 than rsq * rcp (two transcendentals, one multiply)
            float w = inv[g][t] * inv[g][t] * inv[g][t];
            if (CUT) w = r2[g][t] < cut2 ? w : 0.0f;
            ax[t] = __builtin_fmaf(dx[g][t], w, ax[t]);
            ay[t] = __builtin_fmaf(dy[g][t], w, ay[t]);
            az[t] = __builtin_fmaf(dz[g][t], w, az[t]);
        }
}

// All pairs of one staged tile (cnt sources) with the lane's TPT targets.
template <int TPT, int DIFF, bool CUT = false, bool EXACT = false>
__device__ __forceinline__ void tile_terms(
    const float* __restrict__ hxp, const float* __restrict__ hyp, const float* __restrict__ hzp,
    const float* __restrict__ lxp, const float* __restrict__ lyp, const float* __restrict__ lzp,
    uint32_t cnt, const float (&thx)[TPT], const float (&thy)[TPT], const float (&thz)[TPT],
    const float (&tlx)[TPT], const float (&tly)[TPT], const float (&tlz)[TPT], float eps2,
    const float (&rc2)[TPT], float (&bx)[TPT], float (&by)[TPT], float (&bz)[TPT],
    float cut2 = 0.0f, const FieldArgs* ap = nullptr, ExactList* xl = nullptr, uint32_t tgt0 = 0u,
    uint32_t src0 = 0u) {
    constexpr int G = 4 / TPT;  // four pairs of a lane at a time
    uint32_t k = 0;
    for (; k + 4 <= cnt; k += 4) {
        const f32x4 h[3] = {*reinterpret_cast<const f32x4*>(hxp + k),
                            *reinterpret_cast<const f32x4*>(hyp + k),
                            *reinterpret_cast<const f32x4*>(hzp + k)};
        f32x4 l[3] = {};
        if (DIFF == kDiffAll) {
            l[0] = *reinterpret_cast<const f32x4*>(lxp + k);
            l[1] = *reinterpret_cast<const f32x4*>(lyp + k);
            l[2] = *reinterpret_cast<const f32x4*>(lzp + k);
        }
#pragma unroll
        for (int u = 0; u < 4; u += G)
            pair_terms<TPT, DIFF, CUT, EXACT, G>(h, l, u, lxp, lyp, lzp, k + u, thx, thy, thz, tlx,
                                                 tly, tlz, eps2, rc2, bx, by, bz, cut2, ap, xl,
                                                 tgt0, src0);
    }
    for (; k < cnt; ++k) {
        const f32x4 h[3] = {{hxp[k]}, {hyp[k]}, {hzp[k]}}, l[3] = {{lxp[k]}, {lyp[k]}, {lzp[k]}};
        pair_terms<TPT, DIFF, CUT, EXACT, 1>(h, l, 0, lxp, lyp, lzp, k, thx, thy, thz, tlx, tly,
                                             tlz, eps2, rc2, bx, by, bz, cut2, ap, xl, tgt0, src0);
    }
}

template <int TPT, int PREC>
__global__ __launch_bounds__(kFieldThreads) void field_tiles(FieldArgs a) {
    __shared__ __align__(16) float sh[2][6][kTile];
    __shared__ double box[6][kFieldThreads / 64];
    __shared__ double ebox[6][kFieldThreads / 64];  // EVENT mode: the event's source box
    __shared__ double tbox[2][6];  // bounding box of the staged source tile
    __shared__ ExactList xl;       // default precision: close pairs of the item

    const FieldItem it = a.items[blockIdx.x];
    const uint32_t off = a.ev_off[it.event];
    const uint32_t ne = a.ev_off[it.event + 1] - off;
    const uint32_t na = a.ev_active[it.event];
    const uint32_t nt = a.targets_all ? ne : na;
    const uint32_t ns = a.sources_all ? ne : na;
    const uint32_t tbase = it.blk * (uint32_t)(kFieldThreads * TPT);
    if (tbase >= nt) return;  // the whole workgroup leaves before any barrier

    // The item takes the event's source tiles first, first + S, first + 2S,
    // ... below its end.  Each tile is a compact region (the segment is
    // spatially sorted) whose bounding box is precomputed; dealing them
    // round-robin gives every chunk a sample of the whole cloud, so the
    // close pairs -- the costlier ones -- spread evenly over the workgroups.
    const uint32_t ntiles = (ns + kTile - 1) / kTile;
    const uint32_t tile0 = a.ev_tile[it.event];
    const uint32_t chunk = it.group;  // partial-sum group written
    const uint32_t step_t = it.step;
    const uint32_t t_first = it.first;
    const uint32_t t_end = min(it.end, ntiles);
    const int tid = threadIdx.x;
    if (tid == 0) xl.n = 0;  // ordered before any push by the barrier below

    // targets and their bounding box
    double px[TPT], py[TPT], pz[TPT];
    double lo_x = INFINITY, lo_y = INFINITY, lo_z = INFINITY;
    double hi_x = -INFINITY, hi_y = -INFINITY, hi_z = -INFINITY;
#pragma unroll
    for (int t = 0; t < TPT; ++t) {
        const uint32_t ts = tbase + (uint32_t)(t * kFieldThreads + tid);
        px[t] = py[t] = pz[t] = 0.0;
        if (ts < nt) {
            px[t] = a.px[off + ts];
            py[t] = a.py[off + ts];
            pz[t] = a.pz[off + ts];
            lo_x = fmin(lo_x, px[t]);
            lo_y = fmin(lo_y, py[t]);
            lo_z = fmin(lo_z, pz[t]);
            hi_x = fmax(hi_x, px[t]);
            hi_y = fmax(hi_y, py[t]);
            hi_z = fmax(hi_z, pz[t]);
        }
    }
    {
        const int wave = tid >> 6, lane = tid & 63;
        lo_x = wave_min(lo_x);
        lo_y = wave_min(lo_y);
        lo_z = wave_min(lo_z);
        hi_x = wave_max(hi_x);
        hi_y = wave_max(hi_y);
        hi_z = wave_max(hi_z);
        if (lane == 0) {
            box[0][wave] = lo_x;
            box[1][wave] = lo_y;
            box[2][wave] = lo_z;
            box[3][wave] = hi_x;
            box[4][wave] = hi_y;
            box[5][wave] = hi_z;
        }
    }
    __syncthreads();
#pragma unroll
    for (int w = 0; w < kFieldThreads / 64; ++w) {
        lo_x = fmin(lo_x, box[0][w]);
        lo_y = fmin(lo_y, box[1][w]);
        lo_z = fmin(lo_z, box[2][w]);
        hi_x = fmax(hi_x, box[3][w]);
        hi_y = fmax(hi_y, box[4][w]);
        hi_z = fmax(hi_z, box[5][w]);
    }
    lo_x = uniform(lo_x);
    lo_y = uniform(lo_y);
    lo_z = uniform(lo_z);
    hi_x = uniform(hi_x);
    hi_y = uniform(hi_y);
    hi_z = uniform(hi_z);
    // Every lane now holds the same box.  A box of non-finite positions
    // gives a NaN origin; the field is then NaN, and the step kernel flags it.
    double ox = 0.5 * (lo_x + hi_x), oy = 0.5 * (lo_y + hi_y), oz = 0.5 * (lo_z + hi_z);
    if (PREC == GCCD_PRECISION_ABSOLUTE) {
        ox = oy = oz = 0.0;
    } else if (PREC == GCCD_PRECISION_EVENT) {
        // centre of the union of the event's source-tile boxes
        double e[6] = {INFINITY, INFINITY, INFINITY, -INFINITY, -INFINITY, -INFINITY};
        for (uint32_t t = (uint32_t)tid; t < ntiles; t += kFieldThreads) {
            const size_t g = (size_t)tile0 + t;
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                e[d] = fmin(e[d], a.tile_box[(size_t)d * a.tile_stride + g]);
                e[d + 3] = fmax(e[d + 3], a.tile_box[(size_t)(d + 3) * a.tile_stride + g]);
            }
        }
        const int wave = tid >> 6;
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            e[d] = wave_min(e[d]);
            e[d + 3] = wave_max(e[d + 3]);
        }
        if ((tid & 63) == 0) {
#pragma unroll
            for (int d = 0; d < 6; ++d) ebox[d][wave] = e[d];
        }
        __syncthreads();
#pragma unroll
        for (int w = 0; w < kFieldThreads / 64; ++w) {
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                e[d] = fmin(e[d], ebox[d][w]);
                e[d + 3] = fmax(e[d + 3], ebox[d + 3][w]);
            }
        }
        ox = uniform(0.5 * (e[0] + e[3]));
        oy = uniform(0.5 * (e[1] + e[4]));
        oz = uniform(0.5 * (e[2] + e[5]));
    }
    const double hx = 0.5 * (hi_x - lo_x), hy = 0.5 * (hi_y - lo_y), hz = 0.5 * (hi_z - lo_z);
    const double rc2d = 0.0625 * (hx * hx + hy * hy + hz * hz);  // (rho / 4)^2

    // rc2[t]: the close-pair radius squared of target t, a quarter of its own
    // distance from the origin (the error bound 4u (1 + |t - o| / |d|) holds
    // for every target; a lane-wise radius takes the branch less often than
    // the workgroup's rho / 4); 0 for slots past the last target
    float thx[TPT], thy[TPT], thz[TPT], tlx[TPT], tly[TPT], tlz[TPT], rc2[TPT];
    float ax[TPT], ay[TPT], az[TPT];
#pragma unroll
    for (int t = 0; t < TPT; ++t) {
        const double rx = px[t] - ox, ry = py[t] - oy, rz = pz[t] - oz;
        thx[t] = (float)rx;
        thy[t] = (float)ry;
        thz[t] = (float)rz;
        tlx[t] = (float)(rx - (double)thx[t]);
        tly[t] = (float)(ry - (double)thy[t]);
        tlz[t] = (float)(rz - (double)thz[t]);
        const uint32_t ts = tbase + (uint32_t)(t * kFieldThreads + tid);
        rc2[t] = ts < nt ? 0.0625f * (float)((double)thx[t] * thx[t] + (double)thy[t] * thy[t] +
                                             (double)thz[t] * thz[t])
                         : 0.0f;
        if (PREC == GCCD_PRECISION_DEFAULT && ts < nt) rc2[t] = fmaxf(rc2[t], a.acc2);
        ax[t] = 0.0f;
        ay[t] = 0.0f;
        az[t] = 0.0f;
    }

    double qx = 0.0, qy = 0.0, qz = 0.0;  // this lane's source of the next tile
    double qb = 0.0;                      // lanes 0-5: one bound of that tile's box
    auto fetch = [&](uint32_t t) {
        const uint32_t i = t * kTile + (uint32_t)tid;
        qx = ox;
        qy = oy;
        qz = oz;
        if (i < ns) {
            qx = a.px[off + i];
            qy = a.py[off + i];
            qz = a.pz[off + i];
        }
        if (tid < 6) qb = a.tile_box[(size_t)tid * a.tile_stride + tile0 + t];
    };
    auto stage = [&](int b) {
        if (tid < 6) tbox[b][tid] = qb;
        const double rx = qx - ox, ry = qy - oy, rz = qz - oz;
        const float fx = (float)rx, fy = (float)ry, fz = (float)rz;
        sh[b][0][tid] = fx;
        sh[b][1][tid] = fy;
        sh[b][2][tid] = fz;
        sh[b][3][tid] = (float)(rx - (double)fx);
        sh[b][4][tid] = (float)(ry - (double)fy);
        sh[b][5][tid] = (float)(rz - (double)fz);
    };

    int buf = 0;
    if (t_first < t_end) {
        fetch(t_first);
        stage(0);
    }
    __syncthreads();
    for (uint32_t t = t_first; t < t_end; t += step_t) {
        const uint32_t next = t + step_t;
        if (next < t_end) fetch(next);
        const uint32_t cnt = min((uint32_t)kTile, ns - t * kTile);

        float bx[TPT], by[TPT], bz[TPT];
#pragma unroll
        for (int u = 0; u < TPT; ++u) bx[u] = by[u] = bz[u] = 0.0f;

        const float* hxp = sh[buf][0];
        const float* hyp = sh[buf][1];
        const float* hzp = sh[buf][2];
        const float* lxp = sh[buf][3];
        const float* lyp = sh[buf][4];
        const float* lzp = sh[buf][5];
        // A tile whose bounding box is at least rho/4 from the targets' box
        // cannot hold a close pair: its pairs skip the per-pair check.
        const double* tb = tbox[buf];
        const double gx = fmax(0.0, fmax(tb[0] - hi_x, lo_x - tb[3]));
        const double gy = fmax(0.0, fmax(tb[1] - hi_y, lo_y - tb[4]));
        const double gz = fmax(0.0, fmax(tb[2] - hi_z, lo_z - tb[5]));
        const bool far_tile = gx * gx + gy * gy + gz * gz >= fmax(rc2d, a.acc_box2);
        if (PREC == GCCD_PRECISION_COMPENSATED) {
            tile_terms<TPT, kDiffAll>(hxp, hyp, hzp, lxp, lyp, lzp, cnt, thx, thy, thz, tlx, tly,
                                      tlz, a.eps2, rc2, bx, by, bz);
        } else if (PREC != GCCD_PRECISION_DEFAULT || far_tile) {
            tile_terms<TPT, kDiffHi>(hxp, hyp, hzp, lxp, lyp, lzp, cnt, thx, thy, thz, tlx, tly,
                                     tlz, a.eps2, rc2, bx, by, bz);
        } else {
            tile_terms<TPT, kDiffNear, false, true>(hxp, hyp, hzp, lxp, lyp, lzp, cnt, thx, thy,
                                                    thz, tlx, tly, tlz, a.eps2, rc2, bx, by, bz,
                                                    0.0f, &a, &xl, (uint32_t)tid, t * kTile);
        }
#pragma unroll
        for (int u = 0; u < TPT; ++u) {
            ax[u] += bx[u];
            ay[u] += by[u];
            az[u] += bz[u];
        }
        if (next < t_end) stage(buf ^ 1);
        __syncthreads();
        buf ^= 1;
    }

    if (PREC == GCCD_PRECISION_DEFAULT) exact_flush(a, xl, off, tbase);
    float* outx = a.part + (size_t)(chunk * 3 + 0) * a.pstride + off;
    float* outy = a.part + (size_t)(chunk * 3 + 1) * a.pstride + off;
    float* outz = a.part + (size_t)(chunk * 3 + 2) * a.pstride + off;
#pragma unroll
    for (int t = 0; t < TPT; ++t) {
        const uint32_t ts = tbase + (uint32_t)(t * kFieldThreads + tid);
        if (ts < nt) {
            outx[ts] = ax[t];
            outy[ts] = ay[t];
            outz[ts] = az[t];
        }
    }
}

// The cutoff r^2 + eps^2 < cut2 of the near sum as factors of 0 or 1 (see
// diff_quad), on r^2 and on its reciprocal square root.
struct CutoffTest {
    float big_r2 = 0.0f, lim_r2 = 0.0f;    // clamp(lim_r2 - big_r2 r^2)
    float big_inv = 0.0f, lim_inv = 0.0f;  // clamp(big_inv / r - lim_inv)
};

__device__ __forceinline__ float clamp01(float v) { return __builtin_amdgcn_fmed3f(v, 0.0f, 1.0f); }

// One source quadruple of a near (COMP: hi and lo parts) or plain (hi parts) block
// in the difference form: sources k .. k + 3 of the staged tile (sources src ..
// src + 3 of the event) at the lane's target, number tgt of the block.  The four reciprocal square
// roots stand together at raised wave priority: a compute unit issues the
// full-rate FP32 instructions of two waves at once only while neither has a
// transcendental next, so single ones spread through the stream cost every wave
// that pairing (measured, far pairs: 40.3 cycles per wave and source spread,
// 37.5 grouped by four at raised priority).  COMP: one compare with the smallest
// of the four r^2 rules out pairs below acc2 (a compare issues at half rate),
// which are recorded for exact summation.  e2 is the softening and rx the
// exact-sum limit (0 for a lane without a target) in vector registers (an
// instruction with a scalar operand does not pair either).
// CUT: the term counts only while r^2 < cut2, as a factor clamp(big (cut2 -
// r^2)) of 0 or 1 (big: a power of two that makes one unit in the last place
// exceed 1); no pair is recorded.  Two full-rate instructions where compare and
// select are two half-rate ones.
template <bool CUT, bool COMP>
__device__ __forceinline__ void diff_quad(WaveList& xl, uint32_t& nx, uint32_t tgt, uint32_t src,
                                          const float (&hl)[6][kTile], uint32_t k, float thx,
                                          float thy, float thz, float tlx, float tly, float tlz,
                                          float e2, float rx, const CutoffTest& ct, float& bx, float& by,
                                          float& bz) {
    const f32x4 x4 = *reinterpret_cast<const f32x4*>(&hl[0][k]);
    const f32x4 y4 = *reinterpret_cast<const f32x4*>(&hl[1][k]);
    const f32x4 z4 = *reinterpret_cast<const f32x4*>(&hl[2][k]);
    f32x4 a4, b4, c4;
    if constexpr (COMP) {
        a4 = *reinterpret_cast<const f32x4*>(&hl[3][k]);
        b4 = *reinterpret_cast<const f32x4*>(&hl[4][k]);
        c4 = *reinterpret_cast<const f32x4*>(&hl[5][k]);
    }
    float dx[4], dy[4], dz[4], r2[4], inv[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        // thx + 0.5 (-2 s_x) rounds once, to the same value as thx - s_x
        dx[u] = __builtin_fmaf(x4[u], 0.5f, thx);
        dy[u] = __builtin_fmaf(y4[u], 0.5f, thy);
        dz[u] = __builtin_fmaf(z4[u], 0.5f, thz);
        if constexpr (COMP) {
            dx[u] += tlx - a4[u];
            dy[u] += tly - b4[u];
            dz[u] += tlz - c4[u];
        }
        r2[u] = __builtin_fmaf(dx[u], dx[u], e2);
        r2[u] = __builtin_fmaf(dy[u], dy[u], r2[u]);
        r2[u] = __builtin_fmaf(dz[u], dz[u], r2[u]);
    }
    if constexpr (COMP && !CUT) {
        const float m = fminf(fminf(r2[0], r2[1]), fminf(r2[2], r2[3]));
        if (__builtin_expect(__ballot(m < rx) != 0ull, 0)) {
    #pragma unroll
            for (int u = 0; u < 4; ++u) {
                const bool rec = r2[u] < rx && r2[u] > e2;
                const uint64_t who = __ballot(rec);
                if (who) {
                    const uint32_t i =
                        nx + __builtin_amdgcn_mbcnt_hi((uint32_t)(who >> 32),
                                                       __builtin_amdgcn_mbcnt_lo((uint32_t)who, 0u));
                    if (rec && i < (uint32_t)kWaveCap) {
                        xl.src[i] = src + (uint32_t)u;
                        xl.tgt[i] = (uint8_t)tgt;
                        dx[u] = dy[u] = dz[u] = 0.0f;
                    }
                    nx = min(nx + (uint32_t)__popcll(who), (uint32_t)kWaveCap);
                }
            }
        }
    }
    transcendental_begin();
#pragma unroll
    for (int u = 0; u < 4; ++u) inv[u] = __builtin_amdgcn_rsqf(r2[u]);
    transcendental_end();
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        float w = inv[u] * inv[u] * inv[u];
        if constexpr (CUT) w *= clamp01(__builtin_fmaf(r2[u], -ct.big_r2, ct.lim_r2));
        bx = __builtin_fmaf(dx[u], w, bx);
        by = __builtin_fmaf(dy[u], w, by);
        bz = __builtin_fmaf(dz[u], w, bz);
    }
}

// Default precision, one target per lane.  The wave's 64 targets are four groups
// of 16 (as the matrix cores take them), a source tile up to 16 groups of 16,
// and each of the 64 pairs of groups is summed in one of three forms, chosen by
// the gap between the groups' bounding boxes (rho: the half-diagonal of the
// workgroup's targets, whose centre is the origin; u = 2^-24):
//
// Far (gap above kFarFraction rho = 4/7 rho):
//     r^2 = (|s|^2 + eps^2) + |t|^2 - 2 t.s    on the matrix cores,
//     sum d w = t sum w - sum s w,             w = (r^2)^{-3/2},
// with s and t the hi parts.  One v_mfma_f32_16x16x32_bf16 gives r^2 of a
// block, which leaves 6 VALU instructions and the reciprocal square root per
// pair.  Every FP32 factor is held as three bf16 parts (exactly its 24 bits);
// the products of parts are exact and accumulated in FP32, and those of order
// 2^-27 (second with third part and below) are left out.  The error of r^2 is at
// most 2.1 u (|s| + |t|)^2, the largest of 1e7 random pairs at gaps of 0.15 to 5
// rho with |t| = rho (rms 0.34; four FP32 operations on the vector units 2.9 and
// 0.34 to 0.63), and (|s| + |t|) / |d| is at most 2/f + 1 = 4.5 at a gap of f rho
// = 4/7 rho: 64 u per term, with 11 u of the dropped lo parts, 4 u (1 + 1/f), and 8 u
// of r^-3 and the products 83 u.  (At f = 1/5 the same sum is 413 u, and single
// terms at the very edge were off by up to 1.04e-5; now 1.9e-6.)  t sum w - sum s w is
// formed per tile in FP64 from the tile's FP32 sums, and the tiles add up in FP64
// (launches level with FP32 there; rms error of the field at 1e5 holes 3.2e-8 ->
// 2.8e-8 of its rms, at 3e5 2.6e-8 -> 2.1e-8).
//
// Plain (gap above kPlainFraction rho = rho/4): the difference of the hi parts,
// 4 u (1 + 1/f) = 20 u from the coordinates.
//
// Near (all others): the compensated difference (hi and lo parts) in every
// pair, and the exact sum for pairs within kExactRadius eps.  No pair needs a
// test against a close-pair radius, so the loop has no branch that a dense cloud
// takes.
//
// Shares of near and plain pairs: 0.008 and 0.019 of a 1e5-hole cloud, 0.05 and
// 0.10 of 2e4, 0.09 and 0.18 of 1e4, 0.69 and 0.29 of 1000.  us per step with the
// far limit at rho/5, with it at 4 rho/7 and everything within near, and as it is:
// 1e5 holes 2032, 2124, 2083; 3e5 17487, 17952, 17653; 2e4 141, 157, 148; 400 clouds
// of 200-20000 holes 4291, 5185, 4772; the 62354-hole track 808, 814, 814.  (Far
// where |s| + |t| of the two groups' boxes is within 4.5 gaps, at any rho: level, the
// track 3 % slower.)  Largest error of a hole, in sums of its term magnitudes, and
// rms error in rms fields: 5.4e-8 and 2.5e-8 at 1e5 holes, 5.9e-8 and 3.7e-8 at 2e4,
// 1.5e-7 and 5.8e-8 on the track, 1.6e-7 and 3.4e-8 on 40 clouds; a VALU kernel that
// took r^2 as four FP32 operations per pair in tiles beyond rho and checked
// differences within: 8.0e-8 and 7.2e-8, 1.1e-7 and 1.1e-7, 1.5e-6 and 2.0e-7, 6.6e-7
// and 9.5e-8.
//
// What bounds it: VALU issue.  The far loop runs at 24.7 cycles per wave and
// source (2.4 GHz; its launch run twice over the same groups, minus once), of
// which the reciprocal square root takes 8.1 and six full-rate instructions
// 14.4; the matrix instructions run beside the transcendentals.  The VALU form
// of the same pair took 40.  The rest of a launch is staging, classification and
// the barrier of each tile.
//
// The 32 products of the contraction: eight for each of the lanes' four
// quarters q (A: source lane % 16, B: target lane % 16):
//   q = 0, 1, 2:  -2 s_q as (h, m, m, l, h, h)  with  t_q as (h, h, m, h, m, l)
//   q = 3:        |s|^2 + eps^2 the same way    with  (1, 1, 0, 1, 0, 0)
// and 1, 1 with |t|^2's parts (h, m in q = 0, l in q = 1).  A lane's A operand
// takes eight bytes of LDS; D holds sources 4 q .. 4 q + 3 of target lane % 16,
// so a lane sums four sources of each of four targets, and the quarters' sums are
// added after each tile (blocked summation).
//
// Four waves per SIMD: 128 registers hold four groups' operands, r^2 and sums.
// Two groups at a time in 96 registers (five waves) spill and measured 8 %
// slower at 3e5 holes.
constexpr double kFarFraction = 4.0 / 7.0;
constexpr double kPlainFraction = 0.25;
// A padding source: its r^-3 underflows to 0 in either form.
constexpr float kPadS = 3.0e38f;  // |s|^2
constexpr float kPadX = 2.0e19f;  // -2 s_x of the difference form

struct MatrixLds {
    struct Tile {
        float hl[6][kTile];           // -2 s_x, -2 s_y, -2 s_z, lo_x, lo_y, lo_z
        u32x2 pk[kTile / 16][4][16];  // bf16 parts (h, m), (m, l): [group][quarter][source]
        float gbox[6][16];            // boxes of the 16-source groups, relative to the origin
    } tile[2];
    double box[6][kFieldThreads / 16];
    union {
        WaveList xl[kFieldThreads / 64];  // close pairs of the item
        uint32_t list[1024];              // CUT: groups (tile * 16 + group) to be staged
    };
};

// The sum of v over the lanes of one column (lane % 16), in each of them.
__device__ __forceinline__ float add_quarters(float v) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false,
                                                    false);
    const float h = __uint_as_float(r[0]) + __uint_as_float(r[1]);
    const auto s = __builtin_amdgcn_permlane16_swap(__float_as_uint(h), __float_as_uint(h), false,
                                                    false);
    return __uint_as_float(s[0]) + __uint_as_float(s[1]);
}

// CUT: the near part of the closure's split, the sum over the sources closer
// than a only (r^2 + eps^2 < a^2 + eps^2, gp).  Of the item's tiles, 64 tested at
// a time, the 16-source groups within a of the workgroup's targets are listed,
// and sixteen of them at a time are staged as one tile: the boundary of the
// a-ball cuts through most tiles, and staging whole ones left the waves waiting
// for whichever had most of a tile within reach.  Of the staged tile's blocks those whose boxes
// come within a are summed; far source groups that lie within a as a whole for
// all four target groups skip the cutoff.  No pair is summed exactly.
template <int UNIT, bool CUT>
__device__ __forceinline__ void matrix_item(const FieldArgs& a, const FieldItem it, MatrixLds& L,
                                            uint32_t na0, const GridParams* gp = nullptr) {
    const bool one = a.one_event_n != 0u;
    const uint32_t off = one ? 0u : a.ev_off[it.event];
    const uint32_t ne = one ? a.one_event_n : a.ev_off[it.event + 1] - off;
    const uint32_t na = one ? na0 : a.ev_active[it.event];
    const uint32_t nt = a.targets_all ? ne : na;
    const uint32_t ns = a.sources_all ? ne : na;
    const uint32_t tbase = it.blk * (uint32_t)kFieldThreads;
    if (tbase >= nt) return;  // the whole workgroup leaves before any barrier
    const uint32_t ntiles = (ns + UNIT - 1) / UNIT;
    const uint32_t tile0 = one ? 0u : a.ev_tile[it.event];
    const uint32_t chunk = it.group;  // partial-sum group written
    const uint32_t step_t = it.step;
    const uint32_t t_first = it.first;
    const uint32_t t_end = min(it.end, ntiles);
    const int tid = threadIdx.x;
    const int wave = tid >> 6, lane = tid & 63;
    const int q = lane >> 4, col = lane & 15;

    const uint32_t ts = tbase + (uint32_t)tid;
    double px = 0.0, py = 0.0, pz = 0.0;
    double lo_x = INFINITY, lo_y = INFINITY, lo_z = INFINITY;
    double hi_x = -INFINITY, hi_y = -INFINITY, hi_z = -INFINITY;
    if (ts < nt) {
        px = a.px[off + ts];
        py = a.py[off + ts];
        pz = a.pz[off + ts];
    }
    // The boxes of the block's targets (origin, rho) and of this lane's group of
    // 16, from which source groups are classified.  Where every target is a
    // source, they are boxes of one source tile, which the list holds (the last
    // block's may also hold sources that are no targets); else they are reduced
    // from the positions.
    double gl_x = INFINITY, gl_y = INFINITY, gl_z = INFINITY;
    double gh_x = -INFINITY, gh_y = -INFINITY, gh_z = -INFINITY;
    if (nt <= ns) {
        const double* tb = a.tile_box + tile0 + it.blk;
        const size_t st = a.tile_stride;
        lo_x = tb[0];
        lo_y = tb[st];
        lo_z = tb[2 * st];
        hi_x = tb[3 * st];
        hi_y = tb[4 * st];
        hi_z = tb[5 * st];
        tb += (size_t)(30 + (tid >> 4)) * st;
        gl_x = tb[0];
        gl_y = tb[16 * st];
        gl_z = tb[32 * st];
        gh_x = tb[48 * st];
        gh_y = tb[64 * st];
        gh_z = tb[80 * st];
    } else {
        if (ts < nt) {
            gl_x = gh_x = px;
            gl_y = gh_y = py;
            gl_z = gh_z = pz;
        }
#pragma unroll
        for (int k = 8; k >= 1; k >>= 1) {
            gl_x = fmin(gl_x, __shfl_xor(gl_x, k));
            gl_y = fmin(gl_y, __shfl_xor(gl_y, k));
            gl_z = fmin(gl_z, __shfl_xor(gl_z, k));
            gh_x = fmax(gh_x, __shfl_xor(gh_x, k));
            gh_y = fmax(gh_y, __shfl_xor(gh_y, k));
            gh_z = fmax(gh_z, __shfl_xor(gh_z, k));
        }
        if (col == 0) {
            L.box[0][tid >> 4] = gl_x;
            L.box[1][tid >> 4] = gl_y;
            L.box[2][tid >> 4] = gl_z;
            L.box[3][tid >> 4] = gh_x;
            L.box[4][tid >> 4] = gh_y;
            L.box[5][tid >> 4] = gh_z;
        }
        __syncthreads();
        for (int w = 0; w < kFieldThreads / 16; ++w) {
            lo_x = fmin(lo_x, L.box[0][w]);
            lo_y = fmin(lo_y, L.box[1][w]);
            lo_z = fmin(lo_z, L.box[2][w]);
            hi_x = fmax(hi_x, L.box[3][w]);
            hi_y = fmax(hi_y, L.box[4][w]);
            hi_z = fmax(hi_z, L.box[5][w]);
        }
    }
    lo_x = uniform(lo_x);
    lo_y = uniform(lo_y);
    lo_z = uniform(lo_z);
    hi_x = uniform(hi_x);
    hi_y = uniform(hi_y);
    hi_z = uniform(hi_z);
    const double ox = 0.5 * (lo_x + hi_x), oy = 0.5 * (lo_y + hi_y), oz = 0.5 * (lo_z + hi_z);
    const double hx = 0.5 * (hi_x - lo_x), hy = 0.5 * (hi_y - lo_y), hz = 0.5 * (hi_z - lo_z);
    // no far or unchecked group may hold a pair closer than kExactRadius eps.  The
    // group boxes are held in FP32 relative to the origin, which puts a gap off
    // by a few 1e-7 of itself: the limits carry a margin of 1e-4.
    const double rho2 = hx * hx + hy * hy + hz * hz;
    const float far2 =
        uniform((float)(1.0001 * fmax(kFarFraction * kFarFraction * rho2, a.acc_box2)));
    const float plain2 =
        uniform((float)(1.0001 * fmax(kPlainFraction * kPlainFraction * rho2, a.acc_box2)));
    const float glx = (float)(gl_x - ox), gly = (float)(gl_y - oy), glz = (float)(gl_z - oz),
                ghx = (float)(gh_x - ox), ghy = (float)(gh_y - oy), ghz = (float)(gh_z - oz);
    const bool has_targets = (ts & ~15u) < nt;  // of this lane's group
    const double eps2d = (double)a.eps2;

    double qx = 0.0, qy = 0.0, qz = 0.0;  // this lane's source of the next tile
    double qb = 0.0;                      // lanes 0-95: one bound of one of its groups
    const double ob = (tid >> 4) % 3 == 0 ? ox : (tid >> 4) % 3 == 1 ? oy : oz;  // its origin
    bool qv = false;                      // that source exists
    uint32_t n_list = 0;                  // CUT: groups listed, in L.list
    // tile number i of the batch: the item's tile t_first + i S, or (CUT) sixteen
    // listed groups
    auto fetch = [&](uint32_t i) {
        uint32_t j, row, tile;  // source slot; lanes 0-95: box row and tile of their group
        if constexpr (CUT) {
            const uint32_t g = i * 16u + (uint32_t)(tid >> 4), gb = i * 16u + (uint32_t)col;
            const uint32_t G = L.list[min(g, n_list - 1u)], Gb = L.list[min(gb, n_list - 1u)];
            j = G * 16u + (uint32_t)col;
            qv = g < n_list && j < ns;
            row = 30u + (uint32_t)(tid & ~15) + (Gb & 15u);
            tile = Gb >> 4;
        } else {
            const uint32_t s0 = (t_first + i * step_t) * UNIT;
            j = s0 + (uint32_t)tid;
            qv = tid < UNIT && j < ns;
            // rows 30 + 16 k + g of the 256-source tile that holds the tile
            row = 30u + (uint32_t)(tid & ~15) +
                  min((uint32_t)col + ((s0 & (kTile - 1)) >> 4), 15u);
            tile = s0 / kTile;
        }
        qx = ox;
        qy = oy;
        qz = oz;
        if (qv) {
            qx = a.px[off + j];
            qy = a.py[off + j];
            qz = a.pz[off + j];
        }
        if (tid < 96) qb = a.tile_box[(size_t)row * a.tile_stride + tile0 + tile];
    };
    auto stage = [&](int b) {
        MatrixLds::Tile& S = L.tile[b];
        if (tid < 96) S.gbox[tid >> 4][tid & 15] = (float)(qb - ob);
        const double rx = qx - ox, ry = qy - oy, rz = qz - oz;
        const float fx = (float)rx, fy = (float)ry, fz = (float)rz;
        const float mx = -2.0f * fx, my = -2.0f * fy, mz = -2.0f * fz;
        S.hl[0][tid] = qv ? mx : kPadX;
        S.hl[1][tid] = my;
        S.hl[2][tid] = mz;
        S.hl[3][tid] = (float)(rx - (double)fx);
        S.hl[4][tid] = (float)(ry - (double)fy);
        S.hl[5][tid] = (float)(rz - (double)fz);
        float s2 = (float)fma((double)fx, (double)fx,
                             fma((double)fy, (double)fy, fma((double)fz, (double)fz, eps2d)));
        s2 = qv ? fminf(s2, kPadS) : kPadS;
        const float v[4] = {mx, my, mz, s2};
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const Bf16x3 p = split_bf16(v[k]);
            S.pk[tid >> 4][k][tid & 15] = u32x2{p.hm, p.ml};
        }
    };
    // CUT: lists the groups within a of the targets in the next tiles that have
    // any.  Every wave does the same work, the first one writes.
    uint32_t t_test = t_first;  // the next tile to test
    const double a2 = CUT ? uniform(gp->a2) : 0.0;
    auto gap2 = [&](const double* tb, size_t st) {  // of the targets' box and one at tb
        const double gx = fmax(0.0, fmax(tb[0] - hi_x, lo_x - tb[3 * st]));
        const double gy = fmax(0.0, fmax(tb[st] - hi_y, lo_y - tb[4 * st]));
        const double gz = fmax(0.0, fmax(tb[2 * st] - hi_z, lo_z - tb[5 * st]));
        return gx * gx + gy * gy + gz * gz;
    };
    auto list_groups = [&]() {
        n_list = 0;
        while (n_list == 0 && t_test < t_end) {
            const uint32_t t0 = t_test, m = t0 + (uint32_t)lane * step_t;
            t_test += 64u * step_t;
            uint64_t cand =
                __ballot(m < t_end && gap2(a.tile_box + tile0 + m, a.tile_stride) < a2);
            while (cand) {  // four tiles at a time, sixteen lanes each
                uint32_t t = t_end;
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const uint32_t b = cand ? t0 + (uint32_t)__builtin_ctzll(cand) * step_t : t_end;
                    cand &= cand - 1ull;
                    if (q == k) t = b;
                }
                const bool keep =
                    t < t_end && t * kTile + (uint32_t)col * 16u < ns &&
                    gap2(a.tile_box + (size_t)(30 + col) * a.tile_stride + tile0 + t,
                         16 * (size_t)a.tile_stride) < a2;
                const uint64_t who = __ballot(keep);
                const uint32_t i =
                    n_list + __builtin_amdgcn_mbcnt_hi((uint32_t)(who >> 32),
                                                       __builtin_amdgcn_mbcnt_lo((uint32_t)who, 0u));
                if (keep && wave == 0) L.list[i] = t * 16u + (uint32_t)col;
                n_list += (uint32_t)__popcll(who);
            }
        }
    };
    // the batch: all of the item's tiles, or (CUT) the groups listed at a time
    uint32_t n_batch = t_first < t_end ? (t_end - t_first + step_t - 1) / step_t : 0u;
    if constexpr (CUT) {
        list_groups();
        __syncthreads();
        n_batch = (n_list + 15u) / 16u;
    }
    if (n_batch) fetch(0u);

    // this lane's target (lanes past the last target sit at the origin, their
    // sums unused), and its parts of the B operands of the wave's four groups
    // of 16 targets
    float thx, thy, thz, tlx, tly, tlz;
    bf16x8 B[4];
    {
        const double rx = (ts < nt ? px : ox) - ox, ry = (ts < nt ? py : oy) - oy,
                     rz = (ts < nt ? pz : oz) - oz;
        thx = (float)rx;
        thy = (float)ry;
        thz = (float)rz;
        tlx = (float)(rx - (double)thx);
        tly = (float)(ry - (double)thy);
        tlz = (float)(rz - (double)thz);
        const float T =
            fminf((float)((double)thx * thx + (double)thy * thy + (double)thz * thz), kPadS);
        float(&tl)[6][kTile] = L.tile[1].hl;  // staged only after the first barrier below
        tl[0][tid] = thx;
        tl[1][tid] = thy;
        tl[2][tid] = thz;
        tl[3][tid] = T;
        __syncthreads();
        constexpr uint32_t kOne = 0x3F80u;  // 1.0 in bf16
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const int tg = wave * 64 + g * 16 + col;
            const Bf16x3 c = split_bf16(tl[q < 3 ? q : 0][tg]);
            const Bf16x3 tt = split_bf16(tl[3][tg]);
            u32x4 w;
            w[0] = q < 3 ? c.hh : kOne << 16 | kOne;
            w[1] = q < 3 ? (c.ml & 0xFFFFu) | (c.hh << 16) : kOne << 16;
            w[2] = q < 3 ? (c.hm >> 16) | (c.ml & 0xFFFF0000u) : 0u;
            w[3] = q == 0 ? tt.hm : q == 1 ? tt.ml >> 16 : 0u;
            B[g] = __builtin_bit_cast(bf16x8, w);
        }
    }
    float e2 = a.eps2;
    float rx = ts < nt ? a.acc2 : 0.0f;  // lanes past the last target record nothing
    asm volatile("" : "+v"(e2), "+v"(rx));  // vector registers (see diff_quad)
    CutoffTest ct;
    float in2 = 0.0f, near_a2 = 0.0f;
    if constexpr (CUT) {
        const double cut2 = gp->cut2;
        const float c2 = (float)cut2, ic = (float)(1.0 / sqrt(cut2));
        ct.big_r2 = ldexpf(1.0f, 26 - ilogbf(c2));
        ct.lim_r2 = c2 * ct.big_r2;
        ct.big_inv = ldexpf(1.0f, 26 - ilogbf(ic));
        ct.lim_inv = ic * ct.big_inv;
        asm volatile("" : "+v"(ct.big_r2), "+v"(ct.lim_r2), "+v"(ct.big_inv), "+v"(ct.lim_inv));
        near_a2 = uniform((float)(1.0001 * a2));
        in2 = uniform((float)(0.9999 * a2));
    }
    double fx = 0.0, fy = 0.0, fz = 0.0;  // far blocks
    float ex = 0.0f, ey = 0.0f, ez = 0.0f;
    uint32_t nx = 0;  // pairs in this wave's list

    int buf = 0;
    if (n_batch) stage(0);
    __syncthreads();
    for (uint32_t i = 0; i < n_batch;) {
        const bool more = i + 1 < n_batch;
        if (more) fetch(i + 1);
        const uint32_t src0 = (t_first + i * step_t) * UNIT;  // not CUT: the tile's first source
        const MatrixLds::Tile& S = L.tile[buf];
        const uint32_t cnt = CUT ? min(16u, n_list - i * 16u) * 16u : min((uint32_t)UNIT, ns - src0);
        // lane 16 g + c: target group g of the wave against source group c
        uint64_t far_b, plain_b, near_b, in_b = 0;
        {
            const float gx = fmaxf(0.0f, fmaxf(S.gbox[0][col] - ghx, glx - S.gbox[3][col]));
            const float gy = fmaxf(0.0f, fmaxf(S.gbox[1][col] - ghy, gly - S.gbox[4][col]));
            const float gz = fmaxf(0.0f, fmaxf(S.gbox[2][col] - ghz, glz - S.gbox[5][col]));
            const float g2 = gx * gx + gy * gy + gz * gz;
            bool valid = (uint32_t)col * 16u < cnt && has_targets;
            if constexpr (CUT) {
                valid = valid && g2 < near_a2;
                const float mx = fmaxf(S.gbox[3][col] - glx, ghx - S.gbox[0][col]);
                const float my = fmaxf(S.gbox[4][col] - gly, ghy - S.gbox[1][col]);
                const float mz = fmaxf(S.gbox[5][col] - glz, ghz - S.gbox[2][col]);
                in_b = __ballot(mx * mx + my * my + mz * mz < in2);
            }
            far_b = __ballot(valid && g2 > far2);
            const uint64_t plain = __ballot(g2 > plain2), all = __ballot(valid);
            plain_b = all & plain & ~far_b;
            near_b = all & ~plain & ~far_b;
        }
        const uint32_t far_g[4] = {(uint32_t)far_b & 0xFFFFu, (uint32_t)far_b >> 16,
                                   (uint32_t)(far_b >> 32) & 0xFFFFu, (uint32_t)(far_b >> 48)};
        const uint32_t far_all = far_g[0] & far_g[1] & far_g[2] & far_g[3];
        if (far_b) {
            f32x4 acc[4];  // of target group g: sums of w, -2 s_x w, -2 s_y w, -2 s_z w
#pragma unroll
            for (int g = 0; g < 4; ++g) acc[g] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
            auto source_group = [&](int grp, bf16x8& A, f32x4& x4, f32x4& y4, f32x4& z4) {
                const u32x2 pw = S.pk[grp][q][col];
                const u32x4 aw = {pw[0], pw[1],
                                  __builtin_amdgcn_perm(pw[0], pw[0], 0x05040504u), 0x3F803F80u};
                A = __builtin_bit_cast(bf16x8, aw);
                x4 = *reinterpret_cast<const f32x4*>(&S.hl[0][grp * 16 + q * 4]);
                y4 = *reinterpret_cast<const f32x4*>(&S.hl[1][grp * 16 + q * 4]);
                z4 = *reinterpret_cast<const f32x4*>(&S.hl[2][grp * 16 + q * 4]);
            };
            auto r2_of = [&](const bf16x8& A, int g) {
                return __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                    A, B[g], f32x4{0.0f, 0.0f, 0.0f, 0.0f}, 0, 0, 0);
            };
            auto add_terms = [&](auto cut, int g, const f32x4& inv, const f32x4& x4,
                                 const f32x4& y4, const f32x4& z4) {
                // w of source u in element u ^ 1 of a register quadruple, opposite in
                // parity to the coordinates' element u: an instruction whose three
                // vector registers are all even or all odd takes twice as long
                f32x4 w;
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    w[u ^ 1] = inv[u] * inv[u] * inv[u];
                    if constexpr (decltype(cut)::value)
                        w[u ^ 1] *= clamp01(__builtin_fmaf(inv[u], ct.big_inv, -ct.lim_inv));
                }
                asm("" : "+v"(w));
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    acc[g][0] += w[u ^ 1];
                    acc[g][1] = __builtin_fmaf(x4[u], w[u ^ 1], acc[g][1]);
                    acc[g][2] = __builtin_fmaf(y4[u], w[u ^ 1], acc[g][2]);
                    acc[g][3] = __builtin_fmaf(z4[u], w[u ^ 1], acc[g][3]);
                }
            };
            auto four_groups = [&](auto cut, uint32_t m) {
                while (m) {
                    const int grp = __builtin_ctz(m);
                    m &= m - 1u;
                    bf16x8 A;
                    f32x4 x4, y4, z4, d[4];
                    source_group(grp, A, x4, y4, z4);
#pragma unroll
                    for (int g = 0; g < 4; ++g) d[g] = r2_of(A, g);
#pragma unroll
                    for (int g = 0; g < 4; g += 2) {
                        transcendental_begin();
#pragma unroll
                        for (int u = 0; u < 4; ++u) d[g][u] = __builtin_amdgcn_rsqf(d[g][u]);
#pragma unroll
                        for (int u = 0; u < 4; ++u) d[g + 1][u] = __builtin_amdgcn_rsqf(d[g + 1][u]);
                        transcendental_end();
                        add_terms(cut, g, d[g], x4, y4, z4);
                        add_terms(cut, g + 1, d[g + 1], x4, y4, z4);
                    }
                }
            };
            if constexpr (CUT) {
                const uint32_t in_all = (uint32_t)(in_b & (in_b >> 16) & (in_b >> 32) & (in_b >> 48));
                four_groups(std::false_type{}, far_all & in_all);
                four_groups(std::true_type{}, far_all & ~in_all);
            } else {
                four_groups(std::false_type{}, far_all);
            }
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                uint32_t m = far_g[g] & ~far_all;
                while (m) {
                    const int grp = __builtin_ctz(m);
                    m &= m - 1u;
                    bf16x8 A;
                    f32x4 x4, y4, z4;
                    source_group(grp, A, x4, y4, z4);
                    f32x4 d = r2_of(A, g);
                    transcendental_begin();
#pragma unroll
                    for (int u = 0; u < 4; ++u) d[u] = __builtin_amdgcn_rsqf(d[u]);
                    transcendental_end();
                    add_terms(std::bool_constant<CUT>{}, g, d, x4, y4, z4);
                }
            }
            // add the quarters: lane 16 r + c ends with target c of group r
            float tot[4];
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                auto add32 = [](float u, float v) {
                    const auto r = __builtin_amdgcn_permlane32_swap(
                        __float_as_uint(u), __float_as_uint(v), false, false);
                    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
                };
                auto add16 = [](float u, float v) {
                    const auto r = __builtin_amdgcn_permlane16_swap(
                        __float_as_uint(u), __float_as_uint(v), false, false);
                    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
                };
                tot[c] = add16(add32(acc[0][c], acc[2][c]), add32(acc[1][c], acc[3][c]));
            }
            // t sum w - sum s w of the tile, the second held as -2 sum s w
            const double w = (double)tot[0];
            fx += fma((double)thx, w, 0.5 * (double)tot[1]);
            fy += fma((double)thy, w, 0.5 * (double)tot[2]);
            fz += fma((double)thz, w, 0.5 * (double)tot[3]);
        }
        // near blocks: the lanes' targets of group g, each lane four sources of a group
        for (int g = 0; g < 4; ++g) {
            uint32_t m = (uint32_t)(near_b >> (16 * g)) & 0xFFFFu;
            uint32_t p = (uint32_t)(plain_b >> (16 * g)) & 0xFFFFu;
            if ((m | p) == 0u) continue;
            const int tg = g * 16 + col;
            const float hx_ = __shfl(thx, tg), hy_ = __shfl(thy, tg), hz_ = __shfl(thz, tg);
            const float lx_ = __shfl(tlx, tg), ly_ = __shfl(tly, tg), lz_ = __shfl(tlz, tg);
            const float rx_ = __shfl(rx, tg);
            float bx = 0.0f, by = 0.0f, bz = 0.0f;
            // sources past the last one are staged too, far enough away to add nothing
            while (m) {
                const uint32_t k = (uint32_t)__builtin_ctz(m) * 16u + (uint32_t)q * 4u;
                m &= m - 1u;
                diff_quad<CUT, true>(L.xl[wave], nx, (uint32_t)(wave * 64 + tg), src0 + k, S.hl, k,
                                     hx_, hy_, hz_, lx_, ly_, lz_, e2, rx_, ct, bx, by, bz);
            }
            while (p) {
                const uint32_t k = (uint32_t)__builtin_ctz(p) * 16u + (uint32_t)q * 4u;
                p &= p - 1u;
                diff_quad<CUT, false>(L.xl[wave], nx, (uint32_t)(wave * 64 + tg), src0 + k, S.hl, k,
                                      hx_, hy_, hz_, lx_, ly_, lz_, e2, rx_, ct, bx, by, bz);
            }
            const float tx = add_quarters(bx), ty = add_quarters(by), tz = add_quarters(bz);
            ex += q == g ? tx : 0.0f;
            ey += q == g ? ty : 0.0f;
            ez += q == g ? tz : 0.0f;
        }
        if (more) stage(buf ^ 1);
        __syncthreads();
        buf ^= 1;
        ++i;
        if constexpr (CUT) {
            if (i == n_batch) {  // the next batch; every wave is past the list's last use
                list_groups();
                __syncthreads();
                n_batch = (n_list + 15u) / 16u;
                i = 0;
                if (n_batch) {
                    fetch(0u);
                    stage(buf);
                    __syncthreads();
                }
            }
        }
    }
    for (uint32_t i = (uint32_t)lane; i < nx; i += 64)
        exact_add(a, off + tbase + L.xl[wave].tgt[i], off + L.xl[wave].src[i]);

    if (ts < nt) {
        a.part[(size_t)(chunk * 3 + 0) * a.pstride + off + ts] = (float)(fx + (double)ex);
        a.part[(size_t)(chunk * 3 + 1) * a.pstride + off + ts] = (float)(fy + (double)ey);
        a.part[(size_t)(chunk * 3 + 2) * a.pstride + off + ts] = (float)(fz + (double)ez);
    }
}

// One workgroup per work item.
template <int UNIT>
__global__ __launch_bounds__(kFieldThreads) __attribute__((amdgpu_waves_per_eu(4)))
void field_tiles_matrix(FieldArgs a) {
    const FieldItem it = a.items[blockIdx.x];
    const uint32_t na0 = a.ev_active[0];
    if (a.count_items && blockIdx.x >= *a.n_items) return;  // the whole workgroup
    __shared__ __align__(16) MatrixLds L;
    matrix_item<UNIT, false>(a, it, L, na0);
}

// Persistent form: a fixed grid of workgroups takes the items in list order
// from a counter (queue[0], zero before the launch) until *n_items are taken.
// Every workgroup leaves once the counter has passed the end, so the grid
// drains whatever the item count; the grid and the arguments stay the same
// when the items are rebuilt, which lets a captured graph be replayed.
template <int UNIT>
__global__ __launch_bounds__(kFieldThreads) __attribute__((amdgpu_waves_per_eu(4)))
void field_queue_matrix(FieldArgs a) {
    __shared__ __align__(16) MatrixLds L;
    __shared__ uint32_t next;
    const uint32_t n_items = *a.n_items;
    const uint32_t na0 = a.ev_active[0];
    for (;;) {
        if (threadIdx.x == 0) next = atomicAdd(a.queue, 1u);
        __syncthreads();
        const uint32_t i = next;
        __syncthreads();  // every lane has read `next` before lane 0 writes it again
        if (i >= n_items) break;
        matrix_item<UNIT, false>(a, a.items[i], L, na0);
    }
}

// Eq. (6) entirely in FP64: the difference, q = r^2 + eps^2, r^-3 = q^(-3/2)
// from the hardware's reciprocal square root and a second-order correction,
// and the sums.  Bound by VALU issue, 17 FP64 instructions at 4.3 cycles and the
// estimate at 16: 6.5 ms at 1e5 holes, where 1/(q sqrt q) with IEEE square root
// and division took 12.6.  q is held finite so that a pair farther apart than
// 1e150 um adds nothing; since that also hides a NaN from r^-3, a hole with any NaN
// coordinate takes part with three (whole_nan).  Same work items, tiles
// and source dealing as field_tiles; the FP64 sum of group g is written as
// the FP32 pair hi (group g) and lo (group G + g, G the event's groups),
// which the FP64 reduction of the groups adds back exactly.
__device__ __forceinline__ void whole_nan(double& x, double& y, double& z) {
    if (x != x || y != y || z != z) x = y = z = __builtin_nan("");
}

template <int TPT>
__global__ __launch_bounds__(kFieldThreads) void field_tiles_f64(FieldArgs a) {
    __shared__ double sh[2][3][kTile];

    const FieldItem it = a.items[blockIdx.x];
    const uint32_t off = a.ev_off[it.event];
    const uint32_t ne = a.ev_off[it.event + 1] - off;
    const uint32_t na = a.ev_active[it.event];
    const uint32_t nt = a.targets_all ? ne : na;
    const uint32_t ns = a.sources_all ? ne : na;
    const uint32_t tbase = it.blk * (uint32_t)(kFieldThreads * TPT);
    if (tbase >= nt) return;
    const uint32_t ntiles = (ns + kTile - 1) / kTile;
    const uint32_t chunk = it.group;  // partial-sum group written
    const uint32_t step_t = it.step;
    const uint32_t t_first = it.first;
    const uint32_t t_end = min(it.end, ntiles);
    const int tid = threadIdx.x;
    const double eps2 = a.eps2d;

    double px[TPT], py[TPT], pz[TPT], ax[TPT], ay[TPT], az[TPT];
#pragma unroll
    for (int t = 0; t < TPT; ++t) {
        const uint32_t ts = tbase + (uint32_t)(t * kFieldThreads + tid);
        px[t] = py[t] = pz[t] = 0.0;
        if (ts < nt) {
            px[t] = a.px[off + ts];
            py[t] = a.py[off + ts];
            pz[t] = a.pz[off + ts];
            whole_nan(px[t], py[t], pz[t]);
        }
        ax[t] = ay[t] = az[t] = 0.0;
    }

    double qx = 0.0, qy = 0.0, qz = 0.0;
    auto fetch = [&](uint32_t t) {
        const uint32_t i = t * kTile + (uint32_t)tid;
        qx = qy = qz = 0.0;
        if (i < ns) {
            qx = a.px[off + i];
            qy = a.py[off + i];
            qz = a.pz[off + i];
            whole_nan(qx, qy, qz);
        }
    };
    auto stage = [&](int b) {
        sh[b][0][tid] = qx;
        sh[b][1][tid] = qy;
        sh[b][2][tid] = qz;
    };

    int buf = 0;
    if (t_first < t_end) {
        fetch(t_first);
        stage(0);
    }
    __syncthreads();
    for (uint32_t t = t_first; t < t_end; t += step_t) {
        const uint32_t next = t + step_t;
        if (next < t_end) fetch(next);
        const uint32_t cnt = min((uint32_t)kTile, ns - t * kTile);
        for (uint32_t k = 0; k < cnt; ++k) {
            const double sx = sh[buf][0][k], sy = sh[buf][1][k], sz = sh[buf][2][k];
#pragma unroll
            for (int u = 0; u < TPT; ++u) {
                const double dx = px[u] - sx, dy = py[u] - sy, dz = pz[u] - sz;
                double q = fma(dx, dx, eps2);
                q = fma(dy, dy, q);
                q = fma(dz, dz, q);
                const double w = fp64::rsqrt3_pos(fmin(q, 1e300));
                ax[u] = fma(dx, w, ax[u]);
                ay[u] = fma(dy, w, ay[u]);
                az[u] = fma(dz, w, az[u]);
            }
        }
        if (next < t_end) stage(buf ^ 1);
        __syncthreads();
        buf ^= 1;
    }

#pragma unroll
    for (int t = 0; t < TPT; ++t) {
        const uint32_t ts = tbase + (uint32_t)(t * kFieldThreads + tid);
        if (ts >= nt) continue;
        const double v[3] = {ax[t], ay[t], az[t]};
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            const float hi = (float)v[d];
            const float lo = (float)(v[d] - (double)hi);
            a.part[(size_t)(chunk * 3 + d) * a.pstride + off + ts] = hi;
            a.part[(size_t)((it.groups + chunk) * 3 + d) * a.pstride + off + ts] = lo;
        }
    }
}

// The near part of the closure's split of Eq. (6): matrix_item with the cutoff.
// Bound by VALU issue: 4.3 ms at 1e6 holes, of which (measured with the far limit at
// rho/5, 4.1 ms) 1.6 go to source groups far from all four target groups, 1.0 to
// single far blocks, 0.9 to nearer ones, 0.1 to staging.  A kernel on difference forms
// that culled 16-source groups against 64 targets and staged whole tiles took 6.8.
// rms error of the near sum against 64 bits, that kernel and this one, in its rms:
// 65,536 holes 2.7e-7 and 1.7e-7, 70,001 3.3e-7 and 1.5e-7, 2e5 4.0e-7 and 2.0e-7, 1e6
// 4.0e-7 and 1.7e-7.
__global__ __launch_bounds__(kFieldThreads) __attribute__((amdgpu_waves_per_eu(4)))
void near_matrix(FieldArgs a, const GridParams* gp) {
    __shared__ __align__(16) MatrixLds L;
    matrix_item<kTile, true>(a, a.items[blockIdx.x], L, a.ev_active[0], gp);
}

// ---------------------------------------------------------------------------
// Near part of the closure's split of Eq. (6) for loads below kNearMatrixMin
// holes (see launch_near): the same sum over the sources closer than a only
// (r^2 + eps^2 < a^2 + eps^2), in the difference form of field_tiles with its
// origins, hi and lo parts and close-pair recomputation.  Chunk c of the sum holds
// the source tiles c, c + S, c + 2 S, ..., at most kNearTiles of them.
//
// One wave per workgroup: 64 targets and one chunk, whose tiles are tested by
// one lane each.  The 16-source groups of the tiles that come within a of the
// wave's targets are listed (a group within a of them as a whole skips the
// per-pair cutoff), and the wave stages four at a time, the next four's
// positions in flight, and sums those that come within a of any of its targets.
// The last test matters most for the holes at the cloud's edge, whose boxes are
// large: without it their waves, the longest, set the time.  The sums of a tile
// are taken before they meet those of other tiles.
//
// Four waves that shared whole staged tiles spent over half of their time at
// barriers and in set-up: 5e4 holes 204 us, this kernel 93.  Two chunks per
// wave 111 us, four 145 (fewer set-ups, longer waves); workgroups of four such
// waves 97.
// ---------------------------------------------------------------------------
constexpr int kNearTiles = 8;

__global__ __launch_bounds__(64) void near_waves(FieldArgs a, const GridParams* gp,
                                                 uint32_t n_chunks) {
    __shared__ __align__(16) float sh[2][6][64];
    __shared__ __align__(16) float gbox[2][4][8];  // boxes of the staged groups
    __shared__ uint16_t list[kNearTiles * 16];  // tile | group << 3 | inside << 7 | far << 8

    const uint32_t nwaves = gridDim.x / n_chunks;
    const uint32_t wave = blockIdx.x % nwaves;  // of the event's targets
    const uint32_t chunk = blockIdx.x / nwaves;
    const uint32_t ne = a.pstride, na = a.ev_active[0];
    const uint32_t nt = a.targets_all ? ne : na;
    const uint32_t ns = a.sources_all ? ne : na;
    const uint32_t ts0 = wave * 64u, tbase = ts0 & ~(uint32_t)(kFieldThreads - 1);
    if (ts0 >= nt) return;
    const uint32_t ntiles = (ns + kTile - 1) / kTile;
    const int lane = threadIdx.x;
    const uint32_t ts = ts0 + (uint32_t)lane;
    const size_t st = a.tile_stride;

    double px = 0.0, py = 0.0, pz = 0.0;
    if (ts < nt) {
        px = a.px[ts];
        py = a.py[ts];
        pz = a.pz[ts];
    }
    // The boxes of the 256-target block (its centre is the origin) and of this wave's
    // targets, by which groups are culled: those of a source tile and its quarter
    // where all 256 targets are sources.
    double lo[3], hi[3], wl[3], wh[3];
    if (tbase + (uint32_t)kFieldThreads <= min(nt, ns)) {
        const double* tb = a.tile_box + tbase / kTile;
        const uint32_t qr = (ts0 - tbase) / 64u;
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            lo[k] = tb[k * st];
            hi[k] = tb[(3 + k) * st];
            wl[k] = tb[(6 + 4 * k + qr) * st];
            wh[k] = tb[(6 + 4 * (3 + k) + qr) * st];
        }
    } else {
        for (int k = 0; k < 3; ++k) {
            const double* p = k == 0 ? a.px : k == 1 ? a.py : a.pz;
            lo[k] = wl[k] = INFINITY;
            hi[k] = wh[k] = -INFINITY;
            for (uint32_t w = 0; w < kFieldThreads / 64; ++w) {
                const uint32_t i = tbase + w * 64u + (uint32_t)lane;
                if (i < nt) {
                    const double v = p[i];
                    lo[k] = fmin(lo[k], v);
                    hi[k] = fmax(hi[k], v);
                    if (i == ts) wl[k] = wh[k] = v;
                }
            }
            lo[k] = wave_min(lo[k]);
            hi[k] = wave_max(hi[k]);
            wl[k] = wave_min(wl[k]);
            wh[k] = wave_max(wh[k]);
        }
    }
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        lo[k] = uniform(lo[k]);
        hi[k] = uniform(hi[k]);
        wl[k] = uniform(wl[k]);
        wh[k] = uniform(wh[k]);
    }
    const double ox = 0.5 * (lo[0] + hi[0]), oy = 0.5 * (lo[1] + hi[1]), oz = 0.5 * (lo[2] + hi[2]);
    const double hx = 0.5 * (hi[0] - lo[0]), hy = 0.5 * (hi[1] - lo[1]), hz = 0.5 * (hi[2] - lo[2]);
    const double rc2d = 0.0625 * (hx * hx + hy * hy + hz * hz);
    const double a2 = uniform(gp->a2);
    const float cut2 = uniform((float)gp->cut2);

    const auto tile_of = [&](uint32_t l) { return chunk + l * n_chunks; };
    const auto gap2_of = [&](const double* b, size_t s) {  // b: low x at b[0], ..., stride s
        const double gx = fmax(0.0, fmax(b[0] - wh[0], wl[0] - b[3 * s]));
        const double gy = fmax(0.0, fmax(b[s] - wh[1], wl[1] - b[4 * s]));
        const double gz = fmax(0.0, fmax(b[2 * s] - wh[2], wl[2] - b[5 * s]));
        return gx * gx + gy * gy + gz * gz;
    };
    uint64_t cand;  // tiles within a of the targets
    {
        const uint32_t t = tile_of((uint32_t)lane);
        const bool have = lane < kNearTiles && t < ntiles;
        cand = __ballot(have && gap2_of(a.tile_box + (have ? t : 0u), st) < a2);
    }
    // the groups of those tiles, four tiles at a time, sixteen lanes each
    uint32_t n_list = 0;
    while (cand) {
        uint32_t l = 64u;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const uint32_t bit = cand ? (uint32_t)__builtin_ctzll(cand) : 64u;
            cand &= cand - 1ull;
            if ((lane >> 4) == k) l = bit;
        }
        const uint32_t grp = (uint32_t)lane & 15u, t = l < 64u ? tile_of(l) : 0u;
        const double* gb = a.tile_box + (size_t)(30 + grp) * st + t;  // bound k at gb[16 k st]
        const double gap2 = gap2_of(gb, 16 * st);
        // largest distance between the boxes: every pair well inside a (a margin
        // far above the FP32 error of r^2) needs no per-pair test
        const double mx = fmax(gb[48 * st] - wl[0], wh[0] - gb[0]);
        const double my = fmax(gb[64 * st] - wl[1], wh[1] - gb[16 * st]);
        const double mz = fmax(gb[80 * st] - wl[2], wh[2] - gb[32 * st]);
        const bool inside = mx * mx + my * my + mz * mz < 0.9999 * a2;
        const bool keep = l < 64u && t * kTile + grp * 16u < ns && gap2 < a2;
        const uint64_t who = __ballot(keep);
        if (keep)
            list[n_list + (uint32_t)__popcll(who & ((1ull << lane) - 1ull))] =
                (uint16_t)(l | grp << 3 | (inside ? 1u << 7 : 0u) |
                           (gap2 >= rc2d ? 1u << 8 : 0u));
        n_list += (uint32_t)__popcll(who);
    }
    __syncthreads();

    float thx[1], thy[1], thz[1], tlx[1], tly[1], tlz[1], rc2[1];
    {
        const double rx = px - ox, ry = py - oy, rz = pz - oz;
        thx[0] = (float)rx;
        thy[0] = (float)ry;
        thz[0] = (float)rz;
        tlx[0] = (float)(rx - (double)thx[0]);
        tly[0] = (float)(ry - (double)thy[0]);
        tlz[0] = (float)(rz - (double)thz[0]);
        // close-pair radius of this target, as in field_tiles
        rc2[0] = ts < nt ? 0.0625f * (float)((double)thx[0] * thx[0] + (double)thy[0] * thy[0] +
                                             (double)thz[0] * thz[0])
                         : 0.0f;
    }
    double qx = 0.0, qy = 0.0, qz = 0.0;
    double qb = 0.0;  // lanes 0-23: bound lane % 6 of the box of group lane / 6
    const double ob = lane % 3 == 0 ? ox : lane % 3 == 1 ? oy : oz;  // its origin
    auto fetch = [&](uint32_t i) {  // listed groups i .. i + 3
        qx = ox;
        qy = oy;
        qz = oz;
        const uint32_t e = i + (uint32_t)(lane >> 4);
        if (e < n_list) {
            const uint32_t v = list[e];
            const uint32_t j =
                tile_of(v & 7u) * kTile + ((v >> 3) & 15u) * 16u + ((uint32_t)lane & 15u);
            if (j < ns) {
                qx = a.px[j];
                qy = a.py[j];
                qz = a.pz[j];
            }
        }
        const uint32_t eb = i + (uint32_t)lane / 6u;
        if (lane < 24 && eb < n_list) {
            const uint32_t v = list[eb];
            qb = a.tile_box[(size_t)(30u + 16u * ((uint32_t)lane % 6u) + ((v >> 3) & 15u)) * st +
                            tile_of(v & 7u)];
        }
    };
    auto stage = [&](int b) {
        if (lane < 24) gbox[b][lane / 6][lane % 6] = (float)(qb - ob);
        const double rx = qx - ox, ry = qy - oy, rz = qz - oz;
        const float fx = (float)rx, fy = (float)ry, fz = (float)rz;
        sh[b][0][lane] = fx;
        sh[b][1][lane] = fy;
        sh[b][2][lane] = fz;
        sh[b][3][lane] = (float)(rx - (double)fx);
        sh[b][4][lane] = (float)(ry - (double)fy);
        sh[b][5][lane] = (float)(rz - (double)fz);
    };
    // of FP32 coordinates, with a margin far above their rounding
    const float near_a2 = uniform((float)(1.001 * a2));
    float ax = 0.0f, ay = 0.0f, az = 0.0f;
    float bx[1] = {0.0f}, by[1] = {0.0f}, bz[1] = {0.0f};
    uint32_t tile = 0u;  // (its number in the chunk) whose sums b holds
    auto end_tile = [&]() {
        ax += bx[0];
        ay += by[0];
        az += bz[0];
        bx[0] = by[0] = bz[0] = 0.0f;
    };
    int buf = 0;
    fetch(0u);
    for (uint32_t i = 0; i < n_list; i += 4u) {
        stage(buf);
        __syncthreads();
        fetch(i + 4u);
        const uint32_t m = min(4u, n_list - i);
        for (uint32_t u = 0; u < m; ++u) {
            const uint32_t v = (uint32_t)__builtin_amdgcn_readfirstlane((int)list[i + u]);
            {  // no target of the wave within a of the group's box: no term
                const f32x4 g0 = *reinterpret_cast<const f32x4*>(&gbox[buf][u][0]);
                const float g4 = gbox[buf][u][4], g5 = gbox[buf][u][5];
                const float gx = fmaxf(0.0f, fmaxf(g0[0] - thx[0], thx[0] - g0[3]));
                const float gy = fmaxf(0.0f, fmaxf(g0[1] - thy[0], thy[0] - g4));
                const float gz = fmaxf(0.0f, fmaxf(g0[2] - thz[0], thz[0] - g5));
                if (!__any(ts < nt && gx * gx + gy * gy + gz * gz < near_a2)) continue;
            }
            if ((v & 7u) != tile) {
                end_tile();
                tile = v & 7u;
            }
            const uint32_t j0 = tile_of(tile) * kTile + ((v >> 3) & 15u) * 16u;
            const uint32_t kn = min(16u, ns - j0);
            const float* hxp = sh[buf][0] + u * 16u;
            const float* hyp = sh[buf][1] + u * 16u;
            const float* hzp = sh[buf][2] + u * 16u;
            const float* lxp = sh[buf][3] + u * 16u;
            const float* lyp = sh[buf][4] + u * 16u;
            const float* lzp = sh[buf][5] + u * 16u;
            const bool inside = (v >> 7) & 1u, far = (v >> 8) & 1u;
            if (inside) {
                if (far)
                    tile_terms<1, kDiffHi, false>(hxp, hyp, hzp, lxp, lyp, lzp, kn, thx, thy, thz,
                                                  tlx, tly, tlz, a.eps2, rc2, bx, by, bz);
                else
                    tile_terms<1, kDiffNear, false>(hxp, hyp, hzp, lxp, lyp, lzp, kn, thx, thy, thz,
                                                    tlx, tly, tlz, a.eps2, rc2, bx, by, bz);
            } else {
                if (far)
                    tile_terms<1, kDiffHi, true>(hxp, hyp, hzp, lxp, lyp, lzp, kn, thx, thy, thz,
                                                 tlx, tly, tlz, a.eps2, rc2, bx, by, bz, cut2);
                else
                    tile_terms<1, kDiffNear, true>(hxp, hyp, hzp, lxp, lyp, lzp, kn, thx, thy, thz,
                                                   tlx, tly, tlz, a.eps2, rc2, bx, by, bz, cut2);
            }
        }
        buf ^= 1;
    }
    end_tile();
    if (ts < nt) {
        a.part[(size_t)(chunk * 3 + 0) * a.pstride + ts] = ax;
        a.part[(size_t)(chunk * 3 + 1) * a.pstride + ts] = ay;
        a.part[(size_t)(chunk * 3 + 2) * a.pstride + ts] = az;
    }
}

// The matrix kernel for loads of at least kNearMatrixMin holes, where near_waves'
// kNearTiles tiles per chunk end.  Below, the two are level: closure step at 2e4,
// 3.3e4, 5e4 and 65,535 holes 170, 195, 220 and 247 us with near_waves, 170, 197, 216 and
// 246 with the matrix kernel (measured down to 16,384); rms error of the near sum
// 2.5e-7, 2.5e-7, 2.0e-7, 2.9e-7 and 2.1e-7, 2.2e-7, 1.3e-7, 1.8e-7.  near_waves stays for
// its terms and their order, those that these loads' runs have always had: the FP32
// rounding of a close pair's near sum grows along a run.
hipError_t launch_near(const FieldArgs& a, const GridParams* gp, uint32_t n, uint32_t n_items,
                       uint32_t n_chunks, hipStream_t s) {
    if (n_items == 0) return hipSuccess;
    if (n >= (uint32_t)kNearMatrixMin) {
        near_matrix<<<n_items, kFieldThreads, 0, s>>>(a, gp);
        return hipGetLastError();
    }
    // one event, and no chunk of more than kNearTiles tiles
    const uint32_t tiles = (n + kTile - 1) / kTile;
    if (a.pstride != n || n_chunks == 0 || tiles > n_chunks * (uint32_t)kNearTiles)
        return hipErrorInvalidValue;
    const uint32_t waves = n_items / n_chunks * (kFieldThreads / 64);
    near_waves<<<waves * n_chunks, 64, 0, s>>>(a, gp, n_chunks);
    return hipGetLastError();
}

template <int PREC>
static hipError_t launch_field_prec(const FieldArgs& a, int tpt, uint32_t n_items,
                                    hipStream_t s) {
    switch (tpt) {
        case 1:
            if constexpr (PREC == GCCD_PRECISION_DEFAULT)
                return hipErrorInvalidValue;  // the matrix kernel's
            else
                field_tiles<1, PREC><<<n_items, kFieldThreads, 0, s>>>(a);
            break;
        case 2: field_tiles<2, PREC><<<n_items, kFieldThreads, 0, s>>>(a); break;
        case 4: field_tiles<4, PREC><<<n_items, kFieldThreads, 0, s>>>(a); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

// Workgroups of the Eq. (6) kernel that one compute unit holds at once for
// this shape (registers and LDS permitting); 1 if the runtime cannot say.
int field_queue_slots_per_cu() {
    int n = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(
            &n, reinterpret_cast<const void*>(field_queue_matrix<kTile>), kFieldThreads,
            0) !=
        hipSuccess) {
        (void)hipGetLastError();
        return 1;
    }
    return n > 0 ? n : 1;
}

int field_slots_per_cu(int tpt, int precision) {
    int n = 0;
    hipError_t e = hipErrorInvalidValue;
    if (precision == GCCD_PRECISION_FP64) {
        if (tpt == 1)
            e = hipOccupancyMaxActiveBlocksPerMultiprocessor(
                &n, reinterpret_cast<const void*>(field_tiles_f64<1>), kFieldThreads, 0);
        else if (tpt == 2)
            e = hipOccupancyMaxActiveBlocksPerMultiprocessor(
                &n, reinterpret_cast<const void*>(field_tiles_f64<2>), kFieldThreads, 0);
        else
            e = hipOccupancyMaxActiveBlocksPerMultiprocessor(
                &n, reinterpret_cast<const void*>(field_tiles_f64<4>), kFieldThreads, 0);
    } else if (tpt == 1 && precision == GCCD_PRECISION_DEFAULT) {
        e = hipOccupancyMaxActiveBlocksPerMultiprocessor(
            &n, reinterpret_cast<const void*>(field_tiles_matrix<kTile>), kFieldThreads, 0);
    } else if (tpt == 1) {
        e = hipOccupancyMaxActiveBlocksPerMultiprocessor(
            &n, reinterpret_cast<const void*>(field_tiles<1, GCCD_PRECISION_BLOCK>),
            kFieldThreads, 0);
    } else if (tpt == 2) {
        e = hipOccupancyMaxActiveBlocksPerMultiprocessor(
            &n, reinterpret_cast<const void*>(field_tiles<2, GCCD_PRECISION_DEFAULT>),
            kFieldThreads, 0);
    } else {
        e = hipOccupancyMaxActiveBlocksPerMultiprocessor(
            &n, reinterpret_cast<const void*>(field_tiles<4, GCCD_PRECISION_DEFAULT>),
            kFieldThreads, 0);
    }
    if (e != hipSuccess) {
        (void)hipGetLastError();
        return 1;
    }
    return n > 0 ? n : 1;
}

hipError_t launch_field(const FieldArgs& a, int tpt, int precision, uint32_t n_items,
                        uint32_t queue_grid, hipStream_t s, uint32_t grid_cap) {
    if (grid_cap > 0) {
        if (tpt != 1 || precision != GCCD_PRECISION_DEFAULT || n_items > grid_cap)
            return hipErrorInvalidValue;
        FieldArgs b = a;
        b.count_items = 1;
        switch (b.unit) {
            case kTile / 4:
                field_tiles_matrix<kTile / 4><<<grid_cap, kFieldThreads, 0, s>>>(b);
                break;
            case kTile / 2:
                field_tiles_matrix<kTile / 2><<<grid_cap, kFieldThreads, 0, s>>>(b);
                break;
            case kTile:
                field_tiles_matrix<kTile><<<grid_cap, kFieldThreads, 0, s>>>(b);
                break;
            default: return hipErrorInvalidValue;
        }
        return hipGetLastError();
    }
    if (queue_grid > 0 && tpt == 1 && precision == GCCD_PRECISION_DEFAULT) {
        // the item count is read on the device: launched even with none
        const hipError_t e = launch_fill_u32(a.queue, 1u, 0u, s);
        if (e != hipSuccess) return e;
        switch (a.unit) {
            case kTile / 4:
                field_queue_matrix<kTile / 4><<<queue_grid, kFieldThreads, 0, s>>>(a);
                break;
            case kTile / 2:
                field_queue_matrix<kTile / 2><<<queue_grid, kFieldThreads, 0, s>>>(a);
                break;
            case kTile:
                field_queue_matrix<kTile><<<queue_grid, kFieldThreads, 0, s>>>(a);
                break;
            default: return hipErrorInvalidValue;
        }
        return hipGetLastError();
    }
    if (n_items == 0) return hipSuccess;
    // only the one-target-per-lane default kernel takes smaller tiles
    if (a.unit != kTile && !(tpt == 1 && precision == GCCD_PRECISION_DEFAULT))
        return hipErrorInvalidValue;
    switch (precision) {
        case GCCD_PRECISION_DEFAULT:
            if (tpt == 1) {
                switch (a.unit) {
                    case kTile / 4:
                        field_tiles_matrix<kTile / 4><<<n_items, kFieldThreads, 0, s>>>(a);
                        break;
                    case kTile / 2:
                        field_tiles_matrix<kTile / 2><<<n_items, kFieldThreads, 0, s>>>(a);
                        break;
                    case kTile:
                        field_tiles_matrix<kTile><<<n_items, kFieldThreads, 0, s>>>(a);
                        break;
                    default: return hipErrorInvalidValue;
                }
                return hipGetLastError();
            }
            return launch_field_prec<GCCD_PRECISION_DEFAULT>(a, tpt, n_items, s);
        case GCCD_PRECISION_BLOCK:
            return launch_field_prec<GCCD_PRECISION_BLOCK>(a, tpt, n_items, s);
        case GCCD_PRECISION_EVENT:
            return launch_field_prec<GCCD_PRECISION_EVENT>(a, tpt, n_items, s);
        case GCCD_PRECISION_ABSOLUTE:
            return launch_field_prec<GCCD_PRECISION_ABSOLUTE>(a, tpt, n_items, s);
        case GCCD_PRECISION_COMPENSATED:
            return launch_field_prec<GCCD_PRECISION_COMPENSATED>(a, tpt, n_items, s);
        case GCCD_PRECISION_FP64:
            switch (tpt) {
                case 1: field_tiles_f64<1><<<n_items, kFieldThreads, 0, s>>>(a); break;
                case 2: field_tiles_f64<2><<<n_items, kFieldThreads, 0, s>>>(a); break;
                case 4: field_tiles_f64<4><<<n_items, kFieldThreads, 0, s>>>(a); break;
                default: return hipErrorInvalidValue;
            }
            return hipGetLastError();
        default: return hipErrorInvalidValue;
    }
}

static uint32_t grid_for(uint64_t n, int threads, uint32_t cap) {
    uint64_t g = (n + (uint64_t)threads - 1) / (uint64_t)threads;
    if (g < 1) g = 1;
    if (g > cap) g = cap;
    return (uint32_t)g;
}

// ---------------------------------------------------------------------------
// The sorted list.  make_keys writes every carrier's key (carrier order);
// after the sort, count_active finds in each event's segment the first
// collected key (the segment holds its travelling holes first) and records
// the step's holes and pair interactions; gather_tiles copies the positions
// into slot order and takes the bounding box of every source tile.
// ---------------------------------------------------------------------------
__global__ void make_keys(const double* x, const double* y, const double* z,
                          const int32_t* cstep, const uint32_t* ev_of, const uint32_t* ev_off,
                          uint32_t n, KeyLayout kl, uint64_t* keys) {
    for (uint32_t j = blockIdx.x * blockDim.x + threadIdx.x; j < n; j += gridDim.x * blockDim.x) {
        const uint32_t e = ev_of[j];
        keys[j] = make_key(e, cstep[j] >= 0, x[j], y[j], z[j], j - ev_off[e], kl);
    }
}

hipError_t launch_make_keys(const double* x, const double* y, const double* z,
                            const int32_t* cstep, const uint32_t* ev_of, const uint32_t* ev_off,
                            uint32_t n, KeyLayout kl, uint64_t* keys, hipStream_t s) {
    make_keys<<<grid_for(n, 256, 8192), 256, 0, s>>>(x, y, z, cstep, ev_of, ev_off, n, kl, keys);
    return hipGetLastError();
}

// The travelling holes of each event: the first collected key of its
// segment (travelling holes come first), by binary search.
constexpr int kCountThreads = 256;

__global__ __launch_bounds__(kCountThreads) void count_active(const uint64_t* keys,
                                                              const uint32_t* ev_off,
                                                              uint32_t n_events, KeyLayout kl,
                                                              uint32_t* ev_active) {
    for (uint32_t e = blockIdx.x * blockDim.x + threadIdx.x; e < n_events;
         e += gridDim.x * blockDim.x) {
        const uint32_t off = ev_off[e], ne = ev_off[e + 1] - off;
        uint32_t lo = 0, hi = ne;  // first collected key of the segment in [lo, hi]
        while (lo < hi) {
            const uint32_t mid = (lo + hi) >> 1;
            if (key_collected(keys[off + mid], kl))
                hi = mid;
            else
                lo = mid + 1;
        }
        ev_active[e] = lo;
    }
}

hipError_t launch_count(const uint64_t* keys, const uint32_t* ev_off, uint32_t n_events,
                        KeyLayout kl, uint32_t* ev_active, hipStream_t s) {
    count_active<<<grid_for(n_events, kCountThreads, 1024), kCountThreads, 0, s>>>(
        keys, ev_off, n_events, kl, ev_active);
    return hipGetLastError();
}

// The boxes of source tile g, by kTile threads of a workgroup (tid: index among
// them), one slot each (source: whether the slot is one): bounding box of the tile (rows
// 0-5 of box: low x, y, z, high x, y, z), and the same for each 64-slot
// quarter of the tile (row 6 + 4 k + q for bound k of quarter q) and each
// 16-slot group (row 30 + 16 k + g), which the near-field kernel culls by.
// The group boxes are the first four steps of the lane reduction that gives
// the quarter boxes.
__device__ __forceinline__ void tile_boxes(uint32_t g, uint32_t tid, bool source, double vx,
                                           double vy, double vz, double* box, uint32_t stride,
                                           double (*red)[kTile / 64], bool write = true) {
    double lx = source ? vx : INFINITY, ly = source ? vy : INFINITY, lz = source ? vz : INFINITY;
    double hx = source ? vx : -INFINITY, hy = source ? vy : -INFINITY, hz = source ? vz : -INFINITY;
    // butterfly over lanes: after the strides 1..8 every lane holds its
    // 16-slot group's box, after 16 and 32 its quarter's
#pragma unroll
    for (int m = 1; m <= 8; m <<= 1) {
        lx = fmin(lx, __shfl_xor(lx, m));
        ly = fmin(ly, __shfl_xor(ly, m));
        lz = fmin(lz, __shfl_xor(lz, m));
        hx = fmax(hx, __shfl_xor(hx, m));
        hy = fmax(hy, __shfl_xor(hy, m));
        hz = fmax(hz, __shfl_xor(hz, m));
    }
    if (write && (tid & 15) == 0) {
        const int grp = tid >> 4;  // 0 .. 15
        const double v[6] = {lx, ly, lz, hx, hy, hz};
#pragma unroll
        for (int k = 0; k < 6; ++k) box[(size_t)(30 + 16 * k + grp) * stride + g] = v[k];
    }
#pragma unroll
    for (int m = 16; m <= 32; m <<= 1) {
        lx = fmin(lx, __shfl_xor(lx, m));
        ly = fmin(ly, __shfl_xor(ly, m));
        lz = fmin(lz, __shfl_xor(lz, m));
        hx = fmax(hx, __shfl_xor(hx, m));
        hy = fmax(hy, __shfl_xor(hy, m));
        hz = fmax(hz, __shfl_xor(hz, m));
    }
    const int wave = tid >> 6;
    if ((tid & 63) == 0) {
        red[0][wave] = lx;
        red[1][wave] = ly;
        red[2][wave] = lz;
        red[3][wave] = hx;
        red[4][wave] = hy;
        red[5][wave] = hz;
        const double v[6] = {lx, ly, lz, hx, hy, hz};
#pragma unroll
        for (int k = 0; k < 6; ++k)
            if (write) box[(size_t)(6 + 4 * k + wave) * stride + g] = v[k];
    }
    __syncthreads();
    if (write && tid < 6) {
        const int k = tid;
        double v = red[k][0];
        for (int w = 1; w < kTile / 64; ++w) v = (k < 3) ? fmin(v, red[k][w]) : fmax(v, red[k][w]);
        box[(size_t)k * stride + g] = v;
    }
}

// Source tile g of event e = tile_event[g] (local tile t = g - ev_tile[e]),
// by one workgroup of kTile threads: positions of every slot of the tile
// (key_at(slot) gives the slot's key) and its boxes; ns_or_active is the
// event's travelling holes, the sources unless sources_all.
template <class KeyAt>
__device__ __forceinline__ void gather_tile(uint32_t g, KeyAt key_at, const uint32_t* ev_off,
                                            const uint32_t* ev_tile, const uint32_t* tile_event,
                                            uint32_t ns_or_active, int sources_all, KeyLayout kl,
                                            const double* x, const double* y, const double* z,
                                            double* px, double* py, double* pz, double* box,
                                            uint32_t stride, double (*red)[kTile / 64]) {
    const uint32_t e = tile_event[g];
    const uint32_t t = g - ev_tile[e];
    const uint32_t off = ev_off[e], ne = ev_off[e + 1] - off;
    const uint32_t ns = sources_all ? ne : ns_or_active;
    const uint32_t i = t * kTile + threadIdx.x;
    double vx = 0.0, vy = 0.0, vz = 0.0;
    if (i < ne) {
        // a slot of event e holds a key of event e; the clamp keeps every
        // load inside the event regardless
        const uint32_t c = off + min(key_local(key_at(off + i), kl), ne - 1u);
        vx = x[c];
        vy = y[c];
        vz = z[c];
        px[off + i] = vx;
        py[off + i] = vy;
        pz[off + i] = vz;
    }
    tile_boxes(g, threadIdx.x, i < ne && i < ns, vx, vy, vz, box, stride, red);
}

__global__ __launch_bounds__(kTile) void gather_tiles(
    const uint64_t* keys, const uint32_t* ev_off, const uint32_t* ev_tile,
    const uint32_t* tile_event, const uint32_t* ev_active, int sources_all, KeyLayout kl,
    const double* x, const double* y, const double* z, double* px, double* py, double* pz,
    double* box, uint32_t stride) {
    __shared__ double red[6][kTile / 64];
    const uint32_t g = blockIdx.x;
    gather_tile(
        g, [&](uint32_t slot) { return keys[slot]; }, ev_off, ev_tile, tile_event,
        sources_all ? 0u : ev_active[tile_event[g]], sources_all, kl, x, y, z, px, py, pz, box,
        stride, red);
}

// gather_tiles and count_active in one launch, for lists whose sources are
// every hole (the gather then needs no count): tile g also finds whether the
// event's first collected key -- its travelling count, the keys of a
// segment being ordered travelling before collected -- lies in its slots.
// Exactly one workgroup writes each event's count: the one whose tile holds
// the first collected key (the slot before the tile travelling, or the tile
// first in its event), or the event's last tile if no key is collected;
// workgroup 0 writes 0 for the events with no holes (and no tiles).
__global__ __launch_bounds__(kTile) void gather_count_tiles(
    const uint64_t* keys, const uint32_t* ev_off, const uint32_t* ev_tile,
    const uint32_t* tile_event, uint32_t n_events, KeyLayout kl, const double* x,
    const double* y, const double* z, double* px, double* py, double* pz, double* box,
    uint32_t stride, uint32_t* ev_active) {
    __shared__ double red[6][kTile / 64];
    __shared__ uint32_t first_col[kTile / 64];
    const uint32_t g = blockIdx.x;
    if (g == 0) {
        for (uint32_t e = threadIdx.x; e < n_events; e += kTile)
            if (ev_off[e + 1] == ev_off[e]) ev_active[e] = 0u;
    }
    gather_tile(
        g, [&](uint32_t slot) { return keys[slot]; }, ev_off, ev_tile, tile_event, 0u, 1, kl,
        x, y, z, px, py, pz, box, stride, red);
    const uint32_t e = tile_event[g];
    const uint32_t t0 = (g - ev_tile[e]) * kTile;
    const uint32_t off = ev_off[e], ne = ev_off[e + 1] - off;
    const uint32_t i = t0 + threadIdx.x;
    const bool col = i < ne && key_collected(keys[off + i], kl);
    const uint64_t bal = __ballot(col);
    const uint32_t wave = threadIdx.x >> 6;
    if ((threadIdx.x & 63u) == 0)
        first_col[wave] = bal ? wave * 64u + (uint32_t)__builtin_ctzll(bal) : (uint32_t)kTile;
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t p = (uint32_t)kTile;  // first collected slot of the tile, from its start
        for (uint32_t w = 0; w < kTile / 64; ++w) p = min(p, first_col[w]);
        if (p < (uint32_t)kTile) {
            if (t0 == 0u || !key_collected(keys[off + t0 - 1u], kl)) ev_active[e] = t0 + p;
        } else if (t0 + (uint32_t)kTile >= ne) {
            ev_active[e] = ne;  // the event's last tile, and no key collected
        }
    }
}

hipError_t launch_gather_count(const uint64_t* keys, const uint32_t* ev_off,
                               const uint32_t* ev_tile, const uint32_t* tile_event,
                               uint32_t n_events, uint32_t n_tiles, KeyLayout kl, const double* x,
                               const double* y, const double* z, double* px, double* py,
                               double* pz, double* box, uint32_t stride, uint32_t* ev_active,
                               hipStream_t s) {
    if (n_tiles == 0) return launch_count(keys, ev_off, n_events, kl, ev_active, s);
    gather_count_tiles<<<n_tiles, kTile, 0, s>>>(keys, ev_off, ev_tile, tile_event, n_events, kl,
                                                 x, y, z, px, py, pz, box, stride, ev_active);
    return hipGetLastError();
}

hipError_t launch_gather(const uint64_t* keys, const uint32_t* ev_off, const uint32_t* ev_tile,
                         const uint32_t* tile_event, const uint32_t* ev_active, int sources_all,
                         uint32_t n_tiles, KeyLayout kl, const double* x, const double* y,
                         const double* z, double* px, double* py, double* pz, double* box,
                         uint32_t stride, hipStream_t s) {
    if (n_tiles == 0) return hipSuccess;
    gather_tiles<<<n_tiles, kTile, 0, s>>>(keys, ev_off, ev_tile, tile_event, ev_active,
                                           sources_all, kl, x, y, z, px, py, pz, box, stride);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Random diffusion vectors: Philox4x32-10 (Salmon, Moraes, Dror, Shaw, SC'11),
// ten rounds of two 32x32->64 multiplies whose high halves are XORed into the
// other words together with the round key; the key advances by two Weyl
// constants between rounds.  Counter = (carrier within its event, step,
// event, 0).
// ---------------------------------------------------------------------------
__device__ __forceinline__ void philox4x32_10(uint32_t& c0, uint32_t& c1, uint32_t& c2,
                                              uint32_t& c3, uint32_t k0, uint32_t k1) {
    constexpr uint32_t kMulA = 0xD2511F53u, kMulB = 0xCD9E8D57u;
    constexpr uint32_t kWeylA = 0x9E3779B9u, kWeylB = 0xBB67AE85u;
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        // one 32 x 32 -> 64-bit multiply-add instruction gives both halves
        const uint64_t pA = (uint64_t)kMulA * c0, pB = (uint64_t)kMulB * c2;
        // (0x96: the three-way XOR)
        const uint32_t n0 = __builtin_amdgcn_bitop3_b32((uint32_t)(pB >> 32), c1, k0, 0x96);
        const uint32_t n2 = __builtin_amdgcn_bitop3_b32((uint32_t)(pA >> 32), c3, k1, 0x96);
        c0 = n0;
        c1 = (uint32_t)pB;
        c2 = n2;
        c3 = (uint32_t)pA;
        k0 += kWeylA;
        k1 += kWeylB;
    }
}

__device__ __forceinline__ double unit_open(uint32_t w) {
    return ((double)w + 0.5) * (1.0 / 4294967296.0);
}

// ---------------------------------------------------------------------------
// One time step for every travelling hole (Sec. III.B, Fig. 2): static field
// (Eq. (1)) + Coulomb field (the chunk partials of field_tiles, summed in
// FP64 in chunk order), |E|, mobility (Eq. (2)), drift mu E dt, diffusion
// (Eqs. (3)-(4), Box-Muller on one Philox block), FP64 position update,
// mirror at the back surface, collection at the well.
//   list mode (Coulomb on): one thread per slot of the sorted list; every
//     carrier keeps its slot in the next (unsorted) list with its new key,
//     collected holes copying theirs through; the next sort restores order.
//   kept list (a.keep): a source tile per turn of a workgroup, one thread per slot.
//     The order stays, so no key is made or sorted: the step writes the slots' new
//     positions and its tile's boxes.  1,000 holes, latency-bound: 6.4 us.
//   carrier mode: drift_steps.
// ---------------------------------------------------------------------------
// The FP64 functions of the step (gccd_fp64.h).  Carrier mode (no
// repulsion) is bound by VALU issue and takes the three-operand Horner steps
// (one instruction fewer per step, at the cost of registers); list mode,
// which streams the partial sums, the compiler's own form, which needs
// fewer registers.
template <bool LIST>
__device__ __forceinline__ double exp_fin_s(double x) {
    return fp64::exp_fin<!LIST>(x);
}
template <bool LIST>
__device__ __forceinline__ double log_pos_s(double x) {
    return fp64::log_pos<!LIST>(x);
}
template <bool LIST>
__device__ __forceinline__ double log1p_fin_s(double x) {
    return fp64::log1p_fin<!LIST>(x);
}
template <bool LIST>
__device__ __forceinline__ void sincospi_s(double x, double* s, double* c) {
    fp64::sincospi<!LIST, true>(x, s, c);  // x in (0, 2)
}

// One step of one travelling hole at (x, y, z) in the Coulomb field (ecx, ecy,
// ecz): static field, mobility, drift, diffusion and the mirror at the back surface.
template <bool LIST>
__device__ __forceinline__ void move_hole(const StepArgs& a, uint32_t step, uint32_t e,
                                          uint32_t local, double ecx, double ecy, double ecz,
                                          double& x, double& y, double& z) {
    const double es = a.a1 * z - a.a2;
    const double ex = ecx, ey = ecy, ez = LIST ? ecz + es : es;
    double mu = a.mu0;
    if (a.mobility_model == 0) {
        // Eq. (2), mu0 / (1 + (|E|/Ec)^beta)^(1/beta), as
        // mu0 exp(-log1p(y) / beta) with y = exp(beta (log|E|^2 / 2
        // - log Ec)): four transcendentals instead of two general
        // powers and a square root.  The arguments are held in the
        // functions' finite ranges, so no special case is tested:
        // |E|^2 at or above 2^-1000 (|E| = 0 then gives a y far
        // below the rounding of 1 + y, so mu = mu0 exactly, as
        // y = 0 would), the exponents within [-745, 709]
        const double e2 = fmax(ex * ex + ey * ey + ez * ez, 0x1p-1000);
        const double ly = a.beta * (0.5 * log_pos_s<LIST>(e2) - a.log_ec);
        const double y = exp_fin_s<LIST>(fmin(fmax(ly, -745.0), 709.0));
        mu = a.mu0 * exp_fin_s<LIST>(fmax(-a.inv_beta * log1p_fin_s<LIST>(y), -745.0));
    }
    // v = mu E in cm/s; v dt in cm; 1 cm = 1e4 um.  Without
    // repulsion the field is the static one, along z only: no
    // lateral drift (mu 0 dt = +0 exactly)
    double dx = LIST ? mu * ex * a.dt_s * 1e4 : 0.0;
    double dy = LIST ? mu * ey * a.dt_s * 1e4 : 0.0;
    double dz = mu * ez * a.dt_s * 1e4;
    if (a.diffusion) {
        uint32_t w0 = local, w1 = step, w2 = a.event0 + e, w3 = 0u;
        philox4x32_10(w0, w1, w2, w3, a.key0, a.key1);
        // -2 ln u > 2^-33 for u on the open grid (w + 1/2) 2^-32
        const double r01 = fp64::sqrt_pos(-2.0 * log_pos_s<LIST>(unit_open(w0)));
        const double r23 = fp64::sqrt_pos(-2.0 * log_pos_s<LIST>(unit_open(w2)));
        // the angles 2 pi u in half-turns: 2 u is exact, and one
        // argument reduction serves both sine and cosine
        double s1, c1, s3, c3;
        sincospi_s<LIST>(2.0 * unit_open(w1), &s1, &c1);
        sincospi_s<LIST>(2.0 * unit_open(w3), &s3, &c3);
        (void)s3;
        const double D = a.vt * mu;                        // Eq. (4), cm^2/s
        // Eq. (3), um; 2 D dt > 0 (T > 0, dt > 0), held at or
        // above 2^-1000 so that the square root's estimate stays
        // in range even for a dt that underflows it
        const double s2 = fmax(2.0 * D * a.dt_s, 0x1p-1000);
        const double sigma = fp64::sqrt_pos(s2) * 1e4;
        dx += sigma * (r01 * c1);
        dy += sigma * (r01 * s1);
        dz += sigma * (r23 * c3);
    }
    x += dx;
    y += dy;
    z += dz;
    if (z > a.thickness) z = 2.0 * a.thickness - z;
}

constexpr int kDriftSum = 1024;
constexpr uint32_t kDriftAtomics = 256;

// The step's modes: list mode (a.list_mode, Coulomb on) leaving the new keys for
// a sort of their own, the same for a load whose sort counts places (kRankMax: no
// runs; latency-bound, so more loads in flight), or keeping the list's order
// (a.keep), one tile per workgroup or (kStepTurns) several in turns: the loop over
// them holds 51 more registers and takes 0.5 us more at 1000 holes.  Carrier mode is
// a kernel of its own (drift_steps).
constexpr int kStepList = 0, kStepShort = 1, kStepKept = 2, kStepTurns = 3;

template <int MODE>
__device__ __forceinline__ void step_body(const StepArgs& a) {
    constexpr bool KEEP = MODE == kStepKept || MODE == kStepTurns;
    const uint32_t step = a.step + (a.step_base ? *a.step_base : 0u);
    // travelling holes at the start of this step, of the next one, and the
    // counter of the step after next (cleared now; nobody reads it)
    const uint32_t* cnt_in = a.cnt_ring + step % 3u;
    uint32_t* cnt_out = a.cnt_ring + (step + 1u) % 3u;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        const unsigned long long holes = *cnt_in;
        a.cnt_ring[(step + 2u) % 3u] = 0u;
        if (holes > 0) {
            atomicAdd(&a.stats[0], holes);
            a.misc[1] = (int32_t)(step + 1u);
        }
    }
    const int lane = threadIdx.x & 63;
    uint32_t kept = 0;  // this wave's holes still travelling (wave-uniform)
    unsigned long long pairs = 0;  // this lane's pair interactions of Eq. (6)
    // a.sort_runs: each turn's kStepThreads slots leave their new
    // keys as one sorted run (sort_block_keys), which the next sort only
    // merges; else every slot leaves its key in place
    const bool runs = MODE == kStepList && a.sort_runs != 0;
    __shared__ uint64_t sk[kStepThreads];
    // KEEP: each turn takes one source tile, one slot per thread
    uint32_t te = 0u, toff = 0u, tne = a.n_all, ti = 0u;
    double px = 0.0, py = 0.0, pz = 0.0;  // KEEP: the slot's position
    const uint32_t turns = KEEP ? a.n_tiles : (a.n_all + kStepThreads - 1) / kStepThreads;
    for (uint32_t turn = blockIdx.x; turn < turns; turn += gridDim.x) {
        const uint32_t base = turn * kStepThreads;  // (not KEEP)
        if constexpr (KEEP) {
            ti = turn * kTile + threadIdx.x;
            if (!a.one_event) {
                te = a.tile_event[turn];
                toff = a.ev_off[te];
                tne = a.ev_off[te + 1] - toff;
                ti -= a.ev_tile[te] * kTile;
            }
        }
        const uint32_t slot = KEEP ? toff + ti : base + threadIdx.x;
        uint64_t run_key = ~0ull;  // this slot's new key, when the keys form runs
        bool keep = false;
        if (KEEP ? ti < tne : slot < a.n_all) {
            uint32_t e, j, local, src = 0u;
            bool active;
            uint64_t key = 0;
            if (KEEP) {
                px = a.px[slot];
                py = a.py[slot];
                pz = a.pz[slot];
            }
            {
                // the list may be some steps old (its travelling segment then
                // still holds the holes collected since): the
                // carrier's own collection step decides
                key = a.keys_in[slot];
                uint32_t off, ne;
                if (KEEP) {
                    e = te;
                    off = toff;
                    ne = tne;
                } else if (a.one_event) {
                    e = 0u;
                    off = 0u;
                    ne = a.n_all;
                } else {
                    e = key_event(key, a.kl);
                    off = a.ev_off[e];
                    ne = a.ev_off[e + 1] - off;
                }
                local = min(key_local(key, a.kl), ne - 1u);
                j = off + local;
                active = a.cstep[j] < 0;
                if (active) {
                    src = a.sources_all ? ne : a.ev_active[e];
                } else {
                    // collected in a step that kept the list
                    if ((runs || MODE == kStepShort) && !key_collected(key, a.kl))
                        key = make_key(e, true, a.x[j], a.y[j], a.z[j], local, a.kl);
                }
                if (!active && a.close && slot - off < a.ev_active[e]) {
                    // a target of the field launch collected since the list was sorted:
                    // its close-pair sums are not consumed, so cleared here
                    const size_t ps = a.pstride;
                    a.close[slot] = 0ull;
                    a.close[slot + ps] = 0ull;
                    a.close[slot + 2 * ps] = 0ull;
                }
            }
            if (active) {
                pairs += src;  // sources of the Eq. (6) sum at this target
                double ecx = 0.0, ecy = 0.0, ecz = 0.0;
                if (a.coulomb) {
                    double sx = 0.0, sy = 0.0, sz = 0.0;
                    const int nchunk = a.ev_chunks[e];
                    const float* pp = a.part + slot;
                    const size_t ps = a.pstride;
                    int c = 0;
                    // eight (a small load, latency-bound: sixteen), then four
                    // groups' loads in flight ahead of their adds (the adds in
                    // group order)
                    constexpr int kW = MODE == kStepList ? 8 : 16;
                    for (; c + kW <= nchunk; c += kW) {
                        float v[kW][3];
#pragma unroll
                        for (int u = 0; u < kW; ++u)
#pragma unroll
                            for (int d = 0; d < 3; ++d) v[u][d] = pp[(size_t)((c + u) * 3 + d) * ps];
#pragma unroll
                        for (int u = 0; u < kW; ++u) {
                            sx += (double)v[u][0];
                            sy += (double)v[u][1];
                            sz += (double)v[u][2];
                        }
                    }
                    if (kW > 8 && c + 8 <= nchunk) {
                        float v[8][3];
#pragma unroll
                        for (int u = 0; u < 8; ++u)
#pragma unroll
                            for (int d = 0; d < 3; ++d) v[u][d] = pp[(size_t)((c + u) * 3 + d) * ps];
#pragma unroll
                        for (int u = 0; u < 8; ++u) {
                            sx += (double)v[u][0];
                            sy += (double)v[u][1];
                            sz += (double)v[u][2];
                        }
                        c += 8;
                    }
                    for (; c + 4 <= nchunk; c += 4) {
                        float v[4][3];
#pragma unroll
                        for (int u = 0; u < 4; ++u)
#pragma unroll
                            for (int d = 0; d < 3; ++d) v[u][d] = pp[(size_t)((c + u) * 3 + d) * ps];
#pragma unroll
                        for (int u = 0; u < 4; ++u) {
                            sx += (double)v[u][0];
                            sy += (double)v[u][1];
                            sz += (double)v[u][2];
                        }
                    }
                    for (; c < nchunk; ++c) {
                        sx += (double)pp[(size_t)(c * 3 + 0) * ps];
                        sy += (double)pp[(size_t)(c * 3 + 1) * ps];
                        sz += (double)pp[(size_t)(c * 3 + 2) * ps];
                    }
                    if (a.close) {
                        // the exactly summed close pairs, cleared for the next launch
                        unsigned long long* cp = a.close + slot;
                        const long long cx = (long long)cp[0], cy = (long long)cp[ps],
                                        cz = (long long)cp[2 * ps];
                        if ((cx | cy | cz) != 0ll) {
                            sx += (double)cx * a.close_unit;
                            sy += (double)cy * a.close_unit;
                            sz += (double)cz * a.close_unit;
                            cp[0] = 0ull;
                            cp[ps] = 0ull;
                            cp[2 * ps] = 0ull;
                        }
                    }
                    ecx = a.K * sx;
                    ecy = a.K * sy;
                    ecz = a.K * sz;
                }
                double xn = KEEP ? px : a.x[j], yn = KEEP ? py : a.y[j],
                       zn = KEEP ? pz : a.z[j];
                move_hole<true>(a, step, e, local, ecx, ecy, ecz, xn, yn, zn);
                a.x[j] = xn;
                a.y[j] = yn;
                a.z[j] = zn;
                if (!isfinite(xn) || !isfinite(yn) || !isfinite(zn)) atomicOr(&a.misc[0], 1);
                const bool collected = zn <= a.z_well;
                if (collected) a.cstep[j] = (int32_t)(step + 1u);
                keep = !collected;
                if (KEEP) {
                    a.px[slot] = px = xn;
                    a.py[slot] = py = yn;
                    a.pz[slot] = pz = zn;
                } else {
                    key = make_key(e, collected, xn, yn, zn, local, a.kl);
                }
            }
            if (runs)
                run_key = key;
            else if (!KEEP)
                a.keys_out[slot] = key;
        }
        kept += (uint32_t)__popcll(__ballot(keep));
        if constexpr (KEEP) {
            __shared__ double red[6][kTile / 64];
            tile_boxes(turn, threadIdx.x, ti < tne, px, py, pz, a.tile_box, a.box_stride, red);
            if constexpr (MODE == kStepKept) break;
            __syncthreads();  // red is written again
        }
        if (runs) {  // uniform: every thread of the workgroup takes each turn
            const uint32_t m = min((uint32_t)kStepThreads, a.n_all - base);
            const uint64_t sorted = sort_block_keys(run_key, m, sk);
            if (threadIdx.x < m) a.keys_out[base + threadIdx.x] = sorted;
        }
    }
    // one atomic per workgroup for each count: a counter taking one per wave
    // and grid-stride turn (2.6e5 at 2^24 holes) serialised the whole step
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) pairs += __shfl_xor(pairs, m);
    __shared__ uint32_t wave_kept[kStepThreads / 64];
    __shared__ unsigned long long wave_pairs[kStepThreads / 64];
    if (lane == 0) {
        wave_kept[threadIdx.x >> 6] = kept;
        wave_pairs[threadIdx.x >> 6] = pairs;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t t = 0;
        unsigned long long pr = 0;
        for (int w = 0; w < kStepThreads / 64; ++w) {
            t += wave_kept[w];
            pr += wave_pairs[w];
        }
        if (t) atomicAdd(cnt_out, t);
        if (pr && a.coulomb) atomicAdd(&a.stats[1], pr);
    }
}

template <int MODE>
__global__ __launch_bounds__(kStepThreads) void step_update(StepArgs a) {
    step_body<MODE>(a);
}

// The counts of a workgroup's lanes (missed, last) and waves (gone, the same in every
// lane), left in *out or, where that is NULL, added to the load's.
__device__ __forceinline__ void add_drift_counts(const StepArgs& a, DriftCounts c,
                                                 DriftCounts* out) {
    __shared__ DriftCounts wave[kDriftSum / 64];
    if (c.gone) {  // wave-uniform
#pragma unroll
        for (int m = 32; m >= 1; m >>= 1) {
            c.missed += __shfl_xor(c.missed, m);
            c.last = max(c.last, (uint32_t)__shfl_xor((int)c.last, m));
        }
    }
    if ((threadIdx.x & 63u) == 0) wave[threadIdx.x >> 6] = c;
    __syncthreads();
    if (threadIdx.x != 0) return;
    for (uint32_t w = 1; w < blockDim.x / 64u; ++w) {
        c.missed += wave[w].missed;
        c.last = max(c.last, wave[w].last);
        c.gone += wave[w].gone;
    }
    if (out) {
        *out = c;
        return;
    }
    // every hole that travelled at the start counts as moved in every step
    if (blockIdx.x == 0) atomicAdd(&a.stats[0], a.holes * a.n_steps);
    if (c.gone) {
        atomicAdd(&a.stats[0], 0ull - c.missed);
        atomicMax(reinterpret_cast<uint32_t*>(&a.misc[1]), a.step + c.last);
        atomicSub(a.cnt_ring, c.gone);
    }
}

// a.n_steps steps without repulsion: holes do not see each other, so each
// stays in its thread's registers over all of them.  Bound by VALU issue: about
// 300 FP64 instructions per hole and step.  One launch per step read and wrote
// 52 B per hole each time and stopped at the launch's end: 8 million holes
// 207 us per step, now 104; 1,000 holes 4.4 us, now 1.5.
__global__ __launch_bounds__(kStepThreads) void drift_steps(StepArgs a) {
    unsigned long long missed = 0;  // of this lane's collected holes: steps after that,
    uint32_t last = 0;              // and the last one's step
    uint32_t gone = 0;              // holes collected (wave)
    for (uint32_t base = blockIdx.x * kStepThreads; base < a.n_all;
         base += gridDim.x * kStepThreads) {
        const uint32_t j = base + threadIdx.x;
        const bool was = j < a.n_all && a.cstep[j] < 0;
        if (!__any(was)) continue;
        uint32_t e = 0u, local = j;
        double x = 0.0, y = 0.0, z = 0.0;
        if (was) {
            if (!a.one_event) {
                e = a.ev_of[j];
                local = j - a.ev_off[e];
            }
            x = a.x[j];
            y = a.y[j];
            z = a.z[j];
        }
        bool active = was;
        uint32_t done = 0;  // steps in which this hole travelled
        for (uint32_t i = 0; i < a.n_steps && __any(active); ++i) {
            if (active) {
                move_hole<false>(a, a.step + i, e, local, 0.0, 0.0, 0.0, x, y, z);
                ++done;
                active = !(z <= a.z_well);
            }
        }
        if (was) {
            a.x[j] = x;
            a.y[j] = y;
            a.z[j] = z;
            // a coordinate once infinite or NaN never becomes finite again
            if (!isfinite(x) || !isfinite(y) || !isfinite(z)) atomicOr(&a.misc[0], 1);
            if (!active) {
                a.cstep[j] = (int32_t)(a.step + done);
                missed += a.n_steps - done;
                last = max(last, done);
            }
        }
        gone += (uint32_t)__popcll(__ballot(was && !active));
    }
    add_drift_counts(a, DriftCounts{missed, last, gone},
                     a.counts ? a.counts + blockIdx.x : nullptr);
}

// The sum of the workgroups' counts.
__global__ __launch_bounds__(kDriftSum) void drift_counts(StepArgs a, uint32_t n_counts) {
    DriftCounts c{0ull, 0u, 0u};
#pragma unroll 4
    for (uint32_t i = threadIdx.x; i < n_counts; i += kDriftSum) {
        c.missed += a.counts[i].missed;
        c.last = max(c.last, a.counts[i].last);
        c.gone += a.counts[i].gone;
    }
    // add_drift_counts takes a wave's `gone` from its first lane
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) c.gone += (uint32_t)__shfl_xor((int)c.gone, m);
    add_drift_counts(a, c, nullptr);
}

hipError_t launch_step(const StepArgs& a, uint32_t n_slots, hipStream_t s) {
    static_assert(kTile == kStepThreads, "a turn of a kept step takes one source tile");
    if (a.keep) {
        if (!a.list_mode || !a.sources_all || a.n_tiles == 0) return hipErrorInvalidValue;
        // The workgroups' atomics on the same two words queue up (24 ns per workgroup):
        // 6553 events of 10 holes, a tile each, take 198 us per step in as many
        // workgroups, 109 in 512 (154 in 256, 112 in 1024); 1700 events of 1000 holes
        // 880, 849 (889, 862).
        constexpr uint32_t kMax = 512;
        if (a.n_tiles <= kMax)
            step_update<kStepKept><<<a.n_tiles, kStepThreads, 0, s>>>(a);
        else
            step_update<kStepTurns><<<kMax, kStepThreads, 0, s>>>(a);
    } else if (a.list_mode && n_slots <= kRankMax) {
        step_update<kStepShort>
            <<<(n_slots + kStepThreads - 1) / kStepThreads, kStepThreads, 0, s>>>(a);
    } else if (a.list_mode) {
        step_update<kStepList>
            <<<grid_for(n_slots, kStepThreads, 16384), kStepThreads, 0, s>>>(a);
    } else {
        const uint32_t grid = grid_for(n_slots, kStepThreads, 16384);
        StepArgs d = a;
        // Atomics of many workgroups on the same words queue up (8 ns each): with
        // a set per workgroup a single step of 8 million holes took 755 us.  Above
        // kDriftAtomics workgroups each leaves its counts in memory and a second
        // launch (6 us) adds them: 157 us.
        if (grid <= kDriftAtomics) d.counts = nullptr;
        drift_steps<<<grid, kStepThreads, 0, s>>>(d);
        if (d.counts) drift_counts<<<1, kDriftSum, 0, s>>>(d, grid);
    }
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Taking in a load: the caller's positions copied with z mirrored at the back
// surface, holes at or below the well collected (collection step 0), each
// carrier's event recorded and the travelling ones counted; with repulsion
// also the unsorted list key and the zeroed close sums (LoadArgs).  One pass
// at HBM rate in place of three copies, the boundary pass, the key pass and a
// fill: per carrier 24 B read and 32 B written, 64 B with repulsion (before:
// 128 and 176 B in all).  gccd_load of 8 million holes without repulsion takes
// 141 us in all, most of it this kernel (before, with the allocations: 4.1 ms).
// ---------------------------------------------------------------------------
// LIST: keys and close sums too.  ONE: one event, whose tables are not read (they
// are written by the same launch), and no count.
template <bool LIST, bool ONE>
__device__ __forceinline__ void load_body(const LoadArgs& a) {
    const int lane = threadIdx.x & 63;
    uint32_t kept = 0;  // this wave's travelling holes (wave-uniform)
    for (uint32_t base = blockIdx.x * kStepThreads; base < a.n;
         base += gridDim.x * kStepThreads) {
        const uint32_t j = base + threadIdx.x;
        bool keep = false;
        if (j < a.n) {
            const double xx = a.sx[j], yy = a.sy[j];
            double zz = a.sz[j];
            if (zz > a.thickness) zz = 2.0 * a.thickness - zz;
            a.x[j] = xx;
            a.y[j] = yy;
            a.z[j] = zz;
            const bool collected = zz <= a.z_well;
            a.cstep[j] = collected ? 0 : -1;
            keep = !collected;
            const uint32_t e = ONE ? 0u : event_of(a.ev_off, a.n_events, j);
            a.ev_of[j] = e;
            if constexpr (LIST) {
                a.keys[j] =
                    make_key(e, collected, xx, yy, zz, ONE ? j : j - a.ev_off[e], a.kl);
                a.close[j] = 0ull;
                a.close[(size_t)a.n + j] = 0ull;
                a.close[2 * (size_t)a.n + j] = 0ull;
            }
        }
        kept += (uint32_t)__popcll(__ballot(keep));
    }
    if constexpr (!ONE) {  // one atomic per workgroup, as in step_update
        __shared__ uint32_t wave_kept[kStepThreads / 64];
        if (lane == 0) wave_kept[threadIdx.x >> 6] = kept;
        __syncthreads();
        if (threadIdx.x == 0) {
            uint32_t t = 0;
            for (int w = 0; w < kStepThreads / 64; ++w) t += wave_kept[w];
            if (t) atomicAdd(a.cnt, t);
        }
    }
}

template <bool LIST>
__global__ __launch_bounds__(kStepThreads) void load_prepare(LoadArgs a) {
    load_body<LIST, false>(a);
}

// Taking in a load of one event of at most kSmallLoad holes with its sorted list,
// by one workgroup: what load_prepare, the counted sort and gather_count_tiles do
// in three launches, whose latency is all that such a load costs.  Each wave sorts
// its 64 keys by counting the smaller ones; a key's place is then the number of
// smaller keys of every run, by binary searches side by side.  Each half of the
// workgroup takes one source tile.  gccd_field_noalloc called without waiting, 64
// holes 24 -> 18 us, 300 23.5 -> 20.9, 512 24 -> 23.  (Counting a key's smaller ones over
// the whole list on the one compute unit: 512 holes 29 to 33.)
__device__ __forceinline__ void small_load_body(const LoadArgs& a) {
    __shared__ uint64_t keys[kSmallLoad];
    __shared__ uint16_t from[kSmallLoad];
    __shared__ double pos[3][kSmallLoad];
    __shared__ double red[kSmallLoad / kTile][6][kTile / 64];
    __shared__ uint32_t travelling;
    const uint32_t tid = threadIdx.x, n = a.n;
    if (tid == 0) travelling = 0u;
    double xx = 0.0, yy = 0.0, zz = 0.0;
    bool keep = false;
    if (tid < n) {
        xx = a.sx[tid];
        yy = a.sy[tid];
        zz = a.sz[tid];
        if (zz > a.thickness) zz = 2.0 * a.thickness - zz;
        a.x[tid] = pos[0][tid] = xx;
        a.y[tid] = pos[1][tid] = yy;
        a.z[tid] = pos[2][tid] = zz;
        keep = !(zz <= a.z_well);
        a.cstep[tid] = keep ? -1 : 0;
        a.ev_of[tid] = 0u;
        a.close[tid] = 0ull;
        a.close[(size_t)n + tid] = 0ull;
        a.close[2 * (size_t)n + tid] = 0ull;
    }
    // (past the load: distinct keys above every other)
    const uint64_t key =
        tid < n ? make_key(0u, !keep, xx, yy, zz, tid, a.kl) : ~0ull - (kSmallLoad - tid);
    const uint32_t run = tid & ~63u;
    uint32_t below = 0u;
#pragma unroll 16
    for (int u = 0; u < 64; ++u) {
        const uint64_t k =
            (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(key >> 32), u) << 32 |
            (uint32_t)__builtin_amdgcn_readlane((int)key, u);
        below += k < key ? 1u : 0u;
    }
    keys[run + below] = key;
    __syncthreads();
    const uint32_t kept = (uint32_t)__popcll(__ballot(keep));
    if ((tid & 63u) == 0 && kept) atomicAdd(&travelling, kept);
    constexpr uint32_t kRuns = kSmallLoad / 64;
    uint32_t at[kRuns] = {};
#pragma unroll
    for (uint32_t step = 32u; step >= 1u; step >>= 1) {
#pragma unroll
        for (uint32_t q = 0; q < kRuns; ++q)
            at[q] += keys[q * 64u + at[q] + step - 1u] < key ? step : 0u;
    }
    uint32_t place = 0u;
#pragma unroll
    for (uint32_t q = 0; q < kRuns; ++q) place += at[q] + (keys[q * 64u + at[q]] < key ? 1u : 0u);
    if (tid < n) {
        a.sorted[place] = key;
        from[place] = (uint16_t)tid;
    }
    __syncthreads();
    double px = 0.0, py = 0.0, pz = 0.0;
    if (tid < n) {
        const uint32_t i = from[tid];
        a.px[tid] = px = pos[0][i];
        a.py[tid] = py = pos[1][i];
        a.pz[tid] = pz = pos[2][i];
    }
    const uint32_t active = travelling, g = tid / kTile, tiles = (n + kTile - 1) / kTile;
    // (without a second tile the upper half writes no boxes)
    tile_boxes(g, tid % kTile, tid < n && (a.sources_all || tid < active), px, py, pz, a.box,
               a.box_stride, red[g], g < tiles);
    if (tid == 0) {
        a.ev_active[0] = active;
        if (a.cnt && active) atomicAdd(a.cnt, active);
    }
}

__global__ __launch_bounds__(kSmallLoad) void small_load(LoadArgs a) { small_load_body(a); }

hipError_t launch_small_load(const LoadArgs& a, hipStream_t s) {
    if (a.n == 0 || a.n > (uint32_t)kSmallLoad || a.n_events != 1u) return hipErrorInvalidValue;
    small_load<<<1, kSmallLoad, 0, s>>>(a);
    return hipGetLastError();
}

hipError_t launch_load(const LoadArgs& a, hipStream_t s) {
    const auto grid = grid_for(a.n, kStepThreads, 8192);
    if (a.keys)
        load_prepare<true><<<grid, kStepThreads, 0, s>>>(a);
    else
        load_prepare<false><<<grid, kStepThreads, 0, s>>>(a);
    return hipGetLastError();
}

__global__ void fill_u32(uint32_t* p, uint64_t n, uint32_t v) {
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (uint64_t)gridDim.x * blockDim.x)
        p[i] = v;
}

hipError_t launch_fill_u32(uint32_t* p, uint64_t n, uint32_t v, hipStream_t s) {
    if (n == 0) return hipSuccess;
    fill_u32<<<grid_for(n, 256, 4096), 256, 0, s>>>(p, n, v);
    return hipGetLastError();
}

// Coulomb field of every carrier for gccd_field: chunk partials summed in
// FP64 in chunk order, times K (same reduction as step_update), written back
// to the carrier each slot holds.
__global__ void field_finish(const float* part, uint32_t pstride, const int32_t* ev_chunks,
                             int g0, int groups, const uint64_t* keys, const uint32_t* ev_off,
                             KeyLayout kl, uint32_t n, double K, unsigned long long* close,
                             double close_unit, double* ex, double* ey, double* ez) {
    for (uint32_t slot = blockIdx.x * blockDim.x + threadIdx.x; slot < n;
         slot += gridDim.x * blockDim.x) {
        const uint64_t key = keys[slot];
        const uint32_t e = key_event(key, kl);
        const uint32_t off = ev_off[e], ne = ev_off[e + 1] - off;
        const uint32_t j = off + min(key_local(key, kl), ne - 1u);
        double sx = 0.0, sy = 0.0, sz = 0.0;
        const int g1 = g0 + (groups > 0 ? groups : ev_chunks[e]);
        for (int c = g0; c < g1; ++c) {
            sx += (double)part[(size_t)(c * 3 + 0) * pstride + slot];
            sy += (double)part[(size_t)(c * 3 + 1) * pstride + slot];
            sz += (double)part[(size_t)(c * 3 + 2) * pstride + slot];
        }
        if (close) {
            unsigned long long* cp = close + slot;
            const long long cx = (long long)cp[0], cy = (long long)cp[pstride],
                            cz = (long long)cp[2 * (size_t)pstride];
            if ((cx | cy | cz) != 0ll) {
                sx += (double)cx * close_unit;
                sy += (double)cy * close_unit;
                sz += (double)cz * close_unit;
                cp[0] = 0ull;
                cp[pstride] = 0ull;
                cp[2 * (size_t)pstride] = 0ull;
            }
        }
        ex[j] = K * sx;
        ey[j] = K * sy;
        ez[j] = K * sz;
    }
}

hipError_t launch_field_finish(const float* part, uint32_t pstride, const int32_t* ev_chunks,
                               int g0, int groups, const uint64_t* keys, const uint32_t* ev_off,
                               KeyLayout kl, uint32_t n, double K, unsigned long long* close,
                               double close_unit, double* ex, double* ey, double* ez,
                               hipStream_t s) {
    field_finish<<<grid_for(n, 256, 8192), 256, 0, s>>>(part, pstride, ev_chunks, g0, groups, keys,
                                                         ev_off, kl, n, K, close, close_unit, ex,
                                                         ey, ez);
    return hipGetLastError();
}

// The per-call state of gccd_field_noalloc (one event of n holes, t tiles,
// `blocks` target blocks, g chunks of which the last `tail` form the tail
// layer from tile `split`), written in its scratch memory: event tables,
// zeroed counters, and the work items in the order the context's item builder
// lists them for one event; and, in the same launch, its holes (load_body).
template <bool SMALL>
__global__ __launch_bounds__(SMALL ? kSmallLoad : kStepThreads) void noalloc_setup(
    LoadArgs la, uint32_t tiles, int32_t g, int32_t tail, uint32_t split, uint32_t blocks,
    uint32_t* ev_off, uint32_t* ev_tile, int32_t* ev_chunks, uint32_t* tile_event, uint32_t* words,
    uint32_t n_words, FieldItem* items) {
    if (SMALL)
        small_load_body(la);
    else
        load_body<true, true>(la);
    const uint64_t i0 = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    if (i0 == 0) {
        ev_off[0] = 0u;
        ev_off[1] = la.n;
        ev_tile[0] = 0u;
        ev_tile[1] = tiles;
        ev_chunks[0] = g;
    }
    for (uint64_t i = i0; i < n_words; i += stride) words[i] = 0u;
    for (uint64_t i = i0; i < tiles; i += stride) tile_event[i] = 0u;
    const uint32_t s1 = (uint32_t)(g - tail), s2 = (uint32_t)tail;
    const uint64_t first = (uint64_t)blocks * s1, total = first + (uint64_t)blocks * s2;
    for (uint64_t k = i0; k < total; k += stride) {
        FieldItem it;
        it.event = 0u;
        it.groups = (uint32_t)g;
        it.pad = 0u;
        if (k < first) {
            const uint32_t b = (uint32_t)(k / s1), q = (uint32_t)((k % s1 + b) % s1);
            it.blk = b;
            it.group = q;
            it.first = q;
            it.end = s2 ? split : kTilesToEnd;
            it.step = s1;
        } else {
            const uint64_t kk = k - first;
            const uint32_t b = (uint32_t)(kk / s2), q = (uint32_t)((kk % s2 + b) % s2);
            it.blk = b;
            it.group = s1 + q;
            it.first = split + q;
            it.end = kTilesToEnd;
            it.step = s2;
        }
        items[k] = it;
    }
}

hipError_t launch_noalloc_setup(const LoadArgs& la, uint32_t tiles, int32_t g, int32_t tail,
                                uint32_t split, uint32_t blocks, uint32_t* ev_off,
                                uint32_t* ev_tile, int32_t* ev_chunks, uint32_t* tile_event,
                                uint32_t* words, uint32_t n_words, FieldItem* items,
                                hipStream_t s) {
    if (la.sorted)
        noalloc_setup<true><<<1, kSmallLoad, 0, s>>>(la, tiles, g, tail, split, blocks, ev_off,
                                                     ev_tile, ev_chunks, tile_event, words, n_words,
                                                     items);
    else
        noalloc_setup<false><<<grid_for(la.n, kStepThreads, 1024), kStepThreads, 0, s>>>(
            la, tiles, g, tail, split, blocks, ev_off, ev_tile, ev_chunks, tile_event, words,
            n_words, items);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Sec. V.A image: half-open pixels, index floor((x - x0) / pitch) in IEEE
// FP64 (correctly rounded division), integer atomics into the caller's grid:
// one grid for all events, or one per event (per_event).
// ---------------------------------------------------------------------------
__global__ void image_bin(const double* x, const double* y, const int32_t* cstep,
                          const uint32_t* ev_of, uint32_t n, int per_event, double x0, double y0,
                          double pitch, int32_t nx, int32_t ny, uint32_t* counts,
                          unsigned long long* n_out) {
    for (uint32_t j = blockIdx.x * blockDim.x + threadIdx.x; j < n; j += gridDim.x * blockDim.x) {
        if (cstep[j] < 0) continue;
        const uint64_t e = per_event ? (uint64_t)ev_of[j] : 0ull;
        const double fx = floor((x[j] - x0) / pitch);
        const double fy = floor((y[j] - y0) / pitch);
        if (fx >= 0.0 && fx < (double)nx && fy >= 0.0 && fy < (double)ny) {
            atomicAdd(&counts[e * (uint64_t)nx * (uint64_t)ny + (uint64_t)fy * nx + (uint64_t)fx],
                      1u);
        } else {
            atomicAdd(&n_out[e], 1ull);
        }
    }
}

hipError_t launch_image(const double* x, const double* y, const int32_t* cstep,
                        const uint32_t* ev_of, uint32_t n, int per_event, double x0, double y0,
                        double pitch, int32_t nx, int32_t ny, uint32_t* counts,
                        unsigned long long* n_out, hipStream_t s) {
    image_bin<<<grid_for(n, 256, 8192), 256, 0, s>>>(x, y, cstep, ev_of, n, per_event, x0, y0,
                                                      pitch, nx, ny, counts, n_out);
    return hipGetLastError();
}

}  // namespace gccd
