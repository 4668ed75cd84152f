// Sorting of the 64-bit carrier keys that order the Eq. (6) targets
// spatially (the keys are unique, so every correct sort gives the same
// list).  Written for this list:
//   rank_sort   -- up to kRankMax keys, one launch: every key's place counted;
//   block_sort  -- each workgroup sorts a tile of up to kSortTile keys
//                  (register sorts of kSortItems keys, then merge levels in
//                  LDS), giving sorted runs of kSortTile;
//   merge_all   -- up to kMergeRuns of those runs merged in one launch;
//   merge_runs  -- longer lists, one launch per level that doubles the run
//                  length: each
//                  workgroup writes kSortTile consecutive outputs of one
//                  merged pair of runs, locating its share of both runs by a
//                  64-way search (one wave per end of its output range) and
//                  merging it out of LDS, kSortItems outputs per thread.
// The counting and the searches of merge_all grow with the square of the list
// but take one launch, where the latency of a launch and of the levels within a
// workgroup sets the time of a short list.  us between events around the
// sort (6.2 of them the events' own), merge sort alone / with the short forms:
// 300 keys 15.0 / 6.2, 2048 21.0 / 6.8, 10007 39.9 / 17.3, 12288 40.4 / 19.8 (counted;
// 33.8 merged), 16384 41.0 / 33.9 (28.7 if counted, but 24.1 where the keys come in
// runs of 256, as a step leaves them), 20011 48.8 / 34.4 (40.2 if counted), 50000
// 58.5 / 46.1, 65536 58.4 / 43.3; 1e5 keys take one launch plus five levels, 67.
// The kernels only read and write the two key buffers (no
// memory-set commands, no temporary storage, no host synchronisation), so a
// sequence of steps that sorts can be captured in a HIP graph.
#include "gccd_sort_dev.h"

namespace gccd {

constexpr int kSortThreads = 512;
constexpr uint32_t kSortTile = kSortThreads * kSortItems;  // 4096

// One tile of T = THREADS * kSortItems keys per workgroup, sorted in LDS
// (block_sort_lds; with run0 > 0 the tile's runs of run0 keys are already
// sorted and only merged, merge_sorted_runs); loads and stores of global
// memory are coalesced.
template <int THREADS>
__global__ __launch_bounds__(THREADS) void block_sort(const uint64_t* in, uint64_t* out,
                                                      uint32_t n, uint32_t run0) {
    constexpr uint32_t T = (uint32_t)THREADS * kSortItems;
    __shared__ uint64_t s[T + T / kSortItems];
    const uint32_t b0 = blockIdx.x * T;
    const uint32_t cnt = min(T, n - b0);
    if (run0 != 0u)
        merge_sorted_runs<THREADS>(in + b0, cnt, s, min(run0, T));
    else
        block_sort_lds<THREADS>(in + b0, cnt, s);
    for (uint32_t i = threadIdx.x; i < cnt; i += THREADS) out[b0 + i] = s[lds_slot(i)];
}

// Of the first k outputs of merging A[0, la) and B[0, lb) (sorted, no key in
// both), the number taken from A: the least i in [max(0, k - lb), min(k, la)]
// with i == min(k, la) or A[i] > B[k - 1 - i].  Every lane of the wave calls
// it with the same arguments and gets the same answer; each round tests 64
// candidates (two loads per lane) and keeps the interval between the last
// that fails and the first that holds.
__device__ uint32_t merge_split(const uint64_t* A, uint32_t la, const uint64_t* B, uint32_t lb,
                                uint32_t k) {
    uint32_t lo = k > lb ? k - lb : 0u;
    uint32_t hi = min(k, la);
    const uint32_t lane = threadIdx.x & 63u;
    while (hi > lo) {
        const uint32_t span = hi - lo;
        uint32_t m;
        bool valid;
        if (span <= 64u) {
            m = lo + lane;
            valid = lane < span;
        } else {
            m = lo + (uint32_t)(((uint64_t)span * (lane + 1u)) / 65u);
            valid = true;
        }
        // m < hi <= la and k - 1 - m < lb for every valid candidate
        const bool holds = valid && A[m] > B[k - 1u - m];
        const uint64_t bal = __ballot(holds);
        if (span <= 64u) {
            lo = bal ? lo + (uint32_t)__builtin_ctzll(bal) : hi;
            break;
        }
        const uint32_t f = bal ? (uint32_t)__builtin_ctzll(bal) : 64u;
        const uint32_t mf = __shfl(m, (int)min(f, 63u));
        const uint32_t mb = __shfl(m, (int)(f > 0u ? f - 1u : 0u));
        if (f < 64u) hi = mf;
        if (f > 0u) lo = mb + 1u;
    }
    return lo;
}

// One merge level: runs of width w in `in` become runs of 2 w in `out`.
__global__ __launch_bounds__(kSortThreads) void merge_runs(const uint64_t* in, uint64_t* out,
                                                          uint32_t n, uint32_t w) {
    __shared__ uint64_t buf[kSortTile + kSortTile / kSortItems];
    __shared__ uint32_t cut[2];
    const uint64_t o0 = (uint64_t)blockIdx.x * kSortTile;  // first output of the workgroup
    const uint64_t base = o0 / (2ull * w) * (2ull * w);    // its pair of runs starts here
    const uint32_t la = (uint32_t)min<uint64_t>(w, n - base);
    const uint32_t lb = n - base > w ? (uint32_t)min<uint64_t>(w, n - base - w) : 0u;
    const uint64_t* A = in + base;
    const uint64_t* B = A + la;
    const uint32_t k0 = (uint32_t)(o0 - base);
    const uint32_t k1 = min(k0 + kSortTile, la + lb);
    const uint32_t wave = threadIdx.x >> 6;
    if (wave < 2) {
        const uint32_t k = wave == 0 ? k0 : k1;
        const uint32_t i = merge_split(A, la, B, lb, k);
        if ((threadIdx.x & 63u) == 0) cut[wave] = i;
    }
    __syncthreads();
    const uint32_t i0 = cut[0], i1 = cut[1];
    const uint32_t na = i1 - i0, nb = (k1 - i1) - (k0 - i0);
    for (uint32_t t = threadIdx.x; t < na + nb; t += kSortThreads)
        buf[t] = t < na ? A[i0 + t] : B[k0 - i0 + (t - na)];
    __syncthreads();
    // outputs [kt, kt + kSortItems) of this workgroup's share, merged into
    // registers, then stored through LDS so that the global stores coalesce
    const uint32_t kt = threadIdx.x * kSortItems;
    const uint32_t nk = na + nb;
    uint64_t v[kSortItems];
    if (kt < nk) {
        const uint64_t* a = buf;
        const uint64_t* b = buf + na;
        uint32_t lo = kt > nb ? kt - nb : 0u, hi = min(kt, na);
        while (lo < hi) {
            const uint32_t mid = (lo + hi) >> 1;
            if (a[mid] > b[kt - 1u - mid])
                hi = mid;
            else
                lo = mid + 1u;
        }
        uint32_t ia = lo, ib = kt - lo;
#pragma unroll
        for (uint32_t e = 0; e < (uint32_t)kSortItems; ++e) {
            if (kt + e < nk) {
                const bool take_a = ib >= nb || (ia < na && a[ia] < b[ib]);
                v[e] = take_a ? a[ia++] : b[ib++];
            }
        }
    }
    __syncthreads();  // every read of buf is done
    if (kt < nk) {
#pragma unroll
        for (uint32_t e = 0; e < (uint32_t)kSortItems; ++e)
            if (kt + e < nk) buf[lds_slot(kt + e)] = v[e];
    }
    __syncthreads();
    uint64_t* o = out + base + k0;
    for (uint32_t t = threadIdx.x; t < nk; t += kSortThreads) o[t] = buf[lds_slot(t)];
}

// A short list in one launch: every key's place is the number of smaller keys.
// A workgroup places kRankKeys keys, held as scalars: its waves take 64 keys of the
// list at a time, one per lane, and count the lanes whose key is smaller.
constexpr int kRankWaves = 8;
constexpr uint32_t kRankKeys = 16;

__global__ __launch_bounds__(64 * kRankWaves) void rank_sort(const uint64_t* __restrict__ in,
                                                             uint64_t* __restrict__ out,
                                                             uint32_t n) {
    __shared__ uint32_t part[kRankWaves][kRankKeys];
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const uint32_t i0 = blockIdx.x * kRankKeys;
    uint64_t key[kRankKeys];
    uint32_t below[kRankKeys];
#pragma unroll
    for (uint32_t u = 0; u < kRankKeys; ++u) {
        key[u] = in[min(i0 + u, n - 1u)];
        below[u] = 0;
    }
    for (uint32_t j = wave * 64u; j < n; j += 64u * kRankWaves) {
        const uint64_t k = j + lane < n ? in[j + lane] : ~0ull;
#pragma unroll
        for (uint32_t u = 0; u < kRankKeys; ++u) below[u] += (uint32_t)__popcll(__ballot(k < key[u]));
    }
#pragma unroll
    for (uint32_t u = 0; u < kRankKeys; ++u)
        if (lane == u) part[wave][u] = below[u];
    __syncthreads();
    if (threadIdx.x < kRankKeys && i0 + threadIdx.x < n) {
        uint32_t r = 0;
#pragma unroll
        for (int w = 0; w < kRankWaves; ++w) r += part[w][threadIdx.x];
        out[r] = in[i0 + threadIdx.x];
    }
}

// Up to kMergeRuns sorted runs of kSortTile keys merged in one launch: a key's
// place is its place in its run and, of every other run, the number of smaller
// keys.  A workgroup takes kSortThreads consecutive keys of a run; its waves
// find the part of each other run that lies between the first and the last of
// them, and the threads search those parts, kSearch runs at a time so that their
// loads overlap.
constexpr uint32_t kMergeRuns = 16;
constexpr int kSearch = 8;

// The number of keys below k in the sorted A[0, n), in every lane.
__device__ __forceinline__ uint32_t wave_lower_bound(const uint64_t* A, uint32_t n, uint64_t k) {
    const uint32_t lane = threadIdx.x & 63u;
    uint32_t lo = 0, hi = n;  // the answer lies in [lo, hi]
    while (hi > lo) {
        const uint32_t span = hi - lo, stride = (span + 63u) / 64u;
        const uint32_t m = lo + lane * stride;
        const uint32_t c = (uint32_t)__popcll(__ballot(m < hi && A[m] < k));
        // the tests hold for the first c candidates: the answer is past the last of them
        const uint32_t l2 = c ? lo + (c - 1u) * stride + 1u : lo;
        hi = min(hi, lo + c * stride);
        lo = l2;
    }
    return lo;
}

__global__ __launch_bounds__(kSortThreads) void merge_all(const uint64_t* __restrict__ in,
                                                          uint64_t* __restrict__ out,
                                                          uint32_t n) {
    __shared__ uint32_t from[kMergeRuns], len[kMergeRuns];
    const uint32_t b0 = blockIdx.x * kSortThreads;
    const uint32_t cnt = min((uint32_t)kSortThreads, n - b0);
    const uint32_t own = b0 / kSortTile, runs = (n + kSortTile - 1) / kSortTile;
    const uint64_t first = in[b0], final = in[b0 + cnt - 1u];
    for (uint32_t q = threadIdx.x >> 6; q < kMergeRuns; q += kSortThreads / 64) {
        uint32_t lo = 0, hi = 0;
        if (q < runs && q != own) {
            const uint32_t w = min(kSortTile, n - q * kSortTile);
            lo = wave_lower_bound(in + q * kSortTile, w, first);
            hi = lo + wave_lower_bound(in + q * kSortTile + lo, w - lo, final);
        }
        if ((threadIdx.x & 63u) == 0) {
            from[q] = lo;
            len[q] = hi - lo;
        }
    }
    __syncthreads();
    if (threadIdx.x >= cnt) return;
    const uint64_t key = in[b0 + threadIdx.x];
    uint32_t place = b0 + threadIdx.x - own * kSortTile;
    for (uint32_t q0 = 0; q0 < runs; q0 += kSearch) {
        uint32_t lo[kSearch], m[kSearch], most = 0;
#pragma unroll
        for (int u = 0; u < kSearch; ++u) {
            lo[u] = (q0 + u) * kSortTile + from[q0 + u];
            m[u] = len[q0 + u];
            most = max(most, m[u]);
        }
        for (; most > 0u; most >>= 1) {
            uint64_t v[kSearch];
#pragma unroll
            for (int u = 0; u < kSearch; ++u) v[u] = m[u] ? in[lo[u] + (m[u] >> 1)] : 0ull;
#pragma unroll
            for (int u = 0; u < kSearch; ++u) {
                const uint32_t half = m[u] >> 1;
                const bool right = m[u] != 0u && v[u] < key;
                lo[u] += right ? half + 1u : 0u;
                m[u] = right ? m[u] - half - 1u : half;
            }
        }
#pragma unroll
        for (int u = 0; u < kSearch; ++u) place += lo[u] - (q0 + u) * kSortTile;
    }
    out[place] = key;
}

// Sorts keys[0, n) (clobbered) into out[0, n).
hipError_t sort_keys(uint64_t* keys, uint64_t* out, uint32_t n, hipStream_t s, uint32_t run0) {
    if (n == 0) return hipSuccess;
    if (run0 != 0u && (run0 < (uint32_t)kSortItems || (run0 & (run0 - 1u)) != 0u))
        return hipErrorInvalidValue;
    if (n <= kRankMax) {
        rank_sort<<<(n + kRankKeys - 1) / kRankKeys, 64 * kRankWaves, 0, s>>>(keys, out, n);
        return hipGetLastError();
    }
    const uint32_t tiles = (n + kSortTile - 1) / kSortTile;
    const bool once = tiles <= kMergeRuns;  // one merge launch
    int levels = 0;
    for (uint64_t r = kSortTile; r < n; r <<= 1) ++levels;
    // the block sort writes where `levels` merges, alternating, end in out
    uint64_t* src = once || (levels & 1) ? keys : out;
    block_sort<kSortThreads><<<tiles, kSortThreads, 0, s>>>(keys, src, n, run0);
    if (once) {
        if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
        merge_all<<<(n + kSortThreads - 1) / kSortThreads, kSortThreads, 0, s>>>(keys, out, n);
        return hipGetLastError();
    }
    hipError_t e = hipGetLastError();
    uint64_t w = kSortTile;
    for (int l = 0; l < levels && e == hipSuccess; ++l, w <<= 1) {
        uint64_t* dst = src == keys ? out : keys;
        merge_runs<<<tiles, kSortThreads, 0, s>>>(src, dst, n, (uint32_t)w);
        e = hipGetLastError();
        src = dst;
    }
    return e;
}

}  // namespace gccd
