// Far-field closure kernels (gfx950): the grid part of the split of Eq. (6)
// into an exact near sum and a far field read from a coarse grid.
//   moments_part, grid_params -- placement of the 32^3 grid (centroid, width)
//   deposit_cic, rho_convert  -- cloud-in-cell charge per node, fixed point
//   conv_mfma                 -- 3x3x3 / 1x1x1 convolutions of the linear
//                                U-Net as implicit GEMMs on bf16 MFMA
//   pool2, upsample2          -- the U-Net's resolution changes
//   far_interp                -- Catmull-Rom interpolation to the carriers
#include "gccd_internal.h"

#include <math.h>

namespace gccd {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// float -> bfloat16 bits, round to nearest, ties to even (finite inputs)
__device__ __forceinline__ uint16_t to_bf16(float f) {
    uint32_t b = __float_as_uint(f);
    b += 0x7FFFu + ((b >> 16) & 1u);
    return (uint16_t)(b >> 16);
}

__device__ __forceinline__ float from_bf16(uint16_t h) {
    return __uint_as_float((uint32_t)h << 16);
}

__device__ __forceinline__ double wsum(double v) {
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) v += __shfl_xor(v, m);
    return v;
}

__device__ __forceinline__ double wmin(double v) {
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) v = fmin(v, __shfl_xor(v, m));
    return v;
}

__device__ __forceinline__ double wmax(double v) {
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) v = fmax(v, __shfl_xor(v, m));
    return v;
}

constexpr int kMom = 10;  // sum dx, dy, dz; sum |d|^2; min x, y, z; max x, y, z

}  // namespace

// ---------------------------------------------------------------------------
// Placement.  Block b of a fixed grid of kMomBlocks sums, over its strided
// share of the charges, the offsets d = x - x[0] and |d|^2 and takes the
// per-axis minimum and maximum (and clears the deposit's sums); grid_params adds the block results in a
// fixed order, so the placement is deterministic for a given input.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void moments_part(const double* x, const double* y,
                                                    const double* z, uint32_t n, double* part,
                                                    unsigned long long* acc) {
    __shared__ double red[kMom][4];
    for (uint32_t i = blockIdx.x * 256u + threadIdx.x; i < (uint32_t)kGridNodes;
         i += gridDim.x * 256u)
        acc[i] = 0ull;
    const double rx = x[0], ry = y[0], rz = z[0];
    double v[kMom] = {0.0, 0.0, 0.0, 0.0, INFINITY, INFINITY, INFINITY,
                      -INFINITY, -INFINITY, -INFINITY};
    for (uint32_t j = blockIdx.x * 256u + threadIdx.x; j < n; j += gridDim.x * 256u) {
        const double dx = x[j] - rx, dy = y[j] - ry, dz = z[j] - rz;
        v[0] += dx;
        v[1] += dy;
        v[2] += dz;
        v[3] += dx * dx + dy * dy + dz * dz;
        v[4] = fmin(v[4], x[j]);
        v[5] = fmin(v[5], y[j]);
        v[6] = fmin(v[6], z[j]);
        v[7] = fmax(v[7], x[j]);
        v[8] = fmax(v[8], y[j]);
        v[9] = fmax(v[9], z[j]);
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) v[k] = wsum(v[k]);
#pragma unroll
    for (int k = 4; k < 7; ++k) v[k] = wmin(v[k]);
#pragma unroll
    for (int k = 7; k < 10; ++k) v[k] = wmax(v[k]);
    const int wave = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) {
#pragma unroll
        for (int k = 0; k < kMom; ++k) red[k][wave] = v[k];
    }
    __syncthreads();
    if (threadIdx.x < kMom) {
        const int k = threadIdx.x;
        double r = red[k][0];
        for (int w = 1; w < 4; ++w)
            r = k < 4 ? r + red[k][w] : (k < 7 ? fmin(r, red[k][w]) : fmax(r, red[k][w]));
        part[(size_t)blockIdx.x * kMom + k] = r;
    }
}

hipError_t launch_moments(const double* x, const double* y, const double* z, uint32_t n,
                          double* part, unsigned long long* acc, hipStream_t s) {
    if (n == 0) return hipErrorInvalidValue;
    moments_part<<<kMomBlocks, 256, 0, s>>>(x, y, z, n, part, acc);
    return hipGetLastError();
}

// One workgroup: centroid c, rms width per axis s, largest offset d_max;
// h = max(kSigmaCells s, d_max / kMaxDevCells), node k at c + (k - 15.5) h.
__global__ __launch_bounds__(256) void grid_params(const double* part, const double* x,
                                                   const double* y, const double* z, uint32_t n,
                                                   double eps2, GridParams* gp) {
    __shared__ double red[kMom][256];
    const int t = threadIdx.x;
    double v[kMom] = {0.0, 0.0, 0.0, 0.0, INFINITY, INFINITY, INFINITY,
                      -INFINITY, -INFINITY, -INFINITY};
    for (int b = t; b < kMomBlocks; b += 256) {
        const double* p = part + (size_t)b * kMom;
#pragma unroll
        for (int k = 0; k < 4; ++k) v[k] += p[k];
#pragma unroll
        for (int k = 4; k < 7; ++k) v[k] = fmin(v[k], p[k]);
#pragma unroll
        for (int k = 7; k < 10; ++k) v[k] = fmax(v[k], p[k]);
    }
#pragma unroll
    for (int k = 0; k < kMom; ++k) red[k][t] = v[k];
    __syncthreads();
    for (int half = 128; half >= 1; half >>= 1) {
        if (t < half) {
#pragma unroll
            for (int k = 0; k < 4; ++k) red[k][t] += red[k][t + half];
#pragma unroll
            for (int k = 4; k < 7; ++k) red[k][t] = fmin(red[k][t], red[k][t + half]);
#pragma unroll
            for (int k = 7; k < 10; ++k) red[k][t] = fmax(red[k][t], red[k][t + half]);
        }
        __syncthreads();
    }
    if (t == 0) {
        const double inv_n = 1.0 / (double)n;
        const double mx = red[0][0] * inv_n, my = red[1][0] * inv_n, mz = red[2][0] * inv_n;
        const double c[3] = {x[0] + mx, y[0] + my, z[0] + mz};
        // sum of the three variances: E|d|^2 - |E d|^2, offsets from x[0]
        double var = red[3][0] * inv_n - (mx * mx + my * my + mz * mz);
        var = fmax(var, 0.0);
        const double s = sqrt(var / 3.0);
        double dmax = 0.0;
#pragma unroll
        for (int d = 0; d < 3; ++d) dmax = fmax(dmax, fmax(c[d] - red[4 + d][0], red[7 + d][0] - c[d]));
        double h = fmax(kSigmaCells * s, dmax / kMaxDevCells);
        if (!(h > 1e-6)) h = 1e-6;  // a single point, or non-finite input
        for (int d = 0; d < 3; ++d) gp->origin[d] = c[d] - 0.5 * (kGrid - 1) * h;
        gp->h = h;
        gp->inv_h = 1.0 / h;
        const double a = kNearCells * h;
        gp->a2 = a * a;
        gp->cut2 = a * a + eps2;
        gp->inv_h2 = 1.0 / (h * h);
    }
}

hipError_t launch_grid_params(const double* part, const double* x, const double* y,
                              const double* z, uint32_t n, double eps2, GridParams* gp,
                              hipStream_t s) {
    grid_params<<<1, 256, 0, s>>>(part, x, y, z, n, eps2, gp);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Cloud-in-cell deposit in 32.32 fixed point: integer atomics make the sum
// independent of their order.  The charges come in the spatially sorted slot
// order, so a workgroup's 256 charges touch only a few nodes: they are
// added first into an 8x8x8 window of nodes in LDS (64-bit LDS atomics)
// and the window's non-zero nodes then go to the grid with one global atomic
// each.  A workgroup whose charges span more than the window (sparse edges
// of a cloud) adds its weights to the grid directly.
// ---------------------------------------------------------------------------
constexpr int kWin = 8;

__global__ __launch_bounds__(256) void deposit_cic(const double* px, const double* py,
                                                   const double* pz, uint32_t n,
                                                   const GridParams* gp,
                                                   unsigned long long* acc) {
    __shared__ unsigned long long win[kWin * kWin * kWin];
    __shared__ int red[6][4];
    const double inv_h = gp->inv_h;
    const double o[3] = {gp->origin[0], gp->origin[1], gp->origin[2]};
    const uint32_t j = blockIdx.x * 256u + threadIdx.x;
    const bool valid = j < n;
    int cell[3] = {0, 0, 0};
    double f[3] = {0.0, 0.0, 0.0};
    if (valid) {
        const double p[3] = {px[j], py[j], pz[j]};
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            double u = (p[d] - o[d]) * inv_h;
            // clamp keeps every access in the grid (non-finite input lands at node 0)
            if (!(u >= 0.0)) u = 0.0;
            if (!(u <= (double)(kGrid - 1))) u = (double)(kGrid - 1);
            int i = (int)floor(u);
            if (i > kGrid - 2) i = kGrid - 2;
            cell[d] = i;
            f[d] = u - (double)i;
        }
    }
    unsigned long long w[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        const double wx = (k & 1) ? f[0] : 1.0 - f[0];
        const double wy = (k & 2) ? f[1] : 1.0 - f[1];
        const double wz = (k & 4) ? f[2] : 1.0 - f[2];
        w[k] = valid ? (unsigned long long)__double2ll_rn(wx * wy * wz * 4294967296.0) : 0ull;
    }
    // the workgroup's cell range per axis
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    int lo[3], hi[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        lo[d] = valid ? cell[d] : kGrid;
        hi[d] = valid ? cell[d] : -1;
#pragma unroll
        for (int m = 32; m >= 1; m >>= 1) {
            lo[d] = min(lo[d], __shfl_xor(lo[d], m));
            hi[d] = max(hi[d], __shfl_xor(hi[d], m));
        }
    }
    if (lane == 0) {
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            red[d][wave] = lo[d];
            red[3 + d][wave] = hi[d];
        }
    }
    for (int i = threadIdx.x; i < kWin * kWin * kWin; i += 256) win[i] = 0ull;
    __syncthreads();
    bool fits = true;
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        lo[d] = min(min(red[d][0], red[d][1]), min(red[d][2], red[d][3]));
        hi[d] = max(max(red[3 + d][0], red[3 + d][1]), max(red[3 + d][2], red[3 + d][3]));
        fits = fits && hi[d] + 1 - lo[d] < kWin;  // nodes lo .. hi + 1
    }
    if (!fits) {
        if (!valid) return;
        const int c = (cell[2] * kGrid + cell[1]) * kGrid + cell[0];
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const int node = c + ((k & 4) ? kGrid * kGrid : 0) + ((k & 2) ? kGrid : 0) + (k & 1);
            atomicAdd(&acc[node], w[k]);
        }
        return;
    }
    if (valid) {
        const int c = ((cell[2] - lo[2]) * kWin + (cell[1] - lo[1])) * kWin + (cell[0] - lo[0]);
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const int node = c + ((k & 4) ? kWin * kWin : 0) + ((k & 2) ? kWin : 0) + (k & 1);
            atomicAdd(&win[node], w[k]);
        }
    }
    __syncthreads();
    for (int i = threadIdx.x; i < kWin * kWin * kWin; i += 256) {
        const unsigned long long v = win[i];
        if (v == 0ull) continue;
        const int x = lo[0] + i % kWin, y = lo[1] + (i / kWin) % kWin, z = lo[2] + i / (kWin * kWin);
        if (x < kGrid && y < kGrid && z < kGrid) atomicAdd(&acc[(z * kGrid + y) * kGrid + x], v);
    }
}

hipError_t launch_deposit(const double* px, const double* py, const double* pz, uint32_t n,
                          const GridParams* gp, unsigned long long* acc, hipStream_t s) {
    if (n == 0) return hipSuccess;
    deposit_cic<<<(n + 255) / 256, 256, 0, s>>>(px, py, pz, n, gp, acc);
    return hipGetLastError();
}

// charge per node: bf16 network input, and FP32 (for inspection) if asked
__global__ void rho_convert(const unsigned long long* acc, uint16_t* rho, float* rho_f32) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= kGridNodes) return;
    const float v = (float)((double)acc[i] * (1.0 / 4294967296.0));
    rho[i] = to_bf16(v);
    if (rho_f32) rho_f32[i] = v;
}

hipError_t launch_rho(const unsigned long long* acc, uint16_t* rho_bf16, float* rho_f32,
                      hipStream_t s) {
    rho_convert<<<kGridNodes / 256, 256, 0, s>>>(acc, rho_bf16, rho_f32);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Convolution as an implicit GEMM on v_mfma_f32_16x16x32_bf16: M = 16
// consecutive nodes (row-major z, y, x), N = output channels in tiles of 16,
// K = taps x input channels in slices of 32 (zero padded).  K index k =
// tap * cin + channel, tap = (dz + 1) * 9 + (dy + 1) * 3 + (dx + 1), the
// order of a PyTorch Conv3d weight (c_out, c_in, kz, ky, kx).  Operand
// layout of the instruction, per lane l of the wave: A holds row l % 16,
// K entries 8 (l / 16) .. +7; B holds column l % 16, the same K entries;
// the result holds column l % 16, rows 4 (l / 16) .. +3.  Weights are
// packed on the host in exactly the B order, one 16-byte load per lane.
// Nodes outside the grid read as zero (zero padding).  One wave, and one
// workgroup, per M tile.
//
// What bounds it: latency.  A layer is a chain of up to 54 dependent matrix
// instructions behind loads that hit L2, over as few as four waves (4^3 nodes).
// The K slices keep their order (one accumulation per output, so the bits do not
// depend on the batching); their operands are loaded kBatch slices at a time, all
// in flight together, with tap and channel known at compile time.  A kernel that
// loaded and multiplied slice by slice with runtime divisions took 27 us per
// layer on average (12 layers, 0.32 ms per closure step); this one takes 5.2 us
// (closure step at 5e4 holes 0.667 -> 0.392 ms).
// ---------------------------------------------------------------------------
constexpr int kBatch = 9;

template <int CIN, int NT, int TAPS>
__global__ __launch_bounds__(64) void conv_mfma(ConvArgs a) {
    // The near sum fills the chip beside these short launches, which wait for each
    // other (closure_field): their waves go first.  Closure step at 5e4 holes: one
    // after the other 0.269 ms, beside each other 0.254, with this priority 0.238.
    __builtin_amdgcn_s_setprio(3);
    constexpr int kMax = TAPS * CIN, kSlices = (kMax + 31) / 32;
    const int lane = threadIdx.x;
    const int n = a.n, ln = a.log2n;
    const int v0 = blockIdx.x * 16;
    const int row = lane & 15, kq = lane >> 4;
    const int v = v0 + row;
    const int vx = v & (n - 1), vy = (v >> ln) & (n - 1), vz = v >> (2 * ln);

    f32x4 acc[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
    // node of tap `tap` beside this lane's, or -1
    auto node = [&](int tap) {
        const int x = vx + (TAPS == 27 ? tap % 3 - 1 : 0);
        const int y = vy + (TAPS == 27 ? (tap / 3) % 3 - 1 : 0);
        const int z = vz + (TAPS == 27 ? tap / 9 - 1 : 0);
        const bool in = (unsigned)x < (unsigned)n && (unsigned)y < (unsigned)n &&
                        (unsigned)z < (unsigned)n && tap < TAPS;
        return in ? (((z << ln) + y) << ln) + x : -1;
    };
#pragma unroll
    for (int s0 = 0; s0 < kSlices; s0 += kBatch) {
        uint4 A[kBatch], B[kBatch][NT];
#pragma unroll
        for (int i = 0; i < kBatch; ++i) {
            const int s = s0 + i;
            if (s >= kSlices) break;
#pragma unroll
            for (int t = 0; t < NT; ++t)
                B[i][t] = *reinterpret_cast<const uint4*>(
                    a.wpk + ((size_t)(s * NT + t) * 64 + lane) * 8);
            if constexpr (CIN == 1) {  // one input channel: 8 taps
                uint16_t av[8];
#pragma unroll
                for (int k = 0; k < 8; ++k) {
                    const int w = node(s * 32 + kq * 8 + k);
                    const uint16_t r = a.in[(size_t)max(w, 0) * a.in_stride + a.in_off];
                    av[k] = w >= 0 ? r : (uint16_t)0;
                }
                __builtin_memcpy(&A[i], av, 16);
            } else {  // 8 consecutive channels of one tap: one 16-byte load
                const int k0 = s * 32 + kq * 8;
                const int tap = CIN % 32 == 0 ? s * 32 / CIN : k0 / CIN;
                const int ch = k0 - tap * CIN;
                const int w = node(tap);
                const uint4 r = *reinterpret_cast<const uint4*>(
                    a.in + (size_t)max(w, 0) * a.in_stride + a.in_off + (w >= 0 ? ch : 0));
                A[i] = w >= 0 ? r : make_uint4(0u, 0u, 0u, 0u);
            }
        }
#pragma unroll
        for (int i = 0; i < kBatch; ++i) {
            if (s0 + i >= kSlices) break;
            bf16x8 av;
            __builtin_memcpy(&av, &A[i], 16);
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                bf16x8 bv;
                __builtin_memcpy(&bv, &B[i][t], 16);
                acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, bv, acc[t], 0, 0, 0);
            }
        }
    }
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        const int co = t * 16 + (lane & 15);
        if (co >= a.cout) continue;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int vo = v0 + kq * 4 + i;
            if (a.outf)
                a.outf[(size_t)vo * 4 + co] = acc[t][i];
            else
                a.out[(size_t)vo * a.out_stride + a.out_off + co] = to_bf16(acc[t][i]);
        }
    }
}

hipError_t launch_conv(const ConvArgs& a, hipStream_t s) {
    // grids of a power of two of nodes per axis, at least 4 (whole tiles of 16)
    if (a.n < 4 || (1 << a.log2n) != a.n || a.cout > 16 * a.ntile) return hipErrorInvalidValue;
    if (a.cin != 1 && ((a.in_stride & 7) != 0 || (a.in_off & 7) != 0)) return hipErrorInvalidValue;
    const int tiles = a.n * a.n * a.n / 16;
    auto is = [&](int cin, int nt, int taps) {
        return a.cin == cin && a.ntile == nt && a.taps == taps;
    };
    if (is(1, 1, 27)) conv_mfma<1, 1, 27><<<tiles, 64, 0, s>>>(a);
    else if (is(16, 1, 27)) conv_mfma<16, 1, 27><<<tiles, 64, 0, s>>>(a);
    else if (is(16, 2, 27)) conv_mfma<16, 2, 27><<<tiles, 64, 0, s>>>(a);
    else if (is(32, 2, 27)) conv_mfma<32, 2, 27><<<tiles, 64, 0, s>>>(a);
    else if (is(64, 2, 27)) conv_mfma<64, 2, 27><<<tiles, 64, 0, s>>>(a);
    else if (is(48, 1, 27)) conv_mfma<48, 1, 27><<<tiles, 64, 0, s>>>(a);
    else if (is(16, 1, 1)) conv_mfma<16, 1, 1><<<tiles, 64, 0, s>>>(a);
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

// mean of 2x2x2 fine nodes, channels [in_off, in_off + c) -> dense [m^3][c]
__global__ void pool2(const uint16_t* in, int in_stride, int in_off, int c, int n,
                      uint16_t* out) {
    const int m = n / 2;
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= m * m * m * c) return;
    const int ch = i % c, vo = i / c;
    const int x = vo % m, y = (vo / m) % m, z = vo / (m * m);
    float sum = 0.0f;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        const int fx = 2 * x + (k & 1), fy = 2 * y + ((k >> 1) & 1), fz = 2 * z + (k >> 2);
        sum += from_bf16(in[(size_t)((fz * n + fy) * n + fx) * in_stride + in_off + ch]);
    }
    out[i] = to_bf16(0.125f * sum);
}

hipError_t launch_pool(const uint16_t* in, int in_stride, int in_off, int c, int n_fine,
                       uint16_t* out, hipStream_t s) {
    const int total = (n_fine / 2) * (n_fine / 2) * (n_fine / 2) * c;
    pool2<<<(total + 255) / 256, 256, 0, s>>>(in, in_stride, in_off, c, n_fine, out);
    return hipGetLastError();
}

// x2 linear upsampling: fine 2i <- 3/4 a[i] + 1/4 a[i-1], fine 2i+1 <- 3/4 a[i]
// + 1/4 a[i+1] per axis, neighbours clamped at the edges; dense [m^3][c] in,
// channels [out_off, out_off + c) of rows of out_stride out
__global__ void upsample2(const uint16_t* in, int c, int m, uint16_t* out, int out_stride,
                          int out_off) {
    const int n = 2 * m;
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= n * n * n * c) return;
    const int ch = i % c, vo = i / c;
    const int f[3] = {vo % n, (vo / n) % n, vo / (n * n)};
    int i0[3], i1[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        i0[d] = f[d] >> 1;
        i1[d] = (f[d] & 1) ? min(i0[d] + 1, m - 1) : max(i0[d] - 1, 0);
    }
    float sum = 0.0f;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        const int ix = (k & 1) ? i1[0] : i0[0];
        const int iy = (k & 2) ? i1[1] : i0[1];
        const int iz = (k & 4) ? i1[2] : i0[2];
        const float w = ((k & 1) ? 0.25f : 0.75f) * ((k & 2) ? 0.25f : 0.75f) *
                        ((k & 4) ? 0.25f : 0.75f);
        sum += w * from_bf16(in[(size_t)((iz * m + iy) * m + ix) * c + ch]);
    }
    out[(size_t)vo * out_stride + out_off + ch] = to_bf16(sum);
}

hipError_t launch_upsample(const uint16_t* in, int c, int m, uint16_t* out, int out_stride,
                           int out_off, hipStream_t s) {
    const int total = 8 * m * m * m * c;
    upsample2<<<(total + 255) / 256, 256, 0, s>>>(in, c, m, out, out_stride, out_off);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Far field at target slot t: Catmull-Rom weights of nodes i-1 .. i+2 per
// axis for u = (x - origin) / h = i + f, the 64 node values summed, times
// 1 / h^2 (the network's unit K / h^2, over K).  The placement keeps every
// charge within 1 <= u < 30; the clamp only guards non-finite input.
// ---------------------------------------------------------------------------
__device__ __forceinline__ void cr_weights(float f, float (&w)[4]) {
    const float f2 = f * f, f3 = f2 * f;
    w[0] = 0.5f * (-f3 + 2.0f * f2 - f);
    w[1] = 0.5f * (3.0f * f3 - 5.0f * f2 + 2.0f);
    w[2] = 0.5f * (-3.0f * f3 + 4.0f * f2 + f);
    w[3] = 0.5f * (f3 - f2);
}

__global__ __launch_bounds__(256) void far_interp(const float4* F, const GridParams* gp,
                                                  const double* px, const double* py,
                                                  const double* pz, uint32_t nt, float* ox,
                                                  float* oy, float* oz) {
    const uint32_t t = blockIdx.x * 256u + threadIdx.x;
    if (t >= nt) return;
    const double p[3] = {px[t], py[t], pz[t]};
    int i[3];
    float w[3][4];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        double u = (p[d] - gp->origin[d]) * gp->inv_h;
        if (!(u >= 1.0)) u = 1.0;
        if (!(u <= (double)(kGrid - 2))) u = (double)(kGrid - 2);
        int k = (int)floor(u);
        if (k > kGrid - 3) k = kGrid - 3;
        i[d] = k;
        cr_weights((float)(u - (double)k), w[d]);
    }
    float ex = 0.0f, ey = 0.0f, ez = 0.0f;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            const float wzy = w[2][c] * w[1][b];
            const int rowbase = ((i[2] + c - 1) * kGrid + (i[1] + b - 1)) * kGrid + i[0] - 1;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const float4 v = F[rowbase + q];
                const float wt = wzy * w[0][q];
                ex = __builtin_fmaf(wt, v.x, ex);
                ey = __builtin_fmaf(wt, v.y, ey);
                ez = __builtin_fmaf(wt, v.z, ez);
            }
        }
    }
    const float s = (float)gp->inv_h2;
    ox[t] = ex * s;
    oy[t] = ey * s;
    oz[t] = ez * s;
}

hipError_t launch_far(const float* F, const GridParams* gp, const double* px, const double* py,
                      const double* pz, uint32_t nt, float* ox, float* oy, float* oz,
                      hipStream_t s) {
    if (nt == 0) return hipSuccess;
    far_interp<<<(nt + 255) / 256, 256, 0, s>>>(reinterpret_cast<const float4*>(F), gp, px, py,
                                                pz, nt, ox, oy, oz);
    return hipGetLastError();
}

}  // namespace gccd
