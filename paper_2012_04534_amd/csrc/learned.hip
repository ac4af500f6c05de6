// Learned unrolled shrinkage network: forward, backward, training and inference.
//
// The network unrolls FISTA (paper Alg. 1) into S stages with learned step and
// threshold and a small 3-D convolutional correction; the operator A / A^H of
// the plan is a fixed layer.  Stage i (FISTA iteration i + 1):
//
//   gamma_i = x_i + beta_i (x_i - x_{i-1})           beta_0 = beta_1 = 0, then FISTA's
//   z_i     = gamma_i - s_i A^H (A gamma_i - y)      s_i = exp(rho_i) / L
//   u_i     = soft(z_i, theta_i)                      theta_i = exp(kappa_i) lam / L
//   x_{i+1} = u_i + c conv2(relu(conv1([Re u_i, Im u_i] / c))),  c = lam / L
//
// lam = mu max|A^H y| per measurement.  3x3x3 convolutions with zero padding
// over the [ny][nx][nz] grid, offset e = (e_y, e_x, e_z) indexed 9 (e_y + 1) +
// 3 (e_x + 1) + e_z + 1.  The scale c makes the network homogeneous in y; in
// the backward pass the c factors cancel except on the W2, b2 and b1
// gradients, which carry one factor c.  Backward: the linear layers are transposed
// (z = gamma - s A^H A gamma + const has the self-adjoint Jacobian
// I - s A^H A, run with the same A and A^H kernels), the complex soft
// threshold on R^2 has Jacobian I - theta (I/|z| - z z^T/|z|^3) for |z| > theta
// and 0 otherwise, d/dtheta = -z/|z|.  Parameter gradients are reduced in FP64
// in a fixed order (deterministic); Adam (Kingma & Ba) updates the FP32
// master weights.
#include <cmath>
#include <cstdio>
#include <cstring>
#include <type_traits>
#include <vector>

#include "internal.h"
#include "run.h"

namespace ufss {

static constexpr int kLT = 256;
static constexpr int kMaxCh = 8;

static int nblk(int64_t n) { return (int)std::max<int64_t>(1, std::min<int64_t>(1024, (n + kLT - 1) / kLT)); }

// The convolution kernels give a thread a run of XV columns x at one (y, z):
// lanes are consecutive depths, so every load is coalesced, the XV + 2 columns
// of a neighbour row (e_y, e_z) serve the 3 XV products of each weight, and a
// weight read from LDS serves the whole run.  The channel count is a template
// constant (accumulators in registers).  What bounds them is the latency of the
// neighbour loads: a row is loaded in straight line while the one before it is used.
// 32 x 32 x 256, 8 channels, before (one voxel per thread, run-time channel count), with
// a row at a time and so: conv1 46, 10.6, 9.9 us, conv2 17 + 5 (the extrapolation's own
// pass), 15.9, 14.1, their transposes 52, 13.7, 12.8 and 17, 14.7, 13.1.  (The same ahead
// with a branch per column waits at each join: conv2 19.)
static constexpr int kXC = 2;            // the convolutions: more, shorter runs (4: 14-20 us; 1: 12-16)
static constexpr int kXW = 4;            // the weight gradients: more products per load (2: 22 us)

// Row (e_y, e_z) = (row / 3 - 1, row % 3 - 1) of the neighbours: whether it is
// inside the grid, and the offset to it.  Tap e of a row is e_x = e - 1, offset
// index tap_index(row, e).
__device__ __forceinline__ bool row_inside(const Dims& d, const Run& r, int row, int64_t& o) {
    const int ey = row / 3 - 1, ez = row % 3 - 1;
    o = (int64_t)ey * d.nx * d.nz + ez;
    return (unsigned)(r.y + ey) < (unsigned)d.ny && (unsigned)(r.z + ez) < (unsigned)d.nz;
}
__device__ __forceinline__ int tap_index(int row, int e) { return row / 3 * 9 + 3 * e + row % 3; }

// The row's values at columns x - 1 .. x + N - 2; zero outside the grid.  at(o): the
// value at voxel r.v + o.
template <class T, int N, class F>
__device__ __forceinline__ void row_values(const Dims& d, const Run& r, bool in, int64_t off, F at, T (&v)[N]) {
#pragma unroll
    for (int k = 0; k < N; ++k) {
        const int x = r.x + k - 1;
        v[k] = T{};
        if (in && x >= 0 && x < d.nx) v[k] = at(off + (int64_t)(k - 1) * d.nz);
    }
}

// The columns x - 1 .. x + XV of a run with their loads in straight line, a row ahead:
// a voxel outside the grid is replaced by its nearest one inside, and by zero after the
// load.
template <int XV>
struct RunColumns {
    int64_t at[XV + 2];     // nearest voxel of column k at the run's (y, z)
    bool ok[XV + 2];
    __device__ RunColumns(const Dims& d, const Run& r) {
#pragma unroll
        for (int k = 0; k < XV + 2; ++k) {
            const int x = r.x + k - 1;
            ok[k] = x >= 0 && x < d.nx;
            at[k] = ((int64_t)r.y * d.nx + min(max(x, 0), d.nx - 1)) * d.nz + r.z;
        }
    }
};
// Offset to the row's nearest row inside, and whether it is the row itself.
__device__ __forceinline__ bool row_offset(const Dims& d, const Run& r, int row, int64_t& o) {
    const int y = r.y + row / 3 - 1, z = r.z + row % 3 - 1;
    const int yc = min(max(y, 0), d.ny - 1), zc = min(max(z, 0), d.nz - 1);
    o = (int64_t)(yc - r.y) * d.nx * d.nz + (zc - r.z);
    return yc == y && zc == z;
}

// --- forward kernels ---------------------------------------------------------
__global__ __launch_bounds__(kLT) void k_momentum(int64_t n, const cf32* __restrict__ x,
                                                  const cf32* __restrict__ xp, float beta,
                                                  cf32* __restrict__ gam) {
    for (int64_t i = (int64_t)blockIdx.x * kLT + threadIdx.x; i < n; i += (int64_t)gridDim.x * kLT) {
        cf32 a = x[i], b = xp[i];
        gam[i] = cf32{a.re + beta * (a.re - b.re), a.im + beta * (a.im - b.im)};
    }
}

// stage parameters at par: [rho, kappa, ...]
// (transform plans: in the adjoint's last lateral product, fft_prox)
__global__ __launch_bounds__(kLT) void k_prox(int64_t n, ProxArgs p) {
    const float s = p.step(), th = p.threshold();
    for (int64_t i = (int64_t)blockIdx.x * kLT + threadIdx.x; i < n; i += (int64_t)gridDim.x * kLT) {
        cf32 z, u;
        prox_step(p.gam[i], p.g[i], s, th, z, u);
        p.z[i] = z;
        p.u[i] = u;
    }
}

// Weights in LDS: w[(row * 3 + tap) * CH + channel] = the pair for (Re, Im).
// src(o, c, e): the weight of channel `o` and part c at offset index e.
template <int CH, class F>
__device__ __forceinline__ void stage_weights(float2* w, F src) {
    for (int t = threadIdx.x; t < 27 * CH; t += kLT) {
        const int i = t / CH, o = t - i * CH, e = tap_index(i / 3, i % 3);
        w[t] = make_float2(src(o, 0, e), src(o, 1, e));
    }
}

// h[co][v] = relu(b1[co] + sum_{c, e} W1[co][c][e] u_c(v + e) / c),  c = lam / L
template <int CH>
__global__ __launch_bounds__(kLT) void k_conv1(Dims d, const cf32* __restrict__ u,
                                               const float* __restrict__ W1, const float* __restrict__ b1,
                                               const double* __restrict__ lam, float invL,
                                               float* __restrict__ h) {
    __shared__ __align__(16) float2 w[27 * CH];
    const float ic = 1.0f / ((float)lam[0] * invL);
    stage_weights<CH>(w, [&](int o, int c, int e) { return W1[o * 54 + c * 27 + e]; });
    __syncthreads();
    const int64_t n = run_count<kXC>(d), nz = d.nz;
    for (int64_t t = (int64_t)blockIdx.x * kLT + threadIdx.x; t < n; t += (int64_t)gridDim.x * kLT) {
        const Run r = run_at<kXC>(d, t);
        float acc[kXC][CH];
#pragma unroll
        for (int k = 0; k < kXC; ++k)
#pragma unroll
            for (int o = 0; o < CH; ++o) acc[k][o] = b1[o];
        const RunColumns<kXC> col(d, r);
        cf32 v[kXC + 2], next[kXC + 2];
        bool in = false, in_next;
        auto load = [&](int row) {
            int64_t off;
            in_next = row_offset(d, r, row, off);
#pragma unroll
            for (int k = 0; k < kXC + 2; ++k) next[k] = u[col.at[k] + off];
        };
        load(0);
#pragma unroll 1
        for (int row = 0; row < 9; ++row) {
            in = in_next;
#pragma unroll
            for (int k = 0; k < kXC + 2; ++k) v[k] = in && col.ok[k] ? next[k] : cf32{0.f, 0.f};
            load(min(row + 1, 8));
#pragma unroll
            for (int k = 0; k < kXC + 2; ++k) v[k] = cf32{v[k].re * ic, v[k].im * ic};
#pragma unroll
            for (int e = 0; e < 3; ++e)
#pragma unroll
                for (int o = 0; o < CH; ++o) {
                    const float2 a = w[(row * 3 + e) * CH + o];
#pragma unroll
                    for (int k = 0; k < kXC; ++k) acc[k][o] += a.x * v[k + e].re + a.y * v[k + e].im;
                }
        }
#pragma unroll
        for (int o = 0; o < CH; ++o)
#pragma unroll
            for (int k = 0; k < kXC; ++k)
                if (r.x + k < d.nx) h[(int64_t)o * d.n + r.v + k * nz] = fmaxf(acc[k][o], 0.f);
    }
}

// xout = u + c (b2 + sum_{c, e} W2[o][c][e] h_c(v + e)) as complex (o = re, im), and,
// with gam, the next stage's extrapolation gam = xout + beta (xout - xcur) in the
// same pass.
template <int CH>
__global__ __launch_bounds__(kLT) void k_conv2(Dims d, const float* __restrict__ h,
                                               const float* __restrict__ W2, const float* __restrict__ b2,
                                               const double* __restrict__ lam, float invL,
                                               const cf32* __restrict__ u, cf32* __restrict__ xout,
                                               const cf32* __restrict__ xcur, float beta, cf32* __restrict__ gam) {
    __shared__ __align__(16) float2 w[27 * CH];
    const float cs = (float)lam[0] * invL;
    stage_weights<CH>(w, [&](int c, int o, int e) { return W2[(o * CH + c) * 27 + e]; });
    __syncthreads();
    const int64_t n = run_count<kXC>(d), nz = d.nz;
    for (int64_t t = (int64_t)blockIdx.x * kLT + threadIdx.x; t < n; t += (int64_t)gridDim.x * kLT) {
        const Run r = run_at<kXC>(d, t);
        float ar[kXC], ai[kXC];
#pragma unroll
        for (int k = 0; k < kXC; ++k) {
            ar[k] = b2[0];
            ai[k] = b2[1];
        }
        const RunColumns<kXC> col(d, r);
        float cur[CH][kXC + 2], next[CH][kXC + 2];
        bool in = false, in_next;
        auto load = [&](int row) {
            int64_t off;
            in_next = row_offset(d, r, row, off);
#pragma unroll
            for (int k = 0; k < kXC + 2; ++k)
#pragma unroll
                for (int p = 0; p < CH; ++p) next[p][k] = (h + p * d.n)[col.at[k] + off];
        };
        load(0);
#pragma unroll 1
        for (int row = 0; row < 9; ++row) {
            in = in_next;
#pragma unroll
            for (int p = 0; p < CH; ++p)
#pragma unroll
                for (int k = 0; k < kXC + 2; ++k) cur[p][k] = in && col.ok[k] ? next[p][k] : 0.f;
            load(min(row + 1, 8));
#pragma unroll
            for (int c = 0; c < CH; ++c) {
                const float (&v)[kXC + 2] = cur[c];
#pragma unroll
                for (int e = 0; e < 3; ++e) {
                    const float2 a = w[(row * 3 + e) * CH + c];
#pragma unroll
                    for (int k = 0; k < kXC; ++k) {
                        ar[k] += a.x * v[k + e];
                        ai[k] += a.y * v[k + e];
                    }
                }
            }
        }
#pragma unroll
        for (int k = 0; k < kXC; ++k) {
            if (r.x + k >= d.nx) break;
            const int64_t v = r.v + k * nz;
            const cf32 uu = u[v];
            const cf32 x{uu.re + cs * ar[k], uu.im + cs * ai[k]};
            xout[v] = x;
            if (gam) {
                const cf32 b = xcur[v];
                gam[v] = cf32{x.re + beta * (x.re - b.re), x.im + beta * (x.im - b.im)};
            }
        }
    }
}

// --- backward kernels ---------------------------------------------------------
__global__ __launch_bounds__(kLT) void k_loss_grad(int64_t n, const cf32* __restrict__ x,
                                                   const cf32* __restrict__ aref, const double* __restrict__ ref2,
                                                   cf32* __restrict__ dx, double* __restrict__ part) {
    __shared__ double red[kLT];
    const float sc = (float)(2.0 / ref2[0]);
    double acc = 0.0;
    for (int64_t i = (int64_t)blockIdx.x * kLT + threadIdx.x; i < n; i += (int64_t)gridDim.x * kLT) {
        const cf32 a = x[i], b = aref[i];
        const float er = a.re - b.re, ei = a.im - b.im;
        dx[i] = cf32{sc * er, sc * ei};
        acc += (double)er * er + (double)ei * ei;
    }
    red[threadIdx.x] = acc;
    __syncthreads();
    for (int off = kLT / 2; off > 0; off >>= 1) {
        if (threadIdx.x < off) red[threadIdx.x] += red[threadIdx.x + off];
        __syncthreads();
    }
    if (threadIdx.x == 0) part[blockIdx.x] = red[0];
}

// dh[c][v] = (h[c][v] > 0) * sum_{o, e} W2[o][c][e] dx_o(v - e)
template <int CH>
__global__ __launch_bounds__(kLT) void k_conv2_bwd(Dims d, const cf32* __restrict__ dx,
                                                   const float* __restrict__ W2, const float* __restrict__ h,
                                                   float* __restrict__ dh) {
    __shared__ __align__(16) float2 w[27 * CH];
    stage_weights<CH>(w, [&](int c, int o, int e) { return W2[(o * CH + c) * 27 + 26 - e]; });   // mirrored: v - e
    __syncthreads();
    const int64_t n = run_count<kXC>(d), nz = d.nz;
    for (int64_t t = (int64_t)blockIdx.x * kLT + threadIdx.x; t < n; t += (int64_t)gridDim.x * kLT) {
        const Run r = run_at<kXC>(d, t);
        float acc[kXC][CH];
#pragma unroll
        for (int k = 0; k < kXC; ++k)
#pragma unroll
            for (int c = 0; c < CH; ++c) acc[k][c] = 0.f;
        float hv[CH][kXC];
#pragma unroll
        for (int c = 0; c < CH; ++c)
#pragma unroll
            for (int k = 0; k < kXC; ++k) hv[c][k] = (h + c * d.n)[r.v + min(k, d.nx - 1 - r.x) * nz];
        const RunColumns<kXC> col(d, r);
        cf32 v[kXC + 2], next[kXC + 2];
        bool in = false, in_next;
        auto load = [&](int row) {
            int64_t off;
            in_next = row_offset(d, r, row, off);
#pragma unroll
            for (int k = 0; k < kXC + 2; ++k) next[k] = dx[col.at[k] + off];
        };
        load(0);
#pragma unroll 1
        for (int row = 0; row < 9; ++row) {
            in = in_next;
#pragma unroll
            for (int k = 0; k < kXC + 2; ++k) v[k] = in && col.ok[k] ? next[k] : cf32{0.f, 0.f};
            load(min(row + 1, 8));
#pragma unroll
            for (int e = 0; e < 3; ++e)
#pragma unroll
                for (int c = 0; c < CH; ++c) {
                    const float2 a = w[(row * 3 + e) * CH + c];
#pragma unroll
                    for (int k = 0; k < kXC; ++k) acc[k][c] += a.x * v[k + e].re + a.y * v[k + e].im;
                }
        }
#pragma unroll
        for (int c = 0; c < CH; ++c)
#pragma unroll
            for (int k = 0; k < kXC; ++k)
                if (r.x + k < d.nx) {
                    const int64_t o = (int64_t)c * d.n + r.v + k * nz;
                    dh[o] = hv[c][k] > 0.f ? acc[k][c] : 0.f;
                }
    }
}

// du = dx + sum_{o, e} W1[o][c][e] dh_o(v - e)
template <int CH>
__global__ __launch_bounds__(kLT) void k_conv1_bwd(Dims d, const float* __restrict__ dh,
                                                   const float* __restrict__ W1, const cf32* __restrict__ dx,
                                                   cf32* __restrict__ du) {
    __shared__ __align__(16) float2 w[27 * CH];
    stage_weights<CH>(w, [&](int o, int c, int e) { return W1[o * 54 + c * 27 + 26 - e]; });     // mirrored: v - e
    __syncthreads();
    const int64_t n = run_count<kXC>(d), nz = d.nz;
    for (int64_t t = (int64_t)blockIdx.x * kLT + threadIdx.x; t < n; t += (int64_t)gridDim.x * kLT) {
        const Run r = run_at<kXC>(d, t);
        float ar[kXC], ai[kXC];
#pragma unroll
        for (int k = 0; k < kXC; ++k) ar[k] = ai[k] = 0.f;
        const RunColumns<kXC> col(d, r);
        float cur[CH][kXC + 2], next[CH][kXC + 2];
        bool in = false, in_next;
        auto load = [&](int row) {
            int64_t off;
            in_next = row_offset(d, r, row, off);
#pragma unroll
            for (int k = 0; k < kXC + 2; ++k)
#pragma unroll
                for (int p = 0; p < CH; ++p) next[p][k] = (dh + p * d.n)[col.at[k] + off];
        };
        load(0);
#pragma unroll 1
        for (int row = 0; row < 9; ++row) {
            in = in_next;
#pragma unroll
            for (int p = 0; p < CH; ++p)
#pragma unroll
                for (int k = 0; k < kXC + 2; ++k) cur[p][k] = in && col.ok[k] ? next[p][k] : 0.f;
            load(min(row + 1, 8));
#pragma unroll
            for (int o = 0; o < CH; ++o) {
                const float (&v)[kXC + 2] = cur[o];
#pragma unroll
                for (int e = 0; e < 3; ++e) {
                    const float2 a = w[(row * 3 + e) * CH + o];
#pragma unroll
                    for (int k = 0; k < kXC; ++k) {
                        ar[k] += a.x * v[k + e];
                        ai[k] += a.y * v[k + e];
                    }
                }
            }
        }
#pragma unroll
        for (int k = 0; k < kXC; ++k)
            if (r.x + k < d.nx) {
                const cf32 g = dx[r.v + k * nz];
                du[r.v + k * nz] = cf32{g.re + ar[k], g.im + ai[k]};
            }
    }
}

// Weight gradients: gW[o][c][e] = sum_v dout_o(v) in_c(v + e), gb[o] = sum_v dout_o(v),
// where one of dout / in is a complex field (2 parts) and the other CH planes.
// What bounds it: the loads of both fields per product.  Block (r, row) takes a
// range of voxels and one row (e_y, e_z): every thread forms the 2 CH x 3 products of
// its voxels (each loaded value is used 3 to 3 CH times) in FP32 over at most
// kWgRun runs, then the block sums each of them over its threads in FP64 through
// LDS in fixed order, into part[(r * 9 + row) * (6 CH + CH') + slot]; slots past
// the products are the bias (row 4, the centre, only).  32 x 32 x 256, 8
// channels: 17.5 (gW1) and 15.0 us (gW2) per launch, 98 with one (o, c) pair per
// block, whose 27 products per voxel each took a load of their own; the sum over
// the ranges 4.5 us, 18 with one thread per slot.  PLANES_OUT: dout is the planes (gW1), else in (gW2).
static constexpr int kWgRun = 2;                       // runs of kXW voxels per thread
template <int CH, bool PLANES_OUT>
__global__ __launch_bounds__(kLT) void k_wgrad(Dims d, const float* __restrict__ planes, const cf32* __restrict__ field,
                                               double* __restrict__ part) {
    constexpr int NB = PLANES_OUT ? CH : 2, NV = 6 * CH + NB;
    __shared__ float sv[NV][kLT + 1];
    __shared__ double sd[NV][4];
    const int row = blockIdx.y;
    const int64_t n = run_count<kXW>(d), nz = d.nz;
    float acc[2 * CH][3], bias[NB];
#pragma unroll
    for (int p = 0; p < 2 * CH; ++p)
#pragma unroll
        for (int e = 0; e < 3; ++e) acc[p][e] = 0.f;
#pragma unroll
    for (int o = 0; o < NB; ++o) bias[o] = 0.f;
    for (int q = 0; q < kWgRun; ++q) {
        const int64_t t = ((int64_t)blockIdx.x * kWgRun + q) * kLT + threadIdx.x;
        if (t >= n) break;
        const Run r = run_at<kXW>(d, t);
        int64_t off;
        const bool in = row_inside(d, r, row, off);
        if (PLANES_OUT) {
            cf32 f[kXW + 2];
            row_values(d, r, in, off, [&](int64_t at) { return field[r.v + at]; }, f);
#pragma unroll
            for (int o = 0; o < CH; ++o)
#pragma unroll
                for (int k = 0; k < kXW; ++k) {
                    const float g = r.x + k < d.nx ? planes[(int64_t)o * d.n + r.v + k * nz] : 0.f;
                    bias[o % NB] += g;
#pragma unroll
                    for (int e = 0; e < 3; ++e) {
                        acc[2 * o][e] += g * f[k + e].re;
                        acc[2 * o + 1][e] += g * f[k + e].im;
                    }
                }
        } else {
            cf32 g[kXW];
#pragma unroll
            for (int k = 0; k < kXW; ++k) {
                g[k] = r.x + k < d.nx ? field[r.v + k * nz] : cf32{0.f, 0.f};
                bias[0] += g[k].re;
                bias[1 % NB] += g[k].im;
            }
#pragma unroll
            for (int c = 0; c < CH; ++c) {
                float v[kXW + 2];
                row_values(d, r, in, off, [&](int64_t at) { return planes[(int64_t)c * d.n + r.v + at]; }, v);
#pragma unroll
                for (int k = 0; k < kXW; ++k)
#pragma unroll
                    for (int e = 0; e < 3; ++e) {
                        acc[c][e] += g[k].re * v[k + e];
                        acc[CH + c][e] += g[k].im * v[k + e];
                    }
            }
        }
    }
#pragma unroll
    for (int p = 0; p < 2 * CH; ++p)
#pragma unroll
        for (int e = 0; e < 3; ++e) sv[p * 3 + e][threadIdx.x] = acc[p][e];
#pragma unroll
    for (int o = 0; o < NB; ++o) sv[6 * CH + o][threadIdx.x] = bias[o];
    __syncthreads();
    for (int t = threadIdx.x; t < 4 * NV; t += kLT) {
        const int w = t >> 2, q = t & 3;
        double s = 0.0;
        for (int i = 0; i < kLT / 4; ++i) s += (double)sv[w][4 * i + q];
        sd[w][q] = s;
    }
    __syncthreads();
    for (int w = threadIdx.x; w < NV; w += kLT)
        part[((int64_t)blockIdx.x * 9 + row) * NV + w] = (sd[w][0] + sd[w][1]) + (sd[w][2] + sd[w][3]);
}

// gW[pair * 27 + tap_index(row, e)] += the sum over the voxel ranges of slot (row, pair,
// e), gb[o] += that of the bias; each optionally times c = lam / L (the
// correction's scale, see the stage definition).  One wave per slot: lane l sums
// the ranges l, l + 64, ..., then a fixed tree.
__global__ __launch_bounds__(kLT) void k_wgrad_sum(const double* __restrict__ part, int nsplit, int nw, int nb,
                                                   float* __restrict__ gW, float* __restrict__ gb,
                                                   const double* __restrict__ lam, float invL, int scale_w, int scale_b) {
    const int slot = blockIdx.x * (kLT / 64) + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int nv = nw + nb;
    if (slot >= 9 * nw + nb) return;
    const int row = slot < 9 * nw ? slot / nw : 4, w = slot < 9 * nw ? slot - row * nw : nw + slot - 9 * nw;
    double s = 0.0;
    for (int r = lane; r < nsplit; r += 64) s += part[((int64_t)r * 9 + row) * nv + w];
    for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
    if (lane != 0) return;
    const double cs = lam[0] * (double)invL;
    if (w < nw) gW[(w / 3) * 27 + tap_index(row, w % 3)] += (float)(scale_w ? cs * s : s);
    else gb[w - nw] += (float)(scale_b ? cs * s : s);
}

// Voxel ranges of a weight-gradient launch.
static int wgrad_split(const Dims& d) { return (int)((run_count<kXW>(d) + (int64_t)kLT * kWgRun - 1) / ((int64_t)kLT * kWgRun)); }

// Soft-threshold backward and the step-size gradient partials.
__global__ __launch_bounds__(kLT) void k_soft_bwd(int64_t n, const cf32* __restrict__ z,
                                                  const cf32* __restrict__ du, const cf32* __restrict__ g,
                                                  const float* __restrict__ par, float invL,
                                                  const double* __restrict__ lam, cf32* __restrict__ dz,
                                                  double* __restrict__ part) {
    __shared__ double red[2][kLT];
    const float th = expf(par[1]) * (float)lam[0] * invL;
    double a_th = 0.0, a_s = 0.0;
    for (int64_t i = (int64_t)blockIdx.x * kLT + threadIdx.x; i < n; i += (int64_t)gridDim.x * kLT) {
        const cf32 zz = z[i], d = du[i];
        const float mag = sqrtf(zz.re * zz.re + zz.im * zz.im);
        cf32 o{0.f, 0.f};
        if (mag > th) {
            const float inv = 1.0f / mag;
            const float zd = zz.re * d.re + zz.im * d.im;
            const float k3 = th * zd * inv * inv * inv;
            o.re = d.re - th * inv * d.re + k3 * zz.re;
            o.im = d.im - th * inv * d.im + k3 * zz.im;
            a_th += -(double)zd * inv;
        }
        dz[i] = o;
        const cf32 gg = g[i];
        a_s += -((double)o.re * gg.re + (double)o.im * gg.im);
    }
    red[0][threadIdx.x] = a_th;
    red[1][threadIdx.x] = a_s;
    __syncthreads();
    for (int off = kLT / 2; off > 0; off >>= 1) {
        if (threadIdx.x < off) {
            red[0][threadIdx.x] += red[0][threadIdx.x + off];
            red[1][threadIdx.x] += red[1][threadIdx.x + off];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        part[2 * blockIdx.x] = red[0][0];
        part[2 * blockIdx.x + 1] = red[1][0];
    }
}

// d gamma = dz - s (A^H A dz); dx_i += (1 + beta) d gamma; dx_{i-1} -= beta d gamma
__global__ __launch_bounds__(kLT) void k_dgamma(int64_t n, const cf32* __restrict__ dz,
                                                const cf32* __restrict__ ahadz, const float* __restrict__ par,
                                                float invL, float beta, cf32* __restrict__ dxi,
                                                cf32* __restrict__ dxim1) {
    const float s = expf(par[0]) * invL;
    for (int64_t i = (int64_t)blockIdx.x * kLT + threadIdx.x; i < n; i += (int64_t)gridDim.x * kLT) {
        const cf32 a = dz[i], b = ahadz[i];
        const float gr = a.re - s * b.re, gi = a.im - s * b.im;
        cf32 x = dxi[i];
        dxi[i] = cf32{x.re + (1.f + beta) * gr, x.im + (1.f + beta) * gi};
        if (dxim1) {
            cf32 y = dxim1[i];
            dxim1[i] = cf32{y.re - beta * gr, y.im - beta * gi};
        }
    }
}

// grad[rho] += s * ds, grad[kappa] += theta * dtheta (sums of the partials, fixed order)
__global__ void k_scalar_grads(const double* __restrict__ part, int nb, const float* __restrict__ par,
                               float invL, const double* __restrict__ lam, float* __restrict__ grad) {
    __shared__ double red[2][kLT];
    double a = 0.0, b = 0.0;
    for (int i = threadIdx.x; i < nb; i += kLT) {
        a += part[2 * i];
        b += part[2 * i + 1];
    }
    red[0][threadIdx.x] = a;
    red[1][threadIdx.x] = b;
    __syncthreads();
    for (int off = kLT / 2; off > 0; off >>= 1) {
        if (threadIdx.x < off) {
            red[0][threadIdx.x] += red[0][threadIdx.x + off];
            red[1][threadIdx.x] += red[1][threadIdx.x + off];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        const double s = exp((double)par[0]) * invL;
        const double th = exp((double)par[1]) * lam[0] * invL;
        grad[0] += (float)(red[1][0] * s);
        grad[1] += (float)(red[0][0] * th);
    }
}

__global__ __launch_bounds__(kLT) void k_adam(int64_t n, float* __restrict__ p, const float* __restrict__ g,
                                              float* __restrict__ m, float* __restrict__ v, float lr,
                                              float gscale, float b1t, float b2t, int64_t t) {
    const float b1 = 0.9f, b2 = 0.999f, eps = 1e-8f;
    for (int64_t i = (int64_t)blockIdx.x * kLT + threadIdx.x; i < n; i += (int64_t)gridDim.x * kLT) {
        const float gg = g[i] * gscale;
        const float mm = b1 * m[i] + (1.f - b1) * gg;
        const float vv = b2 * v[i] + (1.f - b2) * gg * gg;
        m[i] = mm;
        v[i] = vv;
        p[i] -= lr * (mm / b1t) / (sqrtf(vv / b2t) + eps);
    }
    (void)t;
}

__global__ void k_mul_scalar(double* x, double f) {
    if (threadIdx.x == 0) x[0] *= f;
}

// --- network object -----------------------------------------------------------
struct Net {
    Plan* P = nullptr;
    int S = 0, ch = 0, sn = 0;
    double L = 0, mu = 0;
    int64_t np = 0;
    float *d_par = nullptr, *d_grad = nullptr, *d_m = nullptr, *d_v = nullptr;
    int64_t adam_t = 0;
    std::vector<cf32*> x, gam, g, z, u, dxs;
    std::vector<float*> h;
    cf32 *du = nullptr, *dz = nullptr, *tmp = nullptr;
    float* dh = nullptr;
    double *d_lam = nullptr, *d_part = nullptr, *d_sc = nullptr, *d_wpart = nullptr;
    std::vector<float> beta;
    std::vector<void*> owned;
};

template <class T>
static T* nalloc(Net& N, size_t count) {
    void* p = nullptr;
    UFSS_HIP(hipMalloc(&p, std::max<size_t>(count, 1) * sizeof(T)));
    N.owned.push_back(p);
    return static_cast<T*>(p);
}

static void net_free(Net* N) {
    if (!N) return;
    for (void* p : N->owned) (void)hipFree(p);
    delete N;
}

static int stage_size(int ch) { return 2 + ch * 54 + ch + 2 * ch * 27 + 2; }

Net* net_create(Plan* P, int S, int ch, double L, double mu, uint64_t seed) {
    if (!P) fail(UFSS_ERR_INVALID_ARG, "plan is NULL");
    if (S < 1 || S > 256 || ch < 1 || ch > kMaxCh) fail(UFSS_ERR_INVALID_ARG, "stages in [1,256], channels in [1,8]");
    if (P->nvox >= (int64_t(1) << 32)) fail(UFSS_ERR_OOM, "no device holds a network of 2^32 voxels");   // see run_at
    if (!(L > 0) || !(mu > 0)) fail(UFSS_ERR_INVALID_ARG, "L and mu must be positive");
    Net* N = new Net();
    try {
        N->P = P;
        N->S = S;
        N->ch = ch;
        N->sn = stage_size(ch);
        N->L = L;
        N->mu = mu;
        N->np = (int64_t)S * N->sn;
        const int64_t nv = P->nvox;
        N->d_par = nalloc<float>(*N, N->np);
        N->d_grad = nalloc<float>(*N, N->np);
        N->d_m = nalloc<float>(*N, N->np);
        N->d_v = nalloc<float>(*N, N->np);
        for (int i = 0; i <= S; ++i) {
            N->x.push_back(nalloc<cf32>(*N, nv));
            N->dxs.push_back(nalloc<cf32>(*N, nv));
        }
        for (int i = 0; i < S; ++i) {
            N->gam.push_back(nalloc<cf32>(*N, nv));
            N->g.push_back(nalloc<cf32>(*N, nv));
            N->z.push_back(nalloc<cf32>(*N, nv));
            N->u.push_back(nalloc<cf32>(*N, nv));
            N->h.push_back(nalloc<float>(*N, (size_t)ch * nv));
        }
        N->du = nalloc<cf32>(*N, nv);
        N->dz = nalloc<cf32>(*N, nv);
        N->tmp = nalloc<cf32>(*N, nv);
        N->dh = nalloc<float>(*N, (size_t)ch * nv);
        N->d_lam = nalloc<double>(*N, 4);
        N->d_part = nalloc<double>(*N, 4096);
        N->d_sc = nalloc<double>(*N, 16);
        N->d_wpart = nalloc<double>(*N, (size_t)wgrad_split(Dims{P->g.nx, P->g.ny, P->g.nz, nv}) * 9 * (6 * ch + std::max(ch, 2)));
        // FISTA momentum weights (stage i = iteration i + 1)
        double t = 1.0;
        for (int i = 0; i < S; ++i) {
            double b = 0.0;
            if (i > 0) {
                const double tn = 0.5 * (1.0 + std::sqrt(1.0 + 4.0 * t * t));
                b = (t - 1.0) / tn;
                t = tn;
            }
            N->beta.push_back((float)b);
        }
        // initial parameters: rho = kappa = 0, W1 ~ N(0, 0.1^2) (SplitMix64 + Box-Muller), rest 0
        std::vector<float> h((size_t)N->np, 0.f);
        uint64_t st = seed;
        auto next = [&]() {
            st += 0x9E3779B97F4A7C15ull;
            uint64_t zz = st;
            zz = (zz ^ (zz >> 30)) * 0xBF58476D1CE4E5B9ull;
            zz = (zz ^ (zz >> 27)) * 0x94D049BB133111EBull;
            return zz ^ (zz >> 31);
        };
        for (int i = 0; i < S; ++i)
            for (int k = 0; k < ch * 54; ++k) {
                const double u1 = ((next() >> 11) + 1.0) * 0x1.0p-53, u2 = (next() >> 11) * 0x1.0p-53;
                h[(size_t)i * N->sn + 2 + k] = (float)(0.1 * std::sqrt(-2.0 * std::log(u1)) * std::cos(2 * M_PI * u2));
            }
        UFSS_HIP(hipMemcpy(N->d_par, h.data(), N->np * sizeof(float), hipMemcpyHostToDevice));
        UFSS_HIP(hipMemset(N->d_grad, 0, N->np * sizeof(float)));
        UFSS_HIP(hipMemset(N->d_m, 0, N->np * sizeof(float)));
        UFSS_HIP(hipMemset(N->d_v, 0, N->np * sizeof(float)));
        UFSS_HIP(hipMemset(N->x[0], 0, nv * sizeof(cf32)));
    } catch (...) {
        net_free(N);
        throw;
    }
    return N;
}

void net_destroy(Net* N) {
    if (!N) fail(UFSS_ERR_INVALID_ARG, "net is NULL");
    UFSS_HIP(hipDeviceSynchronize());
    net_free(N);
}

static Dims dims_of(const Net& N) {
    return Dims{N.P->g.nx, N.P->g.ny, N.P->g.nz, N.P->nvox};
}

// Calls f with the channel count as a compile-time constant.
template <class F>
static void with_channels(int ch, F f) {
    switch (ch) {
        case 1: f(std::integral_constant<int, 1>{}); break;
        case 2: f(std::integral_constant<int, 2>{}); break;
        case 3: f(std::integral_constant<int, 3>{}); break;
        case 4: f(std::integral_constant<int, 4>{}); break;
        case 5: f(std::integral_constant<int, 5>{}); break;
        case 6: f(std::integral_constant<int, 6>{}); break;
        case 7: f(std::integral_constant<int, 7>{}); break;
        default: f(std::integral_constant<int, kMaxCh>{}); break;
    }
}

// Forward pass; with `keep`, all that the backward pass reads is kept.  Result in N.x[S].
static void net_forward(Net& N, const cf32* y, bool keep, hipStream_t s) {
    Plan& P = *N.P;
    const int64_t n = P.nvox;
    const float invL = (float)(1.0 / N.L);
    // lam = mu max |A^H y|
    op_adjoint(P, y, N.tmp, s);
    int nb = launch_absmax(n, N.tmp, N.d_part, s);
    launch_reduce_max(N.d_part, nb, N.d_lam, s);
    hipLaunchKernelGGL(k_mul_scalar, dim3(1), dim3(64), 0, s, N.d_lam, N.mu);
    const Dims d = dims_of(N);
    const int ch = N.ch;
    // the first extrapolation is x_0 itself; every further one is formed by the
    // previous stage's last kernel
    hipLaunchKernelGGL(k_momentum, dim3(nblk(n)), dim3(kLT), 0, s, n, N.x[0], N.x[0], N.beta[0], N.gam[0]);
    const int nbr = nblk(run_count<kXC>(d));
    for (int i = 0; i < N.S; ++i) {
        const float* par = N.d_par + (int64_t)i * N.sn;
        op_residual(P, N.gam[i], y, P.d_part, StatsJob{}, s);
        ProxArgs prox{N.gam[i], par, invL, N.d_lam, N.g[i], N.z[i], N.u[i]};
        if (fft_fused(P)) {
            op_adjoint_spectrum(P, s);
            if (!keep) prox.g = nullptr;
            fft_prox(P, prox, s);
        } else {
            op_adjoint_residual(P, N.g[i], s);
            hipLaunchKernelGGL(k_prox, dim3(nblk(n)), dim3(kLT), 0, s, n, prox);
        }
        const bool more = i + 1 < N.S;
        with_channels(ch, [&](auto chc) {
            constexpr int CH = decltype(chc)::value;
            hipLaunchKernelGGL(k_conv1<CH>, dim3(nbr), dim3(kLT), 0, s, d, N.u[i], par + 2, par + 2 + CH * 54,
                               N.d_lam, invL, N.h[i]);
            hipLaunchKernelGGL(k_conv2<CH>, dim3(nbr), dim3(kLT), 0, s, d, N.h[i], par + 2 + CH * 54 + CH,
                               par + 2 + CH * 54 + CH + 2 * CH * 27, N.d_lam, invL, N.u[i], N.x[i + 1], N.x[i],
                               more ? N.beta[i + 1] : 0.f, more ? N.gam[i + 1] : nullptr);
        });
    }
    UFSS_HIP(hipGetLastError());
}

// Backward pass for one sample; accumulates into d_grad; loss into d_sc[0].
static void net_backward(Net& N, const cf32* aref, hipStream_t s) {
    Plan& P = *N.P;
    const int64_t n = P.nvox;
    const float invL = (float)(1.0 / N.L);
    const Dims d = dims_of(N);
    const int ch = N.ch;
    const int nsp = wgrad_split(d), nbr = nblk(run_count<kXC>(d));
    int nb = launch_norm2(n, aref, P.d_part, s);
    launch_reduce(P.d_part, nb, 2, N.d_sc + 2, s);   // [2] = ||a_ref||^2
    for (int i = 0; i <= N.S; ++i) UFSS_HIP(hipMemsetAsync(N.dxs[i], 0, n * sizeof(cf32), s));
    const int nbl = nblk(n);
    hipLaunchKernelGGL(k_loss_grad, dim3(nbl), dim3(kLT), 0, s, n, N.x[N.S], aref, N.d_sc + 2,
                       N.dxs[N.S], N.d_part);
    launch_reduce(N.d_part, nbl, 1, N.d_sc + 0, s);   // [0] = ||x - a_ref||^2
    for (int i = N.S - 1; i >= 0; --i) {
        const float* par = N.d_par + (int64_t)i * N.sn;
        float* gpar = N.d_grad + (int64_t)i * N.sn;
        const float* W1 = par + 2;
        const float* W2 = par + 2 + ch * 54 + ch;
        float* gW1 = gpar + 2;
        float* gb1 = gpar + 2 + ch * 54;
        float* gW2 = gb1 + ch;
        float* gb2 = gW2 + 2 * ch * 27;
        // conv correction backward
        with_channels(ch, [&](auto chc) {
            constexpr int CH = decltype(chc)::value;
            auto sum = [&](int nb, float* gW, float* gb, int scale_w) {
                const int slots = 9 * 6 * CH + nb;
                hipLaunchKernelGGL(k_wgrad_sum, dim3((slots + kLT / 64 - 1) / (kLT / 64)), dim3(kLT), 0, s, N.d_wpart,
                                   nsp, 6 * CH, nb, gW, gb, N.d_lam, invL, scale_w, 1);
            };
            hipLaunchKernelGGL(k_conv2_bwd<CH>, dim3(nbr), dim3(kLT), 0, s, d, N.dxs[i + 1], W2, N.h[i], N.dh);
            hipLaunchKernelGGL((k_wgrad<CH, false>), dim3(nsp, 9), dim3(kLT), 0, s, d, N.h[i], N.dxs[i + 1], N.d_wpart);
            sum(2, gW2, gb2, 1);
            hipLaunchKernelGGL((k_wgrad<CH, true>), dim3(nsp, 9), dim3(kLT), 0, s, d, N.dh, N.u[i], N.d_wpart);
            sum(CH, gW1, gb1, 0);
            hipLaunchKernelGGL(k_conv1_bwd<CH>, dim3(nbr), dim3(kLT), 0, s, d, N.dh, W1, N.dxs[i + 1], N.du);
        });
        // soft threshold backward, theta / step partials
        hipLaunchKernelGGL(k_soft_bwd, dim3(nbl), dim3(kLT), 0, s, n, N.z[i], N.du, N.g[i], par, invL,
                           N.d_lam, N.dz, N.d_part);
        hipLaunchKernelGGL(k_scalar_grads, dim3(1), dim3(kLT), 0, s, N.d_part, nbl, par, invL, N.d_lam, gpar);
        // gamma backward through I - s A^H A
        op_residual(P, N.dz, nullptr, P.d_part, StatsJob{}, s);
        op_adjoint_residual(P, N.tmp, s);
        hipLaunchKernelGGL(k_dgamma, dim3(nbl), dim3(kLT), 0, s, n, N.dz, N.tmp, par, invL, N.beta[i],
                           N.dxs[i], i >= 1 ? N.dxs[i - 1] : nullptr);
    }
    UFSS_HIP(hipGetLastError());
}

void net_forward_out(Net& N, const cf32* y, cf32* x, hipStream_t s) {
    if (!y || !x) fail(UFSS_ERR_INVALID_ARG, "NULL buffer");
    net_forward(N, y, false, s);
    launch_copy(N.P->nvox, N.x[N.S], x, s);
}

double net_grad(Net& N, const cf32* y, const cf32* aref, int accumulate, hipStream_t s) {
    if (!y || !aref) fail(UFSS_ERR_INVALID_ARG, "NULL buffer");
    if (!accumulate) UFSS_HIP(hipMemsetAsync(N.d_grad, 0, N.np * sizeof(float), s));
    net_forward(N, y, true, s);
    net_backward(N, aref, s);
    double h[3];
    UFSS_HIP(hipMemcpyAsync(h, N.d_sc, 3 * sizeof(double), hipMemcpyDeviceToHost, s));
    UFSS_HIP(hipStreamSynchronize(s));
    return h[0] / h[2];
}

double net_train_step(Net& N, int batch, const cf32* const* ys, const cf32* const* refs, double lr,
                      hipStream_t s) {
    if (batch < 1 || !ys || !refs) fail(UFSS_ERR_INVALID_ARG, "bad batch");
    UFSS_HIP(hipMemsetAsync(N.d_grad, 0, N.np * sizeof(float), s));
    double loss = 0.0;
    for (int b = 0; b < batch; ++b) loss += net_grad(N, ys[b], refs[b], 1, s);
    N.adam_t += 1;
    const double b1t = 1.0 - std::pow(0.9, (double)N.adam_t), b2t = 1.0 - std::pow(0.999, (double)N.adam_t);
    hipLaunchKernelGGL(k_adam, dim3(nblk(N.np)), dim3(kLT), 0, s, N.np, N.d_par, N.d_grad, N.d_m, N.d_v,
                       (float)lr, (float)(1.0 / batch), (float)b1t, (float)b2t, N.adam_t);
    UFSS_HIP(hipGetLastError());
    UFSS_HIP(hipStreamSynchronize(s));
    return loss / batch;
}

void net_params(Net& N, float* get, const float* set, int64_t* count) {
    if (count) *count = N.np;
    if (set) UFSS_HIP(hipMemcpy(N.d_par, set, N.np * sizeof(float), hipMemcpyHostToDevice));
    if (get) UFSS_HIP(hipMemcpy(get, N.d_par, N.np * sizeof(float), hipMemcpyDeviceToHost));
}

void net_grads(Net& N, float* get) {
    if (get) UFSS_HIP(hipMemcpy(get, N.d_grad, N.np * sizeof(float), hipMemcpyDeviceToHost));
}

// Checkpoint: magic, stages, channels, L, mu, adam step, params, m, v.
void net_save(Net& N, const char* path) {
    if (!path) fail(UFSS_ERR_INVALID_ARG, "path is NULL");
    std::vector<float> p(N.np), m(N.np), v(N.np);
    UFSS_HIP(hipMemcpy(p.data(), N.d_par, N.np * 4, hipMemcpyDeviceToHost));
    UFSS_HIP(hipMemcpy(m.data(), N.d_m, N.np * 4, hipMemcpyDeviceToHost));
    UFSS_HIP(hipMemcpy(v.data(), N.d_v, N.np * 4, hipMemcpyDeviceToHost));
    FILE* f = std::fopen(path, "wb");
    if (!f) fail(UFSS_ERR_INVALID_ARG, std::string("cannot write ") + path);
    const char magic[8] = {'U', 'F', 'S', 'S', 'N', 'E', 'T', '1'};
    int32_t hdr[2] = {N.S, N.ch};
    double dd[2] = {N.L, N.mu};
    int64_t t = N.adam_t;
    bool ok = std::fwrite(magic, 1, 8, f) == 8 && std::fwrite(hdr, 4, 2, f) == 2 &&
              std::fwrite(dd, 8, 2, f) == 2 && std::fwrite(&t, 8, 1, f) == 1 &&
              std::fwrite(p.data(), 4, N.np, f) == (size_t)N.np &&
              std::fwrite(m.data(), 4, N.np, f) == (size_t)N.np &&
              std::fwrite(v.data(), 4, N.np, f) == (size_t)N.np;
    std::fclose(f);
    if (!ok) fail(UFSS_ERR_INVALID_ARG, "short write");
}

void net_load(Net& N, const char* path) {
    if (!path) fail(UFSS_ERR_INVALID_ARG, "path is NULL");
    FILE* f = std::fopen(path, "rb");
    if (!f) fail(UFSS_ERR_INVALID_ARG, std::string("cannot read ") + path);
    char magic[8];
    int32_t hdr[2];
    double dd[2];
    int64_t t;
    std::vector<float> p(N.np), m(N.np), v(N.np);
    bool ok = std::fread(magic, 1, 8, f) == 8 && std::memcmp(magic, "UFSSNET1", 8) == 0 &&
              std::fread(hdr, 4, 2, f) == 2 && hdr[0] == N.S && hdr[1] == N.ch &&
              std::fread(dd, 8, 2, f) == 2 && std::fread(&t, 8, 1, f) == 1 &&
              std::fread(p.data(), 4, N.np, f) == (size_t)N.np &&
              std::fread(m.data(), 4, N.np, f) == (size_t)N.np &&
              std::fread(v.data(), 4, N.np, f) == (size_t)N.np;
    std::fclose(f);
    if (!ok) fail(UFSS_ERR_INVALID_ARG, "not a checkpoint of this network shape");
    UFSS_HIP(hipMemcpy(N.d_par, p.data(), N.np * 4, hipMemcpyHostToDevice));
    UFSS_HIP(hipMemcpy(N.d_m, m.data(), N.np * 4, hipMemcpyHostToDevice));
    UFSS_HIP(hipMemcpy(N.d_v, v.data(), N.np * 4, hipMemcpyHostToDevice));
    N.adam_t = t;
    N.L = dd[0];
    N.mu = dd[1];
}

}  // namespace ufss
