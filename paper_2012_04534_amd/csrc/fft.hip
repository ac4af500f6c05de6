// Transform-domain operator (paper Sec. IV-B, Alg. 2): the block two-level
// Toeplitz structure makes A a lateral 2-D correlation, which a cyclic
// transform of size L >= N + W per axis evaluates exactly on the scan grid.
//
//   forward  X^[q][z] = DFT_2(x)              (separable twiddle products)
//            Y^[q][k] = sum_z K^[q][z][k] X^[q][z]
//            y[p][k]  = IDFT_2(Y^) on the N x N grid positions, then H_k
//   adjoint  R^[q][k] = DFT_2(H r)
//            X'[q][z] = sum_k conj(K^[q][z][k]) R^[q][k]
//            x[v][z]  = IDFT_2(X') on the grid voxels
//
// K^[q][z][k] = sum_{|d| <= W} P_d[k][z] exp(-j 2 pi (q_x d_x / L_x + q_y d_y / L_y))
// with P_d the windowed, beam-weighted phasor of the other paths (same
// integer-turn delays).  P_d is even in d_x and in d_y, so K^ is a cosine
// transform, even in q_x and q_y: only the quadrant q_x <= L_x / 2,
// q_y <= L_y / 2 is stored, and each stored entry serves up to four q.
// With both axes alike (same pitch, window and size) K^ is also symmetric in
// (q_y, q_x): half the quadrant is stored, each entry serving up to eight q.
// K^ is built once per plan in FP64 and stored in FP32 (BF16 plans: BF16); the
// applies run in FP32.  The contraction streams K^ once per apply and is bound by
// HBM (or by the last-level cache when K^ fits there); the lateral transforms are
// small products with twiddle tables.
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "internal.h"

namespace ufss {

// Lateral products on the FP32 matrix cores (v_mfma_f32_16x16x4f32: rows i,
// columns c of contiguous channels, reduction over j four at a time), in the
// real tables cos(2 pi i j / L) and sin(2 pi i j / L) with the index mirrored
// about L folded away: with C = sum_j cos v_j and S = sum_j sin v_j
//   forward (v on the grid, j < n):   out[i] = C - j S, out[L - i] = C + j S,
//     rows i <= L / 2 only;
//   inverse (v over the L indices, folded to j <= L / 2 as E = v_j + v_{L-j}
//     and O = v_j - v_{L-j}):         out[p] = sum_j cos E_j + j sin O_j, / L.
// Either way half the products of the complex table (64 x 64 x 512: the depth
// transforms of an apply pair 25 + 29 + 30 + 24 us with it, 18 + 20 + 21 + 17 us
// so; 50 x 50 with 256 bins 32 + 14 + 16 + 37 -> 18 + 10 + 10 + 16 us).
//
// What bounds it: on a small scan the latency of one pass (so the loads of a
// wave's column are issued before the tables are staged, kTwPK steps ahead, and
// a wave takes few row tiles), on a large one the traffic of its operands.
// A workgroup is 4 waves on 4 consecutive (b, 16-channel) columns and one block
// of NI row tiles.  The plan keeps each table in operand order,
//   tab[(T ks + s) 64 + lane] = (cos, sin) at row 16 T + lane % 16, j = 4 s + lane / 16
// (row tile T, reduction step s of ks, zero outside the table), staged in LDS
// kTwKS steps at a time: each lane then reads 8 contiguous bytes per operand.
typedef float f4v __attribute__((ext_vector_type(4)));
static constexpr int kTwPK = 8;
static constexpr int kTwKS = 16;
static constexpr int kTwMaxNI = 4;

template <int NI, bool INV>
__global__ __launch_bounds__(256) void twiddle_kernel(cf32* __restrict__ out, const cf32* __restrict__ in,
                                                      const cf32* __restrict__ tab, int L, int n, int ks, int tiles,
                                                      int units, int nct, int C, int64_t sib, int64_t sij,
                                                      int64_t sob, int64_t soi) {
    __shared__ __align__(16) cf32 wl[NI * kTwKS * 64];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int unit = blockIdx.x * 4 + wave, b = unit / nct;
    const int c = (unit - b * nct) * 16 + (lane & 15), kq = lane >> 4;
    const bool active = unit < units, ok = active && c < C;
    const int t0 = blockIdx.y * NI;
    const int J = INV ? L / 2 + 1 : n;                    // reduction length
    const cf32* src = in + (int64_t)b * sib + c;
    // this lane's column at reduction step s (INV: folded into E and O)
    struct Col { cf32 e, o; };
    auto fetch = [&](int s) {
        Col v{{0.f, 0.f}, {0.f, 0.f}};
        const int j = 4 * s + kq;
        if (ok && j < J) {
            v.e = src[(int64_t)j * sij];
            if (INV && j > 0 && 2 * j < L) v.o = src[(int64_t)(L - j) * sij];
        }
        return v;
    };
    Col cur[kTwPK];
#pragma unroll
    for (int p = 0; p < kTwPK; ++p) cur[p] = fetch(p);
    // forward: C and S (real, imaginary); inverse: the output's real and imaginary part
    constexpr int NA = INV ? 2 : 4;
    f4v acc[NI][NA];
#pragma unroll
    for (int t = 0; t < NI; ++t)
#pragma unroll
        for (int q = 0; q < NA; ++q) acc[t][q] = f4v{0.f, 0.f, 0.f, 0.f};
    for (int k0 = 0; k0 < ks; k0 += kTwKS) {
        const int kn = min(kTwKS, ks - k0);
        if (k0 > 0) __syncthreads();
        for (int t = 0; t < NI; ++t) {
            float4* dst4 = reinterpret_cast<float4*>(wl + t * kTwKS * 64);
            const float4* src4 = reinterpret_cast<const float4*>(tab + ((int64_t)(t0 + t) * ks + k0) * 64);
            for (int q = threadIdx.x; q < kn * 32; q += 256)
                dst4[q] = t0 + t < tiles ? src4[q] : make_float4(0.f, 0.f, 0.f, 0.f);
        }
        __syncthreads();
        if (!active) continue;
        for (int s0 = 0; s0 < kn; s0 += kTwPK) {
#pragma unroll
            for (int p = 0; p < kTwPK; ++p) {
                const int st = s0 + p;
                if (st >= kn) break;                      // wave-uniform
                const Col v = cur[p];
                cur[p] = fetch(k0 + st + kTwPK);
                float er = v.e.re, ei = v.e.im, orr = 0.f, oi = 0.f;
                if constexpr (INV) {
                    // an unmirrored index (0, L / 2) has sin = 0: its O is not used
                    er += v.o.re;
                    ei += v.o.im;
                    orr = v.e.re - v.o.re;
                    oi = v.o.im - v.e.im;                 // -O.im
                }
#pragma unroll
                for (int t = 0; t < NI; ++t) {
                    const cf32 w = wl[(t * kTwKS + st) * 64 + lane];   // (cos, sin)
                    if constexpr (INV) {
                        acc[t][0] = __builtin_amdgcn_mfma_f32_16x16x4f32(w.re, er, acc[t][0], 0, 0, 0);
                        acc[t][1] = __builtin_amdgcn_mfma_f32_16x16x4f32(w.re, ei, acc[t][1], 0, 0, 0);
                        acc[t][0] = __builtin_amdgcn_mfma_f32_16x16x4f32(w.im, oi, acc[t][0], 0, 0, 0);
                        acc[t][1] = __builtin_amdgcn_mfma_f32_16x16x4f32(w.im, orr, acc[t][1], 0, 0, 0);
                    } else {
                        acc[t][0] = __builtin_amdgcn_mfma_f32_16x16x4f32(w.re, er, acc[t][0], 0, 0, 0);
                        acc[t][1] = __builtin_amdgcn_mfma_f32_16x16x4f32(w.re, ei, acc[t][1], 0, 0, 0);
                        acc[t][2] = __builtin_amdgcn_mfma_f32_16x16x4f32(w.im, er, acc[t][2], 0, 0, 0);
                        acc[t][3] = __builtin_amdgcn_mfma_f32_16x16x4f32(w.im, ei, acc[t][3], 0, 0, 0);
                    }
                }
            }
        }
    }
    if (!ok) return;
    cf32* dst = out + (int64_t)b * sob + c;
#pragma unroll
    for (int t = 0; t < NI; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int i = 16 * (t0 + t) + 4 * kq + r;
            if constexpr (INV) {
                if (i < n) dst[(int64_t)i * soi] = cf32{acc[t][0][r], acc[t][1][r]};
            } else {
                const float cr = acc[t][0][r], ci = acc[t][1][r], sr = acc[t][2][r], si = acc[t][3][r];
                if (2 * i <= L) dst[(int64_t)i * soi] = cf32{cr + si, ci - sr};
                if (i > 0 && 2 * i < L) dst[(int64_t)(L - i) * soi] = cf32{cr - si, ci + sr};
            }
        }
}

// One lateral product over B batches of C channels: forward n -> L indices or
// inverse L -> n.
template <bool INV>
static void twiddle(cf32* out, const cf32* in, const cf32* tab, int B, int L, int n, int C, int64_t sib,
                    int64_t sij, int64_t sob, int64_t soi, hipStream_t s) {
    const int rows = INV ? n : L / 2 + 1, J = INV ? L / 2 + 1 : n;
    const int tiles = (rows + 15) / 16, ks = (J + 3) / 4;
    const int nct = (C + 15) / 16;
    const int64_t units = (int64_t)B * nct;
    // row tiles per wave: as many as the accumulators allow, fewer (more waves,
    // each input column read by more of them) while the launch has under 2048 waves
    int ni = std::min(tiles, kTwMaxNI);
    while (ni > 1 && units * ((tiles + ni - 1) / ni) < 2048) --ni;
    while (ni > 1 && (tiles + ni - 2) / (ni - 1) == (tiles + ni - 1) / ni) --ni;   // the same rounds with fewer
    const dim3 grid((unsigned)((units + 3) / 4), (tiles + ni - 1) / ni);
#define UFSS_TW(T) hipLaunchKernelGGL((twiddle_kernel<T, INV>), grid, dim3(256), 0, s, out, in, tab, L, n, ks, tiles, \
                                      (int)units, nct, C, sib, sij, sob, soi)
    if (ni == 1) UFSS_TW(1); else if (ni == 2) UFSS_TW(2); else if (ni == 3) UFSS_TW(3); else UFSS_TW(4);
#undef UFSS_TW
    UFSS_HIP(hipGetLastError());
}

// The transform indices (q_y, q_x) that share the stored entry (oy, ox): q_y = oy
// or ly - oy (a) and q_x = ox or lx - ox (b), one of each on an axis's
// self-mirrored entries, and, where the axes are alike (SWAP), the same with
// the axes exchanged.  Up to 4, or 8 with SWAP.
struct Orbit {
    int oy, ox, ly, lx, nx2, n4, n;
    __device__ Orbit(int2 o, int ly_, int lx_, bool swap) : oy(o.x), ox(o.y), ly(ly_), lx(lx_) {
        const int ny2 = (oy == 0 || 2 * oy == ly) ? 1 : 2;
        nx2 = (ox == 0 || 2 * ox == lx) ? 1 : 2;
        n4 = ny2 * nx2;
        n = swap && oy != ox ? 2 * n4 : n4;
    }
    // row index q_y lx + q_x of member q
    __device__ int64_t row(int q) const {
        const int e = q >= n4, w = q - e * n4;
        const int a = w / nx2, b = w - a * nx2;
        const int qa = a ? ly - oy : oy, qb = b ? lx - ox : ox;
        return e ? (int64_t)qb * lx + qa : (int64_t)qa * lx + qb;
    }
};

// Contraction, both directions, on one stored table K^[o][z][k] (rows of k
// padded to an even stride): forward out[q][k] = sum_z K^[o][z][k] in[q][z],
// adjoint out[q][z] = sum_k conj(K^[o][z][k]) in[q][k] for the members q of
// entry o.
//
// What bounds it: the table, read once per apply.  It runs on the FP32 matrix
// cores because they do what the two directions need on one layout: with
// v_mfma_f32_16x16x4f32 the 16 columns are the real and imaginary parts of up to
// 8 members, the rows 16 outputs and the reduction 4 entries, so the adjoint
// reduces along the contiguous index without a transposed copy of the table,
// and an entry loaded once serves all members (8 FMAs per byte, 20 TB/s of
// table at the FP32 matrix rate; the earlier vector form took 4 members, a
// transposed copy and a broadcast LDS read per entry and member).  A complex
// product is two real ones into one accumulator: K_re times the column, K_im
// times the neighbouring column with a sign.
//   forward: lane l loads entries (z = 4 s + l / 16, k = 2 (l % 16), + 1) of 32
//   outputs: two tiles of 16 rows, rows 2 i and 2 i + 1
//   adjoint: lane l loads entries (z = l % 16, k = 16 s + 4 (l / 16) .. + 3): one
//   tile of 16 rows, four steps of the reduction, 128 contiguous bytes per row
// A workgroup of kNW waves takes one entry and a block of its outputs; a wave
// takes one group of TB tiles (16-byte loads kPD steps ahead)
// and, where there are fewer groups than waves, a share of the reduction,
// summed over the waves in LDS in fixed order.  Members are staged in LDS, kRC
// reduction entries at a time, zero past the last; lanes past the last output
// or the last reduction entry load some other finite entry (the table is
// followed by zeros), which meets a zero column or a row that is not stored.
//
// Per launch, forward / adjoint, before (quadrant, vector FMAs) and now: 64 x
// 64 x 512 (128 bins, W = 16) 181 / 176 -> 94 / 100 us (4.8 TB/s of table), 32 x
// 32 x 256 (66 bins, full) 27.5 / 27.3 -> 17.6 / 19.7, 50 x 50 x 50 (256 bins) 53 /
// 52 -> 28 / 26.5; unequal axes (45 x 51 x 301, 76 bins) 45 / 51 -> 35 / 38.
static constexpr int kPD = 2;
static constexpr int kNW = 4;
static constexpr int kRC = 512;
static constexpr int kSeg = 32;          // steps per first-level sum (a multiple of kPD): shorter chains round less

// Outputs of one group (TB tiles), and reduction entries of a step.
__host__ __device__ constexpr int group_rows(bool fwd, int tb) { return (fwd ? 32 : 16) * tb; }
__host__ __device__ constexpr int step_len(bool fwd, bool bf16) { return fwd && !bf16 ? 4 : 16; }

template <bool FWD, int TB, bool SWAP>
__global__ __launch_bounds__(64 * kNW) void contract_kernel(const cf32* __restrict__ tab, const int2* __restrict__ orbits,
                                                       const cf32* __restrict__ in, cf32* __restrict__ out,
                                                       int ly, int lx, int nz, int mus, int C, int R, int groups) {
    extern __shared__ __align__(16) unsigned char smem[];
    float* xs = reinterpret_cast<float*>(smem);               // [kRC][RS] members' columns
    float* red = xs;                                          // [shares][16][rows + 1] after the reduction
    constexpr int NQ = SWAP ? 8 : 4, RS = 2 * NQ + 2;
    constexpr int GR = group_rows(FWD, TB), ND = FWD ? 2 * TB : TB, ST = step_len(FWD, false), NL = FWD ? 1 : 2;
    const Orbit orb(orbits[blockIdx.x], ly, lx, SWAP);
    const int nq = orb.n;
    const cf32* tb = tab + (int64_t)blockIdx.x * nz * mus;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int c0 = blockIdx.y * groups * GR;                  // first output of the block
    const int ng = min(groups, (C - c0 + GR - 1) / GR);       // its groups (1..kNW)
    const int shares = kNW / ng;                              // waves per group
    const int grp = wave % ng, share = wave / ng;
    const bool active = share < shares;
    const int i = lane & 15, kq = lane >> 4;
    const int gc0 = c0 + grp * GR;
    // columns: member i / 2, real (even) or imaginary part; the K_im product
    // takes the other part, negative where the (conjugated) product says so
    const int col = SWAP ? i : (i & 7);
    const float sgn = (FWD == ((i & 1) == 0)) ? -1.f : 1.f;
    auto other = [&](float b) {
        return sgn * __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(b), 0xB1, 0xf, 0xf, true));
    };

    f4v D[ND], sum[ND];                                       // of kSeg steps, of those before
#pragma unroll
    for (int t = 0; t < ND; ++t) D[t] = sum[t] = f4v{0.f, 0.f, 0.f, 0.f};
    // this lane's entries of step 0, and what a step and a tile add
    int off[TB];
#pragma unroll
    for (int t = 0; t < TB; ++t)
        off[t] = FWD ? kq * mus + min(gc0 + 32 * t + 2 * i, mus - 2) : min(gc0 + 16 * t + i, nz - 1) * mus + 4 * kq;
    f4v buf[kPD][TB][NL];                                     // two entries each
    auto load = [&](f4v (&b)[TB][NL], int r0, int st) {
        const cf32* p = tb + (FWD ? (int64_t)(r0 + 4 * st) * mus : (int64_t)(r0 + 16 * st));
#pragma unroll
        for (int t = 0; t < TB; ++t)
#pragma unroll
            for (int h = 0; h < NL; ++h) b[t][h] = *reinterpret_cast<const f4v*>(p + off[t] + 2 * h);
    };
    for (int r0 = 0; r0 < R; r0 += kRC) {
        const int rc = min(kRC, R - r0), nst = (rc + ST - 1) / ST;
#pragma unroll
        for (int p = 0; p < kPD; ++p)
            if (active && share + p * shares < nst) load(buf[p], r0, share + p * shares);
        if (r0 > 0) __syncthreads();                          // the previous chunk's columns are read
        for (int r = threadIdx.x; r < nst * ST; r += 64 * kNW) {
            cf32 v[NQ];
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                v[q] = cf32{0.f, 0.f};
                if (q < nq && r < rc) v[q] = in[orb.row(q) * R + r0 + r];
            }
#pragma unroll
            for (int q = 0; q < NQ; ++q) *reinterpret_cast<cf32*>(xs + r * RS + 2 * q) = v[q];
        }
        __syncthreads();
        if (!active) continue;
        for (int sg = share; sg < nst; sg += kSeg * shares) {
            for (int st0 = sg; st0 < min(nst, sg + kSeg * shares); st0 += kPD * shares) {
#pragma unroll
                for (int p = 0; p < kPD; ++p) {
                    const int st = st0 + p * shares;
                    if (st >= nst) break;                         // wave-uniform
                    const float* xr = xs + (FWD ? 4 * st + kq : 16 * st + 4 * kq) * RS + col;
                    if constexpr (FWD) {
                        const float b0 = xr[0], o0 = other(b0);
#pragma unroll
                        for (int t = 0; t < TB; ++t) {
                            const f4v a = buf[p][t][0];
                            D[2 * t] = __builtin_amdgcn_mfma_f32_16x16x4f32(a.x, b0, D[2 * t], 0, 0, 0);
                            D[2 * t + 1] = __builtin_amdgcn_mfma_f32_16x16x4f32(a.z, b0, D[2 * t + 1], 0, 0, 0);
                            D[2 * t] = __builtin_amdgcn_mfma_f32_16x16x4f32(a.y, o0, D[2 * t], 0, 0, 0);
                            D[2 * t + 1] = __builtin_amdgcn_mfma_f32_16x16x4f32(a.w, o0, D[2 * t + 1], 0, 0, 0);
                        }
                    } else {
#pragma unroll
                        for (int h = 0; h < NL; ++h) {
                            const float b0 = xr[2 * h * RS], b1 = xr[(2 * h + 1) * RS], o0 = other(b0), o1 = other(b1);
                            f4v a[TB];
#pragma unroll
                            for (int t = 0; t < TB; ++t) a[t] = buf[p][t][h];
#pragma unroll
                            for (int t = 0; t < TB; ++t) D[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[t].x, b0, D[t], 0, 0, 0);
#pragma unroll
                            for (int t = 0; t < TB; ++t) D[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[t].y, o0, D[t], 0, 0, 0);
#pragma unroll
                            for (int t = 0; t < TB; ++t) D[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[t].z, b1, D[t], 0, 0, 0);
#pragma unroll
                            for (int t = 0; t < TB; ++t) D[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[t].w, o1, D[t], 0, 0, 0);
                        }
                    }
                    if (st + kPD * shares < nst) load(buf[p], r0, st + kPD * shares);
                }
            }
#pragma unroll
            for (int t = 0; t < ND; ++t) {
                sum[t] += D[t];
                D[t] = f4v{0.f, 0.f, 0.f, 0.f};
            }
        }
    }
    __syncthreads();                                          // the columns are read; red takes their place
    const int rows = min(groups * GR, C - c0), pitch = ng * GR + 1;
    if (active) {
#pragma unroll
        for (int t = 0; t < ND; ++t)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int lr = FWD ? 32 * (t >> 1) + 2 * (4 * kq + r) + (t & 1) : 16 * t + 4 * kq + r;
                red[(share * 16 + i) * pitch + grp * GR + lr] = sum[t][r];
            }
    }
    __syncthreads();
    for (int t = threadIdx.x; t < nq * rows; t += 64 * kNW) {
        const int q = t / rows, c = t - q * rows;
        float re = 0.f, im = 0.f;
        for (int h = 0; h < shares; ++h) {
            re += red[(h * 16 + 2 * q) * pitch + c];
            im += red[(h * 16 + 2 * q + 1) * pitch + c];
        }
        out[orb.row(q) * C + c0 + c] = cf32{re, im};
    }
}

// The same on a BF16 table, with the BF16 matrix cores: v_mfma_f32_16x16x32_bf16
// takes 16 reduction entries a step, (re, im) after one another as they lie in the
// table, against columns that hold (Xre, -+Xim) for a real and (Xim, +-Xre) for an
// imaginary part.  The FP32 members are cut into three BF16 parts (8 leading bits, the
// next 8, the last 8: their sum is the member), so every product is exact and the sums
// stay FP32; where an entry has at most 4 members, the first two parts share a product
// (columns 0-7 and 8-15).  2 or 3 products of 16 cycles take the place of 8 FP32 ones
// of 32, which bounded this kernel (its table is half the FP32 one's): forward / adjoint
// 32 x 32 x 256, 66 bins 20.0 / 17.1 -> 12.8 / 13.9 us, 45 x 51 x 301, 76 bins 32.8 / 30.8 ->
// 21.1 / 23.1 (4.7 / 4.3 TB/s of table), 64 x 64 x 512, 128 bins 57 / 60 -> 44 / 54.
//   forward: lane l loads entries (z = 16 s + 4 (l / 16) .. + 3, k = 2 (l % 16), + 1) of
//   32 outputs: two tiles, rows 2 i and 2 i + 1
//   adjoint: lane l loads entries (z = l % 16, k = 16 s + 4 (l / 16) .. + 3)
// The matrix cores take BF16 values below 2^-126 as zero, which the second and third
// parts of members below 2^-103 can be: where all members of an entry are below 2^-63
// (kSizable, the upper exponent bits, none set) they are cut once more at 2^64 times
// their size and the sums scaled back.  (Next to a larger member each loses under 2^-63
// of that one.)  The sizes are looked at beside the outputs' sums, where it takes under
// 0.5 us: 13.1 / 14.6, 21.9 / 24.3 and 44 / 50 us for the three scans above with members
// of order one, 13.1 / 14.5, 21.9 / 23.8 and 44 / 50 without.
// Columns in LDS: plane, group of 4 entries, column, 4 entries of (re, im): one 16-byte
// read per operand; groups padded by 16 bytes against bank conflicts of the staging.
typedef __bf16 bf8v __attribute__((ext_vector_type(8)));
typedef unsigned int u4v __attribute__((ext_vector_type(4)));
static constexpr int kRB = 256;                               // reduction entries staged at a time
static constexpr int kGP = 16 * 16 + 16;                      // bytes of a group of 4 entries
static constexpr float kLarger = 0x1p64f;
static constexpr unsigned kSizable = 0x60000000u;

template <bool FWD, int TB, bool SWAP>
__global__ __launch_bounds__(64 * kNW) void contract_bf16_kernel(const cbf16* __restrict__ tab, const int2* __restrict__ orbits,
                                                       const cf32* __restrict__ in, cf32* __restrict__ out,
                                                       int ly, int lx, int nz, int mus, int C, int R, int groups) {
    static_assert(kRB == 64 * kNW && kNW == 4, "a thread stages one reduction entry, an int4 holds the waves' sizes");
    __shared__ __align__(16) int sizes[kNW];
    extern __shared__ __align__(16) unsigned char smem[];
    float* red = reinterpret_cast<float*>(smem);              // [shares][16][rows + 1] after the reduction
    constexpr int NQ = SWAP ? 8 : 4, NPL = SWAP ? 3 : 2;
    constexpr int GR = group_rows(FWD, TB), ND = FWD ? 2 * TB : TB, ST = step_len(FWD, true), NL = FWD ? 4 : 2;
    const Orbit orb(orbits[blockIdx.x], ly, lx, SWAP);
    const int nq = orb.n;
    const cbf16* tb = tab + (int64_t)blockIdx.x * nz * mus;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int c0 = blockIdx.y * groups * GR;                  // first output of the block
    const int ng = min(groups, (C - c0 + GR - 1) / GR);       // its groups (1..kNW)
    const int shares = kNW / ng;                              // waves per group
    const int grp = wave % ng, share = wave / ng;
    const bool active = share < shares;
    const int i = lane & 15, kq = lane >> 4;
    const int gc0 = c0 + grp * GR;

    f4v D[ND];
    int off[TB];
#pragma unroll
    for (int t = 0; t < TB; ++t)
        off[t] = FWD ? 4 * kq * mus + min(gc0 + 32 * t + 2 * i, mus - 2) : min(gc0 + 16 * t + i, nz - 1) * mus + 4 * kq;
    uint2 buf[kPD][TB][NL];                                   // two entries each
    auto load = [&](uint2 (&b)[TB][NL], int r0, int st) {
        const cbf16* p = tb + (FWD ? (int64_t)(r0 + 16 * st) * mus : (int64_t)(r0 + 16 * st));
#pragma unroll
        for (int t = 0; t < TB; ++t)
#pragma unroll
            for (int h = 0; h < NL; ++h) b[t][h] = *reinterpret_cast<const uint2*>(p + off[t] + h * (FWD ? mus : 2));
    };
    float scale = 1.f;
    unsigned bits = 0;                                        // all bits of this thread's members
    for (;;) {
#pragma unroll
        for (int t = 0; t < ND; ++t) D[t] = f4v{0.f, 0.f, 0.f, 0.f};
        for (int r0 = 0; r0 < R; r0 += kRB) {
            const int rc = min(kRB, R - r0), nst = (rc + ST - 1) / ST;
#pragma unroll
            for (int p = 0; p < kPD; ++p)
                if (active && share + p * shares < nst) load(buf[p], r0, share + p * shares);
            if (r0 > 0) __syncthreads();                          // the previous chunk's columns are read
            const int r = threadIdx.x;
            if (r < nst * ST) {
                unsigned char* dst = smem + (r >> 2) * kGP + (r & 3) * 4;
                auto put = [&](int plane, int col, float a, float b) {       // the top halves of a and b
                    *reinterpret_cast<unsigned*>(dst + plane * (kRB / 4) * kGP + col * 16) =
                        (__float_as_uint(a) >> 16) | (__float_as_uint(b) & 0xffff0000u);
                };
                auto top = [](float a) { return __uint_as_float(__float_as_uint(a) & 0xffff0000u); };
                cf32 v[NQ];
#pragma unroll
                for (int q = 0; q < NQ; ++q) {
                    v[q] = cf32{0.f, 0.f};
                    if (q < nq && r < rc) v[q] = in[orb.row(q) * R + r0 + r];
                }
#pragma unroll
                for (int q = 0; q < NQ; ++q) {
                    bits |= __float_as_uint(v[q].re) | __float_as_uint(v[q].im);
                    float re = v[q].re, im = v[q].im;
                    if (scale != 1.f) {                           // uniform
                        re *= scale;
                        im *= scale;
                    }
#pragma unroll
                    for (int part = 0; part < 3; ++part) {
                        const float tr = top(re), ti = top(im);
                        const int plane = SWAP ? part : part >> 1, col = 2 * q + (SWAP ? 0 : 8 * (part & 1));
                        put(plane, col, tr, FWD ? -ti : ti);
                        put(plane, col + 1, ti, FWD ? tr : -tr);
                        re -= tr;
                        im -= ti;
                    }
                    if (!SWAP) {
                        put(1, 8 + 2 * q, 0.f, 0.f);
                        put(1, 9 + 2 * q, 0.f, 0.f);
                    }
                }
            }
            __syncthreads();
            if (!active) continue;
            for (int st0 = share; st0 < nst; st0 += kPD * shares) {
#pragma unroll
                for (int p = 0; p < kPD; ++p) {
                    const int st = st0 + p * shares;
                    if (st >= nst) break;                         // wave-uniform
                    const unsigned char* src = smem + (4 * st + kq) * kGP + i * 16;
                    bf8v b[NPL], a[ND];
#pragma unroll
                    for (int w = 0; w < NPL; ++w) b[w] = *reinterpret_cast<const bf8v*>(src + w * (kRB / 4) * kGP);
#pragma unroll
                    for (int t = 0; t < TB; ++t) {
                        const uint2* e = buf[p][t];
                        if constexpr (FWD) {
                            a[2 * t] = __builtin_bit_cast(bf8v, u4v{e[0].x, e[1].x, e[2].x, e[3].x});
                            a[2 * t + 1] = __builtin_bit_cast(bf8v, u4v{e[0].y, e[1].y, e[2].y, e[3].y});
                        } else {
                            a[t] = __builtin_bit_cast(bf8v, u4v{e[0].x, e[0].y, e[1].x, e[1].y});
                        }
                    }
                    // smallest parts first
#pragma unroll
                    for (int w = NPL - 1; w >= 0; --w)
#pragma unroll
                        for (int t = 0; t < ND; ++t) D[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[t], b[w], D[t], 0, 0, 0);
                    if (st + kPD * shares < nst) load(buf[p], r0, st + kPD * shares);
                }
            }
        }
        if (scale == 1.f) {
            const int size = (__any(bits & kSizable) ? 1 : 0) | (__any(bits & 0x7fffffffu) ? 2 : 0);
            if (lane == 0) sizes[wave] = size;
        }
        __syncthreads();                                      // the columns are read; red takes their place
        const int rows = min(groups * GR, C - c0), pitch = ng * GR + 1;
        if (active) {
            const float back = 1.f / scale;
#pragma unroll
            for (int t = 0; t < ND; ++t)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int lr = FWD ? 32 * (t >> 1) + 2 * (4 * kq + r) + (t & 1) : 16 * t + 4 * kq + r;
                    red[(share * 16 + i) * pitch + grp * GR + lr] = D[t][r] * back;
                }
        }
        __syncthreads();
        const int4 w4 = *reinterpret_cast<const int4*>(sizes);
        for (int t = threadIdx.x; t < nq * rows; t += 64 * kNW) {
            const int q = t / rows, c = t - q * rows;
            float re = 0.f, im = 0.f;
            for (int h = 0; h < shares; ++h)
#pragma unroll
                for (int w = 0; w < (SWAP ? 1 : 2); ++w) {
                    re += red[(h * 16 + 8 * w + 2 * q) * pitch + c];
                    im += red[(h * 16 + 8 * w + 2 * q + 1) * pitch + c];
                }
            out[orb.row(q) * C + c0 + c] = cf32{re, im};
        }
        if (scale != 1.f || __builtin_amdgcn_readfirstlane(w4.x | w4.y | w4.z | w4.w) != 2) break;
        scale = kLarger;                                      // small members only: once more
        __syncthreads();                                      // red is read; the columns take its place
    }
}

// ---- plan-time construction of K^ (FP64) -------------------------------------
// P64[dy][dx][z][k] = g(dx, dy, z) exp(-j 2 pi (kb[k] u(dy, dx, z) mod 2^32) / 2^32)
__global__ void phasor64_kernel(const uint32_t* __restrict__ u, const float* __restrict__ amp,
                                const int* __restrict__ kb, int64_t ncell, int mu,
                                double2* __restrict__ out) {
    const int64_t n = ncell * mu;
    for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < n;
         t += (int64_t)gridDim.x * blockDim.x) {
        const int64_t cell = t / mu;
        const int k = (int)(t - cell * mu);
        const uint32_t ph = (uint32_t)kb[k] * u[cell];
        const double turns = (double)ph * (1.0 / 4294967296.0);
        double sn, cs;
        sincos(2.0 * M_PI * turns, &sn, &cs);
        const double g = amp ? (double)amp[cell] : 1.0;
        out[t] = double2{g * cs, -g * sn};
    }
}

// The two cosine transforms of the build take kBI outputs per thread: each FP64
// input is loaded once for them (32 x 32 C-scan: 0.6 + 0.7 ms of the plan with
// one output per thread).
static constexpr int kBI = 8;

// out[b][i][c] = sum_j C[i][j] in[b][j][c] with a real FP64 weight table (over d_x).
__global__ __launch_bounds__(256) void cos_kernel(double2* __restrict__ out, const double2* __restrict__ in,
                                                  const double* __restrict__ Cw, int I, int J,
                                                  int64_t C, int64_t sib, int64_t sij,
                                                  int64_t sob, int64_t soi) {
    const int64_t c = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int i0 = blockIdx.y * kBI, b = blockIdx.z;
    if (c >= C) return;
    double re[kBI], im[kBI];
#pragma unroll
    for (int t = 0; t < kBI; ++t) re[t] = im[t] = 0.0;
    const double2* src = in + (int64_t)b * sib + c;
    for (int j = 0; j < J; ++j) {
        const double2 v = src[(int64_t)j * sij];
#pragma unroll
        for (int t = 0; t < kBI; ++t) {
            const double w = Cw[(int64_t)min(i0 + t, I - 1) * J + j];
            re[t] += w * v.x;
            im[t] += w * v.y;
        }
    }
#pragma unroll
    for (int t = 0; t < kBI; ++t)
        if (i0 + t < I) out[(int64_t)b * sob + (int64_t)(i0 + t) * soi + c] = double2{re[t], im[t]};
}

// Index of the stored entry (oy, ox) (SWAP: oy <= ox), rows of oy one after another.
__host__ __device__ static inline int entry_index(int oy, int ox, int nox, bool swap) {
    return swap ? oy * nox - oy * (oy - 1) / 2 + ox - oy : oy * nox + ox;
}

// The stored table: T[(oy, ox)][z][k] = sum_dy hy[oy][dy] S[dy][ox][z][k], rounded
// to FP32 (and from there to BF16), rows of k padded with zeros to the stride mus.
__device__ __forceinline__ void put(cf32* t, float re, float im) { *t = cf32{re, im}; }
__device__ __forceinline__ void put(cbf16* t, float re, float im) { *t = to_cbf16(re, im); }

template <typename TT>
__global__ __launch_bounds__(256) void table_kernel(TT* __restrict__ tab, const double2* __restrict__ S,
                                                    const double* __restrict__ hy, int J, int nox, int noy, int swap,
                                                    int nz, int mu, int mus) {
    const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int ox = blockIdx.y, oy0 = blockIdx.z * kBI;
    const int oy_end = swap ? min(noy, ox + 1) : noy;
    if (t >= (int64_t)nz * mus || oy0 >= oy_end) return;
    const int z = (int)(t / mus), k = (int)(t - (int64_t)z * mus);
    double re[kBI], im[kBI];
#pragma unroll
    for (int i = 0; i < kBI; ++i) re[i] = im[i] = 0.0;
    if (k < mu) {
        const int64_t zc = (int64_t)nz * mu;
        const double2* src = S + (int64_t)ox * zc + (int64_t)z * mu + k;
        for (int j = 0; j < J; ++j) {
            const double2 v = src[(int64_t)j * nox * zc];
#pragma unroll
            for (int i = 0; i < kBI; ++i) {
                const double w = hy[(int64_t)min(oy0 + i, noy - 1) * J + j];
                re[i] += w * v.x;
                im[i] += w * v.y;
            }
        }
    }
#pragma unroll
    for (int i = 0; i < kBI; ++i) {
        if (oy0 + i >= oy_end) break;
        // two roundings, as FP32 plans followed by a conversion: the compiler would
        // otherwise round FP64 to BF16 at once, another value in the FP32 ties
        float fr = (float)re[i], fi = (float)im[i];
        asm volatile("" : "+v"(fr), "+v"(fi));
        put(tab + (int64_t)entry_index(oy0 + i, ox, nox, swap) * nz * mus + t, fr, fi);
    }
}

// Cyclic transform size per axis: the smallest L >= N + W (and >= 1).
static int fft_len(int n, int w) { return std::max(1, n + w); }

int64_t fft_table_bytes(const Plan& P) {
    const int lx = fft_len(P.g.nx, P.d.wx), ly = fft_len(P.g.ny, P.d.wy);
    return (int64_t)(ly / 2 + 1) * (lx / 2 + 1) * P.g.nz * (int64_t)P.ubins_h.size() * 8;
}

static constexpr int64_t kFftTableMax = int64_t(32) << 30;

void fft_setup(Plan& P) {
    const int nx = P.g.nx, ny = P.g.ny, nz = P.g.nz, wx = P.d.wx, wy = P.d.wy;
    const int mu = (int)P.ubins_h.size();
    const int lx = fft_len(nx, wx), ly = fft_len(ny, wy);
    const int nox = lx / 2 + 1, noy = ly / 2 + 1;
    if (fft_table_bytes(P) > kFftTableMax)
        fail(UFSS_ERR_UNSUPPORTED, "transform table larger than 32 GiB");
    // the sizes that the path takes and is tested up to; its kernels stage chunks of a
    // fixed size and set no limit of their own near these
    if (std::max(lx, ly) > 1024 || std::max(nz, mu) > 1536)
        fail(UFSS_ERR_UNSUPPORTED, "grid too large for the transform path (L <= 1024, nz and bins <= 1536)");
    P.fft_lx = lx;
    P.fft_ly = ly;
    // twiddle tables (FP64 angles from exact integer products, stored FP32) in
    // operand order (see twiddle_kernel)
    auto tw = [](int rows, int cols, int L, double scale) {
        const int tiles = (rows + 15) / 16, ks = (cols + 3) / 4;
        std::vector<cf32> t((size_t)tiles * ks * 64, cf32{0.f, 0.f});
        for (int T = 0; T < tiles; ++T)
            for (int st = 0; st < ks; ++st)
                for (int l = 0; l < 64; ++l) {
                    const int r = 16 * T + (l & 15), c = 4 * st + (l >> 4);
                    if (r >= rows || c >= cols) continue;
                    const int64_t k = ((int64_t)r * c) % L;
                    const double a = 2.0 * M_PI * (double)k / L;
                    // sin(pi) and sin(0) exactly zero: those indices have no mirror
                    t[((size_t)T * ks + st) * 64 + l] = cf32{(float)(scale * std::cos(a)), 2 * k % L == 0 ? 0.f : (float)(scale * std::sin(a))};
                }
        return t;
    };
    auto up = [&](const std::vector<cf32>& h) {
        void* d = nullptr;
        UFSS_HIP(hipMalloc(&d, h.size() * sizeof(cf32)));
        UFSS_HIP(hipMemcpy(d, h.data(), h.size() * sizeof(cf32), hipMemcpyHostToDevice));
        P.ws_bytes += h.size() * sizeof(cf32);
        return static_cast<cf32*>(d);
    };
    P.d_tw_fx = up(tw(lx / 2 + 1, nx, lx, 1.0));          // [qx][nx]
    P.d_tw_fy = up(tw(ly / 2 + 1, ny, ly, 1.0));          // [qy][ny]
    P.d_tw_ix = up(tw(nx, lx / 2 + 1, lx, 1.0 / lx));     // [px][qx]
    P.d_tw_iy = up(tw(ny, ly / 2 + 1, ly, 1.0 / ly));     // [py][qy]
    const int64_t cmax = std::max(nz, mu);
    const int64_t wbytes = (int64_t)ly * lx * cmax * sizeof(cf32);
    const int64_t tbytes = (int64_t)std::max((int64_t)ny * lx, (int64_t)ly * nx) * cmax * sizeof(cf32);
    UFSS_HIP(hipMalloc(&P.d_fa, wbytes));
    UFSS_HIP(hipMalloc(&P.d_fb, wbytes));
    UFSS_HIP(hipMalloc(&P.d_ft, tbytes));
    P.ws_bytes += 2 * wbytes + tbytes;

    // stored entries: the quadrant, or, with both axes alike (K^ is then symmetric
    // in q_y and q_x: half the table), its part oy <= ox
    P.fft_swap = lx == ly && wx == wy && P.g.dx == P.g.dy;
    P.fft_mus = (mu + 1) & ~1;
    std::vector<int2> orb;
    for (int oy = 0; oy < noy; ++oy)
        for (int ox = P.fft_swap ? oy : 0; ox < nox; ++ox) orb.push_back(int2{oy, ox});
    P.fft_entries = (int)orb.size();
    UFSS_HIP(hipMalloc(&P.d_orb, orb.size() * sizeof(int2)));
    UFSS_HIP(hipMemcpy(P.d_orb, orb.data(), orb.size() * sizeof(int2), hipMemcpyHostToDevice));

    // K^ in FP64: phasors, cosine transform over d_x, then over d_y into the table
    const int64_t ncell = (int64_t)(wy + 1) * (wx + 1) * nz;
    const int64_t zc = (int64_t)nz * mu;                 // channels (z, k)
    const int64_t row = (int64_t)nz * P.fft_mus;         // table values per entry
    const size_t tbytes1 = P.dtype == UFSS_BF16 ? sizeof(cbf16) : sizeof(cf32);
    double2 *p64 = nullptr, *s64 = nullptr;
    double *cx = nullptr, *cy = nullptr;
    std::vector<double> hx((size_t)nox * (wx + 1)), hy((size_t)noy * (wy + 1));
    for (int q = 0; q < nox; ++q)
        for (int d = 0; d <= wx; ++d)
            hx[(size_t)q * (wx + 1) + d] = (d == 0 ? 1.0 : 2.0) * std::cos(2.0 * M_PI * (double)(((int64_t)q * d) % lx) / lx);
    for (int q = 0; q < noy; ++q)
        for (int d = 0; d <= wy; ++d)
            hy[(size_t)q * (wy + 1) + d] = (d == 0 ? 1.0 : 2.0) * std::cos(2.0 * M_PI * (double)(((int64_t)q * d) % ly) / ly);
    auto release = [&]() {
        if (p64) (void)hipFree(p64);
        if (s64) (void)hipFree(s64);
        if (cx) (void)hipFree(cx);
        if (cy) (void)hipFree(cy);
    };
    try {
        UFSS_HIP(hipMalloc(&p64, ncell * mu * sizeof(double2)));
        UFSS_HIP(hipMalloc(&s64, (int64_t)(wy + 1) * nox * zc * sizeof(double2)));
        UFSS_HIP(hipMalloc(&cx, hx.size() * sizeof(double)));
        UFSS_HIP(hipMalloc(&cy, hy.size() * sizeof(double)));
        // the contraction may load up to a step past the last entry's rows
        const int64_t slack = 16 * P.fft_mus + 16;
        UFSS_HIP(hipMalloc(&P.d_khat, (P.fft_entries * row + slack) * tbytes1));
        UFSS_HIP(hipMemset(static_cast<char*>(P.d_khat) + P.fft_entries * row * tbytes1, 0, slack * tbytes1));
        P.ws_bytes += (P.fft_entries * row + slack) * (int64_t)tbytes1 + P.fft_entries * (int64_t)sizeof(int2);
        UFSS_HIP(hipMemcpy(cx, hx.data(), hx.size() * sizeof(double), hipMemcpyHostToDevice));
        UFSS_HIP(hipMemcpy(cy, hy.data(), hy.size() * sizeof(double), hipMemcpyHostToDevice));
        const int64_t n = ncell * mu;
        const int blocks = (int)std::min<int64_t>((n + 255) / 256, 65536);
        hipLaunchKernelGGL(phasor64_kernel, dim3(blocks), dim3(256), 0, nullptr, P.d_u, P.d_amp,
                           P.d_ubins, ncell, mu, p64);
        UFSS_HIP(hipGetLastError());
        // S[dy][qx][z][k] = sum_dx hx[qx][dx] P[dy][dx][z][k]
        hipLaunchKernelGGL(cos_kernel, dim3((unsigned)((zc + 255) / 256), (nox + kBI - 1) / kBI, wy + 1), dim3(256),
                           0, nullptr, s64, p64, cx, nox, wx + 1, zc, (int64_t)(wx + 1) * zc, zc,
                           (int64_t)nox * zc, zc);
        UFSS_HIP(hipGetLastError());
        const dim3 grid((unsigned)((row + 255) / 256), nox, (noy + kBI - 1) / kBI);
        if (P.dtype == UFSS_BF16)
            hipLaunchKernelGGL(table_kernel<cbf16>, grid, dim3(256), 0, nullptr, static_cast<cbf16*>(P.d_khat), s64, cy,
                               wy + 1, nox, noy, P.fft_swap, nz, mu, P.fft_mus);
        else
            hipLaunchKernelGGL(table_kernel<cf32>, grid, dim3(256), 0, nullptr, static_cast<cf32*>(P.d_khat), s64, cy,
                               wy + 1, nox, noy, P.fft_swap, nz, mu, P.fft_mus);
        UFSS_HIP(hipGetLastError());
        UFSS_HIP(hipDeviceSynchronize());
    } catch (...) {
        release();
        throw;
    }
    release();
}

// One contraction launch.  Tiles per wave: forward one block of 32 outputs where a
// workgroup has a wave for each, else two (BF16 tables, half the bytes per load: up to
// 3, as few padded ones as possible); adjoint up to 2 tiles of 16.  Groups per
// workgroup: at most kNW, one per wave (FP32 adjoint 2, so that two waves share a reduction),
// fewer while the grid has too few workgroups to spread evenly over 256 CUs: with 528 of
// 3 blocks each, the busiest CU had 3 of them for a mean of 2.
// FP32, forward / adjoint, with 3 blocks per wave, 4 groups and 512 workgroups -> so: 32 x
// 32 x 256, 66 bins 20.3 / 22.5 -> 17.6 / 19.7 us; 45 x 51 x 301, 76 bins 38.7 / 41.7 ->
// 35.0 / 37.8; 64 x 64 x 512, 132 bins 100 / 105 -> 93 / 104.  BF16 by the FP32 rule -> so:
// 12.8 / 15.3 -> 12.8 / 13.9; 21.1 / 23.5 -> 21.1 / 23.1; 57 / 57 -> 46 / 56.
template <bool FWD, bool SWAP, bool BF16>
static void contract(const Plan& P, hipStream_t s) {
    const int mu = (int)P.ubins_h.size(), nz = P.g.nz;
    const int C = FWD ? mu : nz, R = FWD ? nz : mu;
    const int blocks = (C + group_rows(FWD, 1) - 1) / group_rows(FWD, 1);
    constexpr bool f32 = !BF16;
    int tb = std::min(blocks, FWD && !f32 ? 3 : 2);
    for (int t = tb - 1; t >= 2; --t)
        if ((blocks + t - 1) / t * t < (blocks + tb - 1) / tb * tb) tb = t;
    if (FWD && f32 && blocks <= kNW) tb = 1;
    const int all = (blocks + tb - 1) / tb, gr = group_rows(FWD, tb);
    int g = std::min(all, FWD || BF16 ? kNW : 2);
    while (g > 1 && P.fft_entries * ((all + g - 1) / g) < (FWD && f32 ? 768 : 512)) --g;
    const dim3 grid(P.fft_entries, (all + g - 1) / g);
    const int rs = (SWAP ? 16 : 8) + 2;
    const size_t cols = BF16 ? (size_t)(SWAP ? 3 : 2) * (kRB / 4) * kGP / sizeof(float)
                             : (size_t)(std::min(R, kRC) + step_len(FWD, false)) * rs;
    size_t red = 0;                       // over the group counts a block may have
    for (int n : {g, all - (all - 1) / g * g}) red = std::max(red, (size_t)(kNW / n) * 16 * (n * gr + 1));
    const size_t lds = std::max(cols, red) * sizeof(float);
    auto go = [&](auto tbc) {
        constexpr int TB = decltype(tbc)::value;
        if constexpr (BF16)
            hipLaunchKernelGGL((contract_bf16_kernel<FWD, TB, SWAP>), grid, dim3(64 * kNW), lds, s,
                               static_cast<const cbf16*>(P.d_khat), P.d_orb, P.d_fa, P.d_fb, P.fft_ly, P.fft_lx, nz,
                               P.fft_mus, C, R, g);
        else
            hipLaunchKernelGGL((contract_kernel<FWD, TB, SWAP>), grid, dim3(64 * kNW), lds, s,
                               static_cast<const cf32*>(P.d_khat), P.d_orb, P.d_fa, P.d_fb, P.fft_ly, P.fft_lx, nz,
                               P.fft_mus, C, R, g);
    };
    if (tb == 1) go(std::integral_constant<int, 1>{});
    else if (tb == 2) go(std::integral_constant<int, 2>{});
    else if constexpr (FWD && !f32) go(std::integral_constant<int, 3>{});
    UFSS_HIP(hipGetLastError());
}

template <bool FWD>
static void contract(const Plan& P, hipStream_t s) {
    if (P.dtype == UFSS_BF16) {
        if (P.fft_swap) contract<FWD, true, true>(P, s); else contract<FWD, false, true>(P, s);
    } else {
        if (P.fft_swap) contract<FWD, true, false>(P, s); else contract<FWD, false, false>(P, s);
    }
}

// ---------------------------------------------------------------------------
// The passes between two contractions act on one position and channel at a time,
// and the lateral products along y on one (x, channel) column: so the inverse
// product along y, the pass and the next forward product along y are one kernel,
// with the column in registers from one to the next.
//   kPre    measurements, times H -> DFT_y
//   kPost   IDFT_y -> times H (- ymeas) -> measurements
//   kBins   IDFT_y -> H^2 and - H ymeas -> DFT_y       (A x - y on its way to R^)
//   kDepth  IDFT_y -> FISTA update -> DFT_y            (X' on its way to the next X^)
//   kProx   IDFT_y -> a learned stage's gradient and proximal step
//   kSpec   voxels -> DFT_y                            (a first iteration's X^, by kDepth's arithmetic)
// What bounds it: launches and latencies.  On a small scan each product and each
// pass takes 4-6 us as a kernel of its own, of which its arithmetic is under 1 us;
// a FISTA iteration goes from 11 launches to 8.  (A whole plane in LDS, both axes
// at once, 4 launches, gains nothing: 8-byte columns of every row of the array cost
// 3 us to load and 5 us to store.)
// A workgroup of 4 waves takes 16 channels of one x (2 or 4 where NT, the tiles of 16
// rows y, is 2 or 1): wave w the inverse's tile w and every 4 / (units)-th tile of the
// forward product, so that a chain is one tile long; the column goes from one to the
// other through LDS.  A table operand is used once per wave: it is loaded from the
// cache, with the column, kTwPK steps ahead.  Operands and order are twiddle_kernel's.
// 32 x 32 x 256, 66 bins: the bins' side of an iteration (5 launches) 22.5 us -> 18
// with 3, the depths' side (4) 25.5 -> 20.5 with 3, the fused kernels 7.4 and 9.6 us of
// it (8.8 and 11.8 with all tiles in one wave); an apply pair of 45 x 51 x 301 (BF16
// table) 139 -> 133 us with one launch less per operator.
// ---------------------------------------------------------------------------
enum { kPre, kPost, kBins, kDepth, kProx, kSpec };

struct ColumnArgs {
    const cf32* in;                           // [ly][nx][C], or the measurements (kPre) or voxels (kSpec)
    cf32* out;                                // [ly][nx][C], or the measurements (kPost)
    const cf32 *tiy, *tfy;
    int nx, ny, ly, C, nct, units;
    // kPre, kPost, kBins
    const int* inv;                           // [npos][C], or null: measurement c is channel c
    const float* hu;
    const cf32* ymeas;
    int m;
    double* part;                             // per block: 1 value (kPost, kBins) or 5 (kDepth)
    // kDepth
    UpdateArgs upd;
    int more;
    ProxArgs prox;
    StatsJob job;                             // kBins: by the last block
};

// Block-wide FP64 sums of 4 waves in fixed order.
template <int W>
__device__ __forceinline__ void column_sums(double (&v)[W], double* red, double* out) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int w = 0; w < W; ++w) {
        double x = v[w];
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) x += __shfl_xor(x, off, 64);
        if (lane == 0) red[w * 4 + wave] = x;
    }
    __syncthreads();
    if (threadIdx.x < W) {
        const double* q = red + threadIdx.x * 4;
        out[threadIdx.x] = ((q[0] + q[1]) + q[2]) + q[3];
    }
}

// Units (one x, 16 channels) per workgroup.
__host__ __device__ constexpr int column_units(int nt) { return nt == 1 ? 4 : nt == 2 ? 2 : 1; }

template <int NT, int MODE>
__global__ __launch_bounds__(256) void column_kernel(ColumnArgs g) {
    constexpr int UN = column_units(NT), NW = 4 / UN;         // waves per unit
    constexpr bool kIv = MODE != kPre && MODE != kSpec, kFw = MODE != kPost && MODE != kProx;
    constexpr bool kMeas = MODE == kPre || MODE == kPost || MODE == kBins;
    __shared__ __align__(16) double smem[MODE == kBins ? kStatsRed + 6 : UN * NT * 256];
    __shared__ double red[5 * 4];
    if (MODE == kBins && (int)blockIdx.x * UN >= g.units) {
        fista_stats(g.job, smem, smem + kStatsRed);
        return;
    }
    const int nx = g.nx, ny = g.ny, L = g.ly;
    const int64_t C = g.C;
    const int J = L / 2 + 1, ksi = (J + 3) / 4, ksf = (ny + 3) / 4, tf = (J + 15) / 16;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int un = wave / NW, w = wave - un * NW;             // unit in the workgroup, wave in the unit
    const int unit = blockIdx.x * UN + un, px = unit / g.nct;
    const int ch = lane & 15, c = (unit - px * g.nct) * 16 + ch, kq = lane >> 4;
    const bool ok = unit < g.units && c < C;
    const bool mine = w < NT;                                 // the unit's waves that hold a tile
    cf32* xs = reinterpret_cast<cf32*>(smem) + un * NT * 256; // [16 NT rows][16 channels]
    const cf32* src = g.in + (int64_t)px * C + c;
    const cf32* ti = g.tiy + (int64_t)min(w, NT - 1) * ksi * 64 + lane;
    // table operand and column (folded about L / 2) of reduction step s
    struct Col { cf32 a, e, o; };
    auto fetch = [&](int s) {
        Col v{{0.f, 0.f}, {0.f, 0.f}, {0.f, 0.f}};
        if (s < ksi) v.a = ti[s * 64];
        const int j = 4 * s + kq;
        if (ok && j < J) {
            v.e = src[(int64_t)j * nx * C];
            if (j > 0 && 2 * j < L) v.o = src[(int64_t)(L - j) * nx * C];
        }
        return v;
    };
    Col cur[kTwPK];
    if (kIv && mine) {
#pragma unroll
        for (int p = 0; p < kTwPK; ++p) cur[p] = fetch(p);
    }
    // the forward product's first operands
    const bool fw = kFw && (MODE != kDepth || g.more);
    cf32 af[kTwPK];
    auto first = [&](int T) {
#pragma unroll
        for (int p = 0; p < kTwPK; ++p)
            if (p < ksf) af[p] = g.tfy[((int64_t)T * ksf + p) * 64 + lane];
    };
    if (fw && w < tf) first(w);
    // what the pass reads, requested before the product: rows i0 .. i0 + 3
    const int i0 = 16 * w + 4 * kq;
    auto pos = [&](int r) { return (int64_t)(i0 + r) * nx + px; };
    int mi[4];
    cf32 q[4], v[4];
    float h = 0.f;
    if constexpr (kMeas) {
        if (ok) h = g.hu[c];
#pragma unroll
        for (int r = 0; r < 4; ++r) mi[r] = ok && mine && i0 + r < ny ? (g.inv ? g.inv[pos(r) * C + c] : c) : -1;
        const cf32* rows = MODE == kPre ? g.in : g.ymeas;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            q[r] = cf32{0.f, 0.f};
            if (rows && mi[r] >= 0) q[r] = rows[pos(r) * g.m + mi[r]];
        }
    } else {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            q[r] = v[r] = cf32{0.f, 0.f};
            if (!ok || !mine || i0 + r >= ny) continue;
            q[r] = (MODE == kSpec ? g.in : MODE == kProx ? g.prox.gam : g.upd.gamma)[pos(r) * C + c];
            if (MODE == kDepth) v[r] = g.upd.a[pos(r) * C + c];
        }
    }
    f4v acc[2] = {f4v{0.f, 0.f, 0.f, 0.f}, f4v{0.f, 0.f, 0.f, 0.f}};
    if (kIv && mine) {
        for (int s0 = 0; s0 < ksi; s0 += kTwPK) {
#pragma unroll
            for (int p = 0; p < kTwPK; ++p) {
                if (s0 + p >= ksi) break;                     // uniform
                const Col u = cur[p];
                cur[p] = fetch(s0 + p + kTwPK);
                // an unmirrored index (0, L / 2) has sin = 0: its difference is not used
                const float er = u.e.re + u.o.re, ei = u.e.im + u.o.im;
                const float orr = u.e.re - u.o.re, oi = u.o.im - u.e.im;
                acc[0] = __builtin_amdgcn_mfma_f32_16x16x4f32(u.a.re, er, acc[0], 0, 0, 0);
                acc[1] = __builtin_amdgcn_mfma_f32_16x16x4f32(u.a.re, ei, acc[1], 0, 0, 0);
                acc[0] = __builtin_amdgcn_mfma_f32_16x16x4f32(u.a.im, oi, acc[0], 0, 0, 0);
                acc[1] = __builtin_amdgcn_mfma_f32_16x16x4f32(u.a.im, orr, acc[1], 0, 0, 0);
            }
        }
    }
    if constexpr (MODE == kProx) {
        const float st = g.prox.step(), th = g.prox.threshold();
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            if (!ok || !mine || i0 + r >= ny) continue;
            const int64_t at = pos(r) * C + c;
            const cf32 b{acc[0][r], acc[1][r]};
            cf32 z, u;
            prox_step(q[r], b, st, th, z, u);
            if (g.prox.g) g.prox.g[at] = b;
            g.prox.z[at] = z;
            g.prox.u[at] = u;
        }
        return;
    }
    double sum[MODE == kDepth ? 5 : 1] = {};
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        if constexpr (MODE == kDepth) {
            if (ok && mine && i0 + r < ny) {
                const int64_t at = pos(r) * C + c;
                cf32 an, gn;
                fista_step(q[r], v[r], cf32{acc[0][r], acc[1][r]}, g.upd.step, g.upd.thresh, g.upd.beta, g.upd.real,
                           g.upd.aref ? g.upd.aref + at : nullptr, an, gn, sum);
                g.upd.a[at] = an;
                g.upd.gamma[at] = gn;
                v[r] = gn;
            }
        } else if constexpr (MODE == kSpec) {
            v[r] = q[r];
        } else if constexpr (MODE == kPre) {
            v[r] = cf32{h * q[r].re, h * q[r].im};
        } else {
            float re = 0.f, im = 0.f;
            if (mi[r] >= 0) {
                re = acc[0][r] * h;
                im = acc[1][r] * h;
                if (g.ymeas) {
                    re -= q[r].re;
                    im -= q[r].im;
                }
                if (MODE == kPost) g.out[pos(r) * g.m + mi[r]] = cf32{re, im};
            }
            v[r] = cf32{h * re, h * im};
            sum[0] += (double)re * re + (double)im * im;
        }
        if (kFw && mine) xs[(i0 + r) * 16 + ch] = v[r];
    }
    if constexpr (MODE == kDepth) column_sums(sum, red, g.part + 5 * (int64_t)blockIdx.x);
    else if constexpr (MODE == kPost || MODE == kBins) column_sums(sum, red, g.part + blockIdx.x);
    else __syncthreads();                                     // xs is written (column_sums has the barrier too)
    if (!fw || unit >= g.units) return;
    cf32* dst = g.out + (int64_t)px * C + c;
    for (int T = w; T < tf; T += NW) {
        f4v d[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) d[e] = f4v{0.f, 0.f, 0.f, 0.f};
        for (int s0 = 0; s0 < ksf; s0 += kTwPK) {
#pragma unroll
            for (int p = 0; p < kTwPK; ++p) {
                const int s = s0 + p;
                if (s >= ksf) break;                          // uniform
                const cf32 a = af[p], e = xs[(4 * s + kq) * 16 + ch];
                if (s + kTwPK < ksf) af[p] = g.tfy[((int64_t)T * ksf + s + kTwPK) * 64 + lane];
                d[0] = __builtin_amdgcn_mfma_f32_16x16x4f32(a.re, e.re, d[0], 0, 0, 0);
                d[1] = __builtin_amdgcn_mfma_f32_16x16x4f32(a.re, e.im, d[1], 0, 0, 0);
                d[2] = __builtin_amdgcn_mfma_f32_16x16x4f32(a.im, e.re, d[2], 0, 0, 0);
                d[3] = __builtin_amdgcn_mfma_f32_16x16x4f32(a.im, e.im, d[3], 0, 0, 0);
            }
        }
        if (T + NW < tf) first(T + NW);
        if (!ok) continue;                                    // a lane's table operand is of another channel's row
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int i = 16 * T + 4 * kq + r;
            const float cr = d[0][r], ci = d[1][r], sr = d[2][r], si = d[3][r];
            if (2 * i <= L) dst[(int64_t)i * nx * C] = cf32{cr + si, ci - sr};
            if (i > 0 && 2 * i < L) dst[(int64_t)(L - i) * nx * C] = cf32{cr - si, ci + sr};
        }
    }
}

// Rows y of a column: 4 tiles of 16, one per wave.  Longer grids, and grids whose update
// would leave more partials than there is room for, take a kernel per product and pass.
static constexpr int kColTiles = 4;

static int column_blocks(const Plan& P, int C) {
    const int un = column_units((P.g.ny + 15) / 16);
    return (P.g.nx * ((C + 15) / 16) + un - 1) / un;
}

bool fft_fused(const Plan& P) {
    return P.algo == UFSS_ALGO_FFT && !P.mix && P.g.ny <= 16 * kColTiles && column_blocks(P, P.g.nz) * 5 <= P.part_cap &&
           column_blocks(P, (int)P.ubins_h.size()) <= P.part_cap / 2;
}

template <int MODE>
static int column(const Plan& P, const cf32* in, cf32* out, int C, ColumnArgs g, hipStream_t s) {
    g.in = in;
    g.out = out;
    g.tiy = P.d_tw_iy;
    g.tfy = P.d_tw_fy;
    g.nx = P.g.nx;
    g.ny = P.g.ny;
    g.ly = P.fft_ly;
    g.C = C;
    g.nct = (C + 15) / 16;
    g.units = g.nx * g.nct;
    const int nt = (g.ny + 15) / 16, blocks = column_blocks(P, C);
    const dim3 grid(blocks + (MODE == kBins && g.job.stats ? 1 : 0));
    auto go = [&](auto ntc) {
        hipLaunchKernelGGL((column_kernel<decltype(ntc)::value, MODE>), grid, dim3(256), 0, s, g);
    };
    if (nt == 1) go(std::integral_constant<int, 1>{});
    else if (nt == 2) go(std::integral_constant<int, 2>{});
    else if (nt == 3) go(std::integral_constant<int, 3>{});
    else go(std::integral_constant<int, 4>{});
    UFSS_HIP(hipGetLastError());
    return blocks;
}

static ColumnArgs meas_args(const Plan& P, const cf32* ymeas, double* part) {
    ColumnArgs g{};
    g.inv = P.d_inv;
    g.hu = P.d_hu;
    g.ymeas = ymeas;
    g.m = P.m;
    g.part = part;
    return g;
}

// The products along x around the fused ones: [ly][lx][C] -> [ly][nx][C] and back.
static void inverse_x(const Plan& P, int C, hipStream_t s) {
    const int nx = P.g.nx, lx = P.fft_lx, ly = P.fft_ly;
    twiddle<true>(P.d_ft, P.d_fb, P.d_tw_ix, ly, lx, nx, C, (int64_t)lx * C, C, (int64_t)nx * C, C, s);
}
static void forward_x(const Plan& P, int C, hipStream_t s) {
    const int nx = P.g.nx, lx = P.fft_lx, ly = P.fft_ly;
    twiddle<false>(P.d_fa, P.d_ft, P.d_tw_fx, ly, lx, nx, C, (int64_t)nx * C, C, (int64_t)lx * C, C, s);
}

int fft_post(const Plan& P, cf32* y, const cf32* ymeas, double* part, hipStream_t s) {
    const int mu = (int)P.ubins_h.size();
    inverse_x(P, mu, s);
    return column<kPost>(P, P.d_ft, y, mu, meas_args(P, ymeas, part), s);
}

void fft_pre(const Plan& P, const cf32* r, hipStream_t s) {
    const int mu = (int)P.ubins_h.size();
    column<kPre>(P, r, P.d_ft, mu, meas_args(P, nullptr, nullptr), s);
    forward_x(P, mu, s);
}

// The fused kernels work in place: a workgroup has read its columns before it writes them.
int fft_residual(const Plan& P, const cf32* ymeas, double* part, const StatsJob& job, hipStream_t s) {
    const int mu = (int)P.ubins_h.size();
    ColumnArgs g = meas_args(P, ymeas, part);
    g.job = job;
    inverse_x(P, mu, s);
    const int nb = column<kBins>(P, P.d_ft, P.d_ft, mu, g, s);
    forward_x(P, mu, s);
    return nb;
}

void fft_prox(const Plan& P, const ProxArgs& a, hipStream_t s) {
    ColumnArgs g{};
    g.prox = a;
    inverse_x(P, P.g.nz, s);
    column<kProx>(P, P.d_ft, nullptr, P.g.nz, g, s);
}

int fft_update(const Plan& P, const UpdateArgs& u, bool more, hipStream_t s) {
    const int nz = P.g.nz;
    ColumnArgs g{};
    g.upd = u;
    g.part = u.part;
    g.more = more;
    inverse_x(P, nz, s);
    const int nb = column<kDepth>(P, P.d_ft, P.d_ft, nz, g, s);
    if (more) forward_x(P, nz, s);
    return nb;
}

// X^ as fft_update leaves it, in the same order and arithmetic (y, then x).
void fft_spectrum(const Plan& P, const cf32* x, hipStream_t s) {
    column<kSpec>(P, x, P.d_ft, P.g.nz, ColumnArgs{}, s);
    forward_x(P, P.g.nz, s);
}

// Forward, in three steps (the contraction is the core kernel):
//   x[ny][nx][nz] -> T[ny][lx][nz] -> X^[ly][lx][nz]
void fft_fwd_transform(const Plan& P, const cf32* x, hipStream_t s) {
    const int nx = P.g.nx, ny = P.g.ny, nz = P.g.nz, lx = P.fft_lx, ly = P.fft_ly;
    twiddle<false>(P.d_ft, x, P.d_tw_fx, ny, lx, nx, nz, (int64_t)nx * nz, nz, (int64_t)lx * nz, nz, s);
    twiddle<false>(P.d_fa, P.d_ft, P.d_tw_fy, lx, ly, ny, nz, nz, (int64_t)lx * nz, nz, (int64_t)lx * nz, s);
}

//   Y^[q][k] = sum_z K^[q][z][k] X^[q][z]
void fft_fwd_contract(const Plan& P, hipStream_t s) { contract<true>(P, s); }

//   Y^[ly][lx][mu] -> U[ly][nx][mu] -> y_raw[ny][nx][mu]
void fft_fwd_inverse(const Plan& P, hipStream_t s) {
    const int nx = P.g.nx, ny = P.g.ny, lx = P.fft_lx, ly = P.fft_ly, mu = (int)P.ubins_h.size();
    twiddle<true>(P.d_ft, P.d_fb, P.d_tw_ix, ly, lx, nx, mu, (int64_t)lx * mu, mu, (int64_t)nx * mu, mu, s);
    twiddle<true>(P.d_yraw, P.d_ft, P.d_tw_iy, nx, ly, ny, mu, mu, (int64_t)nx * mu, mu, (int64_t)nx * mu, s);
}

// Adjoint, in three steps; the operand is the H-scaled union-bin rows in P.d_rop.
void fft_adj_transform(const Plan& P, hipStream_t s) {
    const int nx = P.g.nx, ny = P.g.ny, lx = P.fft_lx, ly = P.fft_ly, mu = (int)P.ubins_h.size();
    const cf32* r = static_cast<const cf32*>(P.d_rop);
    twiddle<false>(P.d_ft, r, P.d_tw_fx, ny, lx, nx, mu, (int64_t)nx * mu, mu, (int64_t)lx * mu, mu, s);
    twiddle<false>(P.d_fa, P.d_ft, P.d_tw_fy, lx, ly, ny, mu, mu, (int64_t)lx * mu, mu, (int64_t)lx * mu, s);
}

void fft_adj_contract(const Plan& P, hipStream_t s) { contract<false>(P, s); }

void fft_adj_inverse(const Plan& P, cf32* out, hipStream_t s) {
    const int nx = P.g.nx, ny = P.g.ny, nz = P.g.nz, lx = P.fft_lx, ly = P.fft_ly;
    twiddle<true>(P.d_ft, P.d_fb, P.d_tw_ix, ly, lx, nx, nz, (int64_t)lx * nz, nz, (int64_t)nx * nz, nz, s);
    twiddle<true>(out, P.d_ft, P.d_tw_iy, nx, ly, ny, nz, nz, (int64_t)nx * nz, nz, (int64_t)nx * nz, s);
}

}  // namespace ufss
