// Windowed complex GEMM kernels for shared frequency subsets, FP32 on MFMA.
//
// The operator is block 2-level Toeplitz in the lateral offset d = p - v
// (paper Sec. IV-B, theorem on the structure of H): for one offset d it is a
// dense complex product between the phase matrix P_d[k, z] and the depth
// profiles of the voxels at p - d.  Instead of the paper's FFT-based
// correlation (Alg. 2) the window is summed directly, one small GEMM per
// offset, which puts the work on the matrix cores.  P_d depends on (|d_x|,
// |d_y|) only, so the (up to four) voxels at mirrored offsets are added first
// and share one product:
//
//   forward  Y[p, k] = sum_{a in [0, W]} sum_z P_a[k, z] sum_{d = (+-a_x, +-a_y)} x[p - d, z]
//   adjoint  G[v, z] = sum_{a in [0, W]} sum_k conj(P_a[k, z]) sum_{d = (+-a_x, +-a_y)} R[v + d, k]
//
// with P_a[k, z] = exp(-j 2 pi (k * u(a, z) mod 2^32) / 2^32), u the
// integer-turn delay table built by the plan (a zero component has one sign,
// voxels outside the grid are zero).  H_k scaling, gathers for per-position
// subsets and residuals live in the small pre/post kernels.
//
// What bounds it: the FP32 MFMAs and the VALU work share issue cycles on this
// chip, so the cost is products + phasors + mirror additions.  One product per
// mirrored offset group is about a quarter of the products and phasors of one
// per offset when the window is narrow against the grid (0.28 on the 64 x 64
// C-scan with W = 16) and about half on a full aperture (0.58 at 32 x 32).
// Core kernels before and after: 64 x 64 x 512 (128 bins, W = 16) forward 12.4 ->
// 4.0 ms, adjoint 13.3 -> 4.0 ms; 32 x 32 x 256 (66 bins, full) 1.20 -> 0.73 and
// 1.23 -> 0.75 ms; 32-position B-scan (128 depths, 32 bins) 0.26 -> 0.013 and
// 0.067 -> 0.014 ms (there from the parts, below).
// Offsets are summed from the far ones in: the near ones, where the phase is
// stationary, make most of a scene's sum, and a chain that starts with them carries
// it through all its roundings.  Relative error against 64 bits of the adjoint of a
// scene's measurements, 22 x 41 x 99 with 16 bins: from the near ones out 3.0e-7, from
// the far ones in 1.7e-7, one product per offset from -W to W 2.1e-7 (random operands:
// 4.4e-7, 4.0e-7, 4.8e-7); the same time.  A B-scan's parts take the offsets in the same
// order (36 positions, 299 depths, 56 bins: near ones in the first part 1.5e-7, far ones 1.3e-7).
//
// MFMA: v_mfma_f32_16x16x4_f32.  Lane l holds A[i = l%16][k = l/16],
// B[k = l/16][j = l%16] and D[i = 4(l/16) + r][j = l%16] for r = 0..3.
// Complex products use three real MFMAs on split real / imaginary parts
// (Gauss's form: one product of sums, two products with combined phasors).
//
// Tiling (both kernels): a workgroup of 4 waves owns one lateral tile of
// NP sub-tiles of 16 positions (SW x 16/SW each, SW = 4 for C-scans, 16 for
// B-scans).  Forward: each wave owns 16 bins, the 4 waves cover 64 bins.
// Adjoint: each wave owns 16 depths.  For one a_y and one chunk of the
// reduction axis the rows at +-a_y are added while they are staged in LDS
// (zero outside the grid); the columns at +-a_x are two LDS reads and an
// addition per operand.  Phasors are generated per lane in registers.
// Accumulation is two level (per a_y in MFMA registers, then into an outer
// FP32 sum) to keep the FP32 error of ~1e5-term sums near 1e-6.
//
// Parts: split-K partials go to separate output slots that the epilogues sum
// in fixed order.  On a C-scan the (chunk of the reduction axis, a_y) steps of
// a tile are dealt to its parts in equal contiguous ranges; a B-scan has one
// a_y, so its parts divide the a_x range instead (a 32-position B-scan is one
// lateral tile: without that it runs on 1 or 2 of the 256 CUs).
#include <type_traits>

#include "internal.h"

namespace ufss {

typedef float f4 __attribute__((ext_vector_type(4)));

static constexpr float kTwoM32 = 2.3283064365386963e-10f;   // 2^-32

// exp(-j 2 pi phi) components for the integer phase k*u (mod 2^32) in turns.
__device__ __forceinline__ void phasor(uint32_t ku, float& c, float& s) {
    float ph = (float)(int32_t)ku * kTwoM32;     // [-0.5, 0.5) turns
    c = __builtin_amdgcn_cosf(ph);              // cos(2 pi ph)
    s = __builtin_amdgcn_sinf(ph);              // sin(2 pi ph)
}

// ---- LDS layout of the staged rows -----------------------------------------
// tpy rows of hc = tpx + 2 wx cells (the columns a tile reaches; those outside
// the grid stay zero), CH complex values per cell at a stride of cell_stride
// values, then a run of zero cells that stands in for the mirrored columns at
// a_x = 0.  Strides: 16-byte aligned cells for the 16-byte reads below, and
// rows 64 bytes apart modulo the 256-byte bank period, so the 4 x 4 cells that
// 16 lanes read together (cells 144 or 80 bytes apart) touch every bank once.
__host__ __device__ constexpr int cell_stride(int ch) { return ch == 4 ? 5 : ch + 2; }
__host__ __device__ static inline int row_pitch(int hc, int ch) {
    const int raw = hc * cell_stride(ch);
    return raw + ((8 - raw) & 31);
}
__host__ __device__ static inline int zero_run(int np, int sw, int ch) {
    return (((np - 1) * sw + 1) * cell_stride(ch) + 1) & ~1;
}

// Stages rows r < TPY, grid columns [x_lo, x_hi], CH values of the reduction
// axis from i0 on: halo[r pitch + (x - xb) cs + e] = src[y0 + r - ay][x][i0 + e]
// (+ src[y0 + r + ay][x][i0 + e] for ay > 0), rows outside the grid counting as
// zero, nothing at or past `ilim`.  Each thread keeps one e and walks the
// columns with a fixed step, U columns of each of the TPY rows (8 loads) in
// flight; whether a row is inside the grid is uniform.
template <int CH, int TPY>
__device__ __forceinline__ void stage_mirrored(cf32* __restrict__ halo, int pitch, const cf32* __restrict__ src,
                                               int ny, int nx, int64_t ld, int y0, int ay, int xb, int x_lo,
                                               int x_hi, int i0, int ilim) {
    constexpr int cs = cell_stride(CH);
    constexpr int U = 4 / TPY;
    const int e = threadIdx.x & (CH - 1);
    const int step = blockDim.x / CH;
    const bool eok = i0 + e < ilim;
    for (int x = x_lo + (int)(threadIdx.x / CH); x <= x_hi; x += U * step) {
        cf32 v[TPY * U], w[TPY * U];
        const cf32* col = src + (int64_t)x * ld + i0 + e;
#pragma unroll
        for (int r = 0; r < TPY; ++r) {
            const int ya = y0 + r - ay, yb = y0 + r + ay;
            const bool oka = ya >= 0 && ya < ny, okb = ay > 0 && yb < ny;
#pragma unroll
            for (int t = 0; t < U; ++t) {
                v[r * U + t] = w[r * U + t] = cf32{0.f, 0.f};
                const bool in = eok && x + t * step <= x_hi;
                const cf32* q = col + (int64_t)t * step * ld;
                if (oka && in) v[r * U + t] = q[(int64_t)ya * nx * ld];
                if (okb && in) w[r * U + t] = q[(int64_t)yb * nx * ld];
            }
        }
        cf32* dst = halo + (x - xb) * cs + e;
#pragma unroll
        for (int r = 0; r < TPY; ++r)
#pragma unroll
            for (int t = 0; t < U; ++t)
                if (x + t * step <= x_hi)
                    dst[r * pitch + t * step * cs] = cf32{v[r * U + t].re + w[r * U + t].re, v[r * U + t].im + w[r * U + t].im};
    }
}

// The CH / 4 values of one lane group (kq = lane / 16): cell entries
// kq CH / 4 .. + CH / 4 - 1, consecutive so that they are 16-byte LDS reads.
template <int CH>
__device__ __forceinline__ void lane_values(const cf32* __restrict__ p, cf32 (&v)[CH / 4]) {
    if constexpr (CH >= 8) {
#pragma unroll
        for (int h = 0; h < CH / 8; ++h) {
            const f4 q = *reinterpret_cast<const f4*>(p + 2 * h);
            v[2 * h] = cf32{q.x, q.y};
            v[2 * h + 1] = cf32{q.z, q.w};
        }
    } else {
        v[0] = p[0];
    }
}

// Last a_x at which a sub-tile of SW columns from c0 on sees the grid (-1:
// the sub-tile itself lies outside).
__host__ __device__ static inline int last_ax(int c0, int sw, int nx) {
    return c0 >= nx ? -1 : max(min(c0 + sw, nx) - 1, nx - 1 - c0);
}

// a_y values at which the rows y0 .. y0 + tpy - 1 see the grid.
__host__ __device__ static inline int tile_nay(int y0, int tpy, int ny, int wy) {
    return min(wy, last_ax(y0, tpy, ny)) + 1;
}

// Sub-tile offsets a_x of a tile's row of np sub-tiles from x0 on.
__host__ __device__ static inline int tile_nax(int x0, int np, int sw, int nx, int wx) {
    int n = 0;
    for (int s = 0; s < np; ++s) n += min(wx, last_ax(x0 + s * sw, sw, nx)) + 1;
    return n;
}

// What a tile and its part of the reduction run over.
struct TileRange {
    int t0, t1;          // steps (chunk of the reduction axis, a_y), a_y fastest, from the far one in
    int nay;             // a_y values of the tile
    int ax_lo, ax_hi;    // a_x range
};

// Tile of np sub-tiles (sw x tpy) at (x0, y0); part `sp` of `split` and `spz`
// of `zsplit`; nch chunks of the reduction axis, a step of the last one costing
// `last` where a step of the others costs `full`.  On a C-scan a tile whose work
// is w of the heaviest tile's `top` uses ceil(parts w / top) of the parts, spread
// evenly, and leaves the others empty, so every workgroup with work has about
// the same (on a full aperture a corner tile has 2.5 times a central one's
// offsets).
__device__ __forceinline__ TileRange tile_range(int x0, int y0, int np, int sw, int tpy, int nx, int ny, int wx, int wy,
                                                int nch, int full, int last, int sp, int split, int spz, int zsplit,
                                                int top) {
    TileRange R;
    R.nay = tile_nay(y0, tpy, ny, wy);
    const int nax = min(wx, last_ax(x0, np * sw, nx)) + 1;
    R.ax_lo = 0;
    R.ax_hi = nax - 1;
    if (ny == 1) {
        R.t0 = spz * nch / zsplit;
        R.t1 = (spz + 1) * nch / zsplit;
        R.ax_lo = (split - 1 - sp) * nax / split;                  // the far ones in the first part
        R.ax_hi = (split - sp) * nax / split - 1;
    } else {
        const int part = sp + split * spz;
        const int64_t w = (int64_t)R.nay * tile_nax(x0, np, sw, nx, wx);
        const int slots = split * zsplit;
        const int parts = (int)((slots * w + top - 1) / top);
        const int64_t head = (int64_t)(nch - 1) * R.nay * full, cost = head + (int64_t)R.nay * last;
        auto step_at = [&](int64_t c) {                            // first step not before cost c
            return (int)(c <= head ? (c + full - 1) / full : head / full + (c - head + last - 1) / last);
        };
        const int q = (int)((int64_t)part * parts / slots);        // the slot's part, if it has one
        const bool has = (int)((int64_t)(part + 1) * parts / slots) > q;
        R.t0 = has ? step_at(q * cost / parts) : 0;
        R.t1 = has ? step_at((q + 1) * cost / parts) : 0;
    }
    return R;
}

// Block b of `groups` x `parts` -> (group, part).  Blocks are dealt round-robin
// to the 8 XCDs; where that comes out even, XCD k takes the k-th eighth of the
// parts of every group: neighbouring parts and neighbouring tiles read the same
// rows, which then stay in that XCD's L2.
__device__ __forceinline__ void deal(int b, int groups, int parts, int& group, int& part) {
    const int per_xcd = groups * parts / 8;
    if (per_xcd * 8 == groups * parts) b = (b & 7) * per_xcd + (b >> 3);
    part = b / groups;
    group = b - part * groups;
}

struct FwdArgs {
    const cf32* x;
    cf32* yraw;            // [split * zsplit][npos][mu]
    const uint32_t* u;     // [wy+1][wx+1][nz]
    const float* amp;      // beam amplitude, same layout (DIR kernels only)
    const int* kb;         // [mu]
    int nx, ny, nz, wx, wy, mu;
    int sw;                // sub-tile width (4 or 16)
    int ntx, nty;          // lateral tiles
    int nbt;               // bin tiles of 16 * nw
    int nw;                // waves with a bin sub-tile (<= blockDim / 64)
    int ft;                // bins past the last full tile (1..4) folded into it, else 0
    int zc;                // depth chunk (multiple of 4)
    int split;             // parts, see tile_range
    int zsplit;
    int top;               // the heaviest tile's work
    int64_t npos;
    int nblk;              // blocks of this plan's grid
};

// ZC: the depth chunk a.zc as a compile-time constant (16, 8 or 4).
// DIR: scale each phasor by the beam amplitude g(a, z) (staged in LDS beside
// the delay table).
// FOLD: the plan folds a.ft tail bins into its last bin tile (below).
template <int NP, int ZC, int SW, bool DIR = false, bool FOLD = false>
__device__ __forceinline__ void fwd_f32_body(const FwdArgs& a, const int b, unsigned char* smem) {
    constexpr int NJ = ZC / 4, cs = cell_stride(ZC);
    constexpr int tpx = SW * NP, tpy = 16 / SW;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int hc = tpx + 2 * a.wx;            // halo columns
    const int pitch = row_pitch(hc, ZC);
    const int zrun = zero_run(NP, SW, ZC);
    cf32* halo = reinterpret_cast<cf32*>(smem);
    uint32_t* ulds = reinterpret_cast<uint32_t*>(halo + (size_t)tpy * pitch + zrun);
    float* glds = reinterpret_cast<float*>(ulds + (size_t)(a.wx + 1) * ZC);

    // block -> (part, bin tile, lateral tile)
    const int ntile = a.ntx * a.nty;
    int tile, sp_all;                                // sp_all: partial slot
    deal(b, ntile * a.nbt, a.split * a.zsplit, tile, sp_all);
    const int bt = tile / ntile;
    tile -= bt * ntile;
    const int px0 = (tile % a.ntx) * tpx, py0 = (tile / a.ntx) * tpy;
    const TileRange R = tile_range(px0, py0, NP, SW, tpy, a.nx, a.ny, a.wx, a.wy, (a.nz + ZC - 1) / ZC, 1, 1,
                                   sp_all % a.split, a.split, sp_all / a.split, a.zsplit, a.top);
    const int x_lo = max(0, px0 - a.wx), x_hi = min(a.nx - 1, px0 + tpx - 1 + a.wx);
    int axl[NP];
#pragma unroll
    for (int s = 0; s < NP; ++s) axl[s] = last_ax(px0 + s * SW, SW, a.nx);

    for (int t = threadIdx.x; t < tpy * pitch + zrun; t += blockDim.x) halo[t] = cf32{0.f, 0.f};

    const int bin0 = bt * 16 * a.nw + wave * 16;               // this wave's first bin
    const bool wave_active = wave < a.nw && bin0 < a.mu;
    const int i = lane & 15, ix = i % SW, iy = i / SW;
    const int kq = lane >> 4;                                  // depths NJ kq .. NJ kq + NJ - 1 of a chunk
    // A wave left with at most 4 bins (the short last one of a union such as
    // 66 = 4 x 16 + 2) runs v_mfma_f32_4x4x1_16b_f32 instead: 16 blocks of a
    // 4 x 4 product with one depth each, the same rate per flop, a quarter of
    // the 16 x 16 x 4 cycles.  Its A operand is the same (lane l: position
    // l % 16, depth group l / 16), its B operand takes bin l % 4 (block l / 4 =
    // (position group, depth group)), and the four depth blocks of a position
    // group are summed across lanes at the end.
    const bool tail = wave_active && a.mu - bin0 <= 4;
    // Folded tail (four waves, a.ft bins past the last full bin tile, e.g. the
    // 2 of 66 = 64 + 2): the last tile's waves share those bins' products on the
    // same 4 x 4 x 1 form, wave w at the offsets a_x = w (mod 4), reusing the
    // A operands of their own products; the four partial sums meet in LDS at
    // the end.  Every wave keeps the same work per offset range, where a fifth
    // wave for the tail shares a SIMD with another wave.
    const bool fold = FOLD && bt == a.nbt - 1;
    const int tb = FOLD ? a.nbt * 16 * a.nw + (lane & 3) : 0;   // this lane's folded bin
    // this lane's cells at a_x = 0 and the zero cells that stand in there
    const cf32* cell0 = halo + iy * pitch + (ix + a.wx) * cs + NJ * kq;
    const cf32* zcell = halo + tpy * pitch;
    auto run = [&](auto tailc) {
        constexpr bool TAIL = decltype(tailc)::value;
        const int mb = bin0 + (TAIL ? (lane & 3) : (lane & 15));   // this lane's bin column
        const uint32_t kbin = (mb < a.mu) ? (uint32_t)a.kb[mb] : 0u;
        uint32_t kbt = 0u;
        if constexpr (FOLD) kbt = (fold && tb < a.mu) ? (uint32_t)a.kb[tb] : 0u;
        auto mfma = [](float av, float bv, f4 acc) {
            if constexpr (TAIL) return __builtin_amdgcn_mfma_f32_4x4x1f32(av, bv, acc, 0, 0, 0);
            else return __builtin_amdgcn_mfma_f32_16x16x4f32(av, bv, acc, 0, 0, 0);
        };

        f4 out_re[NP], out_im[NP], t_re[FOLD ? NP : 1], t_im[FOLD ? NP : 1];
#pragma unroll
        for (int s = 0; s < NP; ++s) out_re[s] = out_im[s] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < (FOLD ? NP : 1); ++s) t_re[s] = t_im[s] = f4{0.f, 0.f, 0.f, 0.f};

        for (int t = R.t0; t < R.t1; ++t) {
            const int zi = t / R.nay, ay = R.nay - 1 - (t - zi * R.nay), z0 = zi * ZC;
            __syncthreads();
            stage_mirrored<ZC, tpy>(halo, pitch, a.x, a.ny, a.nx, a.nz, py0, ay, px0 - a.wx, x_lo, x_hi, z0, a.nz);
            for (int q = threadIdx.x; q < (a.wx + 1) * ZC; q += blockDim.x) {
                const int ax = q / ZC, z = z0 + (q & (ZC - 1));
                const int64_t o = ((int64_t)ay * (a.wx + 1) + ax) * a.nz + z;
                ulds[q] = z < a.nz ? a.u[o] : 0u;
                if (DIR) glds[q] = z < a.nz ? a.amp[o] : 0.f;
            }
            __syncthreads();
            if (!wave_active) continue;
            // Gauss's three-product form of (xr + j xi)(c - j s):
            //   m1 = c (xr + xi), m2 = xr (-s - c), m3 = xi (c - s);
            //   Re = m1 - m3 = xr c + xi s,  Im = m1 + m2 = xi c - xr s
            f4 m1[NP], m2[NP], m3[NP];
#pragma unroll
            for (int s = 0; s < NP; ++s) m1[s] = m2[s] = m3[s] = f4{0.f, 0.f, 0.f, 0.f};
            for (int ax = R.ax_hi; ax >= R.ax_lo; --ax) {
                const uint32_t* urow = ulds + ax * ZC;
                const cf32* lrow = cell0 - ax * cs;
                const cf32* rrow = ax > 0 ? cell0 + ax * cs : zcell;
                float cz[NJ], bmz[NJ], bpz[NJ];
#pragma unroll
                for (int j = 0; j < NJ; ++j) {
                    float c, sn;
                    phasor(kbin * urow[NJ * kq + j], c, sn);
                    if (DIR) {
                        const float gv = glds[ax * ZC + NJ * kq + j];
                        c *= gv;
                        sn *= gv;
                    }
                    cz[j] = c;
                    bmz[j] = -sn - c;
                    bpz[j] = c - sn;
                }
                // this wave's offsets for the folded bins, and their phasors: the
                // wave's 4 bins x ZC depths are one phasor per lane (bin l % 4,
                // depth l / 4), handed to the lanes that take them
                const bool folds = FOLD && !TAIL && fold && (ax & 3) == wave;
                float cj[NJ], sj[NJ];
                if (folds) {
                    const int dz = min(lane >> 2, ZC - 1);
                    float c0, s0;
                    phasor(kbt * urow[dz], c0, s0);
                    if (DIR) {
                        const float gv = glds[ax * ZC + dz];
                        c0 *= gv;
                        s0 *= gv;
                    }
#pragma unroll
                    for (int j = 0; j < NJ; ++j) {
                        const int src = 4 * (NJ * kq + j) + (lane & 3);
                        cj[j] = __shfl(c0, src, 64);
                        sj[j] = __shfl(s0, src, 64);
                    }
                }
#pragma unroll
                for (int s = 0; s < NP; ++s) {
                    // past the last a_x at which a sub-tile sees the grid its
                    // operands are zero: no products (wave-uniform test)
                    if (ax > axl[s]) continue;
                    cf32 l[NJ], r[NJ];
                    lane_values<ZC>(lrow + s * SW * cs, l);
                    lane_values<ZC>(rrow + s * SW * cs, r);
                    float xr[NJ], xi[NJ];
#pragma unroll
                    for (int j = 0; j < NJ; ++j) {
                        xr[j] = l[j].re + r[j].re;
                        xi[j] = l[j].im + r[j].im;
                        m1[s] = mfma(xr[j] + xi[j], cz[j], m1[s]);
                        m2[s] = mfma(xr[j], bmz[j], m2[s]);
                        m3[s] = mfma(xi[j], bpz[j], m3[s]);
                    }
                    if constexpr (FOLD && !TAIL) {
                        if (folds) {
                            // (xr + j xi)(c - j s) for the folded bins, four real products
#pragma unroll
                            for (int j = 0; j < NJ; ++j) {
                                t_re[s] = __builtin_amdgcn_mfma_f32_4x4x1f32(xr[j], cj[j], t_re[s], 0, 0, 0);
                                t_im[s] = __builtin_amdgcn_mfma_f32_4x4x1f32(xi[j], cj[j], t_im[s], 0, 0, 0);
                                t_re[s] = __builtin_amdgcn_mfma_f32_4x4x1f32(xi[j], sj[j], t_re[s], 0, 0, 0);
                                t_im[s] = __builtin_amdgcn_mfma_f32_4x4x1f32(xr[j], -sj[j], t_im[s], 0, 0, 0);
                            }
                        }
                    }
                }
            }
#pragma unroll
            for (int s = 0; s < NP; ++s) {
                out_re[s] += m1[s] - m3[s];
                out_im[s] += m1[s] + m2[s];
            }
        }
        if constexpr (FOLD && !TAIL) {
            if (fold) {
                cf32* yo = a.yraw + (int64_t)sp_all * a.npos * a.mu;
                // the four waves' folded sums, added in wave order, then the four
                // depth blocks of each position group as in the tail wave below
                float* red = reinterpret_cast<float*>(smem);     // [4][NP][8][64]
                __syncthreads();                                 // halo reads done
                if (wave < 4) {
#pragma unroll
                    for (int s = 0; s < NP; ++s)
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            red[((wave * NP + s) * 8 + r) * 64 + lane] = t_re[s][r];
                            red[((wave * NP + s) * 8 + 4 + r) * 64 + lane] = t_im[s][r];
                        }
                }
                __syncthreads();
                if (wave == 0) {
#pragma unroll
                    for (int s = 0; s < NP; ++s)
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            float vr = red[(s * 8 + r) * 64 + lane], vi = red[(s * 8 + 4 + r) * 64 + lane];
#pragma unroll
                            for (int w = 1; w < 4; ++w) {
                                vr += red[((w * NP + s) * 8 + r) * 64 + lane];
                                vi += red[((w * NP + s) * 8 + 4 + r) * 64 + lane];
                            }
                            vr += __shfl_xor(vr, 16, 64);
                            vi += __shfl_xor(vi, 16, 64);
                            vr += __shfl_xor(vr, 32, 64);
                            vi += __shfl_xor(vi, 32, 64);
                            const int irow = 4 * (lane >> 2) + r;
                            const int px = px0 + s * SW + irow % SW, py = py0 + irow / SW;
                            if (lane < 16 && tb < a.mu && px < a.nx && py < a.ny)
                                yo[((int64_t)py * a.nx + px) * a.mu + tb] = cf32{vr, vi};
                        }
                }
            }
        }
        if (!wave_active) return;
        cf32* yo = a.yraw + (int64_t)sp_all * a.npos * a.mu;
        if constexpr (TAIL) {
            // lane l holds rows r = 0..3 (positions 4 (l / 4 % 4) + r) of column
            // l % 4 of block l / 4; the blocks of the four depth groups (lanes l,
            // l ^ 16, l ^ 32, l ^ 48) are summed in a fixed order
#pragma unroll
            for (int s = 0; s < NP; ++s)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    out_re[s][r] += __shfl_xor(out_re[s][r], 16, 64);
                    out_im[s][r] += __shfl_xor(out_im[s][r], 16, 64);
                    out_re[s][r] += __shfl_xor(out_re[s][r], 32, 64);
                    out_im[s][r] += __shfl_xor(out_im[s][r], 32, 64);
                }
            if (lane >= 16 || mb >= a.mu) return;
#pragma unroll
            for (int s = 0; s < NP; ++s) {
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int irow = 4 * (lane >> 2) + r;
                    const int px = px0 + s * SW + irow % SW, py = py0 + irow / SW;
                    if (px < a.nx && py < a.ny)
                        yo[((int64_t)py * a.nx + px) * a.mu + mb] = cf32{out_re[s][r], out_im[s][r]};
                }
            }
        } else {
            if (mb >= a.mu) return;
#pragma unroll
            for (int s = 0; s < NP; ++s) {
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    int irow = 4 * kq + r;
                    int px = px0 + s * SW + irow % SW, py = py0 + irow / SW;
                    if (px < a.nx && py < a.ny)
                        yo[((int64_t)py * a.nx + px) * a.mu + mb] = cf32{out_re[s][r], out_im[s][r]};
                }
            }
        }
    };
    if (tail) run(std::true_type{});
    else run(std::false_type{});
}

// Registers for at least 3 (4 sub-tiles per wave) or 4 waves per SIMD: two
// workgroups of a CU already keep its issue slots full, the third covers their
// staging rounds.
template <int NP, int ZC, int SW, bool DIR = false, bool FOLD = false>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(NP == 4 ? 3 : 4)))
void fwd_gemm_f32_kernel(FwdArgs a) {
    extern __shared__ __align__(16) unsigned char smem[];
    fwd_f32_body<NP, ZC, SW, DIR, FOLD>(a, blockIdx.x, smem);
}

// Grouped launch: block -> (plan index, block index inside that plan's grid).
template <int NP>
__global__ __launch_bounds__(512) void fwd_gemm_f32_kernel_grouped(const FwdArgs* __restrict__ descs,
                                                 const int2* __restrict__ blk) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int2 sb = blk[blockIdx.x];
    const FwdArgs a = descs[sb.x];
    // scans of one batch may differ in depth chunk and in sub-tile shape
    if (a.sw == 4) {
        if (a.zc == 16) fwd_f32_body<NP, 16, 4>(a, sb.y, smem);
        else if (a.zc == 8) fwd_f32_body<NP, 8, 4>(a, sb.y, smem);
        else fwd_f32_body<NP, 4, 4>(a, sb.y, smem);
    } else {
        if (a.zc == 16) fwd_f32_body<NP, 16, 16>(a, sb.y, smem);
        else if (a.zc == 8) fwd_f32_body<NP, 8, 16>(a, sb.y, smem);
        else fwd_f32_body<NP, 4, 16>(a, sb.y, smem);
    }
}

// Product steps per offset of the last bin chunk (of kc bins; a last chunk of at
// most 2 bins takes two offsets per product, half a step each).
__device__ __forceinline__ int last_chunk_cost(int mu, int kc) {
    const int left = mu - (mu - 1) / kc * kc;
    return (left + 3) / 4;
}

struct AdjArgs {
    const cf32* r;         // H-scaled operand [npos][mu]
    cf32* out;             // [ny][nx][nz]
    const uint32_t* u;
    const float* amp;      // beam amplitude, same layout as u (DIR kernels only)
    const int* kb;
    int nx, ny, nz, wx, wy, mu;
    int sw, ntx, nty, nzt; // lateral tiles, depth tiles (of 16 * waves)
    int kc;                // bin chunk (multiple of 4)
    int split;             // parts, see tile_range; split > 1 writes partials
    int top;               // the heaviest tile's work
    int kcons;             // the union is consecutive bins
    cf32* part;            // [split][ny][nx][nz] when split > 1
    int64_t nvox;
    int nblk;              // blocks of this plan's grid
};

// KC: the bin chunk a.kc as a compile-time constant (16, 8 or 4).
// DIR: scale each phasor by the beam amplitude (staged in LDS after the bins).
// NW: waves per workgroup, each on its own 16 depths; the staged halo
// (positions x bins) is the same for every depth, so 8 waves share one halo
// over 128 depths where 4 waves cover 64.
template <int NP, int KC, int SW, bool DIR = false, int NW = 4>
__device__ __forceinline__ void adj_f32_body(const AdjArgs& a, const int b, unsigned char* smem) {
    constexpr int NJ = KC / 4, cs = cell_stride(KC);
    constexpr int tpx = SW * NP, tpy = 16 / SW;
    constexpr int zspan = 16 * NW;                   // depths per workgroup
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int hc = tpx + 2 * a.wx;
    const int pitch = row_pitch(hc, KC);
    const int zrun = zero_run(NP, SW, KC);
    cf32* halo = reinterpret_cast<cf32*>(smem);
    uint32_t* ulds = reinterpret_cast<uint32_t*>(halo + (size_t)tpy * pitch + zrun);
    int* klds = reinterpret_cast<int*>(ulds + (size_t)(a.wx + 1) * zspan);
    float* glds = reinterpret_cast<float*>(klds + KC);

    const int ntile = a.ntx * a.nty;
    int tile, sp;
    deal(b, ntile * a.nzt, a.split, tile, sp);
    const int zt = tile / ntile;
    tile -= zt * ntile;
    const int vx0 = (tile % a.ntx) * tpx, vy0 = (tile / a.ntx) * tpy;
    const int zw0 = zt * zspan;                      // first depth of the workgroup
    const TileRange R = tile_range(vx0, vy0, NP, SW, tpy, a.nx, a.ny, a.wx, a.wy, (a.mu + KC - 1) / KC, NJ,
                                   last_chunk_cost(a.mu, KC), sp, a.split, 0, 1, a.top);
    const int x_lo = max(0, vx0 - a.wx), x_hi = min(a.nx - 1, vx0 + tpx - 1 + a.wx);
    int axl[NP];
#pragma unroll
    for (int s = 0; s < NP; ++s) axl[s] = last_ax(vx0 + s * SW, SW, a.nx);

    for (int t = threadIdx.x; t < tpy * pitch + zrun; t += 64 * NW) halo[t] = cf32{0.f, 0.f};

    const int i = lane & 15, ix = i % SW, iy = i / SW;
    const int kq = lane >> 4;
    const bool wave_active = zw0 + wave * 16 < a.nz;
    const cf32* cell0 = halo + iy * pitch + (ix + a.wx) * cs;
    const cf32* zcell = halo + tpy * pitch;
    const uint32_t* ucol = ulds + wave * 16 + i;
    const float* gcol = glds + wave * 16 + i;

    f4 out_re[NP], out_im[NP];
#pragma unroll
    for (int s = 0; s < NP; ++s) out_re[s] = out_im[s] = f4{0.f, 0.f, 0.f, 0.f};

    for (int t = R.t0; t < R.t1; ++t) {
        const int ki = t / R.nay, ay = R.nay - 1 - (t - ki * R.nay), k0 = ki * KC;
        const int left = a.mu - k0;                       // bins of this chunk, if fewer than KC
        __syncthreads();
        stage_mirrored<KC, tpy>(halo, pitch, a.r, a.ny, a.nx, a.mu, vy0, ay, vx0 - a.wx, x_lo, x_hi, k0, a.mu);
        for (int q = threadIdx.x; q < (a.wx + 1) * zspan; q += 64 * NW) {
            const int ax = q / zspan, z = zw0 + (q & (zspan - 1));
            const int64_t o = ((int64_t)ay * (a.wx + 1) + ax) * a.nz + z;
            ulds[q] = z < a.nz ? a.u[o] : 0u;
            if (DIR) glds[q] = z < a.nz ? a.amp[o] : 0.f;
        }
        for (int q = threadIdx.x; q < KC; q += 64 * NW) klds[q] = q < left ? a.kb[k0 + q] : 0;
        __syncthreads();
        if (!wave_active) continue;
        // Gauss's three-product form of (rr + j ri)(c + j s):
        //   m1 = c (rr + ri), m2 = rr (s - c), m3 = ri (c + s);
        //   Re = m1 - m3 = rr c - ri s,  Im = m1 + m2 = rr s + ri c
        f4 m1[NP], m2[NP], m3[NP];
#pragma unroll
        for (int s = 0; s < NP; ++s) m1[s] = m2[s] = m3[s] = f4{0.f, 0.f, 0.f, 0.f};
        auto products = [&](const int s, const float rr, const float ri, const float c, const float bm, const float bp) {
            m1[s] = __builtin_amdgcn_mfma_f32_16x16x4f32(rr + ri, c, m1[s], 0, 0, 0);
            m2[s] = __builtin_amdgcn_mfma_f32_16x16x4f32(rr, bm, m2[s], 0, 0, 0);
            m3[s] = __builtin_amdgcn_mfma_f32_16x16x4f32(ri, bp, m3[s], 0, 0, 0);
        };
        if (left >= KC) {
            // a whole chunk: lane group kq takes bins NJ kq .. NJ kq + NJ - 1 of it.
            // CONS (8-wave workgroups, a union of consecutive bins): the lane's
            // phasor steps by exp(-j 2 pi u) from one to the next: one rotation
            // (4 FMAs) instead of a cos/sin pair, whose issue does not hide under
            // the products; the chain restarts from cos/sin at every offset.
            // Three rotations in a row have about twice a cos/sin pair's error, so
            // the other kernels, whose callers cannot choose, do without
            auto offsets = [&](auto consc) {
                constexpr bool CONS = decltype(consc)::value;
                uint32_t kl[NJ];
#pragma unroll
                for (int j = 0; j < NJ; ++j) kl[j] = (uint32_t)klds[NJ * kq + j];
                for (int ax = R.ax_hi; ax >= R.ax_lo; --ax) {
                    const uint32_t uz = ucol[ax * zspan];
                    const float gz = DIR ? gcol[ax * zspan] : 1.f;
                    const cf32* lrow = cell0 - ax * cs + NJ * kq;
                    const cf32* rrow = ax > 0 ? cell0 + ax * cs + NJ * kq : zcell;
                    float pc, ps, rc, rsn;
                    if constexpr (CONS) {
                        phasor(kl[0] * uz, pc, ps);
                        phasor(uz, rc, rsn);
                    }
                    float cj[NJ], bm[NJ], bp[NJ];
#pragma unroll
                    for (int j = 0; j < NJ; ++j) {
                        float c, sn;
                        if constexpr (CONS) {
                            c = pc;
                            sn = ps;
                            if (j + 1 < NJ) {
                                pc = c * rc - sn * rsn;
                                ps = sn * rc + c * rsn;
                            }
                        } else {
                            phasor(kl[j] * uz, c, sn);
                        }
                        if (DIR) {
                            c *= gz;
                            sn *= gz;
                        }
                        cj[j] = c;
                        bm[j] = sn - c;
                        bp[j] = c + sn;
                    }
#pragma unroll
                    for (int s = 0; s < NP; ++s) {
                        if (ax > axl[s]) continue;        // operands zero (wave-uniform)
                        cf32 l[NJ], r[NJ];
                        lane_values<KC>(lrow + s * SW * cs, l);
                        lane_values<KC>(rrow + s * SW * cs, r);
#pragma unroll
                        for (int j = 0; j < NJ; ++j)
                            products(s, l[j].re + r[j].re, l[j].im + r[j].im, cj[j], bm[j], bp[j]);
                    }
                }
            };
            if constexpr (NW == 8 && NJ > 1) {
                if (a.kcons) offsets(std::true_type{});
                else offsets(std::false_type{});
            } else {
                offsets(std::false_type{});
            }
        } else if (left <= 2) {
            // a last chunk of at most 2 bins: the K = 4 of one product takes
            // those bins at two offsets, lane groups kq = 0, 1 at a_x and
            // kq = 2, 3 at a_x - 1 (zero past the first), so the chunk runs half
            // the offset steps and no product lane carries a padding bin
            const uint32_t k = (uint32_t)klds[kq & 1];
            for (int ax = R.ax_hi; ax >= R.ax_lo; ax -= 2) {
                const int al = ax - (kq >> 1);
                const bool ok = al >= R.ax_lo;
                const int ad = ok ? al : ax;
                const cf32* lrow = cell0 - ad * cs + (kq & 1);
                const cf32* rrow = cell0 + ad * cs + (kq & 1);
                float c, sn;
                phasor(k * ucol[ad * zspan], c, sn);
                if (DIR) {
                    const float gv = gcol[ad * zspan];
                    c *= gv;
                    sn *= gv;
                }
                const float bm = sn - c, bp = c + sn;
#pragma unroll
                for (int s = 0; s < NP; ++s) {
                    cf32 l = lrow[s * SW * cs], r = rrow[s * SW * cs];
                    if (!ok) l = cf32{0.f, 0.f};
                    if (!ok || ad == 0) r = cf32{0.f, 0.f};
                    products(s, l.re + r.re, l.im + r.im, c, bm, bp);
                }
            }
        } else {
            // a short last chunk: bins 4 j + kq, as many steps as it has fours
            const int nj = (left + 3) >> 2;
            for (int ax = R.ax_hi; ax >= R.ax_lo; --ax) {
                const uint32_t uz = ucol[ax * zspan];
                const float gz = DIR ? gcol[ax * zspan] : 1.f;
                const cf32* lrow = cell0 - ax * cs + kq;
                const cf32* rrow = ax > 0 ? cell0 + ax * cs + kq : zcell;
                for (int j = 0; j < nj; ++j) {
                    float c, sn;
                    phasor((uint32_t)klds[4 * j + kq] * uz, c, sn);
                    if (DIR) {
                        c *= gz;
                        sn *= gz;
                    }
                    const float bm = sn - c, bp = c + sn;
#pragma unroll
                    for (int s = 0; s < NP; ++s) {
                        if (ax > axl[s]) continue;
                        const cf32 l = lrow[s * SW * cs + 4 * j], r = rrow[s * SW * cs + (ax > 0 ? 4 * j : 0)];
                        products(s, l.re + r.re, l.im + r.im, c, bm, bp);
                    }
                }
            }
        }
#pragma unroll
        for (int s = 0; s < NP; ++s) {
            out_re[s] += m1[s] - m3[s];
            out_im[s] += m1[s] + m2[s];
        }
    }
    if (!wave_active) return;
    cf32* dst = a.split > 1 ? a.part + (int64_t)sp * a.nvox : a.out;
#pragma unroll
    for (int s = 0; s < NP; ++s)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            int irow = 4 * kq + r;
            int vx = vx0 + s * SW + irow % SW, vy = vy0 + irow / SW;
            int z = zw0 + wave * 16 + i;
            if (vx < a.nx && vy < a.ny && z < a.nz)
                dst[((int64_t)vy * a.nx + vx) * a.nz + z] = cf32{out_re[s][r], out_im[s][r]};
        }
}

template <int NP, int KC, int SW, bool DIR = false, int NW = 4>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(NP == 4 ? 3 : 4)))
void adj_gemm_f32_kernel(AdjArgs a) {
    extern __shared__ __align__(16) unsigned char smem[];
    adj_f32_body<NP, KC, SW, DIR, NW>(a, blockIdx.x, smem);
}

// Grouped launch: block -> (plan index, block index inside that plan's grid).
template <int NP>
__global__ __launch_bounds__(256) void adj_gemm_f32_kernel_grouped(const AdjArgs* __restrict__ descs,
                                                 const int2* __restrict__ blk) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int2 sb = blk[blockIdx.x];
    const AdjArgs a = descs[sb.x];
    if (a.sw == 4) {
        if (a.kc == 16) adj_f32_body<NP, 16, 4>(a, sb.y, smem);
        else if (a.kc == 8) adj_f32_body<NP, 8, 4>(a, sb.y, smem);
        else adj_f32_body<NP, 4, 4>(a, sb.y, smem);
    } else {
        if (a.kc == 16) adj_f32_body<NP, 16, 16>(a, sb.y, smem);
        else if (a.kc == 8) adj_f32_body<NP, 8, 16>(a, sb.y, smem);
        else adj_f32_body<NP, 4, 16>(a, sb.y, smem);
    }
}

// ---------------------------------------------------------------------------
// Host launchers.
// ---------------------------------------------------------------------------
static constexpr int kGroupNP = 2;   // grouped (batched) launches: one shape for every scan

int fwd_tile_np(const Plan& P) { return P.fwd_np == 4 ? 4 : 2; }
int adj_tile_np(const Plan& P) { return P.adj_np == 4 ? 4 : 2; }
int adj_waves(const Plan& P) { return adj_tile_np(P) == 2 && P.adj_nw == 8 ? 8 : 4; }

static int fwd_args(const Plan& P, const cf32* x, FwdArgs& a, size_t& lds, int np, bool fold = true);
static int adj_args(const Plan& P, cf32* out, AdjArgs& a, size_t& lds, int np, int nw = 4);

int fwd_chunk(const Plan& P) {
    FwdArgs a;
    size_t lds;
    fwd_args(P, nullptr, a, lds, fwd_tile_np(P));
    return a.zc;
}

int adj_chunk(const Plan& P) {
    AdjArgs a;
    size_t lds;
    adj_args(P, nullptr, a, lds, adj_tile_np(P), adj_waves(P));
    return a.kc;
}
static constexpr size_t kLdsMax = 64 * 1024;

static int sub_width(const Plan& P) { return P.g.ny == 1 ? 16 : 4; }

// The heaviest tile's work (see tile_range).
static int top_work(const Plan& P, int np) {
    const int sw = sub_width(P), tpx = sw * np, tpy = 16 / sw;
    int mx = 1, my = 1;
    for (int x0 = 0; x0 < P.g.nx; x0 += tpx) mx = std::max(mx, tile_nax(x0, np, sw, P.g.nx, P.d.wx));
    for (int y0 = 0; y0 < P.g.ny; y0 += tpy) my = std::max(my, tile_nay(y0, tpy, P.g.ny, P.d.wy));
    return mx * my;
}

// Default number of parts for `groups` workgroups per part and lateral tile: as
// many as make about 3072 workgroups with work (12 per CU: the dispatcher evens
// out their differences; fewer, larger ones measured up to 25% slower on the
// 32 x 32 C-scan), within 64 parts, the steps of a tile and kPartsMax.
static int default_split(const Plan& P, int np, int groups, int steps, int64_t part_bytes) {
    const int sw = sub_width(P), tpx = sw * np, tpy = 16 / sw;
    int64_t sx = 0, sy = 0;
    for (int x0 = 0; x0 < P.g.nx; x0 += tpx) sx += tile_nax(x0, np, sw, P.g.nx, P.d.wx);
    for (int y0 = 0; y0 < P.g.ny; y0 += tpy) sy += tile_nay(y0, tpy, P.g.ny, P.d.wy);
    const double full = std::max(1.0, (double)sx * sy / top_work(P, np) * groups);   // workgroups with work per part
    const int64_t most = std::max<int64_t>(1, kPartsMax / part_bytes);
    const int64_t split = std::max<int64_t>(1, std::min<int64_t>({(int64_t)(3072.0 / full + 0.5), 64, steps, most}));
    return (int)(split >= 8 ? split & ~(int64_t)7 : split);      // whole eighths for the XCDs
}

int gemm_split(const Plan& P) {
    const int mu = (int)P.ubins_h.size();
    const int nw = std::max(1, std::min(P.fwd_nw, (mu + 15) / 16));
    const int steps = P.g.ny == 1 ? std::min(P.d.wx + 1, 4) : (P.d.wy + 1) * ((P.g.nz + 15) / 16);
    return default_split(P, fwd_tile_np(P), (mu + 16 * nw - 1) / (16 * nw), steps, (int64_t)P.npos * mu * 8 * gemm_zsplit(P));
}

// A B-scan's forward: its parts are depth chunks first (a workgroup walks its
// chunks one after the other, each with a staging round of its own), then a_x.
int gemm_zsplit(const Plan& P) {
    if (P.g.ny > 1) return 1;
    const int64_t most = std::max<int64_t>(1, kPartsMax / ((int64_t)P.npos * (int64_t)P.ubins_h.size() * 8));
    return (int)std::min<int64_t>({(P.g.nz + 15) / 16, 8, most});
}

int adj_split(const Plan& P) {
    const int mu = (int)P.ubins_h.size();
    const int steps = P.g.ny == 1 ? std::min(P.d.wx + 1, 16) : (P.d.wy + 1) * ((mu + 15) / 16);
    return default_split(P, adj_tile_np(P), (P.g.nz + 63) / 64, steps, P.nvox * 8);
}

// LDS bytes of one workgroup: the staged rows, the zero cells and the delay
// (and beam) rows of `tcols` entries per a_x, plus `extra`.
static size_t gemm_lds(int tpy, int hc, int np, int sw, int ch, int wx, int tcols, bool beam, size_t extra) {
    return ((size_t)tpy * row_pitch(hc, ch) + zero_run(np, sw, ch)) * sizeof(cf32) +
           (size_t)(wx + 1) * tcols * (beam ? 8 : 4) + extra;
}

// Staged chunk: the preferred one, halved until the LDS fits kLdsMax (powers of
// two: the staging needs the chunk to divide the workgroup), at least 4, which
// may take more.  Windows whose unpadded chunk of 4 exceeds kLdsMax are refused.
static int pick_chunk(int prefer, int tpy, int hc, int np, int sw, int wx, int tcols_per, int tcols, bool beam) {
    const size_t least = (size_t)tpy * hc * 5 * sizeof(cf32) + (tcols ? 16 : 0) +
                         (size_t)(wx + 1) * (tcols ? tcols : 4 * tcols_per) * (beam ? 8 : 4);
    if (least > kLdsMax) fail(UFSS_ERR_UNSUPPORTED, "aperture window too wide for the GEMM path");
    int ch = prefer == 8 ? 8 : 16;
    while (ch > 4 && gemm_lds(tpy, hc, np, sw, ch, wx, tcols ? tcols : ch * tcols_per, beam, (size_t)ch * 4) > kLdsMax)
        ch /= 2;
    return ch;
}

// Descriptor of one plan's forward GEMM launch; returns the block count.
// `fold`: allow the folded tail (single-plan launches; grouped launches keep
// one kernel body for every plan).
static int fwd_args(const Plan& P, const cf32* x, FwdArgs& a, size_t& lds, int np, bool fold) {
    a = FwdArgs{};
    a.x = x;
    a.yraw = P.d_yraw;
    a.u = P.d_u;
    a.amp = P.d_amp;
    a.kb = P.d_ubins;
    a.nx = P.g.nx;
    a.ny = P.g.ny;
    a.nz = P.g.nz;
    a.wx = P.d.wx;
    a.wy = P.d.wy;
    a.mu = (int)P.ubins_h.size();
    a.sw = sub_width(P);
    const int tpx = a.sw * np, tpy = 16 / a.sw;
    a.ntx = (a.nx + tpx - 1) / tpx;
    a.nty = (a.ny + tpy - 1) / tpy;
    a.nw = std::max(1, std::min(P.fwd_nw, (a.mu + 15) / 16));
    a.nbt = (a.mu + 16 * a.nw - 1) / (16 * a.nw);
    // four waves and at most 4 bins past the last full tile: fold them into it
    const int rem = a.mu % (16 * a.nw);
    a.ft = (fold && a.nw == 4 && a.mu > 64 && rem >= 1 && rem <= 4) ? rem : 0;
    if (a.ft) a.nbt = a.mu / 64;
    a.split = P.fwd_split;
    a.npos = P.npos;
    const int hc = tpx + 2 * a.wx;
    a.zc = pick_chunk(P.fwd_zc, tpy, hc, np, a.sw, a.wx, 1, 0, P.d_amp != nullptr);
    lds = gemm_lds(tpy, hc, np, a.sw, a.zc, a.wx, a.zc, P.d_amp != nullptr, 0);
    if (a.ft) lds = std::max(lds, (size_t)4 * np * 8 * 64 * sizeof(float));   // the folded sums
    a.zsplit = std::max(1, P.fwd_zsplit);
    a.top = top_work(P, np);
    a.nblk = a.ntx * a.nty * a.nbt * a.split * a.zsplit;
    return a.nblk;
}

// nw: waves per workgroup (4, or 8 with two sub-tiles per wave), 16 depths each.
static int adj_args(const Plan& P, cf32* out, AdjArgs& a, size_t& lds, int np, int nw) {
    a = AdjArgs{};
    a.r = static_cast<const cf32*>(P.d_rop);
    a.out = out;
    a.u = P.d_u;
    a.amp = P.d_amp;
    a.kb = P.d_ubins;
    a.nx = P.g.nx;
    a.ny = P.g.ny;
    a.nz = P.g.nz;
    a.wx = P.d.wx;
    a.wy = P.d.wy;
    a.mu = (int)P.ubins_h.size();
    a.sw = sub_width(P);
    const int tpx = a.sw * np, tpy = 16 / a.sw;
    a.ntx = (a.nx + tpx - 1) / tpx;
    a.nty = (a.ny + tpy - 1) / tpy;
    const int zspan = 16 * nw;
    a.nzt = (a.nz + zspan - 1) / zspan;
    const int hc = tpx + 2 * a.wx;
    a.kc = pick_chunk(P.adj_kc, tpy, hc, np, a.sw, a.wx, 0, zspan, P.d_amp != nullptr);
    lds = gemm_lds(tpy, hc, np, a.sw, a.kc, a.wx, zspan, P.d_amp != nullptr, (size_t)a.kc * 4);
    a.split = P.adj_split;
    a.top = top_work(P, np);
    a.kcons = P.ubins_h.back() - P.ubins_h.front() == a.mu - 1;
    a.part = P.d_gpart;
    a.nvox = P.nvox;
    a.nblk = a.ntx * a.nty * a.nzt * a.split;
    return a.nblk;
}

// A kernel may use up to 160 KiB of LDS per workgroup; above 64 KiB it has to be
// asked for (only windows whose smallest chunk needs more come here).
template <class K, class A>
static void launch_with_lds(K kernel, dim3 grid, dim3 block, size_t lds, hipStream_t s, const A& a) {
    if (lds > kLdsMax)
        UFSS_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    hipLaunchKernelGGL(kernel, grid, block, lds, s, a);
    UFSS_HIP(hipGetLastError());
}

template <int NP, int ZC, int SW, bool DIR>
static void launch_fwd(const FwdArgs& a, size_t lds, hipStream_t s) {
    const dim3 grid(a.nblk), block(64 * a.nw);
    if (a.ft) launch_with_lds(fwd_gemm_f32_kernel<NP, ZC, SW, DIR, true>, grid, block, lds, s, a);
    else launch_with_lds(fwd_gemm_f32_kernel<NP, ZC, SW, DIR, false>, grid, block, lds, s, a);
}

template <int NP, int SW, bool DIR>
static void launch_fwd_zc(const FwdArgs& a, size_t lds, hipStream_t s) {
    if (a.zc == 16) launch_fwd<NP, 16, SW, DIR>(a, lds, s);
    else if (a.zc == 8) launch_fwd<NP, 8, SW, DIR>(a, lds, s);
    else launch_fwd<NP, 4, SW, DIR>(a, lds, s);
}

void launch_forward_gemm(const Plan& P, const cf32* x, hipStream_t s) {
    FwdArgs a;
    size_t lds;
    const int np = fwd_tile_np(P);
    fwd_args(P, x, a, lds, np);
    auto go = [&](auto npc, auto swc) {
        constexpr int NP = decltype(npc)::value, SW = decltype(swc)::value;
        if (a.amp) launch_fwd_zc<NP, SW, true>(a, lds, s);
        else launch_fwd_zc<NP, SW, false>(a, lds, s);
    };
    using I2 = std::integral_constant<int, 2>;
    using I4 = std::integral_constant<int, 4>;
    using I16 = std::integral_constant<int, 16>;
    if (np == 4) {
        if (a.sw == 4) go(I4{}, I4{}); else go(I4{}, I16{});
    } else {
        if (a.sw == 4) go(I2{}, I4{}); else go(I2{}, I16{});
    }
}

template <int NP, int SW, bool DIR, int NW>
static void launch_adj_kc(const AdjArgs& a, size_t lds, hipStream_t s) {
    const dim3 grid(a.nblk), block(64 * NW);
    if (a.kc == 16) launch_with_lds(adj_gemm_f32_kernel<NP, 16, SW, DIR, NW>, grid, block, lds, s, a);
    else if (a.kc == 8) launch_with_lds(adj_gemm_f32_kernel<NP, 8, SW, DIR, NW>, grid, block, lds, s, a);
    else launch_with_lds(adj_gemm_f32_kernel<NP, 4, SW, DIR, NW>, grid, block, lds, s, a);
}

void launch_adjoint_gemm(const Plan& P, cf32* out, hipStream_t s, bool sum) {
    AdjArgs a;
    size_t lds;
    const int np = adj_tile_np(P), nw = adj_waves(P);
    adj_args(P, out, a, lds, np, nw);
    auto go = [&](auto npc, auto swc, auto nwc) {
        constexpr int NP = decltype(npc)::value, SW = decltype(swc)::value, NW = decltype(nwc)::value;
        if (a.amp) launch_adj_kc<NP, SW, true, NW>(a, lds, s);
        else launch_adj_kc<NP, SW, false, NW>(a, lds, s);
    };
    using I2 = std::integral_constant<int, 2>;
    using I4 = std::integral_constant<int, 4>;
    using I8 = std::integral_constant<int, 8>;
    using I16 = std::integral_constant<int, 16>;
    if (np == 4) {
        if (a.sw == 4) go(I4{}, I4{}, I4{}); else go(I4{}, I16{}, I4{});
    } else if (nw == 8) {
        if (a.sw == 4) go(I2{}, I4{}, I8{}); else go(I2{}, I16{}, I8{});
    } else {
        if (a.sw == 4) go(I2{}, I4{}, I4{}); else go(I2{}, I16{}, I4{});
    }
    if (a.split > 1 && sum) launch_sum_parts(P.d_gpart, a.split, P.nvox, out, s);
}

// Grouped launches (one grid for many plans).  Descriptors are opaque bytes.
size_t desc_size(GemmKind k) {
    switch (k) {
        case GemmKind::FwdF32: return sizeof(FwdArgs);
        case GemmKind::AdjF32: return sizeof(AdjArgs);
        default: return bf16_desc_size(k);
    }
}

int make_desc(GemmKind k, const Plan& P, const void* in, void* out, void* desc, size_t* lds, int* threads) {
    if (P.d_amp) fail(UFSS_ERR_UNSUPPORTED, "grouped launches do not take a Gaussian beam");
    if (P.mix) fail(UFSS_ERR_UNSUPPORTED, "grouped launches do not take mixed plans");
    switch (k) {
        case GemmKind::FwdF32: {
            FwdArgs& a = *static_cast<FwdArgs*>(desc);
            const int nb = fwd_args(P, static_cast<const cf32*>(in), a, *lds, kGroupNP, false);
            *threads = 64 * a.nw;                   // the waves with a bin sub-tile
            return nb;
        }
        case GemmKind::AdjF32:
            *threads = 256;
            return adj_args(P, static_cast<cf32*>(out), *static_cast<AdjArgs*>(desc), *lds, kGroupNP);
        default:
            *threads = 256;
            return bf16_make_desc(k, P, in, out, desc, lds);
    }
}

void launch_grouped(GemmKind k, const void* descs, const int2* blk, int nblocks, size_t lds, int threads,
                    hipStream_t s) {
    if (nblocks <= 0) return;
    auto raise = [&](const void* kernel) {
        if (lds > kLdsMax) UFSS_HIP(hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    };
    switch (k) {
        case GemmKind::FwdF32:
            if (threads < 64 || threads > 512 || threads % 64)
                fail(UFSS_ERR_INVALID_ARG, "grouped forward: workgroup size must be 64 to 512 in steps of 64");
            raise(reinterpret_cast<const void*>(fwd_gemm_f32_kernel_grouped<kGroupNP>));
            hipLaunchKernelGGL(fwd_gemm_f32_kernel_grouped<kGroupNP>, dim3(nblocks), dim3(threads), lds, s,
                               static_cast<const FwdArgs*>(descs), blk);
            break;
        case GemmKind::AdjF32:
            raise(reinterpret_cast<const void*>(adj_gemm_f32_kernel_grouped<kGroupNP>));
            hipLaunchKernelGGL(adj_gemm_f32_kernel_grouped<kGroupNP>, dim3(nblocks), dim3(256), lds, s,
                               static_cast<const AdjArgs*>(descs), blk);
            break;
        default: bf16_launch_grouped(k, descs, blk, nblocks, lds, s); return;
    }
    UFSS_HIP(hipGetLastError());
}

}  // namespace ufss
