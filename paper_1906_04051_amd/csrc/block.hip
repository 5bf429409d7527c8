// Block GMRES(m) for k <= 16 right-hand sides sharing A (A X = B).
//
// The paper solves one right-hand side at a time (Sec. 3.2); with several,
// the same minimisation over the block Krylov space span{R0, A R0, ...}
// turns the Gram-Schmidt work into tall-skinny matrix products, which run
// here on the FP64 matrix cores (v_mfma_f64_16x16x4f64):
//   - vectors are 16-wide row-major panels (n_pad x 16, columns >= k zero):
//     one row of a panel is one 128-byte line;
//   - SpMM Y = A X: 16 lanes per row, one per column, so every gather reads
//     one line of X;
//   - C = [V_0 .. V_j]^T W: one 16x16 MFMA accumulator per panel, 4 rows of
//     every panel per instruction (one coalesced 512-byte load per panel);
//   - W -/+= sum_i V_i C_i: one 16-row tile per wavefront, the coefficients in
//     LDS;
//   - block Gram-Schmidt applied twice (BCGS2), then the new block by
//     Cholesky QR applied twice (CholQR2): H_{j+1,j} = R2 R1;
//   - the band Hessenberg least-squares problem by Householder reflections
//     updated per block step in one workgroup (the oracle refactors it from
//     scratch; equal in exact arithmetic), the per-column residual estimate
//     from the transformed right-hand side (analogue of eq. res).
// Readings shared with the oracle: iterations are block steps; a cycle runs on
// the columns whose true residual has not passed; a new column whose norm
// after orthogonalisation is <= 1e-10 times its norm before ends the cycle
// after that block step (its new basis block is never used); at a restart a
// residual column dependent on the earlier ones (same test) adds no basis
// vector but stays a right-hand side of the least-squares problem (kb <= ka
// basis columns per block); a zero initial residual column is rejected.
#include <hip/hip_ext.h>

#include <cmath>
#include <mutex>
#include <new>

#include "internal.hpp"

namespace gm {

namespace {

constexpr int kBW = 16;            // panel width
constexpr int kPan = kBW * kBW;    // entries of one 16 x 16 coefficient block
constexpr int kDotGrid = 1024;     // workgroups of the dot kernel (partials)
constexpr int kSplit = 16;         // first-level splits of the partial sums
constexpr int kNormGrid = 1024;    // workgroups of the residual kernel
constexpr int kLdH = (kBlockStepsMax + 1) * kBW;   // rows of the least-squares arrays
constexpr double kBdTol = 1e-10;
constexpr int kZtChunksMax = 64;   // workgroups per row of Z^T in the panel's Z^T W (at most)

typedef double d4 __attribute__((ext_vector_type(4)));

// D += A B for A 16x4, B 4x16: lane l feeds A[l % 16][l / 16] and
// B[l / 16][l % 16]; register r of lane l holds D[l / 16 + 4 r][l % 16].
__device__ __forceinline__ d4 mfma16(double a, double b, d4 c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// Rows n .. n_pad - 1 of three panels that follow each other (stride ps).
__global__ __launch_bounds__(kWG) void k_bpad(int64_t n, int64_t n_pad, int pw, int64_t ps, double* __restrict__ P) {
    const int cnt = (int)(n_pad - n) * pw;
    for (int e = threadIdx.x; e < 3 * cnt; e += kWG) P[e / cnt * ps + n * pw + e % cnt] = 0.0;
}

// Row-major n x k (caller layout) <-> panel of pw columns (pw = 8 or 16,
// k <= pw; rows of pw doubles).
__global__ __launch_bounds__(kWG) void k_bpack(int64_t n, int k, int pw, const double* __restrict__ src,
                                               double* __restrict__ P) {
    const int64_t e = (int64_t)blockIdx.x * kWG + threadIdx.x;
    if (e >= n * pw) return;
    const int64_t row = e / pw;
    const int c = (int)(e % pw);
    P[e] = (c < k && src) ? src[row * k + c] : 0.0;
}

__global__ __launch_bounds__(kWG) void k_bunpack(int64_t n, int k, int pw, const double* __restrict__ P,
                                                 double* __restrict__ dst) {
    const int64_t e = (int64_t)blockIdx.x * kWG + threadIdx.x;
    if (e >= n * k) return;
    const int64_t row = e / k;
    const int c = (int)(e % k);
    dst[e] = P[row * pw + c];
}

// Deflation of a panel (Sec. 3.3, eq. precond1, applied to each of the 16
// columns): T = Z^T W, S = E^{-1} T, then W -= (A Z) S (projection) or
// X += Z S (coarse correction at exit, eq. precond2).
//
// Partial sums of T: workgroup (c, ch) sums chunk ch (of nch) of row c of
// Z^T, kWG / PW entries per round with one lane per panel column, four
// rounds' index loads issued before their gathers; fixed order.  Columns
// PW..15 of a partial are zero.
template <int PW>
__global__ __launch_bounds__(kWG) void k_bzt(int nch, const int* __restrict__ ztrp,
                                             const int* __restrict__ ztci, const double* __restrict__ ztv,
                                             const double* __restrict__ W, double* __restrict__ zpart,
                                             const int* __restrict__ stop) {
    constexpr int RG = kWG / PW;   // entries per round
    constexpr int U = 4;
    __shared__ double red[kWG];
    if (stop && *stop) return;   // a later step of a cycle that has ended
    const int c = blockIdx.x, ch = blockIdx.y;
    const int q0 = ztrp[c], q1 = ztrp[c + 1];
    const int cl = (q1 - q0 + nch - 1) / nch;
    const int a0 = q0 + ch * cl, a1 = min(q1, a0 + cl);
    const int l = threadIdx.x & (PW - 1), g = threadIdx.x / PW;
    double acc = 0.0;
    for (int q = a0 + g; q < a1; q += U * RG) {
        int row[U];
        double zvv[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int qu = q + u * RG;
            row[u] = qu < a1 ? ztci[qu] : 0;
            zvv[u] = qu < a1 ? ztv[qu] : 0.0;
        }
#pragma unroll
        for (int u = 0; u < U; ++u) acc += zvv[u] * W[(int64_t)row[u] * PW + l];
    }
    red[threadIdx.x] = acc;
    __syncthreads();
    if (threadIdx.x < kBW) {
        double t = 0.0;
        if (threadIdx.x < PW)
            for (int i = 0; i < RG; ++i) t += red[i * PW + threadIdx.x];
        zpart[((int64_t)c * nch + ch) * kBW + threadIdx.x] = t;
    }
}

// S = E^{-1} T (R x 16, row c of T the sum of its chunks in order); one
// workgroup, T and E^{-1} staged in LDS.
__global__ __launch_bounds__(kWG) void k_bcoarse(int R, int nch, const double* __restrict__ zpart,
                                                 const double* __restrict__ Einv, double* __restrict__ S,
                                                 const int* __restrict__ stop) {
    __shared__ double T[kBlockZMax * kBW];
    __shared__ double Ei[kBlockZMax * kBlockZMax];
    if (stop && *stop) return;
    for (int e = threadIdx.x; e < R * kBW; e += kWG) {
        const int c = e / kBW, l = e % kBW;
        double t = 0.0;
        for (int ch = 0; ch < nch; ++ch) t += zpart[((int64_t)c * nch + ch) * kBW + l];
        T[e] = t;
    }
    for (int e = threadIdx.x; e < R * R; e += kWG) Ei[e] = Einv[e];
    __syncthreads();
    for (int e = threadIdx.x; e < R * kBW; e += kWG) {
        const int i = e / kBW, l = e % kBW;
        double t = 0.0;
        for (int a = 0; a < R; ++a) t += Ei[a * R + i] * T[a * kBW + l];
        S[e] = t;
    }
}

// P += sign * M S over the rows of the CSR matrix M (n x R, local columns):
// sign -1 with M = A Z projects W, sign +1 with M = Z corrects X.  PW lanes
// per row (one per panel column), S (R x 16) staged in LDS.
template <int PW>
__global__ __launch_bounds__(kWG) void k_bzapply(int64_t n, int R, const int* __restrict__ mrp,
                                                 const int* __restrict__ mci, const double* __restrict__ mv,
                                                 const double* __restrict__ S, double sign, double* __restrict__ P,
                                                 const int* __restrict__ stop) {
    constexpr int rpr = kWG / PW;   // rows per round
    __shared__ double Ss[kBlockZMax * kBW];
    if (stop && *stop) return;
    for (int e = threadIdx.x; e < R * kBW; e += kWG) Ss[e] = S[e];
    __syncthreads();
    const int l = threadIdx.x & (PW - 1), rl = threadIdx.x / PW;
    for (int64_t r0 = (int64_t)blockIdx.x * rpr; r0 < n; r0 += (int64_t)gridDim.x * rpr) {
        const int64_t row = r0 + rl;
        if (row >= n) continue;
        double t = 0.0;
        for (int q = mrp[row]; q < mrp[row + 1]; ++q) {
            GM_DCHECK(mci[q] >= 0 && mci[q] < R, kDbgBlockCol);
            t += mv[q] * Ss[mci[q] * kBW + l];
        }
        P[row * PW + l] += sign * t;
    }
}

// Per-workgroup partial sums of squares of the 16 columns of a panel.
__global__ __launch_bounds__(kWG) void k_bnorm(int64_t n, int pw, const double* __restrict__ W,
                                               double* __restrict__ part) {
    __shared__ double red[kWG];
    const int l = threadIdx.x & (kBW - 1), rl = threadIdx.x / kBW;
    double acc = 0.0;
    for (int64_t r0 = (int64_t)blockIdx.x * (kWG / kBW); r0 < n; r0 += (int64_t)gridDim.x * (kWG / kBW)) {
        const int64_t row = r0 + rl;
        if (row < n && l < pw) {
            const double y = W[row * pw + l];
            acc += y * y;
        }
    }
    red[threadIdx.x] = acc;
    __syncthreads();
    if (threadIdx.x < kBW) {
        double t = 0.0;
        for (int i = 0; i < kWG / kBW; ++i) t += red[i * kBW + threadIdx.x];
        part[(int64_t)blockIdx.x * kBW + threadIdx.x] = t;
    }
}

// Y = A X (MODE 0), or Y = B - A X with per-workgroup partial sums of squares
// of every column (MODE 1).  PW / 2 lanes per row, two columns each; a
// wavefront takes 64 / (PW / 2) rows a round, a workgroup one contiguous range
// of rows, and each die a contiguous range of workgroups, so the three mesh
// lines a row gathers from meet in one L2.  What bounds it is the rate at
// which addresses are processed (16 cycles a load, whatever it reads): the
// lanes of a row would all load its column and value, 18 of 29 loads a Q1 row.
// So a wavefront loads its rows' entries once, side by side, into its part of
// LDS, reads them from there, and gathers X with 16-byte loads; the next
// entries are in flight meanwhile.  1,050,625 rows of 9, 16 columns: 182 us
// (MODE 0) and 265 (MODE 1) with a column a lane and rows dealt round the dies,
// 152 and 187 with two columns a lane, 130 and 155 with the entries staged
// (368 MB: 75 us at the rate of a copy).  A stage holds 32 entries a row: of
// longer rows it holds a few whole ones, and the lanes of the others wait.
template <int PW>
constexpr int kSpRows = kWG / (PW / 2);
constexpr int kSpC = 9;        // gathers in flight a lane (a whole Q1 row)
constexpr int kSpRounds = 2;   // rounds a workgroup when there are rows enough

template <int MODE, int PW>
__global__ __launch_bounds__(kWG) void k_bspmm(int64_t n, int rounds, const int* __restrict__ rowptr,
                                               const int* __restrict__ colind,
                                               const double* __restrict__ vals,
                                               const double* __restrict__ X,
                                               const double* __restrict__ B, double* __restrict__ Y,
                                               double* __restrict__ part, const int* __restrict__ stop) {
    constexpr int lpr = PW / 2, rpr = kSpRows<PW>;
    constexpr int NL = 32 / lpr, cap = NL * kWave;   // entries a lane, a wavefront (32 a row)
    __shared__ int sc[kWG / kWave][cap];
    __shared__ double sv[kWG / kWave][cap];
    __shared__ double red[2 * kWG];
    if (stop && *stop) return;   // a later step of a cycle that has ended
    const int l = threadIdx.x & (kWave - 1), wv = threadIdx.x / kWave;
    const int c = (l & (lpr - 1)) * 2;
    double n0 = 0.0, n1 = 0.0;
    int64_t row = (int64_t)xcd_block(blockIdx.x, gridDim.x) * rounds * rpr + wv * (kWave / lpr) + l / lpr;
    int ec[NL];
    double ev[NL];
    // Entries [base, e) into registers (at most cap of them).
    auto fetch = [&](int base, int e) {
#pragma unroll
        for (int u = 0; u < NL; ++u) {
            const int p = u * kWave + l;
            ec[u] = 0;
            ev[u] = 0.0;
            if (p < e - base) {
                ec[u] = colind[base + p];
                ev[u] = vals[base + p];
                GM_DCHECK(ec[u] >= 0 && ec[u] < n, kDbgBlockCol);
            }
        }
    };
    // Rows past n have no entries; the bounds of this round and the next.
    auto bound = [&](int64_t r) { return rowptr[r < n ? r : n]; };
    int q0 = bound(row), q1 = bound(row + 1), p0 = bound(row + rpr), p1 = bound(row + rpr + 1);
    fetch(__builtin_amdgcn_readfirstlane(q0), __builtin_amdgcn_readlane(q1, kWave - 1));
    for (int it = 0; it < rounds; ++it, row += rpr) {
        const int b0 = __builtin_amdgcn_readfirstlane(q0), e0 = __builtin_amdgcn_readlane(q1, kWave - 1);
        const int b1 = __builtin_amdgcn_readfirstlane(p0), e1 = __builtin_amdgcn_readlane(p1, kWave - 1);
        const int t0 = bound(row + 2 * rpr), t1 = bound(row + 2 * rpr + 1);
        double s0 = 0.0, s1 = 0.0;
        int base = b0;
        bool more;
        do {
            wave_lds_sync();   // the entries before these have been read
#pragma unroll
            for (int u = 0; u < NL; ++u) {
                sc[wv][u * kWave + l] = ec[u];
                sv[wv][u * kWave + l] = ev[u];
            }
            wave_lds_sync();
            more = e0 - base > cap;
            fetch(more ? base + cap : b1, more ? e0 : it + 1 < rounds ? e1 : b1);
            const int f = max(q0 - base, 0), t = min(q1 - base, cap);
            for (int q = f; q < t; q += kSpC) {
                double2 x[kSpC];
#pragma unroll
                for (int e = 0; e < kSpC; ++e)   // past the row: its last entry, dropped below
                    x[e] = *reinterpret_cast<const double2*>(X + (int64_t)sc[wv][min(q + e, t - 1)] * PW + c);
#pragma unroll
                for (int e = 0; e < kSpC; ++e)
                    if (q + e < t) {
                        const double a = sv[wv][q + e];
                        s0 += a * x[e].x;
                        s1 += a * x[e].y;
                    }
            }
            if (more) base += cap;
        } while (more);
        if (row < n) {
            double2* y = reinterpret_cast<double2*>(Y + row * PW + c);
            if (MODE == 0) {
                *y = make_double2(s0, s1);
            } else {
                const double2 b = *reinterpret_cast<const double2*>(B + row * PW + c);
                const double y0 = b.x - s0, y1 = b.y - s1;
                *y = make_double2(y0, y1);
                n0 += y0 * y0;
                n1 += y1 * y1;
            }
        }
        q0 = p0;
        q1 = p1;
        p0 = t0;
        p1 = t1;
    }
    if (MODE == 1) {
        red[2 * threadIdx.x] = n0;
        red[2 * threadIdx.x + 1] = n1;
        __syncthreads();
        if (threadIdx.x < kBW) {
            double s = 0.0;
            if (threadIdx.x < PW)
                for (int i = 0; i < rpr; ++i) s += red[i * PW + threadIdx.x];
            part[(int64_t)blockIdx.x * kBW + threadIdx.x] = s;
        }
    }
}

// The same with PW lanes per row, a column each, that read their row's entries
// themselves: every row of a workgroup advances at once, whatever its length,
// and nothing is staged before the first gather.
template <int MODE, int PW>
__global__ __launch_bounds__(kWG) void k_bspmm_rows(int64_t n, const int* __restrict__ rowptr,
                                                    const int* __restrict__ colind,
                                                    const double* __restrict__ vals,
                                                    const double* __restrict__ X,
                                                    const double* __restrict__ B, double* __restrict__ Y,
                                                    double* __restrict__ part, const int* __restrict__ stop) {
    __shared__ double red[kWG];
    if (stop && *stop) return;   // a later step of a cycle that has ended
    constexpr int rpr = kWG / PW;
    const int c = threadIdx.x & (PW - 1), rl = threadIdx.x / PW;
    double nrm = 0.0;
    for (int64_t r0 = (int64_t)blockIdx.x * rpr; r0 < n; r0 += (int64_t)gridDim.x * rpr) {
        const int64_t row = r0 + rl;
        if (row < n) {
            const int q0 = rowptr[row], q1 = rowptr[row + 1];
            double acc = 0.0;
            int q = q0;
            for (; q + 4 <= q1; q += 4) {
                const int c0 = colind[q], c1 = colind[q + 1], c2 = colind[q + 2], c3 = colind[q + 3];
                GM_DCHECK(min(min(c0, c1), min(c2, c3)) >= 0 && max(max(c0, c1), max(c2, c3)) < n,
                          kDbgBlockCol);
                const double a0 = vals[q], a1 = vals[q + 1], a2 = vals[q + 2], a3 = vals[q + 3];
                const double x0 = X[(int64_t)c0 * PW + c], x1 = X[(int64_t)c1 * PW + c];
                const double x2 = X[(int64_t)c2 * PW + c], x3 = X[(int64_t)c3 * PW + c];
                acc += a0 * x0;
                acc += a1 * x1;
                acc += a2 * x2;
                acc += a3 * x3;
            }
            for (; q < q1; ++q) {
                GM_DCHECK(colind[q] >= 0 && colind[q] < n, kDbgBlockCol);
                acc += vals[q] * X[(int64_t)colind[q] * PW + c];
            }
            if (MODE == 0) {
                Y[row * PW + c] = acc;
            } else {
                const double y = B[row * PW + c] - acc;
                Y[row * PW + c] = y;
                nrm += y * y;
            }
        }
    }
    if (MODE == 1) {
        red[threadIdx.x] = nrm;
        __syncthreads();
        if (threadIdx.x < kBW) {
            double s = 0.0;
            if (threadIdx.x < PW)
                for (int i = 0; i < rpr; ++i) s += red[i * PW + threadIdx.x];
            part[(int64_t)blockIdx.x * kBW + threadIdx.x] = s;
        }
    }
}

// Column sums of squares: out[c] = sum_b part[b * 16 + c].
__global__ __launch_bounds__(kWG) void k_bcolsum(int nblk, const double* __restrict__ part,
                                                 double* __restrict__ out) {
    __shared__ double red[kWG];
    const int c = threadIdx.x & (kBW - 1), s = threadIdx.x / kBW;
    double acc = 0.0;
#pragma unroll 16
    for (int b = s; b < nblk; b += kWG / kBW) acc += part[(int64_t)b * kBW + c];
    red[threadIdx.x] = acc;
    __syncthreads();
    if (threadIdx.x < kBW) {
        double t = 0.0;
        for (int i = 0; i < kWG / kBW; ++i) t += red[i * kBW + threadIdx.x];
        out[threadIdx.x] = t;
    }
}

// Partial products C_i = P_i^T W (P_i = panel i of V for i < nv; with gram,
// P_nv = W) over 4-row chunks, one MFMA accumulator per panel; workgroups
// with blockIdx.y = g take panels [NG g, NG g + NG) (W is read once per
// group; NG accumulators per lane);
// per-workgroup partials part[(blockIdx.x * nb + i) * 256 + m * 16 + n]
// (fixed order).  Panels beyond nb are loaded (W again) and multiplied but
// never stored, so the loop body is branch-free.
// Entry t of a workgroup's 16 x 16 block of partial dots from the
// wavefronts' accumulators red[w] (row-major).  16-wide panels: the sum over
// the wavefronts.  8-wide panels (lanes l%16 >= 8 on the second half of each
// 8-row run): entry (i, j) < 8 is quadrant (i, j) plus quadrant (i+8, j+8);
// the other entries are zero, as the 16-wide layout leaves them.
template <int PW>
__device__ __forceinline__ double fold_partial(const double (*red)[kPan], int t) {
    double s = 0.0;
    if (PW == 16) {
#pragma unroll
        for (int w = 0; w < kWG / kWave; ++w) s += red[w][t];
    } else if (t / kBW < 8 && t % kBW < 8) {
#pragma unroll
        for (int w = 0; w < kWG / kWave; ++w) s += red[w][t] + red[w][t + 8 * kBW + 8];
    }
    return s;
}

template <int NG, int PW>
__global__ __launch_bounds__(kWG, NG <= 5 ? 4 : 3) void k_bdots(int64_t n_pad, int64_t ps, const double* __restrict__ V,
                                               int nv, const double* __restrict__ W, int gram,
                                               double* __restrict__ part, const int* __restrict__ stop) {
    __shared__ double red[kWG / kWave][kPan];
    if (stop && *stop) return;   // a later step of a cycle that has ended

    const int l = threadIdx.x & (kWave - 1), wv = threadIdx.x / kWave;
    const int nb = nv + gram, i0 = blockIdx.y * NG;
    d4 acc[NG];
#pragma unroll
    for (int i = 0; i < NG; ++i) acc[i] = d4{0.0, 0.0, 0.0, 0.0};
    const double* src[NG];
#pragma unroll
    for (int i = 0; i < NG; ++i) src[i] = i0 + i < nv ? V + (i0 + i) * ps : W;
    // 16-wide panels: lane l holds row r0 + l/16, column l%16, four rows a
    // step.  8-wide panels: lanes with l%16 >= 8 take the next four rows,
    // row r0 + l/16 + 4, column l%16 - 8, so a step covers eight whole rows
    // (one contiguous 512-byte run) with no idle lane; the 8x8 diagonal
    // quadrants of the accumulator then hold the products of the two row
    // halves (the off-diagonal quadrants mix them and are dropped), and their
    // sum is the 8x8 block of dots.
    constexpr int pw = PW;
    constexpr int rows = PW == 8 ? 8 : 4;   // rows per step and wavefront
    const int64_t e = PW == 8 ? (int64_t)(l / kBW + 4 * ((l & (kBW - 1)) >> 3)) * pw + (l & 7)
                              : (int64_t)(l / kBW) * pw + (l & (kBW - 1));
    const int64_t nw = (int64_t)gridDim.x * (kWG / kWave);
    // The next step's loads are all on their way before this one's products
    // (left to itself the compiler trades them for registers).
    int64_t r0 = ((int64_t)blockIdx.x * (kWG / kWave) + wv) * rows;
    double a[NG], b = 0.0;
#pragma unroll
    for (int i = 0; i < NG; ++i) a[i] = 0.0;
    if (r0 < n_pad) {
        b = W[r0 * pw + e];
#pragma unroll
        for (int i = 0; i < NG; ++i) a[i] = src[i][r0 * pw + e];
    }
    for (; r0 < n_pad; r0 += nw * rows) {
        const int64_t r1 = r0 + nw * rows < n_pad ? r0 + nw * rows : r0;
        const double b1 = W[r1 * pw + e];
        double a1[NG];
#pragma unroll
        for (int i = 0; i < NG; ++i) a1[i] = src[i][r1 * pw + e];
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < NG; ++i) acc[i] = mfma16(a[i], b, acc[i]);
        b = b1;
#pragma unroll
        for (int i = 0; i < NG; ++i) a[i] = a1[i];
    }
#pragma unroll
    for (int i = 0; i < NG; ++i) {
        if (i0 + i < nb) {
#pragma unroll
            for (int r = 0; r < 4; ++r) red[wv][(l / kBW + 4 * r) * kBW + (l & (kBW - 1))] = acc[i][r];
            __syncthreads();
            part[((int64_t)blockIdx.x * nb + i0 + i) * kPan + threadIdx.x] = fold_partial<PW>(red, threadIdx.x);
            __syncthreads();
        }
    }
}

// Sum of the dot partials over the workgroups, fixed order: a workgroup
// takes 16 entries; its 16 x 16 threads each sum split s (workgroups s,
// s + 16, ...) of one entry, then the splits are added in order.  out = the
// sums; with acc_into: acc_into[e] = (first ? 0 : acc_into[e]) + out[e] for
// e < acc_cnt, and (diag_blk >= 0) the diagonal of block diag_blk saved to
// nb2.  Bound by load latency: kSumAhead partials are in flight a thread
// (1,024 workgroups' blocks: 5.7 us with eight, 5.0 now).
constexpr int kSumAhead = 32;
__global__ __launch_bounds__(kWG) void k_breduce(int nblk, int cnt, const double* __restrict__ part,
                                                 double* __restrict__ out, double* acc_into, int acc_cnt,
                                                 int first, int diag_blk, double* __restrict__ nb2,
                                                 const int* __restrict__ stop) {
    static_assert(kSplit * kBW == kWG, "16 entries x 16 splits per workgroup");
    __shared__ double ps[kSplit][kBW + 1];
    if (stop && *stop) return;   // a later step of a cycle that has ended
    const int el = threadIdx.x % kBW, sp = threadIdx.x / kBW;
    const int e = blockIdx.x * kBW + el;
    double acc = 0.0;
    if (e < cnt) {
        for (int b = sp; b < nblk; b += kSumAhead * kSplit) {
            double v[kSumAhead];
#pragma unroll
            for (int u = 0; u < kSumAhead; ++u)
                v[u] = b + u * kSplit < nblk ? part[(int64_t)(b + u * kSplit) * cnt + e] : 0.0;
#pragma unroll
            for (int u = 0; u < kSumAhead; ++u) acc += v[u];
        }
    }
    ps[sp][el] = acc;
    __syncthreads();
    if (sp == 0 && e < cnt) {
        double a = 0.0;
        for (int q = 0; q < kSplit; ++q) a += ps[q][el];
        out[e] = a;
        if (acc_into && e < acc_cnt) acc_into[e] = (first ? 0.0 : acc_into[e]) + a;
        if (nb2 && diag_blk >= 0) {
            const int d = e - diag_blk * kPan;
            if (d >= 0 && d < kPan && d / kBW == d % kBW) nb2[d / kBW] = a;
        }
    }
}

// sum_{i < nb} P_i C_i over the 16-row tile at r0 (C_i row-major 16 x 16 in
// LDS): lane l feeds row r0 + l%16, columns l/16 + 4q of each panel (the
// MFMA A operand, pw/4 steps a panel) and comes out holding rows
// r0 + l/16 + 4r, column l%16.  For 8-wide panels the B operand repeats C's
// first 8 columns in its upper 8, so both halves of the result hold the tile.
template <int PW>
__device__ __forceinline__ d4 tile_product(const double* V, int64_t ps, int nb, const double* cs, int64_t r0,
                                           int l) {
    d4 acc = {0.0, 0.0, 0.0, 0.0};
    const int col = PW == 8 ? (l & 7) : (l & (kBW - 1));
    for (int i = 0; i < nb; ++i) {
        const double* P = V + i * ps + (r0 + (l & (kBW - 1))) * PW + l / kBW;
        const double* Ci = cs + i * kPan + (l / kBW) * kBW + col;
        double a[PW / 4], b[PW / 4];
#pragma unroll
        for (int q = 0; q < PW / 4; ++q) {
            a[q] = P[4 * q];
            b[q] = Ci[4 * q * kBW];
        }
#pragma unroll
        for (int q = 0; q < PW / 4; ++q) acc = mfma16(a[q], b[q], acc);
    }
    return acc;
}

// OUT = IN + sign * sum_{i < nb} P_i C_i (P_i = panel i of V, C_i = C[i*256 ..]
// row-major 16x16, staged in nb * 2 KB of dynamic LDS given at launch), one
// 16-row tile per wavefront; IN may be NULL; IN, OUT and the panels may alias
// (a tile is read completely before it is written, by the same wavefront).
template <int PW>
__global__ __launch_bounds__(kWG) void k_bgemm(int64_t n_pad, int64_t ps, const double* V, int nb,
                                               const double* __restrict__ C, const double* IN,
                                               double sign, double* OUT, const int* __restrict__ stop) {
    if (stop && *stop) return;   // a later step of a cycle that has ended
    constexpr int pw = PW;
    extern __shared__ double cs[];   // nb coefficient blocks (dynamic)
    for (int t = threadIdx.x; t < nb * kPan; t += kWG) cs[t] = C[t];
    __syncthreads();
    const int l = threadIdx.x & (kWave - 1), wv = threadIdx.x / kWave;
    const int64_t ntile = n_pad / kBW;
    for (int64_t tile = (int64_t)blockIdx.x * (kWG / kWave) + wv; tile < ntile;
         tile += (int64_t)gridDim.x * (kWG / kWave)) {
        const int64_t r0 = tile * kBW;
        d4 acc = tile_product<PW>(V, ps, nb, cs, r0, l);
        if (PW == 8) {
            // both column halves of the accumulator hold the tile; lane l
            // stores rows r0 + l/16 + 4 h + 8 s (h = its half, s = 0, 1)
            const int h = (l & (kBW - 1)) >> 3;
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                const int64_t idx = (r0 + l / kBW + 4 * (2 * s + h)) * pw + (l & 7);
                OUT[idx] = (IN ? IN[idx] : 0.0) + sign * (h ? acc[2 * s + 1] : acc[2 * s]);
            }
        } else {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int64_t idx = (r0 + l / kBW + 4 * r) * pw + (l & (kBW - 1));
                OUT[idx] = (IN ? IN[idx] : 0.0) + sign * acc[r];
            }
        }
    }
}

// First projection and second dot pass of BCGS2 in one sweep over the basis:
// OUT = IN - sum_{i < NB} P_i C_i (as k_bgemm with sign -1), then the partial
// dots P_i^T OUT of this workgroup's tiles (as k_bdots, no Gram block).  One
// 16-row tile per wavefront.  Bound by the panels' bytes: every panel's tile
// is loaded once, whole lines a load and all panels in flight together, in the
// layout of the dots (lane l rows r0 + l/16 + 4r, column l%16), and turned
// through LDS into the layout of the product (row l%16, columns l/16 + 4q); the
// product leaves the new tile in the layout of the dots.  1,050,625 rows, 16
// columns, 1 to 8 panels: 236 us on average (3.7 TB/s) with the panels read a
// second time for the dots, 167 (5.1 TB/s at 8 panels) now.
template <int NB, int PW>
__global__ __launch_bounds__(kWG, NB <= 4 ? 3 : 2) void k_bgemm_dots(int64_t n_pad, int64_t ps,
                                                                     const double* V,
                                                                     const double* __restrict__ C,
                                                                     const double* IN, double* OUT,
                                                                     double* __restrict__ part,
                                                                     const int* __restrict__ stop) {
    if (stop && *stop) return;   // a later step of a cycle that has ended
    constexpr int pw = PW, np = PW / 4, ld = PW + 1;
    constexpr int kTurn = 2 * kBW * ld;   // two tiles a wavefront
    __shared__ double cs[NB * kPan];
    __shared__ double buf[kWG / kWave * (kTurn > kPan ? kTurn : kPan)];
    for (int t = threadIdx.x; t < NB * kPan; t += kWG) cs[t] = C[t];
    __syncthreads();
    const int l = threadIdx.x & (kWave - 1), wv = threadIdx.x / kWave;
    double* turn = buf + wv * kTurn;
    const int col = PW == 8 ? (l & 7) : (l & (kBW - 1));   // 8-wide: C's columns repeated
    const int hf = (l & (kBW - 1)) >> 3;                   // 8-wide: the lane's column half
    // Entry s of a lane in the layout of the dots: its row in the tile.
    auto trow = [&](int s) { return PW == 8 ? l / kBW + 4 * (2 * s + hf) : l / kBW + 4 * s; };
    d4 dacc[NB];
#pragma unroll
    for (int i = 0; i < NB; ++i) dacc[i] = d4{0.0, 0.0, 0.0, 0.0};
    const int64_t ntile = n_pad / kBW;
    for (int64_t tile = (int64_t)blockIdx.x * (kWG / kWave) + wv; tile < ntile;
         tile += (int64_t)gridDim.x * (kWG / kWave)) {
        const int64_t r0 = tile * kBW;
        double a[NB][np], wn[np];
#pragma unroll
        for (int i = 0; i < NB; ++i)
#pragma unroll
            for (int s = 0; s < np; ++s) a[i][s] = V[i * ps + (r0 + trow(s)) * pw + col];
#pragma unroll
        for (int s = 0; s < np; ++s) wn[s] = IN[(r0 + trow(s)) * pw + col];
        d4 acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int i = 0; i < NB; ++i) {
            double* tb = turn + (i & 1) * kBW * ld;
            wave_lds_sync();
#pragma unroll
            for (int s = 0; s < np; ++s) tb[trow(s) * ld + col] = a[i][s];
            wave_lds_sync();
            const double* Ci = cs + i * kPan + (l / kBW) * kBW + col;
#pragma unroll
            for (int q = 0; q < np; ++q)
                acc = mfma16(tb[(l & (kBW - 1)) * ld + l / kBW + 4 * q], Ci[4 * q * kBW], acc);
        }
#pragma unroll
        for (int s = 0; s < np; ++s) {
            // 8-wide: both column halves of acc hold the tile.
            wn[s] -= PW == 8 ? (hf ? acc[(2 * s + 1) & 3] : acc[(2 * s) & 3]) : acc[s];
            OUT[(r0 + trow(s)) * pw + col] = wn[s];
        }
#pragma unroll
        for (int i = 0; i < NB; ++i)
#pragma unroll
            for (int s = 0; s < np; ++s) dacc[i] = mfma16(a[i][s], wn[s], dacc[i]);
    }
    double (*red)[kPan] = reinterpret_cast<double (*)[kPan]>(buf);
    __syncthreads();
#pragma unroll
    for (int i = 0; i < NB; ++i) {
#pragma unroll
        for (int r = 0; r < 4; ++r) red[wv][(l / kBW + 4 * r) * kBW + (l & (kBW - 1))] = dacc[i][r];
        __syncthreads();
        part[((int64_t)blockIdx.x * NB + i) * kPan + threadIdx.x] = fold_partial<PW>(red, threadIdx.x);
        __syncthreads();
    }
}

// OUT = IN + sign * sum_{i < nb} P_i C_i (as k_bgemm), then the partial Gram
// block OUT^T OUT of this workgroup's tiles.  The new tile leaves the product
// in the layout both operands of the dot step take (as in k_bgemm_dots), so
// the Gram block needs no second read of OUT.  One 16-row tile per wavefront;
// the coefficients' LDS (sized for max(nb, kWG / kWave) blocks at launch)
// holds the wavefronts' accumulators at the end.
template <int PW>
__global__ __launch_bounds__(kWG) void k_bgemm_gram(int64_t n_pad, int64_t ps, const double* V, int nb,
                                                    const double* __restrict__ C, const double* IN, double sign,
                                                    double* OUT, double* __restrict__ part,
                                                    const int* __restrict__ stop) {
    if (stop && *stop) return;   // a later step of a cycle that has ended
    constexpr int pw = PW;
    extern __shared__ double cs[];   // max(nb, 4) blocks (dynamic): coefficients, then accumulators
    for (int t = threadIdx.x; t < nb * kPan; t += kWG) cs[t] = C[t];
    __syncthreads();
    const int l = threadIdx.x & (kWave - 1), wv = threadIdx.x / kWave;
    d4 g = {0.0, 0.0, 0.0, 0.0};
    const int64_t ntile = n_pad / kBW;
    for (int64_t tile = (int64_t)blockIdx.x * (kWG / kWave) + wv; tile < ntile;
         tile += (int64_t)gridDim.x * (kWG / kWave)) {
        const int64_t r0 = tile * kBW;
        const d4 acc = tile_product<PW>(V, ps, nb, cs, r0, l);
        if (PW == 8) {
            // lane l: rows r0 + l/16 + 4 h + 8 s, column l%8 (h = its column
            // half); each s is one 8-row Gram step in the k_bdots layout
            const int h = (l & (kBW - 1)) >> 3;
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                const int64_t idx = (r0 + l / kBW + 4 * (2 * s + h)) * pw + (l & 7);
                const double v = (IN ? IN[idx] : 0.0) + sign * (h ? acc[2 * s + 1] : acc[2 * s]);
                OUT[idx] = v;
                g = mfma16(v, v, g);
            }
        } else {
            double v[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int64_t idx = (r0 + l / kBW + 4 * r) * pw + (l & (kBW - 1));
                v[r] = (IN ? IN[idx] : 0.0) + sign * acc[r];
                OUT[idx] = v[r];
            }
#pragma unroll
            for (int r = 0; r < 4; ++r) g = mfma16(v[r], v[r], g);
        }
    }
    __syncthreads();   // every wavefront is done with the coefficients
    double (*red)[kPan] = reinterpret_cast<double (*)[kPan]>(cs);
#pragma unroll
    for (int r = 0; r < 4; ++r) red[wv][(l / kBW + 4 * r) * kBW + (l & (kBW - 1))] = g[r];
    __syncthreads();
    part[(int64_t)blockIdx.x * kPan + threadIdx.x] = fold_partial<PW>(red, threadIdx.x);
}

// R^T R = G for the 16x16 Gram matrix G (row-major); rows/columns >= k are
// the identity.  Rinv = R^{-1}; Rout = R Rprev (Rprev NULL: R).  With test,
// a pivot <= kBdTol times the column's norm before orthogonalisation
// (sqrt(nb2[c]), else sqrt(G_cc)) sets *flag |= 2, bdmask[c] = 1, and makes
// row c of R and of R^{-1} zero (the column counts as dependent).
//
// One wavefront, bound by the latency of its chain of k pivots: lane l holds
// rows 4 (l/16) .. + 3 of column l%16 in registers, a pivot is a lane
// broadcast, and only the pivot row goes through LDS; the inverse is one
// column a lane with R's entries broadcast from LDS.  20.3 us at k = 16 and
// 15.8 us at k = 5 with the matrices in LDS and a barrier a pivot;
// 12.0 and 7.5 us now.
__global__ __launch_bounds__(kWave) void k_bchol(int k, const double* __restrict__ G,
                                                 const double* __restrict__ nb2, int test,
                                                 const double* __restrict__ Rprev, double* __restrict__ Rout,
                                                 double* __restrict__ Rinv, int* flag,
                                                 int* __restrict__ bdmask, const int* __restrict__ stop) {
    if (stop && *stop) return;   // a later step of a cycle that has ended
    __shared__ __align__(16) double R[kPan], Rp[kPan];
    const int l = threadIdx.x, c = l & (kBW - 1), r0 = (l / kBW) * 4;
    double a[4], diag[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        a[e] = (r0 + e < k && c < k) ? G[(r0 + e) * kBW + c] : 0.0;
        diag[e] = a[e];
        Rp[(r0 + e) * kBW + c] = Rprev ? Rprev[(r0 + e) * kBW + c] : 0.0;
        R[(r0 + e) * kBW + c] = r0 + e == c ? 1.0 : 0.0;
    }
    const double nbl = nb2 ? nb2[c] : 0.0;
    unsigned bd = 0;
    wave_lds_sync();
#pragma unroll
    for (int j = 0; j < kBW; ++j) {
        if (j >= k) break;
        const int gl = (j / 4) * kBW;   // first lane of the pivot row's group
        const double p = lane_value(a[j % 4], gl + j);
        const double before = nb2 ? lane_value(nbl, j) : lane_value(diag[j % 4], gl + j);
        // A broken column counts as dependent: zero row of R.
        if (test && !(p > kBdTol * kBdTol * before)) bd |= 1u << j;
        const double d = (p > 0.0 && !((bd >> j) & 1)) ? sqrt(p) : 0.0;
        const double row = c == j ? d : (c > j && d > 0.0) ? a[j % 4] / d : 0.0;
        if (l / kBW == j / 4) R[j * kBW + c] = row;
        wave_lds_sync();
        const double rc = R[j * kBW + c];
        // Rows up to j are finished: what this leaves there is not used.
#pragma unroll
        for (int e = 0; e < 4; ++e) a[e] -= R[j * kBW + r0 + e] * rc;
    }
    // Column c of R^{-1} by back substitution (broken pivots give zeros).
    double x[kBW];
#pragma unroll
    for (int i = kBW - 1; i >= 0; --i) {
        double s = i == c ? 1.0 : 0.0;
#pragma unroll
        for (int q = i + 1; q < kBW; ++q) s -= R[i * kBW + q] * x[q];
        const double d = R[i * kBW + i];
        x[i] = s;
        if (i < k) x[i] = d > 0.0 ? s / d : 0.0;
    }
#pragma unroll
    for (int i = 0; i < kBW; ++i)
        if (l / kBW == i / 4) Rinv[i * kBW + c] = x[i];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int i = r0 + e;
        double o = 0.0;
        if (Rprev) {
#pragma unroll
            for (int q = 0; q < kBW; ++q)
                if (q >= i && q <= c) o += R[i * kBW + q] * Rp[q * kBW + c];
        } else {
            o = R[i * kBW + c];
        }
        Rout[i * kBW + c] = o;
    }
    if (test && bdmask && l < kBW) bdmask[l] = (bd >> l) & 1;
    if (test && bd && l == 0) *flag |= 2;
}

// In-place column selection of a panel: column i <- column map[i] (map[i] < 0:
// zero), one entry per thread.  pw divides the wavefront, so a row lies in
// one wavefront, whose loads of the row complete before any of its stores.
__global__ __launch_bounds__(kWG) void k_bselect(int64_t n, int pw, const int* __restrict__ map, double* P) {
    const int64_t e = (int64_t)blockIdx.x * kWG + threadIdx.x;
    if (e >= n * pw) return;
    const int c = (int)(e % pw);
    const int q = map[c];
    const double v = q >= 0 && q < pw ? P[e - c + q] : 0.0;
    P[e] = v;
}

// X[:, act[c]] += T[:, c] for c < ka.
__global__ __launch_bounds__(kWG) void k_bscatter(int64_t n, int pw, int ka, const int* __restrict__ act,
                                                  const double* __restrict__ T, double* __restrict__ X) {
    const int64_t e = (int64_t)blockIdx.x * kWG + threadIdx.x;
    if (e >= n * pw) return;
    const int64_t row = e / pw;
    const int c = (int)(e % pw);
    if (c < ka) X[row * pw + act[c]] += T[e];
}

// Least-squares state, column-major with kLdH rows: H (transformed Hbar),
// reflectors v (k + 1 entries per column) and beta, G (transformed [S; 0]).
struct LsView {
    double* H;      // kLdH * (kBlockStepsMax * kBW)
    double* v;      // (kBlockStepsMax * kBW) * (kBW + 1)
    double* beta;   // kBlockStepsMax * kBW
    double* G;      // kLdH * kBW
    double* rho0;   // kBW
    double* est;    // kBW
};

// G = [S; 0] for the cycle's starting block (S kb x ka, row-major in 16x16).
__global__ __launch_bounds__(kWG) void k_bls_init(int kb, int ka, const double* __restrict__ S, LsView ls) {
    for (int e = threadIdx.x; e < kLdH * kBW; e += kWG) {
        const int c = e / kLdH, i = e % kLdH;
        ls.G[e] = (c < ka && i < kb) ? S[i * kBW + c] : 0.0;
    }
}

// Block step j (k basis columns per block, ka right-hand sides): append the
// block column (rows 0 .. (j+2)k-1) built from the accumulated projection
// coefficients Csum (blocks 0..j) and H_{j+1,j} = Rj, apply the previous
// reflectors, make k new ones, apply them to G, and estimate each right-hand
// side's residual.  flag[0] |= 1 when every one passes.  It ends the block
// step: flag[2] counts the cycle's steps, and flag[1] (the gate of every later
// kernel of the cycle) is set once flag[0] is (this step ended the cycle).
//
// One workgroup, bound by the latency of the chain of reflectors (j k earlier
// ones, k new ones): sixteen lanes a column, entries in registers that move
// along the lanes, sums on the vector unit, one barrier a new reflector.
// k = 16, steps 1 to 8: 41 us on average with the columns in LDS and shuffled
// sums, 28 us now.
__global__ __launch_bounds__(kWG) void k_bls(int j, int k, int ka, double rtol,
                                             const double* __restrict__ Csum,
                                             const double* __restrict__ Rj, LsView ls, int* flag) {
    if (flag[1]) return;   // a later step of a cycle that has ended
    // Columns padded by one entry: threads that walk different columns at
    // the same row then hit different LDS banks.
    __shared__ double h[kBW][kLdH + 1];
    __shared__ double vl[(kBlockStepsMax - 1) * kBW * (kBW + 1)];   // previous reflectors
    __shared__ double bl[(kBlockStepsMax - 1) * kBW];
    __shared__ double col[2][kBW + 1];   // the column whose reflector is made
    __shared__ double est2[kBW];
    const int t = threadIdx.x;
    const int rows = (j + 2) * k, c0 = j * k;
    const int ct = t / kBW, li = t & (kBW - 1);
    // Rows c0 .. c0 + k - 1 of G; the rows below are still zero.
    double gw = (ct < ka && li < k) ? ls.G[(int64_t)ct * kLdH + c0 + li] : 0.0, gx = 0.0;
    // Every global load of the inputs is issued before the first is stored
    // to LDS (fixed trip counts, registers in between).
    constexpr int kVIt = ((kBlockStepsMax - 1) * kBW * (kBW + 1) + kWG - 1) / kWG;
    constexpr int kHIt = (kBW * kLdH + kWG - 1) / kWG;
    double vr[kVIt], hr[kHIt];
#pragma unroll
    for (int u = 0; u < kVIt; ++u) {
        const int e = t + u * kWG;
        vr[u] = e < c0 * (kBW + 1) ? ls.v[e] : 0.0;
    }
#pragma unroll
    for (int u = 0; u < kHIt; ++u) {
        const int e = t + u * kWG;
        const int col = e / kLdH, row = e % kLdH;
        double val = 0.0;
        if (e < kBW * kLdH && col < k && row < rows) {
            const int blk = row / k, kk = row % k;
            if (blk <= j) val = Csum[blk * kPan + kk * kBW + col];
            else val = kk <= col ? Rj[kk * kBW + col] : 0.0;
        }
        hr[u] = val;
    }
    for (int e = t; e < c0; e += kWG) bl[e] = ls.beta[e];
#pragma unroll
    for (int u = 0; u < kVIt; ++u) {
        const int e = t + u * kWG;
        if (e < c0 * (kBW + 1)) vl[e] = vr[u];
    }
#pragma unroll
    for (int u = 0; u < kHIt; ++u) {
        const int e = t + u * kWG;
        if (e < kBW * kLdH) h[e / kLdH][e % kLdH] = hr[u];
    }
    __syncthreads();
    // Sixteen lanes hold a column's window: lane i entry p + i, lane 0 also
    // entry p + 16 (x).  After reflector p the window moves down by one: entry
    // p is final, and entry p + 16 enters at lane 15.
    double w = h[ct][li], x = h[ct][kBW];
    for (int p = 0; p < c0; ++p) {
        const double v0 = li <= k ? vl[p * (kBW + 1) + li] : 0.0;
        const double v16 = k == kBW ? vl[p * (kBW + 1) + kBW] : 0.0;
        const double nx = h[ct][p + kBW + 1];
        const double sp = ggroup_sum(v0 * w + (li == 0 ? v16 * x : 0.0), kBW) * bl[p];
        w -= sp * v0;
        x -= sp * v16;
        if (li == 0 && ct < k) ls.H[(int64_t)(c0 + ct) * kLdH + p] = w;
        w = gdpp<0x12F>(li == 0 ? x : w);
        x = nx;
    }
    // New reflectors: column q's window goes to LDS, every group forms its
    // reflector and applies it to its own column and right-hand side.
    for (int q = 0; q < k; ++q) {
        double* cq = col[q & 1];
        if (ct == q) {
            cq[li] = w;
            if (li == 0) cq[kBW] = x;
        }
        __syncthreads();
        const double a0 = cq[0], x0 = li <= k ? cq[li] : 0.0, x16 = k == kBW ? cq[kBW] : 0.0;
        const double nrm = sqrt(ggroup_sum(x0 * x0 + (li == 0 ? x16 * x16 : 0.0), kBW));
        const double alpha = a0 >= 0.0 ? -nrm : nrm;
        const double v0 = nrm > 0.0 ? (li == 0 ? a0 - alpha : x0) : 0.0;
        const double v16 = nrm > 0.0 ? x16 : 0.0;
        const double vv = ggroup_sum(v0 * v0 + (li == 0 ? v16 * v16 : 0.0), kBW);
        const double beta = (nrm > 0.0 && vv > 0.0) ? 2.0 / vv : 0.0;
        if (ct == 0) {
            if (li <= k) ls.v[(int64_t)(c0 + q) * (kBW + 1) + li] = v0;
            if (li == 0) {
                if (k == kBW) ls.v[(int64_t)(c0 + q) * (kBW + 1) + kBW] = v16;
                ls.beta[c0 + q] = beta;
            }
        }
        if (beta != 0.0) {
            const double sp = ggroup_sum(v0 * w + (li == 0 ? v16 * x : 0.0), kBW) * beta;
            const double sg = ggroup_sum(v0 * gw + (li == 0 ? v16 * gx : 0.0), kBW) * beta;
            w -= sp * v0;
            x -= sp * v16;
            gw -= sg * v0;
            gx -= sg * v16;
        }
        if (li == 0) {
            if (ct >= q && ct < k) ls.H[(int64_t)(c0 + ct) * kLdH + c0 + q] = w;
            if (ct < ka) ls.G[(int64_t)ct * kLdH + c0 + q] = gw;
        }
        w = gdpp<0x12F>(li == 0 ? x : w);
        x = h[ct][min(c0 + q + kBW + 1, kLdH - 1)];   // past the block's rows: zero
        gw = gdpp<0x12F>(li == 0 ? gx : gw);
        gx = 0.0;
    }
    // Residual estimate of each right-hand side: the norm of its transformed
    // rows (j+1)k .. (j+2)k-1, now in the window.
    if (ct < ka && li < k) ls.G[(int64_t)ct * kLdH + c0 + k + li] = gw;
    const double e2 = ggroup_sum(li < k ? gw * gw : 0.0, kBW);
    if (li == 0) est2[ct] = e2;
    __syncthreads();
    if (t == 0) {
        int conv = 1;
        for (int c = 0; c < ka; ++c) {
            const double est = sqrt(est2[c]);
            ls.est[c] = est;
            if (est > rtol * ls.rho0[c]) conv = 0;
        }
        const int f = flag[0] | (conv ? 1 : 0);
        flag[0] = f;
        flag[2] += 1;
        if (f) flag[1] = 1;
    }
}

// Y = R^{-1} G_top (R: leading J x J upper triangle of H, J = nblk * k; ka
// right-hand sides), written as nblk padded 16x16 coefficient blocks
// Cy[blk * 256 + kk * 16 + c].  One workgroup, bound by the chain of J rows:
// three barriers per strip of eight rows, whose small triangle is solved in
// registers.  J = 128: 82 us with two barriers a row, 39 us now.
__global__ __launch_bounds__(kWG) void k_bsolve(int nblk, int k, int ka, LsView ls, double* __restrict__ Cy) {
    constexpr int kStrip = 8;   // rows of H staged in LDS at a time
    constexpr int kLd = (kStrip * kBlockStepsMax * kBW) / kWG;
    __shared__ double y[kLdH][kBW];
    __shared__ double part[kBW][kBW + 1];
    __shared__ double hs[kStrip][kBlockStepsMax * kBW + 1];
    const int J = nblk * k;
    const int c = threadIdx.x & (kBW - 1), g = threadIdx.x / kBW;
    // y starts as the right-hand side G; row i is overwritten by the solution
    // once the rows below it are solved.
    for (int e = threadIdx.x; e < kLdH * kBW; e += kWG) {
        const int i = e % kLdH, cc = e / kLdH;
        y[i][cc] = i < J ? ls.G[(int64_t)cc * kLdH + i] : 0.0;
    }
    double ld[kLd];   // the next strip, in flight
    auto load = [&](int i0) {
#pragma unroll
        for (int u = 0; u < kLd; ++u) {
            const int e = threadIdx.x + u * kWG, q = e / kStrip, r = e % kStrip;
            ld[u] = (i0 >= 0 && q < J && i0 + r < J && q >= i0 + r) ? ls.H[(int64_t)q * kLdH + i0 + r] : 0.0;
        }
    };
    const int last = (J - 1) / kStrip * kStrip;
    if (J > 0) load(last);
    for (int i0 = last; i0 >= 0 && J > 0; i0 -= kStrip) {
        __syncthreads();   // the previous strip is done with hs and y
#pragma unroll
        for (int u = 0; u < kLd; ++u) {
            const int e = threadIdx.x + u * kWG;
            hs[e % kStrip][e / kStrip] = ld[u];
        }
        load(i0 - kStrip);
        __syncthreads();
        // The strip's rows less the solved ones' products: two groups a row.
        {
            double s = 0.0;
#pragma unroll 4
            for (int q = i0 + kStrip + (g & 1); q < J; q += 2) s += hs[g / 2][q] * y[q][c];
            part[g][c] = s;
        }
        __syncthreads();
        if (g == 0) {
            double yy[kStrip];
#pragma unroll
            for (int r = kStrip - 1; r >= 0; --r) {
                yy[r] = 0.0;
                if (i0 + r < J) {
                    double acc = y[i0 + r][c] - part[2 * r][c] - part[2 * r + 1][c];
#pragma unroll
                    for (int q = r + 1; q < kStrip; ++q) acc -= hs[r][i0 + q] * yy[q];
                    yy[r] = c < ka ? acc / hs[r][i0 + r] : 0.0;
                    y[i0 + r][c] = yy[r];
                }
            }
        }
    }
    __syncthreads();
    for (int e = threadIdx.x; e < nblk * kPan; e += kWG) {
        const int blk = e / kPan, kk = (e % kPan) / kBW, cc = e % kBW;
        Cy[e] = (kk < k && cc < ka) ? y[blk * k + kk][cc] : 0.0;
    }
}

// Launch through the timing hook when there is one: the kernel carries the
// armed start/stop events in its own dispatch.
template <typename... KA, typename... A>
void blaunch_shm(BlockTimer* tm, int kind, double bytes, void (*k)(KA...), dim3 g, dim3 b, size_t shm,
                 hipStream_t st, A... args) {
    hipEvent_t e0, e1;
    if (tm) tm->begin(kind, bytes);
    if (tm && take_kernel_events(&e0, &e1))
        hipExtLaunchKernelGGL(k, g, b, shm, st, e0, e1, 0u, static_cast<KA>(args)...);
    else
        k<<<g, b, shm, st>>>(static_cast<KA>(args)...);
    if (tm) tm->end();
}

template <typename... KA, typename... A>
void blaunch(BlockTimer* tm, int kind, double bytes, void (*k)(KA...), dim3 g, dim3 b, hipStream_t st,
             A... args) {
    blaunch_shm(tm, kind, bytes, k, g, b, 0, st, args...);
}

constexpr int kDotGroup = 9;   // panels per workgroup of the dot kernel (at most)

}  // namespace

struct BlockWork {
    int64_t n = 0, n_pad = 0, ps = 0;
    int m = 0;
    int pw = kBW;                // panel width of the current solve (8 for k <= 8, else 16)
    double* panels = nullptr;   // (m + 1) basis panels, W, B, X
    double *part = nullptr, *C = nullptr, *Csum = nullptr;
    double *R1 = nullptr, *R = nullptr, *Rinv = nullptr, *nb2 = nullptr, *Cy = nullptr;
    double *npart = nullptr, *nsq = nullptr;
    double *lsbuf = nullptr, *S = nullptr;
    double *zpart = nullptr, *Sz = nullptr;   // deflation: Z^T W partials, E^{-1} Z^T W
    int* flag = nullptr;
    int* imap = nullptr;   // [0,16): column map; [16,32): active columns; [32,48): broken mask
    LsView ls{};
    double* V() const { return panels; }
    double* W() const { return panels + (int64_t)(m + 1) * ps; }
    double* Bp() const { return panels + (int64_t)(m + 2) * ps; }
    double* Xp() const { return panels + (int64_t)(m + 3) * ps; }
};

// Scratch of gmres_solve_block_noalloc, for callers that cannot allocate
// device memory: one array per GPU, held until the process ends.  Host code
// never passes `scratch` itself (its host-side name is not the device
// address); it uses the address looked up once per device below.
constexpr size_t kStaticScratchBytes = size_t(64) << 20;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices] = {};
}  // namespace

int static_scratch_init(int device) {
    if (device < 0 || device >= kMaxDevices) return kStatusInval;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (g_scratch_ptr[device]) return kStatusOk;
    int cur = -1;
    if (hipGetDevice(&cur) != hipSuccess || cur != device) return kStatusDevice;
    void* ptr = nullptr;
    if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) return kStatusDevice;
    g_scratch_ptr[device] = ptr;
    return kStatusOk;
}

void* static_scratch(int device, size_t* bytes) {
    *bytes = kStaticScratchBytes;
    if (device < 0 || device >= kMaxDevices) return nullptr;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    return g_scratch_ptr[device];
}

BlockWork* block_new() { return new (std::nothrow) BlockWork(); }
void block_delete(BlockWork* w) { delete w; }

namespace {

int64_t ls_entries() {
    return (int64_t)kLdH * kBlockStepsMax * kBW + (int64_t)kBlockStepsMax * kBW * (kBW + 1) +
           (int64_t)kBlockStepsMax * kBW + (int64_t)kLdH * kBW + 2 * kBW;
}

// Carves the block workspace for n rows and m block steps from an arena
// (sizing or real).
void block_carve(BlockWork* w, Arena& ar, int64_t n, int m) {
    w->n = n;
    w->n_pad = (n + 63) / 64 * 64;
    w->ps = w->n_pad * kBW;
    w->m = m;
    const int64_t nbmax = m + 2;
    w->panels = ar.take_n<double>((int64_t)(m + 4) * w->ps);
    w->part = ar.take_n<double>((int64_t)kDotGrid * nbmax * kPan);
    w->C = ar.take_n<double>(nbmax * kPan);
    w->Csum = ar.take_n<double>(nbmax * kPan);
    w->R1 = ar.take_n<double>(kPan);
    w->R = ar.take_n<double>(kPan);
    w->Rinv = ar.take_n<double>(kPan);
    w->nb2 = ar.take_n<double>(kBW);
    w->Cy = ar.take_n<double>((int64_t)(m + 1) * kPan);
    w->npart = ar.take_n<double>((int64_t)kNormGrid * kBW);
    w->nsq = ar.take_n<double>(kBW);
    w->lsbuf = ar.take_n<double>(ls_entries());
    w->S = ar.take_n<double>(kPan);
    w->zpart = ar.take_n<double>((int64_t)kBlockZMax * kZtChunksMax * kBW);
    w->Sz = ar.take_n<double>((int64_t)kBlockZMax * kBW);
    w->flag = ar.take_n<int>(3);
    w->imap = ar.take_n<int>(3 * kBW);
}

}  // namespace

size_t block_workspace_bytes(int64_t n, int m) {
    BlockWork w;
    Arena ar;
    ar.sizing = true;
    block_carve(&w, ar, n, m);
    return ar.peak;
}

int block_bind(BlockWork* w, void* mem, size_t bytes, hipStream_t st, int64_t n, int m) {
    Arena ar;
    ar.base = reinterpret_cast<uintptr_t>(mem);
    ar.cap = bytes;
    block_carve(w, ar, n, m);
    if (ar.short_ || (ar.base & 255) != 0) return kStatusNoMem;
    if (hipMemsetAsync(w->lsbuf, 0, (size_t)ls_entries() * sizeof(double), st) != hipSuccess)
        return kStatusDevice;
    double* q = w->lsbuf;
    w->ls.H = q;
    q += (int64_t)kLdH * kBlockStepsMax * kBW;
    w->ls.v = q;
    q += (int64_t)kBlockStepsMax * kBW * (kBW + 1);
    w->ls.beta = q;
    q += (int64_t)kBlockStepsMax * kBW;
    w->ls.G = q;
    q += (int64_t)kLdH * kBW;
    w->ls.rho0 = q;
    q += kBW;
    w->ls.est = q;
    return kStatusOk;
}

namespace {

// Workgroups of a sweep that leaves one partial per workgroup: one round of
// resident workgroups of `kernel` with shm bytes of dynamic LDS (at most
// kDotGrid, the partial-sum capacity), looked up once per device into cache.
std::mutex g_grid_mu;
int resident_grid(const void* kernel, int* cache, size_t shm = 0) {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return kDotGrid;
    std::lock_guard<std::mutex> lk(g_grid_mu);
    if (cache[dev] == 0) {
        int per_cu = 0, cus = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, kWG, shm) != hipSuccess || per_cu < 1)
            per_cu = 1;
        if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 1)
            cus = 1;
        cache[dev] = std::min(kDotGrid, per_cu * cus);
    }
    return cache[dev];
}

// k_bdots over nb = nv + gram blocks: ceil(nb / kDotGroup) groups of workgroups
// with the fewest slots each that hold the blocks (nb = 10: two groups of
// five).  Every slot loads a panel and issues a matrix-core step per row
// step, used or not, and every group reads W: 1,050,625 rows, 16 columns, the
// 2 to 9 blocks of a cycle of eight steps: 1,300 us in groups of at most four,
// 1,140 (5.3 TB/s at nine blocks) in groups of at most nine.
template <int NG, int PW>
int launch_dots_ng(const BlockWork& w, BlockTimer* tm, double bytes, hipStream_t st, int ng, int groups,
                    const double* V, int nv, const double* W, int gram, const int* stop) {
    if constexpr (NG > 1)
        if (ng < NG) return launch_dots_ng<NG - 1, PW>(w, tm, bytes, st, ng, groups, V, nv, W, gram, stop);
    static int cache[64] = {};
    const int grid = resident_grid(reinterpret_cast<const void*>(k_bdots<NG, PW>), cache);
    blaunch(tm, 5, bytes, k_bdots<NG, PW>, dim3(grid, groups), dim3(kWG), st, w.n_pad, w.ps, V, nv, W, gram, w.part,
            stop);
    return grid;
}

template <int PW>
int launch_dots(const BlockWork& w, BlockTimer* tm, double bytes, hipStream_t st, const double* V, int nv,
                 const double* W, int gram, const int* stop) {
    const int nb = nv + gram;
    const int groups = (nb + kDotGroup - 1) / kDotGroup;
    return launch_dots_ng<kDotGroup, PW>(w, tm, bytes, st, (nb + groups - 1) / groups, groups, V, nv, W, gram, stop);
}

// C[0 .. nb) = P^T W (panels of V, then W itself when gram), summed.
void dots(const BlockWork& w, BlockTimer* tm, hipStream_t st, const double* V, int nv, const double* W,
          int gram, double* acc_into, int acc_blocks, int first, int diag_blk, double* nb2,
          const int* stop) {
    const int nb = nv + gram;
    const double bytes = (double)(nv + 1) * (double)w.n * w.pw * sizeof(double);   // panels and W, once
    const int grid = w.pw == 8 ? launch_dots<8>(w, tm, bytes, st, V, nv, W, gram, stop)
                               : launch_dots<kBW>(w, tm, bytes, st, V, nv, W, gram, stop);
    const int cnt = nb * kPan;
    k_breduce<<<(cnt + kBW - 1) / kBW, kWG, 0, st>>>(grid, cnt, w.part, w.C, acc_into, acc_blocks * kPan,
                                                     first, diag_blk, nb2, stop);
}

void gemm(const BlockWork& w, BlockTimer* tm, hipStream_t st, const double* V, int nb, const double* C,
          const double* IN, double sign, double* OUT, const int* stop) {
    const int64_t ntile = w.n_pad / kBW;
    const int grid = (int)std::min<int64_t>((ntile + 3) / 4, 8192);
    const double bytes = (double)(nb + (IN ? 1 : 0) + 1) * (double)w.n * w.pw * sizeof(double);
    const size_t shm = (size_t)nb * kPan * sizeof(double);   // the coefficient blocks
    if (w.pw == 8)
        blaunch_shm(tm, 6, bytes, k_bgemm<8>, dim3(grid), dim3(kWG), shm, st, w.n_pad, w.ps, V, nb, C, IN, sign, OUT,
                    stop);
    else
        blaunch_shm(tm, 6, bytes, k_bgemm<kBW>, dim3(grid), dim3(kWG), shm, st, w.n_pad, w.ps, V, nb, C, IN, sign,
                    OUT, stop);
}

// W -= V C (C: the first projection's coefficients in w.C), then the second
// projection's coefficients V^T W into w.C, accumulated into acc_into (as the
// dots() call without a Gram block would); one sweep over the panels.
constexpr int kFuseMax = 8;   // panels of the fused sweep (accumulators per lane)

// Dynamic LDS of k_bgemm_gram for nb coefficient blocks (the wavefronts'
// accumulators reuse it), and its resident grid.
size_t gram_shm(int nb) { return (size_t)std::max(nb, kWG / kWave) * kPan * sizeof(double); }

template <int PW>
int gram_grid(int nb) {
    static int cache[kBlockStepsMax + 2][64] = {};
    const int blocks = std::max(nb, kWG / kWave);
    return resident_grid(reinterpret_cast<const void*>(k_bgemm_gram<PW>), cache[blocks], gram_shm(nb));
}

// Launches the sweep over nb panels (one instance each); returns its grid.
template <int NB, int PW>
int launch_gemm_dots(const BlockWork& w, BlockTimer* tm, double bytes, hipStream_t st, int nb, const double* V,
                     double* W, const int* stop) {
    if constexpr (NB > 1)
        if (nb < NB) return launch_gemm_dots<NB - 1, PW>(w, tm, bytes, st, nb, V, W, stop);
    static int cache[64] = {};
    const int grid = resident_grid(reinterpret_cast<const void*>(k_bgemm_dots<NB, PW>), cache);
    blaunch(tm, 6, bytes, k_bgemm_dots<NB, PW>, dim3(grid), dim3(kWG), st, w.n_pad, w.ps, V, (const double*)w.C,
            (const double*)W, W, w.part, stop);
    return grid;
}

void gemm_dots(const BlockWork& w, BlockTimer* tm, hipStream_t st, const double* V, int nb, double* W,
               double* acc_into, int acc_blocks, const int* stop) {
    const double bytes = (double)(nb + 2) * (double)w.n * w.pw * sizeof(double);   // panels once, W in and out
    const int grid = w.pw == 8 ? launch_gemm_dots<kFuseMax, 8>(w, tm, bytes, st, nb, V, W, stop)
                               : launch_gemm_dots<kFuseMax, kBW>(w, tm, bytes, st, nb, V, W, stop);
    const int cnt = nb * kPan;
    k_breduce<<<(cnt + kBW - 1) / kBW, kWG, 0, st>>>(grid, cnt, w.part, w.C, acc_into, acc_blocks * kPan, 0,
                                                     -1, nullptr, stop);
}

// OUT = IN + sign * V C (as gemm), and OUT^T OUT summed into w.C (as the
// dots() call of OUT's Gram block alone would); one sweep.
void gemm_gram(const BlockWork& w, BlockTimer* tm, hipStream_t st, const double* V, int nb, const double* C,
               const double* IN, double sign, double* OUT, const int* stop) {
    const double bytes = (double)(nb + (IN ? 1 : 0) + 1) * (double)w.n * w.pw * sizeof(double);
    int grid;
    if (w.pw == 8) {
        grid = gram_grid<8>(nb);
        blaunch_shm(tm, 6, bytes, k_bgemm_gram<8>, dim3(grid), dim3(kWG), gram_shm(nb), st, w.n_pad, w.ps, V, nb, C,
                    IN, sign, OUT, w.part, stop);
    } else {
        grid = gram_grid<kBW>(nb);
        blaunch_shm(tm, 6, bytes, k_bgemm_gram<kBW>, dim3(grid), dim3(kWG), gram_shm(nb), st, w.n_pad, w.ps, V, nb,
                    C, IN, sign, OUT, w.part, stop);
    }
    k_breduce<<<kPan / kBW, kWG, 0, st>>>(grid, kPan, w.part, w.C, nullptr, 0, 0, -1, nullptr, stop);
}

// Cholesky QR applied twice to the panel `src` into `dst` (may alias):
// dst R = src, R = R2 R1 (into w.R).  test: breakdown test of the first pass
// against nb2 (NULL: the Gram diagonal).  gram_ready: w.C already holds
// src^T src (the sweep that wrote src formed it).
void cholqr2(const BlockWork& w, BlockTimer* tm, hipStream_t st, int k, const double* src, double* dst,
             int test, const double* nb2, const int* stop, bool gram_ready = false) {
    if (!gram_ready) dots(w, tm, st, nullptr, 0, src, 1, nullptr, 0, 0, -1, nullptr, stop);
    k_bchol<<<1, kWave, 0, st>>>(k, w.C, nb2, test, nullptr, w.R1, w.Rinv, w.flag, w.imap + 2 * kBW, stop);
    gemm_gram(w, tm, st, src, 1, w.Rinv, nullptr, 1.0, dst, stop);   // and dst^T dst into w.C
    k_bchol<<<1, kWave, 0, st>>>(k, w.C, nullptr, 0, w.R1, w.R, w.Rinv, w.flag, nullptr, stop);
    gemm(w, tm, st, dst, 1, w.Rinv, nullptr, 1.0, dst, stop);
}

// Residual panel W = B - A X and the column norms on the host.
// Algorithmic bytes of one SpMM: A (8-byte values, 4-byte indices, row
// pointers), the input panel (one line per row), the output panel (and B).
double spmm_bytes(const BlockWork& w, const BlockArgs& a, int mode) {
    return 12.0 * (double)a.nnz + 4.0 * (double)(w.n + 1) + (2.0 + mode) * (double)w.n * w.pw * sizeof(double);
}

// Whether the SpMM stages its entries (k_bspmm) or its rows read them
// (k_bspmm_rows), by the mean row length and the work.  us a product, rows /
// staged, 16 columns: 8,000 rows of 9: 4.8 / 5.3, of 17: 7.3 / 6.2; 250,000 of 9:
// 32.4 / 26.1, of 33: 115 / 62; past the 32 entries a stage holds of a row, 20,000
// of 41: 15.5 / 17.9, of 151: 44.5 / 102; 60,000 of 65: 58.1 / 52.8, of 101: 85.1 /
// 106.  8 columns: 20,000 of 33: 10.3 / 11.1; 60,000 of 17: 12.2 / 9.9, of 65: 33.3 /
// 35.3; 250,000 of 9: 16.9 / 17.2, of 65: 134 / 127, of 101: 215 / 269.
template <int PW>
bool spmm_staged(int64_t n, int64_t nnz) {
    constexpr int64_t kEntries = PW == 8 ? 900000 : 100000, kRowsLong = PW == 8 ? 200000 : 60000;
    return nnz >= kEntries && (nnz <= 33 * n || (nnz <= 66 * n && n >= kRowsLong));
}

// Y = A X (mode 0; staged: up to kSpRounds rounds a workgroup while kNormGrid of
// them are left) or Y = B - A X with column partial sums of squares (mode 1,
// kNormGrid workgroups), the instance for the solve's panel width.
template <int MODE, int PW>
void spmm_pw(const BlockWork& w, const BlockArgs& a, const double* X, const double* B, double* Y, double* part,
             const int* stop) {
    if (!spmm_staged<PW>(w.n, a.nnz)) {
        constexpr int64_t rows = kWG / PW;
        blaunch(a.timer, 7, spmm_bytes(w, a, MODE), k_bspmm_rows<MODE, PW>,
                dim3((unsigned)(MODE == 0 ? (w.n + rows - 1) / rows : kNormGrid)), dim3(kWG), a.st, w.n, a.rowptr,
                a.colind, a.vals, X, B, Y, part, stop);
        return;
    }
    constexpr int64_t rpr = kSpRows<PW>;
    const int64_t rounds = MODE == 0 ? std::max<int64_t>(1, std::min<int64_t>(kSpRounds, w.n / (kNormGrid * rpr)))
                                     : (w.n + kNormGrid * rpr - 1) / (kNormGrid * rpr);
    const int64_t grid = MODE == 0 ? (w.n + rounds * rpr - 1) / (rounds * rpr) : kNormGrid;
    blaunch(a.timer, 7, spmm_bytes(w, a, MODE), k_bspmm<MODE, PW>, dim3((unsigned)grid), dim3(kWG), a.st, w.n,
            (int)rounds, a.rowptr, a.colind, a.vals, X, B, Y, part, stop);
}

template <int MODE>
void spmm(const BlockWork& w, const BlockArgs& a, const double* X, const double* B, double* Y, double* part,
          const int* stop) {
    if (w.pw == 8)
        spmm_pw<MODE, 8>(w, a, X, B, Y, part, stop);
    else
        spmm_pw<MODE, kBW>(w, a, X, B, Y, part, stop);
}

// S = E^{-1} Z^T P into w.Sz (deflation basis of a).
void coarse(const BlockWork& w, const BlockArgs& a, const double* P, const int* stop) {
    // About 256 entries of Z^T per workgroup (Z's rows are shared out over
    // its columns), at most kZtChunksMax workgroups per column.
    const int nch = (int)std::max<int64_t>(1, std::min<int64_t>(kZtChunksMax, (w.n + 256LL * a.R - 1) / (256LL * a.R)));
    if (w.pw == 8)
        k_bzt<8><<<dim3((unsigned)a.R, (unsigned)nch), kWG, 0, a.st>>>(nch, a.ztrp, a.ztci, a.ztv, P, w.zpart, stop);
    else
        k_bzt<kBW><<<dim3((unsigned)a.R, (unsigned)nch), kWG, 0, a.st>>>(nch, a.ztrp, a.ztci, a.ztv, P, w.zpart,
                                                                        stop);
    k_bcoarse<<<1, kWG, 0, a.st>>>(a.R, nch, w.zpart, a.Einv, w.Sz, stop);
}

// P += sign * M S (k_bzapply, S in w.Sz): pw lanes per row, kWG / pw rows per
// workgroup and round, 4096 workgroups at most.
void zapply(const BlockWork& w, hipStream_t st, int R, const int* mrp, const int* mci, const double* mv,
            double sign, double* P, const int* stop) {
    const int rpr = kWG / w.pw;
    const unsigned g = (unsigned)std::min<int64_t>((w.n + rpr - 1) / rpr, 4096);
    if (w.pw == 8)
        k_bzapply<8><<<g, kWG, 0, st>>>(w.n, R, mrp, mci, mv, w.Sz, sign, P, stop);
    else
        k_bzapply<kBW><<<g, kWG, 0, st>>>(w.n, R, mrp, mci, mv, w.Sz, sign, P, stop);
}

// W = P W = W - A Z E^{-1} Z^T W (no-op without a deflation basis).
void project(const BlockWork& w, const BlockArgs& a, double* W, const int* stop) {
    if (a.R == 0) return;
    coarse(w, a, W, stop);
    zapply(w, a.st, a.R, a.azrp, a.azci, a.azv, -1.0, W, stop);
}

// W = B - A X, h_raw[c] = ||w_c||; then W = P W and h_nrm[c] = ||P w_c||
// (h_nrm = h_raw without a deflation basis).
int residual(const BlockWork& w, const BlockArgs& a, double* h_raw, double* h_nrm) {
    spmm<1>(w, a, w.Xp(), w.Bp(), w.W(), w.npart, nullptr);
    k_bcolsum<<<1, kWG, 0, a.st>>>(kNormGrid, w.npart, w.nsq);
    double sq[kBW], sp[kBW];
    if (hipMemcpyAsync(sq, w.nsq, sizeof(sq), hipMemcpyDeviceToHost, a.st) != hipSuccess) return kStatusDevice;
    if (a.R > 0) {
        project(w, a, w.W(), nullptr);
        k_bnorm<<<kNormGrid, kWG, 0, a.st>>>(w.n, w.pw, w.W(), w.npart);
        k_bcolsum<<<1, kWG, 0, a.st>>>(kNormGrid, w.npart, w.nsq);
        if (hipMemcpyAsync(sp, w.nsq, sizeof(sp), hipMemcpyDeviceToHost, a.st) != hipSuccess)
            return kStatusDevice;
    }
    if (hipStreamSynchronize(a.st) != hipSuccess) return kStatusDevice;
    for (int c = 0; c < kBW; ++c) {
        h_raw[c] = std::sqrt(sq[c]);
        h_nrm[c] = a.R > 0 ? std::sqrt(sp[c]) : h_raw[c];
    }
    return kStatusOk;
}


}  // namespace

int block_solve(BlockWork* w, const BlockArgs& a, BlockResult* res) {
    const hipStream_t st = a.st;
    const int k = a.k, m = a.m;
    *res = BlockResult{};
    // Panels of 8 columns for up to 8 right-hand sides (half the bytes of
    // the 16-wide rows), else 16; both fit the workspace carved for 16.
    w->pw = k <= 8 ? 8 : kBW;
    w->ps = w->n_pad * w->pw;
    const int64_t pe = w->n * w->pw;
    const unsigned gpe = (unsigned)((pe + kWG - 1) / kWG);
    // Panel rows beyond n and columns beyond k stay zero through the solve:
    // set here for W, B and X; a basis panel is written whole, from W, before
    // it is read (clearing all panels took 0.27 ms at 1,050,625 rows, m = 8).
    if (w->n_pad > w->n) k_bpad<<<1, kWG, 0, st>>>(w->n, w->n_pad, w->pw, w->ps, w->W());
    k_bpack<<<gpe, kWG, 0, st>>>(w->n, k, w->pw, a.B, w->Bp());
    k_bpack<<<gpe, kWG, 0, st>>>(w->n, k, w->pw, a.X0, w->Xp());
    // rho0_c = ||b_c - A x0_c|| (unprojected); the tests use ||P (b_c - A x_c)||.
    double rho0[kBW], rn[kBW], raw[kBW];
    int s = residual(*w, a, rho0, rn);
    if (s != kStatusOk) return s;
    double rho_max = 0.0;
    for (int c = 0; c < k; ++c) {
        if (!(rho0[c] > 0.0)) return kStatusInval;   // zero (or non-finite) initial residual column
        rho_max = std::max(rho_max, rho0[c]);
    }
    res->rho0 = rho_max;
    int64_t steps = 0;
    int cycles = 0, status = kStatusMaxIter;
    double est_max = 1.0;
    for (;;) {
        // Active columns: residual not yet below rtol * rho0_c.
        int act[kBW], ka = 0;
        for (int c = 0; c < k; ++c)
            if (rn[c] > a.rtol * rho0[c]) act[ka++] = c;
        if (ka == 0) {
            status = kStatusOk;
            break;
        }
        if (steps >= a.max_steps) {
            status = kStatusMaxIter;
            break;
        }
        // Starting block from the active residual columns: V_0 S = R.
        int hmap[3 * kBW];
        for (int c = 0; c < kBW; ++c) {
            hmap[c] = c < ka ? act[c] : -1;
            hmap[kBW + c] = c < ka ? act[c] : 0;
        }
        if (hipMemcpyAsync(w->imap, hmap, 2 * kBW * sizeof(int), hipMemcpyHostToDevice, st) != hipSuccess ||
            hipMemsetAsync(w->flag, 0, sizeof(int), st) != hipSuccess ||
            hipMemsetAsync(w->imap + 2 * kBW, 0, kBW * sizeof(int), st) != hipSuccess)
            return kStatusDevice;
        k_bselect<<<gpe, kWG, 0, st>>>(w->n, w->pw, w->imap, w->W());
        cholqr2(*w, a.timer, st, ka, w->W(), w->V(), 1, nullptr, nullptr);
        // A residual column dependent on the earlier ones adds no basis
        // vector: keep kb independent columns, S = their rows of R (kb x ka).
        double hR[kPan];
        if (hipMemcpyAsync(hR, w->R, sizeof(hR), hipMemcpyDeviceToHost, st) != hipSuccess ||
            hipMemcpyAsync(hmap + 2 * kBW, w->imap + 2 * kBW, kBW * sizeof(int), hipMemcpyDeviceToHost, st) !=
                hipSuccess ||
            hipStreamSynchronize(st) != hipSuccess)
            return kStatusDevice;
        int indep[kBW], kb = 0;
        for (int c = 0; c < ka; ++c)
            if (!hmap[2 * kBW + c]) indep[kb++] = c;
        double hS[kPan] = {};
        for (int q = 0; q < kb; ++q)
            for (int c = 0; c < ka; ++c) hS[q * kBW + c] = hR[indep[q] * kBW + c];
        double r0a[kBW] = {};
        for (int c = 0; c < ka; ++c) r0a[c] = rho0[act[c]];
        if (hipMemcpyAsync(w->S, hS, sizeof(hS), hipMemcpyHostToDevice, st) != hipSuccess ||
            hipMemcpyAsync(w->ls.rho0, r0a, sizeof(r0a), hipMemcpyHostToDevice, st) != hipSuccess)
            return kStatusDevice;
        if (kb < ka) {
            int cmap[kBW];
            for (int c = 0; c < kBW; ++c) cmap[c] = c < kb ? indep[c] : -1;
            if (hipMemcpyAsync(w->imap, cmap, kBW * sizeof(int), hipMemcpyHostToDevice, st) != hipSuccess)
                return kStatusDevice;
            k_bselect<<<gpe, kWG, 0, st>>>(w->n, w->pw, w->imap, w->V());
        }
        // flag[0]: breakdown / convergence bits, flag[1]: the cycle has
        // ended (gate of its later kernels), flag[2]: steps done.  The
        // cycle's steps are enqueued without waiting for the host; the steps
        // after the one that ends the cycle return at once.
        if (hipMemsetAsync(w->flag, 0, 3 * sizeof(int), st) != hipSuccess) return kStatusDevice;
        k_bls_init<<<1, kWG, 0, st>>>(kb, ka, w->S, w->ls);
        ++cycles;
        const int* stop = w->flag + 1;
        const int nst = (int)std::min<int64_t>(m, a.max_steps - steps);
        for (int j = 0; j < nst; ++j) {
            if (a.timer) a.timer->step(j);
            double* Vj = w->V() + (int64_t)j * w->ps;
            double* Vn = w->V() + (int64_t)(j + 1) * w->ps;
            spmm<0>(*w, a, Vj, nullptr, w->W(), nullptr, stop);
            project(*w, a, w->W(), stop);   // W = P A V_j
            // BCGS2: two projections onto V_0..V_j; the first also gives the
            // squared column norms of A V_j (the breakdown reference).
            dots(*w, a.timer, st, w->V(), j + 1, w->W(), 1, w->Csum, j + 1, 1, j + 1, w->nb2, stop);
            if (j + 1 <= kFuseMax) {
                // First projection and second dot pass in one sweep.
                gemm_dots(*w, a.timer, st, w->V(), j + 1, w->W(), w->Csum, j + 1, stop);
            } else {
                gemm(*w, a.timer, st, w->V(), j + 1, w->C, w->W(), -1.0, w->W(), stop);
                dots(*w, a.timer, st, w->V(), j + 1, w->W(), 0, w->Csum, j + 1, 0, -1, nullptr, stop);
            }
            // Second projection; its sweep also forms W^T W for the CholQR.
            gemm_gram(*w, a.timer, st, w->V(), j + 1, w->C, w->W(), -1.0, w->W(), stop);
            cholqr2(*w, a.timer, st, kb, w->W(), Vn, 1, w->nb2, stop, true);
            k_bls<<<1, kWG, 0, st>>>(j, kb, ka, a.rtol, w->Csum, w->R, w->ls, w->flag);
        }
        double est[kBW];
        int hf[3] = {0, 0, 0};
        if (hipMemcpyAsync(est, w->ls.est, sizeof(est), hipMemcpyDeviceToHost, st) != hipSuccess ||
            hipMemcpyAsync(hf, w->flag, sizeof(hf), hipMemcpyDeviceToHost, st) != hipSuccess ||
            hipStreamSynchronize(st) != hipSuccess)
            return kStatusDevice;
        const int jd = hf[2];
        steps += jd;
        if (a.timer) a.timer->cycle_done(jd);
        est_max = 0.0;
        for (int c = 0; c < ka; ++c) est_max = std::max(est_max, est[c] / r0a[c]);
        // X[:, act] += V Y (through the free W panel).
        k_bsolve<<<1, kWG, 0, st>>>(jd, kb, ka, w->ls, w->Cy);
        gemm(*w, a.timer, st, w->V(), jd, w->Cy, nullptr, 1.0, w->W(), nullptr);
        k_bscatter<<<gpe, kWG, 0, st>>>(w->n, w->pw, ka, w->imap + kBW, w->W(), w->Xp());
        if ((s = residual(*w, a, raw, rn)) != kStatusOk) return s;
        for (int c = 0; c < k; ++c)
            if (!std::isfinite(rn[c])) return kStatusNonFinite;
    }
    if (a.R > 0) {
        // x_c = x_hat_c + Z E^{-1} Z^T (b_c - A x_hat_c) (eq. precond2); the
        // true residuals are then recomputed.
        spmm<1>(*w, a, w->Xp(), w->Bp(), w->W(), w->npart, nullptr);
        coarse(*w, a, w->W(), nullptr);
        zapply(*w, st, a.R, a.zrp, a.zci, a.zv, 1.0, w->Xp(), nullptr);
        if ((s = residual(*w, a, raw, rn)) != kStatusOk) return s;
        for (int c = 0; c < k; ++c) rn[c] = raw[c];
    }
    const int64_t ue = w->n * k;
    k_bunpack<<<(unsigned)((ue + kWG - 1) / kWG), kWG, 0, st>>>(w->n, k, w->pw, w->Xp(), a.X);
    if (hipStreamSynchronize(st) != hipSuccess) return kStatusDevice;
    double tr = 0.0;
    for (int c = 0; c < k; ++c) tr = std::max(tr, rn[c] / rho0[c]);
    res->steps = steps;
    res->cycles = cycles;
    res->status = status;
    res->rel_res_est = est_max;
    res->rel_res_true = tr;
    return kStatusOk;
}

GM_DEBUG_ACCESSOR(dbg_take_block)

}  // namespace gm
