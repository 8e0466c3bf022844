// FP64 solve and update kernels: gauge fix and Levenberg-Marquardt damping, blocked
// Cholesky factorisation of the dense 6N x 6N system, the two triangular solves, the
// pose update X <- X exp(dx) (Supplementary: exp(dx) = [R(dq), dt], R(dq) the rotation
// of the unit quaternion with imaginary part dq) and the device-side accept/reject of a
// step, so that a whole iteration runs without returning to the host.

#include "pba_internal.h"

#include <algorithm>
#include <cstdlib>

namespace pba {

constexpr int NB = 64;   // Cholesky block size

// A = gauge-fixed H with Marquardt damping, rhs = -b (anchor rows zero); also clears the failure flag.
// lam_override >= 0 replaces the device-side lambda (direct solve calls).
__global__ void damp_copy_kernel(const double *__restrict__ H, const double *__restrict__ b,
                                 double *__restrict__ A, double *__restrict__ rhs, int n, int anchor,
                                 const LmState *lm, double lam_override, int32_t *fail, Stamp stamp)
{
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        put_stamp(stamp, 2);
        *fail = 0;
    }
    const double lam = lam_override >= 0.0 ? lam_override : lm->lam;
    const int a0 = 6 * anchor, a1 = a0 + 6;
    const int64_t nn = (int64_t)n * n;
    for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < nn; e += (int64_t)gridDim.x * blockDim.x) {
        const int i = (int)(e / n), j = (int)(e - (int64_t)i * n);
        const bool ai = i >= a0 && i < a1, aj = j >= a0 && j < a1;
        double v = H[e];
        if (ai || aj) v = (i == j) ? 1.0 : 0.0;
        if (i == j) v += lam * v;
        A[e] = v;
        if (j == 0) rhs[i] = ai ? 0.0 : -b[i];
    }
}

// The same system in a nested-dissection order: factor row R holds row perm[R] of the 6 NP system
// (perm[R] < 0: padding, a unit diagonal and no coupling).  Only the lower tiles of the factor's
// pattern are written (one workgroup per tile, dtiles), the diagonal tiles in full; rhs is the
// permuted -b.  Also clears the failure flag ahead of the level launches.
__global__ void __launch_bounds__(256) damp_copy_perm_kernel(const double *__restrict__ H,
                                                             const double *__restrict__ b, double *__restrict__ A,
                                                             double *__restrict__ rhs, int n0, int n,
                                                             const int32_t *__restrict__ perm,
                                                             const int32_t *__restrict__ dtiles, int anchor,
                                                             const LmState *lm, double lam_override, int32_t *fail,
                                                             Stamp stamp)
{
    if (blockIdx.x == 0 && threadIdx.x == 0) put_stamp(stamp, 2);
    const double lam = lam_override >= 0.0 ? lam_override : lm->lam;
    const int a0 = 6 * anchor, a1 = a0 + 6;
    const int ti = dtiles[2 * blockIdx.x], tj = dtiles[2 * blockIdx.x + 1];
    const int C = tj * NB + (threadIdx.x & 63), oc = perm[C];
    const bool ac = oc >= a0 && oc < a1;
    for (int r = threadIdx.x >> 6; r < NB; r += 4) {
        const int R = ti * NB + r, orow = perm[R];
        const bool ar = orow >= a0 && orow < a1;
        double v = (orow >= 0 && oc >= 0) ? H[(int64_t)orow * n0 + oc] : 0.0;
        if (orow < 0 || oc < 0 || ar || ac) v = (R == C) ? 1.0 : 0.0;
        if (R == C) v += lam * v;
        A[(int64_t)R * n + C] = v;
    }
    if (ti == tj && threadIdx.x < NB) {
        const int R = ti * NB + threadIdx.x, o = perm[R];
        rhs[R] = (o < 0 || (o >= a0 && o < a1)) ? 0.0 : -b[o];
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) *fail = 0;
}

void launch_damp_copy_perm(const double *H, const double *b, double *A, double *rhs, int n0, int anchor,
                           const LmState *lm, double lam_override, const CholPlan &plan, int32_t *fail,
                           const Stamp &stamp, hipStream_t st)
{
    hipLaunchKernelGGL(damp_copy_perm_kernel, dim3(plan.ndt), dim3(256), 0, st, H, b, A, rhs, n0, plan.n, plan.perm,
                       plan.dtiles, anchor, lm, lam_override, fail, stamp);
}

void launch_damp_copy(const double *H, const double *b, double *A, double *rhs, int n, int anchor,
                      const LmState *lm, double lam_override, int32_t *fail, const Stamp &stamp, hipStream_t st)
{
    int64_t nn = (int64_t)n * n;
    int64_t blocks = (nn + 255) / 256;
    if (blocks > 8192) blocks = 8192;
    hipLaunchKernelGGL(damp_copy_kernel, dim3((unsigned)blocks), dim3(256), 0, st, H, b, A, rhs, n, anchor, lm,
                       lam_override, fail, stamp);
}

// ---- blocked right-looking Cholesky, lower triangle, A row-major n x n, 64-wide block columns.
// The columns of one level of the elimination tree of block columns go together, in two launches: one forms the
// factor's panels X_ak = A_ak W_k^T, W_k = L_kk^-1 (a workgroup per panel tile, each factoring its column's
// diagonal block for itself), the next subtracts X_a X_b^T from the tiles right of them.  A itself keeps the
// panels' input; the panels go to L and, transposed, to LT, the inverted diagonal blocks to Winv for the solves.
// 64-wide products run on the FP64 matrix cores.

typedef double d4 __attribute__((ext_vector_type(4)));

// 1/sqrt(d) in FP64 to about an ulp: the hardware estimate refined by two Newton steps.
__device__ __forceinline__ double rsqrt_f64(double d)
{
    double y = __builtin_amdgcn_rsq(d);
    y = y * fma(-0.5 * d * y, y, 1.5);
    return y * fma(-0.5 * d * y, y, 1.5);
}

// x of lane K of each 16-lane row, in every lane of the row (one 64-bit DPP move).
template <int K>
__device__ __forceinline__ double row_bcast(double x)
{
    return __builtin_amdgcn_update_dpp(0.0, x, 0x150 + K, 0xF, 0xF, true);
}

// c += P Q over 16 k-steps-of-four: operand lane l holds P[l % 16][4 s + l / 16] and Q[4 s + l / 16][l % 16]; element
// c[r] of lane l is row 4 r + l / 16, column l % 16.
__device__ __forceinline__ d4 mma(double p, double q, d4 c) { return __builtin_amdgcn_mfma_f64_16x16x4f64(p, q, c, 0, 0, 0); }

// x += (x of lane K of the 16-lane row) * g, one instruction.  The DPP operand must not have been written by the two
// vector instructions before (the leading s_nop), nor may the two after read the result by DPP.
template <int K>
__device__ __forceinline__ void fmac_bcast(double &x, double g)
{
    asm volatile("s_nop 1\n\tv_fmac_f64_dpp %0, %0, %1 row_newbcast:%2 row_mask:0xf bank_mask:0xf\n\ts_nop 1" : "+v"(x) : "v"(g), "n"(K));
}
// The same for seven values.
template <int K>
__device__ __forceinline__ void fmac_bcast(double &x0, double &x1, double &x2, double &x3, double &x4, double &x5, double &x6, double g)
{
    asm volatile("s_nop 1\n\t"
                 "v_fmac_f64_dpp %0, %0, %7 row_newbcast:%8 row_mask:0xf bank_mask:0xf\n\t"
                 "v_fmac_f64_dpp %1, %1, %7 row_newbcast:%8 row_mask:0xf bank_mask:0xf\n\t"
                 "v_fmac_f64_dpp %2, %2, %7 row_newbcast:%8 row_mask:0xf bank_mask:0xf\n\t"
                 "v_fmac_f64_dpp %3, %3, %7 row_newbcast:%8 row_mask:0xf bank_mask:0xf\n\t"
                 "v_fmac_f64_dpp %4, %4, %7 row_newbcast:%8 row_mask:0xf bank_mask:0xf\n\t"
                 "v_fmac_f64_dpp %5, %5, %7 row_newbcast:%8 row_mask:0xf bank_mask:0xf\n\t"
                 "v_fmac_f64_dpp %6, %6, %7 row_newbcast:%8 row_mask:0xf bank_mask:0xf\n\t"
                 "s_nop 1"
                 : "+v"(x0), "+v"(x1), "+v"(x2), "+v"(x3), "+v"(x4), "+v"(x5), "+v"(x6) : "v"(g), "n"(K));
}

// Pivots K .. 15 of the 16 x 16 factor-and-invert below.  The next pivot's column is updated first and its
// reciprocal started before the other 14, so the chain from pivot to pivot overlaps them.
template <int K>
__device__ __forceinline__ void pivots16(double (&a)[16], int r, double p, double q, double &pown, bool &bad)
{
    const bool ok = p > 0.0;
    bad = bad || !ok;
    q = fma(q, fma(-p, q, 1.0), q);
    q = fma(q, fma(-p, q, 1.0), q);
    const bool below = r > K;
    const double g = below && ok ? -a[K] * q : 0.0;
    pown = r == K && ok ? p : pown;
    // (a[K] itself becomes g below the pivot; its old value is not needed any more)
#define PBA_COL(d) a[(K + d) & 15]
    fmac_bcast<K>(PBA_COL(1), g);
    double pn = 1.0, qn = 1.0;
    if constexpr (K < 15) {
        pn = row_bcast<K + 1>(a[K + 1]);
        qn = __builtin_amdgcn_rcp(pn);
        __builtin_amdgcn_sched_barrier(0);
    }
    fmac_bcast<K>(PBA_COL(2), PBA_COL(3), PBA_COL(4), PBA_COL(5), PBA_COL(6), PBA_COL(7), PBA_COL(8), g);
    fmac_bcast<K>(PBA_COL(9), PBA_COL(10), PBA_COL(11), PBA_COL(12), PBA_COL(13), PBA_COL(14), PBA_COL(15), g);
#undef PBA_COL
    a[K] = below ? g : a[K];
    if constexpr (K < 15) pivots16<K + 1>(a, r, pn, qn, pown, bad);
}

constexpr int kLd = NB + 1;   // LDS row pitch of a 64-wide tile (odd: rows 16 apart fall in distinct banks)
struct FactorLds {
    double X[NB - 16][17];    // the block column's factor below the diagonal block
    double Wd[16][17];        // the diagonal block's inverse factor
};

// W = L^-1 for the 64 x 64 symmetric matrix M = L L^T, in place in M's lower triangle (strictly upper 16 x 16
// blocks are left as they are; the upper part of the diagonal ones becomes zero).  Only M's lower blocks and the
// whole of its diagonal 16 x 16 blocks are read.  256 threads; false where a pivot is not positive.
//
// Block Gauss-Jordan over four 16-wide block columns.  Every wave factors and inverts the diagonal block for
// itself: lane l holds row l % 16 (the four 16-lane rows alike), pivot k subtracts row k times c_i / p from the
// rows below, where columns right of k are the remaining matrix and columns left of it already rows of the inverse
// (column k itself becomes the new one, -c_i / p), so one update of 15 values serves both; a pivot row's
// values reach the lanes by DPP, no LDS, no barrier.  W's rows are those, scaled by 1 / sqrt(p_i).  Then each wave
// forms one block: X_w = M_w,k W_k^T below, R_w = W_k M_k,w left of the diagonal; and the blocks below take
// M_it -= X_i X_t^T (t > k), M_it -= X_i R_t (t < k), M_ik = -X_i W_k; two barriers per block column.  A latency
// chain: 16 pivots take 3300 cycles (the reciprocal and its refinement, 200 each), a block column's products 2200 on
// average; 10.7 us a tile, and about 5 more while the launch's instructions come from memory.  64 single pivots
// exchanged through LDS took 700 cycles each (20 us); a DPP move and an FMA per value 450 (the move's latency).
__device__ __forceinline__ bool factor64(double (*M)[kLd], FactorLds &F)
{
    const int l = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int r = l & 15, q = l >> 4;
    bool bad = false;
#pragma unroll 1
    for (int kb = 0; kb < 4; ++kb) {
        const int d0 = 16 * kb;
        double a[16], pown = 1.0, m[4];
#pragma unroll
        for (int j = 0; j < 16; ++j) a[j] = M[d0 + r][d0 + j];
        // the wave's own block of phase 1 (M_w,k below the diagonal block, M_k,w left of it), ahead of the pivots
        {
            const double *mb = w > kb ? &M[16 * w + r][d0 + q] : &M[d0 + q][16 * w + r];
            const int step = w > kb ? 4 : 4 * kLd;
#pragma unroll
            for (int s = 0; s < 4; ++s) m[s] = mb[s * step];
        }
        const double p0 = row_bcast<0>(a[0]);
        pivots16<0>(a, r, p0, __builtin_amdgcn_rcp(p0), pown, bad);
        const double rs = rsqrt_f64(pown);
        // W_k's rows before scaling as an operand: row l % 16, columns 4 s + l / 16
        double v[4];
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const double t = q < 2 ? (q == 0 ? a[4 * s] : a[4 * s + 1]) : (q == 2 ? a[4 * s + 2] : a[4 * s + 3]);
            v[s] = 4 * s + q < r ? t : (4 * s + q == r ? 1.0 : 0.0);
        }
        d4 c = {0.0, 0.0, 0.0, 0.0};
        if (w > kb) {   // X's column l % 16 is scaled by that row's factor, which this lane has
#pragma unroll
            for (int s = 0; s < 4; ++s) c = mma(m[s], v[s], c);
#pragma unroll
            for (int e = 0; e < 4; ++e) F.X[16 * (w - kb - 1) + 4 * e + q][r] = c[e] * rs;
        } else if (w < kb) {
#pragma unroll
            for (int s = 0; s < 4; ++s) c = mma(v[s] * rs, m[s], c);
#pragma unroll
            for (int e = 0; e < 4; ++e) M[d0 + 4 * e + q][16 * w + r] = c[e];
        } else {
#pragma unroll
            for (int s = 0; s < 4; ++s) F.Wd[r][4 * s + q] = v[s] * rs;
        }
        __syncthreads();
        // phase 2: block b of the list (i, t), i = kb + 1 .. 3, t = 0 .. i, to wave b % 4; the operands of a wave's
        // next block are read while one is multiplied
        const int nb2 = kb == 0 ? 9 : kb == 1 ? 7 : kb == 2 ? 4 : 0;
        auto locate = [&](int b, int &i, int &t) {
            i = kb + 1;
            while (b > i) { b -= i + 1; ++i; }
            t = b;
        };
        struct Ops { d4 v; double x[4], y[4]; };
        auto read = [&](int b, Ops &o) {
            int i, t;
            locate(b, i, t);
            const double *xb = &F.X[16 * (i - kb - 1) + r][q];
            const double *yb = t > kb ? &F.X[16 * (t - kb - 1) + r][q] : t == kb ? &F.Wd[q][r] : &M[d0 + q][16 * t + r];
            const int ys = t > kb ? 4 : t == kb ? 4 * 17 : 4 * kLd;
#pragma unroll
            for (int s = 0; s < 4; ++s) { o.x[s] = xb[4 * s]; o.y[s] = yb[s * ys]; }
#pragma unroll
            for (int e = 0; e < 4; ++e) o.v[e] = t == kb ? 0.0 : M[16 * i + 4 * e + q][16 * t + r];
        };
        auto multiply = [&](int b, Ops &o) {
            int i, t;
            locate(b, i, t);
#pragma unroll
            for (int s = 0; s < 4; ++s) o.v = mma(-o.x[s], o.y[s], o.v);
#pragma unroll
            for (int e = 0; e < 4; ++e) M[16 * i + 4 * e + q][16 * t + r] = o.v[e];
        };
        if (w < nb2) {
            Ops o0, o1;
            read(w, o0);
            if (w + 4 < nb2) read(w + 4, o1);
            multiply(w, o0);
            if (w + 8 < nb2) read(w + 8, o0);
            if (w + 4 < nb2) multiply(w + 4, o1);
            if (w + 8 < nb2) multiply(w + 8, o0);
        }
        if (w == kb)   // W_k in its place
#pragma unroll
            for (int s = 0; s < 4; ++s) M[d0 + r][d0 + 4 * s + q] = v[s] * rs;
        __syncthreads();
    }
    return !bad;
}

// The diagonal tile at k0 (nb rows) into M, its upper part mirrored from the lower (which alone is kept up to date),
// padded with the identity.
__device__ __forceinline__ void load_diag(double (*M)[kLd], const double *A, int64_t n, int k0, int nb)
{
    double v[NB * NB / 256];
#pragma unroll
    for (int it = 0; it < NB * NB / 256; ++it) {
        const int e = it * 256 + (int)threadIdx.x, i = e >> 6, j = e & 63;
        v[it] = (j <= i && i < nb) ? A[(int64_t)(k0 + i) * n + k0 + j] : (i == j ? 1.0 : 0.0);
    }
#pragma unroll
    for (int it = 0; it < NB * NB / 256; ++it) {
        const int e = it * 256 + (int)threadIdx.x, i = e >> 6, j = e & 63;
        if (j <= i) { M[i][j] = v[it]; M[j][i] = v[it]; }
    }
}

// Panels of one level: workgroup = entry (k, a) of `panels`, column k's diagonal block and its tile row a (a < 0: a
// column without rows below).  Every workgroup of a column factors the diagonal block for itself (bitwise alike),
// so no workgroup waits for another; the column's first one writes W and W^T and, with x, the forward
// substitution's y_k = W r_k (x_k holds r_k, from which every earlier column's part has been subtracted).
// Latency-bound: 21 us a launch, of which the factor takes 16 and the panel's products 2 (lidar64's eight levels:
// diagonal blocks 24 us and updates that formed the panels from LDS 14 to 53 us; now 21 and 5 to 11).
__global__ void __launch_bounds__(256) chol_panel_kernel(const double *__restrict__ A, double *__restrict__ L,
                                                         double *__restrict__ LT, int n,
                                                         const int2 *__restrict__ panels, double *__restrict__ Winv,
                                                         int32_t *fail, double *x)
{
    __shared__ double M[NB][kLd], T[NB][kLd];
    __shared__ FactorLds F;
    // (no early return on a failure: this launch sets the flag itself, so its waves could disagree)
    const int2 ka = panels[blockIdx.x];
    const bool first = blockIdx.x == 0 || panels[(int)blockIdx.x - 1].x != ka.x;
    const int k0 = ka.x * NB, ra = ka.y * NB, nb = min(NB, n - k0), tid = threadIdx.x;
    const int l = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6), r = l & 15, q = l >> 4;
    // the panel tile's input is fetched ahead of the factorisation (its columns are whole: only the last block
    // column can be ragged, and that has no rows below)
    double2 t[NB * NB / 512];
#pragma unroll
    for (int it = 0; it < NB * NB / 512; ++it) {
        const int e = it * 256 + tid, i = e >> 5, j = (e & 31) * 2;
        t[it] = ka.y >= 0 && ra + i < n ? *reinterpret_cast<const double2 *>(A + (int64_t)(ra + i) * n + k0 + j)
                                        : make_double2(0.0, 0.0);
    }
    load_diag(M, A, n, k0, nb);
    __syncthreads();
    if (!factor64(M, F) && first && tid == 0) *fail = 1;
    if (first) {
        double *Wb = Winv + (int64_t)ka.x * NB * NB, *Wtb = Wb + (int64_t)((n + NB - 1) / NB) * NB * NB;
#pragma unroll
        for (int it = 0; it < NB * NB / 256; ++it) {
            const int e = it * 256 + tid, i = e >> 6, j = e & 63;
            Wb[e] = j <= i && i < nb ? M[i][j] : 0.0;
            Wtb[e] = i <= j && j < nb ? M[j][i] : 0.0;
        }
        if (x) {   // rows i = tid / 4, columns 16 (tid % 4) .. +15
            const int i = tid >> 2, j0 = (tid & 3) * 16;
            double y = 0.0;
#pragma unroll
            for (int j = 0; j < 16; ++j)
                if (j0 + j <= i) y = fma(M[i][j0 + j], x[k0 + j0 + j], y);
            y += __shfl_xor(y, 1, 64);
            y += __shfl_xor(y, 2, 64);
            __syncthreads();   // every r_k read (x has whole blocks)
            if ((tid & 3) == 0) x[k0 + i] = y;
        }
    }
    if (ka.y < 0) return;   // uniform over the workgroup
#pragma unroll
    for (int it = 0; it < NB * NB / 512; ++it) {
        const int e = it * 256 + tid, i = e >> 5, j = (e & 31) * 2;
        T[i][j] = t[it].x;
        T[i][j + 1] = t[it].y;
    }
    __syncthreads();
    // X = A_ak W^T: wave w rows 16 w .. +15 (it alone reads and writes them); W is lower triangular
    double p[16];
#pragma unroll
    for (int s = 0; s < 16; ++s) p[s] = T[16 * w + r][4 * s + q];
#pragma unroll
    for (int jb = 0; jb < 4; ++jb) {
        d4 c = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int s = 0; s < 4 * (jb + 1); ++s) c = mma(p[s], M[16 * jb + r][4 * s + q], c);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int i = 16 * w + 4 * e + q, j = 16 * jb + r;
            T[i][j] = c[e];
            if (ra + i < n) L[(int64_t)(ra + i) * n + k0 + j] = c[e];
        }
    }
    __syncthreads();
#pragma unroll
    for (int it = 0; it < NB * NB / 256; ++it) {   // L^T, read back column-wise so the stores run along its rows
        const int e = it * 256 + tid, j = e >> 6, i = e & 63;
        if (ra + i < n) LT[(int64_t)(k0 + j) * n + ra + i] = T[i][j];
    }
}

// Updates of one level after its panels: every block column k of the level contributes A_ab -= X_a X_b^T to the
// tiles (a, b), b <= a, of its tile rows.  They belong to higher levels, so nothing this level reads is written.  One
// task per target tile lists its contributing columns (ascending); workgroup (task, qi, qj) owns one 32 x 32
// quarter, a 16 x 16 block of it per wave, and sums the contributions in that order before subtracting them, so
// the result does not depend on the schedule.  The next contributor's rows are fetched while one is multiplied.
// With x, the diagonal targets' workgroups with qj = 0 subtract L_ak y_k from their rows of x (the forward
// substitution; y_k was written by this level's panels, and only this task writes those rows).
__global__ void __launch_bounds__(256) chol_update_kernel(double *A, const double *__restrict__ L, int n,
                                                          const int32_t *__restrict__ tasks,
                                                          const int32_t *__restrict__ contrib, const int32_t *fail,
                                                          double *x)
{
    constexpr int H = NB / 2, kIt = H * NB / 512;
    __shared__ double Xi[H][kLd], Xj[H][kLd];
    if (*fail) return;
    const int4 tk = reinterpret_cast<const int4 *>(tasks)[blockIdx.x >> 2];
    const int qi = (blockIdx.x >> 1) & 1, qj = blockIdx.x & 1;
    const bool diag = tk.x == tk.y;
    const int ri = tk.x * NB + H * qi, rj = tk.y * NB + H * qj;
    if ((diag && qj > qi) || ri >= n) return;   // uniform over the workgroup
    const bool fwd = diag && qj == 0 && x;
    const int tid = threadIdx.x, l = tid & 63, w = tid >> 6, r = l & 15, q = l >> 4;
    const int bi = 16 * (w >> 1), bj = 16 * (w & 1);
    double2 ti[kIt], tj[kIt];
    auto fetch = [&](int e) {
        const int k0 = contrib[tk.z + e] * NB;
#pragma unroll
        for (int it = 0; it < kIt; ++it) {
            const int o = it * 256 + tid, i = o >> 5, k = (o & 31) * 2;
            ti[it] = ri + i < n ? *reinterpret_cast<const double2 *>(L + (int64_t)(ri + i) * n + k0 + k) : make_double2(0.0, 0.0);
            tj[it] = rj + i < n ? *reinterpret_cast<const double2 *>(L + (int64_t)(rj + i) * n + k0 + k) : make_double2(0.0, 0.0);
        }
    };
    d4 c = {0.0, 0.0, 0.0, 0.0};
    double z = 0.0;   // fwd: sum over the contributors of L_ak y_k, row tid / 8 of the quarter
    fetch(0);
    for (int e = 0; e < tk.w; ++e) {
#pragma unroll
        for (int it = 0; it < kIt; ++it) {
            const int o = it * 256 + tid, i = o >> 5, k = (o & 31) * 2;
            Xi[i][k] = ti[it].x; Xi[i][k + 1] = ti[it].y;
            Xj[i][k] = tj[it].x; Xj[i][k + 1] = tj[it].y;
        }
        if (e + 1 < tk.w) fetch(e + 1);
        __syncthreads();
#pragma unroll
        for (int s = 0; s < 16; ++s) c = mma(Xi[bi + r][4 * s + q], Xj[bj + r][4 * s + q], c);
        if (fwd) {
            const int i = tid >> 3, j0 = (tid & 7) * 8, k0 = contrib[tk.z + e] * NB;   // 8 lanes per row, 8 columns each
#pragma unroll
            for (int j = 0; j < 8; ++j) z = fma(Xi[i][j0 + j], x[k0 + j0 + j], z);
        }
        __syncthreads();
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int i = bi + 4 * e + q, j = bj + r;
        if (ri + i < n && rj + j < n && (!diag || H * qj + j <= H * qi + i)) A[(int64_t)(ri + i) * n + rj + j] -= c[e];
    }
    if (fwd) {
        z += __shfl_xor(z, 1, 64);
        z += __shfl_xor(z, 2, 64);
        z += __shfl_xor(z, 4, 64);
        if ((tid & 7) == 0) x[ri + (tid >> 3)] -= z;
    }
}

void launch_cholesky(double *A, double *L, double *LT, int n, double *Winv, const CholPlan &plan, int32_t *fail,
                     hipStream_t st, double *x)
{
    for (size_t s = 0; s < plan.pcnt.size(); ++s) {
        hipLaunchKernelGGL(chol_panel_kernel, dim3(plan.pcnt[s]), dim3(256), 0, st, A, L, LT, n,
                           reinterpret_cast<const int2 *>(plan.panels) + plan.pbeg[s], Winv, fail, plan.nd ? x : nullptr);
        if (plan.tcnt[s] > 0)
            hipLaunchKernelGGL(chol_update_kernel, dim3(4 * plan.tcnt[s]), dim3(256), 0, st, A, L, n,
                               plan.tasks + 4 * (int64_t)plan.tbeg[s], plan.contrib, fail, plan.nd ? x : nullptr);
    }
}

// A system of one block (n <= 64): damping and gauge, factorisation and both triangular solves in one launch of
// one workgroup (three launches, 33 us, before; 17 us so).  x receives the step, zero if the factorisation failed.
__global__ void __launch_bounds__(256) solve_small_kernel(const double *__restrict__ H, const double *__restrict__ b,
                                                          int n, int anchor, const LmState *lm, double lam_override,
                                                          double *__restrict__ x, int32_t *fail, Stamp stamp)
{
    __shared__ double M[NB][kLd];
    __shared__ FactorLds F;
    __shared__ double v[NB], y[NB];
    const int tid = threadIdx.x;
    if (tid == 0) put_stamp(stamp, 2);
    const double lam = lam_override >= 0.0 ? lam_override : lm->lam;
    const int a0 = 6 * anchor, a1 = a0 + 6;
#pragma unroll 4
    for (int it = 0; it < NB * NB / 256; ++it) {
        const int e = it * 256 + tid, i = e >> 6, j = e & 63;
        const bool fixed = (i >= a0 && i < a1) || (j >= a0 && j < a1);
        double h = i == j ? 1.0 : 0.0;
        if (i < n && j < n && !fixed) h = H[(int64_t)i * n + j];
        if (i == j && i < n) h += lam * h;
        M[i][j] = h;
    }
    if (tid < NB) v[tid] = (tid < n && !(tid >= a0 && tid < a1)) ? -b[tid] : 0.0;
    __syncthreads();
    const bool ok = factor64(M, F);
    // y = W v, x = W^T y: four lanes to a row, 16 columns each
    const int i = tid >> 2, j0 = (tid & 3) * 16;
    double u = 0.0;
#pragma unroll
    for (int j = 0; j < 16; ++j)
        if (j0 + j <= i) u = fma(M[i][j0 + j], v[j0 + j], u);
    u += __shfl_xor(u, 1, 64);
    u += __shfl_xor(u, 2, 64);
    if ((tid & 3) == 0) y[i] = u;
    __syncthreads();
    u = 0.0;
#pragma unroll
    for (int j = 0; j < 16; ++j)
        if (j0 + j >= i) u = fma(M[j0 + j][i], y[j0 + j], u);
    u += __shfl_xor(u, 1, 64);
    u += __shfl_xor(u, 2, 64);
    if ((tid & 3) == 0 && i < n) x[i] = ok ? u : 0.0;
    if (tid == 0) *fail = ok ? 0 : 1;
}

void launch_solve_small(const double *H, const double *b, int n, int anchor, const LmState *lm, double lam_override,
                        double *x, int32_t *fail, const Stamp &stamp, hipStream_t st)
{
    hipLaunchKernelGGL(solve_small_kernel, dim3(1), dim3(256), 0, st, H, b, n, anchor, lm, lam_override, x, fail, stamp);
}

// L y = rhs, then L^T x = y, both in one launch of one 1024-thread workgroup that walks the
// block columns forward and then backward: the factor couples each block to a few tiles, so a
// block step is a few thousand FMAs and a launch per step would cost more than the step.  The
// vector being solved for sits in LDS when it fits (kTrsvLds doubles), else in x itself; it holds
// the right-hand side, then y block by block, then the solution (x is zeroed instead if the
// factorisation failed).  The two sweeps are the same
// loop: block k takes u_k = M_k v_k in place of v_k, then v_i -= F_ik u_k for the tiles i listed
// for k, with M = W_kk, F = L (tile rows below k) forward and M = W_kk^T, F = L^T (tile columns
// left of k, read as rows of L^T) backward, so every product runs along rows: 16 lanes per row,
// 4 columns each, summed within the lanes' row by DPP.  The next step's M_k and first kTrsvPre
// tiles (listed per block, -1 padded, after the plan's counts) are fetched into registers while
// the current step runs: they do not depend on the vector, so only LDS traffic and barriers
// remain on the chain of steps.  A barrier also makes global writes before it visible to the
// whole workgroup.
constexpr int kTrsvLds = 16384;
constexpr int kTrsvPre = kCholPre;
constexpr int kTrsvLpr = 16;   // lanes per row of the products (per solve at n = 1800: 4 -> 393 us, 8 -> 240, 16 -> 192)

// Workgroup barrier that orders LDS accesses only: global loads issued before it stay in flight
// (__syncthreads() also waits for those).
__device__ __forceinline__ void lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Lane permutations without LDS round trips.  DPP row_ror:n rotates each 16-lane row by n.
template <int CTRL>
__device__ __forceinline__ double dpp_f64(double x)
{
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(x), CTRL, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(x), CTRL, 0xF, 0xF, false);
    return __hiloint2double(hi, lo);
}
constexpr int kRowRor8 = 0x128, kRowRor4 = 0x124;

constexpr int kHalfMirror = 0x141, kQuadXor2 = 0x4E, kQuadXor1 = 0xB1;

// Sum over each aligned group of G lanes (16: rotations of the 16-lane row by 8, 4, 2, 1; 8: the
// half-row mirror, which pairs lane i with 7 - i, then quad permutes xor 2 and xor 1; 4: the quad
// permutes), in every lane of the group.  Groups may be active or inactive as a whole.
template <int G>
__device__ __forceinline__ double group_sum(double u)
{
    if constexpr (G == 16) {
        u += dpp_f64<kRowRor8>(u);
        u += dpp_f64<kRowRor4>(u);
    } else if constexpr (G == 8) {
        u += dpp_f64<kHalfMirror>(u);
    }
    u += dpp_f64<kQuadXor2>(u);
    return u + dpp_f64<kQuadXor1>(u);
}

// Two doubles at p (16-byte aligned) if ok, else the two at `safe`, without a branch, so every
// call issues exactly one load and the compiler can count the loads still in flight (a select
// to zero would be placed right after the load and wait for it).  The callers skip a value that
// was not ok, or multiply it by an exact zero, and `safe` holds finite values.
__device__ __forceinline__ void load2_or_safe(const double *p, bool ok, double &a, double &b, const double *safe)
{
    const double2 v = *reinterpret_cast<const double2 *>(ok ? p : safe);
    a = v.x;
    b = v.y;
}

template <bool kInLds, int LPR>
__global__ void __launch_bounds__(64 * LPR) trsv_band_kernel(const double *__restrict__ L,
                                                         const double *__restrict__ LT,
                                                         const double *__restrict__ Winv, double *x, int n,
                                                         const int32_t *__restrict__ rows,
                                                         const int32_t *__restrict__ cols,
                                                         const int32_t *__restrict__ meta, const int32_t *fail)
{
    __shared__ double vs[kInLds ? kTrsvLds : 1];
    __shared__ double vk[NB];
    if (*fail) {   // no factor: the step is zero
        for (int e = threadIdx.x; e < n; e += blockDim.x) x[e] = 0.0;
        return;
    }
    double *v = kInLds ? vs : x;
    // with the vector in LDS the barriers need not wait for the prefetches
    auto sync = [] {
        if constexpr (kInLds) lds_barrier();
        else __syncthreads();
    };
    const int t = threadIdx.x, nblk = (n + NB - 1) / NB;
    const int32_t *rbeg = meta, *rcnt = meta + nblk, *cbeg = meta + 2 * nblk, *ccnt = meta + 3 * nblk;
    const int32_t *rpre = meta + 4 * nblk, *cpre = rpre + kTrsvPre * nblk;   // first tiles, -1 padded
    if (kInLds) {
        for (int e = t; e < n; e += blockDim.x) vs[e] = x[e];
        sync();
    }
    constexpr int CPL = NB / LPR;   // columns per lane
    const int row = t / LPR, c4 = (t % LPR) * CPL;   // thread = (row of the product, CPL columns)
    auto sweep = [&](const double *M, const double *F, const int32_t *pre, const int32_t *beg, const int32_t *cnt,
                     const int32_t *list, bool forward) {
        double wa[CPL], la[kTrsvPre][CPL], wb[CPL], lb[kTrsvPre][CPL];
        auto fetch = [&](int kb, double (&wn)[CPL], double (&ln)[kTrsvPre][CPL]) {
            const int k0 = kb * NB, nb = min(NB, n - k0);
            const double2 *Mr = reinterpret_cast<const double2 *>(M + ((int64_t)kb * NB + row) * NB + c4);
#pragma unroll
            for (int h = 0; h < CPL / 2; ++h) {   // the block is zero-padded
                const double2 m = Mr[h];
                wn[2 * h] = m.x;
                wn[2 * h + 1] = m.y;
            }
#pragma unroll
            for (int e = 0; e < kTrsvPre; ++e) {
                const int tile = pre[kTrsvPre * kb + e];
                const int i = tile >= 0 ? tile * NB + row : n;
#pragma unroll
                for (int h = 0; h < CPL / 2; ++h)   // columns c4 + 2 h, c4 + 2 h + 1 (nb is even)
                    load2_or_safe(F + (int64_t)i * n + k0 + c4 + 2 * h, i < n && c4 + 2 * h < nb, ln[e][2 * h],
                                  ln[e][2 * h + 1], M);
            }
        };
        auto step = [&](int kb, const double (&w)[CPL], const double (&l)[kTrsvPre][CPL]) {
            const int k0 = kb * NB, nb = min(NB, n - k0);
            double u = 0.0;
#pragma unroll
            for (int q = 0; q < CPL; ++q) u = fma(w[q], c4 + q < nb ? v[k0 + c4 + q] : 0.0, u);
            u = group_sum<LPR>(u);   // zero for rows beyond the block (M is zero-padded)
            const bool lead = t % LPR == 0;
            if (lead) vk[row] = u;
            sync();
            if (lead && row < nb) v[k0 + row] = u;
            double vq[CPL];
#pragma unroll
            for (int q = 0; q < CPL; ++q) vq[q] = vk[c4 + q];
#pragma unroll
            for (int e = 0; e < kTrsvPre; ++e) {
                const int tile = pre[kTrsvPre * kb + e];
                const int i = tile >= 0 ? tile * NB + row : n;
                if (i < n) {   // uniform over the row's lanes
                    double z = 0.0;
#pragma unroll
                    for (int q = 0; q < CPL; ++q) z = fma(l[e][q], vq[q], z);
                    z = group_sum<LPR>(z);
                    if (lead) v[i] -= z;
                }
            }
            for (int e = kTrsvPre; e < cnt[kb]; ++e) {
                const int i = list[beg[kb] + e] * NB + row;
                if (i >= n) continue;
                double z = 0.0;
#pragma unroll
                for (int q = 0; q < CPL; ++q)
                    if (c4 + q < nb) z = fma(F[(int64_t)i * n + k0 + c4 + q], vq[q], z);
                z = group_sum<LPR>(z);
                if (lead) v[i] -= z;
            }
            sync();
        };
        // Two steps per pass with the register sets swapped (static indexing keeps them in registers;
        // a copy out of the prefetch set would wait for its loads).  The fetches are unconditional
        // (past the end they repeat the last block), so that the loads in flight are the same on
        // every path and the waits for them can be counted.
        const int first = forward ? 0 : nblk - 1, dir = forward ? 1 : -1;
        auto clampb = [&](int kb) { return min(max(kb, 0), nblk - 1); };
        fetch(first, wa, la);
        for (int s = 0; s < nblk; s += 2) {
            const int kb = first + dir * s;
            fetch(clampb(kb + dir), wb, lb);
            step(kb, wa, la);
            if (s + 1 >= nblk) break;
            fetch(clampb(kb + 2 * dir), wa, la);
            step(kb + dir, wb, lb);
        }
    };
    sweep(Winv, L, rpre, rbeg, rcnt, rows, true);
    sweep(Winv + (int64_t)nblk * NB * NB, LT, cpre, cbeg, ccnt, cols, false);
    if (kInLds)
        for (int e = t; e < n; e += blockDim.x) x[e] = vs[e];
}

// One elimination-tree level of the triangular solves in a nested-dissection order, one workgroup
// per block column k of the level, gathering what the finished levels contribute (the library
// runs the forward sweep with the factorisation instead, and this kernel for the backward one):
//   forward   y_k = W_k (r_k - sum_j L_kj y_j)      over the tile columns j < k of block row k,
//   backward  x_k = W_k^T (y_k - sum_i L_ik^T x_i)  over the tile rows i > k of block column k,
// with F = L (tile (k, j)) or F = L^T (tile (k, i), rows of L^T) and M = W_k or W_k^T.  The tiles
// gathered belong to lower levels (forward) or higher ones (backward), finished by earlier
// launches.  Four lanes per row, 16 columns each; the sums of a row's lanes by quad permutes.
// x is zeroed instead if the factorisation failed.
__global__ void __launch_bounds__(256) trsv_level_kernel(const double *__restrict__ F, const double *__restrict__ M,
                                                         double *x, int n, const int32_t *__restrict__ lcols,
                                                         const int32_t *__restrict__ adj,
                                                         const int32_t *__restrict__ beg,
                                                         const int32_t *__restrict__ cnt, const int32_t *fail)
{
    __shared__ double sv[NB];
    const int kb = lcols[blockIdx.x], k0 = kb * NB;
    const int t = threadIdx.x, row = t >> 2, c16 = (t & 3) * 16;
    const bool lead = (t & 3) == 0;
    if (*fail) {
        if (t < NB) x[k0 + t] = 0.0;
        return;
    }
    double z = 0.0;
    const int b0 = beg[kb], m = cnt[kb];
    for (int e = 0; e < m; ++e) {
        const int j0 = adj[b0 + e] * NB;
        const double2 *Fr = reinterpret_cast<const double2 *>(F + (int64_t)(k0 + row) * n + j0 + c16);
        const double2 *xr = reinterpret_cast<const double2 *>(x + j0 + c16);
#pragma unroll
        for (int h = 0; h < 8; ++h) {
            const double2 f = Fr[h], v = xr[h];
            z = fma(f.x, v.x, z);
            z = fma(f.y, v.y, z);
        }
    }
    z = group_sum<4>(z);
    if (lead) sv[row] = x[k0 + row] - z;
    __syncthreads();
    const double2 *Mr = reinterpret_cast<const double2 *>(M + ((int64_t)kb * NB + row) * NB + c16);
    double u = 0.0;
#pragma unroll
    for (int h = 0; h < 8; ++h) {
        const double2 w = Mr[h];
        u = fma(w.x, sv[c16 + 2 * h], u);
        u = fma(w.y, sv[c16 + 2 * h + 1], u);
    }
    u = group_sum<4>(u);
    if (lead) x[k0 + row] = u;
}

void launch_chol_solve(const double *L, const double *LT, double *Winv, double *x, int n, const CholPlan &plan,
                       const int32_t *fail, hipStream_t st)
{
    if (plan.nd) {   // the forward substitution ran with the factorisation (launch_cholesky with x)
        const int nblk = n / NB, nlev = (int)plan.lcnt.size();
        const int32_t *rbeg = plan.meta, *rcnt = rbeg + nblk;
        for (int l = nlev - 1; l >= 0; --l)
            hipLaunchKernelGGL(trsv_level_kernel, dim3(plan.lcnt[l]), dim3(256), 0, st, LT,
                               Winv + (int64_t)nblk * NB * NB, x, n, plan.lcols + plan.lbeg[l], plan.rows, rbeg,
                               rcnt, fail);
        return;
    }
    // PBA_TRSV_LDS_MAX (doubles, at most kTrsvLds) lowers the size up to which the vector is kept
    // in LDS; 0 selects the global-memory variant for every size.  PBA_TRSV_LPR (4, 8 or 16) sets
    // the lanes per row of the products.
    int lds_max = kTrsvLds, lpr = kTrsvLpr;
    if (const char *e = std::getenv("PBA_TRSV_LDS_MAX")) lds_max = std::min(kTrsvLds, std::max(0, std::atoi(e)));
    if (const char *e = std::getenv("PBA_TRSV_LPR")) lpr = std::atoi(e);
    const bool in_lds = n <= lds_max;
#define PBA_TRSV_LAUNCH(LDS, G)                                                                                 \
    hipLaunchKernelGGL((trsv_band_kernel<LDS, G>), dim3(1), dim3(64 * G), 0, st, L, LT, Winv, x, n, plan.rows, \
                       plan.cols, plan.meta, fail)
    if (lpr == 4) {
        if (in_lds) PBA_TRSV_LAUNCH(true, 4);
        else PBA_TRSV_LAUNCH(false, 4);
    } else if (lpr == 16) {
        if (in_lds) PBA_TRSV_LAUNCH(true, 16);
        else PBA_TRSV_LAUNCH(false, 16);
    } else {
        if (in_lds) PBA_TRSV_LAUNCH(true, 8);
        else PBA_TRSV_LAUNCH(false, 8);
    }
#undef PBA_TRSV_LAUNCH
}

// ---- pose update

// Xo_k = X_k exp(dx_k), one thread per pose (inside an iteration the pair setup applies the step instead).
// off: first element of each pose's 6 in dx (a nested-dissection solve's layout), nullptr = 6 k.
__global__ void __launch_bounds__(128) boxplus_kernel(const double *__restrict__ X, const double *__restrict__ dx,
                                                      const int32_t *__restrict__ off, double *__restrict__ Xo, int N)
{
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= N) return;
    double o[12];
    boxplus_pose(X + 12 * (int64_t)k, dx + (off ? (int64_t)off[k] : 6 * (int64_t)k), o);
    for (int i = 0; i < 12; ++i) Xo[12 * (int64_t)k + i] = o[i];
}

void launch_boxplus(const double *X, const double *dx, const int32_t *off, double *Xout, int N, hipStream_t st)
{
    hipLaunchKernelGGL(boxplus_kernel, dim3((N + 127) / 128), dim3(128), 0, st, X, dx, off, Xout, N);
}

// dst[6 k + i] = src[off[k] + i]: a nested-dissection solve's step in pose order.
__global__ void gather_step_kernel(double *__restrict__ dst, const double *__restrict__ src,
                                   const int32_t *__restrict__ off, int N)
{
    for (int e = blockIdx.x * blockDim.x + threadIdx.x; e < 6 * N; e += gridDim.x * blockDim.x)
        dst[e] = src[off[e / 6] + e % 6];
}

void launch_gather_step(double *dst, const double *src, const int32_t *off, int N, hipStream_t st)
{
    const int blocks = std::max(1, std::min(1024, (6 * N + 255) / 256));
    hipLaunchKernelGGL(gather_step_kernel, dim3(blocks), dim3(256), 0, st, dst, src, off, N);
}

// Take or leave the candidate, as the assembly decided (lm->accepted: Gauss-Newton, use_lm = 0, takes every
// solved step; LM takes it if F decreases): the candidate's blocks of H, its gradient and poses become current,
// and the first thread updates the scalars (nothing that another thread reads) and writes the log row {F,
// lambda, step_norm, valid, accepted, failed} and the iteration's end stamp.  Only the nonzero blocks of H move
// (blk_rc): at n = 3600 the dense matrix took 29 us.
__global__ void __launch_bounds__(256) lm_decide_kernel(LmState *lm, const double *__restrict__ totals_cand,
                                                        double *totals_cur, const int2 *__restrict__ blk_rc, int nblk,
                                                        double *H_cur, const double *__restrict__ H_cand, double *b_cur,
                                                        const double *__restrict__ b_cand, double *X_cur,
                                                        const double *__restrict__ X_cand, int N, double *logbuf,
                                                        int log_cap)
{
    const bool accept = lm->accepted != 0;
    const int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x, nH = 36 * (int64_t)nblk;
    if (accept) {
        if (e < nH) {
            const int2 rc = blk_rc[e / 36];
            const int i = (int)(e % 36) / 6, j = (int)(e % 6);
            const int64_t at = (int64_t)(6 * rc.x + i) * (6 * N) + 6 * rc.y + j;
            H_cur[at] = H_cand[at];
        } else if (e < nH + 6 * N) {
            b_cur[e - nH] = b_cand[e - nH];
        } else if (e < nH + 18 * (int64_t)N) {
            X_cur[e - nH - 6 * N] = X_cand[e - nH - 6 * N];
        }
    }
    if (e != 0) return;
    // the row is chosen on the device so that every iteration launches identical arguments
    double *log_row = logbuf + kLogRow * (int64_t)min(lm->iter, log_cap - 1);
    const bool solved = !lm->fail;
    if (accept) {
        for (int k = 0; k < 4; ++k) totals_cur[k] = totals_cand[k];
        lm->F_cur = totals_cand[0];
        lm->valid_cur = (int64_t)totals_cand[2];
        if (lm->use_lm) lm->lam = fmax(lm->lam / 10.0, 1e-12);
    } else if (lm->use_lm) {
        lm->lam *= 10.0;
    }
    log_row[0] = lm->F_cur;
    log_row[1] = lm->use_lm ? lm->lam : 0.0;
    log_row[2] = solved ? lm->step_norm : 0.0;
    log_row[3] = (double)lm->valid_cur;
    log_row[4] = accept ? 1.0 : 0.0;
    log_row[5] = solved ? 0.0 : 1.0;
    reinterpret_cast<uint64_t *>(log_row)[9] = (uint64_t)wall_clock64();
    lm->iter += 1;
}

void launch_lm_decide(LmState *lm, const double *totals_cand, const int2 *blk_rc, int nblk, double *H_cur,
                      const double *H_cand, double *b_cur, const double *b_cand, double *X_cur, const double *X_cand,
                      int N, double *totals_cur, double *logbuf, int log_cap, hipStream_t st)
{
    const int64_t total = 36 * (int64_t)nblk + 18 * (int64_t)N;
    hipLaunchKernelGGL(lm_decide_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st, lm, totals_cand,
                       totals_cur, blk_rc, nblk, H_cur, H_cand, b_cur, b_cand, X_cur, X_cand, N, logbuf, log_cap);
}

// The state ahead of the first iteration: F and the valid count from the current system's totals (read here, so
// that the host waits for nothing before it enqueues the iterations).
__global__ void lm_init_kernel(LmState *lm, const double *__restrict__ totals, double lam, int use_lm)
{
    LmState s{};
    s.lam = lam;
    s.F_cur = totals[0];
    s.valid_cur = (int64_t)totals[2];
    s.use_lm = use_lm;
    *lm = s;
}

void launch_lm_init(LmState *lm, const double *totals, double lam, int use_lm, hipStream_t st)
{
    hipLaunchKernelGGL(lm_init_kernel, dim3(1), dim3(1), 0, st, lm, totals, lam, use_lm);
}

__global__ void copy_kernel(double *__restrict__ dst, const double *__restrict__ src, int64_t n)
{
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        dst[i] = src[i];
}

void launch_copy(double *dst, const double *src, int64_t n, hipStream_t st)
{
    if (n <= 0) return;
    int64_t blocks = (n + 255) / 256;
    if (blocks > 8192) blocks = 8192;
    hipLaunchKernelGGL(copy_kernel, dim3((unsigned)blocks), dim3(256), 0, st, dst, src, n);
}

}  // namespace pba
