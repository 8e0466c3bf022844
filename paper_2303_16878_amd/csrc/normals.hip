// Normal estimation from depth (Sec. IV-A): the normal at u is the normal of the least-squares
// plane through the unprojected neighbours u' with |u - u'| < tau_u, tau_u inversely proportional
// to the range at u, oriented towards the observer.
//
// tau_u = clamp(radius_m |fx| / d(u), min_px, max_px) pixels (a fixed metric radius seen at range
// d); neighbours need valid depth within tau (the sensor model's occlusion threshold) of d(u);
// the fit is the eigenvector of the smallest eigenvalue of the neighbours' covariance (cyclic
// Jacobi on the 3 x 3 matrix, FP64); at least min_count points and a second eigenvalue above
// 1e-12 of the trace; oriented so that n . q_u < 0.  Pixels without a normal get 0.

#include "pba_internal.h"

#include <algorithm>
#include <cmath>

namespace pba {

// 1/x and 1/sqrt(x) for x > 0 within a few ulps: the hardware estimates (relative error below 2^-24) refined by two
// Newton steps (an IEEE division or square root is some 25 instructions, and a rotation had four).
__device__ __forceinline__ double rcp2(double x)
{
    double r = __builtin_amdgcn_rcp(x);
    r = fma(r, fma(-x, r, 1.0), r);
    return fma(r, fma(-x, r, 1.0), r);
}
__device__ __forceinline__ double rsq2(double x)
{
    double y = __builtin_amdgcn_rsq(x);
    y = y * fma(-0.5 * x * y, y, 1.5);
    return y * fma(-0.5 * x * y, y, 1.5);
}

// Eigenvector of the smallest eigenvalue of the symmetric 3 x 3 matrix a (row-major), by cyclic
// Jacobi rotations; also the two smallest eigenvalues.  The matrix is scaled to unit trace, so that no square
// of its entries leaves FP64's range.
__device__ static void smallest_eigvec(double (&a)[9], double (&v)[3], double &lmin, double &lmid)
{
    double V[9] = {1, 0, 0, 0, 1, 0, 0, 0, 1};
    for (int sweep = 0; sweep < 12; ++sweep) {
        const double off = a[1] * a[1] + a[2] * a[2] + a[5] * a[5];
        const double dia = a[0] * a[0] + a[4] * a[4] + a[8] * a[8];
        if (!(off > 1e-34 * dia)) break;
#pragma unroll
        for (int pq = 0; pq < 3; ++pq) {
            const int p = pq == 2 ? 1 : 0, q = pq == 0 ? 1 : 2;
            const double apq = a[3 * p + q];
            if (apq == 0.0) continue;
            // t = sign(theta) / (|theta| + sqrt(theta^2 + 1)), theta = (a_qq - a_pp) / (2 a_pq), with theta's denominator
            // multiplied through; then c = 1 / sqrt(t^2 + 1)
            const double h = a[3 * q + q] - a[3 * p + p], g = 2.0 * apq;
            const double w = h * h + g * g;
            const double t = (h >= 0.0 ? g : -g) * rcp2(fabs(h) + w * rsq2(w));
            const double c = rsq2(t * t + 1.0), s = t * c;
            // a <- J^T a J with the rotation in the (p, q) plane
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                const double akp = a[3 * k + p], akq = a[3 * k + q];
                a[3 * k + p] = c * akp - s * akq;
                a[3 * k + q] = s * akp + c * akq;
            }
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                const double apk = a[3 * p + k], aqk = a[3 * q + k];
                a[3 * p + k] = c * apk - s * aqk;
                a[3 * q + k] = s * apk + c * aqk;
            }
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                const double vkp = V[3 * k + p], vkq = V[3 * k + q];
                V[3 * k + p] = c * vkp - s * vkq;
                V[3 * k + q] = s * vkp + c * vkq;
            }
        }
    }
    // (selects, not indexed: an array with a variable index would live in memory)
    const bool b1 = a[4] < a[0], b2 = a[8] < (b1 ? a[4] : a[0]);
    lmin = b2 ? a[8] : b1 ? a[4] : a[0];
    lmid = b2 ? fmin(a[0], a[4]) : b1 ? fmin(a[0], a[8]) : fmin(a[4], a[8]);
    v[0] = b2 ? V[2] : b1 ? V[1] : V[0];
    v[1] = b2 ? V[5] : b1 ? V[4] : V[3];
    v[2] = b2 ? V[8] : b1 ? V[7] : V[6];
}

// Tiles of 32 x 8 pixels of keyframe kf0 + blockIdx.y (those of one sensor model; one launch for all keyframes), one
// thread per pixel.  The tile's depths and its rays with a margin of R = floor(max_px) sit in LDS; outside the image
// the depth is negative.  A neighbour at (dx, dy) is inside the radius where sqrt(dx^2 + dy^2) < rad, that is
// where dx^2 + dy^2 <= klim, found once per pixel, and each row's loop runs over its neighbours only.  Bound by
// FP64 issue (69 neighbours of 20 instructions at a radius of 5, the rotations about as much again): 16 keyframes of
// 640x480 take 516 us, 2680 with a square root, bounds tests and global loads per window position, IEEE divisions and
// square roots in the rotations and a launch per keyframe.
constexpr int kTw = 32, kTh = 8, kMaxR = 16;
template <bool SPH>
__global__ void __launch_bounds__(kTw * kTh) normals_kernel(const float *__restrict__ dep_all, void *__restrict__ att4, int bf,
                                                            const KfDev *__restrict__ kfs,
                                                            const SensorDev *__restrict__ sensors,
                                                            const double2 *__restrict__ lut, int kf0, double radius_m,
                                                            double min_px, double max_px, int min_count, int R)
{
    __shared__ float D[kTh + 2 * kMaxR][kTw + 2 * kMaxR];
    __shared__ double2 Rc[kTw + 2 * kMaxR], Rr[kTh + 2 * kMaxR];
    const KfDev kf = kfs[kf0 + blockIdx.y];
    const SensorDev &sen = sensors[kf.sensor];
    if ((sen.model == MODEL_SPHERICAL) != SPH) return;
    const int H = kf.H, W = kf.W, tiles_x = (W + kTw - 1) / kTw, tiles = tiles_x * ((H + kTh - 1) / kTh);
    const float *dep = dep_all + kf.off;
    const double2 *lcol = lut + sen.lut_col, *lrow = lut + sen.lut_row;
    const double scale = radius_m * fabs(sen.fxd), tau = sen.taud;
    const int tid = threadIdx.x, tx = tid % kTw, ty = tid / kTw, w = kTw + 2 * R, h = kTh + 2 * R;
    for (int tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
        const int c0 = tile % tiles_x * kTw, r0 = tile / tiles_x * kTh;
        __syncthreads();   // the previous tile is done with
        for (int e = tid; e < w * h; e += kTw * kTh) {
            const int i = e / w, j = e - i * w, y = r0 - R + i, x = c0 - R + j;
            D[i][j] = (y >= 0 && y < H && x >= 0 && x < W) ? dep[(int64_t)y * W + x] : kNoDepth;
        }
        for (int e = tid; e < w + h; e += kTw * kTh) {
            if (e < w) Rc[e] = lcol[min(max(c0 - R + e, 0), W - 1)];
            else Rr[e - w] = lrow[min(max(r0 - R + e - w, 0), H - 1)];
        }
        __syncthreads();
        const int r = r0 + ty, c = c0 + tx;
        if (r >= H || c >= W) continue;
        const int64_t at = kf.off + (int64_t)r * W + c;
        const double d = (double)D[ty + R][tx + R];
        float4 out = att_get4(att4, bf, at);
        out.y = out.z = out.w = 0.f;
        if (d > 0.0) {
            auto point = [&](double dn, const double2 &lc, const double2 &lr, double &q0, double &q1, double &q2) {
                if (SPH) { q0 = dn * (lr.x * lc.x); q1 = dn * (lr.x * lc.y); q2 = dn * lr.y; }
                else { q0 = dn * lc.x; q1 = dn * lr.x; q2 = dn; }
            };
            const double rad = fmin(fmax(scale / d, min_px), max_px);
            int klim = (int)(rad * rad);   // the largest whole k with sqrt(k) < rad, -1 if there is none
            while (klim >= 0 && !(sqrt((double)klim) < rad)) --klim;
            while (sqrt((double)(klim + 1)) < rad) ++klim;
            int n = 0;
            double s1[3] = {0, 0, 0}, s2[6] = {0, 0, 0, 0, 0, 0};
            for (int dy = -R; dy <= R; ++dy) {
                const int left = klim - dy * dy;
                if (left < 0) continue;
                const int xm = min((int)sqrtf((float)left), R);
                const double2 lr = Rr[ty + R + dy];
                for (int dx = -xm; dx <= xm; ++dx) {
                    const double dn = (double)D[ty + R + dy][tx + R + dx];
                    if (!(dn > 0.0) || !(fabs(dn - d) <= tau)) continue;
                    double q0, q1, q2;
                    point(dn, Rc[tx + R + dx], lr, q0, q1, q2);
                    ++n;
                    s1[0] += q0; s1[1] += q1; s1[2] += q2;
                    s2[0] += q0 * q0; s2[1] += q0 * q1; s2[2] += q0 * q2;
                    s2[3] += q1 * q1; s2[4] += q1 * q2; s2[5] += q2 * q2;
                }
            }
            const double cn = (double)(n > 0 ? n : 1);
            const double m0 = s1[0] / cn, m1 = s1[1] / cn, m2 = s1[2] / cn;
            double A[9];
            A[0] = s2[0] / cn - m0 * m0; A[1] = s2[1] / cn - m0 * m1; A[2] = s2[2] / cn - m0 * m2;
            A[4] = s2[3] / cn - m1 * m1; A[5] = s2[4] / cn - m1 * m2; A[8] = s2[5] / cn - m2 * m2;
            const double tr = A[0] + A[4] + A[8], unit = 1.0 / fmax(tr, 1e-300);
            A[0] *= unit; A[1] *= unit; A[2] *= unit; A[4] *= unit; A[5] *= unit; A[8] *= unit;
            A[3] = A[1]; A[6] = A[2]; A[7] = A[5];
            double v[3], lmin, lmid;
            smallest_eigvec(A, v, lmin, lmid);
            if (n >= min_count && lmid > 1e-12 && tr > 0.0) {
                double q0, q1, q2;
                point(d, Rc[tx + R], Rr[ty + R], q0, q1, q2);
                const double sg = v[0] * q0 + v[1] * q1 + v[2] * q2 > 0.0 ? -1.0 : 1.0;
                out.y = (float)(sg * v[0]);
                out.z = (float)(sg * v[1]);
                out.w = (float)(sg * v[2]);
            }
        }
        att_put4(att4, bf, at, out);
    }
}

void launch_normals(const float *dep, void *att4, int bf, const KfDev *kfs, const SensorDev *sensors, const double2 *lut,
                    int n, int max_tiles, bool spherical, double radius_m, double min_px, double max_px, int min_count,
                    hipStream_t st)
{
    for (int k = 0; k < n; k += 32768) {   // (a grid's y extent is at most 65535)
        const dim3 grid(std::max(1, std::min(max_tiles, 65536)), std::min(n - k, 32768));
        const int R = std::min((int)floor(max_px), kMaxR);
        if (spherical)
            hipLaunchKernelGGL(normals_kernel<true>, grid, dim3(kTw * kTh), 0, st, dep, att4, bf, kfs, sensors, lut, k,
                               radius_m, min_px, max_px, min_count, R);
        else
            hipLaunchKernelGGL(normals_kernel<false>, grid, dim3(kTw * kTh), 0, st, dep, att4, bf, kfs, sensors, lut, k,
                               radius_m, min_px, max_px, min_count, R);
    }
}

int normals_tiles(int H, int W) { return ((W + kTw - 1) / kTw) * ((H + kTh - 1) / kTh); }

}  // namespace pba
