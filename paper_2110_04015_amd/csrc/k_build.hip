// System build kernels: the damped normal-equation blocks and the reduced
// camera system of Sec. 3.1, eq. (8)-(15), and the block-Jacobi preconditioner
// D(S) of Sec. 3.2 (before Algorithm 1), all in FP64.
#include "ba_internal.h"
#include "kernels.h"
#include "dev_la.h"

namespace ba {

// ---------------------------------------------------------------- validation

// Sets the flag when a value of a (count0), b (count1) or c (count2, all even) is not finite:
// its exponent bits are all set.  Sixteen-byte loads, eight of a contiguous 32 KiB in flight
// (1.06 GB just written by k_project: 221 us; with the eight a grid's width apart 251).
__device__ __forceinline__ bool not_finite(const Dbl2 *__restrict__ a, int64_t n) {
    uint32_t top = 0;   // the exponent bits of a value that is not finite are the largest
    for (int64_t i = (int64_t)blockIdx.x * 2048 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 2048) {
        Dbl2 v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = a[i + u * 256 < n ? i + u * 256 : i];
#pragma unroll
        for (int u = 0; u < 8; ++u)
            top = max(top, max((uint32_t)__double2hiint(v[u].x) & 0x7FF00000u, (uint32_t)__double2hiint(v[u].y) & 0x7FF00000u));
    }
    return top == 0x7FF00000u;
}

__global__ __launch_bounds__(256) void k_check_finite(const Dbl2 *__restrict__ a, int64_t na, const Dbl2 *__restrict__ b,
                                                      int64_t nb, const Dbl2 *__restrict__ c, int64_t nc,
                                                      int32_t *status) {
    const bool bad = not_finite(a, na) | not_finite(b, nb) | not_finite(c, nc);
    if (__any(bad) && (threadIdx.x & 63) == 0) atomicOr(status, kStatusNonfinite);
}

// ---------------------------------------------------------------- packing

// Record of one observation in the tile stream: J_p rows 0 and 1 (DP values each),
// then J_l rows 0 and 1 (3 each): RecordShape<DP>::kVals values, stored as FP64 pairs,
// FP32 quads or BF16 octets (the last word zero-padded).
template <int DP>
__device__ __forceinline__ void write_record(const double *v, int64_t tile, int lane, double *J64, float *J32,
                                             uint16_t *J16) {
    typedef RecordShape<DP> R;
    if (J64) {
        double2 *d2 = reinterpret_cast<double2 *>(J64);
        for (int q = 0; q < R::kW64; ++q) d2[(tile * R::kW64 + q) * kTile + lane] = make_double2(v[2 * q], v[2 * q + 1]);
    }
    if (J32) {
        float4 *f4 = reinterpret_cast<float4 *>(J32);
        for (int q = 0; q < R::kW32; ++q) {
            float w[4];
            for (int h = 0; h < 4; ++h) w[h] = 4 * q + h < R::kVals ? (float)v[4 * q + h] : 0.0f;
            f4[(tile * R::kW32 + q) * kTile + lane] = make_float4(w[0], w[1], w[2], w[3]);
        }
    }
    if (J16) {
        uint4 *u4 = reinterpret_cast<uint4 *>(J16);
        for (int q = 0; q < R::kW16; ++q) {
            uint32_t w[4];
            for (int h = 0; h < 4; ++h) {
                const int a = 8 * q + 2 * h;
                const uint32_t lo = a < R::kVals ? f32_to_bf16((float)v[a]) : 0u;
                const uint32_t hi = a + 1 < R::kVals ? f32_to_bf16((float)v[a + 1]) : 0u;
                w[h] = lo | (hi << 16);
            }
            u4[(tile * R::kW16 + q) * kTile + lane] = make_uint4(w[0], w[1], w[2], w[3]);
        }
    }
}

// One thread per tile slot: gathers the observation's 2 x DP and 2 x 3 blocks and
// writes them in the tile layout (plus FP32 / BF16 copies).  A wavefront is a tile, so it
// also leaves its landmarks' sums that do not depend on lambda, as segmented sums across
// their lanes: J_l^T J_l (eq. (10), six entries: 00 01 02 11 12 22) and b_l = J_l^T r0
// (eq. (12)).  5.08M observations, 2.1 GB read and written: 437 us (4.9 TB/s, above a device
// copy's 4.4), against 390 us for the packing alone and 294 us for a kernel of a thread per
// landmark that read J_l and r once more.
template <int DP>
__global__ __launch_bounds__(256) void k_pack(const int64_t *__restrict__ slot_obs, const uint32_t *__restrict__ meta,
                                              const int32_t *__restrict__ tile_lmk_base, int64_t nslots,
                                              const double *__restrict__ Jp, const double *__restrict__ Jl,
                                              const double *__restrict__ r, double *__restrict__ J64,
                                              float *__restrict__ J32, uint16_t *__restrict__ J16,
                                              double *__restrict__ Vraw, double *__restrict__ bl) {
    constexpr int NV = RecordShape<DP>::kVals;
    const int64_t s = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (s >= nslots) return;   // whole wavefronts
    const int lane = threadIdx.x & 63;
    const int64_t o = slot_obs[s], tile = s / kTile;
    const uint32_t mt = meta[s];
    double v[NV], r0 = 0.0, r1 = 0.0;
    if (o >= 0) {
        const Dbl2 *p = reinterpret_cast<const Dbl2 *>(Jp + o * 2 * DP), *l = reinterpret_cast<const Dbl2 *>(Jl + o * 6);
#pragma unroll
        for (int k = 0; k < DP; ++k) {
            const Dbl2 d = p[k];
            v[2 * k] = d.x;
            v[2 * k + 1] = d.y;
        }
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const Dbl2 d = l[k];
            v[2 * DP + 2 * k] = d.x;
            v[2 * DP + 2 * k + 1] = d.y;
        }
        const Dbl2 d = reinterpret_cast<const Dbl2 *>(r)[o];
        r0 = d.x;
        r1 = d.y;
    } else {
#pragma unroll
        for (int k = 0; k < NV; ++k) v[k] = 0.0;
    }
    write_record<DP>(v, tile, lane, J64, J32, J16);
    const int ll = (int)((mt >> 16) & 63u);
    const Segs sg = key_segments(mt != kPad ? ll : 64 + lane, lane);
    const double *a = v + 2 * DP, *b = a + 3;   // J_l rows 0 and 1
    const double x[9] = {a[0] * a[0] + b[0] * b[0], a[0] * a[1] + b[0] * b[1], a[0] * a[2] + b[0] * b[2],
                         a[1] * a[1] + b[1] * b[1], a[1] * a[2] + b[1] * b[2], a[2] * a[2] + b[2] * b[2],
                         a[0] * r0 + b[0] * r1,     a[1] * r0 + b[1] * r1,     a[2] * r0 + b[2] * r1};
    double t[9];
#pragma unroll
    for (int k = 0; k < 9; ++k) t[k] = segment_scan(x[k], sg);
    if (mt != kPad && sg.end == lane) {
        const int64_t l = tile_lmk_base[tile] + ll;
#pragma unroll
        for (int k = 0; k < 6; ++k) Vraw[l * 6 + k] = t[k];
#pragma unroll
        for (int k = 0; k < 3; ++k) bl[l * 3 + k] = t[6 + k];
    }
}

// Lower-precision copies of an existing FP64 tile stream (one thread per slot).
template <int DP>
__global__ void k_convert(const double *__restrict__ J64, int64_t nslots, float *__restrict__ J32,
                          uint16_t *__restrict__ J16) {
    typedef RecordShape<DP> R;
    int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= nslots) return;
    int64_t tile = s / kTile;
    int lane = (int)(s % kTile);
    const double2 *d2 = reinterpret_cast<const double2 *>(J64);
    double v[R::kVals];
    for (int q = 0; q < R::kW64; ++q) {
        double2 d = d2[(tile * R::kW64 + q) * kTile + lane];
        v[2 * q] = d.x;
        v[2 * q + 1] = d.y;
    }
    write_record<DP>(v, tile, lane, nullptr, J32, J16);
}

void launch_convert(const double *J64, int64_t nslots, float *J32, uint16_t *J16, hipStream_t s, int dp) {
    if (nslots <= 0) return;
    const dim3 g((unsigned)((nslots + 255) / 256));
    if (dp == 6) hipLaunchKernelGGL(k_convert<6>, g, dim3(256), 0, s, J64, nslots, J32, J16);
    else hipLaunchKernelGGL(k_convert<9>, g, dim3(256), 0, s, J64, nslots, J32, J16);
}

// ---------------------------------------------------------------- landmarks

// One thread per landmark: V_lambda = V + lambda diag(V) (eq. (10) with Marquardt
// damping), V_lambda^-1 (symmetric, 6 entries) by its 3x3 Cholesky factor, and
// h0 = V_lambda^-1 b_l.
__global__ void k_landmarks_lambda(int nl, const double *__restrict__ Vraw, const double *__restrict__ bl,
                                   double lambda, double *__restrict__ vinv, double *__restrict__ h0,
                                   int32_t *status) {
    int s = blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= nl) return;
    double V[6], b[3];
    for (int k = 0; k < 6; ++k) V[k] = Vraw[(int64_t)s * 6 + k];
    for (int k = 0; k < 3; ++k) b[k] = bl[(int64_t)s * 3 + k];
    V[0] += lambda * V[0];
    V[3] += lambda * V[3];
    V[5] += lambda * V[5];
    // 3x3 Cholesky V = L L^T
    double l00 = V[0];
    bool ok = l00 > 0.0;
    l00 = sqrt(ok ? l00 : 1.0);
    double l10 = V[1] / l00, l20 = V[2] / l00;
    double l11 = V[3] - l10 * l10;
    ok = ok && l11 > 0.0;
    l11 = sqrt(ok ? l11 : 1.0);
    double l21 = (V[4] - l20 * l10) / l11;
    double l22 = V[5] - l20 * l20 - l21 * l21;
    ok = ok && l22 > 0.0;
    l22 = sqrt(ok ? l22 : 1.0);
    if (!ok) atomicOr(status, kStatusNotSpdLandmark);
    // L^-1 (lower), then V^-1 = L^-T L^-1
    double i00 = 1.0 / l00, i11 = 1.0 / l11, i22 = 1.0 / l22;
    double i10 = -l10 * i00 * i11;
    double i21 = -l21 * i11 * i22;
    double i20 = -(l20 * i00 + l21 * i10) * i22;
    double w[6];
    w[0] = i00 * i00 + i10 * i10 + i20 * i20;
    w[1] = i11 * i10 + i21 * i20;
    w[2] = i22 * i20;
    w[3] = i11 * i11 + i21 * i21;
    w[4] = i22 * i21;
    w[5] = i22 * i22;
    for (int k = 0; k < 6; ++k) vinv[(int64_t)s * 6 + k] = w[k];
    h0[(int64_t)s * 3 + 0] = w[0] * b[0] + w[1] * b[1] + w[2] * b[2];
    h0[(int64_t)s * 3 + 1] = w[1] * b[0] + w[3] * b[1] + w[4] * b[2];
    h0[(int64_t)s * 3 + 2] = w[2] * b[0] + w[4] * b[1] + w[5] * b[2];
}

// ---------------------------------------------------------------- cameras

// The observations' tile slots, from the slots' observations (-1: padding).
__global__ __launch_bounds__(256) void k_obs_slots(int64_t slots, const int64_t *__restrict__ slot_obs,
                                                   int64_t *__restrict__ obs_slot) {
    const int64_t sl = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (sl >= slots) return;
    const int64_t o = slot_obs[sl];
    if (o >= 0) obs_slot[o] = sl;
}

void launch_obs_slots(int64_t slots, const int64_t *slot_obs, int64_t *obs_slot, hipStream_t s) {
    hipLaunchKernelGGL(k_obs_slots, dim3((unsigned)((slots + 255) / 256)), dim3(256), 0, s, slots, slot_obs, obs_slot);
}

__global__ __launch_bounds__(256) void k_cam_slots(int64_t m, const int64_t *__restrict__ cam_obs,
                                                   const int64_t *__restrict__ obs_slot,
                                                   const int32_t *__restrict__ obs_lm,
                                                   const int32_t *__restrict__ lmk_store,
                                                   uint32_t *__restrict__ cam_slot, int32_t *__restrict__ cam_lmk) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= m) return;
    const int64_t o = cam_obs[i];
    cam_slot[i] = (uint32_t)obs_slot[o];
    cam_lmk[i] = lmk_store[obs_lm[o]];
}

void launch_cam_slots(int64_t m, const int64_t *cam_obs, const int64_t *obs_slot, const int32_t *obs_lm,
                      const int32_t *lmk_store, uint32_t *cam_slot, int32_t *cam_lmk, hipStream_t s) {
    hipLaunchKernelGGL(k_cam_slots, dim3((unsigned)((m + 255) / 256)), dim3(256), 0, s, m, cam_obs, obs_slot, obs_lm,
                       lmk_store, cam_slot, cam_lmk);
}

// Sums over a camera's observations, on the FP64 matrix cores:
//   U = sum J_p^T J_p, b_p = sum J_p^T r0            (eq. (9), (11); independent of lambda)
//   E = sum W V_lambda^-1 W^T, w = sum W h0, W = J_p^T J_l
// With the 2 x 2 block B = J_l V_lambda^-1 J_l^T and q = J_l h0 of an observation,
// E = sum J_p^T B J_p and w = sum J_p^T q, so all four are products of J_p^T with a few
// columns.  One work-group takes up to kCamObs observations of a camera, 64 per wavefront:
//   1. lane l loads observation l's record (12 scattered 16-byte words of the tile stream),
//      V_lambda^-1 and h0, forms B and q and leaves them and J_p in LDS;
//   2. four observations at a time, v_mfma_f64_16x16x4f64 once per Jacobian row adds
//      A^T C with A = [J_p | first 16 - DP columns of B J_p] and
//      C = [J_p | r0 | q | remaining columns of B J_p]: U, b_p, w and E (by its symmetry)
//      all lie in the one 16 x 16 result.
// The work-groups run in the order of their first slot, consecutive ones on one XCD, so that
// the cameras that share tiles read them from its L2 at about the same time.  r0 = 0 when
// only the lambda-dependent sums are asked for: the others' accumulators do not see it.
// Lane layouts as in the Gram kernel of the solvers.  No unit is full: the address units (twenty
// scattered 16-byte loads per observation) are busy for 70 % of the time, vector issue for 30 %,
// the matrix cores for 14 %, and a wavefront waits for memory for 42 % of its own.  Loads,
// barrier and products of a work-group follow each other, and 53 KB of LDS leave three of them
// to a compute unit to overlap.  Fewer address cycles alone gain nothing (camera rows read from
// the caller's Jacobians by lanes in turn: 508 against 517 us).  5.08M observations of 1,936
// cameras: 506 us, against 354 (U, b_p) + 1,389 us (E, w) with a wavefront per camera and the
// sums on the vector units; ba_set_lambda 1,420 -> 500 us.  571 cameras of very uneven
// popularity, 897k observations: an update 6.1 -> 0.45 ms.
typedef double dbl2_t __attribute__((ext_vector_type(2)));
typedef double dbl4_t __attribute__((ext_vector_type(4)));

template <int DP>
__global__ __launch_bounds__(256) void k_cameras(CameraArgs a) {
    typedef RecordShape<DP> R;
    constexpr int T = DP * (DP + 1) / 2, NA = T + DP;
    constexpr int RB = 16 - DP < DP ? 16 - DP : DP;   // columns of B J_p that A takes
    __shared__ __align__(16) double sJ[4][64][2 * DP];
    __shared__ __align__(16) double sB[4][64][8];     // B00, B01, B11, q0, q1, r0, r1
    const int lane = threadIdx.x & 63, i = lane & 15, o = lane >> 4;
    const int w = threadIdx.x >> 6;
    const int per = (a.n_blocks + 7) / 8;
    const int at = ((int)blockIdx.x & 7) * per + ((int)blockIdx.x >> 3);
    if (at >= a.n_blocks) return;   // uniform (the grid is a multiple of eight)
    const int blk = a.blk_order[at];
    const int c = a.blk_cam[blk];
    const int64_t b0 = a.cam_obs_ptr[c] + (int64_t)(blk - a.cam_blk[c]) * kCamObs + w * 64;
    const int cnt = (int)min((int64_t)64, a.cam_obs_ptr[c + 1] - b0);   // may be <= 0
    if (lane < cnt) {
        const uint32_t sl = a.cam_slot[b0 + lane];
        const int64_t l = a.cam_lmk[b0 + lane];
        const dbl2_t *rec = reinterpret_cast<const dbl2_t *>(a.J64) + (int64_t)(sl / kTile) * R::kW64 * kTile + sl % kTile;
        dbl2_t x[R::kW64];
#pragma unroll
        for (int q = 0; q < R::kW64; ++q) x[q] = rec[q * kTile];
        const dbl2_t *vp = reinterpret_cast<const dbl2_t *>(a.vinv + l * 6);
        const dbl2_t v01 = vp[0], v23 = vp[1], v45 = vp[2];
        const double g0 = a.h0[l * 3], g1 = a.h0[l * 3 + 1], g2 = a.h0[l * 3 + 2];
        double r0 = 0.0, r1 = 0.0;
        if (a.r) {
            const Dbl2 rr = reinterpret_cast<const Dbl2 *>(a.r)[a.cam_obs[b0 + lane]];
            r0 = rr.x;
            r1 = rr.y;
        }
        dbl2_t *dj = reinterpret_cast<dbl2_t *>(sJ[w][lane]);
#pragma unroll
        for (int q = 0; q < DP; ++q) dj[q] = x[q];
        // J_l rows m (x[DP].x, x[DP].y, x[DP+1].x) and k (x[DP+1].y, x[DP+2].x, x[DP+2].y)
        const double m0 = x[DP].x, m1 = x[DP].y, m2 = x[DP + 1].x;
        const double k0 = x[DP + 1].y, k1 = x[DP + 2].x, k2 = x[DP + 2].y;
        const double t0 = v01.x * m0 + v01.y * m1 + v23.x * m2;
        const double t1 = v01.y * m0 + v23.y * m1 + v45.x * m2;
        const double t2 = v23.x * m0 + v45.x * m1 + v45.y * m2;
        const double u0 = v01.x * k0 + v01.y * k1 + v23.x * k2;
        const double u1 = v01.y * k0 + v23.y * k1 + v45.x * k2;
        const double u2 = v23.x * k0 + v45.x * k1 + v45.y * k2;
        double *db = sB[w][lane];
        db[0] = m0 * t0 + m1 * t1 + m2 * t2;
        db[1] = k0 * t0 + k1 * t1 + k2 * t2;
        db[2] = k0 * u0 + k1 * u1 + k2 * u2;
        db[3] = m0 * g0 + m1 * g1 + m2 * g2;
        db[4] = k0 * g0 + k1 * g1 + k2 * g2;
        db[5] = r0;
        db[6] = r1;
    } else {   // no observation: zeros
        for (int k = 0; k < 2 * DP; ++k) sJ[w][lane][k] = 0.0;
        for (int k = 0; k < 8; ++k) sB[w][lane][k] = 0.0;
    }
    __syncthreads();
    // A: column i of J_p, or column i - DP of B J_p; C: column i of J_p, r0, q, then B J_p
    const int ka = i < DP ? i : min(i - DP, DP - 1);
    const int kc = i < DP + 2 ? 0 : min(RB + i - (DP + 2), DP - 1);
    // (two accumulators, so that the products of a step do not wait for each other)
    dbl4_t acc = dbl4_t{0.0, 0.0, 0.0, 0.0}, acc1 = acc;
    for (int j = 0; j < cnt; j += 4) {
        const double *J = sJ[w][j + o];
        const double *B = sB[w][j + o];
        const double b00 = B[0], b01 = B[1], b11 = B[2], q0 = B[3], q1 = B[4], r0 = B[5], r1 = B[6];
        const double x0 = J[ka], x1 = J[DP + ka], y0 = J[kc], y1 = J[DP + kc];
        const double A0 = i < DP ? x0 : b00 * x0 + b01 * x1;
        const double A1 = i < DP ? x1 : b01 * x0 + b11 * x1;
        const double C0 = i < DP ? x0 : i == DP ? r0 : i == DP + 1 ? q0 : b00 * y0 + b01 * y1;
        const double C1 = i < DP ? x1 : i == DP ? r1 : i == DP + 1 ? q1 : b01 * y0 + b11 * y1;
        acc = __builtin_amdgcn_mfma_f64_16x16x4f64(A0, C0, acc, 0, 0, 0);
        acc1 = __builtin_amdgcn_mfma_f64_16x16x4f64(A1, C1, acc1, 0, 0, 0);
    }
    __syncthreads();
    double (*sh)[16][16] = reinterpret_cast<double (*)[16][16]>(&sJ[0][0][0]);
    static_assert(sizeof(sJ) >= sizeof(double) * 4 * 256, "room for the wavefronts' results");
#pragma unroll
    for (int e = 0; e < 4; ++e) sh[w][o + 4 * e][i] = acc[e] + acc1[e];
    __syncthreads();
    // E and w, then U and b_p, each as packed upper triangle and vector
    const int n = a.r ? 2 * NA : NA;
    for (int t = threadIdx.x; t < n; t += 256) {
        int k = t < NA ? t : t - NA, row, col;
        if (k >= T) {
            row = k - T;
            col = t < NA ? DP + 1 : DP;
        } else {
            int p = 0;
            while (k >= DP - p) k -= DP - p++;
            const int q = p + k;   // entry (p, q), p <= q
            if (t >= NA) row = p, col = q;
            else if (p < RB) row = DP + p, col = q;
            else row = q, col = DP + 2 + (p - RB);
        }
        a.partial[(int64_t)blk * (2 * NA) + t] = (sh[0][row][col] + sh[1][row][col]) + (sh[2][row][col] + sh[3][row][col]);
    }
}

// One wavefront per camera: adds its work-groups' sums in order (U and b_p are kept), then
//   D(S)_c = U + lambda diag(U) - E   (diagonal block of eq. (14))
//   b~_c   = b_p - w                  (eq. (15))
// the damping lambda diag(U) of the S product, and the Cholesky factor of D(S)_c.
template <int DP>
__global__ __launch_bounds__(64) void k_cameras_finish(CameraArgs a) {
    constexpr int T = DP * (DP + 1) / 2, NA = T + DP;
    __shared__ double sE[NA], sU[NA], D[DP][DP], L[DP][DP];
    const int c = blockIdx.x, lane = threadIdx.x;
    const int b0 = a.cam_blk[c], b1 = a.cam_blk[c + 1];
    for (int t = lane; t < (a.r ? 2 * NA : NA); t += 64) {
        const double *p = a.partial + t;
        double s = 0.0;
        for (int b = b0; b < b1; b += 16) {   // sixteen loads in flight, added in order
            double v[16];
#pragma unroll
            for (int u = 0; u < 16; ++u) v[u] = p[(int64_t)(b + u < b1 ? b + u : b) * (2 * NA)];
#pragma unroll
            for (int u = 0; u < 16; ++u)
                if (b + u < b1) s += v[u];
        }
        if (t < NA) {
            sE[t] = s;
        } else {
            sU[t - NA] = s;
            if (t - NA < T) a.Uraw[(int64_t)c * T + t - NA] = s;
            else a.bp[(int64_t)c * DP + t - NA - T] = s;
        }
    }
    if (!a.r) {
        if (lane < T) sU[lane] = a.Uraw[(int64_t)c * T + lane];
        if (lane < DP) sU[T + lane] = a.bp[(int64_t)c * DP + lane];
    }
    __syncthreads();
    const auto packed = [](int p, int q) { return p * DP - p * (p - 1) / 2 + q - p; };   // (p, q), p <= q
    for (int t = lane; t < DP * DP; t += 64) {
        const int p = t / DP, q = t - p * DP;
        const int e = p <= q ? packed(p, q) : packed(q, p);
        double u = sU[e];
        if (p == q) u += a.lambda * sU[e];
        D[p][q] = u - sE[e];
        a.Dblk[(int64_t)c * DP * DP + t] = D[p][q];
    }
    if (lane < DP) {
        a.dU[(int64_t)c * DP + lane] = a.lambda * sU[packed(lane, lane)];
        a.bt[(int64_t)c * DP + lane] = sU[T + lane] - sE[T + lane];
    }
    __syncthreads();
    // Cholesky factor, column by column: lane i > j takes row i
    bool ok = true;
    for (int j = 0; j < DP; ++j) {
        double d = D[j][j];
        for (int p = 0; p < j; ++p) d -= L[j][p] * L[j][p];
        if (!(d > 0.0)) {
            ok = false;
            d = 1.0;
        }
        d = sqrt(d);
        if (lane == j) L[j][j] = d;
        if (lane > j && lane < DP) {
            double s = D[lane][j];
            for (int p = 0; p < j; ++p) s -= L[lane][p] * L[j][p];
            L[lane][j] = s / d;
        }
        __syncthreads();
    }
    if (!ok && lane == 0) atomicOr(a.status, kStatusNotSpdCamera);
    if (lane < T) {   // packed lower factor, row p holds L[p][0..p]
        int p = 0, k = lane;
        while (k > p) k -= ++p;
        a.Dchol[(int64_t)c * T + lane] = L[p][k];
    }
}

// ---------------------------------------------------------------- launchers

void launch_check_finite(const double *Jp, const double *Jl, const double *r, int64_t m, int dp, int32_t *status,
                         hipStream_t s) {
    const int64_t na = m * dp;
    const int blocks = (int)std::min<int64_t>((na + 2047) / 2048, 2048);
    hipLaunchKernelGGL(k_check_finite, dim3(blocks), dim3(256), 0, s, reinterpret_cast<const Dbl2 *>(Jp), na,
                       reinterpret_cast<const Dbl2 *>(Jl), m * 3, reinterpret_cast<const Dbl2 *>(r), m, status);
}

void launch_pack(const PackArgs &a, hipStream_t s) {
    const dim3 g((unsigned)((a.nslots + 255) / 256));
    if (a.dp == 6)
        hipLaunchKernelGGL(k_pack<6>, g, dim3(256), 0, s, a.slot_obs, a.meta, a.tile_lmk_base, a.nslots, a.Jp, a.Jl, a.r,
                           a.J64, a.J32, a.J16, a.Vraw, a.bl);
    else
        hipLaunchKernelGGL(k_pack<9>, g, dim3(256), 0, s, a.slot_obs, a.meta, a.tile_lmk_base, a.nslots, a.Jp, a.Jl, a.r,
                           a.J64, a.J32, a.J16, a.Vraw, a.bl);
}

void launch_landmarks_lambda(int nl, const double *Vraw, const double *bl, double lambda, double *vinv, double *h0,
                             int32_t *status, hipStream_t s) {
    hipLaunchKernelGGL(k_landmarks_lambda, dim3((nl + 255) / 256), dim3(256), 0, s, nl, Vraw, bl, lambda, vinv, h0,
                       status);
}

void launch_cameras(const CameraArgs &a, hipStream_t s) {
    const dim3 g((unsigned)((a.n_blocks + 7) / 8 * 8));
    if (a.dp == 6) {
        hipLaunchKernelGGL(k_cameras<6>, g, dim3(256), 0, s, a);
        hipLaunchKernelGGL(k_cameras_finish<6>, dim3(a.np), dim3(64), 0, s, a);
    } else {
        hipLaunchKernelGGL(k_cameras<9>, g, dim3(256), 0, s, a);
        hipLaunchKernelGGL(k_cameras_finish<9>, dim3(a.np), dim3(64), 0, s, a);
    }
}

}  // namespace ba
