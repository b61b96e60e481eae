// Implicit Schur products of the reduced camera system (Sec. 3.1, eq. (14)):
//   S v = U_lambda v - W V_lambda^-1 W^T v
// computed from the per-observation Jacobian blocks without forming W or S:
//   e_o = J_p,o v_c                    (2)
//   g_l = sum_{o in l} J_l,o^T e_o     (3)   = (W^T v)_l
//   h_l = V_l^-1 g_l
//   y_c = sum_{o in c} J_p,o^T (e_o - J_l,o h_l) + lambda diag(U_c) v_c
// One wavefront owns one chunk of landmark tiles: landmark sums are reduced in
// LDS inside the tile, camera sums in a per-wavefront LDS accumulator indexed
// by chunk-local camera slot.  Each chunk writes one partial row per slot and a
// second kernel adds the partial rows of every camera in a fixed order, so the
// result does not depend on scheduling and no global atomics are used.
//
// The multidirectional product (Sec. 3.2, "Optimized implementation",
// eq. (19)) applies S to the N columns Z[:, p] = z restricted to the poses of
// subset p.  An observation of camera c in subset q contributes e_o to column q
// only; its landmark then carries one h_{l,p} per subset p among its observers,
// and every observation of l receives a contribution in each such column.
#include <utility>

#include "ba_internal.h"
#include "kernels.h"
#include "dev_la.h"

namespace ba {

typedef double dbl2_t __attribute__((ext_vector_type(2)));
typedef float flt4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));

// Per-observation stream record of one lane: 2 DP + 6 values (J_p rows 0, 1, then J_l
// rows 0, 1; DP = 9, or 6 for extrinsics only) as RecordShape<DP> 16 B words in FP64,
// FP32 or BF16.  Loads fetch the raw 16-byte words; unpacking (and the BF16
// conversion) is left to the point of use so that a prefetched record needs no wait.
template <int PREC, int DP>
struct Stream;
template <int DP>
struct Stream<0, DP> {
    typedef dbl2_t word_t;
    static constexpr int kWords = RecordShape<DP>::kW64;
    template <typename T>
    static __device__ __forceinline__ void unpack(const word_t (&w)[kWords], T (&v)[2 * DP + 6]) {
#pragma unroll
        for (int q = 0; q < kWords; ++q) {
            v[2 * q] = (T)w[q].x;
            v[2 * q + 1] = (T)w[q].y;
        }
    }
};
template <int DP>
struct Stream<1, DP> {
    typedef flt4_t word_t;
    static constexpr int kWords = RecordShape<DP>::kW32;
    template <typename T>
    static __device__ __forceinline__ void unpack(const word_t (&w)[kWords], T (&v)[2 * DP + 6]) {
#pragma unroll
        for (int q = 0; q < kWords; ++q) {
            const float x[4] = {w[q].x, w[q].y, w[q].z, w[q].w};
#pragma unroll
            for (int h = 0; h < 4; ++h)
                if (4 * q + h < 2 * DP + 6) v[4 * q + h] = (T)x[h];
        }
    }
};
template <int DP>
struct Stream<2, DP> {
    typedef u32x4_t word_t;
    static constexpr int kWords = RecordShape<DP>::kW16;
    template <typename T>
    static __device__ __forceinline__ void unpack(const word_t (&w)[kWords], T (&v)[2 * DP + 6]) {
#pragma unroll
        for (int q = 0; q < kWords; ++q) {
            const uint32_t u[4] = {w[q].x, w[q].y, w[q].z, w[q].w};
#pragma unroll
            for (int h = 0; h < 4; ++h) {
                if (8 * q + 2 * h < 2 * DP + 6) v[8 * q + 2 * h] = (T)bf16_to_f32(u[h] & 0xFFFFu);
                if (8 * q + 2 * h + 1 < 2 * DP + 6) v[8 * q + 2 * h + 1] = (T)bf16_to_f32(u[h] >> 16);
            }
        }
    }
};

template <int PREC, int DP>
__device__ __forceinline__ void load_words(const void *J, int64_t tile, int lane,
                                           typename Stream<PREC, DP>::word_t (&w)[Stream<PREC, DP>::kWords]) {
    typedef typename Stream<PREC, DP>::word_t W;
    constexpr int K = Stream<PREC, DP>::kWords;
    const W *p = reinterpret_cast<const W *>(J) + tile * K * kTile + lane;
#pragma unroll
    for (int q = 0; q < K; ++q) w[q] = __builtin_nontemporal_load(p + q * kTile);
}

template <int PREC, int DP>
struct Loader {
    template <typename T>
    static __device__ __forceinline__ void load(const void *J, int64_t tile, int lane, T (&v)[2 * DP + 6]) {
        typename Stream<PREC, DP>::word_t w[Stream<PREC, DP>::kWords];
        load_words<PREC, DP>(J, tile, lane, w);
        Stream<PREC, DP>::template unpack<T>(w, v);
    }
};

// ---------------------------------------------------------------- one column

// The work-group of the chunk kernels is one wavefront.  A wavefront's LDS
// instructions are performed in issue order, so ordering them needs only a
// code-motion barrier with wavefront-scope fences, not s_barrier -- which would
// also wait for the global loads of the next tile that are already in flight.
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Record, V_l^-1 and slot word of one tile for one lane.  FP64 and FP32 records
// are kept as the 24 values themselves (loading them is the unpacking); BF16
// records are kept as raw words and converted when the tile is processed, so
// that no conversion waits on a load in flight.
template <int PREC, typename T, int DP>
struct TileBuf {
    T v[2 * DP + 6];
    dbl2_t vi[3];
    uint32_t mt;
};
template <typename T, int DP>
struct TileBuf<2, T, DP> {
    u32x4_t w[RecordShape<DP>::kW16];
    dbl2_t vi[3];
    uint32_t mt;
};

template <int PREC, typename T, int DP>
__device__ __forceinline__ void fetch_record(const void *J, int t, int lane, TileBuf<PREC, T, DP> &b) {
    if constexpr (PREC == 0) {
        constexpr int K = RecordShape<DP>::kW64;
        const dbl2_t *p = reinterpret_cast<const dbl2_t *>(J) + (int64_t)t * K * kTile + lane;
#pragma unroll
        for (int q = 0; q < K; ++q) {
            const dbl2_t d = __builtin_nontemporal_load(p + q * kTile);
            b.v[2 * q] = d.x;
            b.v[2 * q + 1] = d.y;
        }
    } else if constexpr (PREC == 1) {
        constexpr int K = RecordShape<DP>::kW32;
        const flt4_t *p = reinterpret_cast<const flt4_t *>(J) + (int64_t)t * K * kTile + lane;
#pragma unroll
        for (int q = 0; q < K; ++q) {
            const flt4_t f = __builtin_nontemporal_load(p + q * kTile);
            const float x[4] = {f.x, f.y, f.z, f.w};
#pragma unroll
            for (int h = 0; h < 4; ++h)
                if (4 * q + h < 2 * DP + 6) b.v[4 * q + h] = x[h];
        }
    } else {
        load_words<2, DP>(J, t, lane, b.w);
    }
}

// Requests the record and V^-1 of tile t (slot word m, already loaded) into b.
// Padding slots read V^-1 of the tile's first landmark (every tile holds at
// least one) and ignore it.
template <int PREC, typename T, int DP>
__device__ __forceinline__ void fetch_tile(const SchurArgs &a, int t, int lane, uint32_t m, TileBuf<PREC, T, DP> &b) {
    b.mt = m;
    fetch_record<PREC, T, DP>(a.J, t, lane, b);
    const int ll = m != kPad ? (int)((m >> 16) & 63u) : 0;
    const dbl2_t *p = reinterpret_cast<const dbl2_t *>(a.vinv + (int64_t)(a.tile_lmk_base[t] + ll) * 6);
#pragma unroll
    for (int q = 0; q < 3; ++q) b.vi[q] = p[q];
}

// Segment layout of a tile's lanes: a landmark's observations occupy consecutive lanes, so
// each lane's segment is the run of lanes with its landmark index (padding lanes form
// segments of their own); the scan itself is in dev_la.h.
__device__ __forceinline__ Segs tile_segments(uint32_t mt, int lane) {
    return key_segments(mt != kPad ? (int)((mt >> 16) & 63u) : 64 + lane, lane);
}

// e = J_p v, g_l = sum J_l^T e, h_l = V_l^-1 g_l, y_c += J_p^T (e - J_l h_l) (LDS).  Products
// are formed in T; the sums g_l and y_c accumulate in FP64 for every precision.  Besides
// being the more accurate choice, it is the faster one on gfx950: with FP32 LDS accumulators
// (ds_add_f32) the FP32 product took 370 us on the F-1936-shaped problem, with FP64 ones
// (ds_add_f64) 131 us.  Landmark sums: with SEG, segmented sums across the landmark's lanes
// in registers (no LDS, no wavefront sync; the reduced-precision products, which the LDS
// work bounds); without, FP64 LDS atomics into a per-landmark row (the FP64 product, which
// HBM bounds and which keeps three wavefronts per SIMD within its registers).  The camera
// sums go to LDS, whose atomics one wavefront issues in program order (lane order within
// an instruction).
template <typename T, int DP, bool SEG>
__device__ __forceinline__ void schur_tile(const T (&J)[2 * DP + 6], const dbl2_t (&vi)[3], uint32_t mt, int lane,
                                           const T *vloc, double *yloc, double *gloc) {
    constexpr int L0 = 2 * DP, L1 = 2 * DP + 3;   // J_l rows 0 and 1
    const bool valid = mt != kPad;
    const int slot = valid ? (int)(mt & 0xFFFFu) : 0;
    const int ll = valid ? (int)((mt >> 16) & 63u) : 0;
    T vc[DP];
#pragma unroll
    for (int k = 0; k < DP; ++k) vc[k] = vloc[slot * DP + k];
    T e0 = 0, e1 = 0;
#pragma unroll
    for (int k = 0; k < DP; ++k) {
        e0 += J[k] * vc[k];
        e1 += J[DP + k] * vc[k];
    }
    T gs[3];   // g_l, rounded to T where h = V^-1 g is formed
    if constexpr (SEG) {
        const Segs sg = tile_segments(mt, lane);
#pragma unroll
        for (int k = 0; k < 3; ++k)
            gs[k] = segment_sum<T>(valid ? (double)(J[L0 + k] * e0 + J[L1 + k] * e1) : 0.0, sg);
    } else {
        gloc[lane * 3 + 0] = 0;
        gloc[lane * 3 + 1] = 0;
        gloc[lane * 3 + 2] = 0;
        wave_sync();
        if (valid) {
#pragma unroll
            for (int k = 0; k < 3; ++k) atomicAdd(&gloc[ll * 3 + k], (double)(J[L0 + k] * e0 + J[L1 + k] * e1));
        }
        wave_sync();
#pragma unroll
        for (int k = 0; k < 3; ++k) gs[k] = (T)gloc[ll * 3 + k];
    }
    if (valid) {
        const T w0 = (T)vi[0].x, w1 = (T)vi[0].y, w2 = (T)vi[1].x;
        const T w3 = (T)vi[1].y, w4 = (T)vi[2].x, w5 = (T)vi[2].y;
        const T g0 = gs[0], g1 = gs[1], g2 = gs[2];
        const T h0 = w0 * g0 + w1 * g1 + w2 * g2;
        const T h1 = w1 * g0 + w3 * g1 + w4 * g2;
        const T h2 = w2 * g0 + w4 * g1 + w5 * g2;
        const T f0 = e0 - (J[L0] * h0 + J[L0 + 1] * h1 + J[L0 + 2] * h2);
        const T f1 = e1 - (J[L1] * h0 + J[L1 + 1] * h1 + J[L1 + 2] * h2);
#pragma unroll
        for (int k = 0; k < DP; ++k) atomicAdd(&yloc[slot * DP + k], (double)(J[k] * f0 + J[DP + k] * f1));
    }
    if constexpr (!SEG) wave_sync();   // the landmark rows are reset by the next tile
}

template <int PREC, typename T, int DP>
__device__ __forceinline__ void process_tile(const TileBuf<PREC, T, DP> &b, int lane, const T *vloc, double *yloc,
                                             double *gloc) {
    if constexpr (PREC == 2) {
        T J[2 * DP + 6];
        Stream<2, DP>::template unpack<T>(b.w, J);
        schur_tile<T, DP, true>(J, b.vi, b.mt, lane, vloc, yloc, gloc);
    } else {
        schur_tile<T, DP, PREC != 0>(b.v, b.vi, b.mt, lane, vloc, yloc, gloc);
    }
}

// P_{i+1} = Z - beta P_i (Alg. 1), rounded alike wherever it is formed
__device__ __forceinline__ double next_direction(double z, double beta, double p) { return fma(-beta, p, z); }

// Software pipeline over the tiles of the chunk with two buffers: the record and
// V^-1 of tile t + 1 and the slot word of tile t + 2 are requested before tile t
// is processed, so a wavefront keeps up to two tiles of the stream in flight.  PCG: the
// product's vector is z - beta v.  A small problem's product lasts as long as its reads take
// one after another, those of the arguments among them: 50 cameras 4.56 us, 4.72 with PCG's
// test at run time, 4.80 with a test of its own as well for each of the reasons not to run.
template <int PREC, typename T, int DP, bool PCG = false>
__global__ __launch_bounds__(64) void k_schur1(SchurArgs a, const double *__restrict__ v) {
    extern __shared__ __align__(16) unsigned char smem[];
    // (the flag and beta are requested with the chunk's bounds)
    double done = 0.0;
    if (a.done || a.seg_skip) {
        if (a.seg_skip && a.seg_skip[a.chunk_seg[blockIdx.x]]) return;
        if (a.done) done = *a.done;
    }
    const double beta = PCG ? *a.beta : 0.0;
    double *yloc = reinterpret_cast<double *>(smem);
    double *gloc = yloc + a.max_slots * DP;                                   // FP64: landmark rows
    T *vloc = reinterpret_cast<T *>(gloc + (PREC == 0 ? 3 * kTile : 0));
    const int chunk = blockIdx.x;
    const int lane = threadIdx.x;
    const int pb = a.chunk_part[chunk];
    const int ns = a.chunk_part[chunk + 1] - pb;
    const int t0 = a.chunk_tile[chunk], t1 = a.chunk_tile[chunk + 1];
    const uint32_t *meta = a.meta + lane;
    const int tl = t1 - 1;   // slot words past the chunk's end are read from its last tile
    if (done != 0.0) return;
    TileBuf<PREC, T, DP> A, B;
    uint32_t mA, mB = 0;
    if (t0 < t1) {
        fetch_tile<PREC, T, DP>(a, t0, lane, meta[(int64_t)t0 * kTile], A);
        mB = meta[(int64_t)min(t0 + 1, tl) * kTile];
    }
    for (int i = lane; i < ns * DP; i += kTile) {
        const int64_t k = (int64_t)a.part_cam[pb + i / DP] * DP + i % DP;
        vloc[i] = (T)(PCG ? next_direction(a.z[k], beta, v[k]) : v[k]);
        yloc[i] = 0.0;
    }
    wave_sync();
    // steady state: tiles t, t + 1 and t + 2 exist, so both requests are unconditional
    // (a branch around a load leaves the compiler waiting for it at the join)
    int t = t0;
    for (; t + 2 < t1; t += 2) {
        fetch_tile<PREC, T, DP>(a, t + 1, lane, mB, B);
        mA = meta[(int64_t)(t + 2) * kTile];
        process_tile<PREC, T, DP>(A, lane, vloc, yloc, gloc);
        fetch_tile<PREC, T, DP>(a, t + 2, lane, mA, A);
        mB = meta[(int64_t)min(t + 3, tl) * kTile];
        process_tile<PREC, T, DP>(B, lane, vloc, yloc, gloc);
    }
    // the last one or two tiles
    if (t + 1 < t1) {
        fetch_tile<PREC, T, DP>(a, t + 1, lane, mB, B);
        process_tile<PREC, T, DP>(A, lane, vloc, yloc, gloc);
        process_tile<PREC, T, DP>(B, lane, vloc, yloc, gloc);
    } else if (t < t1) {
        process_tile<PREC, T, DP>(A, lane, vloc, yloc, gloc);
    }
    // row of slot k goes to its camera-major position
    for (int i = lane; i < ns * DP; i += kTile) {
        const int64_t row = a.part_dst[pb + i / DP];
        a.partial[row * DP + i % DP] = (double)yloc[i];
    }
}

// Sum of the DP-vectors rows[a..b) by the calling wavefront, R = 64 / DP rows at a
// time (7 for DP = 9, 10 for DP = 6): lane l < R DP adds component l % DP of rows
// a + l / DP + R i, eight rows per batch with all eight loads in flight (rows past b read
// row a and are dropped), row i into running sum i mod 4; then the 4 R sums of a
// component are added in a fixed order through sh (64 doubles of the wavefront).  Every
// lane returns its component's total (lanes past R DP return component 0's).
template <int DP>
__device__ __forceinline__ double wave_rows(const double *__restrict__ rows, int64_t a, int64_t b, double *sh) {
    constexpr int R = 64 / DP;
    const int lane = threadIdx.x & 63;
    double s[4] = {0.0, 0.0, 0.0, 0.0};
    if (lane < R * DP) {
        const int r0 = lane / DP, k = lane - r0 * DP;
        for (int64_t j = a + r0; j < b; j += 8 * R) {
            double v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int64_t jj = j + u * R;
                v[u] = rows[(jj < b ? jj : a) * DP + k];
            }
#pragma unroll
            for (int u = 0; u < 8; ++u)
                if (j + u * R < b) s[u & 3] += v[u];
        }
    }
    sh[lane] = (s[0] + s[1]) + (s[2] + s[3]);
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    const int k = lane < R * DP ? lane % DP : 0;
    double t = 0.0;
    for (int m = 0; m < R; ++m) t += sh[k + DP * m];
    return t;
}

// y_c = lambda diag(U_c) v_c + sum of the partial rows of camera c, which are
// contiguous (camera-major); one wavefront per camera (wave_rows).  With gram, block b
// also leaves gram[2 b] = sum of y_c . v_c and gram[2 b + 1] = sum of v_c . gr_c over its
// four cameras (the Gram products Q^T P and P^T r of a one-column block, Q = S P).
// The skip flag, the camera's row range and its entries of v, diag(U) and gr are
// requested together, before anything waits on one of them (a wavefront past the last
// camera reads the last camera's and drops them).  PCG: the product's vector is z - beta v,
// which every chunk formed for its cameras and this kernel, after all of them, stores in v: a
// launch less per iteration (571 cameras and fewer: 2 us and the gap of one).  (An instance of
// its own: with d_p = 6 the run-time test took four more registers and 0.3 us, 5.20 against
// 4.89 us after the BF16 product of 70 cameras.)
template <int DP, bool HIST = false, bool PCG = false>
__global__ __launch_bounds__(256) void k_reduce1(int np, const int32_t *__restrict__ ptr,
                                                 const double *__restrict__ partial,
                                                 const double *__restrict__ dU, double *__restrict__ v,
                                                 const double *__restrict__ z, const double *__restrict__ beta,
                                                 double *__restrict__ y, const double *__restrict__ done,
                                                 const int32_t *__restrict__ cam_seg,
                                                 const int32_t *__restrict__ seg_skip, double *__restrict__ gram,
                                                 const double *__restrict__ gr, float *__restrict__ y32,
                                                 const BatchProb *__restrict__ prob,
                                                 const BatchDyn *__restrict__ dyn, double *__restrict__ hist) {
    __shared__ double sh[4][64];
    __shared__ double gsum[2][4];
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int c = blockIdx.x * 4 + w;
    const int cl = c < np ? c : np - 1;
    const int64_t i = (int64_t)cl * DP + (lane < DP ? lane : 0);
    const double dn = done ? *done : 0.0;
    const int32_t ra = ptr[cl], rb = ptr[cl + 1];
    double vi = v[i];
    const double du = dU[i], zi = PCG ? z[i] : 0.0, be = PCG ? *beta : 0.0;
    const double gi = gram ? gr[i] : 0.0;
    double *yo = HIST ? nullptr : y + i;
    if (HIST) {   // the row's place in its problem's next history column
        const int b = cam_seg[cl];
        const BatchProb P = prob[b];
        yo = hist + P.hbase + (int64_t)dyn[b].hcols * P.n + (i - P.row0);
    }
    if (dn != 0.0) return;
    if (PCG) vi = next_direction(zi, be, vi);
    double qp = 0.0, pr = 0.0;
    if (c < np && !(seg_skip && seg_skip[cam_seg[c]])) {   // uniform per wavefront
        const double t = wave_rows<DP>(partial, ra, rb, sh[w]);
        if (lane < DP) {
            const double yi = du * vi + t;
            *yo = yi;
            if (PCG) v[i] = vi;
            if (y32) y32[i] = (float)yi;
            if (gram) {
                qp = yi * vi;
                pr = vi * gi;
            }
        }
    }
    if (!gram) return;   // the same for the whole launch
    qp = wave_sum(qp);
    pr = wave_sum(pr);
    if (lane == 0) {
        gsum[0][w] = qp;
        gsum[1][w] = pr;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        gram[2 * blockIdx.x] = (gsum[0][0] + gsum[0][1]) + (gsum[0][2] + gsum[0][3]);
        gram[2 * blockIdx.x + 1] = (gsum[1][0] + gsum[1][1]) + (gsum[1][2] + gsum[1][3]);
    }
}

template <int PREC, typename T>
static auto schur1_kernel(int dp, bool pcg) {
    if (dp == 6) return pcg ? k_schur1<PREC, T, 6, true> : k_schur1<PREC, T, 6>;
    return pcg ? k_schur1<PREC, T, 9, true> : k_schur1<PREC, T, 9>;
}

void launch_schur_chunks(const SchurArgs &a, const double *v, hipStream_t s) {
    if (a.n_chunks > 0) {
        // FP64 camera rows (and, for the FP64 product, landmark rows), v in the product precision
        const size_t esz = a.precision == 0 ? sizeof(double) : sizeof(float);
        const size_t lds = (size_t)(a.max_slots * a.dp + (a.precision == 0 ? 3 * kTile : 0)) * sizeof(double) +
                           (size_t)a.max_slots * a.dp * esz;
        auto kernel = a.precision == 0   ? schur1_kernel<0, double>(a.dp, a.z)
                      : a.precision == 1 ? schur1_kernel<1, float>(a.dp, a.z)
                                         : schur1_kernel<2, float>(a.dp, a.z);
        hipLaunchKernelGGL(kernel, dim3(a.n_chunks), dim3(kTile), lds, s, a, v);
    }
}

int schur_gram_blocks(int np) { return (np + 3) / 4; }

void launch_schur_reduce(const SchurArgs &a, const double *v, double *y, hipStream_t s) {
    const dim3 g((unsigned)schur_gram_blocks(a.np)), b(256);
    double *vw = const_cast<double *>(v);   // written with a.z only (then the caller's own vector)
    auto kernel = a.dp == 6 ? (a.z ? k_reduce1<6, false, true> : k_reduce1<6>)
                  : a.hist  ? k_reduce1<9, true>   // batches: d_p = 9
                  : a.z     ? k_reduce1<9, false, true>
                            : k_reduce1<9>;
    hipLaunchKernelGGL(kernel, g, b, 0, s, a.np, a.cam_part_ptr, a.partial, a.dU, vw, a.z, a.beta, y, a.done, a.cam_seg,
                       a.seg_skip, a.gram, a.gram_r, a.y32, a.prob, a.dyn, a.hist);
}

void launch_schur_matvec(const SchurArgs &a, const double *v, double *y, hipStream_t s) {
    launch_schur_chunks(a, v, s);
    launch_schur_reduce(a, v, y, s);
}

// ---------------------------------------------------------------- N columns

// Slot words of one lane of a tile for the multidirectional product: the pair word
// (own pair, first pair of the landmark, pair count; kPad on padding slots), the
// camera, the pair's landmark (0xFF past the tile's pairs) and the offset of the
// slot's output indices.
struct MultiSlot {
    uint32_t mm;
    int32_t cam;
    uint32_t pll;
    uint32_t ooff;
};

__device__ __forceinline__ MultiSlot fetch_mslot(const MultiArgs &a, int64_t sidx) {
    MultiSlot m;
    m.mm = a.mmeta[sidx];
    m.cam = a.slot_cam[sidx];
    m.pll = a.pair_ll[sidx];
    m.ooff = a.slot_ooff[sidx];
    return m;
}

// Record, z of the slot's camera, V^-1 of the lane's pair landmark and the slot words
// of one tile (see TileBuf).  Padding slots read camera 0's z and the tile's first
// landmark's V^-1 and ignore them.
template <int PREC, typename T, int DP>
struct MultiBuf {
    TileBuf<PREC, T, DP> r;   // record (r.vi and r.mt unused)
    double z[DP];             // z_c
    dbl2_t vi[3];
    MultiSlot m;
    uint32_t obase;           // tile_oidx of the tile
    int o0, o1;               // output rows of the slot's first two pairs (kept with the tile's loads)
};

// The reduced-precision products sum each pair across its lanes (a pair's observations
// occupy consecutive lanes: a landmark's slots are in camera order and the subsets are
// ranges of consecutive cameras), so every lane takes V^-1 of its own observation's
// landmark; the FP64 product forms h of pair p on lane p, from V^-1 of that pair's landmark.
template <int PREC, typename T, int DP>
__device__ __forceinline__ void fetch_mtile(const MultiArgs &a, const double *__restrict__ z, int t, int lane,
                                            const MultiSlot &m, MultiBuf<PREC, T, DP> &b) {
    b.m = m;
    fetch_record<PREC, T, DP>(a.J, t, lane, b.r);
    const bool valid = m.mm != kPad;
    const double *zc = z + (int64_t)(valid ? m.cam : 0) * DP;
#pragma unroll
    for (int k = 0; k < DP; ++k) b.z[k] = zc[k];
    int ll;
    if constexpr (PREC != 0) {
        const uint32_t mt = a.meta[(int64_t)t * kTile + lane];
        ll = mt != kPad ? (int)((mt >> 16) & 63u) : 0;
    } else {
        ll = m.pll != 0xFFu ? (int)m.pll : 0;
    }
    const dbl2_t *p = reinterpret_cast<const dbl2_t *>(a.vinv + (int64_t)(a.tile_lmk_base[t] + ll) * 6);
#pragma unroll
    for (int q = 0; q < 3; ++q) b.vi[q] = p[q];
    b.obase = a.tile_oidx[t];
    // The first two output rows travel with the tile: a load issued while the tile is
    // processed would wait for every load in flight, the next tile's included.  A padding
    // slot reads the tile's first entry (every tile holds an observation) and ignores it.
    const uint16_t *oi = a.oidx + b.obase + (valid ? m.ooff : 0u);
    const int cnt = valid ? (int)((m.mm >> 16) & 0xFFu) : 1;
    b.o0 = oi[0];
    b.o1 = oi[cnt > 1 ? 1 : 0];
}

// First half of one tile: e = J_p z_c; g per (landmark, subset) pair = sum over the pair's
// observations of J_l^T e; h = V^-1 g.  In the reduced-precision products g is a segmented
// sum across the pair's lanes in registers and the pair's last lane holds h; in FP64 g goes
// through LDS atomics and lane p forms h of pair p.
template <typename T>
struct PairVals {
    T e0, e1;       // e of the lane's observation
    T h0, h1, h2;   // h of pair `pair`
    int pair;       // -1: the lane holds no pair's h
};

template <int PREC, typename T, int DP, bool TWO>
__device__ __forceinline__ PairVals<T> pair_tile(const T (&J)[2 * DP + 6], const double (&zb)[DP],
                                                 const dbl2_t (&vi)[3], const MultiSlot &m, int lane, double *gloc) {
    constexpr int L0 = 2 * DP, L1 = 2 * DP + 3;   // J_l rows 0 and 1
    const bool valid = m.mm != kPad;
    PairVals<T> r;
    T e0 = 0, e1 = 0;
#pragma unroll
    for (int k = 0; k < DP; ++k) {
        e0 += J[k] * (T)zb[k];
        e1 += J[DP + k] * (T)zb[k];
    }
    r.e0 = e0;
    r.e1 = e1;
    const int own = (int)(m.mm & 0xFFu);
    const T w0 = (T)vi[0].x, w1 = (T)vi[0].y, w2 = (T)vi[1].x;
    const T w3 = (T)vi[1].y, w4 = (T)vi[2].x, w5 = (T)vi[2].y;
    T g0, g1, g2;
    if constexpr (PREC != 0) {
        // segments: the pairs (own pair index), padding lanes one each
        const Segs sg = tile_segments(valid ? (uint32_t)own << 16 : kPad, lane);
        double gs[3];   // the pair's total, in its last lane (the only one that uses it)
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            // TWO: contracted as this compiler contracts the one-pass kernel's short chunks (the
            // dense problems the two-pass form takes), so that both give the same term.  Another
            // compiler may choose otherwise in the one-pass kernel: then the two forms part by
            // one FP32 rounding of a term, as that kernel's two copies of this code do already
            // (written out for both, its results move by as much against what they were)
            T t;
            if constexpr (!TWO) t = J[L0 + k] * e0 + J[L1 + k] * e1;
            else if constexpr (PREC == 2 && DP == 6) t = fmaf(J[L0 + k], e0, J[L1 + k] * e1);
            else t = fmaf(J[L1 + k], e1, J[L0 + k] * e0);
            gs[k] = segment_scan(valid ? (double)t : 0.0, sg);
        }
        r.pair = valid && sg.end == lane ? own : -1;
        g0 = (T)gs[0], g1 = (T)gs[1], g2 = (T)gs[2];
    } else {
        gloc[lane * 3 + 0] = 0;
        gloc[lane * 3 + 1] = 0;
        gloc[lane * 3 + 2] = 0;
        wave_sync();
        if (valid) {
#pragma unroll
            for (int k = 0; k < 3; ++k) atomicAdd(&gloc[own * 3 + k], (double)(J[L0 + k] * e0 + J[L1 + k] * e1));
        }
        wave_sync();
        r.pair = m.pll != 0xFFu ? lane : -1;
        g0 = (T)gloc[lane * 3], g1 = (T)gloc[lane * 3 + 1], g2 = (T)gloc[lane * 3 + 2];
    }
    r.h0 = w0 * g0 + w1 * g1 + w2 * g2;
    r.h1 = w1 * g0 + w3 * g1 + w4 * g2;
    r.h2 = w2 * g0 + w4 * g1 + w5 * g2;
    return r;
}

// One tile: h per pair (pair_tile), then every observation of the landmark adds
// J_p^T (e [own pair] - J_l h_pair) to its (camera, pair subset) row.
template <int PREC, typename T, int DP>
__device__ __forceinline__ void multi_tile(const MultiArgs &a, const T (&J)[2 * DP + 6], const double (&zb)[DP],
                                           const dbl2_t (&vi)[3], const MultiSlot &m, uint32_t obase, int o0, int o1,
                                           int lane, double *yloc, double *gloc, double *hloc) {
    constexpr int L0 = 2 * DP, L1 = 2 * DP + 3;   // J_l rows 0 and 1
    const bool valid = m.mm != kPad;
    const PairVals<T> pv = pair_tile<PREC, T, DP, false>(J, zb, vi, m, lane, gloc);
    const T e0 = pv.e0, e1 = pv.e1;
    const int own = (int)(m.mm & 0xFFu);
    if (pv.pair >= 0) {
        hloc[pv.pair * 3 + 0] = (double)pv.h0;
        hloc[pv.pair * 3 + 1] = (double)pv.h1;
        hloc[pv.pair * 3 + 2] = (double)pv.h2;
    }
    wave_sync();
    if (valid) {
        const int base = (int)((m.mm >> 8) & 0xFFu), cnt = (int)((m.mm >> 16) & 0xFFu);
        auto add_pair = [&](int pj, int o) {
            const T h0 = (T)hloc[pj * 3], h1 = (T)hloc[pj * 3 + 1], h2 = (T)hloc[pj * 3 + 2];
            T f0 = -(J[L0] * h0 + J[L0 + 1] * h1 + J[L0 + 2] * h2);
            T f1 = -(J[L1] * h0 + J[L1 + 1] * h1 + J[L1 + 2] * h2);
            if (pj == own) {
                f0 += e0;
                f1 += e1;
            }
#pragma unroll
            for (int k = 0; k < DP; ++k) atomicAdd(&yloc[o * DP + k], (double)(J[k] * f0 + J[DP + k] * f1));
        };
        add_pair(base, o0);   // cnt >= 1 on a valid slot
        if (cnt > 1) add_pair(base + 1, o1);
        // landmarks spanning three subsets or more: the rest of the rows from memory
        const uint16_t *oi = a.oidx + obase + m.ooff;
        for (int j = 2; j < cnt; ++j) add_pair(base + j, oi[j]);
    }
    wave_sync();
}

template <int PREC, typename T, int DP>
__device__ __forceinline__ void process_mtile(const MultiArgs &a, const MultiBuf<PREC, T, DP> &b, int lane,
                                              double *yloc, double *gloc, double *hloc) {
    if constexpr (PREC == 2) {
        T J[2 * DP + 6];
        Stream<2, DP>::template unpack<T>(b.r.w, J);
        multi_tile<PREC, T, DP>(a, J, b.z, b.vi, b.m, b.obase, b.o0, b.o1, lane, yloc, gloc, hloc);
    } else {
        multi_tile<PREC, T, DP>(a, b.r.v, b.z, b.vi, b.m, b.obase, b.o0, b.o1, lane, yloc, gloc, hloc);
    }
}

// One wavefront per chunk of tiles, software-pipelined as k_schur1: the record, z
// gather and V^-1 of tile t + 1 and the slot words of tile t + 2 are requested before
// tile t is processed.
template <int PREC, typename T, int DP>
__global__ __launch_bounds__(64) void k_schur_multi(MultiArgs a, const double *__restrict__ z) {
    if (a.skip && *a.skip != 0.0) return;
    if (a.seg_skip && a.seg_skip[a.chunk_seg[blockIdx.x]]) return;
    extern __shared__ __align__(16) unsigned char smem[];
    double *yloc = reinterpret_cast<double *>(smem);   // FP64 sums for every precision (see schur_tile)
    double *gloc = yloc + a.max_out * DP;
    double *hloc = gloc + 3 * kTile;
    const int chunk = blockIdx.x;
    const int lane = threadIdx.x;
    const int pb = a.chunk_part[chunk];
    const int no = a.chunk_part[chunk + 1] - pb;
    const int t0 = a.chunk_tile[chunk], t1 = a.chunk_tile[chunk + 1];
    const int tl = t1 - 1;   // slot words past the chunk's end are read from its last tile
    MultiBuf<PREC, T, DP> A, B;
    MultiSlot mA, mB{};
    if (t0 < t1) {
        fetch_mtile<PREC, T, DP>(a, z, t0, lane, fetch_mslot(a, (int64_t)t0 * kTile + lane), A);
        mB = fetch_mslot(a, (int64_t)min(t0 + 1, tl) * kTile + lane);
    }
    for (int i = lane; i < no * DP; i += kTile) yloc[i] = 0.0;
    wave_sync();
    int t = t0;
    for (; t + 2 < t1; t += 2) {
        fetch_mtile<PREC, T, DP>(a, z, t + 1, lane, mB, B);
        mA = fetch_mslot(a, (int64_t)(t + 2) * kTile + lane);
        process_mtile<PREC, T, DP>(a, A, lane, yloc, gloc, hloc);
        fetch_mtile<PREC, T, DP>(a, z, t + 2, lane, mA, A);
        mB = fetch_mslot(a, (int64_t)min(t + 3, tl) * kTile + lane);
        process_mtile<PREC, T, DP>(a, B, lane, yloc, gloc, hloc);
    }
    if (t + 1 < t1) {
        fetch_mtile<PREC, T, DP>(a, z, t + 1, lane, mB, B);
        process_mtile<PREC, T, DP>(a, A, lane, yloc, gloc, hloc);
        process_mtile<PREC, T, DP>(a, B, lane, yloc, gloc, hloc);
    } else if (t < t1) {
        process_mtile<PREC, T, DP>(a, A, lane, yloc, gloc, hloc);
    }
    for (int i = lane; i < no * DP; i += kTile) {
        const int64_t row = a.part_dst[pb + i / DP];
        a.partial[row * DP + i % DP] = (double)yloc[i];
    }
}

// Y[p][c] = [group(c) == p] lambda diag(U_c) z_c + sum of the partial rows of (c, p),
// which are contiguous ((camera, subset)-major); one wavefront per (c, p) (wave_rows)
template <int DP>
__global__ __launch_bounds__(256) void k_reduce_multi(int np, int N, const int32_t *__restrict__ ptr,
                                                      const double *__restrict__ partial,
                                                      const double *__restrict__ dU,
                                                      const int32_t *__restrict__ group,
                                                      const double *__restrict__ z, double *__restrict__ Y,
                                                      const int32_t *__restrict__ cam_seg,
                                                      const int32_t *__restrict__ seg_skip,
                                                      const double *__restrict__ skip) {
    if (skip && *skip != 0.0) return;
    __shared__ double sh[4][64];
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int64_t key = (int64_t)blockIdx.x * 4 + w;   // c * N + p
    if (key >= (int64_t)np * N) return;                 // uniform per wavefront
    const int c = (int)(key / N), p = (int)(key - (int64_t)c * N);
    if (seg_skip && seg_skip[cam_seg[c]]) return;
    const double t = wave_rows<DP>(partial, ptr[key], ptr[key + 1], sh[w]);
    if (lane < DP) {
        const int64_t rem = (int64_t)c * DP + lane;
        Y[(int64_t)p * np * DP + rem] = (group[c] == p ? dU[rem] * z[rem] : 0.0) + t;
    }
}

// ---------------------------------------------------------------- N columns in two passes
//
// Where a landmark's observers fall in many subsets the one-pass form pays for every
// (observation, subset) pair an LDS row of its own: a tile of the 571-camera dense problem
// with 47 subsets touches up to 1,600 of them, one wavefront fills a CU's LDS, and its rows
// go to memory as partials (369 MB).  Here the landmark side and the camera side are split:
//   k_pair_h (landmark-major tiles): h = V^-1 g per (landmark, subset) and
//     f = e - J_l h_own per observation, the own subset's term;
//   k_pair_out (camera-major records): a work-group sums the columns of up to kCamObs
//     observations of one camera, sum_o J_p^T ([p = own] f_o - [p != own] J_l h_{l,p});
//   k_pair_reduce: the work-groups of a camera, in order.
// Every term is formed as the one-pass form forms it.
// The 571-camera dense problem (897k observations, N = 47), one-pass form -> this one: FP64
// 845 + 100 us (product, reduction) -> 38 + 98 + 12 us, FP32 888 + 101 us -> 24 + 79 + 13 us.
// k_pair_h streams the records (5 TB/s); the camera side is bound by the issue of its vector
// instructions (95 per four observations in FP64, beside 35 us of the matrix cores).

// h of a (landmark, subset) pair and the subset
template <typename T>
struct alignas(4 * sizeof(T)) PairH;
template <>
struct alignas(32) PairH<double> {
    double h[3];
    int64_t grp;
};
template <>
struct alignas(16) PairH<float> {
    float h[3];
    int32_t grp;
};

// a . b, in the order in which the one-pass form rounds it
template <typename T>
__device__ __forceinline__ T dot3(const T *a, const T *b) {
    return __builtin_elementwise_fma(a[2], b[2], __builtin_elementwise_fma(a[0], b[0], a[1] * b[1]));
}

// a - b, never contracted with the operations that formed a
template <typename T>
__device__ __forceinline__ T sub_plain(T a, T b) {
#pragma clang fp contract(off)
    return a - b;
}

// -f of every slot's own subset (F, two values) and the entry of every pair (H, at
// 64 tile + pair).  One wavefront per tile.
template <int PREC, typename T, int DP>
__global__ __launch_bounds__(256) void k_pair_h(MultiArgs a, const double *__restrict__ z) {
    if (a.skip && *a.skip != 0.0) return;
    constexpr int L0 = 2 * DP, L1 = 2 * DP + 3;   // J_l rows 0 and 1
    __shared__ double gsh[PREC == 0 ? 4 * 3 * kTile : 1];
    __shared__ T hsh[4][3 * kTile];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int64_t t = (int64_t)blockIdx.x * 4 + w;
    if (t >= a.n_tiles) return;   // uniform per wavefront
    if (a.seg_skip && a.seg_skip[a.tile_seg[t]]) return;
    const int64_t si = t * kTile + lane;
    MultiSlot m;
    m.mm = a.mmeta[si];
    m.cam = a.slot_cam[si];
    m.pll = a.pair_ll[si];
    m.ooff = 0;
    TileBuf<PREC, T, DP> b;
    fetch_record<PREC, T, DP>(a.J, (int)t, lane, b);
    const bool valid = m.mm != kPad;
    const double *zc = z + (int64_t)(valid ? m.cam : 0) * DP;
    double zb[DP];
#pragma unroll
    for (int k = 0; k < DP; ++k) zb[k] = zc[k];
    int ll;
    if constexpr (PREC != 0) {
        const uint32_t mt = a.meta[si];
        ll = mt != kPad ? (int)((mt >> 16) & 63u) : 0;
    } else {
        ll = m.pll != 0xFFu ? (int)m.pll : 0;
    }
    const dbl2_t *vp = reinterpret_cast<const dbl2_t *>(a.vinv + (int64_t)(a.tile_lmk_base[t] + ll) * 6);
    dbl2_t vi[3];
#pragma unroll
    for (int q = 0; q < 3; ++q) vi[q] = vp[q];
    T J[2 * DP + 6];
    if constexpr (PREC == 2) {
        Stream<2, DP>::template unpack<T>(b.w, J);
    } else {
#pragma unroll
        for (int k = 0; k < 2 * DP + 6; ++k) J[k] = b.v[k];
    }
    const PairVals<T> r = pair_tile<PREC, T, DP, true>(J, zb, vi, m, lane, gsh + (PREC == 0 ? w * 3 * kTile : 0));
    T *hl = hsh[w];
    if (r.pair >= 0) {
        hl[r.pair * 3 + 0] = r.h0;
        hl[r.pair * 3 + 1] = r.h1;
        hl[r.pair * 3 + 2] = r.h2;
        PairH<T> e;
        e.h[0] = r.h0;
        e.h[1] = r.h1;
        e.h[2] = r.h2;
        e.grp = a.pair_grp[t * kTile + r.pair];
        reinterpret_cast<PairH<T> *>(a.pair_h)[t * kTile + r.pair] = e;
    }
    wave_sync();
    if (valid) {
        const int own = (int)(m.mm & 0xFFu);
        T *F = reinterpret_cast<T *>(a.pair_f) + si * 2;
        F[0] = sub_plain(dot3(J + L0, hl + own * 3), r.e0);
        F[1] = sub_plain(dot3(J + L1, hl + own * 3), r.e1);
    }
}

// The share of wavefront w of work-group `block`: observations [lo, hi) of those at b0.
struct PairShare {
    int64_t b0;
    int c, lo, hi;
};
__device__ __forceinline__ PairShare pair_share(const MultiArgs &a, int block, int w) {
    PairShare s;
    s.c = a.blk_cam[block];
    s.b0 = a.cam_obs_ptr[s.c] + (int64_t)(block - a.cam_blk[s.c]) * kCamObs;
    const int cnt = (int)min((int64_t)kCamObs, a.cam_obs_ptr[s.c + 1] - s.b0);
    const int per = (cnt + 3) / 4;
    s.lo = min(cnt, w * per);
    s.hi = min(cnt, s.lo + per);
    return s;
}

// The four wavefronts' column sums (negated terms), [component][column], to the block's partials.
template <int DP>
__device__ __forceinline__ void pair_store(const double (&sh)[4][DP][64], int N, double *__restrict__ partial) {
    __syncthreads();
    double *out = partial + (int64_t)blockIdx.x * DP * N;
    for (int i = threadIdx.x; i < DP * 64; i += 256) {
        const int k = i >> 6, p = i & 63;
        if (p < N) out[k * N + p] = -((sh[0][k][p] + sh[1][k][p]) + (sh[2][k][p] + sh[3][k][p]));
    }
}

// In both forms of the camera side a wavefront takes four observations at a time: lane
// (o, i) = (lane / 16, lane mod 16) works for observation j + o on pair i of its landmark
// (a landmark with more than 16 pairs takes further rounds), so the work follows the pairs
// there are and not the number of subsets.  pair_obs: the observation's first pair entry and,
// in y, its slot in that tile (bits 0..5) and its landmark's pairs (bits 8..14).
// DIRECT: there is no room for camera-major records, and they are read from the tile stream
// (a record's 16-byte words 64 words apart), to the same bits.  The product of the dense problem
// above takes 310 us so in FP64 and 173 us with records, 188 / 134 us in FP32, 140 / 125 in BF16.

// x of lane `AT` of the lane's row of 16, in every lane of the row (all lanes active)
template <int AT>
__device__ __forceinline__ float row_bcast(float x) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x150 + AT, 0xF, 0xF, true));
}

// Component C of a record that lies two components per lane in the lanes of a row
template <int C>
__device__ __forceinline__ float row_comp(const float (&x)[2]) {
    return row_bcast<C / 2>(x[C & 1]);
}

// Terms J_p^T f of a pair, rounded as the one-pass form rounds them
template <int DP, int... K>
__device__ __forceinline__ void pair_terms(const float (&x)[2], float f0, float f1, float (&t)[DP],
                                           std::integer_sequence<int, K...>) {
    ((t[K] = fmaf(row_comp<K>(x), f0, row_comp<DP + K>(x) * f1)), ...);
}

// FP32 and BF16: the lane forms its pair's column terms and adds them in the wavefront's
// column sums in LDS.  The 16 lanes of an observation hold its record between them, two
// components each, and its F in lane 15; row broadcasts hand every lane the component that an
// operation needs.  Bound by the LDS atomics, which take 24 cycles of the CU each: their
// columns are scattered.  FP32 on the problem above 84 us with the whole record in every lane
// (six 1 KB loads for four observations), 79 us so; 111 us with a column per lane and the
// records in scalar registers, the terms of the subsets that do not see a landmark being work
// too.
template <int PREC, typename T, int DP, bool DIRECT>
__global__ __launch_bounds__(256) void k_pair_out(MultiArgs a, const void *__restrict__ records,
                                                  const uint2 *__restrict__ obs, const T *__restrict__ F,
                                                  const PairH<T> *__restrict__ H, double *__restrict__ partial) {
    if (a.skip && *a.skip != 0.0) return;
    constexpr int kLanes = DP + 3;                // lanes that hold a pair of components
    constexpr int kPairWords = PREC == 1 ? 2 : 1;    // 4-byte words of a pair
    constexpr int kRecWords = Stream<PREC, DP>::kWords * 4;
    static_assert(kLanes < 16, "lane 15 of a row holds F");
    __shared__ double sh[4][DP][64];
    const int lane = threadIdx.x & 63, i = lane & 15, o = lane >> 4;
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const PairShare me = pair_share(a, blockIdx.x, w);
    if (a.seg_skip && a.seg_skip[a.cam_seg[me.c]]) return;
    const int lo = me.lo, hi = me.hi;
    const int own = a.group[me.c];
    const int e = (i < kLanes ? i : 0) * kPairWords;   // the lane's first 4-byte word of a record
    const uint32_t *rec = reinterpret_cast<const uint32_t *>(records) +
                          (DIRECT ? (e & ~3) * kTile + (e & 3) : me.b0 * kRecWords + e);
    obs += me.b0;
#pragma unroll
    for (int k = 0; k < DP; ++k) sh[w][k][lane] = 0.0;
    wave_sync();
    struct Group {
        uint2 x;      // FP32: the lane's two components, lane 15: F
        float f[2];   // BF16: F
        PairH<T> h;
        int cnt;
        uint32_t first;
    };
    auto words = [&](int j) { return obs[min(j + o, hi - 1)]; };
    auto load = [&](int j, const uint2 &d, Group &g) {
        const int at = min(j + o, hi - 1);
        const uint32_t slot = (d.x & ~63u) | (d.y & 63u);
        const uint32_t *r = rec + (DIRECT ? (int64_t)(slot >> 6) * (kRecWords * kTile) + (slot & 63u) * 4
                                          : (int64_t)at * kRecWords);
        const uint32_t *f = reinterpret_cast<const uint32_t *>(F + (int64_t)slot * 2);
        if constexpr (PREC == 1) {
            g.x = *reinterpret_cast<const uint2 *>(i == 15 ? f : r);
        } else {
            g.x.x = *r;
            const uint2 fw = *reinterpret_cast<const uint2 *>(f);
            g.f[0] = __uint_as_float(fw.x);
            g.f[1] = __uint_as_float(fw.y);
        }
        g.cnt = j + o < hi ? (int)(d.y >> 8) : 0;
        g.first = d.x;
        g.h = H[d.x + (i < g.cnt ? i : 0)];
    };
    auto add = [&](Group &g) {
        float x[2], fo[2];
        if constexpr (PREC == 1) {
            x[0] = __uint_as_float(g.x.x);
            x[1] = __uint_as_float(g.x.y);
            fo[0] = row_bcast<15>(x[0]);
            fo[1] = row_bcast<15>(x[1]);
        } else {
            x[0] = bf16_to_f32(g.x.x & 0xFFFFu);
            x[1] = bf16_to_f32(g.x.x >> 16);
            fo[0] = g.f[0];
            fo[1] = g.f[1];
        }
        for (int p = i;;) {
            // every lane takes part up to here: the broadcasts read their neighbours
            const float l0[3] = {row_comp<2 * DP>(x), row_comp<2 * DP + 1>(x), row_comp<2 * DP + 2>(x)};
            const float l1[3] = {row_comp<2 * DP + 3>(x), row_comp<2 * DP + 4>(x), row_comp<2 * DP + 5>(x)};
            float f0 = dot3(l0, g.h.h), f1 = dot3(l1, g.h.h);
            if (g.h.grp == own) {
                f0 = fo[0];
                f1 = fo[1];
            }
            float t[DP];
            pair_terms<DP>(x, f0, f1, t, std::make_integer_sequence<int, DP>());
            if (p < g.cnt) {
#pragma unroll
                for (int k = 0; k < DP; ++k) atomicAdd(&sh[w][k][g.h.grp], (double)t[k]);
            }
            p += 16;
            if (!__any(p < g.cnt)) break;
            g.h = H[g.first + (p < g.cnt ? p : 0)];
        }
    };
    if (lo < hi) {
        Group A, B;
        load(lo, words(lo), A);
        uint2 d = words(lo + 4);
        int j = lo;
        for (; j + 4 < hi; j += 8) {
            load(j + 4, d, B);
            d = words(j + 8);
            add(A);
            load(j + 8, d, A);
            d = words(j + 12);
            add(B);
        }
        if (j < hi) add(A);
    }
    pair_store<DP>(sh, a.N, partial);
}

typedef double dbl4_t __attribute__((ext_vector_type(4)));

// x of lane `AT` of the lane's row of 16, in every lane of the row
template <int AT>
__device__ __forceinline__ double row_bcast(double x) {
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(x), 0x150 + AT, 0xF, 0xF, true);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(x), 0x150 + AT, 0xF, 0xF, true);
    return __hiloint2double(hi, lo);
}

// FP64, on the matrix cores: lane (o, i) of v_mfma_f64_16x16x4f64 supplies
// A[i][o] = J_p,o[row][i] and B[o][i] = f_{o, column}[row], NT tiles of 16 columns, one
// product per row and tile.  J_l rides in the lanes past DP of the first row's load, F in lane
// 15, and DPP hands them to the row; the pairs' f go to their columns through LDS (98 us on
// the problem above; with f formed per column from gathered h 112 us, a column per lane with
// FMAs and scalar loads 141 us).
template <int DP, int NT, bool DIRECT>
__global__ __launch_bounds__(256) void k_pair_out_mfma(MultiArgs a, const double *__restrict__ records,
                                                       const uint2 *__restrict__ obs,
                                                       const double *__restrict__ F,
                                                       const PairH<double> *__restrict__ H,
                                                       double *__restrict__ partial) {
    if (a.skip && *a.skip != 0.0) return;
    constexpr int NV = 2 * DP + 6;
    __shared__ double sh[4][DP][64];
    __shared__ double fsh[4][4][2][16 * NT];
    const int lane = threadIdx.x & 63, i = lane & 15, o = lane >> 4;
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const PairShare me = pair_share(a, blockIdx.x, w);
    if (a.seg_skip && a.seg_skip[a.cam_seg[me.c]]) return;
    const int lo = me.lo, hi = me.hi;
    const int own = a.group[me.c];
    // record values of the lane: J_p row 0 (i < DP), then J_l; J_p row 1; lane 15: F
    const int e0 = i < DP ? i : i < DP + 6 ? DP + i : 0, e1 = DP + (i < DP ? i : 0);
    const double *rec0 = records + (DIRECT ? (e0 & ~1) * kTile + (e0 & 1) : me.b0 * NV + e0);
    const double *rec1 = records + (DIRECT ? (e1 & ~1) * kTile + (e1 & 1) : me.b0 * NV + e1);
    obs += me.b0;
    double (*fc)[2][16 * NT] = fsh[w];
#pragma unroll
    for (int q = 0; q < NT; ++q) fc[o][0][16 * q + i] = fc[o][1][16 * q + i] = 0.0;
    wave_sync();
    dbl4_t acc[NT];
#pragma unroll
    for (int q = 0; q < NT; ++q) acc[q] = dbl4_t{0.0, 0.0, 0.0, 0.0};
    struct Group {
        double x0, x1;
        PairH<double> h;
        int cnt;
        uint32_t first;
    };
    auto words = [&](int j) { return obs[min(j + o, hi - 1)]; };
    auto load = [&](int j, const uint2 &d, Group &g) {
        const uint32_t slot = (d.x & ~63u) | (d.y & 63u);
        const int64_t at = DIRECT ? (int64_t)(slot >> 6) * (NV * kTile) + (slot & 63u) * 2 : (int64_t)min(j + o, hi - 1) * NV;
        const double *fp = F + (int64_t)slot * 2;
        g.x0 = *(i == 15 ? fp : rec0 + at);
        g.x1 = *(i == 15 ? fp + 1 : rec1 + at);
        g.cnt = j + o < hi ? (int)(d.y >> 8) : 0;   // past the share: no pair, so f = 0
        g.first = d.x;
        g.h = H[d.x + (i < g.cnt ? i : 0)];
    };
    auto add = [&](Group &g) {
        const double l0 = row_bcast<DP + 0>(g.x0), l1 = row_bcast<DP + 1>(g.x0), l2 = row_bcast<DP + 2>(g.x0);
        const double l3 = row_bcast<DP + 3>(g.x0), l4 = row_bcast<DP + 4>(g.x0), l5 = row_bcast<DP + 5>(g.x0);
        const double own0 = row_bcast<15>(g.x0), own1 = row_bcast<15>(g.x1);
        auto put = [&](int p, double f0, double f1) {
            if (p < g.cnt) {
                fc[o][0][g.h.grp] = f0;
                fc[o][1][g.h.grp] = f1;
            }
        };
        auto pair = [&](int p) {
            const double f0 = l0 * g.h.h[0] + l1 * g.h.h[1] + l2 * g.h.h[2];
            const double f1 = l3 * g.h.h[0] + l4 * g.h.h[1] + l5 * g.h.h[2];
            const bool mine = g.h.grp == own;
            put(p, mine ? own0 : f0, mine ? own1 : f1);
        };
        const int64_t grp = g.h.grp;
        pair(i);
        bool more = false;
        for (int p = i + 16; __any(p < g.cnt); p += 16) {
            more = true;
            g.h = H[g.first + (p < g.cnt ? p : 0)];
            pair(p);
        }
        wave_sync();
#pragma unroll
        for (int q = 0; q < NT; ++q) {
            acc[q] = __builtin_amdgcn_mfma_f64_16x16x4f64(g.x0, fc[o][0][16 * q + i], acc[q], 0, 0, 0);
            acc[q] = __builtin_amdgcn_mfma_f64_16x16x4f64(g.x1, fc[o][1][16 * q + i], acc[q], 0, 0, 0);
        }
        wave_sync();
        // the columns are zero again before the next four observations
        if (more) {
#pragma unroll
            for (int q = 0; q < NT; ++q) fc[o][0][16 * q + i] = fc[o][1][16 * q + i] = 0.0;
        } else if (i < g.cnt) {
            fc[o][0][grp] = 0.0;
            fc[o][1][grp] = 0.0;
        }
        wave_sync();
    };
    if (lo < hi) {   // four observations in flight while four are added, their words earlier still
        Group A, B;
        load(lo, words(lo), A);
        uint2 d = words(lo + 4);
        int j = lo;
        for (; j + 4 < hi; j += 8) {
            load(j + 4, d, B);
            d = words(j + 8);
            add(A);
            load(j + 8, d, A);
            d = words(j + 12);
            add(B);
        }
        if (j < hi) add(A);
    }
#pragma unroll
    for (int q = 0; q < NT; ++q)
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (o + 4 * e < DP) sh[w][o + 4 * e][16 * q + i] = acc[q][e];
    pair_store<DP>(sh, a.N, partial);
}

template <int DP, bool DIRECT>
static void launch_pair_out_mfma(const MultiArgs &a, const void *records, hipStream_t s) {
    const dim3 g((unsigned)a.n_blocks), b(256);
    const double *rec = reinterpret_cast<const double *>(records);
    const double *F = reinterpret_cast<const double *>(a.pair_f);
    const PairH<double> *H = reinterpret_cast<const PairH<double> *>(a.pair_h);
    switch ((a.N + 15) / 16) {
    case 1: hipLaunchKernelGGL((k_pair_out_mfma<DP, 1, DIRECT>), g, b, 0, s, a, rec, a.pair_obs, F, H, a.pair_partial); break;
    case 2: hipLaunchKernelGGL((k_pair_out_mfma<DP, 2, DIRECT>), g, b, 0, s, a, rec, a.pair_obs, F, H, a.pair_partial); break;
    case 3: hipLaunchKernelGGL((k_pair_out_mfma<DP, 3, DIRECT>), g, b, 0, s, a, rec, a.pair_obs, F, H, a.pair_partial); break;
    default: hipLaunchKernelGGL((k_pair_out_mfma<DP, 4, DIRECT>), g, b, 0, s, a, rec, a.pair_obs, F, H, a.pair_partial);
    }
}

// Y[p][c] = [group(c) == p] lambda diag(U_c) z_c + sum of camera c's blocks, in order:
// wavefront w of the work-group of (c, component) adds blocks w, w + 4, ..., lane p column p.
template <int DP>
__global__ __launch_bounds__(256) void k_pair_reduce(MultiArgs a, const double *__restrict__ partial,
                                                     const double *__restrict__ z, double *__restrict__ Y) {
    if (a.skip && *a.skip != 0.0) return;
    const int c = blockIdx.x / DP, k = blockIdx.x - c * DP;
    if (a.seg_skip && a.seg_skip[a.cam_seg[c]]) return;
    __shared__ double sh[4][64];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int b1 = a.cam_blk[c + 1], N = a.N;
    const double *p0 = partial + (int64_t)k * N + (lane < N ? lane : 0);
    double s = 0.0;
    for (int b = a.cam_blk[c] + w; b < b1; b += 32) {
        double v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = p0[(int64_t)(b + 4 * u < b1 ? b + 4 * u : b) * DP * N];
#pragma unroll
        for (int u = 0; u < 8; ++u)
            if (b + 4 * u < b1) s += v[u];
    }
    sh[w][lane] = s;
    __syncthreads();
    if (w == 0 && lane < N) {
        const int64_t row = (int64_t)c * DP + k;
        const double t = (sh[0][lane] + sh[1][lane]) + (sh[2][lane] + sh[3][lane]);
        Y[(int64_t)lane * a.np * DP + row] = (a.group[c] == lane ? a.dU[row] * z[row] : 0.0) + t;
    }
}

// Camera-major copy of the tile stream: 16-byte word q of the i-th observation of the
// camera order goes to word i kw + q (consecutive threads take consecutive words; a thread
// takes several where there are more words than a launch has threads).
__global__ __launch_bounds__(256) void k_pair_records(int64_t m, int kw, const uint32_t *__restrict__ cam_slot,
                                                      const u32x4_t *__restrict__ J, u32x4_t *__restrict__ out) {
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < m * kw; i += (int64_t)gridDim.x * 256) {
        const int64_t o = i / kw;
        const int q = (int)(i - o * kw);
        const int64_t s = cam_slot[o];
        out[i] = J[(s / kTile * kw + q) * kTile + s % kTile];
    }
}

void launch_pair_records(int64_t m, int precision, int dp, const uint32_t *cam_slot, const void *J, void *out,
                         hipStream_t s) {
    const int kw = record_words(precision, dp);
    const int64_t blocks = std::min<int64_t>((m * kw + 255) / 256, 1 << 23);
    hipLaunchKernelGGL(k_pair_records, dim3((unsigned)blocks), dim3(256), 0, s, m, kw, cam_slot,
                       reinterpret_cast<const u32x4_t *>(J), reinterpret_cast<u32x4_t *>(out));
}

// pair_obs of every observation, in camera order (see k_pair_out).
__global__ __launch_bounds__(256) void k_pair_obs(int64_t m, const uint32_t *__restrict__ cam_slot,
                                                  const uint32_t *__restrict__ mmeta, uint2 *__restrict__ obs) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= m) return;
    const uint32_t s = cam_slot[i], mm = mmeta[s];
    obs[i] = make_uint2((s & ~63u) + ((mm >> 8) & 0xFFu), (s & 63u) | ((mm >> 16) & 0xFFu) << 8);
}

void launch_pair_obs(int64_t m, const uint32_t *cam_slot, const uint32_t *mmeta, uint2 *obs, hipStream_t s) {
    hipLaunchKernelGGL(k_pair_obs, dim3((unsigned)((m + 255) / 256)), dim3(256), 0, s, m, cam_slot, mmeta, obs);
}

template <int PREC, typename T, int DP, bool DIRECT>
static void launch_pair_out(const MultiArgs &a, const void *records, hipStream_t s) {
    if constexpr (PREC == 0)
        launch_pair_out_mfma<DP, DIRECT>(a, records, s);
    else
        hipLaunchKernelGGL((k_pair_out<PREC, T, DP, DIRECT>), dim3((unsigned)a.n_blocks), dim3(256), 0, s, a, records,
                           a.pair_obs, reinterpret_cast<const T *>(a.pair_f),
                           reinterpret_cast<const PairH<T> *>(a.pair_h), a.pair_partial);
}

template <int PREC, typename T, int DP>
static void launch_two_pass(const MultiArgs &a, const double *z, double *Y, hipStream_t s) {
    hipLaunchKernelGGL((k_pair_h<PREC, T, DP>), dim3((unsigned)((a.n_tiles + 3) / 4)), dim3(256), 0, s, a, z);
    if (a.records) launch_pair_out<PREC, T, DP, false>(a, a.records, s);
    else launch_pair_out<PREC, T, DP, true>(a, a.J, s);
    hipLaunchKernelGGL(k_pair_reduce<DP>, dim3((unsigned)(a.np * DP)), dim3(256), 0, s, a, a.pair_partial, z, Y);
}

void launch_schur_multi(const MultiArgs &a, const double *z, double *Y, hipStream_t s) {
    if (a.two_pass) {
        if (a.dp == 6) {
            switch (a.precision) {
                case 0: launch_two_pass<0, double, 6>(a, z, Y, s); break;
                case 1: launch_two_pass<1, float, 6>(a, z, Y, s); break;
                default: launch_two_pass<2, float, 6>(a, z, Y, s); break;
            }
        } else {
            switch (a.precision) {
                case 0: launch_two_pass<0, double, 9>(a, z, Y, s); break;
                case 1: launch_two_pass<1, float, 9>(a, z, Y, s); break;
                default: launch_two_pass<2, float, 9>(a, z, Y, s); break;
            }
        }
        return;
    }
    if (a.n_chunks > 0) {
        const size_t lds = (size_t)(a.max_out * a.dp + 6 * kTile) * sizeof(double);
        const dim3 g(a.n_chunks), b(kTile);
        if (a.dp == 6) {
            switch (a.precision) {
                case 0: hipLaunchKernelGGL((k_schur_multi<0, double, 6>), g, b, lds, s, a, z); break;
                case 1: hipLaunchKernelGGL((k_schur_multi<1, float, 6>), g, b, lds, s, a, z); break;
                default: hipLaunchKernelGGL((k_schur_multi<2, float, 6>), g, b, lds, s, a, z); break;
            }
        } else {
            switch (a.precision) {
                case 0: hipLaunchKernelGGL((k_schur_multi<0, double, 9>), g, b, lds, s, a, z); break;
                case 1: hipLaunchKernelGGL((k_schur_multi<1, float, 9>), g, b, lds, s, a, z); break;
                default: hipLaunchKernelGGL((k_schur_multi<2, float, 9>), g, b, lds, s, a, z); break;
            }
        }
    }
    const int64_t keys = (int64_t)a.np * a.N;
    const dim3 g((unsigned)((keys + 3) / 4));
    if (a.dp == 6)
        hipLaunchKernelGGL(k_reduce_multi<6>, g, dim3(256), 0, s, a.np, a.N, a.cg_ptr, a.partial, a.dU, a.group, z, Y,
                           a.cam_seg, a.seg_skip, a.skip);
    else
        hipLaunchKernelGGL(k_reduce_multi<9>, g, dim3(256), 0, s, a.np, a.N, a.cg_ptr, a.partial, a.dU, a.group, z, Y,
                           a.cam_seg, a.seg_skip, a.skip);
}

// ---------------------------------------------------------------- eq. (16)

// dx_l = -V^-1 (b_l + W^T dx_p) for every landmark; the first observation of a
// landmark inside its tile writes the result.  A work-group of up to eight wavefronts takes a
// chunk, its cameras' rows of dx_p in LDS, and each wavefront a share of its tiles: the
// product's few chunks would leave too few wavefronts.  Bound by latency and the landmarks'
// scattered values: 1,936 cameras, 5.08M observations 188 -> 186 us against a wavefront per
// chunk of 2,961, a dense cap of 571 cameras 52 -> 48 us with the call; with the next tile
// requested ahead (one landmark per lane) no faster and 55 us on the cap.
constexpr int kBackWaves = 8;
template <int DP>
__global__ __launch_bounds__(64 * kBackWaves) void k_backsub(const double *__restrict__ J64, const uint32_t *__restrict__ meta,
                                                 const int32_t *__restrict__ tile_lmk_base,
                                                 const int32_t *__restrict__ chunk_tile,
                                                 const int32_t *__restrict__ chunk_part,
                                                 const int32_t *__restrict__ part_cam, int max_slots,
                                                 const double *__restrict__ vinv, const double *__restrict__ bl,
                                                 const int32_t *__restrict__ lmk_order,
                                                 const double *__restrict__ dxp, double *__restrict__ dxl) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int chunk = blockIdx.x, waves = blockDim.x / kTile;
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    double *vloc = reinterpret_cast<double *>(smem);
    double *gloc = vloc + max_slots * DP + w * 3 * kTile;
    const int pb = chunk_part[chunk];
    const int ns = chunk_part[chunk + 1] - pb;
    const int c0 = chunk_tile[chunk], len = chunk_tile[chunk + 1] - c0;
    for (int i = threadIdx.x; i < ns * DP; i += blockDim.x) vloc[i] = dxp[(int64_t)part_cam[pb + i / DP] * DP + i % DP];
    __syncthreads();
    for (int t = c0 + len * w / waves; t < c0 + len * (w + 1) / waves; ++t) {
        double J[2 * DP + 6];
        Loader<0, DP>::load(J64, t, lane, J);
        const uint32_t mt = meta[(int64_t)t * kTile + lane];
        const bool valid = mt != kPad;
        const int slot = valid ? (int)(mt & 0xFFFFu) : 0;
        const int ll = valid ? (int)((mt >> 16) & 63u) : 0;
        const uint32_t prev = lane > 0 ? meta[(int64_t)t * kTile + lane - 1] : kPad;
        const bool first = valid && (prev == kPad || ((prev >> 16) & 63u) != (uint32_t)ll);
        double e0 = 0, e1 = 0;
#pragma unroll
        for (int k = 0; k < DP; ++k) {
            e0 += J[k] * vloc[slot * DP + k];
            e1 += J[DP + k] * vloc[slot * DP + k];
        }
        gloc[lane * 3 + 0] = 0;
        gloc[lane * 3 + 1] = 0;
        gloc[lane * 3 + 2] = 0;
        wave_sync();
        if (valid)
            for (int k = 0; k < 3; ++k) atomicAdd(&gloc[ll * 3 + k], J[2 * DP + k] * e0 + J[2 * DP + 3 + k] * e1);
        wave_sync();
        if (first) {
            const int64_t ls = tile_lmk_base[t] + ll;
            const double *vi = vinv + ls * 6;
            const double g0 = gloc[ll * 3] + bl[ls * 3], g1 = gloc[ll * 3 + 1] + bl[ls * 3 + 1],
                         g2 = gloc[ll * 3 + 2] + bl[ls * 3 + 2];
            double *o = dxl + (int64_t)lmk_order[ls] * 3;
            o[0] = -(vi[0] * g0 + vi[1] * g1 + vi[2] * g2);
            o[1] = -(vi[1] * g0 + vi[3] * g1 + vi[4] * g2);
            o[2] = -(vi[2] * g0 + vi[4] * g1 + vi[5] * g2);
        }
        wave_sync();   // the landmark rows are reset by the next tile
    }
}

void launch_back_substitute(const double *J64, const uint32_t *meta, const int32_t *tile_lmk_base,
                            const int32_t *chunk_tile, const int32_t *chunk_part, const int32_t *part_cam,
                            int n_chunks, int max_slots, int max_tiles, const double *vinv, const double *bl,
                            const int32_t *lmk_order, const double *dxp, double *dxl, hipStream_t s, int dp) {
    if (n_chunks <= 0) return;
    const int waves = std::min(kBackWaves, std::max(1, max_tiles));
    const size_t lds = (size_t)(max_slots * dp + waves * 3 * kTile) * sizeof(double);
    auto kernel = dp == 6 ? k_backsub<6> : k_backsub<9>;
    hipLaunchKernelGGL(kernel, dim3(n_chunks), dim3(waves * kTile), lds, s, J64, meta, tile_lmk_base, chunk_tile,
                       chunk_part, part_cam, max_slots, vinv, bl, lmk_order, dxp, dxl);
}

// Chunk wavefronts of a kernel the device keeps resident at once (register-limited
// occupancy times compute units); 0 when it cannot be queried
static int resident_waves(const void *f) {
    int dev = 0, cus = 0, per = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, f, kTile, 0) != hipSuccess)
        return 0;
    return per * cus;
}

int schur1_resident_chunks(int dp) {
    return resident_waves(dp == 6 ? reinterpret_cast<const void *>(&k_schur1<0, double, 6>)
                                  : reinterpret_cast<const void *>(&k_schur1<0, double, 9>));
}

int schur1_few_chunks() {
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
        return 0;
    return 3 * cus * 31 / 32;
}

int schur_multi_resident_chunks(int dp) {
    return resident_waves(dp == 6 ? reinterpret_cast<const void *>(&k_schur_multi<0, double, 6>)
                                  : reinterpret_cast<const void *>(&k_schur_multi<0, double, 9>));
}

}  // namespace ba
