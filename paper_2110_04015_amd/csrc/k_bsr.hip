// Explicit reduced camera system in block-sparse rows (9 x 9 FP64 blocks), the
// paper's own representation of S (Sec. 3.2, "Optimized implementation": S_jk is
// nonzero iff cameras j and k observe a common point; Sec. 4.1 forms it as a
// row-major sparse matrix).
//
// Value layout of block row j (nb blocks, starting at block b0 = row_ptr[j]): the 81 nb
// values at val + 81 b0 are stored row-of-the-block-major, [r][t][c] = S_(j, col t)[r][c]
// at r (9 nb) + 9 t + c.  Each of the nine rows r of the block row is then one contiguous
// run of 9 nb values, multiplied entry by entry with the same gathered vector
// (v_(col t))_c, which the products load once for all nine.
//   S_jj = D(S)_j                                   (already formed by the build)
//   S_jk = - sum_{l observed by j and k} W_jl V_l^-1 W_kl^T,   W_jl = J_p,jl^T J_l,jl
// Assembly: one wavefront per kBsrPiece blocks of a row holds them in LDS and adds their
// contributions, 64 at a time, in a fixed order.
#include "ba_internal.h"
#include "kernels.h"
#include "dev_la.h"

namespace ba {

typedef double dbl2b_t __attribute__((ext_vector_type(2)));

// ---- pattern on the device: row j's columns are the cameras that share a landmark
// with camera j (j included).  One work-group per row marks them in an LDS bitmap of
// n_cams bits (every observation o of camera j, then every observation slot of o's
// landmark); the set bits, read in word order, are the row's columns in ascending order.
__device__ void row_bitmap(int j, const int64_t *__restrict__ cam_ptr, const int64_t *__restrict__ cam_obs,
                           const int32_t *__restrict__ obs_lm, const int32_t *__restrict__ lmk_store,
                           const int64_t *__restrict__ lmk_first_slot, const int32_t *__restrict__ lmk_count,
                           const int32_t *__restrict__ slot_cam, int nwords, uint32_t *bm) {
    for (int w = threadIdx.x; w < nwords; w += blockDim.x) bm[w] = 0u;
    __syncthreads();
    for (int64_t u = cam_ptr[j] + threadIdx.x; u < cam_ptr[j + 1]; u += blockDim.x) {
        const int s = lmk_store[obs_lm[cam_obs[u]]];
        const int64_t f = lmk_first_slot[s];
        const int c = lmk_count[s];
        for (int q = 0; q < c; ++q) {
            const int k = slot_cam[f + q];
            atomicOr(&bm[k >> 5], 1u << (k & 31));
        }
    }
    __syncthreads();
}

__global__ __launch_bounds__(256) void k_bsr_rowcount(int nwords, const int64_t *__restrict__ cam_ptr,
                                                      const int64_t *__restrict__ cam_obs,
                                                      const int32_t *__restrict__ obs_lm,
                                                      const int32_t *__restrict__ lmk_store,
                                                      const int64_t *__restrict__ lmk_first_slot,
                                                      const int32_t *__restrict__ lmk_count,
                                                      const int32_t *__restrict__ slot_cam, int32_t *__restrict__ nnz) {
    extern __shared__ uint32_t bm[];
    __shared__ int part[256 / 64];
    const int j = blockIdx.x;
    row_bitmap(j, cam_ptr, cam_obs, obs_lm, lmk_store, lmk_first_slot, lmk_count, slot_cam, nwords, bm);
    int c = 0;
    for (int w = threadIdx.x; w < nwords; w += blockDim.x) c += __popc(bm[w]);
    for (int o = 32; o > 0; o >>= 1) c += __shfl_xor(c, o, 64);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = c;
    __syncthreads();
    if (threadIdx.x == 0) nnz[j] = part[0] + part[1] + part[2] + part[3];
}

// Writes row j's columns (ascending) at col[row_ptr[j] ...]: words are taken 256 at a
// time, each thread's set bits go after the set bits of the words before it.
__global__ __launch_bounds__(256) void k_bsr_rowfill(int nwords, const int64_t *__restrict__ cam_ptr,
                                                     const int64_t *__restrict__ cam_obs,
                                                     const int32_t *__restrict__ obs_lm,
                                                     const int32_t *__restrict__ lmk_store,
                                                     const int64_t *__restrict__ lmk_first_slot,
                                                     const int32_t *__restrict__ lmk_count,
                                                     const int32_t *__restrict__ slot_cam,
                                                     const int32_t *__restrict__ row_ptr, int32_t *__restrict__ col) {
    extern __shared__ uint32_t bm[];
    __shared__ int scan[256];
    const int j = blockIdx.x;
    row_bitmap(j, cam_ptr, cam_obs, obs_lm, lmk_store, lmk_first_slot, lmk_count, slot_cam, nwords, bm);
    int base = row_ptr[j];
    for (int w0 = 0; w0 < nwords; w0 += 256) {
        const int w = w0 + (int)threadIdx.x;
        const uint32_t bits = w < nwords ? bm[w] : 0u;
        scan[threadIdx.x] = __popc(bits);
        __syncthreads();
        for (int o = 1; o < 256; o <<= 1) {   // inclusive scan (Hillis-Steele)
            const int add = (int)threadIdx.x >= o ? scan[threadIdx.x - o] : 0;
            __syncthreads();
            scan[threadIdx.x] += add;
            __syncthreads();
        }
        int pos = base + scan[threadIdx.x] - __popc(bits);
        for (uint32_t b = bits; b; b &= b - 1) col[pos++] = w * 32 + __ffs(b) - 1;
        base += scan[255];
        __syncthreads();
    }
}

// One wavefront per piece, at most kBsrPiece consecutive blocks of a block row j, the piece's
// blocks in LDS.  It goes through camera j's observations o (of landmark l) 64 at a time and
// queues the pairs (o, q) with the other observations q of l whose camera's block lies in the
// piece; whenever 64 are queued, a lane takes each and adds -W_o V_l^-1 W_q^T = -J_p,o^T B
// J_p,q, B = J_l,o V_l^-1 J_l,q^T, into the block.  One wavefront issues all the LDS atomics
// of a block, so they resolve in program order and, within an instruction, in lane order: the
// sums are reproducible.  Every piece goes through the row's observations.  The diagonal block
// is D(S)_j.
// Bound by the latency of the scattered record loads, so pieces are small (many wavefronts per
// compute unit, where a piece of all the blocks that LDS holds left one) and the lanes work on
// queued pairs (with 8 blocks few of an observation's pairs are wanted).  The pieces are
// listed, so that a row takes no work-groups but its own however wide the widest row is.  A
// dense cap of 571
// cameras (897k observations, 257k blocks) 100 -> 16.5 ms, of 120 17.8 -> 2.8, 1,936
// cameras along a walk 19.4 -> 8.0, a ring of 333 3.3 -> 1.4 (ba_set_lambda).  A row's pieces
// each go through its observations, so the work grows with the square of a row's width; it
// stays ahead of pieces of 250 blocks in the widest rows tried: 1,500 cameras dense (740 blocks
// a row) 326 -> 53 ms, 1,000 cameras with every row full 45.8 -> 29.6, one camera covisible with
// 20,000 others 9.5 -> 0.9.
__global__ __launch_bounds__(64) void k_bsr_assemble(const int64_t *__restrict__ cam_ptr,
                                                     const uint32_t *__restrict__ cam_slot,
                                                     const int32_t *__restrict__ cam_lmk,
                                                     const int64_t *__restrict__ lmk_first_slot,
                                                     const int32_t *__restrict__ lmk_count,
                                                     const int32_t *__restrict__ slot_cam,
                                                     const double *__restrict__ J64, const double *__restrict__ vinv,
                                                     const double *__restrict__ Dblk,
                                                     const int32_t *__restrict__ row_ptr,
                                                     const int2 *__restrict__ pieces,
                                                     const int32_t *__restrict__ col, double *__restrict__ val) {
    __shared__ double acc[kBsrPiece * 81];
    __shared__ int32_t rc[kBsrPiece];                 // the piece's columns, ascending
    __shared__ uint64_t queue[64 * (kBsrPiece + 1)];  // pairs: o << 6 | q, o in the camera order
    const int lane = threadIdx.x;
    const int j = pieces[blockIdx.x].x, pb = pieces[blockIdx.x].y;   // the row, the piece's first block in it
    const int b0 = row_ptr[j], nb = row_ptr[j + 1] - b0;
    const int pn = min(kBsrPiece, nb - pb);
    for (int e = lane; e < pn * 81; e += 64) acc[e] = 0.0;
    if (lane < pn) rc[lane] = col[b0 + pb + lane];
    auto lds_order = [] {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    };
    lds_order();
    const int kfirst = rc[0], klast = rc[pn - 1];
    // block of column k in the piece (present: k lies in its range and in the row)
    auto block_of = [&](int k) {
        int lo = 0, hi = pn - 1;
        while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if (rc[mid] < k) lo = mid + 1;
            else hi = mid;
        }
        return lo;
    };
    auto add_pair = [&](uint64_t e) {
        const int64_t u = (int64_t)(e >> 6);
        const int64_t l = cam_lmk[u], sq = lmk_first_slot[l] + (int64_t)(e & 63u), so = cam_slot[u];
        const dbl2b_t *po = reinterpret_cast<const dbl2b_t *>(J64) + (so >> 6) * 12 * 64 + (so & 63);
        const dbl2b_t *pq = reinterpret_cast<const dbl2b_t *>(J64) + (sq >> 6) * 12 * 64 + (sq & 63);
        double a[24], c[24];
#pragma unroll
        for (int q = 0; q < 12; ++q) {
            const dbl2b_t d = po[q * 64], g = pq[q * 64];
            a[2 * q] = d.x;
            a[2 * q + 1] = d.y;
            c[2 * q] = g.x;
            c[2 * q + 1] = g.y;
        }
        const double *vi = vinv + l * 6;
        const double v0 = vi[0], v1 = vi[1], v2 = vi[2], v3 = vi[3], v4 = vi[4], v5 = vi[5];
        double *blk = acc + (size_t)block_of(slot_cam[sq]) * 81;
        double B[2][2];
#pragma unroll
        for (int m = 0; m < 2; ++m) {   // row m of J_l,o V^-1 (V^-1 symmetric, packed), times J_l,q^T
            const double x0 = a[18 + 3 * m], x1 = a[19 + 3 * m], x2 = a[20 + 3 * m];
            const double t0 = x0 * v0 + x1 * v1 + x2 * v2;
            const double t1 = x0 * v1 + x1 * v3 + x2 * v4;
            const double t2 = x0 * v2 + x1 * v4 + x2 * v5;
            B[m][0] = t0 * c[18] + t1 * c[19] + t2 * c[20];
            B[m][1] = t0 * c[21] + t1 * c[22] + t2 * c[23];
        }
#pragma unroll
        for (int r = 0; r < 9; ++r) {
            const double m0 = -(a[r] * B[0][0] + a[9 + r] * B[1][0]), m1 = -(a[r] * B[0][1] + a[9 + r] * B[1][1]);
#pragma unroll
            for (int cc = 0; cc < 9; ++cc) atomicAdd(&blk[r * 9 + cc], m0 * c[cc] + m1 * c[9 + cc]);
        }
    };
    const int64_t u1 = cam_ptr[j + 1];
    int queued = 0;   // uniform, below 64 between trips
    for (int64_t u0 = cam_ptr[j]; u0 < u1; u0 += 64) {
        const int64_t u = u0 + lane;
        uint64_t todo = 0;   // observations q of the landmark with a block here: at most pn of them
        if (u < u1) {
            const int s = cam_lmk[u];
            const int64_t f = lmk_first_slot[s];
            const int c = lmk_count[s];
            for (int q = 0; q < c; ++q) {
                const int k = slot_cam[f + q];
                if (k >= kfirst && k <= klast && k != j) todo |= 1ull << q;
            }
        }
        // queue places: lanes in order, a lane's pairs in slot order
        const int n = __popcll(todo);
        const uint64_t below = (1ull << lane) - 1;
        int at = queued, total = 0;
#pragma unroll
        for (int b = 0; (1 << b) <= kBsrPiece; ++b) {
            const uint64_t bits = __ballot((n >> b) & 1);
            at += __popcll(bits & below) << b;
            total += __popcll(bits) << b;
        }
        for (; todo; todo &= todo - 1) queue[at++] = (uint64_t)u << 6 | (uint64_t)(__ffsll((unsigned long long)todo) - 1);
        queued += total;
        lds_order();
        int done = 0;
        for (; done + 64 <= queued; done += 64) add_pair(queue[done + lane]);
        if (done > 0) {   // the rest to the front (fewer than 64)
            queued -= done;
            const uint64_t e = lane < queued ? queue[done + lane] : 0;
            lds_order();
            if (lane < queued) queue[lane] = e;
            lds_order();
        }
    }
    if (lane < queued) add_pair(queue[lane]);
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    // diagonal block: D(S)_j, formed by the build from the same sums
    const int lo = block_of(j);
    if (rc[lo] == j)
        for (int e = lane; e < 81; e += 64) acc[(size_t)lo * 81 + e] = Dblk[(int64_t)j * 81 + e];
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    // out in the row-of-the-block-major layout: run r holds 9 nb values
    const int64_t L = (int64_t)nb * 9;
    double *out = val + (int64_t)b0 * 81;
    for (int e = lane; e < pn * 81; e += 64) {
        const int t = e / 81, rc = e - t * 81, r = rc / 9, c = rc - r * 9;
        out[r * L + (int64_t)(pb + t) * 9 + c] = acc[e];
    }
}

// Loads of kBsrAhead positions e0 + STEP u of a block row (its nine runs of L values at S,
// columns cj): the nine values sv[u][r] = S[r L + e] and the gathered vector entry
// vg[u] = v[9 col(e / 9) + e mod 9]; with group, also gk[u] = group[col(e / 9)].
// Positions at or beyond `hi` (<= L) read nothing and give zeros.
constexpr int kBsrAhead = 4;

template <int STEP>
__device__ __forceinline__ void bsr_fetch(const double *__restrict__ S, const int32_t *__restrict__ cj,
                                          const double *__restrict__ v, int L, int hi, int e0,
                                          double (&sv)[kBsrAhead][9], double (&vg)[kBsrAhead], const int32_t *__restrict__ group = nullptr,
                                          int *gk = nullptr) {
    int k[kBsrAhead], c[kBsrAhead];
#pragma unroll
    for (int u = 0; u < kBsrAhead; ++u) {
        const int e = e0 + u * STEP;
        const int t = e < hi ? e / 9 : 0;
        c[u] = e - t * 9;
        k[u] = cj[t];
    }
#pragma unroll
    for (int u = 0; u < kBsrAhead; ++u) {
        const int e = e0 + u * STEP;
#pragma unroll
        for (int r = 0; r < 9; ++r) sv[u][r] = e < hi ? S[(int64_t)r * L + e] : 0.0;
    }
#pragma unroll
    for (int u = 0; u < kBsrAhead; ++u) {
        const bool ok = e0 + u * STEP < hi;
        vg[u] = ok ? v[(int64_t)k[u] * 9 + c[u]] : 0.0;
        if (group) gk[u] = group[k[u]];
    }
}

// y_j = sum_t S_(j, col t) v_(col t).  One work-group of 256 threads per block row; thread
// i takes positions e = i, i + 256, ... of the row's 9 nb entries per block row r (block t
// = e / 9, column c = e % 9): it gathers (v_(col t))_c once and multiplies it with the nine
// entries S[r][e], which the work-group reads as nine coalesced runs.  Each output row r
// is added over the lanes of a wavefront, then over the four wavefronts in a fixed order.
// With gram, row j also leaves gram[2 j] = y_j . v_j and gram[2 j + 1] = v_j . gr_j (the
// Gram products Q^T P and P^T r of a one-column block, Q = S P).  When `done` is set and
// nonzero, the launch does nothing.
__global__ __launch_bounds__(256) void k_bsr_mv(int np, const int32_t *__restrict__ row_ptr,
                                                const int32_t *__restrict__ col, const double *__restrict__ val,
                                                const double *__restrict__ v, double *__restrict__ y,
                                                const double *__restrict__ done, double *__restrict__ gram,
                                                const double *__restrict__ gr) {
    if (done && *done != 0.0) return;
    __shared__ double sh[4][9];
    const int j = blockIdx.x;
    const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63;
    const int b0 = row_ptr[j];
    const int L = (row_ptr[j + 1] - b0) * 9;
    const double *S = val + (int64_t)b0 * 81;
    const int32_t *cj = col + b0;
    double acc[9];
#pragma unroll
    for (int r = 0; r < 9; ++r) acc[r] = 0.0;
    // kBsrAhead positions per trip (e0, e0 + 256, ...), all their loads issued before the
    // first multiply; each thread still adds its positions in ascending order
    for (int e0 = tid; e0 < L; e0 += kBsrAhead * 256) {
        double sv[kBsrAhead][9], vg[kBsrAhead];
        bsr_fetch<256>(S, cj, v, L, L, e0, sv, vg);
#pragma unroll
        for (int u = 0; u < kBsrAhead; ++u)
#pragma unroll
            for (int r = 0; r < 9; ++r) acc[r] += sv[u][r] * vg[u];
    }
#pragma unroll
    for (int r = 0; r < 9; ++r) {
        const double t = wave_sum(acc[r]);
        if (lane == 0) sh[w][r] = t;
    }
    __syncthreads();
    if (tid >= 64) return;
    double yr = 0.0, qp = 0.0, pr = 0.0;
    if (tid < 9) {
        yr = (sh[0][tid] + sh[1][tid]) + (sh[2][tid] + sh[3][tid]);
        const int64_t i = (int64_t)j * 9 + tid;
        y[i] = yr;
        if (gram) {
            const double vi = v[i];
            qp = yr * vi;
            pr = vi * gr[i];
        }
    }
    if (!gram) return;   // the same for the whole launch
    qp = wave_sum(qp);
    pr = wave_sum(pr);
    if (tid == 0) {
        gram[2 * j] = qp;
        gram[2 * j + 1] = pr;
    }
}

// Sums of the nine values a[r] over the lanes of a wavefront: after two exchanges of halves
// each row of 16 lanes holds two of the first eight, after the third each 8 lanes one, so
// that eight sums take little more than the last three steps of one.  The sum of a[r] is
// returned in lane 8 r (r < 8) and in `last` (r = 8, every lane).
__device__ __forceinline__ double wave_sum9(const double (&a)[9], double &last) {
    double h[4], q[2];
#pragma unroll
    for (int r = 0; r < 4; ++r) h[r] = add_halves32(a[r], a[r + 4]);   // lanes >= 32: r + 4
#pragma unroll
    for (int r = 0; r < 2; ++r) q[r] = add_halves16(h[r], h[r + 2]);   // odd rows: r + 2
    const bool up = threadIdx.x & 8;
    const double keep = up ? q[1] : q[0], send = up ? q[0] : q[1];
    double x = keep + dpp_move<0x128>(send);   // row_ror:8; lanes 8..15 of a row: the second
    x += dpp_move<0x141>(x);                   // row_half_mirror
    x = quad_sum(x);
    last = wave_sum(a[8]);
    return x;
}

// Y[p][row of j] = sum over blocks t of row j with group(col t) == p of S_(j, col t) z_(col t)
// (the multidirectional product of eq. (19)'s input).  One work-group of 256 threads per
// block row, each wavefront a quarter of the row's positions in trips of 64 consecutive
// ones.  The subsets are ranges of consecutive cameras and a row's columns ascend, so a
// subset's positions follow each other: the lanes add their products for the current
// subset up, and only where the subset changes are the nine rows added over the lanes and
// into the wavefront's LDS row of that subset (any order of the subsets would do, each
// change just costs a reduction).  The four wavefronts' rows are then added in a fixed
// order.  Bound by reading S (8 bytes for one multiplication): 571 cameras, dense (211 MB),
// 47 subsets 36.6 us, 5.8 TB/s; 58.7 us with a segmented scan of every row in every trip.
__global__ __launch_bounds__(256) void k_bsr_mm_grouped(int np, int N, int64_t n, const int32_t *__restrict__ row_ptr,
                                                        const int32_t *__restrict__ col,
                                                        const double *__restrict__ val,
                                                        const int32_t *__restrict__ group,
                                                        const double *__restrict__ z, double *__restrict__ Y,
                                                        const double *__restrict__ skip) {
    if (skip && *skip != 0.0) return;
    __shared__ double yl[4][kMaxBlock * 9];
    const int j = blockIdx.x;
    const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63;
    for (int e = lane; e < N * 9; e += 64) yl[w][e] = 0.0;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    const int b0 = row_ptr[j];
    const int L = (row_ptr[j + 1] - b0) * 9;
    const double *S = val + (int64_t)b0 * 81;
    const int32_t *cj = col + b0;
    const int part = (L + 255) / 256 * 64;   // whole trips per wavefront
    const int lo = w * part, hi = min(L, lo + part);
    int cur = 0;   // the subset being added up (uniform)
    double acc[9];
#pragma unroll
    for (int r = 0; r < 9; ++r) acc[r] = 0.0;
    auto flush = [&]() {
        double last;
        const double x = wave_sum9(acc, last);
        if ((lane & 7) == 0) yl[w][cur * 9 + (lane >> 3)] += x;
        if (lane == 0) yl[w][cur * 9 + 8] += last;
#pragma unroll
        for (int r = 0; r < 9; ++r) acc[r] = 0.0;
    };
    for (int e0 = lo; e0 < hi; e0 += kBsrAhead * 64) {
        double sv[kBsrAhead][9], zg[kBsrAhead];
        int gk[kBsrAhead];
        bsr_fetch<64>(S, cj, z, L, hi, e0 + lane, sv, zg, group, gk);
#pragma unroll
        for (int u = 0; u < kBsrAhead; ++u) {
            const bool ok = e0 + u * 64 + lane < hi;
            uint64_t left = __ballot(ok);
            while (left) {   // once, and once more for every change of the subset
                const bool mine = ok && gk[u] == cur;
                if (mine) {
#pragma unroll
                    for (int r = 0; r < 9; ++r) acc[r] += sv[u][r] * zg[u];
                }
                left &= ~__ballot(mine);
                if (!left) break;
                flush();
                cur = __builtin_amdgcn_readlane(gk[u], __ffsll((unsigned long long)left) - 1);
            }
        }
    }
    flush();
    __syncthreads();
    for (int e = tid; e < N * 9; e += 256) {
        const int p = e / 9, rr = e - p * 9;
        Y[(int64_t)p * n + (int64_t)j * 9 + rr] = (yl[0][e] + yl[1][e]) + (yl[2][e] + yl[3][e]);
    }
}

void launch_bsr_rowcount(int np, const BsrGather &g, int32_t *nnz, hipStream_t s) {
    const int nwords = (np + 31) / 32;
    hipLaunchKernelGGL(k_bsr_rowcount, dim3(np), dim3(256), (size_t)nwords * 4, s, nwords, g.cam_ptr, g.cam_obs,
                       g.obs_lm, g.lmk_store, g.lmk_first_slot, g.lmk_count, g.slot_cam, nnz);
}

void launch_bsr_rowfill(int np, const BsrGather &g, const int32_t *row_ptr, int32_t *col, hipStream_t s) {
    const int nwords = (np + 31) / 32;
    hipLaunchKernelGGL(k_bsr_rowfill, dim3(np), dim3(256), (size_t)nwords * 4, s, nwords, g.cam_ptr, g.cam_obs,
                       g.obs_lm, g.lmk_store, g.lmk_first_slot, g.lmk_count, g.slot_cam, row_ptr, col);
}

void launch_bsr_assemble(const BsrGather &g, const uint32_t *cam_slot, const int32_t *cam_lmk, const double *J64,
                         const double *vinv, const double *Dblk, const int32_t *row_ptr, const int2 *pieces,
                         int64_t n_pieces, const int32_t *col, double *val, hipStream_t s) {
    hipLaunchKernelGGL(k_bsr_assemble, dim3((unsigned)n_pieces), dim3(64), 0, s, g.cam_ptr, cam_slot, cam_lmk,
                       g.lmk_first_slot, g.lmk_count, g.slot_cam, J64, vinv, Dblk, row_ptr, pieces, col, val);
}

void launch_bsr_mv(int np, const int32_t *row_ptr, const int32_t *col, const double *val, const double *v, double *y,
                   const double *done, hipStream_t s, double *gram, const double *gram_r) {
    hipLaunchKernelGGL(k_bsr_mv, dim3(np), dim3(256), 0, s, np, row_ptr, col, val, v, y, done, gram, gram_r);
}

void launch_bsr_mm_grouped(int np, int N, const int32_t *row_ptr, const int32_t *col, const double *val,
                           const int32_t *group, const double *z, double *Y, hipStream_t s, const double *skip) {
    hipLaunchKernelGGL(k_bsr_mm_grouped, dim3(np), dim3(256), 0, s, np, N, (int64_t)np * 9, row_ptr, col, val, group,
                       z, Y, skip);
}

}  // namespace ba
