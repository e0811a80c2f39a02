// Scaling-vector step of SKIM (Sec. 4.3, Alg. 2 inner loop; Alg. 3, training loop)
// for gfx950: centroids from fixed labels, the layer-wise (L-full, Sec. 3.4)
// loss tr(dW H dW^T), its gradient with respect to alpha and the Adam update.
//
//   c_ik  = sum_{j in k} s~_ij w~_ij / sum_{j in k} s~_ij      (calc_centroids(W*alpha^-1, L))
//   dW_ij = w_ij - alpha_j c_{i,L_ij}                           (W - replace(c, L) * alpha)
//   P     = dW H            matrix cores, float32 accumulation (the path's one dense contraction): fp16 MFMA on
//                           two-piece splits of the scaled float32 operands; where only the loss is wanted, half of it.
//                           The diagonal of H in float64
//   loss  = sum_ij P_ij dW_ij                                   float64 reduction
//   dloss/dalpha_l = -2 sum_i [ P_il c_{i,L_il}
//                    + Q_{i,L_il} s_il (w_il - 2 alpha_l c_{i,L_il}) / D_{i,L_il} ],
//   Q_ik = sum_{j in k} P_ij alpha_j,  D_ik = sum_{j in k} s~_ij  (gradient through the centroids).
#include "skim_tiles.h"

#include <math.h>

#include <type_traits>

namespace {

// Pieces of a float32 value for the contraction on the matrix cores (see dwh_kernel): two binary16 values, the rounding of
// x and the rounding of the rest.  |x| < 2^15.  From 2^-1 up they carry 23 of its 24 bits or all (the rest has 12 bits of
// which the second piece keeps 11: every fourth x loses its last), below that everything down to 2^-25.
__device__ __forceinline__ void split2(float x, uint32_t &p1, uint32_t &p2) {
    const _Float16 h = (_Float16)x;
    const _Float16 l = (_Float16)(x - (float)h);       // (the difference is exact)
    p1 = (uint32_t)__builtin_bit_cast(uint16_t, h);
    p2 = (uint32_t)__builtin_bit_cast(uint16_t, l);
}
__device__ __forceinline__ float piece_f32(uint32_t h) { return (float)__builtin_bit_cast(_Float16, (uint16_t)h); }

// The diagonal of H stays out of the pieces: its share of the loss and of P is added up in float64 (row_prep_kernel, grad_rows_kernel).
// What a weak channel's column of P mostly is -- its own dW_il H_ll -- thus keeps its digits however strong the other channels are.
// The scales, powers of two, which cost no digits.  binary16 has little range, so both operands are balanced first:
//   e_j   half the exponent of the largest finite magnitude in row j and column j of H, the diagonal aside (-63 where there is none: a
//         channel without couplings takes no part in the scales of the others).  |H_jl| <= min(max_j, max_l) for j != l, so
//         H''_jl = H_jl 2^(H_SHIFT - e_j - e_l) lies below 2^15, whatever H is; for an H of activations that are alike coupled it is
//         their correlations times 2^H_SHIFT over the largest one, within a factor of two.
//   r_i   the exponent of the largest dW_ij 2^e_j of row i; dW''_ij = dW_ij 2^(e_j - r_i + D_SHIFT) lies below 2^15.
//   P_il  = 2^(r_i + e_l - H_SHIFT - D_SHIFT) sum_j dW''_ij H''_jl  +  dW_il H_ll
//   dW_i H dW_i^T = 2^(2 (r_i - D_SHIFT) - H_SHIFT) sum_jl dW''_ij H''_jl dW''_il  +  sum_l dW_il^2 H_ll
// Digits are lost where an entry is 2^16 times smaller than the largest of its row of dW'' (or a coupling 2^15 times smaller than the
// largest its channels allow), and what such an entry loses is below 2^-39 of that largest one.
constexpr int H_SHIFT = 14, D_SHIFT = 15;
__device__ __forceinline__ int h_exponent(uint32_t max_bits) { return ((int)(max_bits >> 23) - 126) >> 1; }      // -63 .. 64; max < 2^(2 e + 1)
// bits of |h| for the maximum over couplings: the diagonal and what is not finite don't count (an infinity or NaN then stays with the
// columns and rows of P that meet it)
__device__ __forceinline__ uint32_t coupling_bits(float h, bool diagonal) {
    const uint32_t b = __float_as_uint(h) & 0x7FFFFFFFu;
    return diagonal || b >= 0x7F800000u ? 0u : b;
}
__device__ __forceinline__ int value_exponent(float x) { return x == 0.0f ? -1024 : __builtin_amdgcn_frexp_expf(x); }      // |x| < 2^this

// Layout of a split matrix ("planes"): groups of 4 rows; a group holds, for every block of 16 k, its 4 rows' [piece 1 (16) |
// piece 2 (16)], 256 contiguous bytes.  A tile reads whole 128-byte lines for a 16-k step, and the four
// rows one workgroup writes are one contiguous region of memory.
constexpr int GK = 16;
__host__ __device__ __forceinline__ size_t plane_rows(long long rows) { return (size_t)(rows + 3) & ~(size_t)3; }      // rows stored
__device__ __forceinline__ size_t plane_index(long long row, long long k, long long m) {
    return ((size_t)(row >> 2) * (size_t)(m >> 4) + (size_t)(k >> 4)) * 128 + (size_t)(row & 3) * 32 + (size_t)(k & 15);     // piece p at + 16 p
}

constexpr int PREP_THREADS = 256;
constexpr int STRIP = 8;           // rows per workgroup in the gradient kernel

__device__ __forceinline__ double block_sum_256(double x, double *scratch /* >= 4 doubles */) {
    for (int d = 32; d >= 1; d >>= 1) x += __shfl_down(x, d, 64);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    __syncthreads();
    if (lane == 0) scratch[wave] = x;
    __syncthreads();
    return scratch[0] + scratch[1] + scratch[2] + scratch[3];
}

// Per-cluster sums of a row with fixed labels: every wavefront adds into bins of its own in LDS (float64
// atomic adds), four copies per wavefront picked by the lane so that lanes with the same label seldom meet
// on one address; the copies are then added in a fixed order.
constexpr int BIN_COPIES = 4;
constexpr int BIN_SETS = (PREP_THREADS / 64) * BIN_COPIES;

__device__ __forceinline__ double bin_total(const double (*bins)[16], int k) {
    double t = 0.0;
#pragma unroll
    for (int b = 0; b < BIN_SETS; ++b) t += bins[b][k];
    return t;
}

// four neighbouring values, in one load where the caller's rows allow it
__device__ __forceinline__ float4 load4(const float *p, bool vec) { return vec ? *(const float4 *)p : make_float4(p[0], p[1], p[2], p[3]); }
__device__ __forceinline__ uint32_t load4(const uint8_t *p, bool vec) {
    return vec ? *(const uint32_t *)p : (uint32_t)p[0] | ((uint32_t)p[1] << 8) | ((uint32_t)p[2] << 16) | ((uint32_t)p[3] << 24);
}

// H (m x m float32, m % 16 == 0) -> its planes.
//   SPLIT_ROWS     row j of the planes = row j of H (its column j where H is symmetric)
//   SPLIT_COLUMNS  row j of the planes = column j of H
//   SPLIT_LOWER    what the loss needs: the columns up to the end of the 256-column block that holds j; those ahead of the
//                  block are the mean of H and its transpose (dW_i H dW_i^T is that of the mean; with H symmetric, H itself)
// The diagonal is left out of all of them.
// A workgroup takes 64 rows x 32 k; the transposed tile goes through LDS, so both are read in whole lines.
enum SplitMode { SPLIT_ROWS, SPLIT_COLUMNS, SPLIT_LOWER };
constexpr int SPLIT_J = 64, SPLIT_K = 32, SPLIT_THREADS = 256;
struct SplitTile {
    float t[SPLIT_K][SPLIT_J + 1];
};
__device__ __forceinline__ void split_tile(const float *__restrict__ H, long long m, const uint32_t *__restrict__ hmax,
                                           uint16_t *__restrict__ Hp, int mode, long long tile, SplitTile &tr) {
    const int tid = threadIdx.x;
    const long long tk = (m + SPLIT_K - 1) / SPLIT_K;
    const long long j0 = tile / tk * SPLIT_J, k0 = tile % tk * SPLIT_K;
    if (mode == SPLIT_LOWER && k0 > (j0 | (TILE - 1))) return;
    const bool turned = mode == SPLIT_COLUMNS || (mode == SPLIT_LOWER && k0 < (j0 & ~(long long)(TILE - 1)));
    if (turned) {          // (the same in the whole workgroup)
        const long long k = k0 + (tid >> 3), j = j0 + 8 * (tid & 7);
        if (k < m && j < m) {
            const float4 a = *(const float4 *)(H + k * m + j), b = *(const float4 *)(H + k * m + j + 4);
            float *o = &tr.t[tid >> 3][8 * (tid & 7)];
            o[0] = a.x; o[1] = a.y; o[2] = a.z; o[3] = a.w;
            o[4] = b.x; o[5] = b.y; o[6] = b.z; o[7] = b.w;
        }
        __syncthreads();
    }
    const int oct = tid & 3;
    const long long j = j0 + (tid >> 2), k = k0 + 8 * oct;       // 8 consecutive k of one row
    if (j >= m || k >= m) return;
    float x[8];
    if (mode != SPLIT_COLUMNS) {
        const float4 a = *(const float4 *)(H + j * m + k), b = *(const float4 *)(H + j * m + k + 4);
        x[0] = a.x; x[1] = a.y; x[2] = a.z; x[3] = a.w;
        x[4] = b.x; x[5] = b.y; x[6] = b.z; x[7] = b.w;
    }
    if (turned) {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const float y = tr.t[8 * oct + e][tid >> 2];
            x[e] = (mode == SPLIT_COLUMNS || x[e] == y) ? y : 0.5f * x[e] + 0.5f * y;
        }
    }
#pragma unroll
    for (int e = 0; e < 8; ++e)
        if (k + e == j) x[e] = 0.0f;
    const uint4 ma = *(const uint4 *)(hmax + k), mb = *(const uint4 *)(hmax + k + 4);
    const uint32_t mk[8] = {ma.x, ma.y, ma.z, ma.w, mb.x, mb.y, mb.z, mb.w};
    const int ej = H_SHIFT - h_exponent(hmax[j]);
    uint32_t p[2][8];
#pragma unroll
    for (int e = 0; e < 8; ++e) split2(ldexpf(x[e], ej - h_exponent(mk[e])), p[0][e], p[1][e]);
    uint16_t *dst = Hp + plane_index(j, k, m);
#pragma unroll
    for (int q = 0; q < 2; ++q)
        *(uint4 *)(dst + 16 * q) = make_uint4(p[q][0] | (p[q][1] << 16), p[q][2] | (p[q][3] << 16), p[q][4] | (p[q][5] << 16),
                                              p[q][6] | (p[q][7] << 16));
}
inline long long split_tiles(int64_t m) { return (m + SPLIT_J - 1) / SPLIT_J * ((m + SPLIT_K - 1) / SPLIT_K); }
__global__ void __launch_bounds__(SPLIT_THREADS) split_rows_kernel(const float *__restrict__ H, long long m, const uint32_t *__restrict__ hmax,
                                                                   uint16_t *__restrict__ Hp, int mode) {
    __shared__ SplitTile tr;
    split_tile(H, m, hmax, Hp, mode, blockIdx.x, tr);
}

// hdiag = the diagonal of H; hmax[j] = bits of the largest coupling in row j and column j of H (bits of magnitudes order like the magnitudes).
// Short matrices: a workgroup works out 16 of them, no atomics between workgroups and nothing to clear.
constexpr int HMAX_DIRECT = 1024;
__global__ void __launch_bounds__(256) hmax_direct_kernel(const float *__restrict__ H, int m, uint32_t *__restrict__ hmax, float *__restrict__ hdiag) {
    __shared__ uint32_t top[16];
    const int a = threadIdx.x & 15, b = threadIdx.x >> 4, j0 = 16 * blockIdx.x;       // m is a multiple of 16
    if (threadIdx.x < 16) top[threadIdx.x] = 0u;
    __syncthreads();
    uint32_t r = 0u, c = 0u;
#pragma unroll 4
    for (int k = 0; k < m; k += 16) {
        r = max(r, coupling_bits(H[(long long)(j0 + b) * m + k + a], j0 + b == k + a));
        c = max(c, coupling_bits(H[(long long)(k + b) * m + j0 + a], j0 + a == k + b));
    }
    atomicMax(&top[b], r);
    atomicMax(&top[a], c);
    __syncthreads();
    if (threadIdx.x < 16) {
        hmax[j0 + threadIdx.x] = top[threadIdx.x];
        hdiag[j0 + threadIdx.x] = H[(long long)(j0 + threadIdx.x) * (m + 1)];
    }
}
// Longer ones: H is read once, 64 rows x 256 columns a workgroup, into a cleared hmax (12288 columns 115 us, 604 MB).
constexpr int HMAX_ROWS = 64, HMAX_COLS = 256;
__global__ void __launch_bounds__(256) hmax_clear_kernel(const float *__restrict__ H, long long m, uint32_t *__restrict__ hmax, float *__restrict__ hdiag) {
    const long long j = (long long)blockIdx.x * 256 + threadIdx.x;
    if (j >= m) return;
    hmax[j] = 0u;
    hdiag[j] = H[j * (m + 1)];
}
__global__ void __launch_bounds__(256) hmax_kernel(const float *__restrict__ H, long long m, int tiles_x, uint32_t *__restrict__ hmax) {
    __shared__ uint32_t cols[4][HMAX_COLS];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const long long j0 = (long long)(blockIdx.x / tiles_x) * HMAX_ROWS + 16 * wave, k = (long long)(blockIdx.x % tiles_x) * HMAX_COLS + 4 * lane;
    uint32_t c[4] = {0u, 0u, 0u, 0u};
    uint32_t mine = 0u;          // lane i < 16: the largest of row j0 + i
#pragma unroll 1
    for (int i0 = 0; i0 < 16; i0 += 8) {       // (eight rows at a time: 16 at once leave room for half as many wavefronts)
        float4 x[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) x[i] = (j0 + i0 + i < m && k < m) ? *(const float4 *)(H + (j0 + i0 + i) * m + k) : make_float4(0.f, 0.f, 0.f, 0.f);
        const int d = (int)min(max(j0 + i0 - k, -64ll), 64ll);      // column k + d is the diagonal of row j0 + i0
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const uint32_t b[4] = {coupling_bits(x[i].x, d + i == 0), coupling_bits(x[i].y, d + i == 1), coupling_bits(x[i].z, d + i == 2),
                                   coupling_bits(x[i].w, d + i == 3)};
            uint32_t r = 0u;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                c[q] = max(c[q], b[q]);
                r = max(r, b[q]);
            }
#pragma unroll
            for (int o = 32; o >= 1; o >>= 1) r = max(r, (uint32_t)__shfl_xor((int)r, o, 64));
            if (lane == i0 + i) mine = r;
        }
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) cols[wave][4 * lane + q] = c[q];
    if (lane < 16 && j0 + lane < m) atomicMax(&hmax[j0 + lane], mine);
    __syncthreads();
    const long long l = (long long)(blockIdx.x % tiles_x) * HMAX_COLS + tid;
    if (l < m) atomicMax(&hmax[l], max(max(cols[0][tid], cols[1][tid]), max(cols[2][tid], cols[3][tid])));
}

// Per row: weighted cluster sums with fixed labels -> centroids c (n x 16 float64),
// masses Den (n x 16 float64), and the row of dW as two scaled pieces per value with the exponent of its scale (rexp).
// BITS == 0: labels are read.  BITS == 1 .. 4: the labels are worked out from the clusters' upper bounds (the largest member of each
// cluster, -inf for an empty one) at upper + row * upper_stride: the cluster with the smallest bound >= w~; labels_out
// (optional) receives them.  The centroids are those of the clustering then, at given + row * given_stride -- the weighted means of
// these labels, and for a cluster whose members carry no sensitivity mass what the clustering kept -- and S is not read.
// A workgroup takes 4 rows (one group of the planes: it writes one contiguous region), four wavefronts each, four columns
// per lane and step.  KEEP > 0: the row takes at most KEEP steps, and its weights and labels (then its dW and their columns' exponents)
// stay in registers; 0: longer rows are read three times, the largest entry of dW being needed ahead of the first piece.  Bound: HBM
// (9 to 13 bytes read and 4 written per weight): 61 us at 4096 x 4096 (67 with three pieces), 218 MB; held to 64 registers two workgroups
// share a compute unit (69 registers: 75 us).  With labels from bounds 4 bytes read: 42 us (60 to 75 with the sums of S).
// WPR: wavefronts per row: four, or one for rows of up to 256 columns, which one step of a wavefront holds (11008 x 32: 25.6 ->
// 10.1 us).  That variant cuts H into its pieces as well, in workgroups behind those of the rows: such a layer's call is
// mostly launches.
constexpr int ROWP_ROWS = 4, ROWP_COPIES = 8;      // copies of the bins per wavefront, picked by the lane
constexpr int ROWP_NARROW = 256;
// DIAG: for the loss, the row's share of the diagonal of H as well.
template <int BITS, int KEEP, int WPR, bool DIAG>
__global__ void __launch_bounds__(64 * ROWP_ROWS * WPR) __attribute__((amdgpu_waves_per_eu(KEEP > 4 || KEEP == 0 ? 4 : 8))) row_prep_kernel(const float *W, const float *S, const float *alpha, long long n,
                                                                   long long m, long long ld, const uint8_t *labels, const float *upper,
                                                                   long long upper_stride, uint8_t *labels_out, double *cent, double *Den,
                                                                   uint16_t *dWp, const double *given, long long given_stride,
                                                                   bool vec4, const float *H, const uint32_t *hmax, uint16_t *Hp,
                                                                   int split_mode, int *rexp, const float *hdiag, double *rdiag) {
    if constexpr (WPR == 1) {
        __shared__ SplitTile tr;
        const long long groups = (n + ROWP_ROWS - 1) / ROWP_ROWS;
        if (blockIdx.x >= groups) {
            split_tile(H, m, hmax, Hp, split_mode, blockIdx.x - groups, tr);
            return;
        }
    }
    constexpr int WAVES = ROWP_ROWS * WPR, STEP = 256 * WPR, K = 1 << BITS, NSC = BITS == 4 ? 3 : K - 1;
    __shared__ double binD[BITS == 0 ? WAVES : 1][ROWP_COPIES][16], binN[BITS == 0 ? WAVES : 1][ROWP_COPIES][16];
    __shared__ double csh[WAVES][16];             // centroids by label; BITS > 0: by position among the ascending bounds
    __shared__ __align__(16) float thr[WAVES][16];
    __shared__ int thl[WAVES][16];
    __shared__ int wexp[WAVES];
    __shared__ double wdiag[WAVES];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int sub = wave % WPR;                                     // its share of the row's steps
    const bool live = (long long)blockIdx.x * ROWP_ROWS + wave / WPR < n;
    const long long row = live ? (long long)blockIdx.x * ROWP_ROWS + wave / WPR : n - 1;
    const long long mm = live ? m : 0;                              // (a row past the end has no columns)
    const float *Wr = W + row * ld, *Sr = S + row * ld;
    const uint8_t *Lr = BITS == 0 ? labels + row * m : nullptr;
    uint8_t *Lo = BITS > 0 && labels_out ? labels_out + row * m : nullptr;
    float ts[NSC > 0 ? NSC : 1];
    if constexpr (BITS > 0) {
        // bounds ascending (empty clusters, -inf, first; equal ones by cluster), +inf beyond the last
        if (lane < 16) {
            const float *up_row = upper + row * upper_stride;
            const float up = lane < K ? up_row[lane] : INFINITY;
            int rank = lane;
            if (lane < K) {
                rank = 0;
                for (int j = 0; j < K; ++j) {
                    const float uj = up_row[j];
                    rank += (uj < up || (uj == up && j < lane)) ? 1 : 0;
                }
            }
            thr[wave][rank] = up;
            thl[wave][rank] = lane;
            if (lane < K) csh[wave][rank] = given[row * given_stride + lane];
        }
        __builtin_amdgcn_wave_barrier();      // (one wavefront's LDS accesses execute in order)
#pragma unroll
        for (int k = 0; k < NSC; ++k)
            ts[k] = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(thr[wave][BITS == 4 ? 4 * k + 3 : k])));
    }
    auto position_of = [&](float wt) -> int {      // number of bounds below the weight
        int pos = 0;
        if (BITS == 4) {
            int q = 0;
#pragma unroll
            for (int k = 0; k < 3; ++k) q += (ts[k] < wt) ? 1 : 0;
            const float4 t4 = *(const float4 *)&thr[wave][4 * q];
            pos = 4 * q + ((t4.x < wt) ? 1 : 0) + ((t4.y < wt) ? 1 : 0) + ((t4.z < wt) ? 1 : 0);
        } else {
#pragma unroll
            for (int k = 0; k < NSC; ++k) pos += (ts[k] < wt) ? 1 : 0;
        }
        return pos;
    };
    const float4 ones = make_float4(1.f, 1.f, 1.f, 1.f);
    const long long j0 = 4ll * (lane + 64 * sub);
    float4 wk[KEEP > 0 ? KEEP : 1];
    uint32_t lk[KEEP > 0 ? KEEP : 1];
    if constexpr (BITS == 0) {
#pragma unroll
        for (int q = 0; q < ROWP_COPIES / 4; ++q) {
            (&binD[wave][0][0])[64 * q + lane] = 0.0;
            (&binN[wave][0][0])[64 * q + lane] = 0.0;
        }
        double *myD = binD[wave][lane & (ROWP_COPIES - 1)], *myN = binN[wave][lane & (ROWP_COPIES - 1)];
        auto add_step = [&](int it, long long j) {
            const float4 w4 = load4(Wr + j, vec4), s4 = load4(Sr + j, vec4);
            const float4 a4 = alpha ? load4(alpha + j, vec4) : ones;
            const uint32_t l4 = load4(Lr + j, vec4);
            const float wv[4] = {w4.x, w4.y, w4.z, w4.w}, sv[4] = {s4.x, s4.y, s4.z, s4.w}, av[4] = {a4.x, a4.y, a4.z, a4.w};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float wt = alpha ? __fdiv_rn(wv[e], av[e]) : wv[e];
                const float st = alpha ? __fmul_rn(__fmul_rn(sv[e], av[e]), av[e]) : sv[e];
                const int l = (int)((l4 >> (8 * e)) & 15u);
                atomicAdd(&myD[l], (double)st);
                atomicAdd(&myN[l], (double)st * (double)wt);
            }
            if (KEEP > 0) {
                wk[KEEP > 0 ? it : 0] = w4;
                lk[KEEP > 0 ? it : 0] = l4;
            }
        };
        if constexpr (KEEP > 0) {
#pragma unroll
            for (int it = 0; it < KEEP; ++it)
                if (j0 + STEP * it < mm) add_step(it, j0 + STEP * it);
        } else {
#pragma unroll 2
            for (long long j = j0; j < mm; j += STEP) add_step(0, j);
        }
        __syncthreads();
        // 16 clusters; four wavefronts a row: the bins of one of them in every 16 lanes
        double d = 0.0, nn = 0.0;
        const int bw = WPR == 4 ? (wave & ~3) + (lane >> 4) : wave;
#pragma unroll
        for (int q = 0; q < ROWP_COPIES; ++q) {
            d += binD[bw][q][lane & 15];
            nn += binN[bw][q][lane & 15];
        }
        if constexpr (WPR == 4) {
            d += __shfl_xor(d, 16, 64);
            nn += __shfl_xor(nn, 16, 64);
            d += __shfl_xor(d, 32, 64);
            nn += __shfl_xor(nn, 32, 64);
        }
        if (lane < 16) {
            const double c = d > 0.0 ? nn / d : 0.0;
            csh[wave][lane] = c;
            if (sub == 0 && live) {
                cent[row * 16 + lane] = c;
                Den[row * 16 + lane] = d;
            }
        }
        __builtin_amdgcn_wave_barrier();
    }
    // four entries of dW and the exponents e_j of their columns (a byte each); the largest exponent of the row so far
    // and, for the loss, its diagonal share: the sum of dW_ij^2 H_jj in float64
    int top = -1024;
    double dsum = 0.0;
    auto form_four = [&](float4 &w4, const float4 &a4, uint32_t &l4, long long j) {
        const float wv[4] = {w4.x, w4.y, w4.z, w4.w}, av[4] = {a4.x, a4.y, a4.z, a4.w};
        const uint4 h4 = *(const uint4 *)(hmax + j);
        const uint32_t hv[4] = {h4.x, h4.y, h4.z, h4.w};
        const float4 g4 = DIAG ? *(const float4 *)(hdiag + j) : ones;
        const float gv[4] = {g4.x, g4.y, g4.z, g4.w};
        float d[4];
        uint32_t ex = 0u;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const double dd = (double)wv[e] - (double)av[e] * csh[wave][(l4 >> (8 * e)) & 15u];
            if (DIAG) dsum = fma(dd * dd, (double)gv[e], dsum);
            d[e] = (float)dd;
            const int ej = h_exponent(hv[e]);
            top = max(top, value_exponent(d[e]) + ej);
            ex |= ((uint32_t)ej & 0xFFu) << (8 * e);
        }
        w4 = make_float4(d[0], d[1], d[2], d[3]);
        l4 = ex;
    };
    auto write_four = [&](const float4 &d4, uint32_t e4, int shift, long long j) {
        const float d[4] = {d4.x, d4.y, d4.z, d4.w};
        uint32_t pc[2][4];
#pragma unroll
        for (int e = 0; e < 4; ++e) split2(ldexpf(d[e], shift + (int)(int8_t)(e4 >> (8 * e))), pc[0][e], pc[1][e]);
        uint16_t *o = dWp + plane_index(row, j, m);   // four neighbouring k stay inside one block of 16
#pragma unroll
        for (int q = 0; q < 2; ++q)
            *(uint2 *)(o + 16 * q) = make_uint2(pc[q][0] | (pc[q][1] << 16), pc[q][2] | (pc[q][3] << 16));
    };
    // one step of the row from memory: labels (or positions, then the labels go out where they are wanted), dW, exponents
    auto form_step = [&](float4 &w4, uint32_t &l4, long long j, bool out) {
        w4 = load4(Wr + j, vec4);
        const float4 a4 = alpha ? load4(alpha + j, vec4) : ones;
        if (BITS == 0) {
            l4 = load4(Lr + j, vec4);
        } else {
            const float wv[4] = {w4.x, w4.y, w4.z, w4.w}, av[4] = {a4.x, a4.y, a4.z, a4.w};
            int pos[4];
            l4 = 0u;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                pos[e] = position_of(alpha ? __fdiv_rn(wv[e], av[e]) : wv[e]);
                l4 |= (uint32_t)pos[e] << (8 * e);
            }
            if (out && Lo) {
                uint32_t lab = 0u;
#pragma unroll
                for (int e = 0; e < 4; ++e) lab |= (uint32_t)thl[wave][pos[e]] << (8 * e);
                if (vec4) *(uint32_t *)(Lo + j) = lab;
                else
                    for (int e = 0; e < 4; ++e) Lo[j + e] = (uint8_t)(lab >> (8 * e));
            }
        }
        form_four(w4, a4, l4, j);
    };
    // (rows that do not stay in registers are formed for their largest entry, and again to be written)
    if constexpr (KEEP > 0) {
#pragma unroll
        for (int it = 0; it < KEEP; ++it)
            if (j0 + STEP * it < mm) {
                const long long j = j0 + STEP * it;
                if (BITS == 0) form_four(wk[it], alpha ? load4(alpha + j, vec4) : ones, lk[it], j);
                else form_step(wk[it], lk[it], j, true);
            }
    } else {
#pragma unroll 2
        for (long long j = j0; j < mm; j += STEP) {
            float4 w4;
            uint32_t l4;
            form_step(w4, l4, j, true);
        }
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
        top = max(top, __shfl_xor(top, o, 64));
        if (DIAG) dsum += __shfl_xor(dsum, o, 64);
    }
    if constexpr (WPR == 4) {
        if (lane == 0) {
            wexp[wave] = top;
            wdiag[wave] = dsum;
        }
        __syncthreads();
        dsum = 0.0;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            top = max(top, wexp[(wave & ~3) + q]);
            dsum += wdiag[(wave & ~3) + q];
        }
    }
    if (top < -1000) top = 0;          // a row of zeros
    if (sub == 0 && lane == 0 && live) {
        rexp[row] = top;
        if (DIAG) rdiag[row] = dsum;
    }
    if constexpr (KEEP > 0) {
#pragma unroll
        for (int it = 0; it < KEEP; ++it)
            if (j0 + STEP * it < mm) write_four(wk[it], lk[it], D_SHIFT - top, j0 + STEP * it);
    } else {
#pragma unroll 2
        for (long long j = j0; j < mm; j += STEP) {
            float4 w4;
            uint32_t l4;
            form_step(w4, l4, j, false);
            write_four(w4, l4, D_SHIFT - top, j);
        }
    }
}

// ---- the contraction on the matrix cores -------------------------------------------------------------------------
// A float32 value x scaled as above is p1 + p2, two binary16 values, up to its last bit (see split2), so x y is the sum of four
// products of pieces, each exact in float32.  The three with p1 q1, p1 q2, p2 q1 carry everything but p2 q2, at most 2^-22
// of |x y| and 2^-25 in the mean square, of either sign.  v_mfma_f32_32x32x16_f16 does one of them for 16 k in 32 clocks: 96, where
// the six leading products of three bfloat16 pieces took 192 and v_mfma_f32_32x32x2_f32 takes 512.  Accumulation is float32 in the
// matrix core either way.  Half as many roundings of the sums and a diagonal that is left to float64 outweigh the last bit of the
// operands.  Against float64, relative 2-norms here / with three bfloat16 pieces and the diagonal among them, channels of calibration
// activations: P 0.08 / 2.2e-7 at 512 columns, 0.15 / 2.2e-7 at 1552, 0.26 / 1.9e-7 at 4096, 0.63 / 3.3e-7 at 8192; gradient 0.25 / 1.7e-7, 0.23 /
// 2.5e-7, 0.23 / 1.6e-7, 0.27 / 3.1e-7; row losses 0.02 / 0.6e-7 to 0.06 / 0.7e-7.  Channels correlated through 8 common factors: P 1.3 / 1.9e-7,
// 1.7 / 2.1e-7, 2.0 / 2.2e-7, 3.5 / 4.2e-7; gradient 0.7 / 1.5e-7, 0.7 / 1.2e-7, 1.1 / 1.8e-7, 2.3 / 3.6e-7; row losses 0.7 / 1.1e-7 to 2.0 / 2.6e-7.
// (The diagonal among the pieces here too: correlated channels, 512 columns, P 2.2e-7, gradient 2.0e-7: further off than with three pieces.)
typedef _Float16 half8_t __attribute__((ext_vector_type(8)));
typedef __attribute__((address_space(3))) half8_t lds_half8;
constexpr int G_THREADS = 512;                     // 8 wavefronts, two per SIMD: 2 x 4, each 128 x 64 of the 256 x 256 tile
constexpr int G_BUFS = 4;                          // a power of two
constexpr uint32_t G_PANEL_BYTES = TILE * 64;      // one operand of one 16-k stage: 16 KB
constexpr uint32_t G_STAGE_BYTES = 2 * G_PANEL_BYTES;
constexpr size_t G_LDS_BYTES = (size_t)G_BUFS * G_STAGE_BYTES;      // 131072
constexpr int G_LOADS = G_STAGE_BYTES / (1024 * (G_THREADS / 64));  // 1 KB copies of a wavefront per stage: 4
constexpr int G_MIN_STAGES = 16;
constexpr int G_PHASE_COST = 20;                   // a phase of split tiles with its partial tiles, in stages

// What a lane needs to know about the LDS.  A panel holds its rows one after the other (64 bytes each: four 16-byte units,
// unit 2 p + h = piece p, k 8 h .. 8 h + 7), the units of row r rotated by r / 4: any 16 rows then read one unit from 64
// different banks.
struct DwhLane {
    uint32_t voff[G_LOADS];      // source of its copies inside the tile's rows
    uint32_t dst;                // their first kilobyte (the same in the whole wavefront)
    uint32_t ra[2], rb[2];       // operand addresses of the two pieces, A block x at + x * 2048, B block y likewise
    int swave, wr, wc, l32, lhi;
    __device__ __forceinline__ DwhLane(uint32_t lds0, int tid, long long m) {
        const int lane = tid & 63, wave = tid >> 6;
        swave = __builtin_amdgcn_readfirstlane(wave);
        wr = wave >> 2;
        wc = wave & 3;
        l32 = lane & 31;
        lhi = lane >> 5;
#pragma unroll
        for (int i = 0; i < G_LOADS; ++i) {
            const int c = ((wave & 3) * G_LOADS + i) * 64 + lane;
            const int row = c >> 2, unit = (c - (row >> 2)) & 3;
            voff[i] = (uint32_t)((row >> 2) * m * 16) + (uint32_t)((row & 3) * 64 + unit * 16);
        }
        dst = lds0 + (uint32_t)(swave >> 2) * G_PANEL_BYTES + (uint32_t)(swave & 3) * (G_LOADS * 1024);
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            const uint32_t u = (uint32_t)((2 * p + lhi + (l32 >> 2)) & 3) * 16;
            ra[p] = lds0 + (uint32_t)(wr * 128 + l32) * 64 + u;
            rb[p] = lds0 + G_PANEL_BYTES + (uint32_t)(wc * 64 + l32) * 64 + u;
        }
    }
};

// acc = (rows arow0 .. of A) (rows brow0 .. of B)^T over the 16-k stages [s0, s1), from the planes of two matrices of m columns;
// with HALVED the sums are doubled ahead of stage sdouble.  Rows past the end of either matrix carry no meaning.
// 16 k are 24 MFMAs and 12 operand reads per wavefront.  The operands of the next quarter of a stage are read between the
// MFMAs of this one; the barrier stands ahead of the last quarter: past it the next stage is complete in LDS and this
// one's place is free for the stage after the next three.
template <bool HALVED>
__device__ __forceinline__ void dwh_accumulate(floatx16 (&acc)[4][2], const DwhLane &L, const uint16_t *Ap, long long arows,
                                               long long arow0, const uint16_t *Bp, long long brows, long long brow0, long long m,
                                               int s0, int s1, int sdouble) {
#pragma unroll
    for (int x = 0; x < 4; ++x)
#pragma unroll
        for (int y = 0; y < 2; ++y)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[x][y][e] = 0.f;
    const bool isb = L.swave >= 4;
    const long long rows = isb ? brows : arows, skip = ((isb ? brow0 : arow0) >> 2) * m * 16 + (long long)s0 * 256;
    LdsSource src{(uint64_t)(uintptr_t)(isb ? Bp : Ap) + (uint64_t)skip, (long long)plane_rows(rows) * m * 4 - skip};
    int ahead = s1 - s0;         // stages still to be requested (past the end nothing is read: zeros arrive)
    auto issue = [&](uint32_t buf) {
        if (ahead-- <= 0) src.left = 0;
        const int4v rs = src.rsrc();
#pragma unroll
        for (int i = 0; i < G_LOADS; ++i) copy_to_lds(L.dst + buf + i * 1024, L.voff[i], rs);
        src.advance(256);
    };
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");      // the LDS is free
#pragma unroll
    for (int q = 0; q < G_BUFS; ++q) issue(q * G_STAGE_BYTES);
    asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"((G_BUFS - 1) * G_LOADS) : "memory");
    half8_t a[2][2], b[2][2][2];
    auto read_a = [&](int set, uint32_t buf, int x) {
#pragma unroll
        for (int p = 0; p < 2; ++p) a[set][p] = *(lds_half8 *)(L.ra[p] + buf + x * 2048);
    };
    auto read_b = [&](int set, uint32_t buf) {
#pragma unroll
        for (int y = 0; y < 2; ++y)
#pragma unroll
            for (int p = 0; p < 2; ++p) b[set][y][p] = *(lds_half8 *)(L.rb[p] + buf + y * 2048);
    };
    auto multiply = [&](int x, int as, int bs) {     // smallest products first
        constexpr int PA[3] = {1, 0, 0}, PB[3] = {0, 1, 0};
#pragma unroll
        for (int q = 0; q < 3; ++q)
#pragma unroll
            for (int y = 0; y < 2; ++y)
                acc[x][y] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[as][PA[q]], b[bs][y][PB[q]], acc[x][y], 0, 0, 0);
    };
    uint32_t cur = 0;
    read_b(0, cur);
    read_a(0, cur, 0);
    auto stage = [&](auto par, int st) {
        constexpr int BS = decltype(par)::value;
        if (HALVED && st == sdouble) {
#pragma unroll
            for (int x = 0; x < 4; ++x)
#pragma unroll
                for (int y = 0; y < 2; ++y)
#pragma unroll
                    for (int e = 0; e < 16; ++e) acc[x][y][e] += acc[x][y][e];
        }
        const uint32_t nxt = (cur + G_STAGE_BYTES) & (G_BUFS * G_STAGE_BYTES - 1);
#pragma unroll
        for (int x = 0; x < 3; ++x) {
            read_a((x + 1) & 1, cur, x + 1);
            multiply(x, x & 1, BS);
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);       // an MFMA, the two reads, the other MFMAs
            __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
            __builtin_amdgcn_sched_group_barrier(0x008, 5, 0);
        }
        asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"((G_BUFS - 2) * G_LOADS) : "memory");
        issue(cur);
        read_b(BS ^ 1, nxt);
        read_a(0, nxt, 0);
        multiply(3, 1, BS);
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        }
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        cur = nxt;
    };
    for (int st = s0;;) {
        stage(std::integral_constant<int, 0>{}, st);
        if (++st >= s1) break;
        stage(std::integral_constant<int, 1>{}, st);
        if (++st >= s1) break;
    }
}

// Row and column of tile t: column by column in bands of 4 rows of tiles, so that the 32 tiles an XCD works on share 4 panels of dW
// and 8 of H.
__device__ __forceinline__ void tile_place(int t, int rows, int tj, int &i, int &j) {
    const int band = t / (4 * tj), h = min(4, rows - 4 * band), rem = t - band * 4 * tj;
    j = rem / h;
    i = 4 * band + rem - j * h;
}

// What bounds it: the power the matrix cores draw.  4096^3: 0.31 ms = 1.32 PFLOP/s of executed piece products (a bf16
// product of the same size by the library: 1.10), MFMAs busy 84 % of the cycles at 1.66 GHz instead of 2.4, no bank
// conflicts.  Six products of bfloat16 pieces: 0.54 ms.
// P = dW H (H without its diagonal), tile by tile as the plan says: a whole tile goes straight into P, a part of a split one into its slot.
__global__ void __launch_bounds__(G_THREADS) __attribute__((amdgpu_waves_per_eu(2, 2)))
dwh_kernel(const uint16_t *__restrict__ Ap, const uint16_t *__restrict__ Hp, const int *__restrict__ rexp, const uint32_t *__restrict__ hmax,
           long long n, long long m, int tj, TilePlan plan, float *__restrict__ P, floatx4 *__restrict__ slots) {
    extern __shared__ __align__(16) unsigned char g_smem[];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const DwhLane L((uint32_t)(uintptr_t)(lds_byte *)g_smem, tid, m);
    const int nk = (int)(m / GK);
    const int G = gridDim.x, me = xcd_order(blockIdx.x, G);
    for (int p = 0; p < plan.nph; ++p) {
        const int ntile = plan.ntile[p], split = plan.split[p];
        for (int v = me; v < ntile * split; v += G) {
            const int part = v / ntile, t = plan.tile0[p] + v - part * ntile;
            int ti, tc;
            tile_place(t, (int)((n + TILE - 1) / TILE), tj, ti, tc);
            const long long row0 = (long long)ti * TILE, col0 = (long long)tc * TILE;
            const int s0 = (int)((long long)nk * part / split), s1 = (int)((long long)nk * (part + 1) / split);
            floatx16 acc[4][2];
            dwh_accumulate<false>(acc, L, Ap, n, row0, Hp, m, col0, m, s0, s1, -1);
            // accumulator element e of a 32 x 32 block: row = 8*(e/4) + 4*(lane/32) + e%4, column = lane%32
            if (split > 1) {
                floatx4 *sp = slots + ((size_t)(plan.slot0[p] + v) * 8 + wave) * (8 * 4 * 64) + lane;
#pragma unroll
                for (int xy = 0; xy < 8; ++xy)
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const floatx16 &c = acc[xy >> 1][xy & 1];
                        sp[(xy * 4 + q) * 64] = floatx4{c[4 * q], c[4 * q + 1], c[4 * q + 2], c[4 * q + 3]};
                    }
            } else {
                const long long rb = row0 + L.wr * 128 + 4 * L.lhi, cb = col0 + L.wc * 64 + L.l32;
                float *pp = P + rb * m + cb;
                const int *re = rexp + rb;
                long long mm = m;
                int rlim = (int)min(n - rb, 4096ll), clim = (int)min(m - cb, 4096ll);
                asm volatile("" : "+v"(pp), "+v"(re), "+s"(mm), "+v"(rlim), "+v"(clim));     // the addresses are worked out here, not ahead of the loop
                const int e0 = clim > 0 ? h_exponent(hmax[cb]) - H_SHIFT - D_SHIFT : 0, e1 = clim > 32 ? h_exponent(hmax[cb + 32]) - H_SHIFT - D_SHIFT : 0;
#pragma unroll
                for (int x = 0; x < 4; ++x)
#pragma unroll
                    for (int q4 = 0; q4 < 4; ++q4) {
                        const int4v ri = *(const int4v *)(re + x * 32 + 8 * q4);       // (rexp has room for whole tiles)
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            const int r = x * 32 + 8 * q4 + e;
                            float *q = pp + r * mm;
                            if (r < rlim) {
                                if (clim > 0) q[0] = ldexpf(acc[x][0][4 * q4 + e], ri[e] + e0);
                                if (clim > 32) q[32] = ldexpf(acc[x][1][4 * q4 + e], ri[e] + e1);
                            }
                        }
                    }
            }
        }
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");      // no copy into the LDS is left behind
}

// P of the split tiles: their parts added up.  One wavefront per 32 x 32 block (16 workgroups per tile).
__global__ void __launch_bounds__(256) dwh_parts_kernel(float *__restrict__ P, const int *__restrict__ rexp, const uint32_t *__restrict__ hmax,
                                                        long long n, long long m, int tj, TilePlan plan, int ph,
                                                        const floatx4 *__restrict__ slots) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int l32 = lane & 31, lhi = lane >> 5;
    const int tv = blockIdx.x >> 4, blk = (blockIdx.x & 15) * 4 + wave;
    const int t = plan.tile0[ph] + tv;
    int ti, tc;
    tile_place(t, (int)((n + TILE - 1) / TILE), tj, ti, tc);
    const int ow = blk >> 3, xy = blk & 7;
    const long long rb = (long long)ti * TILE + (ow >> 2) * 128 + (xy >> 1) * 32 + 4 * lhi;
    const long long cb = (long long)tc * TILE + (ow & 3) * 64 + (xy & 1) * 32 + l32;
    const floatx4 *sp = slots + ((size_t)(plan.slot0[ph] + tv) * 8 + ow) * (8 * 4 * 64) + xy * 256 + lane;
    const size_t step = (size_t)plan.ntile[ph] * (8 * 8 * 4 * 64);
    floatx4 s[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) s[q] = sp[q * 64];
    for (int k = 1; k < plan.split[ph]; ++k) {
        sp += step;
#pragma unroll
        for (int q = 0; q < 4; ++q) s[q] += sp[q * 64];
    }
    if (cb >= m) return;
    const int ec = h_exponent(hmax[cb]) - H_SHIFT - D_SHIFT;
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (rb + 8 * q + e < n) P[(rb + 8 * q + e) * m + cb] = ldexpf(s[q][e], rexp[rb + 8 * q + e] + ec);
}

// 4096^3: 0.185 ms (0.33 with six products of bfloat16 pieces), MFMAs busy 75 % of the cycles.
// Loss only: dW_i H dW_i^T = sum over the 256-column blocks J of H of [ 2 sum_{K < J} dW_K H_KJ + dW_J H_JJ ] . dW_J, the H_KJ
// those of the mean of H and its transpose: half the products.  The stages of all tiles -- tile (I, J) has those of the blocks K <= J -- form one line that is
// cut into equal pieces, one per workgroup; the loss is linear in the sums, so the pieces of a tile need not meet: each
// multiplies its own sums by dW_J and leaves 256 row sums (float64) behind, at partial[(tile + workgroup) * 256 ..] (tiles
// and workgroups both count up along the line, so no two pieces share a number).
struct LossLine {
    int tj, G, nk;              // column blocks, workgroups, stages of the longest tile
    long long per_row, total;   // stages of a row of tiles, of all
    // A row's tiles follow each other as J = tj - 1, 0, tj - 2, 1, ...: two neighbours have 16 (tj + 1) stages together, so where the
    // pieces are about half of that, the workgroups of an XCD walk through the same K of dW and of H at the same time
    __host__ __device__ __forceinline__ int tile(int q) const { return (q & 1) ? q >> 1 : tj - 1 - (q >> 1); }
    __host__ __device__ __forceinline__ long long before(int q) const {      // stages ahead of the q-th tile of a row
        return 16ll * (tj + 1) * (q >> 1) + ((q & 1) ? 16ll * (tj - (q >> 1)) : 0) - (q > 0 ? 16 * tj - nk : 0);
    }
    __host__ __device__ __forceinline__ int stages(int j) const { return 16 * (j + 1) < nk ? 16 * (j + 1) : nk; }
    __host__ __device__ __forceinline__ long long start(int g) const { return total * g / G; }               // first stage of workgroup g
    __host__ __device__ __forceinline__ int owner(long long stage) const { return (int)(((stage + 1) * G - 1) / total); }
};
constexpr int LOSS_MAX_WG = 256;
constexpr int LOSS_MIN_STAGES = 4;      // a piece is this long, or a whole tile where that is shorter (256 x 256: 20 us, 31 with 16 stages)
constexpr long long LOSS_SMALL = 40000;
inline LossLine loss_line(int64_t n, int64_t m, int num_cu) {
    LossLine l;
    l.tj = (int)((m + TILE - 1) / TILE);
    l.nk = (int)(m / GK);
    l.per_row = l.before(l.tj - 1) + l.stages(l.tile(l.tj - 1));
    l.total = l.per_row * ((n + TILE - 1) / TILE);
    const int least = l.nk < LOSS_MIN_STAGES ? l.nk : LOSS_MIN_STAGES;
    const long long most = l.total / least > 1 ? l.total / least : 1;
    l.G = num_cu < LOSS_MAX_WG ? num_cu : LOSS_MAX_WG;
    if (l.G > most) l.G = (int)most;
    return l;
}

__global__ void __launch_bounds__(G_THREADS) __attribute__((amdgpu_waves_per_eu(2, 2)))
dwh_loss_kernel(const uint16_t *__restrict__ Ap, const uint16_t *__restrict__ Hp, const int *__restrict__ rexp, long long n, long long m,
                LossLine line, double *__restrict__ partial) {
    extern __shared__ __align__(16) unsigned char g_smem[];
    const int tid = threadIdx.x;
    const DwhLane L((uint32_t)(uintptr_t)(lds_byte *)g_smem, tid, m);
    const int g = xcd_order(blockIdx.x, line.G);
    long long at = line.start(g);
    const long long end = line.start(g + 1);
    while (at < end) {
        const int I = (int)(at / line.per_row);
        const int in_row = (int)(at - (long long)I * line.per_row);
        int q = 0;
        while (q + 1 < line.tj && line.before(q + 1) <= in_row) ++q;
        const int J = line.tile(q), s0 = in_row - (int)line.before(q);
        const int s1 = (int)min((long long)line.stages(J), s0 + (end - at));
        const long long row0 = (long long)I * TILE, col0 = (long long)J * TILE;
        floatx16 acc[4][2];
        // H takes the rows of the tile here and dW its columns: a lane then holds 4 neighbouring columns of dW_i H for a row i of
        // its own, and multiplies them by 8 bytes of each piece.
        // (a piece that starts inside the diagonal block is not doubled; one that ends ahead of it is, at the end)
        dwh_accumulate<true>(acc, L, Hp, m, col0, Ap, n, row0, m, s0, s1, s0 < 16 * J ? 16 * J : -1);
        const double twice = s1 <= 16 * J ? 2.0 : 1.0;
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");       // the tiles in LDS are no longer read or written
        double *rsum = (double *)g_smem;                                              // [2][256]
#pragma unroll
        for (int y = 0; y < 2; ++y) {
            const int rl = L.wc * 64 + 32 * y + L.l32;
            const long long r = row0 + rl;
            double t = 0.0;
            if (r < n) {
#pragma unroll
                for (int x = 0; x < 4; ++x) {
                    __builtin_amdgcn_sched_barrier(0);      // (one block's loads at a time: the registers hold the sums)
                    const long long c = col0 + L.wr * 128 + x * 32 + 4 * L.lhi;
                    uint2 d[4][2];
#pragma unroll
                    for (int q = 0; q < 4; ++q)
#pragma unroll
                        for (int p = 0; p < 2; ++p)
                            d[q][p] = c + 8 * q < m ? *(const uint2 *)(Ap + plane_index(r, c + 8 * q, m) + 16 * p) : make_uint2(0u, 0u);
#pragma unroll
                    for (int q = 0; q < 4; ++q)
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            const int sh = (e & 1) * 16;
                            auto piece = [&](int p) { return piece_f32(((e < 2 ? d[q][p].x : d[q][p].y) >> sh) & 0xFFFFu); };
                            const float dw = piece(0) + piece(1);     // exact
                            t += (double)acc[x][y][4 * q + e] * (double)dw;         // (columns past the matrix: dw = 0)
                        }
                }
            }
            t += __shfl_xor(t, 32, 64);
            if (L.lhi == 0) rsum[L.wr * TILE + rl] = t;
        }
        __syncthreads();
        if (tid < TILE) {
            double *o = partial + ((long long)I * line.tj + q + g) * TILE + tid;
            o[0] = ldexp((rsum[tid] + rsum[TILE + tid]) * twice, 2 * (rexp[row0 + tid] - D_SHIFT) - H_SHIFT);
            // (a workgroup that starts with a tile leaves a number unused behind the piece before it)
            if (s0 == 0 && at == line.start(g) && g > 0) o[-TILE] = 0.0;
        }
        at += s1 - s0;
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
}

// row_loss[i] = the share of the diagonal and the pieces of the tiles of its row; left in rows[i] for the total.  Four threads a row take every
// fourth piece each (one, 256 x 12288, 304 pieces a row: 27 us).
__global__ void __launch_bounds__(4 * TILE) loss_rows_kernel(const double *__restrict__ partial, const double *__restrict__ rdiag, LossLine line, long long n, double *rows,
                                                             double *row_loss, long long row_stride) {
    __shared__ double share[3][TILE];
    const int r = threadIdx.x % TILE, part = threadIdx.x / TILE, I = blockIdx.x;
    const long long i = (long long)I * TILE + r;
    const long long first = (long long)I * line.per_row;
    const long long p0 = (long long)I * line.tj + line.owner(first), p1 = (long long)I * line.tj + line.tj - 1 + line.owner(first + line.per_row - 1);
    double tot = part == 0 && i < n ? rdiag[i] : 0.0;
#pragma unroll 8
    for (long long p = p0 + part; p <= p1; p += 4) tot += partial[p * TILE + r];       // (there are numbers for whole tiles of rows)
    if (part > 0) share[part - 1][r] = tot;
    __syncthreads();
    if (part > 0 || i >= n) return;
    tot = ((tot + share[0][r]) + share[1][r]) + share[2][r];
    if (row_loss) row_loss[i * row_stride] = tot;
    rows[i] = tot;
}

// That and the total in one workgroup, for few and short rows: such a layer's call is mostly launches (4096 x 32 34 -> 32 us; 11008 rows
// take it 9 us, the two kernels 4 + 4.5 and the gap between them).
__global__ void __launch_bounds__(1024) loss_small_kernel(const double *__restrict__ partial, const double *__restrict__ rdiag, LossLine line, int n,
                                                          double *row_loss, double *loss) {
    __shared__ double sh[16];
    double acc = 0.0;
    const uint32_t per_row = (uint32_t)line.per_row, total = (uint32_t)line.total, G = (uint32_t)line.G, tj = (uint32_t)line.tj;
#pragma unroll 2
    for (int i = threadIdx.x; i < n; i += 1024) {
        const uint32_t I = (uint32_t)i >> 8, first = I * per_row;
        const uint32_t p0 = I * tj + ((first + 1) * G - 1) / total, p1 = I * tj + tj - 1 + ((first + per_row) * G - 1) / total;
        double tot = rdiag[i];
#pragma unroll 4
        for (uint32_t p = p0; p <= p1; ++p) tot += partial[(size_t)p * TILE + (i & 255)];
        if (row_loss) row_loss[i] = tot;
        acc += tot;
    }
    for (int d = 32; d >= 1; d >>= 1) acc += __shfl_down(acc, d, 64);
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
        double s = 0.0;
        for (int w = 0; w < 16; ++w) s += sh[w];
        *loss = s;
    }
}

// loss = sum_i rows[i] (single workgroup, fixed order).
__global__ void __launch_bounds__(1024) loss_total_kernel(const double *rows, long long n, double *loss) {
    __shared__ double sh[16];
    double acc = 0.0;
    for (long long i = threadIdx.x; i < n; i += 1024) acc += rows[i];
    for (int d = 32; d >= 1; d >>= 1) acc += __shfl_down(acc, d, 64);
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
        double s = 0.0;
        for (int w = 0; w < 16; ++w) s += sh[w];
        *loss = s;
    }
}

// Gradient terms.  P here is what dwh_kernel leaves (P without the diagonal's share) plus dW_ij H_jj, in float64.
// One workgroup walks STRIP consecutive rows; per row it forms
// Q_ik = sum_{j in k} P_ij alpha_j (LDS bins as in row_prep_kernel), then adds each column's term to the
// thread's private column sums.  A thread owns the columns tid, tid + 256, ...: with REG (m <= 16 * 256)
// their sums, alpha and the row's P and labels stay in registers, so a row is read from HBM once;
// otherwise the sums live in gpart and the row is read twice.  gpart[strip][l] is reduced over the strips
// afterwards.  The strip's share of the loss, sum P_ij dW_ij, falls out on the way.
// Column groups that lie outside the row cost nothing, and alpha and the diagonal are requested together: 11008 x 32 62 -> 46 us; 4096 x 4096 58,
// bound by the 13 bytes per weight; 256 x 12288 (not REG) 349 -> 294 with four columns in flight.
constexpr int GRAD_NC = 16;

template <bool REG, bool VEC>
__global__ void __launch_bounds__(PREP_THREADS) __attribute__((amdgpu_waves_per_eu(2, 2))) grad_rows_kernel(const float *W, const float *S, const float *alpha,
                                                                 long long n, long long m, long long ld,
                                                                 const uint8_t *labels, const float *P, const float *hdiag,
                                                                 const double *cent, const double *Den,
                                                                 double *gpart, double *lossp) {
    __shared__ double lsum[4];
    double lacc = 0.0;
    __shared__ double binQ[BIN_SETS][16];
    __shared__ double rsh[16], cshs[2][16];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const long long r0 = (long long)blockIdx.x * STRIP;
    double *gp = gpart + (long long)blockIdx.x * m;
    double gacc[GRAD_NC];
    float al[GRAD_NC];
    __shared__ __align__(16) float hds[REG ? GRAD_NC : 1][PREP_THREADS];      // a thread's diagonal entries (it alone reads them)
    // The columns of a thread (REG): tid, tid + 256, ... -- or, when the rows can be read 16 bytes at a time (VEC),
    // four groups of four neighbouring columns 4 (tid + 256 q) .. + 3: a quarter of the load instructions, and a
    // row then arrives in a third of the time.
    auto colof = [&](int c) -> long long {
        return VEC ? 4ll * (tid + (long long)(c >> 2) * PREP_THREADS) + (c & 3) : tid + (long long)c * PREP_THREADS;
    };
    auto any = [&](int c) { return (VEC ? 4 * PREP_THREADS * (c >> 2) : PREP_THREADS * c) < (int)m; };      // whether any thread has a column there
    if (REG) {
        float hd[GRAD_NC];         // (all requested before the first is used)
        if constexpr (VEC) {
#pragma unroll
            for (int q = 0; q < GRAD_NC / 4; ++q) {
                const long long l = min(colof(4 * q), m - 4);
                const float4 a4 = *(const float4 *)(alpha + l), h4 = *(const float4 *)(hdiag + l);
                al[4 * q] = a4.x; al[4 * q + 1] = a4.y; al[4 * q + 2] = a4.z; al[4 * q + 3] = a4.w;
                hd[4 * q] = h4.x; hd[4 * q + 1] = h4.y; hd[4 * q + 2] = h4.z; hd[4 * q + 3] = h4.w;
            }
        } else {
#pragma unroll
            for (int c = 0; c < GRAD_NC; ++c) {
                const long long l = min(colof(c), m - 1);
                al[c] = alpha[l];
                hd[c] = hdiag[l];
            }
        }
#pragma unroll
        for (int c = 0; c < GRAD_NC; ++c) {
            const bool in = colof(c) < m;
            gacc[c] = 0.0;
            al[c] = in ? al[c] : 0.0f;
            asm("" : "+v"(al[c]));
            hds[c][tid] = in ? hd[c] : 0.0f;
        }
    } else {
        for (long long l = tid; l < m; l += PREP_THREADS) gp[l] = 0.0;
    }
    double *myQ = binQ[wave * BIN_COPIES + (lane & (BIN_COPIES - 1))];
    // a row's centroids are requested while the row before it is worked on
    double cen_k = tid < 16 ? cent[r0 * 16 + tid] : 0.0;
    for (long long row = r0; row < min(n, r0 + STRIP); ++row) {
        double *csh = cshs[row & 1];
        const float *Pr = P + row * m;
        const uint8_t *Lr = labels + row * m;
        const float *Wr = W + row * ld, *Sr = S + row * ld;
        (&binQ[0][0])[tid] = 0.0;
        // the row's cluster masses are requested now by the 16 threads that need them between the
        // barriers below, where every other thread waits for them
        double den_k = 0.0;
        if (tid < 16) {
            den_k = Den[row * 16 + tid];
            csh[tid] = cen_k;
            if (row + 1 < min(n, r0 + STRIP)) cen_k = cent[(row + 1) * 16 + tid];
        }
        __syncthreads();      // bins cleared; the previous row's rsh is no longer read
        float pv[GRAD_NC], wv[GRAD_NC], sv[GRAD_NC];
        double pd[GRAD_NC];
        int lv[GRAD_NC];
        if (REG) {
            if constexpr (VEC) {
#pragma unroll
                for (int q = 0; q < GRAD_NC / 4; ++q) {
                    const long long l = colof(4 * q);
                    float4 p4 = make_float4(0.f, 0.f, 0.f, 0.f), w4 = p4, s4 = p4;
                    uint32_t l4 = 0u;
                    if (l < m) {          // m is a multiple of 4 here: the four columns are inside together
                        p4 = *(const float4 *)(Pr + l);
                        w4 = *(const float4 *)(Wr + l);
                        s4 = *(const float4 *)(Sr + l);
                        l4 = *(const uint32_t *)(Lr + l);
                    }
                    pv[4 * q] = p4.x; pv[4 * q + 1] = p4.y; pv[4 * q + 2] = p4.z; pv[4 * q + 3] = p4.w;
                    wv[4 * q] = w4.x; wv[4 * q + 1] = w4.y; wv[4 * q + 2] = w4.z; wv[4 * q + 3] = w4.w;
                    sv[4 * q] = s4.x; sv[4 * q + 1] = s4.y; sv[4 * q + 2] = s4.z; sv[4 * q + 3] = s4.w;
                    lv[4 * q] = (int)(l4 & 15u); lv[4 * q + 1] = (int)((l4 >> 8) & 15u);
                    lv[4 * q + 2] = (int)((l4 >> 16) & 15u); lv[4 * q + 3] = (int)((l4 >> 24) & 15u);
                }
            } else {
#pragma unroll
                for (int c = 0; c < GRAD_NC; ++c) {
                    const long long l = colof(c);
                    const bool in = l < m;
                    pv[c] = in ? Pr[l] : 0.0f;
                    lv[c] = in ? (Lr[l] & 15) : 0;
                    wv[c] = in ? Wr[l] : 0.0f;
                    sv[c] = in ? Sr[l] : 0.0f;
                }
            }
#pragma unroll
            for (int c = 0; c < GRAD_NC; ++c) asm("" : "+v"(pv[c]), "+v"(wv[c]), "+v"(sv[c]));      // (not converted to doubles until used: registers)
#pragma unroll
            for (int c = 0; c < GRAD_NC; ++c) {
                if (!any(c)) continue;
                const double dw = (double)wv[c] - (double)al[c] * csh[lv[c]];
                pd[c] = fma(dw, (double)hds[c][tid], (double)pv[c]);
                lacc = fma(pd[c], dw, lacc);        // (columns past the row: all zero)
                if (colof(c) < m) atomicAdd(&myQ[lv[c]], pd[c] * (double)al[c]);
            }
        } else {
#pragma unroll 4
            for (long long j = tid; j < m; j += PREP_THREADS) {
                const int k = Lr[j] & 15;
                const double a = (double)alpha[j], dw = (double)Wr[j] - a * csh[k], p = fma(dw, (double)hdiag[j], (double)Pr[j]);
                lacc = fma(p, dw, lacc);
                atomicAdd(&myQ[k], p * a);
            }
        }
        __syncthreads();
        if (tid < 16) {
            const double q = bin_total(binQ, tid), d = den_k;
            rsh[tid] = d > 0.0 ? q / d : 0.0;
        }
        __syncthreads();
        if (REG) {
#pragma unroll
            for (int c = 0; c < GRAD_NC; ++c) {
                if (!any(c)) continue;
                const double a = (double)al[c], cc = csh[lv[c]];
                const double term = pd[c] * cc + rsh[lv[c]] * (double)sv[c] * ((double)wv[c] - 2.0 * a * cc);
                gacc[c] += -2.0 * term;
            }
        } else {
#pragma unroll 4
            for (long long l = tid; l < m; l += PREP_THREADS) {
                const int k = Lr[l] & 15;
                const double a = (double)alpha[l], cc = csh[k];
                const double p = fma((double)Wr[l] - a * cc, (double)hdiag[l], (double)Pr[l]);
                const double term = p * cc + rsh[k] * (double)Sr[l] * ((double)Wr[l] - 2.0 * a * cc);
                gp[l] += -2.0 * term;   // the same thread owns column l for every row of the strip
            }
        }
    }
    if (REG) {
#pragma unroll
        for (int c = 0; c < GRAD_NC; ++c) {
            const long long l = colof(c);
            if (l < m) gp[l] = gacc[c];
        }
    }
    const double l = block_sum_256(lacc, lsum);
    if (tid == 0) lossp[blockIdx.x] = l;
}

// Column sums of the per-strip gradient terms, then the Adam update.  16 columns per workgroup (m / 16 workgroups:
// one per CU at 4096 columns); the strips are shared out to 64 groups of threads (a column's 64 partial sums are
// added in a fixed order).  One more workgroup adds up the strips' shares of the loss.
constexpr int ADAM_COLS = 16, ADAM_GROUPS = 64;

__global__ void __launch_bounds__(ADAM_COLS * ADAM_GROUPS) adam_kernel(const double *gpart, int nstrip, long long m,
                                                                      float *alpha, float *am, float *av, float lr,
                                                                      float beta1, float beta2, float eps, float bc1,
                                                                      float bc2, float *grad_out, const double *lossp, double *loss) {
    __shared__ double part[ADAM_GROUPS][ADAM_COLS];
    if (blockIdx.x == gridDim.x - 1) {
        double *sh = &part[0][0];
        double a = 0.0;
        for (int i = threadIdx.x; i < nstrip; i += ADAM_COLS * ADAM_GROUPS) a += lossp[i];
        for (int d = 32; d >= 1; d >>= 1) a += __shfl_down(a, d, 64);
        if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = a;
        __syncthreads();
        if (threadIdx.x == 0) {
            double s = 0.0;
            for (int w = 0; w < ADAM_COLS * ADAM_GROUPS / 64; ++w) s += sh[w];
            *loss = s;
        }
        return;
    }
    const int c = threadIdx.x % ADAM_COLS, g = threadIdx.x / ADAM_COLS;
    const long long l = (long long)blockIdx.x * ADAM_COLS + c;
    double acc = 0.0;
    if (l < m)
        for (int st = g; st < nstrip; st += ADAM_GROUPS) acc += gpart[(long long)st * m + l];
    part[g][c] = acc;
    __syncthreads();
    if (g != 0 || l >= m) return;
    double g64 = 0.0;
#pragma unroll
    for (int k = 0; k < ADAM_GROUPS; ++k) g64 += part[k][c];
    const float gr = (float)g64;
    if (grad_out) grad_out[l] = gr;
    const float m1 = beta1 * am[l] + (1.0f - beta1) * gr;
    const float v1 = beta2 * av[l] + (1.0f - beta2) * gr * gr;
    am[l] = m1;
    av[l] = v1;
    const float mh = m1 / bc1, vh = v1 / bc2;
    alpha[l] = alpha[l] - lr * mh / (sqrtf(vh) + eps);
}

struct LossWs {
    float *P;                // dW H without the diagonal of H
    uint16_t *dWp, *Hp;      // pieces of dW and of H
    uint32_t *hmax;          // largest couplings of H (the channels' scales)
    float *hdiag;            // the diagonal of H
    int *rexp;               // exponents of the rows of dW
    double *rdiag;           // the rows' losses on the diagonal
    double *cent, *Den, *partial, *rows, *gpart, *lossp;
    floatx4 *slots;
    TilePlan plan;
    LossLine line;
    int nstrip, tj;
    long long tiles;
};

// The plan of dwh_kernel; whole tiles go straight into P, only the parts of split ones have slots.  Returns their number.
long long dwh_plan(TilePlan &plan, int64_t n, int64_t m, int num_cu) {
    const long long tiles = (n + TILE - 1) / TILE * ((m + TILE - 1) / TILE);
    (void)skim_make_plan(plan, num_cu, tiles, (int)(m / GK), G_MIN_STAGES, G_PHASE_COST, false);
    long long slots = 0;
    for (int p = 0; p < plan.nph; ++p) {
        plan.slot0[p] = (int)slots;
        if (plan.split[p] > 1) slots += (long long)plan.ntile[p] * plan.split[p];
    }
    return slots;
}

// grad: what a scale step needs (P and the gradient's partial sums) instead of what the loss needs
skim_status carve(skim_ctx *ctx, int64_t n, int64_t m, bool grad, LossWs &w) {
    skim_ws_cursor cur{(char *)ctx->ws, 0, ctx->ws_bytes};
    w.nstrip = (int)((n + STRIP - 1) / STRIP);
    w.tj = (int)((m + TILE - 1) / TILE);
    w.tiles = (n + TILE - 1) / TILE * w.tj;
    // (H first: skim_train_scale and skim_error_table_lfull keep its pieces across their steps)
    w.Hp = (uint16_t *)cur.take((size_t)m * m * 2 * sizeof(uint16_t));
    w.hmax = (uint32_t *)cur.take((size_t)m * sizeof(uint32_t));
    w.hdiag = (float *)cur.take((size_t)m * sizeof(float));
    w.dWp = (uint16_t *)cur.take(plane_rows(n) * m * 2 * sizeof(uint16_t));
    w.rexp = (int *)cur.take((((size_t)n + TILE - 1) & ~(size_t)(TILE - 1)) * sizeof(int));
    w.cent = (double *)cur.take((size_t)n * 16 * sizeof(double));
    w.Den = (double *)cur.take((size_t)n * 16 * sizeof(double));
    bool ok = w.dWp && w.Hp && w.hmax && w.hdiag && w.rexp && w.cent && w.Den;
    if (grad) {
        w.P = (float *)cur.take((size_t)n * m * sizeof(float));
        w.gpart = (double *)cur.take((size_t)w.nstrip * m * sizeof(double));
        w.lossp = (double *)cur.take((size_t)w.nstrip * sizeof(double));
        const long long slots = dwh_plan(w.plan, n, m, ctx->num_cu);
        w.slots = (floatx4 *)cur.take((size_t)slots * TILE_SLOT_BYTES);
        if (!w.slots) (void)skim_make_plan(w.plan, ctx->num_cu, w.tiles, (int)(m / GK), G_MIN_STAGES, G_PHASE_COST, true);
        ok = ok && w.P && w.gpart && w.lossp;
    } else {
        w.line = loss_line(n, m, ctx->num_cu);
        w.partial = (double *)cur.take((size_t)(w.tiles + w.line.G) * TILE * sizeof(double));
        w.rows = (double *)cur.take((size_t)n * sizeof(double));
        w.rdiag = (double *)cur.take((size_t)n * sizeof(double));
        ok = ok && w.partial && w.rows && w.rdiag;
    }
    if (!ok) SKIM_FAIL(ctx, SKIM_ERR_WORKSPACE, "workspace missing or smaller than skim_workspace_bytes(n, m)");
    return SKIM_OK;
}

skim_status enable_lds(skim_ctx *ctx) {
    if (ctx->gemm3_lds_enabled) return SKIM_OK;
    SKIM_HIP(ctx, hipFuncSetAttribute((const void *)dwh_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)G_LDS_BYTES));
    SKIM_HIP(ctx, hipFuncSetAttribute((const void *)dwh_loss_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)G_LDS_BYTES));
    ctx->gemm3_lds_enabled = 1;
    return SKIM_OK;
}

void launch_split(skim_ctx *ctx, const LossWs &w, const float *H, int64_t m, SplitMode mode) {
    hipLaunchKernelGGL(split_rows_kernel, dim3((unsigned)split_tiles(m)), dim3(SPLIT_THREADS), 0, ctx->stream, H, (long long)m, (const uint32_t *)w.hmax, w.Hp,
                       (int)mode);
}
void launch_hmax(skim_ctx *ctx, const LossWs &w, const float *H, int64_t m) {
    if (m <= HMAX_DIRECT) {
        hipLaunchKernelGGL(hmax_direct_kernel, dim3((unsigned)(m / 16)), dim3(256), 0, ctx->stream, H, (int)m, w.hmax, w.hdiag);
        return;
    }
    const int64_t tx = (m + HMAX_COLS - 1) / HMAX_COLS, ty = (m + HMAX_ROWS - 1) / HMAX_ROWS;
    hipLaunchKernelGGL(hmax_clear_kernel, dim3((unsigned)((m + 255) / 256)), dim3(256), 0, ctx->stream, H, (long long)m, w.hmax, w.hdiag);
    hipLaunchKernelGGL(hmax_kernel, dim3((unsigned)(tx * ty)), dim3(256), 0, ctx->stream, H, (long long)m, (int)tx, w.hmax);
}
// P = dW H, and with rows of H for its columns only where H has to be symmetric (m a multiple of 32 from 128 up)
SplitMode step_split(int64_t m) { return (m % 32) != 0 || m < 128 ? SPLIT_COLUMNS : SPLIT_ROWS; }

// rows of W and S start 16-byte aligned, alpha is, and the labels of a row start 4-byte aligned (m is a multiple of 16)
bool rows_vec4(const float *W, const float *S, const float *alpha, const uint8_t *labels, int64_t ld) {
    return (ld % 4) == 0 && (((uintptr_t)W | (uintptr_t)S | (uintptr_t)alpha) & 15) == 0 && ((uintptr_t)labels & 3) == 0;
}

// split: what to cut H into as well (the caller launches it where it is still to be done on return)
template <int BITS, bool DIAG>
void launch_row_prep_bits(skim_ctx *ctx, const float *W, const float *S, const float *alpha, int64_t n, int64_t m, int64_t ld,
                          const uint8_t *labels, const skim_label_bounds &bd, const LossWs &w, const float *H, bool &split, SplitMode mode) {
    const bool vec4 = rows_vec4(W, S, alpha, BITS == 0 ? labels : bd.labels_out, ld);
    const long long groups = (n + ROWP_ROWS - 1) / ROWP_ROWS;
    auto launch = [&](auto keep, auto wpr, long long blocks) {
        constexpr int WPR = decltype(wpr)::value;
        hipLaunchKernelGGL((row_prep_kernel<BITS, decltype(keep)::value, WPR, DIAG>), dim3((unsigned)blocks), dim3(64 * ROWP_ROWS * WPR), 0, ctx->stream,
                           W, S, alpha, (long long)n, (long long)m, (long long)ld, labels, bd.upper, (long long)bd.upper_stride, bd.labels_out,
                           w.cent, w.Den, w.dWp, bd.centroids, (long long)bd.centroid_stride, vec4, H, (const uint32_t *)w.hmax, w.Hp, (int)mode, w.rexp,
                           (const float *)w.hdiag, w.rdiag);
    };
    using four = std::integral_constant<int, 4>;
    if (m <= ROWP_NARROW) {
        launch(std::integral_constant<int, 1>{}, std::integral_constant<int, 1>{}, groups + (split ? split_tiles(m) : 0));
        split = false;
    } else if (m <= 4 * 1024) launch(std::integral_constant<int, 4>{}, four{}, groups);
    else if (m <= 11 * 1024) launch(std::integral_constant<int, 11>{}, four{}, groups);
    else launch(std::integral_constant<int, 0>{}, four{}, groups);
}
void launch_row_prep(skim_ctx *ctx, const float *W, const float *S, const float *alpha, int64_t n, int64_t m, int64_t ld,
                     const uint8_t *labels, const skim_label_bounds &bd, const LossWs &w, const float *H, bool split,
                     SplitMode mode) {
    if (split) launch_hmax(ctx, w, H, m);
    switch (bd.bits) {
        case 0:
            if (mode == SPLIT_LOWER) launch_row_prep_bits<0, true>(ctx, W, S, alpha, n, m, ld, labels, bd, w, H, split, mode);
            else launch_row_prep_bits<0, false>(ctx, W, S, alpha, n, m, ld, labels, bd, w, H, split, mode);
            break;
        case 1: launch_row_prep_bits<1, true>(ctx, W, S, alpha, n, m, ld, labels, bd, w, H, split, mode); break;
        case 2: launch_row_prep_bits<2, true>(ctx, W, S, alpha, n, m, ld, labels, bd, w, H, split, mode); break;
        case 3: launch_row_prep_bits<3, true>(ctx, W, S, alpha, n, m, ld, labels, bd, w, H, split, mode); break;
        default: launch_row_prep_bits<4, true>(ctx, W, S, alpha, n, m, ld, labels, bd, w, H, split, mode); break;
    }
    if (split) launch_split(ctx, w, H, m, mode);
}

skim_status check_shape(skim_ctx *ctx, int64_t n, int64_t m, int64_t ld) {
    if (n < 1 || n > 0x7fffffff || m < GK || m > 0x7fffffff || ld < m || (m % GK) != 0)
        SKIM_FAIL(ctx, SKIM_ERR_SHAPE, "layer loss needs n >= 1, m a multiple of %d, ld >= m (n=%lld m=%lld ld=%lld)", GK,
                  (long long)n, (long long)m, (long long)ld);
    return SKIM_OK;
}

}  // namespace

// A bound that grows with n and m, so that a workspace made for the largest layer serves every smaller one: the plan cuts a
// tile into stages of at least G_MIN_STAGES, and no more than PLAN_SPLIT_PHASES of its phases hold split tiles, each at
// most one piece per compute unit (256 of them).
size_t skim_dwh_slot_bytes(int64_t n, int64_t m) {
    const int64_t maxsplit = m / GK / G_MIN_STAGES, most = PLAN_SPLIT_PHASES * 256;
    if (n < 1 || maxsplit < 2) return 0;
    const int64_t ti = (n + TILE - 1) / TILE, tj = (m + TILE - 1) / TILE;
    if (ti >= most || tj >= most || maxsplit >= most) return (size_t)most * TILE_SLOT_BYTES;
    const int64_t slots = ti * tj * maxsplit;
    return (size_t)(slots < most ? slots : most) * TILE_SLOT_BYTES;
}

extern "C" skim_status skim_layer_loss(skim_ctx *ctx, const float *W, const float *S, const float *alpha,
                                       const float *H, int64_t n, int64_t m, int64_t ld, const uint8_t *labels,
                                       double *loss, double *row_loss) {
    if (ctx && !loss) SKIM_FAIL(ctx, SKIM_ERR_ARG, "skim_layer_loss: NULL argument");
    return skim_layer_loss_strided(ctx, W, S, alpha, H, n, m, ld, labels, skim_label_bounds{}, loss, row_loss, 1, false);
}

skim_status skim_layer_loss_strided(skim_ctx *ctx, const float *W, const float *S, const float *alpha, const float *H,
                                    int64_t n, int64_t m, int64_t ld, const uint8_t *labels, const skim_label_bounds &bounds, double *loss,
                                    double *row_loss, int64_t row_stride, bool h_ready) {
    skim_status st = skim_enter(ctx);
    if (st != SKIM_OK) return st;
    if (!W || !S || !H || (!labels && !bounds.upper)) SKIM_FAIL(ctx, SKIM_ERR_ARG, "skim_layer_loss: NULL argument");
    if ((st = check_shape(ctx, n, m, ld)) != SKIM_OK) return st;
    if ((uintptr_t)H & 15) SKIM_FAIL(ctx, SKIM_ERR_ARG, "skim_layer_loss: H must be 16-byte aligned");
    LossWs w;
    if ((st = carve(ctx, n, m, false, w)) != SKIM_OK) return st;
    if ((st = enable_lds(ctx)) != SKIM_OK) return st;
    launch_row_prep(ctx, W, S, alpha, n, m, ld, labels, bounds, w, H, !h_ready, SPLIT_LOWER);
    hipLaunchKernelGGL(dwh_loss_kernel, dim3((unsigned)w.line.G), dim3(G_THREADS), G_LDS_BYTES, ctx->stream, w.dWp, w.Hp, (const int *)w.rexp,
                       (long long)n, (long long)m, w.line, w.partial);
    // one launch for what takes hardly longer than that (numbers to add up: those of the tiles, and a row of tiles is cut into up to cuts + 1)
    const long long cuts = (w.line.G * (long long)TILE + n - 1) / n + 1;
    if (loss && row_stride == 1 && n * (w.line.tj + cuts) <= LOSS_SMALL && w.line.total * w.line.G <= 0x7fffffff) {
        hipLaunchKernelGGL(loss_small_kernel, dim3(1), dim3(1024), 0, ctx->stream, (const double *)w.partial, (const double *)w.rdiag, w.line, (int)n, row_loss,
                           loss);
        SKIM_HIP(ctx, hipGetLastError());
        return SKIM_OK;
    }
    hipLaunchKernelGGL(loss_rows_kernel, dim3((unsigned)((n + TILE - 1) / TILE)), dim3(4 * TILE), 0, ctx->stream, (const double *)w.partial,
                       (const double *)w.rdiag, w.line, (long long)n, w.rows, row_loss, (long long)row_stride);
    if (loss) hipLaunchKernelGGL(loss_total_kernel, dim3(1), dim3(1024), 0, ctx->stream, (const double *)w.rows, (long long)n, loss);
    SKIM_HIP(ctx, hipGetLastError());
    return SKIM_OK;
}

namespace {
skim_status scale_step_impl(skim_ctx *ctx, const float *W, const float *S, const float *H, int64_t n, int64_t m,
                            int64_t ld, const uint8_t *labels, float *alpha, float *adam_m, float *adam_v, int64_t t,
                            const skim_adam_opts *opts, double *loss_before, float *grad_out, bool h_ready);
}

extern "C" skim_status skim_scale_step(skim_ctx *ctx, const float *W, const float *S, const float *H, int64_t n,
                                       int64_t m, int64_t ld, const uint8_t *labels, float *alpha, float *adam_m,
                                       float *adam_v, int64_t t, const skim_adam_opts *opts, double *loss_before,
                                       float *grad_out) {
    return scale_step_impl(ctx, W, S, H, n, m, ld, labels, alpha, adam_m, adam_v, t, opts, loss_before, grad_out, false);
}

namespace {
skim_status scale_step_impl(skim_ctx *ctx, const float *W, const float *S, const float *H, int64_t n, int64_t m,
                            int64_t ld, const uint8_t *labels, float *alpha, float *adam_m, float *adam_v, int64_t t,
                            const skim_adam_opts *opts, double *loss_before, float *grad_out, bool h_ready) {
    skim_status st = skim_enter(ctx);
    if (st != SKIM_OK) return st;
    if (!W || !S || !H || !labels || !alpha || !adam_m || !adam_v || !opts || !loss_before)
        SKIM_FAIL(ctx, SKIM_ERR_ARG, "skim_scale_step: NULL argument");
    if (t < 1 || opts->decay_every < 1) SKIM_FAIL(ctx, SKIM_ERR_ARG, "skim_scale_step: t and decay_every must be >= 1");
    if ((st = check_shape(ctx, n, m, ld)) != SKIM_OK) return st;
    if ((uintptr_t)H & 15) SKIM_FAIL(ctx, SKIM_ERR_ARG, "skim_scale_step: H must be 16-byte aligned");
    LossWs w;
    if ((st = carve(ctx, n, m, true, w)) != SKIM_OK) return st;
    if ((st = enable_lds(ctx)) != SKIM_OK) return st;
    launch_row_prep(ctx, W, S, alpha, n, m, ld, labels, skim_label_bounds{}, w, H, !h_ready, step_split(m));
    {
        long long grid = 0;
        for (int p = 0; p < w.plan.nph; ++p) grid = max(grid, (long long)w.plan.ntile[p] * w.plan.split[p]);
        if (grid > ctx->num_cu) grid = ctx->num_cu;
        hipLaunchKernelGGL(dwh_kernel, dim3((unsigned)grid), dim3(G_THREADS), G_LDS_BYTES, ctx->stream, w.dWp, w.Hp, (const int *)w.rexp,
                           (const uint32_t *)w.hmax, (long long)n, (long long)m, w.tj, w.plan, w.P, w.slots);
        for (int p = 0; p < w.plan.nph; ++p)
            if (w.plan.split[p] > 1)
                hipLaunchKernelGGL(dwh_parts_kernel, dim3((unsigned)(w.plan.ntile[p] * 16)), dim3(256), 0, ctx->stream, w.P,
                                   (const int *)w.rexp, (const uint32_t *)w.hmax, (long long)n, (long long)m, w.tj, w.plan, p, (const floatx4 *)w.slots);
    }
    // rows of W, S, P start 16-byte aligned and the labels of a row 4-byte aligned (m is a multiple of 16)
    const bool vec4 = rows_vec4(W, S, alpha, labels, ld) && ((uintptr_t)w.P & 15) == 0;
    auto grad = [&](auto reg, auto vec) {
        hipLaunchKernelGGL((grad_rows_kernel<decltype(reg)::value, decltype(vec)::value>), dim3(w.nstrip), dim3(PREP_THREADS), 0, ctx->stream, W, S,
                           (const float *)alpha, (long long)n, (long long)m, (long long)ld, labels, (const float *)w.P, (const float *)w.hdiag,
                           (const double *)w.cent, (const double *)w.Den, w.gpart, w.lossp);
    };
    if (m > (int64_t)GRAD_NC * PREP_THREADS) grad(std::false_type{}, std::false_type{});
    else if (vec4) grad(std::true_type{}, std::true_type{});
    else grad(std::true_type{}, std::false_type{});
    const double lr = (double)opts->lr0 * pow((double)opts->decay, (double)((t - 1) / opts->decay_every));
    const double bc1 = 1.0 - pow((double)opts->beta1, (double)t), bc2 = 1.0 - pow((double)opts->beta2, (double)t);
    hipLaunchKernelGGL(adam_kernel, dim3((unsigned)((m + ADAM_COLS - 1) / ADAM_COLS) + 1u), dim3(ADAM_COLS * ADAM_GROUPS), 0, ctx->stream, w.gpart, w.nstrip,
                       (long long)m, alpha, adam_m, adam_v, (float)lr, opts->beta1, opts->beta2, opts->eps, (float)bc1,
                       (float)bc2, grad_out, (const double *)w.lossp, loss_before);
    SKIM_HIP(ctx, hipGetLastError());
    return SKIM_OK;
}
}  // namespace

// Scaling-vector training (Alg. 2): `outer` rounds of { labels = K-means of W * alpha^-1 at the given bit
// widths; `steps` optimiser steps on alpha with the labels fixed }, then the centroids and the loss at the
// final alpha.  Composition of skim_cluster_rows, skim_scale_step and the layer-loss kernels.
extern "C" skim_status skim_train_scale(skim_ctx *ctx, const float *W, const float *S, const float *H, int64_t n,
                                        int64_t m, int64_t ld, const uint8_t *bits, int kmeans_iters, int outer,
                                        int steps, int64_t t0, const skim_adam_opts *opts, float *alpha,
                                        float *adam_m, float *adam_v, uint8_t *labels, double *centroids,
                                        double *loss_trace) {
    skim_status st = skim_enter(ctx);
    if (st != SKIM_OK) return st;
    if (!W || !S || !H || !bits || !opts || !alpha || !adam_m || !adam_v || !labels || !centroids || !loss_trace)
        SKIM_FAIL(ctx, SKIM_ERR_ARG, "skim_train_scale: NULL argument");
    if (outer < 1 || steps < 0 || t0 < 1 || kmeans_iters < 1)
        SKIM_FAIL(ctx, SKIM_ERR_ARG, "skim_train_scale: need outer >= 1, steps >= 0, t0 >= 1, kmeans_iters >= 1");
    if (ctx->ws_bytes < skim_workspace_least(n, m))
        SKIM_FAIL(ctx, SKIM_ERR_WORKSPACE, "workspace missing or smaller than skim_workspace_bytes(n, m)");
    // per-row clustering outputs that the caller does not ask for live at the tail of the workspace
    // (the calls below carve from its start)
    const size_t tail_bytes = (((size_t)n * 16 * sizeof(float) + 255) & ~(size_t)255) +
                              (((size_t)n * sizeof(double) + 255) & ~(size_t)255);
    char *tail = (char *)ctx->ws + ((ctx->ws_bytes - tail_bytes) & ~(size_t)255);
    float *upper = (float *)tail;
    double *err = (double *)(tail + (((size_t)n * 16 * sizeof(float) + 255) & ~(size_t)255));
    int64_t t = t0;
    int64_t slot = 0;
    for (int round = 0; round < outer; ++round) {
        if ((st = skim_cluster_rows(ctx, W, S, alpha, n, m, ld, bits, kmeans_iters, labels, centroids, upper, err)) !=
            SKIM_OK)
            return st;
        // H is cut into its pieces once per round (the re-clustering has written over that part of the workspace)
        for (int k = 0; k < steps; ++k, ++t, ++slot) {
            if ((st = scale_step_impl(ctx, W, S, H, n, m, ld, labels, alpha, adam_m, adam_v, t, opts, loss_trace + slot,
                                      nullptr, k > 0)) != SKIM_OK)
                return st;
        }
    }
    // centroids of the fixed labels at the final alpha, and the loss there
    if ((st = check_shape(ctx, n, m, ld)) != SKIM_OK) return st;
    LossWs w;
    if ((st = carve(ctx, n, m, false, w)) != SKIM_OK) return st;
    // (the loss takes other pieces of H than the steps)
    if ((st = skim_layer_loss_strided(ctx, W, S, alpha, H, n, m, ld, labels, skim_label_bounds{}, loss_trace + slot, nullptr, 1, false)) !=
        SKIM_OK)
        return st;
    SKIM_HIP(ctx, hipMemcpyAsync(centroids, w.cent, (size_t)n * 16 * sizeof(double), hipMemcpyDeviceToDevice, ctx->stream));
    return SKIM_OK;
}
