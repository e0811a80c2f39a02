// Readers of the packed model (Sec. 4.2 last paragraph and App. D.2: rows of equal bit width
// are gathered and processed together; Sec. 5.4: binary16 codebooks): dequantisation to a
// dense matrix and the matrix-vector product that looks every weight up in its row's
// codebook.  Both walk the layout skim_pack writes: rows by (bits, row index), a b-bit row =
// ceil(m*b/32) little-endian words, column j at bit j*b.
#include "skim_common.h"

#include <hip/hip_fp16.h>

#include <type_traits>

namespace {

constexpr int UNPACK_THREADS = 256;

struct RowPlace {        // where packed row p lives
    int b;               // its bit width
    long long word0;     // first code word
    long long cb0;       // first codebook entry
};

// group_word_offset[b] .. [b+1] holds the b-bit rows, each ceil(m*b/32) words.  (The number of rows is a quotient without
// a remainder of two numbers below 2^53: the float64 division returns it exactly, in a tenth of the instructions of the
// 64-bit integer one, which every workgroup went through four times before it could ask for its first code.)
__device__ __forceinline__ RowPlace place_row(const long long *gwo, long long m, long long p) {
    RowPlace r{0, 0, 0};
    long long rows_before = 0, cb = 0;
    for (int b = 1; b <= 4; ++b) {
        const long long wpr = (m * b + 31) / 32;
        const long long rows = (long long)((double)(gwo[b + 1] - gwo[b]) / (double)wpr);
        if (p < rows_before + rows) {
            r.b = b;
            r.word0 = gwo[b] + (p - rows_before) * wpr;
            r.cb0 = cb + (p - rows_before) * (1ll << b);
            return r;
        }
        rows_before += rows;
        cb += rows * (1ll << b);
    }
    return r;   // b == 0: p is past the last row
}

// The dense matrix, bound by the 4 bytes written per weight.  A row is cut into segments of up to 4096 columns (multiples of 32: a
// segment's codes are whole words); a workgroup takes one segment of every so many rows.  The codes, codebook and index of its
// next row are on their way while the current one is written: with one workgroup per row and its codes asked for step by step,
// codes that are not in a cache cost four trips to memory in a row, twice over.  The words go through LDS; a thread expands four
// neighbouring columns at a time into one 16-byte store.  The columns ahead of the first 16-byte border of the segment (any m, any
// address of Wq) and behind the last whole four go one by one.  ALIGNED: m is a multiple of 4, so the borders are the same in every row
// and alpha stays in registers.
// STREAM: stores that pass the caches by.  A matrix that the 256 MB of the last cache hold stays there for whoever reads it next, which costs a
// call whose outputs are not read 12 us at 180 MB (each evicts an older one) and saves the reader more; a larger one would only
// drive itself out.  us with alpha, codes of four layers in turn, alone / with torch.mv behind it, streamed and not: 4096 x 4096 18 / 43 and
// 18 / 36, 4096 x 11008 40 / 96 and 37 / 78 (every output in memory of its own: 37 and 48), 5120 x 11008 49 / 131 and 57 / 106, 5632 x 11008
// 53 / 140 and 63 / 132, 6144 x 11008 58 / 149 and 69 / 155, 8192 x 22016 164 / 376 and 188 / 414.  One workgroup per row, 4096 x 11008: 43 / 78, in
// memory of its own 68.
constexpr int64_t UNPACK_CACHED_BYTES = 240ll << 20;
constexpr uint32_t UNPACK_SEGMENT = 4096;
constexpr int UNPACK_QUADS = UNPACK_SEGMENT / (4 * UNPACK_THREADS);       // of a thread, at most
constexpr int UNPACK_WORDS = UNPACK_SEGMENT * 4 / 32 / UNPACK_THREADS;    // of a thread, at 4 bits

typedef float float4v __attribute__((ext_vector_type(4)));

template <int B, bool ALPHA, bool ALIGNED, bool STREAM>
__device__ __forceinline__ void unpack_segment(const uint32_t *words, const float *cbf, uint32_t cols, uint32_t head, bool alpha_vec,
                                               const float *__restrict__ alpha, const float4 (&al)[UNPACK_QUADS], float *__restrict__ out) {
    const uint32_t tid = threadIdx.x;
    const uint32_t quads = (cols - head) >> 2;
    constexpr uint32_t mask = (1u << B) - 1u;
#pragma unroll
    for (int u = 0; u < UNPACK_QUADS; ++u) {
        const uint32_t q = tid + u * UNPACK_THREADS;
        if (q < quads) {
            const uint32_t j = head + 4u * q, bit = j * B, wi = bit >> 5, sh = bit & 31u;
            const uint32_t v = (uint32_t)((((unsigned long long)words[wi + 1] << 32) | words[wi]) >> sh);      // (room for one word more)
            float4 c = make_float4(cbf[v & mask], cbf[(v >> B) & mask], cbf[(v >> (2 * B)) & mask], cbf[(v >> (3 * B)) & mask]);
            if (ALPHA) {
                float4 a = al[u];
                if (!ALIGNED) a = alpha_vec ? *(const float4 *)(alpha + j) : make_float4(alpha[j], alpha[j + 1], alpha[j + 2], alpha[j + 3]);
                c = make_float4(__fmul_rn(a.x, c.x), __fmul_rn(a.y, c.y), __fmul_rn(a.z, c.z), __fmul_rn(a.w, c.w));
            }
            if (STREAM) __builtin_nontemporal_store(float4v{c.x, c.y, c.z, c.w}, (float4v *)(out + j));
            else *(float4 *)(out + j) = c;
        }
    }
    // at most three columns at either end
    const uint32_t tail = head + 4u * quads;
    if (tid < head + (cols - tail)) {
        const uint32_t j = tid < head ? tid : tail + (tid - head);
        const uint32_t bit = j * B, wi = bit >> 5, sh = bit & 31u;
        const uint32_t x = (uint32_t)((((unsigned long long)words[wi + 1] << 32) | words[wi]) >> sh);
        const float c = cbf[x & mask];
        out[j] = ALPHA ? __fmul_rn(alpha[j], c) : c;
    }
}

template <bool ALPHA, bool ALIGNED, bool STREAM>
__global__ void __launch_bounds__(UNPACK_THREADS) unpack_kernel(const uint32_t *__restrict__ codes, const long long *__restrict__ gwo,
                                                               const int *__restrict__ row_perm, const uint16_t *__restrict__ codebooks,
                                                               const float *__restrict__ alpha, long long n, long long m, uint32_t seglen,
                                                               float *__restrict__ Wq) {
    __shared__ uint32_t words[2][UNPACK_WORDS * UNPACK_THREADS + 4];
    __shared__ float cbf[2][16];
    const uint32_t tid = threadIdx.x;
    const long long c0 = (long long)blockIdx.x * seglen;
    const uint32_t cols = (uint32_t)min((long long)seglen, m - c0);
    const uint32_t base = (uint32_t)((uintptr_t)Wq >> 2) & 3u;            // (c0 is a multiple of 4)
    auto head_of = [&](long long row) -> uint32_t {      // columns ahead of the first 16-byte border
        const uint32_t skew = ALIGNED ? 0u : (uint32_t)(((unsigned long long)row * (unsigned long long)m) & 3u);
        return min(cols, (0u - base - skew) & 3u);
    };
    // a row's words of this segment, its codebook and its index, on their way
    uint32_t w[UNPACK_WORDS];
    uint16_t cb = 0;
    int row = 0, bits = 0;
    auto fetch = [&](long long p) {
        bits = 0;
        if (p >= n) return;
        const RowPlace pl = place_row(gwo, m, p);
        bits = pl.b;
        if (bits == 0) return;
        const uint32_t count = (cols * (uint32_t)bits + 31u) >> 5;
        const uint32_t *rw = codes + pl.word0 + (c0 >> 5) * bits;
#pragma unroll
        for (int k = 0; k < UNPACK_WORDS; ++k) w[k] = tid + k * UNPACK_THREADS < count ? rw[tid + k * UNPACK_THREADS] : 0u;
        if (tid < (1u << bits)) cb = codebooks[pl.cb0 + tid];
        row = row_perm[p];
    };
    long long p = blockIdx.y;
    fetch(p);
    float4 al[UNPACK_QUADS];
    if (ALPHA && ALIGNED) {
        alpha += c0;
        const uint32_t head = head_of(0);
        const bool vec = (((uintptr_t)(alpha + head)) & 15) == 0;
#pragma unroll
        for (int u = 0; u < UNPACK_QUADS; ++u) {
            const uint32_t j = head + 4u * (tid + u * UNPACK_THREADS);
            al[u] = make_float4(0.f, 0.f, 0.f, 0.f);
            if (j + 4 <= cols) al[u] = vec ? *(const float4 *)(alpha + j) : make_float4(alpha[j], alpha[j + 1], alpha[j + 2], alpha[j + 3]);
        }
    } else if (ALPHA) {
        alpha += c0;
    }
    for (int buf = 0; bits != 0; buf ^= 1) {
#pragma unroll
        for (int k = 0; k < UNPACK_WORDS; ++k) words[buf][tid + k * UNPACK_THREADS] = w[k];
        if (tid < 16) cbf[buf][tid] = __half2float(__ushort_as_half(cb));
        __syncthreads();
        const int b = bits;
        const uint32_t head = head_of(row);
        float *out = Wq + (long long)row * m + c0;
        p += gridDim.y;
        fetch(p);
        const bool vec = ALPHA && !ALIGNED && (((uintptr_t)(alpha + head)) & 15) == 0;
        switch (b) {
            case 1: unpack_segment<1, ALPHA, ALIGNED, STREAM>(words[buf], cbf[buf], cols, head, vec, alpha, al, out); break;
            case 2: unpack_segment<2, ALPHA, ALIGNED, STREAM>(words[buf], cbf[buf], cols, head, vec, alpha, al, out); break;
            case 3: unpack_segment<3, ALPHA, ALIGNED, STREAM>(words[buf], cbf[buf], cols, head, vec, alpha, al, out); break;
            default: unpack_segment<4, ALPHA, ALIGNED, STREAM>(words[buf], cbf[buf], cols, head, vec, alpha, al, out); break;
        }
    }
}

// Segments of equal length, and as many workgroups as are resident at once (6 a compute unit), in equal numbers of rows.
void launch_unpack(skim_ctx *ctx, const uint32_t *codes, const int64_t *gwo, const int32_t *row_perm, const uint16_t *codebooks,
                   const float *alpha, int64_t n, int64_t m, float *Wq) {
    int64_t nseg = (m + UNPACK_SEGMENT - 1) / UNPACK_SEGMENT;
    const int64_t seglen = ((m + nseg - 1) / nseg + 31) / 32 * 32;
    nseg = (m + seglen - 1) / seglen;
    const int64_t resident = 6ll * ctx->num_cu, rounds = (n * nseg + resident - 1) / resident;
    const int64_t stride = (n + rounds - 1) / rounds;
    auto launch = [&](auto al, auto aligned, auto stream) {
        hipLaunchKernelGGL((unpack_kernel<decltype(al)::value, decltype(aligned)::value, decltype(stream)::value>), dim3((unsigned)nseg, (unsigned)stride), dim3(UNPACK_THREADS), 0,
                           ctx->stream, codes, (const long long *)gwo, row_perm, codebooks, alpha, (long long)n, (long long)m, (uint32_t)seglen, Wq);
    };
    auto pick_stores = [&](auto al, auto aligned) {
        if (n * m > UNPACK_CACHED_BYTES / (int64_t)sizeof(float)) launch(al, aligned, std::true_type{});
        else launch(al, aligned, std::false_type{});
    };
    auto pick = [&](auto al) {
        if (m % 4 == 0) pick_stores(al, std::true_type{});
        else pick_stores(al, std::false_type{});
    };
    if (alpha) pick(std::true_type{});
    else pick(std::false_type{});
}

// The matrix-vector product.  A workgroup takes ROWS packed rows (8, or 4 or 2 where fewer leave compute units idle) and
// reads x and alpha once for all of them.  A lane takes 8 neighbouring columns a step: two 16-byte loads each of x and
// alpha, and per row the 8 B code bits out of one or two words, with neighbouring lanes on neighbouring memory, the next
// step's loads in flight while this one is worked off.  (Lanes with 32 columns each, whole words of every row, put the 64
// lanes of a load of x on 64 lines of memory, and the address unit was what the kernel waited for.)  Per weight: a shift and
// a mask (the code, scaled to a byte offset), one LDS read of the codebook entry, the product's instructions.
//   T = double:  y_i = sum_j fl64(fl32(alpha_j c_ij)) x_j
//   T = float:   y_i = sum_j c_ij (alpha_j x_j), fused multiply-adds in float32
// 4096 x 11008: float32 17.8 -> 13 us, float64 17 us.
constexpr int MV_THREADS = 256;

template <typename T>
struct MvColumns {       // 8 columns of x and alpha
    T x[8];              // float: alpha_j x_j
    float a[8];          // double: alpha_j
};

// (columns past the row: code 0 times 0)
template <typename T, bool ALIGNED>
__device__ __forceinline__ void mv_columns(MvColumns<T> &c, const float *__restrict__ x, const float *__restrict__ alpha,
                                           uint32_t j0, uint32_t m) {
    float xv[8], av[8];
    if (ALIGNED && j0 + 8 <= m) {
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const float4 v = *(const float4 *)(x + j0 + 4 * q);
            xv[4 * q] = v.x; xv[4 * q + 1] = v.y; xv[4 * q + 2] = v.z; xv[4 * q + 3] = v.w;
            const float4 w = alpha ? *(const float4 *)(alpha + j0 + 4 * q) : make_float4(1.0f, 1.0f, 1.0f, 1.0f);
            av[4 * q] = w.x; av[4 * q + 1] = w.y; av[4 * q + 2] = w.z; av[4 * q + 3] = w.w;
        }
    } else {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const bool in = j0 + e < m;
            xv[e] = in ? x[j0 + e] : 0.0f;
            av[e] = (in && alpha) ? alpha[j0 + e] : 1.0f;
        }
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        if constexpr (sizeof(T) == 4) {
            c.x[e] = av[e] * xv[e];
        } else {
            c.x[e] = (T)xv[e];
            c.a[e] = av[e];
        }
    }
}

// the 8 codes of octet o of a B-bit row of wpr words, in the low 8 B bits
template <int B>
__device__ __forceinline__ uint32_t mv_codes(const uint32_t *__restrict__ rw, uint32_t o, uint32_t wpr) {
    const uint32_t bit = o * (8u * B), wi = bit >> 5, sh = bit & 31u;
    const uint32_t w0 = rw[wi];
    if (32 % (8 * B) == 0) return w0 >> sh;
    const uint32_t w1 = rw[min(wi + 1u, wpr - 1u)];        // (3 bits: the octet may reach into the next word, if there is one)
    return (uint32_t)((((unsigned long long)w1 << 32) | w0) >> sh);
}

// (Four octets go into one sum, and that into the lane's; float: an octet's products in two chains of four ahead of that.  One
// chain through all of a lane's columns rounds at the size of the whole sum each time: in float32 1.4 times the error
// at 11008 columns, 1.8 at 22016.)
template <int B, typename T>
__device__ __forceinline__ T mv_dot(uint32_t v, const float *cb, const MvColumns<T> &c, T acc) {
    constexpr uint32_t mask4 = ((1u << B) - 1u) << 2;       // the code times 4: byte offset of a float
    T half[2];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const int sh = e * B;
        const uint32_t off = (sh >= 2 ? v >> (sh - 2) : v << (2 - sh)) & mask4;
        const float w = *(const float *)((const char *)cb + off);
        if constexpr (sizeof(T) == 4) half[e & 1] = e < 2 ? w * c.x[e] : fmaf(w, c.x[e], half[e & 1]);
        else acc = fma((T)__fmul_rn(c.a[e], w), c.x[e], acc);
    }
    if constexpr (sizeof(T) == 4) acc += half[0] + half[1];
    return acc;
}

// All rows of the workgroup have B bits (rows are packed by bit width, so this is every workgroup but the few that lie
// across two groups).
template <int B, typename T, bool ALIGNED, int ROWS>
__device__ __forceinline__ void mv_same(const uint32_t *__restrict__ codes, const RowPlace *places, uint32_t m,
                                        const float *__restrict__ x, const float *__restrict__ alpha, const float (*cbf)[16],
                                        T (&acc)[ROWS]) {
    const uint32_t noct = (m + 7) >> 3, nth = blockDim.x, wpr = (uint32_t)(((long long)m * B + 31) / 32);
    uint32_t o = threadIdx.x;
    if (o >= noct) return;
    const uint32_t *rw = codes + places[0].word0;           // (rows of one group lie one behind the other)
    MvColumns<T> c;
    uint32_t v[ROWS];
    mv_columns<T, ALIGNED>(c, x, alpha, o * 8, m);
#pragma unroll
    for (int r = 0; r < ROWS; ++r) v[r] = mv_codes<B>(rw + (size_t)r * wpr, o, wpr);
    T part[ROWS];                // the sums of up to four octets
#pragma unroll
    for (int r = 0; r < ROWS; ++r) part[r] = (T)0;
    for (uint32_t step = 1;; ++step) {
        const uint32_t on = o + nth;
        const bool more = on < noct;
        MvColumns<T> cn;
        uint32_t vn[ROWS];
        if (more) {
            mv_columns<T, ALIGNED>(cn, x, alpha, on * 8, m);
#pragma unroll
            for (int r = 0; r < ROWS; ++r) vn[r] = mv_codes<B>(rw + (size_t)r * wpr, on, wpr);
        }
#pragma unroll
        for (int r = 0; r < ROWS; ++r) part[r] = mv_dot<B, T>(v[r], cbf[r], c, part[r]);
        if ((step & 3) == 0) {
#pragma unroll
            for (int r = 0; r < ROWS; ++r) {
                acc[r] += part[r];
                part[r] = (T)0;
            }
        }
        if (!more) break;
        c = cn;
#pragma unroll
        for (int r = 0; r < ROWS; ++r) v[r] = vn[r];
        o = on;
    }
#pragma unroll
    for (int r = 0; r < ROWS; ++r) acc[r] += part[r];
}

template <typename T, bool ALIGNED, int ROWS>
__global__ void __launch_bounds__(MV_THREADS) matvec_kernel(const uint32_t *codes, const long long *gwo, const int *row_perm,
                                                           const uint16_t *codebooks, const float *alpha, long long n,
                                                           long long m, const float *x, T *y) {
    __shared__ float cbf[ROWS][16];
    __shared__ T red[ROWS][MV_THREADS / 64];
    __shared__ RowPlace places[ROWS];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, nth = blockDim.x;
    const long long p0 = (long long)blockIdx.x * ROWS;
    // where the rows live and their codebooks as floats: every thread works its entry's row out for itself
    for (int t = tid; t < ROWS * 16; t += nth) {
        const int r = t >> 4, k = t & 15;
        RowPlace pl{0, 0, 0};
        if (p0 + r < n) pl = place_row(gwo, m, p0 + r);
        if (k == 0) places[r] = pl;
        cbf[r][k] = (pl.b > 0 && k < (1 << pl.b)) ? __half2float(__ushort_as_half(codebooks[pl.cb0 + k])) : 0.0f;
    }
    __syncthreads();
    T acc[ROWS];
#pragma unroll
    for (int r = 0; r < ROWS; ++r) acc[r] = (T)0;
    // the bit width all rows of this workgroup share, 0 when they differ (or some are past the end)
    int same_b = places[0].b;
#pragma unroll
    for (int r = 1; r < ROWS; ++r) same_b = (places[r].b == same_b) ? same_b : 0;
    same_b = __builtin_amdgcn_readfirstlane(same_b);
    const uint32_t mm = (uint32_t)m;
    switch (same_b) {
        case 1: mv_same<1, T, ALIGNED, ROWS>(codes, places, mm, x, alpha, cbf, acc); break;
        case 2: mv_same<2, T, ALIGNED, ROWS>(codes, places, mm, x, alpha, cbf, acc); break;
        case 3: mv_same<3, T, ALIGNED, ROWS>(codes, places, mm, x, alpha, cbf, acc); break;
        case 4: mv_same<4, T, ALIGNED, ROWS>(codes, places, mm, x, alpha, cbf, acc); break;
        default:
            for (uint32_t o = tid; o < (mm + 7) >> 3; o += nth) {
                MvColumns<T> c;
                mv_columns<T, ALIGNED>(c, x, alpha, o * 8, mm);
#pragma unroll
                for (int r = 0; r < ROWS; ++r) {
                    const uint32_t *rw = codes + places[r].word0;
                    switch (places[r].b) {
                        case 1: acc[r] = mv_dot<1, T>(mv_codes<1>(rw, o, 0u), cbf[r], c, acc[r]); break;
                        case 2: acc[r] = mv_dot<2, T>(mv_codes<2>(rw, o, 0u), cbf[r], c, acc[r]); break;
                        case 3: acc[r] = mv_dot<3, T>(mv_codes<3>(rw, o, (uint32_t)((m * 3 + 31) / 32)), cbf[r], c, acc[r]); break;
                        case 4: acc[r] = mv_dot<4, T>(mv_codes<4>(rw, o, 0u), cbf[r], c, acc[r]); break;
                        default: break;
                    }
                }
            }
    }
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
        T a = acc[r];
        for (int d = 32; d >= 1; d >>= 1) a += __shfl_down(a, d, 64);
        if (lane == 0) red[r][wave] = a;
    }
    __syncthreads();
    if (tid < ROWS && places[tid].b > 0) {
        T sum = (T)0;
        for (int w = 0; w < nth / 64; ++w) sum += red[tid][w];
        y[row_perm[p0 + tid]] = sum;
    }
}

// One launch.  Threads: enough for the row's octets in equal steps.  Rows per workgroup: 8 as long as that gives every
// compute unit four workgroups.
template <typename T>
void launch_matvec(skim_ctx *ctx, const uint32_t *codes, const int64_t *gwo, const int32_t *row_perm, const uint16_t *codebooks,
                   const float *alpha, int64_t n, int64_t m, const float *x, T *y) {
    const int64_t noct = (m + 7) / 8, steps = (noct + MV_THREADS - 1) / MV_THREADS;
    const int threads = (int)(((noct + steps - 1) / steps + 63) / 64 * 64);
    int rows = 8;
    while (rows > 2 && n < 4ll * ctx->num_cu * rows) rows >>= 1;
    const bool aligned = (((uintptr_t)x | (uintptr_t)alpha) & 15) == 0;
    auto launch = [&](auto al, auto rws) {
        constexpr int R = decltype(rws)::value;
        hipLaunchKernelGGL((matvec_kernel<T, decltype(al)::value, R>), dim3((unsigned)((n + R - 1) / R)), dim3(threads), 0, ctx->stream,
                           codes, (const long long *)gwo, row_perm, codebooks, alpha, (long long)n, (long long)m, x, y);
    };
    auto pick = [&](auto al) {
        if (rows == 8) launch(al, std::integral_constant<int, 8>{});
        else if (rows == 4) launch(al, std::integral_constant<int, 4>{});
        else launch(al, std::integral_constant<int, 2>{});
    };
    if (aligned) pick(std::true_type{});
    else pick(std::false_type{});
}

skim_status check_packed(skim_ctx *ctx, const void *codes, const void *gwo, const void *perm, const void *cbs, int64_t n,
                         int64_t m, const char *who) {
    if (!codes || !gwo || !perm || !cbs) SKIM_FAIL(ctx, SKIM_ERR_ARG, "%s: NULL argument", who);
    if (n < 1 || n > 0x7fffffff || m < 1 || m >= (1ll << 29))
        SKIM_FAIL(ctx, SKIM_ERR_SHAPE, "%s: bad shape n=%lld m=%lld", who, (long long)n, (long long)m);
    return SKIM_OK;
}

}  // namespace

extern "C" skim_status skim_unpack(skim_ctx *ctx, const uint32_t *codes, const int64_t *group_word_offset,
                                   const int32_t *row_perm, const uint16_t *codebooks_fp16, const float *alpha,
                                   int64_t n, int64_t m, float *Wq) {
    skim_status st = skim_enter(ctx);
    if (st != SKIM_OK) return st;
    if ((st = check_packed(ctx, codes, group_word_offset, row_perm, codebooks_fp16, n, m, "skim_unpack")) != SKIM_OK) return st;
    if (!Wq) SKIM_FAIL(ctx, SKIM_ERR_ARG, "skim_unpack: Wq must not be NULL");
    launch_unpack(ctx, codes, group_word_offset, row_perm, codebooks_fp16, alpha, n, m, Wq);
    SKIM_HIP(ctx, hipGetLastError());
    return SKIM_OK;
}

extern "C" skim_status skim_dequant_matvec(skim_ctx *ctx, const uint32_t *codes, const int64_t *group_word_offset,
                                           const int32_t *row_perm, const uint16_t *codebooks_fp16, const float *alpha,
                                           int64_t n, int64_t m, const float *x, double *y) {
    skim_status st = skim_enter(ctx);
    if (st != SKIM_OK) return st;
    if ((st = check_packed(ctx, codes, group_word_offset, row_perm, codebooks_fp16, n, m, "skim_dequant_matvec")) != SKIM_OK)
        return st;
    if (!x || !y) SKIM_FAIL(ctx, SKIM_ERR_ARG, "skim_dequant_matvec: x and y must not be NULL");
    launch_matvec(ctx, codes, group_word_offset, row_perm, codebooks_fp16, alpha, n, m, x, y);
    SKIM_HIP(ctx, hipGetLastError());
    return SKIM_OK;
}

extern "C" skim_status skim_dequant_matvec_f32(skim_ctx *ctx, const uint32_t *codes, const int64_t *group_word_offset,
                                               const int32_t *row_perm, const uint16_t *codebooks_fp16,
                                               const float *alpha, int64_t n, int64_t m, const float *x, float *y) {
    skim_status st = skim_enter(ctx);
    if (st != SKIM_OK) return st;
    if ((st = check_packed(ctx, codes, group_word_offset, row_perm, codebooks_fp16, n, m, "skim_dequant_matvec_f32")) != SKIM_OK)
        return st;
    if (!x || !y) SKIM_FAIL(ctx, SKIM_ERR_ARG, "skim_dequant_matvec_f32: x and y must not be NULL");
    launch_matvec(ctx, codes, group_word_offset, row_perm, codebooks_fp16, alpha, n, m, x, y);
    SKIM_HIP(ctx, hipGetLastError());
    return SKIM_OK;
}
