// Greedy mixed-precision bit allocation (Alg. 1, unit costs) on the device, so that the
// path error table -> allocation -> pack needs no round trip to the host.
//
// Same order as the host function: upgrade j of a row is taken when the running minimum
// k_j = min(g_1 .. g_j) of the row's reductions comes up, and the greedy loop takes the
// upgrades in the order (k descending, row ascending, j ascending).  The first T = budget -
// n * bmin of them are found in one workgroup: by cuts of the keys' interval with the keys in registers
// (greedy_rows_kernel: the usual tables), or by a most-significant-digit radix selection (greedy_select_kernel:
// 8 digits of 8 bits), ties at the threshold value in index order.
#include "skim_common.h"

#include <math.h>

#include <type_traits>

namespace {

constexpr int GA_THREADS = 1024;
constexpr size_t GA_LDS_KEYS = 128 * 1024;      // keys kept in LDS up to this many bytes (16384 keys)
typedef unsigned long long u64;

// float64 -> uint64 whose unsigned order is the order of the doubles (-0 folded into +0).
__device__ __forceinline__ u64 ordered_key(double x) {
    if (x == 0.0) x = 0.0;
    const u64 u = (u64)__double_as_longlong(x);
    return (u >> 63) ? ~u : (u | 0x8000000000000000ull);
}

// hist[dig] += 1 for the lanes with `valid`.  The lanes that share the digit of the first valid lane are
// counted with one atomic (the high digits of the keys are nearly constant; one atomic per key would
// serialise on a single LDS address); the others add on their own.
__device__ __forceinline__ void hist_add(unsigned *hist, bool valid, unsigned dig) {
    const u64 act = __ballot(valid);
    if (act == 0) return;
    const int leader = __ffsll((long long)act) - 1;
    const unsigned first = (unsigned)__builtin_amdgcn_readlane((int)dig, leader);   // leader is the same in every lane
    const u64 same = __ballot(valid && dig == first);
    if ((int)(threadIdx.x & 63) == leader) atomicAdd(&hist[first], (unsigned)__popcll(same));
    else if (valid && dig != first) atomicAdd(&hist[dig], 1u);
}

__global__ void __launch_bounds__(GA_THREADS) greedy_select_kernel(const double *__restrict__ E, long long n, int bmin,
                                                                  int nb, long long T, u64 *keys_global,
                                                                  uint8_t *__restrict__ bits, long long *__restrict__ info,
                                                                  long long budget, int keys_in_lds) {
    // the keys are written, re-read for the ties, marked and read again for the bits: in LDS when they fit
    // (one workgroup: every trip to global memory is pure latency), else in the caller's workspace
    extern __shared__ __align__(16) unsigned char ga_smem[];
    u64 *keys = keys_in_lds ? (u64 *)ga_smem : keys_global;
    __shared__ unsigned hist[256];
    __shared__ u64 sh_prefix;
    __shared__ long long sh_rank;
    __shared__ int sh_single;
    __shared__ long long wsum[GA_THREADS / 64];
    __shared__ long long cnt[8];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int nu = nb - 1;
    const long long nk = n * nu;

    // keys: running minima of the reductions, row by row
    for (long long i = tid; i < n; i += GA_THREADS) {
        double k = 0.0;
        for (int j = 0; j < nu; ++j) {
            const double g = E[i * nb + j] - E[i * nb + j + 1];
            k = (j == 0 || g < k) ? g : k;
            keys[i * nu + j] = ordered_key(k);
        }
    }
    if (tid < 8) cnt[tid] = 0;
    __syncthreads();

    // up to 16 keys per thread stay in registers over the eight passes (tables of up to 4096 rows
    // at four upgrades per row); larger tables re-read the keys from global memory
    constexpr int KPT = 16;
    const bool in_regs = nk <= (long long)GA_THREADS * KPT;
    u64 rk[KPT];
    if (in_regs) {
#pragma unroll
        for (int k = 0; k < KPT; ++k) {
            const long long q = tid + (long long)k * GA_THREADS;
            rk[k] = (q < nk) ? keys[q] : 0ull;
        }
    }

    // threshold = the T-th largest key (T >= 1): fix its digits from the top
    u64 prefix = 0;
    long long rank = T;            // rank among the keys that share the prefix fixed so far
    u64 thr = 0;
    long long R = 0;               // keys equal to the threshold that are still taken
    bool lone = false;             // exactly one key equals the threshold and it is taken: taken <=> key >= thr
    if (T > 0 && T < nk) {
        for (int d = 7; d >= 0; --d) {
            if (tid < 256) hist[tid] = 0;
            __syncthreads();
            const u64 hi_mask = (d == 7) ? 0ull : (~0ull << (8 * (d + 1)));
            if (in_regs) {
#pragma unroll
                for (int k = 0; k < KPT; ++k) {
                    const long long q = tid + (long long)k * GA_THREADS;
                    hist_add(hist, q < nk && (rk[k] & hi_mask) == prefix, (unsigned)(rk[k] >> (8 * d)) & 255u);
                }
            } else {
                for (long long q = tid; q < nk; q += GA_THREADS) {
                    const u64 key = keys[q];
                    hist_add(hist, (key & hi_mask) == prefix, (unsigned)(key >> (8 * d)) & 255u);
                }
            }
            __syncthreads();
            if (wave == 0) {
                // the bin that holds the rank-th largest key: lane l owns bins 4l .. 4l+3; suffix sums over the lanes
                const unsigned h0 = hist[4 * lane], h1 = hist[4 * lane + 1], h2 = hist[4 * lane + 2], h3 = hist[4 * lane + 3];
                const long long mine = (long long)h0 + h1 + h2 + h3;
                long long inc = mine;                       // sum over lanes >= this one
                for (int dd = 1; dd < 64; dd <<= 1) {
                    const long long u = __shfl_down(inc, dd, 64);
                    if (lane + dd < 64) inc += u;
                }
                const long long above = inc - mine;         // keys in higher bins than this lane's
                if (above < rank && rank <= inc) {          // exactly one lane
                    long long r = rank - above;
                    int bin = 4 * lane + 3;
                    if ((long long)h3 < r) { r -= h3; bin = 4 * lane + 2;
                        if ((long long)h2 < r) { r -= h2; bin = 4 * lane + 1;
                            if ((long long)h1 < r) { r -= h1; bin = 4 * lane; } } }
                    sh_prefix = prefix | ((u64)bin << (8 * d));
                    sh_rank = r;
                    sh_single = (hist[bin] == 1u) ? 1 : 0;   // one key left under the new prefix: it is the threshold
                }
            }
            __syncthreads();
            prefix = sh_prefix;
            rank = sh_rank;
            const bool single = sh_single != 0;
            if (single && d > 0) {
                // the remaining digits are those of that key: its owner publishes it
                __syncthreads();   // every thread has read sh_prefix / sh_single before it is overwritten
                const u64 lo_mask = ~0ull << (8 * d);
                if (in_regs) {
#pragma unroll
                    for (int k = 0; k < KPT; ++k) {
                        const long long q = tid + (long long)k * GA_THREADS;
                        if (q < nk && (rk[k] & lo_mask) == prefix) sh_prefix = rk[k];
                    }
                } else {
                    for (long long q = tid; q < nk; q += GA_THREADS) {
                        const u64 key = keys[q];
                        if ((key & lo_mask) == prefix) sh_prefix = key;
                    }
                }
                __syncthreads();
                prefix = sh_prefix;
                lone = true;
                break;             // rank == 1 here
            }
        }
        thr = prefix;
        R = rank;                  // the first R keys equal to thr, in index order, are taken
    }

    // keys equal to the threshold: positions in index order (contiguous index ranges per thread)
    const long long per = (nk + GA_THREADS - 1) / GA_THREADS;
    const long long q0 = min(nk, per * tid), q1 = min(nk, q0 + per);
    long long eq_before = 0;
    if (T > 0 && T < nk && !lone) {
        long long mine = 0;
        for (long long q = q0; q < q1; ++q) mine += (keys[q] == thr) ? 1 : 0;
        long long inc = mine;
        for (int dd = 1; dd < 64; dd <<= 1) {
            const long long u = __shfl_up(inc, dd, 64);
            if (lane >= dd) inc += u;
        }
        if (lane == 63) wsum[wave] = inc;
        __syncthreads();
        long long before = 0;
        for (int w2 = 0; w2 < wave; ++w2) before += wsum[w2];
        eq_before = before + inc - mine;
    }
    __syncthreads();
    // taken: key > thr, or key == thr among the first R equal ones; T >= nk takes everything.
    // Mark by overwriting the key with 1 / 0 (each thread owns its index range).  With a lone key at the threshold
    // the comparison key >= thr says it all and the rows are counted from the keys themselves.
    for (long long q = q0; q < q1 && !lone; ++q) {
        const u64 key = keys[q];
        bool take;
        if (T <= 0) take = false;
        else if (T >= nk) take = true;
        else if (key > thr) take = true;
        else if (key == thr) take = (eq_before++ < R);
        else take = false;
        keys[q] = take ? 1ull : 0ull;
    }
    __syncthreads();
    // rows per bit width: counted per wavefront with ballots (one LDS atomic per wavefront and width instead of
    // one per row on a handful of addresses)
    long long wcnt[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    for (long long i0 = 0; i0 < n; i0 += GA_THREADS) {
        const long long i = i0 + tid;
        int b = -1;
        if (i < n) {
            b = bmin;
            for (int j = 0; j < nu; ++j) {
                const u64 key = keys[i * nu + j];
                b += lone ? (key >= thr ? 1 : 0) : (int)key;
            }
            bits[i] = (uint8_t)b;
        }
#pragma unroll
        for (int v = 0; v < 8; ++v) wcnt[v] += __popcll(__ballot(b == v));
    }
    if (lane == 0) {
#pragma unroll
        for (int v = 0; v < 8; ++v)
            if (wcnt[v]) atomicAdd((unsigned long long *)&cnt[v], (unsigned long long)wcnt[v]);
    }
    __syncthreads();
    if (tid < 8) info[tid] = cnt[tid];
    if (tid == 0) {
        long long spent = 0;
        for (int b = 0; b < 8; ++b) spent += cnt[b] * b;
        info[8] = spent;
        info[9] = budget;
    }
}

// Tables of at most three upgrades per row and GR_THREADS * 12 rows, which is every table of 1 .. 4 bits on a layer of up
// to 12288 rows: a thread keeps the keys of its rows in registers from the error table to the bit widths, so that no key
// is written or read again.  One workgroup, bound by the length of its chain of barriers: the threshold is found by cutting
// the interval between the least and the largest key into 1024 bins and going on inside the bin that holds the T-th
// largest, until at most 64 keys are left, which every wavefront ranks against each other (two or three cuts; a cut by
// the keys' own digits took up to eight, the first two with all keys in a handful of bins).  Every wavefront works the
// outcome of a cut out for itself.  Tables of 8192 rows 112 -> 22.6 us, 11008 rows 74 -> 32.5, 4096 24 -> 14.8, 512 10 -> 7.3
// (kernel times; larger tables and wider bit ranges take greedy_select_kernel: whole calls of 12288 / 12289 / 22016 rows
// 28 / 57 / 106 us).
constexpr int GR_NU = 3, GR_BINS = 1024, GR_LIST = 64;
constexpr int GR_MAX_RPT = 12;

// inclusive sum over the 64 lanes / over each row of 16 lanes
template <bool ROWS16>
__device__ __forceinline__ int scan_incl(int x) {
    x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xF, 0xF, false);   // row_shr:1
    x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xF, 0xF, false);   // row_shr:2
    x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xF, 0xF, false);   // row_shr:4
    x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xF, 0xF, false);   // row_shr:8
    if (!ROWS16) {
        x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xA, 0xF, false);   // row_bcast:15 into rows 1, 3
        x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xC, 0xF, false);   // row_bcast:31 into rows 2, 3
    }
    return x;
}
__device__ __forceinline__ u64 readlane_u64(u64 x, int l) {
    const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)x, l);
    const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(x >> 32), l);
    return ((u64)hi << 32) | lo;
}

// RPT: rows per thread (row tid + r * GA_THREADS in slot r).
template <int RPT>
__global__ void __launch_bounds__(GA_THREADS) greedy_rows_kernel(const double *__restrict__ E, int n, int bmin, int nb, int T,
                                                                uint8_t *__restrict__ bits, long long *__restrict__ info,
                                                                long long budget) {
    // three sets of bins in turn: the set of the next cut is cleared while this one is filled, and the set of the cut
    // before may still be read then
    __shared__ __align__(16) int hist[3][GR_BINS];
    __shared__ u64 list[GR_LIST];
    __shared__ u64 wmin[GA_THREADS / 64], wmax[GA_THREADS / 64];
    __shared__ int wsum[RPT][GA_THREADS / 64];
    __shared__ int listn, cnt[8];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int nu = nb - 1, nk = n * nu;

    u64 key[RPT][GR_NU];
    {
        double e[RPT][GR_NU + 1];
#pragma unroll
        for (int r = 0; r < RPT; ++r) {
            const int i = min(tid + r * GA_THREADS, n - 1);
#pragma unroll
            for (int j = 0; j <= GR_NU; ++j) e[r][j] = E[(long long)i * nb + min(j, nu)];
        }
#pragma unroll
        for (int r = 0; r < RPT; ++r) {
            double k = 0.0;
#pragma unroll
            for (int j = 0; j < GR_NU; ++j) {
                const double g = e[r][j] - e[r][j + 1];
                k = (j == 0 || g < k) ? g : k;
                key[r][j] = ordered_key(k);
            }
        }
    }
    auto valid = [&](int r, int j) -> bool { return j < nu && tid + r * GA_THREADS < n; };

    u64 thr = 0;
    int R = 0;                     // keys equal to the threshold that are still taken, in index order
    bool ties = false;             // fewer than there are
    if (T > 0 && T < nk) {
        u64 lo = ~0ull, hi = 0ull;
#pragma unroll
        for (int r = 0; r < RPT; ++r)
#pragma unroll
            for (int j = 0; j < GR_NU; ++j)
                if (valid(r, j)) {
                    lo = min(lo, key[r][j]);
                    hi = max(hi, key[r][j]);
                }
        for (int d = 32; d >= 1; d >>= 1) {
            lo = min(lo, (u64)__shfl_xor((long long)lo, d, 64));
            hi = max(hi, (u64)__shfl_xor((long long)hi, d, 64));
        }
        if (lane == 0) {
            wmin[wave] = lo;
            wmax[wave] = hi;
        }
        hist[0][tid] = 0;
        if (tid == 0) listn = 0;
        __syncthreads();
        for (int w = 0; w < GA_THREADS / 64; ++w) {
            lo = min(lo, wmin[w]);
            hi = max(hi, wmax[w]);
        }
        lo = readlane_u64(lo, 0);
        hi = readlane_u64(hi, 0);
        // the least shift that leaves fewer than GR_BINS bins
        int shift = max(0, 64 - 10 - (int)__builtin_clzll((hi - lo) | 1ull));
        int rank = T;              // among the keys of [lo, hi]
        static_assert(GR_BINS == 1024 && GA_THREADS == GR_BINS, "10 bits a cut, one bin cleared per thread");
        for (int pass = 0;; ++pass) {
            int *h = hist[pass % 3];
            hist[(pass + 1) % 3][tid] = 0;
            const u64 span = hi - lo;
#pragma unroll
            for (int r = 0; r < RPT; ++r)
#pragma unroll
                for (int j = 0; j < GR_NU; ++j) {
                    const u64 x = key[r][j] - lo;      // (keys below lo wrap around to large values)
                    if (valid(r, j) && x <= span) atomicAdd(&h[(int)(x >> shift)], 1);
                }
            __syncthreads();
            // the bin of the rank-th largest: 16 bins per lane, then the 16 bins of that lane
            const int4 *h4 = (const int4 *)(h + 16 * lane);
            int mine = 0;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int4 c = h4[q];
                mine += (c.x + c.y) + (c.z + c.w);
            }
            const int inc = scan_incl<false>(mine);
            const int above = __builtin_amdgcn_readlane(inc, 63) - inc;       // keys in the bins of higher lanes
            const int L = __ffsll((long long)__ballot(above < rank && rank <= above + mine)) - 1;      // exactly one lane
            const int aboveL = __builtin_amdgcn_readlane(above, L), mineL = __builtin_amdgcn_readlane(mine, L);
            const int c1 = lane < 16 ? h[16 * L + lane] : 0;
            const int above1 = aboveL + mineL - scan_incl<true>(c1);
            const int L1 = __ffsll((long long)__ballot(lane < 16 && above1 < rank && rank <= above1 + c1)) - 1;
            rank -= __builtin_amdgcn_readlane(above1, L1);
            const int left = __builtin_amdgcn_readlane(c1, L1);
            lo += (u64)(16 * L + L1) << shift;
            hi = lo + ((1ull << shift) - 1ull);
            if (shift == 0) {      // one value left
                thr = lo;
                R = rank;
                ties = left > rank;
                break;
            }
            if (left <= GR_LIST) {
                const u64 sp = hi - lo;
#pragma unroll
                for (int r = 0; r < RPT; ++r)
#pragma unroll
                    for (int j = 0; j < GR_NU; ++j)
                        if (valid(r, j) && key[r][j] - lo <= sp) list[min(atomicAdd(&listn, 1), GR_LIST - 1)] = key[r][j];
                __syncthreads();
                const u64 x = lane < left ? list[lane] : 0ull;
                int gt = 0, eq = 0;
                for (int q = 0; q < left; ++q) {
                    const u64 y = list[q];
                    gt += y > x ? 1 : 0;
                    eq += y == x ? 1 : 0;
                }
                const int l = __ffsll((long long)__ballot(lane < left && gt < rank && rank <= gt + eq)) - 1;
                thr = readlane_u64(x, l);
                R = rank - __builtin_amdgcn_readlane(gt, l);
                ties = __builtin_amdgcn_readlane(eq, l) > R;
                break;
            }
            shift = max(0, shift - 10);
        }
    }
    // equal keys ahead of this thread's, in index order (rows ascending: slot by slot, thread by thread)
    int before[RPT];
    if (tid < 8) cnt[tid] = 0;
    if (ties) {                    // (the same in every thread)
#pragma unroll
        for (int r = 0; r < RPT; ++r) {
            int c = 0;
#pragma unroll
            for (int j = 0; j < GR_NU; ++j) c += (valid(r, j) && key[r][j] == thr) ? 1 : 0;
            const int inc = scan_incl<false>(c);
            before[r] = inc - c;
            if (lane == 63) wsum[r][wave] = inc;
        }
    }
    __syncthreads();
    if (ties) {
        int total = 0;
#pragma unroll
        for (int r = 0; r < RPT; ++r) {
            for (int w = 0; w < GA_THREADS / 64; ++w) {
                if (w == wave) before[r] += total;
                total += wsum[r][w];
            }
        }
    }
    // the widths, counted per wavefront with ballots
    int wcnt[GR_NU + 1] = {0, 0, 0, 0};
#pragma unroll
    for (int r = 0; r < RPT; ++r) {
        int up = 0, eqs = ties ? before[r] : 0;
#pragma unroll
        for (int j = 0; j < GR_NU; ++j) {
            if (j >= nu) continue;
            bool take;
            if (T <= 0) take = false;
            else if (T >= nk) take = true;
            else if (!ties) take = key[r][j] >= thr;
            else take = key[r][j] > thr || (key[r][j] == thr && eqs++ < R);
            up += take ? 1 : 0;
        }
        const int i = tid + r * GA_THREADS;
        if (i < n) bits[i] = (uint8_t)(bmin + up);
#pragma unroll
        for (int v = 0; v <= GR_NU; ++v) wcnt[v] += __popcll(__ballot(i < n && up == v));
    }
    if (lane == 0) {
#pragma unroll
        for (int v = 0; v <= GR_NU; ++v)
            if (wcnt[v]) atomicAdd(&cnt[bmin + v], wcnt[v]);
    }
    __syncthreads();
    if (tid < 8) info[tid] = cnt[tid];
    if (tid == 0) {
        long long spent = 0;
        for (int b = 0; b < 8; ++b) spent += (long long)cnt[b] * b;
        info[8] = spent;
        info[9] = budget;
    }
}

}  // namespace

extern "C" skim_status skim_greedy_allocate_device(skim_ctx *ctx, const double *E, int64_t n, int bmin, int bmax,
                                                   double avg_bits, uint8_t *bits, int64_t *info) {
    skim_status st = skim_enter(ctx);
    if (st != SKIM_OK) return st;
    if (!E || !bits || !info) SKIM_FAIL(ctx, SKIM_ERR_ARG, "skim_greedy_allocate_device: NULL argument");
    if (n < 1 || n > (1ll << 24)) SKIM_FAIL(ctx, SKIM_ERR_SHAPE, "skim_greedy_allocate_device: n = %lld out of range", (long long)n);
    if (bmin < 1 || bmax < bmin || bmax > 7) SKIM_FAIL(ctx, SKIM_ERR_ARG, "bit range [%d,%d] outside 1..7", bmin, bmax);
    const int64_t B = (int64_t)floor(avg_bits * (double)n + 1e-9);
    if (B < (int64_t)bmin * n || B > (int64_t)bmax * n)
        SKIM_FAIL(ctx, SKIM_ERR_BUDGET, "budget %lld outside [%lld, %lld]", (long long)B, (long long)(bmin * n), (long long)(bmax * n));
    const int nb = bmax - bmin + 1;
    const int64_t T = B - (int64_t)bmin * n;      // upgrades to take
    const size_t need = (size_t)n * (nb > 1 ? nb - 1 : 1) * sizeof(u64);
    if (!ctx->ws || ctx->ws_bytes < need)
        SKIM_FAIL(ctx, SKIM_ERR_WORKSPACE, "workspace missing or smaller than skim_workspace_bytes(n, m)");
    if (nb - 1 <= GR_NU && n <= (int64_t)GR_MAX_RPT * GA_THREADS) {
        auto launch = [&](auto rpt) {
            hipLaunchKernelGGL(greedy_rows_kernel<decltype(rpt)::value>, dim3(1), dim3(GA_THREADS), 0, ctx->stream, E, (int)n, bmin,
                               nb, (int)T, bits, (long long *)info, (long long)B);
        };
        if (n <= GA_THREADS) launch(std::integral_constant<int, 1>{});
        else if (n <= 4 * GA_THREADS) launch(std::integral_constant<int, 4>{});
        else if (n <= 8 * GA_THREADS) launch(std::integral_constant<int, 8>{});
        else launch(std::integral_constant<int, GR_MAX_RPT>{});
        SKIM_HIP(ctx, hipGetLastError());
        return SKIM_OK;
    }
    const size_t key_bytes = (size_t)n * (nb > 1 ? nb - 1 : 1) * sizeof(u64);
    const int keys_in_lds = key_bytes <= GA_LDS_KEYS;
    if (keys_in_lds && !ctx->greedy_lds_enabled) {
        SKIM_HIP(ctx, hipFuncSetAttribute((const void *)greedy_select_kernel, hipFuncAttributeMaxDynamicSharedMemorySize,
                                          (int)GA_LDS_KEYS));
        ctx->greedy_lds_enabled = 1;
    }
    hipLaunchKernelGGL(greedy_select_kernel, dim3(1), dim3(GA_THREADS), keys_in_lds ? key_bytes : 0, ctx->stream, E,
                       (long long)n, bmin, nb, (long long)T, (u64 *)ctx->ws, bits, (long long *)info,
                       (long long)B, keys_in_lds);
    SKIM_HIP(ctx, hipGetLastError());
    return SKIM_OK;
}
