// Layer-wise Hessian proxy from calibration activations (Sec. 3.4: H ~ X X^T in the paper's
// column convention; here X is N x m row-major, one activation vector per row, so
// H = X^T X / N, m x m).  bf16 inputs, bf16 MFMA (v_mfma_f32_32x32x16_bf16) with float32
// accumulation over chunks of at most 8192 activations.  Only the 256 x 256 tiles on and above the
// diagonal are computed; where there are fewer of them than compute units the activations of a tile are
// split over several workgroups, whose partial tiles a second kernel adds up (float64) and mirrors.
#include "skim_tiles.h"

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef short short4v __attribute__((ext_vector_type(4)));
typedef short short8v __attribute__((ext_vector_type(8)));
typedef __attribute__((address_space(3))) short4v lds_short4v;

constexpr int XT = TILE;                   // output tile (rows and columns of H = columns of X)
constexpr int XK = 32;                     // activations per stage
constexpr int X_BUFS = 4;                  // stages in LDS: one in use, three on their way
constexpr int X_WAVES = 8, X_WC = X_WAVES / 2, X_BY = 8 / X_WC;   // wavefronts: 2 x X_WC, each 4 x X_BY blocks of 32 x 32
constexpr int X_THREADS = 64 * X_WAVES;
constexpr int X_LOADS = (XK * XT * 4) / (1024 * X_WAVES);   // 1 KB loads of a wavefront per stage
constexpr int X_PANEL_BYTES = XK * XT * 2; // one operand panel of a stage, activation-major: 16 KB
constexpr int X_STAGE_BYTES = 2 * X_PANEL_BYTES;
constexpr size_t X_LDS_BYTES = (size_t)X_BUFS * X_STAGE_BYTES;
constexpr int X_CHUNK = 8192 / XK;         // stages summed in float32 registers before they are added to memory
constexpr int X_MIN_STAGES = 8;            // no workgroup gets a shorter share of the activations than this
constexpr int X_PHASE_COST = 24;           // a phase and its partial tiles, in stages of 0.8 us (256 KB per workgroup)

// Tile number -> (bi, bj), bi <= bj: bands of 8 tile rows; inside a band column by column, first the columns the
// diagonal cuts short.  Consecutive tiles share operand panels (32 of them cover about 8 x 4 tiles: 12 panels).
__device__ __forceinline__ void tile_of(int v, int nt, int &bi, int &bj) {
    bi = bj = 0;
    for (int rb = 0; rb < nt; rb += 8) {
        const int hb = min(8, nt - rb);
        const int tri = hb * (hb + 1) / 2, cnt = tri + hb * (nt - rb - hb);
        if (v < cnt) {
            if (v < tri) {          // column rb + t holds the t + 1 rows rb .. rb + t
                int t = 0;
                while (v >= t + 1) {
                    v -= t + 1;
                    ++t;
                }
                bj = rb + t;
                bi = rb + v;
            } else {
                v -= tri;
                bj = rb + hb + v / hb;
                bi = rb + v % hb;
            }
            break;
        }
        v -= cnt;
    }
}

__device__ __forceinline__ bf16x8 operand(uint32_t addr, int off) {
    const short4v lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4v *)(addr + off));
    const short4v hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4v *)(addr + off + 4 * 2 * XT));
    const short8v v = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    return __builtin_bit_cast(bf16x8, v);
}

// 8 wavefronts, two per SIMD, of 128 x 64 each (12 operand reads for 8 MFMAs; 4 wavefronts of 128 x 128 would read a
// third less, but their 256 accumulators and two operand sets spill: 4.3 ms).  Four stages of 32 activations in LDS (128
// KB): the loads of stage s + 4 go out as soon as everybody has read stage s, i.e. three and a half stages ahead; the
// operands of the next half stage are read between the MFMAs of this one, so the barrier in the middle costs little.
// Bound: the power the matrix cores draw.  131072 x 4096 (1.18 PFLOP/s executed): MFMAs busy 76 % of the cycles, at 1.4 GHz
// instead of 2.4; no bank conflicts; 4.3 GB read past L2 of 1.07 GB.  1.90 ms; with one workgroup per tile on 136 of the
// 256 CUs, X staged through registers and transposed there: 3.60.  16384 x 2048: 85 us, of which the partial tiles (66 MB
// written, read again by xtx_finish_kernel) take about 30; the 128 x 128 full-product kernel this replaces: 485.
// DIRECT: the partial sums are added up in H itself (every tile is one workgroup's), not in slots.
template <bool DIRECT>
__global__ void __launch_bounds__(X_THREADS) __attribute__((amdgpu_waves_per_eu(X_WAVES / 4, X_WAVES / 4)))
xtx_big_kernel(const uint16_t *__restrict__ X, long long N, long long m, float *H, int nt, TilePlan plan, float4 *slots) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wr = wave / X_WC, wc = wave % X_WC;
    const int l32 = lane & 31, lhi = lane >> 5;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_byte *)smem;
    const int swave = __builtin_amdgcn_readfirstlane(wave);

    // Staging: wavefronts 0-3 move the i panel, 4-7 the j panel, 8 activations each, two per load (512 contiguous
    // bytes of either), straight from memory into LDS.  LDS row of an activation: its 256 values in 16-byte units,
    // unit u of the panel at place u ^ 4 (activation % 4): the transposing reads below take four activations
    // at once, which would share their banks otherwise.
    const int srow = 2 * X_LOADS * (wave % X_WC) + lhi;
    uint32_t voff_row[X_LOADS];
    int unit[X_LOADS];
#pragma unroll
    for (int i = 0; i < X_LOADS; ++i) {
        unit[i] = l32 ^ (((2 * i + lhi) & 3) << 2);
        voff_row[i] = (uint32_t)((long long)(srow + 2 * i) * m * 2);
    }
    const uint32_t stage_dst = lds0 + (uint32_t)((swave / X_WC) * X_PANEL_BYTES + (swave % X_WC) * 2 * X_LOADS * 2 * XT);

    // Operand reads (ds_read_b64_tr_b16): 16 lanes read 4 activations x 16 columns, 8 bytes each, and get 4
    // activations of one column each.  A lane's operand is column lane % 32 of a 32-column block, 8 activations.
    const int g = lane >> 4, i16 = lane & 15;
    const int rrow = 8 * (g >> 1) + (i16 >> 2);
    auto read_addr = [&](int block) -> uint32_t {
        const int u = (4 * (block ^ (i16 >> 2))) + 2 * (g & 1) + ((i16 & 3) >> 1);
        return (uint32_t)(rrow * 2 * XT + u * 16 + (i16 & 1) * 8);
    };
    uint32_t ra[4], rb[X_BY];
#pragma unroll
    for (int x = 0; x < 4; ++x) ra[x] = lds0 + read_addr(4 * wr + x);
#pragma unroll
    for (int y = 0; y < X_BY; ++y) rb[y] = lds0 + X_PANEL_BYTES + read_addr(X_BY * wc + y);

    const double inv = 1.0 / (double)N;
    const int nstage = (int)((N + XK - 1) / XK);
    const int G = gridDim.x;
    const int me = xcd_order(blockIdx.x, G);
    for (int p = 0; p < plan.nph; ++p) {
        const int ntile = plan.ntile[p], split = plan.split[p];
        for (int v = me; v < ntile * split; v += G) {
            const int part = v / ntile, t = v - part * ntile;
            int bi, bj;
            tile_of(plan.tile0[p] + t, nt, bi, bj);
            const int s0 = (int)((long long)nstage * part / split), s1 = (int)((long long)nstage * (part + 1) / split);
            const long long i0 = (long long)bi * XT, j0 = (long long)bj * XT;
            const long long sc0 = swave >= X_WC ? j0 : i0;
            uint32_t voff[X_LOADS];
#pragma unroll
            for (int i = 0; i < X_LOADS; ++i) {
                // a column group past the matrix reads zeros (out of the buffer's range); one that the matrix ends in
                // reads on into the next row: those columns only reach entries that are never stored
                const long long c = sc0 + 8 * unit[i];
                voff[i] = c < m ? voff_row[i] + (uint32_t)(c * 2) : 0x80000000u;
            }
            // the stage that is requested next: its first activation, and the bytes from there to the end of the part (a stage
            // past it is requested like any other, to keep the count of loads in flight, but reads nothing: zeros arrive)
            const uint64_t stage_bytes = (uint64_t)XK * (uint64_t)m * 2;
            LdsSource src{(uint64_t)(uintptr_t)X + (uint64_t)s0 * stage_bytes,
                          min(N, (long long)s1 * XK) * m * 2 - (long long)((uint64_t)s0 * stage_bytes)};
            auto issue = [&](int st) {
                const int4v rs = src.rsrc();
                const uint32_t dst = stage_dst + (uint32_t)(st & (X_BUFS - 1)) * X_STAGE_BYTES;
#pragma unroll
                for (int i = 0; i < X_LOADS; ++i) copy_to_lds(dst + i * 2 * 2 * XT, voff[i], rs);
                src.advance(stage_bytes);
            };
            floatx16 acc[4][X_BY];
#pragma unroll
            for (int x = 0; x < 4; ++x)
#pragma unroll
                for (int y = 0; y < X_BY; ++y)
#pragma unroll
                    for (int e = 0; e < 16; ++e) acc[x][y][e] = 0.f;
            // (the piece before is done with the LDS)
            asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
#pragma unroll
            for (int i = 0; i < X_BUFS; ++i) issue(s0 + i);
            asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(3 * X_LOADS) : "memory");
            bf16x8 a0[4], b0[X_BY], a1[4], b1[X_BY];
            auto read_ops = [&](int st, int ks, bf16x8 (&a)[4], bf16x8 (&b)[X_BY]) {
                const uint32_t sb = (uint32_t)(st & (X_BUFS - 1)) * X_STAGE_BYTES;
#pragma unroll
                for (int y = 0; y < X_BY; ++y) b[y] = operand(rb[y] + sb, ks * 16 * 2 * XT);
#pragma unroll
                for (int x = 0; x < 4; ++x) a[x] = operand(ra[x] + sb, ks * 16 * 2 * XT);
            };
            auto multiply = [&](const bf16x8 (&a)[4], const bf16x8 (&b)[X_BY]) {
#pragma unroll
                for (int x = 0; x < 4; ++x)
#pragma unroll
                    for (int y = 0; y < X_BY; ++y)
                        acc[x][y] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[x], b[y], acc[x][y], 0, 0, 0);
            };
            read_ops(s0, 0, a0, b0);
            bool first = true;
            for (int c0 = s0; c0 < s1; c0 += X_CHUNK) {
                const int c1 = min(c0 + X_CHUNK, s1);
                for (int st = c0; st < c1; ++st) {
                    read_ops(st, 1, a1, b1);
                    multiply(a0, b0);
                    #pragma unroll
                    for (int q = 0; q < 4 + X_BY; ++q) {
                        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                        __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
                    }
                    __builtin_amdgcn_sched_group_barrier(0x008, 4 * X_BY - 4 - X_BY, 0);
                    // the loads of the next stage have landed (those of the two after it may be in flight), and everybody has
                    // read all of this stage, whose place the new loads take
                    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(2 * X_LOADS) : "memory");
                    issue(st + X_BUFS);
                    read_ops(st + 1, 0, a0, b0);
                    multiply(a1, b1);
                    #pragma unroll
                    for (int q = 0; q < 4 + X_BY; ++q) {
                        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                        __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
                    }
                    __builtin_amdgcn_sched_group_barrier(0x008, 4 * X_BY - 4 - X_BY, 0);
                }
                // the chunk's sums go to memory.  Accumulator element e of a 32 x 32 tile: row = 8*(e/4) + 4*(lane/32)
                // + e%4, column = lane%32.
                if constexpr (!DIRECT) {
                    // partial tile: wavefront by wavefront, its accumulators' quarters as 16 bytes per lane
                    constexpr int XY = 4 * X_BY;
                    // (not through buffer stores with a scalar offset: their first data register may not be overwritten by the
                    // very next instruction on this chip, and the compiler does not know)
                    floatx4 *sp = (floatx4 *)slots + ((size_t)(plan.slot0[p] + v) * X_WAVES + swave) * (XY * 4 * 64) + lane;
                    floatx4 o[2][4];      // what is there already, one accumulator block ahead
                    auto old = [&](int xy) {
                        if (first) return;
#pragma unroll
                        for (int q = 0; q < 4; ++q) o[xy & 1][q] = sp[(xy * 4 + q) * 64];
                    };
                    old(0);
#pragma unroll
                    for (int xy = 0; xy < XY; ++xy) {
                        if (xy + 1 < XY) old(xy + 1);
                        const floatx16 &c = acc[xy / X_BY][xy % X_BY];
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            floatx4 t;
#pragma unroll
                            for (int e = 0; e < 4; ++e) t[e] = c[4 * q + e] + (first ? 0.f : o[xy & 1][q][e]);
                            sp[(xy * 4 + q) * 64] = t;
                        }
                    }
                } else {
                    const double scale = c1 == s1 ? inv : 1.0;
                    const long long ib = i0 + wr * 128 + 4 * lhi, jb = j0 + wc * 32 * X_BY + l32;
                    float *hp = H + ib * m + jb;
                    long long mm = m;
                    int rlim = (int)min(m - ib, 4096ll), clim = (int)min(m - jb, 4096ll);
                    asm volatile("" : "+v"(hp), "+s"(mm), "+v"(rlim), "+v"(clim));     // the addresses are worked out here, not ahead of the loop
                    if (rlim > 0 && clim > 0) {
#pragma unroll
                        for (int x = 0; x < 4; ++x)
#pragma unroll
                            for (int y = 0; y < X_BY; ++y) {
                                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                                for (int e = 0; e < 16; ++e) {
                                    const int r = x * 32 + 8 * (e >> 2) + (e & 3), c = y * 32;
                                    const bool valid = r < rlim && c < clim;
                                    float *q = valid ? hp + r * mm + c : hp;     // (no branch per entry: add nothing to the first one)
                                    const float old = *q;
                                    const float t = (first ? 0.f : old) + acc[x][y][e];
                                    *q = valid ? (float)((double)t * scale) : old;
                                }
                            }
                    }
                }
                first = false;
#pragma unroll
                for (int x = 0; x < 4; ++x)
#pragma unroll
                    for (int y = 0; y < X_BY; ++y)
#pragma unroll
                        for (int e = 0; e < 16; ++e) acc[x][y][e] = 0.f;
            }
        }
    }
    // no load may still be on its way into the LDS when the workgroup gives it back
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
}

// The partial tiles of a split tile added up, and every tile off the diagonal mirrored.  One wavefront per 32 x 32 block.
__global__ void __launch_bounds__(256) xtx_finish_kernel(float *H, long long N, long long m, int nt, TilePlan plan,
                                                         const float4 *__restrict__ slots) {
    __shared__ float tr[4][32][33];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int l32 = lane & 31, lhi = lane >> 5;
    const int tile = blockIdx.x >> 4, blk = (blockIdx.x & 15) * 4 + wave;       // 64 blocks of a tile
    int p = 0;
    while (p + 1 < plan.nph && tile >= plan.tile0[p + 1]) ++p;
    int bi, bj;
    tile_of(tile, nt, bi, bj);
    const int split = slots ? plan.split[p] : 0;           // 0: the sums are in H already
    constexpr int XY = 4 * X_BY;
    const int ow = blk / XY, xy = blk % XY;                 // the wavefront of xtx_big_kernel that owned the block, and which of its blocks
    const long long ib = (long long)bi * XT + (ow / X_WC) * 128 + (xy / X_BY) * 32, jb = (long long)bj * XT + (ow % X_WC) * 32 * X_BY + (xy % X_BY) * 32;
    if (ib < m && jb < m) {
        const int rlim = (int)min(m - ib, 32ll), clim = (int)min(m - jb, 32ll);
        float v[16];
        if (split > 0) {
            const double inv = 1.0 / (double)N;
            const float4 *sp = slots + ((size_t)(plan.slot0[p] + tile - plan.tile0[p]) * X_WAVES + ow) * (XY * 4 * 64) + xy * 256 + lane;
            const size_t step = (size_t)plan.ntile[p] * (8 * 8 * 4 * 64);       // from one part's slot to the next
            double s[16];
#pragma unroll
            for (int e = 0; e < 16; ++e) s[e] = 0.0;
            for (int q = 0; q < split; ++q, sp += step) {
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const float4 o = sp[k * 64];
                    s[4 * k] += o.x;
                    s[4 * k + 1] += o.y;
                    s[4 * k + 2] += o.z;
                    s[4 * k + 3] += o.w;
                }
            }
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const int r = 8 * (e >> 2) + 4 * lhi + (e & 3);
                v[e] = (float)(s[e] * inv);
                if (r < rlim && l32 < clim) H[(ib + r) * m + jb + l32] = v[e];
            }
        } else if (bi != bj) {
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const int r = 8 * (e >> 2) + 4 * lhi + (e & 3);
                v[e] = (r < rlim && l32 < clim) ? H[(ib + r) * m + jb + l32] : 0.f;
            }
        }
        if (bi != bj) {
#pragma unroll
            for (int e = 0; e < 16; ++e) tr[wave][l32][8 * (e >> 2) + 4 * lhi + (e & 3)] = v[e];
            // (one wavefront's LDS accesses execute in order: no barrier)
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const int c = 2 * e + lhi;
                if (c < clim && l32 < rlim) H[(jb + c) * m + ib + l32] = tr[wave][c][l32];
            }
        }
    }
}

}  // namespace

extern "C" size_t skim_hessian_workspace_bytes(const skim_ctx *ctx, int64_t N, int64_t m) {
    if (!ctx || N < 1 || m < 1 || m > 0x7fffffff) return 0;
    TilePlan plan;
    const int64_t nt = (m + XT - 1) / XT;
    return (size_t)skim_make_plan(plan, ctx->num_cu, nt * (nt + 1) / 2, (int)((N + XK - 1) / XK), X_MIN_STAGES, X_PHASE_COST, false) *
           TILE_SLOT_BYTES;
}

extern "C" skim_status skim_hessian_from_activations(skim_ctx *ctx, const uint16_t *X_bf16, int64_t N, int64_t m,
                                                     float *H) {
    return skim_hessian_from_activations_scratch(ctx, X_bf16, N, m, H, ctx ? ctx->ws : nullptr, ctx ? ctx->ws_bytes : 0);
}

extern "C" skim_status skim_hessian_from_activations_scratch(skim_ctx *ctx, const uint16_t *X_bf16, int64_t N, int64_t m, float *H,
                                                             void *scratch, size_t scratch_bytes) {
    skim_status st = skim_enter(ctx);
    if (st != SKIM_OK) return st;
    if (!X_bf16 || !H) SKIM_FAIL(ctx, SKIM_ERR_ARG, "skim_hessian_from_activations: NULL argument");
    if (N < 1 || m < 2 || (m & 1) || m > 0x7fffffff || ((uintptr_t)X_bf16 & 3))
        SKIM_FAIL(ctx, SKIM_ERR_SHAPE, "skim_hessian_from_activations: need N >= 1, m even, X 4-byte aligned (N=%lld m=%lld)",
                  (long long)N, (long long)m);
    if (scratch && ((uintptr_t)scratch & 255)) SKIM_FAIL(ctx, SKIM_ERR_ARG, "skim_hessian_from_activations: scratch must be 256-byte aligned");
    if (!ctx->xtx_lds_enabled) {
        SKIM_HIP(ctx, hipFuncSetAttribute((const void *)xtx_big_kernel<false>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)X_LDS_BYTES));
        SKIM_HIP(ctx, hipFuncSetAttribute((const void *)xtx_big_kernel<true>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)X_LDS_BYTES));
        ctx->xtx_lds_enabled = 1;
    }
    const int nt = (int)((m + XT - 1) / XT);
    const int G = ctx->num_cu;
    // Without scratch that holds the partial tiles the splits are given up, then the slots altogether
    TilePlan plan;
    const long long tiles = (long long)nt * (nt + 1) / 2;
    const int nstage = (int)((N + XK - 1) / XK);
    bool direct = true;
    for (int whole = 0; whole < 2 && direct; ++whole)
        direct = !scratch || (size_t)skim_make_plan(plan, G, tiles, nstage, X_MIN_STAGES, X_PHASE_COST, whole != 0) * TILE_SLOT_BYTES >
                                 scratch_bytes;
    if (direct) (void)skim_make_plan(plan, G, tiles, nstage, X_MIN_STAGES, X_PHASE_COST, true);
    long long grid = 0;
    for (int p = 0; p < plan.nph; ++p) {
        const long long items = (long long)plan.ntile[p] * plan.split[p];
        if (items > grid) grid = items;
    }
    if (grid > G) grid = G;
    float4 *slots = direct ? nullptr : (float4 *)scratch;
    if (direct)
        hipLaunchKernelGGL(xtx_big_kernel<true>, dim3((unsigned)grid), dim3(X_THREADS), X_LDS_BYTES, ctx->stream, X_bf16, (long long)N,
                           (long long)m, H, nt, plan, slots);
    else
        hipLaunchKernelGGL(xtx_big_kernel<false>, dim3((unsigned)grid), dim3(X_THREADS), X_LDS_BYTES, ctx->stream, X_bf16, (long long)N,
                           (long long)m, H, nt, plan, slots);
    hipLaunchKernelGGL(xtx_finish_kernel, dim3((unsigned)(tiles * 16)), dim3(256), 0, ctx->stream, H, (long long)N, (long long)m, nt,
                       plan, (const float4 *)slots);
    SKIM_HIP(ctx, hipGetLastError());
    return SKIM_OK;
}
