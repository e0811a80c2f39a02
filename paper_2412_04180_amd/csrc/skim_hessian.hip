// Layer-wise Hessian proxy from calibration activations (Sec. 3.4: H ~ X X^T in the paper's
// column convention; here X is N x m row-major, one activation vector per row, so
// H = X^T X / N, m x m).  bf16 inputs, bf16 MFMA (v_mfma_f32_32x32x16_bf16) with float32
// accumulation over chunks of activations.  Only the 256 x 256 tiles on and above the diagonal are
// computed; where there are fewer of them than compute units the activations of a tile are
// split over several workgroups, whose partial tiles a second kernel adds up (float64) and mirrors.
// Layers of up to 2560 columns (and wider ones that the 16-byte loads of rows do not divide) have chunks of at most 2048
// activations, all added up in float64; the others chunks of 8192, those of one workgroup added up in float32.
// Without scratch for partial tiles the former take a kernel of 128 x 128 tiles with float64 sums in registers.
#include "skim_tiles.h"

#include <type_traits>

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
constexpr int X_PIECE = 2048 / XK;         // ... before their leading halves go to memory (float64 sums)
constexpr int X_WIDE_TILES = 11;           // rows of so many tiles or more may be summed in chunks of X_CHUNK
constexpr size_t X_PIECE_BYTES = TILE_SLOT_BYTES / 2;
constexpr size_t X_SCRATCH_MOST = 256ull << 20;
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
// Bound: the power the matrix cores draw.  131072 x 4096 (1.23 PFLOP/s executed): MFMAs busy 76 % of the cycles, at 1.4 GHz
// instead of 2.4; no bank conflicts; 4.3 GB read past L2 of 1.07 GB.  1.90 ms; with one workgroup per tile on 136 of the
// 256 CUs, X staged through registers and transposed there: 3.60.  16384 x 2048: 94 us, of which the partial tiles and pieces
// (99 MB written, read again by xtx_finish_kernel) take about 35; the 128 x 128 full-product kernel: 484.
// SUM_IN_H: the chunks are added up in H itself (every tile is one workgroup's); SUM_IN_SLOTS: in the partial tiles.
// SUM_PIECES: nothing is added up here.  At the end of a chunk that is not a workgroup's last, the leading 8 bits of the
// sums, a bfloat16 each, go to memory (128 KB) and only what is left of them stays in the accumulators, exactly: the
// roundings of the next chunk are those of sums that start from next to nothing, and xtx_finish_kernel adds all of it up in
// float64.  (Whole partial tiles per chunk would be twice the memory and as much more to write and read.)  rms error of all
// entries, in units of sqrt(H_jj H_ll), of float64 registers in the 128 x 128 kernel / chunks of 8192 in float32 / pieces:
// 16384 x 2048 3.1 / 3.5 / 2.5 e-9 (484 / 88 / 94 us), 131072 x 2048 1.8 / 2.9 / 1.8 e-9 (4149 / 524 / 598 us), 65536 x 2560
// 1.9 / 3.3 / 1.9 e-9; the diagonal's 1.04 / 1.19 / 0.86, 0.75 / 1.11 / 0.76, 0.81 / 1.30 / 0.79 e-7.
enum SumMode { SUM_IN_H, SUM_IN_SLOTS, SUM_PIECES };
// pieces of a workgroup's share of `stages` stages beyond its last chunk
__host__ __device__ __forceinline__ int pieces_of(int stages) { return (stages - 1) / X_PIECE; }
template <int MODE>
__global__ void __launch_bounds__(X_THREADS) __attribute__((amdgpu_waves_per_eu(X_WAVES / 4, X_WAVES / 4)))
xtx_big_kernel(const uint16_t *__restrict__ X, long long N, long long m, float *H, int nt, TilePlan plan, float4 *slots, uint4 *pieces,
               int nslot) {
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
            // (pieces: as many for every share of the phase, in chunks of equal length)
            const int npiece = MODE == SUM_PIECES ? pieces_of((nstage + split - 1) / split) : 0;
            for (int c0 = s0, c1, piece = 0; c0 < s1; c0 = c1, ++piece) {
                c1 = MODE == SUM_PIECES ? s0 + (int)((long long)(s1 - s0) * (piece + 1) / (npiece + 1)) : min(c0 + X_CHUNK, s1);
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
                if constexpr (MODE == SUM_PIECES) {
                    if (c1 < s1) {
                        uint4 *pp = pieces + (((size_t)piece * nslot + plan.slot0[p] + v) * X_WAVES + swave) * (4 * X_BY * 2 * 64) + lane;
#pragma unroll
                        for (int xy = 0; xy < 4 * X_BY; ++xy) {
                            floatx16 &c = acc[xy / X_BY][xy % X_BY];
                            uint32_t o[8];
#pragma unroll
                            for (int e = 0; e < 16; ++e) {
                                const uint32_t u = __float_as_uint(c[e]);
                                if (e & 1) o[e >> 1] |= u & 0xFFFF0000u;
                                else o[e >> 1] = u >> 16;
                                // (an infinite sum stays in both)
                                c[e] = fabsf(c[e]) <= __FLT_MAX__ ? c[e] - __uint_as_float(u & 0xFFFF0000u) : c[e];
                            }
                            pp[(2 * xy) * 64] = make_uint4(o[0], o[1], o[2], o[3]);
                            pp[(2 * xy + 1) * 64] = make_uint4(o[4], o[5], o[6], o[7]);
                        }
                        continue;
                    }
                }
                // the chunk's sums go to memory.  Accumulator element e of a 32 x 32 tile: row = 8*(e/4) + 4*(lane/32)
                // + e%4, column = lane%32.
                if constexpr (MODE != SUM_IN_H) {
                    // partial tile: wavefront by wavefront, its accumulators' quarters as 16 bytes per lane
                    constexpr int XY = 4 * X_BY;
                    // (not through buffer stores with a scalar offset: their first data register may not be overwritten by the
                    // very next instruction on this chip, and the compiler does not know)
                    floatx4 *sp = (floatx4 *)slots + ((size_t)(plan.slot0[p] + v) * X_WAVES + swave) * (XY * 4 * 64) + lane;
                    floatx4 o[2][4];      // what is there already, one accumulator block ahead
                    auto old = [&](int xy) {
                        if (MODE == SUM_PIECES || first) return;
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
                            for (int e = 0; e < 4; ++e) t[e] = c[4 * q + e] + (MODE == SUM_PIECES || first ? 0.f : o[xy & 1][q][e]);
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

// The partial tiles (and pieces) of a tile added up, and every tile off the diagonal mirrored.  One wavefront per 32 x 32 block.
// (PIECES: of a launch of that kind; the other one keeps more wavefronts resident without its code.)
// run (NULL: none): running sums of the tiles from tile0 on, where the activations are taken in several passes; first: it
// holds nothing yet; last: the sums go to H.
template <bool PIECES>
__global__ void __launch_bounds__(256) xtx_finish_kernel(float *H, double inv, int nstage, long long m, int nt, TilePlan plan,
                                                         const float4 *__restrict__ slots, const uint4 *__restrict__ pieces, int nslot,
                                                         int tile0, double2 *__restrict__ run, bool first, bool last) {
    __shared__ float tr[4][32][33];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int l32 = lane & 31, lhi = lane >> 5;
    const int tile = tile0 + (blockIdx.x >> 4), blk = (blockIdx.x & 15) * 4 + wave;       // 64 blocks of a tile
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
            const size_t slot = (size_t)(plan.slot0[p] + tile - plan.tile0[p]), step = (size_t)plan.ntile[p];       // from one part's to the next
            double s[16];
            double2 *rp = run + ((size_t)(tile - tile0) * 64 + blk) * (8 * 64) + lane;
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const double2 r = PIECES && run && !first ? rp[k * 64] : make_double2(0.0, 0.0);
                s[2 * k] = r.x;
                s[2 * k + 1] = r.y;
            }
            const int npiece = PIECES ? pieces_of((nstage + split - 1) / split) : 0;
            const uint4 *pp = pieces + (slot * X_WAVES + ow) * (XY * 2 * 64) + xy * 128 + lane;
            for (int c = 0; c < npiece; ++c, pp += (size_t)nslot * (X_PIECE_BYTES / 16)) {
#pragma unroll 4
                for (int q = 0; q < split; ++q) {
                    const uint4 *o = pp + q * step * (X_PIECE_BYTES / 16);
                    const uint4 lo = o[0], hi = o[64];
                    const uint32_t w[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
#pragma unroll
                    for (int e = 0; e < 16; ++e) s[e] += (double)__uint_as_float(e & 1 ? w[e >> 1] & 0xFFFF0000u : w[e >> 1] << 16);
                }
            }
            const float4 *sp = slots + (slot * X_WAVES + ow) * (XY * 4 * 64) + xy * 256 + lane;
#pragma unroll 2
            for (int q = 0; q < split; ++q) {
                const float4 *f = sp + q * step * (TILE_SLOT_BYTES / 16);
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const float4 o = f[k * 64];
                    s[4 * k] += o.x;
                    s[4 * k + 1] += o.y;
                    s[4 * k + 2] += o.z;
                    s[4 * k + 3] += o.w;
                }
            }
            if (PIECES && !last) {
#pragma unroll
                for (int k = 0; k < 8; ++k) rp[k * 64] = make_double2(s[2 * k], s[2 * k + 1]);
                return;
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

// How `tiles` tiles (at most one per compute unit) are summed in float64 with at most `cap` bytes of scratch: all activations
// in one pass, or in several with running sums, whatever needs no more.  False: not with so little.
struct PiecePlan {
    TilePlan plan;
    int passes, nslot, npiece;
    size_t bytes;
    size_t run_offset() const { return (size_t)nslot * (TILE_SLOT_BYTES + npiece * X_PIECE_BYTES); }
};
bool piece_plan(PiecePlan &pp, int G, int tiles, int nstage, size_t cap) {
    for (pp.passes = 1; pp.passes <= nstage; ++pp.passes) {
        const int stages = (nstage + pp.passes - 1) / pp.passes;
        pp.nslot = (int)skim_make_plan(pp.plan, G, tiles, stages, X_MIN_STAGES, X_PHASE_COST, false);
        pp.npiece = 0;
        for (int p = 0; p < pp.plan.nph; ++p) {
            const int n = pieces_of((stages + pp.plan.split[p] - 1) / pp.plan.split[p]);
            if (n > pp.npiece) pp.npiece = n;
        }
        pp.bytes = pp.run_offset() + (pp.passes > 1 ? (size_t)tiles * 2 * TILE_SLOT_BYTES : 0);
        if (pp.bytes <= cap) return true;
        if (pp.npiece == 0 && stages <= X_PIECE) break;
    }
    return false;
}
// tiles of one group: all, or an equal share of them that leaves no compute unit two
int group_tiles(long long tiles, int G) {
    const long long groups = (tiles + G - 1) / G;
    return (int)((tiles + groups - 1) / groups);
}
size_t piece_bytes(long long tiles, int nstage, int G) {
    PiecePlan pp;
    const int T = group_tiles(tiles, G), rest = (int)(tiles % T);
    size_t b = piece_plan(pp, G, T, nstage, X_SCRATCH_MOST) ? pp.bytes : 0;
    if (rest && piece_plan(pp, G, rest, nstage, X_SCRATCH_MOST) && pp.bytes > b) b = pp.bytes;
    return b;
}

// How the tiles of the other layers are summed with `slots` partial tiles: in groups of whole rounds of one tile per compute
// unit, the last of them with the rest, whose tiles are split.  Whole tiles have slots, too: entry by entry, 16384 x 11008
// took 1.98 ms instead of 1.74, 1024 x 4096 79 us instead of 49.
struct WidePlan {
    int G;
    long long tiles, at, per_group;      // tiles in all, of the groups so far, of whole rounds per group
    int rest, rest_slots, most;          // tiles beyond the whole rounds and their slots; slots of the largest group
    long long slots;
    TilePlan rest_plan;
    WidePlan(int G, long long tiles, int nstage, long long slots) : G(G), tiles(tiles), at(0), slots(slots) {
        rest = (int)(tiles % G);
        rest_slots = 0;
        for (int whole = 0; whole < 2 && rest && (whole == 0 || rest_slots > slots); ++whole)
            rest_slots = (int)skim_make_plan(rest_plan, G, rest, nstage, X_MIN_STAGES, X_PHASE_COST, whole != 0);
        per_group = slots / G * G;
        TilePlan p;
        most = 0;
        for (int tile0, n, ns; fits() && next(p, tile0, n, ns);) most = most > ns ? most : ns;
        at = 0;
    }
    bool fits() const { return rest_slots <= slots && (tiles < G || per_group > 0); }
    bool next(TilePlan &plan, int &tile0, int &ntile, int &nslot) {
        if (at >= tiles) return false;
        plan = TilePlan{};
        tile0 = (int)at;
        nslot = 0;
        const long long whole = tiles - rest - at < per_group ? tiles - rest - at : per_group;
        if (whole > 0) {
            plan.tile0[0] = (int)at;
            plan.ntile[0] = (int)whole;
            plan.split[0] = 1;
            plan.nph = 1;
            nslot = (int)whole;
            at += whole;
        }
        if (rest && at == tiles - rest && nslot + rest_slots <= slots) {
            for (int p = 0; p < rest_plan.nph; ++p, ++plan.nph) {
                plan.tile0[plan.nph] = (int)at + rest_plan.tile0[p];
                plan.ntile[plan.nph] = rest_plan.ntile[p];
                plan.split[plan.nph] = rest_plan.split[p];
                plan.slot0[plan.nph] = nslot + rest_plan.slot0[p];
            }
            nslot += rest_slots;
            at = tiles;
        }
        ntile = (int)(at - tile0);
        return true;
    }
};
static_assert(1 + PLAN_SPLIT_PHASES <= PLAN_MAX_PHASES, "a round of whole tiles ahead of the rest's phases");

// float64 sums (what every N of up to 2048 has in any case): rows that are narrow, or not whole 16-byte pieces
bool needs_float64(const void *X, long long N, long long m, int nt) {
    return (nt < X_WIDE_TILES || (m % 8) != 0 || ((uintptr_t)X & 15) != 0) && N > (long long)X_PIECE * XK;
}

// ---- without scratch: 128 x 128 tiles, all of them, the chunks (2048 activations) added up in float64 registers --------------
// (131072 x 512: 3.9 ms, 16384 x 2048: 0.48 ms; with a workgroup per 256 x 256 tile a narrow layer has fewer of them than
// compute units, and 1024 x 512 took 47 us instead of 32)
constexpr int HT = 128;            // output tile (rows and columns of H = columns of X)
constexpr int HK = 64;             // activations per LDS tile
constexpr int HK_PAD = HK + 8;     // bf16 per LDS row: 144 bytes (16-byte aligned; operand reads and staging
                                   // stores of a 16-lane group fall into distinct banks)
constexpr int H_THREADS = 256;
constexpr int FLUSH_TILES = 32;    // float32 accumulators are added into float64 every 32 tiles = 2048 activations

// LDS tile T[c][k]: column c of the X tile, HK consecutive activations (k contiguous: one
// ds_read_b128 gives a lane its 8 bf16 of an MFMA operand).
struct XTile {
    uint16_t t[HT][HK_PAD];
};
constexpr size_t H_LDS_BYTES = 4 * sizeof(XTile);     // two operands, double-buffered

// Half of the workgroup stages each operand tile.  One thread moves 8 activations x 8 neighbouring columns:
// eight 16-byte loads (a wavefront covers 8 activation rows x 128 contiguous bytes per instruction), an
// 8 x 8 transpose of 16-bit values in registers, eight 16-byte LDS stores (one per column).
struct Staged {
    uint32_t r[8][4];
};
__device__ __forceinline__ void load_task(const uint16_t *__restrict__ X, long long N, long long m, long long k0,
                                          long long c0, int st, bool vec, Staged &s) {
    const int ab = st & 7, cg = st >> 3;             // 8-activation block, 8-column group
    const long long c = c0 + 8 * cg;
#pragma unroll
    for (int t = 0; t < 8; ++t) {
        const long long k = k0 + 8 * ab + t;
        uint4 v = make_uint4(0u, 0u, 0u, 0u);
        if (k < N) {
            const uint16_t *src = X + k * m + c;
            if (vec && c + 8 <= m) {
                v = *(const uint4 *)src;             // m % 8 == 0 and X 16-byte aligned
            } else {
                uint32_t e[8];
#pragma unroll
                for (int q = 0; q < 8; ++q) e[q] = (c + q < m) ? src[q] : 0u;
                v = make_uint4(e[0] | (e[1] << 16), e[2] | (e[3] << 16), e[4] | (e[5] << 16), e[6] | (e[7] << 16));
            }
        }
        s.r[t][0] = v.x; s.r[t][1] = v.y; s.r[t][2] = v.z; s.r[t][3] = v.w;
    }
}
// columns [cb, ce) of the task's 8 (compile-time bounds once the caller's loop is unrolled): the 8 activations of
// column 8 cg + c go to 16-byte slot `slot` of that column's LDS row
__device__ __forceinline__ void store_cols(uint16_t (*T)[HK_PAD], int cg, int slot, const Staged &s, int cb, int ce) {
#pragma unroll
    for (int c = 0; c < 8; ++c) {
        if (c < cb || c >= ce) continue;
        uint32_t o[4];
#pragma unroll
        for (int d = 0; d < 4; ++d) {
            const uint32_t a = s.r[2 * d][c >> 1], b = s.r[2 * d + 1][c >> 1];
            o[d] = (c & 1) ? ((a >> 16) | (b & 0xffff0000u)) : ((a & 0xffffu) | (b << 16));
        }
        *(uint4 *)&T[8 * cg + c][8 * slot] = make_uint4(o[0], o[1], o[2], o[3]);
    }
}
__device__ __forceinline__ void store_task(XTile &T, int st, const Staged &s) { store_cols(T.t, st >> 3, st & 7, s, 0, 8); }

__global__ void __launch_bounds__(H_THREADS) __attribute__((amdgpu_waves_per_eu(2, 2))) xtx_kernel(const uint16_t *__restrict__ X, long long N, long long m,
                                                        float *__restrict__ H, int vec) {
    extern __shared__ __align__(16) unsigned char smem[];
    XTile *TI = (XTile *)smem, *TJ = TI + 2;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wr = wave >> 1, wc = wave & 1;
    const int l32 = lane & 31, lhi = lane >> 5;
    const long long i0 = (long long)blockIdx.y * HT, j0 = (long long)blockIdx.x * HT;
    // threads 0..127 stage the tile of columns i0.., threads 128..255 the tile of columns j0..
    const int st = tid & 127;
    const bool stage_j = tid >= 128;
    const long long sc0 = stage_j ? j0 : i0;
    XTile *const ST = stage_j ? TJ : TI;

    floatx16 acc[2][2];
    double acc64[2][2][16];
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                acc[a][b][e] = 0.f;
                acc64[a][b][e] = 0.0;
            }

    const long long ntile = (N + HK - 1) / HK;
    Staged sg;
    load_task(X, N, m, 0, sc0, st, vec != 0, sg);
    store_task(ST[0], st, sg);
    __syncthreads();
    for (long long kt = 0; kt < ntile; ++kt) {
        const int buf = (int)(kt & 1);
        if (kt + 1 < ntile) load_task(X, N, m, (kt + 1) * HK, sc0, st, vec != 0, sg);
#pragma unroll
        for (int ks = 0; ks < HK / 16; ++ks) {
            // operand of a lane: 8 consecutive activations 16 ks + 8 (lane / 32) .. + 7 of one column
            const int kk = 16 * ks + 8 * lhi;
            const bf16x8 a0 = *(const bf16x8 *)&TI[buf].t[wr * 64 + l32][kk];
            const bf16x8 a1 = *(const bf16x8 *)&TI[buf].t[wr * 64 + 32 + l32][kk];
            const bf16x8 b0 = *(const bf16x8 *)&TJ[buf].t[wc * 64 + l32][kk];
            const bf16x8 b1 = *(const bf16x8 *)&TJ[buf].t[wc * 64 + 32 + l32][kk];
            acc[0][0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a0, b0, acc[0][0], 0, 0, 0);
            acc[0][1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a0, b1, acc[0][1], 0, 0, 0);
            acc[1][0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a1, b0, acc[1][0], 0, 0, 0);
            acc[1][1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a1, b1, acc[1][1], 0, 0, 0);
        }
        if ((kt % FLUSH_TILES) == FLUSH_TILES - 1 || kt + 1 == ntile) {
#pragma unroll
            for (int a = 0; a < 2; ++a)
#pragma unroll
                for (int b = 0; b < 2; ++b)
#pragma unroll
                    for (int e = 0; e < 16; ++e) {
                        acc64[a][b][e] += (double)acc[a][b][e];
                        acc[a][b][e] = 0.f;
                    }
        }
        if (kt + 1 < ntile) store_task(ST[buf ^ 1], st, sg);
        __syncthreads();
    }

    // accumulator element e of a 32 x 32 tile: row = 8*(e/4) + 4*(lane/32) + e%4, column = lane%32
    const double inv = 1.0 / (double)N;
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const long long i = i0 + wr * 64 + a * 32 + 8 * (e >> 2) + 4 * lhi + (e & 3);
                const long long j = j0 + wc * 64 + b * 32 + l32;
                if (i < m && j < m) H[i * m + j] = (float)(acc64[a][b][e] * inv);
            }
}

}  // namespace

extern "C" size_t skim_hessian_workspace_bytes(const skim_ctx *ctx, int64_t N, int64_t m) {
    if (!ctx || N < 1 || m < 1 || m > 0x7fffffff) return 0;
    const int64_t nt = (m + XT - 1) / XT, tiles = nt * (nt + 1) / 2;
    const int nstage = (int)((N + XK - 1) / XK);
    if (needs_float64(nullptr, N, m, (int)nt)) return piece_bytes(tiles, nstage, ctx->num_cu);
    return (size_t)WidePlan(ctx->num_cu, tiles, nstage, X_SCRATCH_MOST / TILE_SLOT_BYTES).most * TILE_SLOT_BYTES;
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
        SKIM_HIP(ctx, hipFuncSetAttribute((const void *)xtx_big_kernel<SUM_IN_H>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)X_LDS_BYTES));
        SKIM_HIP(ctx, hipFuncSetAttribute((const void *)xtx_big_kernel<SUM_IN_SLOTS>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)X_LDS_BYTES));
        SKIM_HIP(ctx, hipFuncSetAttribute((const void *)xtx_big_kernel<SUM_PIECES>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)X_LDS_BYTES));
        SKIM_HIP(ctx, hipFuncSetAttribute((const void *)xtx_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)H_LDS_BYTES));
        ctx->xtx_lds_enabled = 1;
    }
    const int nt = (int)((m + XT - 1) / XT);
    const int G = ctx->num_cu;
    TilePlan plan;
    const long long tiles = (long long)nt * (nt + 1) / 2;
    const int nstage = (int)((N + XK - 1) / XK);
    const double inv = 1.0 / (double)N;
    auto launch = [&](auto mode, const TilePlan &plan, const uint16_t *X, long long Np, float4 *slots, uint4 *pieces, int nslot) {
        long long grid = 0;
        for (int p = 0; p < plan.nph; ++p) {
            const long long items = (long long)plan.ntile[p] * plan.split[p];
            if (items > grid) grid = items;
        }
        if (grid > G) grid = G;
        hipLaunchKernelGGL(xtx_big_kernel<decltype(mode)::value>, dim3((unsigned)grid), dim3(X_THREADS), X_LDS_BYTES, ctx->stream, X, Np,
                           (long long)m, H, nt, plan, slots, pieces, nslot);
    };
    auto finish = [&](const TilePlan &plan, int stages, const float4 *slots, const uint4 *pieces, int nslot, int tile0, long long ntile,
                      double2 *run, bool first, bool last) {
        hipLaunchKernelGGL(pieces ? xtx_finish_kernel<true> : xtx_finish_kernel<false>, dim3((unsigned)(ntile * 16)), dim3(256), 0, ctx->stream, H,
                           inv, stages, (long long)m, nt, plan, slots, pieces, nslot, tile0, run, first, last);
    };
    const bool float64 = needs_float64(X_bf16, N, m, nt);
    PiecePlan pp;
    bool fits = false;
    int T = group_tiles(tiles, G);
    if (float64 && scratch)
        for (;; T = (T + 1) / 2) {
            const int rest = (int)(tiles % T);
            fits = (!rest || piece_plan(pp, G, rest, nstage, scratch_bytes)) && piece_plan(pp, G, T, nstage, scratch_bytes);
            if (fits || T == 1) break;
        }
    if (fits) {
        for (long long t0 = 0; t0 < tiles; t0 += T) {
            const int ntile = (int)(tiles - t0 < T ? tiles - t0 : T);
            if (ntile < T) (void)piece_plan(pp, G, ntile, nstage, scratch_bytes);
            plan = pp.plan;
            for (int p = 0; p < plan.nph; ++p) plan.tile0[p] += (int)t0;
            float4 *slots = (float4 *)scratch;
            uint4 *pieces = (uint4 *)((char *)scratch + (size_t)pp.nslot * TILE_SLOT_BYTES);
            double2 *run = pp.passes > 1 ? (double2 *)((char *)scratch + pp.run_offset()) : nullptr;
            for (int q = 0; q < pp.passes; ++q) {
                const long long s0 = (long long)nstage * q / pp.passes, s1 = (long long)nstage * (q + 1) / pp.passes;
                const long long Np = (N < s1 * XK ? N : s1 * XK) - s0 * XK;
                launch(std::integral_constant<int, SUM_PIECES>{}, plan, X_bf16 + s0 * XK * m, Np, slots, pieces, pp.nslot);
                finish(plan, (int)(s1 - s0), slots, pieces, pp.nslot, (int)t0, ntile, run, q == 0, q == pp.passes - 1);
            }
        }
        SKIM_HIP(ctx, hipGetLastError());
        return SKIM_OK;
    }
    WidePlan wide(G, tiles, nstage, (long long)((scratch ? (scratch_bytes < X_SCRATCH_MOST ? scratch_bytes : X_SCRATCH_MOST) : 0) / TILE_SLOT_BYTES));
    const bool direct = !wide.fits();
    if (float64 || (direct && nt < X_WIDE_TILES)) {
        const int vec = (m % 8 == 0) && (((uintptr_t)X_bf16 & 15) == 0);     // rows of X start 16-byte aligned
        const unsigned ntiles = (unsigned)((m + HT - 1) / HT);
        hipLaunchKernelGGL(xtx_kernel, dim3(ntiles, ntiles), dim3(H_THREADS), H_LDS_BYTES, ctx->stream, X_bf16, (long long)N, (long long)m, H, vec);
        SKIM_HIP(ctx, hipGetLastError());
        return SKIM_OK;
    }
    if (direct) {
        (void)skim_make_plan(plan, G, tiles, nstage, X_MIN_STAGES, X_PHASE_COST, true);
        launch(std::integral_constant<int, SUM_IN_H>{}, plan, X_bf16, (long long)N, nullptr, nullptr, 0);
        finish(plan, nstage, nullptr, nullptr, 0, 0, tiles, nullptr, true, true);
    } else {
        float4 *slots = (float4 *)scratch;
        for (int tile0, ntile, nslot; wide.next(plan, tile0, ntile, nslot);) {
            launch(std::integral_constant<int, SUM_IN_SLOTS>{}, plan, X_bf16, (long long)N, slots, nullptr, 0);
            finish(plan, nstage, slots, nullptr, 0, tile0, ntile, nullptr, true, true);
        }
    }
    SKIM_HIP(ctx, hipGetLastError());
    return SKIM_OK;
}
