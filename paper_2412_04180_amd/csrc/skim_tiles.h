// Shared by the kernels that work on 256 x 256 output tiles with the matrix cores: copies straight from memory into
// LDS, and the plan that shares the tiles of a product out to the compute units.
#pragma once

#include "skim_common.h"

typedef int int4v __attribute__((ext_vector_type(4)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef __attribute__((address_space(3))) unsigned char lds_byte;

// Source of such copies: a region of memory that a wavefront walks in equal steps.  Bytes past `left` read as zero.
struct LdsSource {
    uint64_t base;
    long long left;
    // descriptor of a raw buffer that starts at base (scalar registers)
    __device__ __forceinline__ int4v rsrc() const {
        int4v rs;
        rs.x = (int)(uint32_t)base;
        rs.y = (int)((uint32_t)(base >> 32) & 0xFFFFu);
        rs.z = (int)max(min(left, 0x7FFFFFFFll), 0ll);
        rs.w = 0x00020000;
        return rs;
    }
    __device__ __forceinline__ void advance(uint64_t bytes) {
        base += bytes;
        left -= (long long)bytes;
    }
};
// 64 lanes x 16 bytes from voff into 1 KB of LDS at dst (the same in every lane).  The compiler does not see these
// loads: the kernels count them with s_waitcnt vmcnt themselves, and wait for the last of them before a workgroup
// ends (its LDS may be another's by then).
__device__ __forceinline__ void copy_to_lds(uint32_t dst, uint32_t voff, int4v rs) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds" ::"s"(dst), "v"(voff), "s"(rs) : "memory", "m0");
}

constexpr int TILE = 256;
constexpr size_t TILE_SLOT_BYTES = (size_t)TILE * TILE * sizeof(float);
constexpr int PLAN_MAX_PHASES = 6;
constexpr int PLAN_SPLIT_PHASES = 4;       // at most so many of them hold split tiles

// How the tiles of a product are shared out: phase p takes tiles tile0 .. tile0 + ntile - 1 and cuts the summation of
// each into `split` equal parts; part q of tile t is one piece of work.  Its sums go to a partial tile ("slot") of its own,
// number slot0 + q * ntile + (t - tile0).
struct TilePlan {
    int nph;
    int tile0[PLAN_MAX_PHASES], ntile[PLAN_MAX_PHASES], split[PLAN_MAX_PHASES], slot0[PLAN_MAX_PHASES];
};
// The plan for G workgroups and a summation of `nstage` stages, no part shorter than min_stages (whole: no tile is split).
// phase_cost: what starting a phase and writing its partial tiles costs, in stages.  Returns the number of slots.
long long skim_make_plan(TilePlan &plan, int G, long long tiles, int nstage, int min_stages, int phase_cost, bool whole);

// Workgroups of one XCD (ids equal modulo 8) get neighbouring numbers
__device__ __forceinline__ int xcd_order(int id, int G) {
    const int q8 = G >> 3, r8 = G & 7, xcd = id & 7;
    return xcd * q8 + min(xcd, r8) + (id >> 3);
}
