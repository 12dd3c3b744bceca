// Device-side helpers shared by the level kernels (cos_level.hip) and the
// sublattice level kernels (cos_sub.hip).
#pragma once
#include "cos_internal.hpp"

namespace libcos {

#define COS_RF(x) __builtin_amdgcn_readfirstlane(x)

typedef __attribute__((address_space(3))) double lds_double;
typedef __attribute__((address_space(3))) int lds_int;
// read-only tables read at wave-uniform addresses: through the constant
// address space they are fetched with scalar loads
typedef const __attribute__((address_space(4))) int32_t cint32;

// LDS byte address of a __shared__ pointer
__device__ __forceinline__ uint32_t lds_addr(double *p) {
    return (uint32_t)(uintptr_t)(lds_double *)p;
}

// accesses of the level kernels: a buffer descriptor over a plane of states
// (scalar registers), a byte offset per lane (one vector register) and a
// wave-uniform byte offset (one scalar register): no address arithmetic beyond
// one scalar add per slot.  Offsets inside a plane stay below 2^32.
typedef __amdgpu_buffer_rsrc_t plane_t;
typedef unsigned int __attribute__((ext_vector_type(2))) u32x2;
constexpr int kPlaneFlags = 0x00020000, kNt = 2;   // raw buffer; the nontemporal hint
__device__ __forceinline__ plane_t make_plane(const double *base) {
    return __builtin_amdgcn_make_buffer_rsrc((void *)base, 0, 0xffffffffu, kPlaneFlags);
}
__device__ __forceinline__ double slot_ld(plane_t p, uint32_t lane_off, uint32_t off) {
    return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(p, (int)lane_off, (int)off, 0));
}
__device__ __forceinline__ void slot_st(plane_t p, uint32_t lane_off, uint32_t off, double x) {
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, x), p, (int)lane_off, (int)off, 0);
}
// STREAM: with the nontemporal hint, for states far larger than the caches, which
// a level reads or writes once: they stream past the caches instead of evicting
// the tables and matrices
template <bool STREAM>
__device__ __forceinline__ double state_ld(plane_t p, uint32_t lane_off, uint32_t off) {
    return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(p, (int)lane_off, (int)off, STREAM ? kNt : 0));
}
template <bool STREAM>
__device__ __forceinline__ void state_st(plane_t p, uint32_t lane_off, uint32_t off, double x) {
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, x), p, (int)lane_off, (int)off, STREAM ? kNt : 0);
}

// Copies `slots` slots of 64 doubles from global memory to LDS by the whole
// workgroup, without passing through registers: every wavefront issues all of
// its 1 KB loads (two slots each, 16 bytes per lane) back to back, so the copy
// costs one memory latency instead of one per iteration of a load-and-write
// loop.  Returns when the caller's wavefront's part has arrived; the caller
// still needs a barrier.  src and dst are 16-byte aligned (slots are 512 bytes).
__device__ __forceinline__ void stage_slots(double *dst, const double *src, int slots) {
    typedef __attribute__((address_space(1))) const void gvoid;
    typedef __attribute__((address_space(3))) void lvoid;
    const int lane = threadIdx.x & 63, wave = COS_RF(threadIdx.x >> 6), waves = blockDim.x >> 6;
    for (int p = wave; 2 * p + 1 < slots; p += waves)
        __builtin_amdgcn_global_load_lds((gvoid *)(src + p * 128 + lane * 2), (lvoid *)(dst + p * 128), 16, 0, 0);
    if ((slots & 1) && wave == waves - 1) {   // an odd last slot: 4 bytes per lane, twice
        const int o = (slots - 1) * 64;
        __builtin_amdgcn_global_load_lds((gvoid *)((const int *)(src + o) + lane), (lvoid *)(dst + o), 4, 0, 0);
        __builtin_amdgcn_global_load_lds((gvoid *)((const int *)(src + o) + 64 + lane), (lvoid *)(dst + o + 32), 4, 0, 0);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
}

// The lane whose configuration a lane works on: its own, or in a group that is
// not full lane 0's.  Padding lanes repeat lane 0's work on lane 0's addresses
// (the same values, so that their stores agree), instead of moving states of
// their own: a group of 22 configurations touches 2 of a slot's 4 cache lines.
// (Orders 6 to 12, 600 configurations with six flavours, 86 a order in two groups:
// 26.0 -> 23.6 ms; one configuration of order 9 with gradients, six flavours: 1.41
// -> 1.03 ms.)
__device__ __forceinline__ uint32_t work_lane(const LvlArgs &A, int g, int lane) {
    return g * 64 + lane < A.count ? (uint32_t)lane : 0u;
}

// every flavour's plane of a level
struct Planes {
    const double *base;
    int64_t stride;   // doubles
    int n;
    __device__ __forceinline__ double sum(uint32_t lane_off, uint32_t at) const {
        double x = 0.0;
        for (int k = 0; k < n; ++k) x += slot_ld(make_plane(base + k * stride), lane_off, at);
        return x;
    }
};

// The workgroups of a launch, nx per group, are dealt to the chip's 8 XCDs round
// robin in the order of blockIdx.  Each XCD takes a contiguous part of them
// (groups one after another), so that the workgroups that run on it at a time
// serve one or two groups: their states lie in few pages and their G is in the
// XCD's own L2 (n = 10, 2048 configurations: forward 3.69 -> 3.64 ms, three
// flavours 6.30 -> 6.22 ms).  Returns false for the padding workgroups.
struct BlockAt {
    int x, group;
};
__device__ __forceinline__ bool xcd_block(const LvlArgs &A, BlockAt &at) {
    const int per = gridDim.x >> 3, id = (int)(blockIdx.x & 7u) * per + (int)(blockIdx.x >> 3);
    at.group = id / A.gridx;
    at.x = id - at.group * A.gridx;
    return at.group < A.ngroups;
}

// the next item of a workgroup's block, claimed by one wavefront
__device__ __forceinline__ int claim(int *next, int lane) {
    int nx = 0;
    if (lane == 0) nx = atomicAdd(next, 1);
    return COS_RF(nx);   // lane 0's claim (every lane is active here)
}

}  // namespace libcos
