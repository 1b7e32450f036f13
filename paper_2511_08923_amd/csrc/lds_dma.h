// Direct loads from memory into LDS, shared by the attention and GEMM kernels.
#pragma once
#include <hip/hip_runtime.h>

namespace {

// 16 bytes per lane straight from a raw buffer into LDS at lds_addr + 16 * lane (the tile's wave-uniform base goes
// through M0).  Written as inline assembly so that only the explicit vmcnt waits of a kernel order these loads
// against the LDS reads: issued through the compiler's builtin, every LDS read waits for *all* loads in flight,
// which is exactly the prefetch this is meant to keep running.
typedef int int4v __attribute__((ext_vector_type(4)));
__device__ inline int4v raw_desc(const void *base, size_t bytes) {
    const unsigned long long p = (unsigned long long)base;
    return (int4v){(int)(p & 0xffffffffull), (int)((p >> 32) & 0xffffull),
                   (int)(bytes > 0x7fffffe0ull ? 0x7fffffe0ull : bytes), 0x00020000};
}
// (M0 is a reserved register that the compiler sets itself right before each of its own uses; the kernels that use this have none.)
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ inline void dma16(unsigned lds_addr, int voff, int4v desc, int soff) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
                 :
                 : "s"(lds_addr), "v"(voff), "s"(desc), "s"(soff)
                 : "memory", "m0");
}
// The same for data that nobody reads again (weights that one workgroup reads once): non-temporal.
__device__ inline void dma16_once(unsigned lds_addr, int voff, int4v desc, int soff) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen nt lds"
                 :
                 : "s"(lds_addr), "v"(voff), "s"(desc), "s"(soff)
                 : "memory", "m0");
}
// The same OFFSET (< 4096) bytes further on, in memory and in LDS alike: tiles that lie side by side in both share lds_addr and
// soff.
template <int OFFSET, bool ONCE>
__device__ inline void dma16_at(unsigned lds_addr, int voff, int4v desc, int soff) {
    if constexpr (ONCE)
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen offset:%4 nt lds"
                     :
                     : "s"(lds_addr), "v"(voff), "s"(desc), "s"(soff), "n"(OFFSET)
                     : "memory", "m0");
    else
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen offset:%4 lds"
                     :
                     : "s"(lds_addr), "v"(voff), "s"(desc), "s"(soff), "n"(OFFSET)
                     : "memory", "m0");
}
#pragma clang diagnostic pop
// Tile i of tiles that lie side by side, 1 KiB each, in memory from soff and in LDS from lds_addr on: four share their base
// addresses.  Not `here`: out of bounds, through a buffer without records.  (i: a constant of the unrolled code; ONCE: as
// dma16_once)
template <bool ONCE = false>
__device__ __attribute__((always_inline)) inline void dma16_tile(unsigned lds_addr, int voff, int4v desc, bool here, int soff,
                                                                 int i) {
    desc[2] = here ? desc[2] : 0;
    lds_addr += (i & ~3) * 1024;
    soff = here ? soff + (i & ~3) * 1024 : 0;
    if ((i & 3) == 0) dma16_at<0, ONCE>(lds_addr, voff, desc, soff);
    else if ((i & 3) == 1) dma16_at<1024, ONCE>(lds_addr, voff, desc, soff);
    else if ((i & 3) == 2) dma16_at<2048, ONCE>(lds_addr, voff, desc, soff);
    else dma16_at<3072, ONCE>(lds_addr, voff, desc, soff);
}
__device__ inline void lds_barrier() {       // workgroup barrier for LDS traffic only: global loads stay in flight
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// The same with the wait as the builtin: the compiler then knows that no LDS read is outstanding and counts exactly which of the
// next ones an MFMA needs.
__device__ __attribute__((always_inline)) inline void lds_barrier_counted() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0xc07f);          // lgkmcnt(0)
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// Wave-uniform LDS address of a pointer into a workgroup's shared memory.
__device__ inline unsigned lds_address(unsigned char *p) {
    typedef __attribute__((address_space(3))) unsigned char lds_byte;
    return (unsigned)(size_t)(lds_byte *)p;
}
// Waits until at most N of the wave's vector-memory loads are in flight (they return in order).
template <int N>
__device__ inline void wait_loads() {
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

}  // namespace
