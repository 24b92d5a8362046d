// LDS-DMA primitives shared by the pipelined kernels: buffer loads that land in LDS without
// passing through registers, issued from inline assembly so that the kernel, not the
// compiler, decides how many of them stay in flight.
#pragma once
#include <hip/hip_runtime.h>

namespace sdconv {

typedef int int4v __attribute__((ext_vector_type(4)));

constexpr unsigned kOutOfRange = 0x80000000u;   // byte offset no tensor here reaches

// Raw buffer descriptor over `bytes` bytes at `p` (stride 0, range-checked on the offset).
__device__ __forceinline__ int4v make_rsrc(const void* p, unsigned bytes)
{
    unsigned long long a = reinterpret_cast<unsigned long long>(p);
    int4v r;
    // readfirstlane pins the words to scalar registers: the descriptor is an "s" operand of
    // the load and the compiler may otherwise keep a copy in vector registers under pressure
    r.x = __builtin_amdgcn_readfirstlane((int)(unsigned)a);
    r.y = __builtin_amdgcn_readfirstlane((int)((a >> 32) & 0xffffu));
    r.z = __builtin_amdgcn_readfirstlane((int)bytes);
    r.w = 0x00020000;
    return r;
}

// 16 bytes per lane from buffer offset voff + soff to LDS address lds_base + lane*16
// (rsrc, soff, lds_base wave-uniform).  A voff at or past the descriptor's size yields zeros
// in LDS and touches no memory.
__device__ __forceinline__ void dma16(unsigned voff, int4v rsrc, unsigned soff, unsigned lds_base)
{
    asm volatile("s_mov_b32 m0, %3\n\ts_nop 0\n\tbuffer_load_dwordx4 %0, %1, %2 offen lds"
                 :: "v"(voff), "s"(rsrc), "s"(soff), "s"(lds_base) : "memory");
}

// N <= 4 loads of 16 bytes per lane whose 1 KiB land one behind the other from lds_base on, with one write of m0: the
// instruction's own offset counts for both addresses, so load i of them reads 1024 i bytes past its offset
// (kRunSlack - run_offset(i) takes that back, with a descriptor that starts kRunSlack before its tensor).
constexpr unsigned kRunSlack = 3072;
__device__ __forceinline__ constexpr unsigned run_offset(int i) { return (i & 3) * 1024u; }
template <int N>
__device__ __forceinline__ void dma16_run(const unsigned* v, int4v rsrc, unsigned soff, unsigned lds_base)
{
    static_assert(N >= 1 && N <= 4, "offsets of 12 bits");
    if constexpr (N == 1)
        asm volatile("s_mov_b32 m0, %3\n\ts_nop 0\n\tbuffer_load_dwordx4 %0, %1, %2 offen lds"
                     :: "v"(v[0]), "s"(rsrc), "s"(soff), "s"(lds_base) : "memory");
    else if constexpr (N == 2)
        asm volatile("s_mov_b32 m0, %4\n\ts_nop 0\n\tbuffer_load_dwordx4 %0, %2, %3 offen lds\n\t"
                     "buffer_load_dwordx4 %1, %2, %3 offen offset:1024 lds"
                     :: "v"(v[0]), "v"(v[1]), "s"(rsrc), "s"(soff), "s"(lds_base) : "memory");
    else if constexpr (N == 3)
        asm volatile("s_mov_b32 m0, %5\n\ts_nop 0\n\tbuffer_load_dwordx4 %0, %3, %4 offen lds\n\t"
                     "buffer_load_dwordx4 %1, %3, %4 offen offset:1024 lds\n\t"
                     "buffer_load_dwordx4 %2, %3, %4 offen offset:2048 lds"
                     :: "v"(v[0]), "v"(v[1]), "v"(v[2]), "s"(rsrc), "s"(soff), "s"(lds_base) : "memory");
    else
        asm volatile("s_mov_b32 m0, %6\n\ts_nop 0\n\tbuffer_load_dwordx4 %0, %4, %5 offen lds\n\t"
                     "buffer_load_dwordx4 %1, %4, %5 offen offset:1024 lds\n\t"
                     "buffer_load_dwordx4 %2, %4, %5 offen offset:2048 lds\n\t"
                     "buffer_load_dwordx4 %3, %4, %5 offen offset:3072 lds"
                     :: "v"(v[0]), "v"(v[1]), "v"(v[2]), "v"(v[3]), "s"(rsrc), "s"(soff), "s"(lds_base) : "memory");
}
// ... and any number of them, four at a time.
template <int N>
__device__ __forceinline__ void dma16_runs(const unsigned* v, int4v rsrc, unsigned soff, unsigned lds_base)
{
    if constexpr (N > 0) {
        dma16_run<(N < 4 ? N : 4)>(v, rsrc, soff, lds_base);
        dma16_runs<(N > 4 ? N - 4 : 0)>(v + 4, rsrc, soff, lds_base + 4096u);
    }
}

template <int N>
__device__ __forceinline__ void wait_vmcnt()
{
    asm volatile("s_waitcnt vmcnt(%0)" :: "n"(N) : "memory");
}

// All LDS reads of this wave have returned.  The builtin, not assembly: the compiler counts it and waits for
// nothing more where it uses their values.
__device__ __forceinline__ void wait_lds_reads() { __builtin_amdgcn_s_waitcnt(0xc07f); }    // lgkmcnt(0)

// Workgroup barrier behind which one stage that the loads above have filled is read and another is given
// back to them.  The compiler, which knows nothing of those writes, may keep no LDS value across it; and the LDS
// reads of this wave have returned: s_barrier itself waits for nothing, and the matrix instructions that
// the compiler waits in front of may move past it.
__device__ __forceinline__ void stage_barrier()
{
    asm volatile("" ::: "memory");
    wait_lds_reads();
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

}  // namespace sdconv
