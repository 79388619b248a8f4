// Loads of operand tiles from memory straight into LDS, and the waits that belong to them: shared by the bf16 MFMA kernels.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace lrd {
namespace {

// Loads go through buffer descriptors: 32-bit byte offsets from a wave-uniform base, and zeros for any
// offset past num_records (into LDS as well).
constexpr uint32_t BUF_FLAGS = 0x00020000u;      // raw buffer, 32-bit data format
constexpr uint32_t BUF_OOB = 0xFFFFFFF0u;        // >= every num_records used here
constexpr int64_t BUF_MAX_LD = int64_t(1) << 22; // keeps (256 rows x ld + K) x 2 bytes below BUF_OOB

// Wave-uniform values the compiler cannot always prove uniform; a descriptor built from them stays
// in scalar registers instead of being looped over per distinct lane value.
__device__ __forceinline__ uint32_t uni(uint32_t v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ int64_t uni64(int64_t v)
{
    uint64_t u = (uint64_t)v;
    return (int64_t)(((uint64_t)uni((uint32_t)(u >> 32)) << 32) | uni((uint32_t)u));
}
__device__ __forceinline__ const char* uni_ptr(const void* p)
{
    return reinterpret_cast<const char*>(uni64((int64_t)reinterpret_cast<uintptr_t>(p)));
}

// What a tile's descriptors are made of, five wait states after whatever vector instructions (readfirstlane) wrote it; the
// results are scalar registers of their own, from which scalar instructions make the base and extent of each K-step.
// (Once per tile: in every K-step it cost the small layers 3 %, 48 x 1024 -> 4096 at rank 256 9.0 -> 9.3 us.)
__device__ __forceinline__ void settle(const char*& base, uint32_t& span)
{
    asm volatile("s_nop 4" : "+s"(base), "+s"(span));
}
__device__ __forceinline__ void settle(const char*& base, int64_t& ld, int& cols)
{
    asm volatile("s_nop 4" : "+s"(base), "+s"(ld), "+s"(cols));
}

// 16 bytes per lane from memory into LDS: lane l's chunk lands at byte address lds + 16 l (lds is wave-uniform).
// As an instruction of its own and not the builtin: the compiler waits for every load of that builtin still in
// flight before each LDS read that might alias it, which is all of them here.  It has no register result; the
// waits are wait_vm's.  (s_nop: M0 must be written one state before an LDS load reads it.)  The compiler does not see a
// vector-memory instruction here, so it does not keep the five wait states between a scalar register written by a vector
// instruction and its use in a descriptor: what descriptors are made of goes through settle() first.  M0 is a reserved
// register, for whose clobber the compiler warns; nothing is kept in it across this, and it has to know of the write.
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ __forceinline__ void load_to_lds(uint32_t lds, const char* base, uint32_t span, uint32_t voff)
{
    __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(base), 0, (int)span, (int)BUF_FLAGS);
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds" ::"s"(lds), "v"(voff), "s"(r) : "memory", "m0");
}
#pragma clang diagnostic pop
// Until all but this wave's newest N vector-memory operations have completed.
template <int N>
__device__ __forceinline__ void wait_vm()
{
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}
// The same for N = min(rem, D) stages of LPS loads each.
template <int D, int LPS>
__device__ __forceinline__ void wait_stages(int rem)
{
    if constexpr (D == 0) wait_vm<0>();
    else if (rem >= D) wait_vm<D * LPS>();
    else wait_stages<D - 1, LPS>(rem);
}
// A barrier after this wave's own LDS reads have returned (not its loads: those are counted by wait_vm).
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// Permutation of the eight 16-byte chunks of a 128-byte LDS row: chunk c of row r lies in slot c ^ kc_swz(r), so that reads
// of one chunk of 16 consecutive rows fall on 16 different 16-byte columns of the banks.
__device__ __forceinline__ constexpr int kc_swz(int row) { return (row >> 1) & 7; }

}  // namespace
}  // namespace lrd
