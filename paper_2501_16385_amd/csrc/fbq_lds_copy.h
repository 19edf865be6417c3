// Copies from global memory straight into LDS and the LDS layout they are used with (device code only).
#ifndef FBQ_LDS_COPY_H
#define FBQ_LDS_COPY_H

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace fbq {

// Sixteen bytes per lane from global memory straight into LDS, `lane_off` + `row_off` bytes behind the descriptor's
// base (row_off the same for all lanes): lane l's go to `dst` + 16 l, dst wave-uniform.  Written as an instruction and
// not with the builtin, because the compiler waits for EVERY load in flight before the first LDS read behind a builtin
// copy - it cannot tell the buffer being read from the ones being filled - which undoes any look-ahead: an earlier
// form of the prefill kernel began every round with vmcnt(0).  The instruction has no destination register; whoever reads
// a copy waits for it by count and passes a barrier (both with a memory clobber).  The compiler's own counted waits only
// get stricter by the copies it does not know of.  M0, the LDS address, is declared as overwritten: the compiler may keep a value there.
__device__ __forceinline__ uint32_t lds_offset(const void *p) { return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const void *)p; }
__device__ __forceinline__ void copy16_to_lds(__amdgpu_buffer_rsrc_t buf, int lane_off, int row_off, uint32_t dst)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds" ::"s"(dst), "v"(lane_off), "s"(buf), "s"(row_off) : "m0");
}
__device__ __forceinline__ void copy12_to_lds(__amdgpu_buffer_rsrc_t buf, int lane_off, int row_off, uint32_t dst)   // (12 bytes per lane, but 16 l apart in LDS)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx3 %1, %2, %3 offen lds" ::"s"(dst), "v"(lane_off), "s"(buf), "s"(row_off) : "m0");
}
__device__ __forceinline__ void copy4_to_lds(__amdgpu_buffer_rsrc_t buf, int lane_off, int row_off, uint32_t dst)    // (4 bytes: dst + 4 l)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dword %1, %2, %3 offen lds" ::"s"(dst), "v"(lane_off), "s"(buf), "s"(row_off) : "m0");
}
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer_of(const void *p, long bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, (int)bytes, 0x00020000);
}

// Piece c (16 bytes) of a row is stored at position c ^ piece_key(row): 8 or 16 consecutive rows reading the same c touch
// every bank once, whether the LDS serves 128 or 256 bytes per clock.
__host__ __device__ __forceinline__ constexpr int piece_key(int row) { return ((row >> 1) & 7) ^ ((row & 1) << 2); }

}  // namespace fbq

#endif
