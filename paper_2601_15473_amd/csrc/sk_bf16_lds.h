// Operands that go from global memory straight into LDS (buffer_load ... lds): the layout they have
// there, how a wave asks for them and how their MFMA fragments are read.
//
// The compiler does not see these loads write LDS (they are inline assembly: a builtin would make it
// wait for every load in flight ahead of each LDS read), so what reads them waits by hand -- on the
// load counter, in which a wave's loads AND stores retire in order.
#pragma once
#include "sk_bf16_tile.h"

// (the compiler remarks that M0, which the loads below name as overwritten, is a register it never
// allocates; naming it keeps its own writes of M0 apart from their uses)
#pragma clang diagnostic ignored "-Winline-asm"

namespace sk {

// A panel of an operand in LDS, 8 KB: [64 rows (m or n)][64 k] for a k-contiguous operand, else
// [64 k][64 m or n] (read through the LDS transpose read).  Either way it is 64 lines of 128
// bytes, one load instruction of a wave fills eight lines, and the 16-byte pieces of a line are
// XOR-swizzled by line so that no read conflicts: the swizzle is in which piece of its line a
// lane asks for.  Panels of more rows follow one another (blocks of 32 rows: two to a panel).
template <bool KC>
struct Panels {
  static __device__ __forceinline__ int swizzle(int line) { return KC ? (line >> 1) & 7 : ((line >> 1) & 1) << 2; }
  // Byte offset from the chunk's origin of what `lane` loads as line 8 `line8` + lane / 8 of panel 0
  static __device__ __forceinline__ unsigned load_offset(int line8, int lane, unsigned ld_bytes) {
    const int line = line8 * 8 + (lane >> 3);
    return (unsigned)line * ld_bytes + (unsigned)((lane & 7) ^ swizzle(line)) * 16u;
  }
  // ... of its first k in the chunk (k-contiguous operands)
  static __device__ __forceinline__ int load_k(int line8, int lane) { return ((lane & 7) ^ swizzle(line8 * 8 + (lane >> 3))) * 8; }
  // LDS address a lane reads block 0, k step 0 of 128 rows `half` at; frag: any block and k step
  static __device__ __forceinline__ unsigned read_address(int half, int lane) {
    if (KC) {
      const int line = lane & 31;
      return half * 16384 + line * 128 + (((lane >> 5) ^ swizzle(line)) << 4);
    } else {   // (see read_frag: lane j of 16 addresses k row j / 4, columns 4 (j % 4) .. + 3)
      const int k = (lane >> 5) * 8 + ((lane & 15) >> 2), col = ((lane >> 4) & 1) * 16 + (lane & 3) * 4;
      return half * 16384 + k * 128 + (((col >> 3) ^ swizzle(k)) << 4) + (col & 4) * 2;
    }
  }
  static __device__ __forceinline__ bf16x8 frag(unsigned address, int block, int ks) {
    if constexpr (KC) {
      typedef __attribute__((address_space(3))) const bf16x8 lds_bf16x8;
      return *(lds_bf16x8*)(uintptr_t)((address ^ (ks << 5)) + block * 4096);
    } else {
      const unsigned p = (address ^ ((block & 1) << 6)) + (block >> 1) * 8192 + ks * 2048;
      const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(uintptr_t)(p));
      const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(uintptr_t)(p + 512));
      typedef short s16x8 __attribute__((ext_vector_type(8)));
      const s16x8 both = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
      return __builtin_bit_cast(bf16x8, both);
    }
  }
};

// Resource descriptor of what is left of an array of `total` elements from element `origin` on.
__device__ __forceinline__ u32x4 descriptor(const void* base, int64_t origin, int64_t total, int esize) {
  int64_t bytes = (total - origin) * esize;
  if (bytes < 0) bytes = 0;
  if (bytes > 0x7fffffff) bytes = 0x7fffffff;
  const uint64_t at = (uint64_t)base + origin * esize;
  return u32x4{(unsigned)at, (unsigned)(at >> 32), (unsigned)bytes, 0x00020000u};
}

// Each lane's 16 bytes at voff + soff of the array (zeros past its end) to LDS byte lds + 16 lane.
// (One wait state between the write of M0 and the load that reads it; in inline assembly the
// compiler does not insert it.)
__device__ __forceinline__ void load_to_lds(unsigned lds, unsigned voff, u32x4 array, unsigned soff) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds" ::"s"(lds), "v"(voff), "s"(array), "s"(soff) : "m0");
}

// A descriptor that is the same in all lanes, in scalar registers (some the compiler would compute in vector ones).
__device__ __forceinline__ u32x4 scalar(u32x4 d) {
  return u32x4{(unsigned)__builtin_amdgcn_readfirstlane((int)d.x), (unsigned)__builtin_amdgcn_readfirstlane((int)d.y),
               (unsigned)__builtin_amdgcn_readfirstlane((int)d.z), (unsigned)__builtin_amdgcn_readfirstlane((int)d.w)};
}

// The lane number computed afresh, for what is not to be kept in registers through the main loop.
__device__ __forceinline__ int lane_again() {
  int zero = 0;
  asm volatile("" : "+v"(zero));
  return __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, zero));
}

}  // namespace sk
