// gfx950 primitives shared by every kernel that stages through LDS without registers: the direct
// global->LDS load, its wait, the raw buffer descriptor whose out-of-range offsets read zeros, and
// the XCD-aware renumbering of workgroups.
#pragma once
#include <hip/hip_runtime.h>

namespace relay {

typedef int intx4 __attribute__((ext_vector_type(4)));

// A buffer offset beyond the num_records of every input and filter buffer (the kernels take at most 2^31 - 1 bytes of them): reads
// zeros.  The residual buffer of conv3x3_halo_kernel alone may be larger (up to 2^32 - 2 bytes).  There an out-of-range lane reads what lies at
// 2^31, inside the tensor, and stores nothing.
constexpr unsigned kOob = 0x80000000u;

// The statement overwrites M0 and says so in its clobber list.  The compiler treats M0 as a reserved
// register (it sets M0 itself right before each of its own instructions that read it and keeps no
// value live there), warns about reserved registers in a clobber list, and honours the entry all the same.
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ __forceinline__ void lds_dma16(intx4 rsrc, unsigned lds_base, unsigned voff) {
  // m0 = wave-uniform LDS byte address; lane i lands at m0 + 16*i
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds" ::"s"(lds_base), "v"(voff),
               "s"(rsrc)
               : "memory", "m0");
}

// Touches 64 memory lines of 128 bytes, one per lane, so that they are on their way to this XCD's L2: the four bytes
// each lane fetches land in a 256-byte dump block of LDS and are never read.
__device__ __forceinline__ void l2_touch(intx4 rsrc, unsigned dump_base, unsigned voff) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dword %1, %2, 0 offen lds" ::"s"(dump_base), "v"(voff), "s"(rsrc)
               : "memory", "m0");
}

#pragma clang diagnostic pop

// Wait until at most N of this wave's global->LDS loads are pending and all of its LDS reads
// have returned (so that the stage they read may be refilled after the barrier).
template <int N>
__device__ __forceinline__ void wait_loads() {
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(N) : "memory");
}

__device__ __forceinline__ intx4 make_rsrc(const void* p, unsigned bytes) {
  const unsigned long long pa = reinterpret_cast<unsigned long long>(p);
  intx4 r;
  r[0] = (int)(unsigned)pa;
  r[1] = (int)(unsigned)((pa >> 32) & 0xffffu);  // stride 0: raw buffer
  r[2] = (int)bytes;                            // num_records
  r[3] = 0x00020000;                            // 32-bit data format, no swizzle
  return r;
}

// Workgroup id -> logical tile id such that consecutive logical ids run on the same XCD
// (workgroups are dealt round-robin over the 8 XCDs, each with its own L2): tiles that
// share input rows or filter tiles then share an L2.
// nb, the workgroups of the launch, is the kernels' leading scalar parameter.  The build has the packet processor put leading scalars into registers
// (-amdgpu-kernarg-preload-count), so this arithmetic runs while the other arguments are on their way; and because the processor has fetched
// the first line of them, the kernel's own loads find it: a batch over eight lines is back after 740 clocks instead of 1130, over one 190 instead of
// 480.  With the blocks' fields in the order of their use (ConvArgs), against neither: ResNet-18 at batch 1 78.5 -> 77.2 us, at batch 7 128.0 ->
// 126.3, int8 batch 16 127.0 -> 124.2, MobileNet-v1 at batch 1 83.3 -> 82.7, at batch 32 220 -> 215 (means of three processes).
__device__ __forceinline__ int xcd_remap(int bid, int nb) {
  const int xcd = bid & 7, idx = bid >> 3;
  const int per = nb >> 3, rem = nb & 7;
  return xcd * per + min(xcd, rem) + idx;
}

// The first touch of a launch's filters, shared by its waves.  Filters that an earlier layer's traffic has pushed
// out of the caches come from HBM, and a reduction that asks for them chunk by chunk, two or three chunks
// ahead, waits most of that latency for every chunk.  So the workgroups an XCD starts with touch, between them,
// every line of the filters that XCD is going to read, right behind their own first loads: with filters from HBM
// 512 -> 512 at 7 x 7, batch 32 takes 16.5 us instead of 19.9, 256 -> 256 at 14 x 14 14.8 instead of 17.7.
// first, bytes: the XCD's range of the packed filters; wid: this wave's place among the `waves` that take part; at
// most MAX touches (8 KiB each); returns how many this wave issued.
template <int MAX>
__device__ __forceinline__ int touch_filters(intx4 rs_w, unsigned dump_base, unsigned first, unsigned bytes, int wid, int waves, int lane) {
#pragma unroll
  for (int j = 0; j < MAX; ++j) {
    const unsigned at = (unsigned)(wid + j * waves) * 8192u;
    if (at >= bytes) return j;  // (uniform)
    l2_touch(rs_w, dump_base, first + at + (unsigned)lane * 128u);
  }
  return MAX;
}

}  // namespace relay
