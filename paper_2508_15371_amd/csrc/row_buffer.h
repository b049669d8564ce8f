// row_buffer.h - one round of a row's 16-byte loads, through a buffer descriptor that ends
// at the row.  Shared by the row kernels (cmsd.hip) and by the probe that shows the range
// check on the device (read_probe.hip).
#ifndef CMSD_ROW_BUFFER_H
#define CMSD_ROW_BUFFER_H

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace {

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

// A raw buffer of 32-bit words (data format 4 in bits 18:15), and the nontemporal hint.
constexpr int kBufferFlags = 0x00020000;
constexpr int kBufferNt = 2;

// Round k of a row of nvec 16-byte vectors at vp: the vectors (k*U + u)*BD + t, u < U, of
// thread t.  Vectors past the row read zeros and no memory: the descriptor's records end at
// the row (none for a round past it), and the whole position of a vector within them is the
// lane's own offset, which is what a raw buffer's range check is defined over.  (The scalar
// offset would save the registers of the further vectors' offsets, but the intrinsic leaves
// it out of the check's contract, whatever the hardware does with it.)  A round takes a
// descriptor per kSpan vectors of a thread, which share the lanes' offsets: one descriptor
// for fp32's eight had two registers of 256-thread rows spilled (200 sequences of 8 drafts
// at V = 128256, GREEDY: 272.8 -> 271.0 us).  nvec and k are 32-bit (a row holds fewer than
// 2^31 logits): the scalar unit has no 64-bit comparison.  The count of records is said to
// be uniform, or the compiler clamps it in the vector unit and wraps every load in a loop
// over the lanes' values (one fp32 row of a million 99.6 -> 71.6 us).
// SKIP: vectors that no thread has are not requested (a load past the records reads nothing,
// but takes its turn in the memory pipeline all the same).
template <int U, int BD, bool SKIP = false>
__device__ __forceinline__ void load_round(const uint4* vp, int nvec, int k, int t, uint4 (&buf)[U]) {
  constexpr int kSpan = 4;
  static_assert(U % kSpan == 0, "whole descriptors");
#pragma unroll
  for (int h = 0; h < U; h += kSpan) {
    const int first = (k * U + h) * BD;  // the span's first vector
    const int left = nvec - first;
    const int n = __builtin_amdgcn_readfirstlane(left < 0 ? 0 : (left < kSpan * BD ? left : kSpan * BD));
    const __amdgpu_buffer_rsrc_t rs =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<uint4*>(vp) + first, 0, 16 * n, kBufferFlags);
#pragma unroll
    for (int u = 0; u < kSpan; ++u) {
      if (SKIP && u * BD >= n) {
        buf[h + u] = make_uint4(0u, 0u, 0u, 0u);
        continue;
      }
      const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(rs, (u * BD + t) * 16, 0, kBufferNt);
      buf[h + u] = make_uint4(v.x, v.y, v.z, v.w);
    }
  }
}

}  // namespace

#endif  // CMSD_ROW_BUFFER_H
