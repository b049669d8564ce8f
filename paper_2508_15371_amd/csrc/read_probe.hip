// Probes for the benchmark and the tests (not part of the cmsd C ABI): the read ceiling, and
// the range check that the row kernels' loads rest on.
//
// A launch of `cmsd_probe_read_rows` reads every logit row the joint row pass reads,
// in the same grid shape (one workgroup per row, drafter rows first, then target
// rows) and with the same nontemporal 16-byte loads, but reduces nothing: each thread
// XORs its words and stores only if the result hits a fixed constant.  Its duration is
// what a single launch of that many bytes can achieve on the chip (ramp-up, tail and
// the HBM itself), so the benchmark can state how far the real kernel sits from a bare
// read of the same rows.  The up-to-15-byte unaligned ends of each row are skipped
// (under 32 bytes of a row of tens of kilobytes).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "row_buffer.h"

namespace {

template <int BD, int UNROLL>
__global__ __launch_bounds__(BD) void k_read_rows(const char* __restrict__ a, int64_t a_rows, int64_t a_stride,
                                                  const char* __restrict__ b, int64_t b_stride, int64_t row_bytes,
                                                  unsigned* __restrict__ sink) {
  const int64_t r = blockIdx.x;
  const char* row = r < a_rows ? a + r * a_stride : b + (r - a_rows) * b_stride;
  const uintptr_t p0 = reinterpret_cast<uintptr_t>(row);
  const uintptr_t v0 = (p0 + 15u) & ~uintptr_t(15);
  const uintptr_t v1 = (p0 + (uintptr_t)row_bytes) & ~uintptr_t(15);
  const int64_t nvec = v1 > v0 ? int64_t((v1 - v0) / 16u) : 0;
  const u32x4* vp = reinterpret_cast<const u32x4*>(v0);
  unsigned acc = 0;
  int64_t j = threadIdx.x;
  for (; j + (UNROLL - 1) * BD < nvec; j += UNROLL * BD) {
    u32x4 v[UNROLL];
#pragma unroll
    for (int u = 0; u < UNROLL; ++u) v[u] = __builtin_nontemporal_load(vp + j + u * BD);
#pragma unroll
    for (int u = 0; u < UNROLL; ++u) acc ^= v[u].x ^ v[u].y ^ v[u].z ^ v[u].w;
  }
  for (; j < nvec; j += BD) {
    const u32x4 v = __builtin_nontemporal_load(vp + j);
    acc ^= v.x ^ v.y ^ v.z ^ v.w;
  }
  if (acc == 0x9e3779b9u) sink[0] = acc;
}

// Rounds 0 .. rounds-1 of a row of nvec vectors at vp, loaded as the row kernels load
// them and written out in order.
template <int U, int BD>
__global__ __launch_bounds__(BD) void k_row_rounds(const uint4* __restrict__ vp, int nvec, int rounds,
                                                   uint4* __restrict__ out) {
  for (int k = 0; k < rounds; ++k) {
    uint4 v[U];
    load_round<U, BD>(vp, nvec, k, threadIdx.x, v);
#pragma unroll
    for (int u = 0; u < U; ++u) out[(k * U + u) * BD + threadIdx.x] = v[u];
  }
}
template <int U>
void launch_rounds(int bd, hipStream_t st, const uint4* vp, int nvec, int rounds, uint4* out) {
  const auto kernel = bd == 64 ? k_row_rounds<U, 64> : bd == 128 ? k_row_rounds<U, 128> : k_row_rounds<U, 256>;
  hipLaunchKernelGGL(kernel, dim3(1), dim3((unsigned)bd), 0, st, vp, nvec, rounds, out);
}

template <int BD>
void launch(int unroll, dim3 grid, hipStream_t st, const char* a, int64_t a_rows, int64_t a_stride, const char* b,
            int64_t b_stride, int64_t row_bytes, unsigned* sink) {
  if (unroll == 8)
    hipLaunchKernelGGL((k_read_rows<BD, 8>), grid, dim3(BD), 0, st, a, a_rows, a_stride, b, b_stride, row_bytes, sink);
  else
    hipLaunchKernelGGL((k_read_rows<BD, 4>), grid, dim3(BD), 0, st, a, a_rows, a_stride, b, b_stride, row_bytes, sink);
}

}  // namespace

extern "C" {

// Reads a_rows rows at a (stride a_stride bytes) and b_rows rows at b (stride
// b_stride), row_bytes bytes each, in one launch of a_rows + b_rows workgroups of bd
// threads (64, 128 or 256), `unroll` (4 or 8) loads in flight per thread.  All
// pointers are device pointers; sink is 4 device bytes the kernel may write.
// Returns 0 on launch, 1 on a bad argument, 3 on a launch error.
int cmsd_probe_read_rows(const void* a, int64_t a_rows, int64_t a_stride, const void* b, int64_t b_rows,
                         int64_t b_stride, int64_t row_bytes, int bd, int unroll, void* sink, void* stream) {
  if (a_rows < 0 || b_rows < 0 || row_bytes < 0 || !sink) return 1;
  if ((a_rows > 0 && (!a || a_stride < row_bytes)) || (b_rows > 0 && (!b || b_stride < row_bytes))) return 1;
  if (a_rows + b_rows > INT32_MAX || (bd != 64 && bd != 128 && bd != 256) || (unroll != 4 && unroll != 8)) return 1;
  if (a_rows + b_rows == 0) return 0;
  const dim3 grid((unsigned)(a_rows + b_rows));
  const hipStream_t st = static_cast<hipStream_t>(stream);
  const char* pa = static_cast<const char*>(a);
  const char* pb = static_cast<const char*>(b);
  unsigned* s = static_cast<unsigned*>(sink);
  if (bd == 64) launch<64>(unroll, grid, st, pa, a_rows, a_stride, pb, b_stride, row_bytes, s);
  else if (bd == 128) launch<128>(unroll, grid, st, pa, a_rows, a_stride, pb, b_stride, row_bytes, s);
  else launch<256>(unroll, grid, st, pa, a_rows, a_stride, pb, b_stride, row_bytes, s);
  return hipGetLastError() == hipSuccess ? 0 : 3;
}

// Loads rounds 0 .. rounds-1 of a row of nvec 16-byte vectors at vp as a row kernel of bd
// threads (64, 128 or 256) and u (4 or 8) vectors per thread does, into out[rounds*u*bd]:
// the row's vectors, then zeros.  The caller's buffer at vp holds all rounds*u*bd vectors,
// so that the loads stay inside it whatever the range check does.  Device pointers, 16-byte
// aligned.  Returns 0 on launch, 1 on a bad argument, 3 on a launch error.
int cmsd_probe_row_rounds(const void* vp, int64_t vp_vectors, int64_t nvec, int rounds, int bd, int u, void* out,
                          int64_t out_vectors, void* stream) {
  if ((bd != 64 && bd != 128 && bd != 256) || (u != 4 && u != 8) || rounds < 1 || rounds > 1024) return 1;
  const int64_t all = (int64_t)rounds * u * bd;
  if (!vp || !out || ((uintptr_t)vp | (uintptr_t)out) % 16 || nvec < 0 || nvec > all || vp_vectors < all ||
      out_vectors < all)
    return 1;
  const hipStream_t st = static_cast<hipStream_t>(stream);
  if (u == 8) launch_rounds<8>(bd, st, static_cast<const uint4*>(vp), (int)nvec, rounds, static_cast<uint4*>(out));
  else launch_rounds<4>(bd, st, static_cast<const uint4*>(vp), (int)nvec, rounds, static_cast<uint4*>(out));
  return hipGetLastError() == hipSuccess ? 0 : 3;
}

}  // extern "C"
