// The fixed-order sum of fp32 partial planes into the output, scaled and converted: second kernel of
// the column-layout applies that split rows (k_mfma.hip) and of the dense sketch (k_gauss.hip).
#pragma once
#include "convert.h"
#include "handle.h"

namespace fs {
namespace {

// out[row][col] = scale * sum_p ws[p][row][col], planes added in index order (PARTS > 1: PARTS
// contiguous shares of them, added in order).
// RUN > 1: plane c of the output block at orbit position pos holds a tile only when
// delta = c*RUN + (pos%RUN + kappa)%RUN - kappa <= RUN-2 (the writer's relative position).
// PARTS: a work-group serves 256/PARTS outputs through PARTS threads each; used when outputs are few
// and planes many (one thread per output then waits for memory once per 8 planes on a chip that is
// mostly idle).
template <typename T, int PARTS>
__global__ __launch_bounds__(256) void reduce_planes_kernel(const float* __restrict__ ws, int planes,
                                                            int64_t k, int64_t ldw, int n,
                                                            T* __restrict__ out, int64_t ldo,
                                                            float scale, int out_vec, int run,
                                                            const uint32_t* __restrict__ blk2pos,
                                                            uint32_t Br, uint32_t kappa) {
  constexpr int OPW = 256 / PARTS;
  constexpr int UN = PARTS > 1 ? 8 : 4;  // loads issued together (with many outputs, the waves of a SIMD hide the rest)
  const int share = PARTS > 1 ? (int)threadIdx.x / OPW : 0;
  const int64_t idx = (int64_t)blockIdx.x * OPW + (int)threadIdx.x % OPW;  // over k * ldw/4
  const int64_t q = ldw / 4;
  const bool valid = idx < k * q;
  if (PARTS == 1 && !valid) return;
  const int64_t row = valid ? idx / q : 0;
  const int col0 = valid ? (int)(idx % q) * 4 : 0;
  uint32_t rho_k = 0;
  if (run > 1) rho_k = (blk2pos[row / Br] % (uint32_t)run + kappa) % (uint32_t)run;
  const float* src = ws + row * ldw + col0;
  float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
  // The planes that count are planes 0 .. nvalid-1 (RUN > 1: once a plane is empty the later ones
  // are too).  UN at a time: their loads are issued together, then added in index order; past
  // the last one the load repeats it (a cache hit) and is ignored.  One load per pass of a loop
  // made this kernel wait for memory once per plane.
  int nvalid = planes;
  if (run > 1) {
    nvalid = 0;
    while (nvalid < planes && (int)(nvalid * run + rho_k) - (int)kappa <= run - 2) ++nvalid;
  }
  const int per = (nvalid + PARTS - 1) / PARTS;
  const int first = share * per, last = min(first + per, nvalid);
  for (int p0 = first; p0 < last; p0 += UN) {
    float4 v[UN];
#pragma unroll
    for (int j = 0; j < UN; ++j)
      v[j] = *reinterpret_cast<const float4*>(src + (int64_t)min(p0 + j, last - 1) * k * ldw);
#pragma unroll
    for (int j = 0; j < UN; ++j)
      if (p0 + j < last) { s.x += v[j].x; s.y += v[j].y; s.z += v[j].z; s.w += v[j].w; }
  }
  if constexpr (PARTS > 1) {
    __shared__ float4 sh[PARTS][OPW];
    sh[share][threadIdx.x % OPW] = s;
    __syncthreads();
    if (share > 0 || !valid) return;
#pragma unroll
    for (int i = 1; i < PARTS; ++i) {
      const float4 v = sh[i][threadIdx.x];
      s.x += v.x; s.y += v.y; s.z += v.z; s.w += v.w;
    }
  }
  float v[4] = {s.x * scale, s.y * scale, s.z * scale, s.w * scale};
  T* dst = out + row * ldo + col0;
  if (out_vec && col0 + 3 < n) {
    if constexpr (sizeof(T) == 2) {
      const uint2 w = pack4<T>(v);
      *reinterpret_cast<uint2*>(dst) = w;
    } else {
      *reinterpret_cast<float4*>(dst) = make_float4(v[0], v[1], v[2], v[3]);
    }
  } else {
#pragma unroll
    for (int c = 0; c < 4; ++c)
      if (col0 + c < n) Elt<T>::store(dst + c, v[c]);
  }
}

// Whether a call's planes are added in shares.  (65536 threads are one per lane of a SIMD on every SIMD.)
inline bool reduce_in_parts(int planes, int64_t k, int64_t ldw) { return planes >= 16 && k * (ldw / 4) < 65536; }

// Enqueues it for element type T.  run / blk2pos / Br / kappa: the orbit-run layout of the planes, or
// run = 1.
template <typename T>
hipError_t launch_reduce_planes(const float* ws, int planes, int64_t k, int64_t ldw, int64_t n, void* out, int64_t ldo,
                                float scale, int run, const uint32_t* blk2pos, uint32_t Br, uint32_t kappa,
                                hipStream_t st) {
  const int out_vec = ((uintptr_t)out % (4 * sizeof(T)) == 0 && ldo % 4 == 0) ? 1 : 0;
  const int64_t work = k * (ldw / 4);
  const bool parts = reduce_in_parts(planes, k, ldw);
  const int64_t opw = parts ? 32 : 256;
  const dim3 grid((unsigned)((work + opw - 1) / opw));
  if (parts)
    hipLaunchKernelGGL((reduce_planes_kernel<T, 8>), grid, dim3(256), 0, st, ws, planes, k, ldw, (int)n, (T*)out, ldo,
                       scale, out_vec, run, blk2pos, Br, kappa);
  else
    hipLaunchKernelGGL((reduce_planes_kernel<T, 1>), grid, dim3(256), 0, st, ws, planes, k, ldw, (int)n, (T*)out, ldo,
                       scale, out_vec, run, blk2pos, Br, kappa);
  return hipGetLastError();
}

}  // namespace
}  // namespace fs
