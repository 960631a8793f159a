// Dense Gaussian sketch S_ij ~ N(0, 1/k) (paper Section 1 and Section 3: the
// canonical JL / OSE sketch) applied as a GEMM on the matrix cores: the
// dense-contraction reference point next to the sparse BlockPerm apply.
//
// S is materialised once at create time from a counter-based generator:
//   c  = mix32(lo32(i*d+j) ^ mix32(hi32(i*d+j) ^ key1 ^ C1))
//   u1 = ((mix32(c ^ 0x9E3779B9) >> 8) + 1) / 2^24,  u2 = (mix32(c ^ 0x85EBCA6B) >> 8) / 2^24
//   S_ij = (float)( sqrt(-2 ln u1) cos(2 pi u2) / sqrt(k) )          (Box-Muller, in fp64)
// and kept as fp32 (export), as bf16 and as half, each rounded to nearest (bf16 and half
// applies), and as an exact three-way bf16 split hi+mid+lo (fp32 applies).  The 16-bit copies are
// stored tile by tile ([row tile of 128][stage of 64 columns][128][64], 16 KiB each), so that what a
// work-group fetches per stage is contiguous.
//
// The GEMM reuses the data path of the sparse kernel: A goes HBM -> registers ->
// MFMA operand (4 columns x 8 rows per lane, transposed with v_perm_b32), S tiles of
// 128 rows x 64 columns are staged in LDS (double buffered, one barrier per stage that orders LDS
// traffic only: the loads of A stay in flight).
// fp32 applies use six bf16 MFMAs per tile (hi*hi, hi*mid, mid*hi, hi*lo, lo*hi,
// mid*mid); the dropped cross terms are below 2^-23 relative.
//
// What bounds it: the matrix cores, if a wave has enough of them per element it loads and (fp32)
// splits: a 128 x 128 wave tile (all 512 registers of a lane) has 96 MFMAs per 208 vector instructions of a
// k-step, a 32 x 128 one 24.  Such tiles are few (256 for k = 4096, n = 1024), so the d columns of S are
// split over grid.z into fp32 planes that a second kernel adds in order.
#include <math.h>

#include <type_traits>

#include "handle.h"
#include "mfma_common.h"
#include "reduce_planes.h"
#include "spec.h"

namespace fs {

namespace {

using namespace mm;

__global__ __launch_bounds__(256) void gauss_fill_kernel(float* __restrict__ S32, uint16_t* __restrict__ Sbf,
                                                         uint16_t* __restrict__ Shi, uint16_t* __restrict__ Smid,
                                                         uint16_t* __restrict__ Slo, uint16_t* __restrict__ Sh,
                                                         int64_t k, int64_t d, uint32_t key1, int tiled, double sqrt_k) {
  // `at`: place in the 16-bit copies, idx: in the matrix by rows.  Tiled: the threads walk the tiles, whose
  // 64-column rows are whole lines of S32 too (shapes no apply takes are left in rows).
  const int64_t at = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (at >= k * d) return;
  int64_t idx = at;
  if (tiled) {
    const int64_t tile = ((int64_t)blockIdx.x * 256) / (128 * KC), per_row = d / KC;  // uniform
    const int64_t trow = tile / per_row;
    idx = (trow * 128 + ((at >> 6) & 127)) * d + (tile - trow * per_row) * KC + (at & 63);
  }
  const uint32_t c = mix32((uint32_t)idx ^ mix32((uint32_t)((uint64_t)idx >> 32) ^ key1 ^ kC1));
  const double u1 = (double)((mix32(c ^ 0x9E3779B9u) >> 8) + 1u) * (1.0 / 16777216.0);
  const double u2 = (double)(mix32(c ^ 0x85EBCA6Bu) >> 8) * (1.0 / 16777216.0);
  const double z = sqrt(-2.0 * log(u1)) * cos(6.283185307179586476925 * u2);
  const float s = (float)(z / sqrt_k);
  S32[idx] = s;
  Sbf[at] = f32_to_bf16_rne(s);
  Sh[at] = f32_to_f16_bits(s);
  const uint32_t sb = __float_as_uint(s);
  const float r1 = s - __uint_as_float(sb & 0xFFFF0000u);
  const uint32_t r1b = __float_as_uint(r1);
  const float r2 = r1 - __uint_as_float(r1b & 0xFFFF0000u);
  Shi[at] = (uint16_t)(sb >> 16);
  Smid[at] = (uint16_t)(r1b >> 16);
  Slo[at] = (uint16_t)(__float_as_uint(r2) >> 16);
}

struct GaussArgs {
  const uint16_t* S[3];  // bf16 and half: S[0] only; fp32: hi, mid, lo
  const void* A;
  void* out;
  float* ws;  // zsplit > 1: planes of k x ldw floats
  int64_t k, d, lda, ldo, ldw;
  int n, total, stages, zsplit, out_vec;
};

// Work-group: 128 = 32*MT*NRG rows of S x 128*NCG columns of A, stages [z*stages, min((z+1)*stages, total)) of
// the d/64; wave: 32*MT rows x 128 columns.
template <typename T, int MT, int NRG, int NCG>
__global__ __launch_bounds__(64 * NRG * NCG) __attribute__((amdgpu_waves_per_eu(MT > 2 || (MT == 2 && sizeof(T) == 4) ? 1 : 2)))
void gauss_kernel(GaussArgs a) {
  using V = typename Ld<T>::V;
  constexpr int PFD = Ld<T>::PFD * (MT > 2 ? 2 : 1) > KSTEPS ? KSTEPS : Ld<T>::PFD * (MT > 2 ? 2 : 1);
  constexpr int PARTS = sizeof(T) == 4 ? 3 : 1;
  constexpr int NW = NRG * NCG, NT = 64 * NW;
  constexpr int RW = 32 * MT * NRG;
  static_assert(RW == 128, "the 16-bit copies of S are stored in tiles of 128 rows");
  constexpr int TILE = RW * PHI_LD;
  constexpr int SREG = RW * 8 / NT;  // 16-byte pieces of one S tile per thread
  static_assert(RW * 8 % NT == 0, "tile copy must divide evenly");

  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  uint16_t* s_tile = reinterpret_cast<uint16_t*>(smem);  // [2][PARTS][TILE]

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int rg = wave / NCG, cg = wave % NCG, kg = lane >> 5;
  const int col0 = (int)blockIdx.y * (WCOLS * NCG) + cg * WCOLS + 4 * (lane & 31);
  const int64_t row_base = (int64_t)blockIdx.x * RW;
  const int t0 = (int)blockIdx.z * a.stages;
  const int T_stages = min(a.stages, a.total - t0);  // >= 1
  const int64_t row_bytes = a.lda * (int64_t)sizeof(T);
  // The whole of A is one buffer (offsets fit 32 bits: checked on the host).  A lane whose columns all
  // lie at or beyond n gets an offset outside its range; a vector that straddles n loads the row's own
  // padding too (or nothing, behind the last row), which feeds only columns that are never stored.
  const uint32_t voff = col0 < a.n ? (uint32_t)(((int64_t)(kg * 8) * a.lda + col0) * (int64_t)sizeof(T)) : 0x80000000u;
  const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<void*>(a.A), 0, (int)((a.d - 1) * row_bytes + ((a.n + 3) & ~3) * (int64_t)sizeof(T)), 0x00020000);

  f32x16 acc[MT][4];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[mt][c][i] = 0.f;

  typedef uint32_t u4 __attribute__((ext_vector_type(4)));  // (an array of uint4 lands in scratch memory here)
  u4 sreg[PARTS * SREG];
  const int64_t s_first = ((int64_t)blockIdx.x * a.total + t0) * (RW * KC) + tid * 8;
  auto s_fetch = [&](int t) {
#pragma unroll
    for (int pt = 0; pt < PARTS; ++pt)
#pragma unroll
      for (int i = 0; i < SREG; ++i)
        sreg[pt * SREG + i] = *reinterpret_cast<const u4*>((pt == 0 ? a.S[0] : pt == 1 ? a.S[1] : a.S[2]) + s_first + (int64_t)t * (RW * KC) + i * NT * 8);
  };
  auto s_store = [&](int buf) {
#pragma unroll
    for (int pt = 0; pt < PARTS; ++pt)
#pragma unroll
      for (int i = 0; i < SREG; ++i) {
        const int e = tid + i * NT, row = e >> 3, c16 = e & 7;
        *reinterpret_cast<u4*>(s_tile + (buf * PARTS + pt) * TILE + row * PHI_LD + c16 * 8) = sreg[pt * SREG + i];
      }
  };
  auto lds_barrier = [&]() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
  };

  V ld[PFD][8];
  auto issue = [&](int kk, V (&dst)[8]) {
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const uint32_t soj = (uint32_t)((t0 * KSTEPS + kk) * 16 + j) * (uint32_t)row_bytes;
      if constexpr (sizeof(T) == 2)
        dst[j] = __builtin_bit_cast(V, __builtin_amdgcn_raw_buffer_load_b64(rs, voff, soj, 0));
      else
        dst[j] = __builtin_bit_cast(V, __builtin_amdgcn_raw_buffer_load_b128(rs, voff, soj, 0));
    }
  };

  auto stage = [&](int t, auto last_tag) {
    constexpr bool LAST = decltype(last_tag)::value;
    lds_barrier();  // tile t is complete, tile t+1's buffer has been read
    if constexpr (!LAST) s_fetch(t + 1);
    const uint16_t* tile = s_tile + (t & 1) * PARTS * TILE;
#pragma unroll
    for (int ks = 0; ks < KSTEPS; ++ks) {
      uint4 pa[PARTS][MT];
#pragma unroll
      for (int pt = 0; pt < PARTS; ++pt)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
          pa[pt][mt] = *reinterpret_cast<const uint4*>(
              tile + pt * TILE + ((rg * MT + mt) * 32 + (lane & 31)) * PHI_LD + ks * 16 + kg * 8);
      V(&cur)[8] = ld[ks % PFD];
      const bool fetch = !LAST || ks + PFD < KSTEPS;
      if constexpr (sizeof(T) == 2) {
        uint4 op[4];
        make_ops(cur, op);
        if (fetch) issue(t * KSTEPS + ks + PFD, cur);
#pragma unroll
        for (int c = 0; c < 4; ++c)
#pragma unroll
          for (int mt = 0; mt < MT; ++mt) acc[mt][c] = mfma<T>(pa[0][mt], op[c], acc[mt][c]);
      } else {
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          uint32_t xs[8];
#pragma unroll
          for (int j = 0; j < 8; ++j)
            xs[j] = c == 0 ? cur[j].x : c == 1 ? cur[j].y : c == 2 ? cur[j].z : cur[j].w;
          uint4 hi, mid, lo;
          split_ops(xs, hi, mid, lo);
          // product by product over the row tiles: with MT = 4 an accumulator is reused only
          // after three other MFMAs (back-to-back dependent MFMAs stall the matrix pipe)
#pragma unroll
          for (int mt = 0; mt < MT; ++mt) acc[mt][c] = mfma<T>(pa[0][mt], hi, acc[mt][c]);
#pragma unroll
          for (int mt = 0; mt < MT; ++mt) acc[mt][c] = mfma<T>(pa[0][mt], mid, acc[mt][c]);
#pragma unroll
          for (int mt = 0; mt < MT; ++mt) acc[mt][c] = mfma<T>(pa[1][mt], hi, acc[mt][c]);
#pragma unroll
          for (int mt = 0; mt < MT; ++mt) acc[mt][c] = mfma<T>(pa[0][mt], lo, acc[mt][c]);
#pragma unroll
          for (int mt = 0; mt < MT; ++mt) acc[mt][c] = mfma<T>(pa[2][mt], hi, acc[mt][c]);
#pragma unroll
          for (int mt = 0; mt < MT; ++mt) acc[mt][c] = mfma<T>(pa[1][mt], mid, acc[mt][c]);
        }
        if (fetch) issue(t * KSTEPS + ks + PFD, cur);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    if constexpr (!LAST) s_store((t + 1) & 1);
  };

#pragma unroll
  for (int i = 0; i < PFD; ++i) issue(i, ld[i]);
  s_fetch(0);
  s_store(0);
  for (int t = 0; t + 1 < T_stages; ++t) stage(t, std::false_type{});
  stage(T_stages - 1, std::true_type{});

  if (col0 >= a.n) return;
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) {
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int64_t row = row_base + (rg * MT + mt) * 32 + 8 * (i >> 2) + 4 * kg + (i & 3);
      const float v[4] = {acc[mt][0][i], acc[mt][1][i], acc[mt][2][i], acc[mt][3][i]};
      if (a.zsplit > 1) {  // a partial sum: plane blockIdx.z (col0 + 3 < ldw)
        *reinterpret_cast<float4*>(a.ws + ((int64_t)blockIdx.z * a.k + row) * a.ldw + col0) = make_float4(v[0], v[1], v[2], v[3]);
        continue;
      }
      T* dst = reinterpret_cast<T*>(a.out) + row * a.ldo + col0;
      if (a.out_vec && col0 + 3 < a.n) {
        if constexpr (sizeof(T) == 2) {
          const uint2 w = pack4<T>(v);
          *reinterpret_cast<uint2*>(dst) = w;
        } else {
          *reinterpret_cast<float4*>(dst) = make_float4(v[0], v[1], v[2], v[3]);
        }
      } else {
#pragma unroll
        for (int c = 0; c < 4; ++c)
          if (col0 + c < a.n) Elt<T>::store(dst + c, v[c]);
      }
    }
  }
}

// Columns per work-group (128, 256 or 512) and splits of the d/64 stages.  128-column waves that own all 128
// rows (512 columns per work-group) do the most matrix work per loaded element; fewer columns leave
// waves without any, so narrower work-groups divide the rows among the waves instead.  The smallest
// modelled time: rounds of resident work-groups times stages, plus the planes (written at 3.4, read at
// 6 TB/s, half that price while they stay in the Infinity Cache) and the reduction's launch.  Measured
// (us per call, one 128 x 512 or 128 x 256 work-group per tile before): fp32 65536 x 1024, k = 4096: 4390 -> 2350
// (1.4 PFLOP/s of bf16 products); fp32 41152 x 672, k = 1792: 5190 -> 614; half 42816 x 148, k = 384 (three
// work-groups with element loads before): 11030 -> 26.
struct GaussPlan { int ncg = 4, zsplit = 1, stages = 1; };
GaussPlan gauss_plan(int64_t k, int64_t d, int64_t n, fs_dtype dt, size_t scratch) {
  GaussPlan pl;
  const int total = (int)(d / KC);
  const double plane = (double)k * (double)((n + 3) & ~(int64_t)3) * 4.0;
  double best = 0;
  for (int ncg = 4; ncg >= 1; ncg /= 2) {
    const int64_t wgs = (k / 128) * ((n + 128 * ncg - 1) / (128 * ncg));
    // us per stage of a work-group that has its CU to itself
    const double stage_us = dt == FS_F32 ? (ncg == 4 ? 9.2 : ncg == 2 ? 5.2 : 4.0) : (ncg == 4 ? 2.0 : ncg == 2 ? 1.3 : 0.9);
    const int per_cu = dt == FS_F32 || ncg == 4 ? 1 : 2;
    for (int z = 1, st; z <= total && z <= 128; z = st > 1 ? (total + st - 2) / (st - 1) : total + 1) {
      st = (total + z - 1) / z;
      if (z > 1 && plane * z > (double)scratch) break;
      const double w = (double)wgs * z, rounds = ceil(w / (256 * per_cu));
      double t = rounds * (w > 256 && per_cu > 1 ? 1.7 : 1.0) * (st * stage_us + 3.0);
      if (z > 1) t += 4.0 + plane * z * (1 / 3.4e6 + 1 / 6e6) * (plane * z < 40e6 ? 0.5 : 1.0);
      if ((ncg == 4 && z == 1) || t < 0.98 * best) { best = t; pl.ncg = ncg; pl.zsplit = z; pl.stages = st; }
    }
  }
  return pl;
}

template <typename K>
hipError_t go(K kernel, dim3 grid, unsigned threads, size_t lds, hipStream_t st, const GaussArgs& a) {
  if (lds > 64 * 1024) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(kernel, grid, dim3(threads), lds, st, a);
  return hipGetLastError();
}

}  // namespace

// fp32, bf16, three pieces of the exact split, half.
size_t gauss_bytes(int64_t k, int64_t d) { return ((size_t)k * (size_t)d * (4 + 5 * 2) + 255) & ~(size_t)255; }

hipError_t gauss_fill(void* storage, int64_t k, int64_t d, uint32_t key1, hipStream_t st) {
  float* S32 = (float*)storage;
  uint16_t* b = (uint16_t*)(S32 + k * d);
  const int64_t blocks = (k * d + 255) / 256;
  if (blocks > 0x7fffffff) return hipErrorInvalidValue;
  const int tiled = d % KC == 0 && k % 128 == 0;
  hipLaunchKernelGGL(gauss_fill_kernel, dim3((unsigned)blocks), dim3(256), 0, st, S32, b, b + k * d,
                     b + 2 * k * d, b + 3 * k * d, b + 4 * k * d, k, d, key1, tiled, sqrt((double)k));
  return hipGetLastError();
}

bool gauss_supported(int64_t k, int64_t d, const void* A, int64_t lda, int64_t n, fs_dtype dt) {
  const int64_t esz = dt == FS_F32 ? 4 : 2;
  if (d % KC || k % 128 || n < 1) return false;
  if ((uintptr_t)A % (4 * esz) || lda % 4) return false;
  if (d * lda * esz >= ((int64_t)1 << 31)) return false;  // 32-bit buffer offsets over all of A
  return (n + 255) / 256 <= 65535;
}

hipError_t launch_gauss(void* storage, size_t scratch, int64_t k, int64_t d, const void* A, int64_t lda,
                        int64_t n, void* out, int64_t ldo, fs_dtype dt, hipStream_t st, EventPair ev) {
  const float* S32 = (const float*)storage;
  const uint16_t* b = (const uint16_t*)(S32 + k * d);
  const size_t esz = dt == FS_F32 ? 4 : 2;
  const GaussPlan pl = gauss_plan(k, d, n, dt, scratch);
  GaussArgs a;
  a.A = A; a.out = out; a.k = k; a.d = d; a.lda = lda; a.ldo = ldo; a.n = (int)n;
  a.total = (int)(d / KC); a.stages = pl.stages; a.zsplit = pl.zsplit;
  a.ldw = (n + 3) & ~(int64_t)3;
  a.ws = (float*)((char*)storage + gauss_bytes(k, d));
  a.out_vec = ((uintptr_t)out % (4 * esz) == 0 && (ldo * esz) % (4 * esz) == 0) ? 1 : 0;
  a.S[1] = a.S[2] = nullptr;
  if (dt == FS_F32) { a.S[0] = b + k * d; a.S[1] = b + 2 * k * d; a.S[2] = b + 3 * k * d; }
  else a.S[0] = dt == FS_BF16 ? b : b + 4 * k * d;
  const dim3 grid((unsigned)(k / 128), (unsigned)((n + 128 * pl.ncg - 1) / (128 * pl.ncg)), (unsigned)pl.zsplit);
  const size_t lds = (size_t)2 * (dt == FS_F32 ? 3 : 1) * 128 * PHI_LD * 2;
  if (ev.start) (void)hipEventRecord(ev.start, st);
  hipError_t e;
#define FS_G(T)                                                          \
  (pl.ncg == 4   ? go(gauss_kernel<T, 4, 1, 4>, grid, 256, lds, st, a)   \
   : pl.ncg == 2 ? go(gauss_kernel<T, 2, 2, 2>, grid, 256, lds, st, a)   \
                 : go(gauss_kernel<T, 1, 4, 1>, grid, 256, lds, st, a))
  e = dt == FS_F32 ? FS_G(float) : dt == FS_BF16 ? FS_G(uint16_t) : FS_G(f16);
#undef FS_G
  if (ev.stop) (void)hipEventRecord(ev.stop, st);
  if (e != hipSuccess || pl.zsplit == 1) return e;
#define FS_R(T) launch_reduce_planes<T>(a.ws, pl.zsplit, k, a.ldw, n, out, ldo, 1.0f, 1, nullptr, 1, 1, st)
  return dt == FS_F32 ? FS_R(float) : dt == FS_BF16 ? FS_R(uint16_t) : FS_R(f16);
#undef FS_R
}

}  // namespace fs
