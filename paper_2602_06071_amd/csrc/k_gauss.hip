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
// Small fp32 applies use six bf16 MFMAs per tile (hi*hi, hi*mid, mid*hi, hi*lo, lo*hi,
// mid*mid); the dropped cross terms are below 2^-23 relative.  Larger ones use three half MFMAs (hi*hi, hi*lo, lo*hi) on
// x*2^e = hi + lo, two halfs of 11 significant bits: off by 2^-23 of x at most (a quarter of all numbers of 24 bits are), or,
// where lo falls under half's normal range (|x*2^e| < 2^-2), by 2^-25; the dropped lo*lo is below 2^-22.  Each column of A has an e of
// its own, by which its largest entry comes to lie between 2^14 and 2^15 (gauss_colmax_kernel), so that 2^-25 is 2^-39 of that entry;
// S has one for all.  Summed over a column of many terms that is less than what half as many rounded additions spare;
// column tiles with a column of few terms, where it would not be (a unit vector's sketch is a column of S), are computed with
// six products by a second launch (gauss_terms).
//
// What bounds it: the matrix cores, if a wave has enough of them per element it loads and (fp32)
// splits: a 128 x 128 wave tile (all 512 registers of a lane) has 48 MFMAs per 80 vector instructions of a
// k-step, a 32 x 128 one 12.  Such tiles are few (256 for k = 4096, n = 1024), so the d columns of S are
// split over grid.z into fp32 planes that a second kernel adds in order.  fp32 65536 x 1024, k = 4096: 1.39 ms, of which 47 us the
// pass for the column maxima (5.7 TB/s, half of them from the Infinity Cache), 1.25 PFLOP/s of half products (a library bf16
// product of 8192^3 on random data: 1.18 to 1.22; registers alone: 1.83 to 1.90).  Counted there: the matrix pipes are busy in
// 67 % of the cycles, 6 % of a wave's cycles wait, and the clock is 1.4 to 1.65 GHz of 2.4.
#include <math.h>
#include <stdio.h>

#include <type_traits>

#include "handle.h"
#include "lds_limit.h"
#include "mfma_common.h"
#include "reduce_planes.h"
#include "spec.h"

namespace fs {

namespace {

using namespace mm;

__global__ __launch_bounds__(256) void gauss_fill_kernel(float* __restrict__ S32, uint16_t* __restrict__ Sbf,
                                                         uint16_t* __restrict__ Shi, uint16_t* __restrict__ Smid,
                                                         uint16_t* __restrict__ Slo, uint16_t* __restrict__ Sh,
                                                         f16* __restrict__ H, f16* __restrict__ L, int es,
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
  if (H) {
    const float t = ldexpf(s, es);
    const f16 h = (f16)t;
    H[at] = h;
    L[at] = (f16)(t - (float)h);
  }
}

// Fourth root of the magnitude with these bits, to 6 %: a quarter of its exponent, and of its significand linearly.  Zero and
// subnormal numbers give kRoot0.  (Two of the root instruction made the pass over A wait for them, on 64 work-groups by 5 to 8 us.)
__device__ __forceinline__ float root4(uint32_t bits) { return __uint_as_float((bits >> 2) + 0x2FA00000u); }
constexpr float kRoot0 = 0x1.4p-32f;

// Of every column over the rows [c*rows, (c+1)*rows), c = blockIdx.y: the largest magnitude, as the bits of a float
// (NaN is above infinity), part[c][column], and the sum of the magnitudes' fourth roots, sums[c][column].  A work-group
// takes 4*2^sh columns, its lanes 4 each.
__global__ __launch_bounds__(1024) void gauss_colmax_kernel(const float* __restrict__ A, int64_t d, int64_t lda, int n,
                                                            int64_t rows, int sh, uint32_t* __restrict__ part,
                                                            float* __restrict__ sums, int64_t ldw) {
  __shared__ uint4 s_max[1024];
  __shared__ float4 s_sum[1024];
  const int tid = threadIdx.x, lanes = 1 << sh, sub = tid >> sh, nsub = 1024 >> sh;
  const int col0 = ((int)blockIdx.x * lanes + (tid & (lanes - 1))) * 4;
  const int64_t first = (int64_t)blockIdx.y * rows, last = min(first + rows, d);
  uint4 m = make_uint4(0, 0, 0, 0);
  float4 f = make_float4(0.f, 0.f, 0.f, 0.f);
  if (col0 < n) {
    constexpr int UN = 8;  // loads in flight
    for (int64_t r0 = first + sub; r0 < last; r0 += UN * nsub) {
      uint4 v[UN];
#pragma unroll
      for (int j = 0; j < UN; ++j)  // (past the end the last row again: a hit)
        v[j] = *reinterpret_cast<const uint4*>(A + min(r0 + j * nsub, last - 1) * lda + col0);
#pragma unroll
      for (int j = 0; j < UN; ++j) {
        const uint32_t mask = r0 + j * nsub < last ? 0x7fffffffu : 0u;
        v[j].x &= mask; v[j].y &= mask; v[j].z &= mask; v[j].w &= mask;
        m.x = max(m.x, v[j].x); m.y = max(m.y, v[j].y); m.z = max(m.z, v[j].z); m.w = max(m.w, v[j].w);
        if (mask) { f.x += root4(v[j].x); f.y += root4(v[j].y); f.z += root4(v[j].z); f.w += root4(v[j].w); }
      }
    }
  }
  s_max[tid] = m;
  s_sum[tid] = f;
  __syncthreads();
  for (int h = 512; h >= lanes; h >>= 1) {
    if (tid < h) {
      const uint4 o = s_max[tid + h];
      m.x = max(m.x, o.x); m.y = max(m.y, o.y); m.z = max(m.z, o.z); m.w = max(m.w, o.w);
      s_max[tid] = m;
      const float4 g = s_sum[tid + h];
      f.x += g.x; f.y += g.y; f.z += g.z; f.w += g.w;
      s_sum[tid] = f;
    }
    __syncthreads();
  }
  if (tid < lanes && col0 < n) {
    *reinterpret_cast<uint4*>(part + (int64_t)blockIdx.y * ldw + col0) = m;
    *reinterpret_cast<float4*>(sums + (int64_t)blockIdx.y * ldw + col0) = f;
  }
}

// x (8 rows of one column) * m as two half pieces each, rounded to nearest: what is left is at most 2^-23 of x*m or 2^-25.
__device__ __forceinline__ void split_half(const uint32_t (&x)[8], float m, uint4& hi, uint4& lo) {
  typedef f16 h2 __attribute__((ext_vector_type(2)));
  uint32_t* h = reinterpret_cast<uint32_t*>(&hi);
  uint32_t* l = reinterpret_cast<uint32_t*>(&lo);
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const float x0 = __uint_as_float(x[2 * q]), x1 = __uint_as_float(x[2 * q + 1]);
    h[q] = __builtin_bit_cast(uint32_t, h2{(f16)(x0 * m), (f16)(x1 * m)});
    asm("" : "+v"(h[q]));  // (or each half is made a second time for the difference)
    const h2 v = __builtin_bit_cast(h2, h[q]);
    // m is a power of two: exact before it is rounded
    l[q] = __builtin_bit_cast(uint32_t, h2{(f16)fmaf(x0, m, -(float)v.x), (f16)fmaf(x1, m, -(float)v.y)});
  }
}

struct GaussArgs {
  const uint16_t* S[3];  // bf16 and half: S[0] only; fp32: hi, mid, lo
  const void* A;
  void* out;
  float* ws;  // zsplit > 1: planes of k x ldw floats
  int64_t k, d, lda, ldo, ldw;
  int n, total, stages, zsplit, out_vec;
  // two half pieces: largest magnitudes of the columns and sums of their fourth roots, `parts` rows of ldw each, and the
  // exponent S was scaled by; `few`: for every column tile of grid.y whether one of its columns has fewer than `terms` terms,
  // written by the kernel of half pieces, which leaves such a tile to the one of three
  const uint32_t* colmax;
  const float* colsum;
  int* few;
  float terms;
  int parts, es;
  int cgroup;  // column tiles (of grid.y, which it divides) that consecutive work-groups take in turn
};

// Work-group: 128 = 32*MT*NRG rows of S x 128*NCG columns of A, stages [z*stages, min((z+1)*stages, total)) of
// the d/64; wave: 32*MT rows x 128 columns.
// HALF (fp32): two half pieces of both operands instead of three bf16 ones.
// ODD: whether a.stages is (only the kernel that walks two stages a pass has to know: a last stage of its own for either
// parity costs the accumulators of a wave their registers, 370 to 930 spilled).  Splits rounded up to an even number
// took longer (us per call): bf16 47808 x 436, k = 2048 121 -> 113, half 7424 x 392, k = 3584 47.2 -> 45.6.
// REST (fp32, three pieces): the column tiles that the kernel of half pieces left.  They are scaled too: below 2^-110 an
// entry's third piece would lie under bf16's range.
template <typename T, int MT, int NRG, int NCG, bool HALF = false, bool ODD = false, bool REST = false>
__global__ __launch_bounds__(64 * NRG * NCG) __attribute__((amdgpu_waves_per_eu(MT > 2 || (MT == 2 && sizeof(T) == 4) ? 1 : 2)))
void gauss_kernel(GaussArgs a) {
  using V = typename Ld<T>::V;
  using P = std::conditional_t<HALF, f16, T>;  // type of the pieces (as mfma() names them)
  // DEEP (one wave per SIMD, many stages): two stages a pass, S tiles and operands fetched earlier, one barrier a stage where
  // it is not waited for.  Short calls of the small tiles are 1.1 to 1.2 times slower with it (its start, its code).
  constexpr bool DEEP = MT == 4;
  constexpr int PFD = Ld<T>::PFD;  // k-steps that the loads of A run ahead
  constexpr int PARTS = sizeof(T) == 4 ? (HALF ? 2 : 3) : 1;
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
  // Which (rows, columns, split) this work-group takes: linear ids are dealt round-robin over the 8 XCDs; renumbered, an
  // XCD's work-groups are consecutive, and consecutive ones share a split and few column tiles (a.cgroup), so that what
  // they read of A and of S they read from one L2.
  uint32_t bx = blockIdx.x, by = blockIdx.y, bz = blockIdx.z;
  if constexpr (DEEP) {  // (the divisions would be a good part of a short call)
    const uint32_t gx = gridDim.x, gy = gridDim.y, total = gx * gy * gridDim.z;
    const uint32_t id = blockIdx.x + gx * (blockIdx.y + gy * blockIdx.z);
    const uint32_t q = total / 8, r = total % 8;
    uint32_t nid = (id % 8) * q + min(id % 8, r) + id / 8;
    const uint32_t C = (uint32_t)a.cgroup;
    by = nid % C; nid /= C;
    bx = nid % gx; nid /= gx;
    by += nid % (gy / C) * C;
    bz = nid / (gy / C);
  }
  const int col0 = (int)by * (WCOLS * NCG) + cg * WCOLS + 4 * (lane & 31);
  const int64_t row_base = (int64_t)bx * RW;
  const int t0 = (int)bz * a.stages;
  const int mine = min(a.stages, a.total - t0);  // >= 1
  // DEEP: odd or even as a.stages; a shorter last split may have one more, of zeros
  const int T_stages = !DEEP ? mine : ODD ? mine | 1 : (mine + 1) & ~1;
  const int64_t row_bytes = a.lda * (int64_t)sizeof(T);
  // A up to the split's last row is one buffer (offsets fit 32 bits: checked on the host), behind which loads give
  // zeros.  A lane whose columns all lie at or beyond n gets an offset outside its range; a vector that straddles n loads the row's own
  // padding too (or nothing, behind the last row), which feeds only columns that are never stored.
  const uint32_t voff = col0 < a.n ? (uint32_t)(((int64_t)(kg * 8) * a.lda + col0) * (int64_t)sizeof(T)) : 0x80000000u;
  const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<void*>(a.A), 0, (int)(((int64_t)(t0 + mine) * KC - 1) * row_bytes + ((a.n + 3) & ~3) * (int64_t)sizeof(T)), 0x00020000);

  f32x16 acc[MT][4];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[mt][c][i] = 0.f;

  if constexpr (REST) {
    if (!a.few[by]) return;  // (uniform)
  }
  // SCALE: the power of two that takes the largest entry of each of the lane's columns to [2^14, 2^15), or as near as
  // the exponents of a float go (columns of subnormals); 1 for columns with an infinity or a NaN
  constexpr bool SCALE = HALF || REST;
  float colm[4];
  if constexpr (SCALE) {
    // The rows of maxima and sums, dealt to the 2*NRG half-waves of a column group, then through LDS: a chain of a few loads
    // in front of the first product (all 64 rows by every lane took 3 to 6 us).
    constexpr int SHARES = 2 * NRG, UN = NCG == 4 ? 16 : 8;  // loads in flight (past the end the last one again)
    uint4* s_m = reinterpret_cast<uint4*>(smem);              // [NCG][SHARES][32]
    float4* s_f = reinterpret_cast<float4*>(s_m + NCG * SHARES * 32);
    int* vote = reinterpret_cast<int*>(s_f + NCG * SHARES * 32);
    uint4 m = make_uint4(0, 0, 0, 0);
    float4 f = make_float4(0.f, 0.f, 0.f, 0.f);
    if (col0 < a.n) {  // (n is rounded up to 4 in the rows)
      for (int i = 2 * rg + kg; i < a.parts; i += UN * SHARES) {
        uint4 v[UN];
        float4 w[UN];
#pragma unroll
        for (int j = 0; j < UN; ++j) {
          const int64_t at = (int64_t)min(i + j * SHARES, a.parts - 1) * a.ldw + col0;
          v[j] = *reinterpret_cast<const uint4*>(a.colmax + at);
          if constexpr (HALF) w[j] = *reinterpret_cast<const float4*>(a.colsum + at);
        }
#pragma unroll
        for (int j = 0; j < UN; ++j) {
          m.x = max(m.x, v[j].x); m.y = max(m.y, v[j].y); m.z = max(m.z, v[j].z); m.w = max(m.w, v[j].w);
          if (HALF && i + j * SHARES < a.parts) { f.x += w[j].x; f.y += w[j].y; f.z += w[j].z; f.w += w[j].w; }
        }
      }
    }
    s_m[(cg * SHARES + 2 * rg + kg) * 32 + (lane & 31)] = m;
    if constexpr (HALF) s_f[(cg * SHARES + 2 * rg + kg) * 32 + (lane & 31)] = f;
    __syncthreads();
    m = make_uint4(0, 0, 0, 0);
    f = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int h = 0; h < SHARES; ++h) {
      const uint4 v = s_m[(cg * SHARES + h) * 32 + (lane & 31)];
      m.x = max(m.x, v.x); m.y = max(m.y, v.y); m.z = max(m.z, v.z); m.w = max(m.w, v.w);
      if constexpr (HALF) {
        const float4 w = s_f[(cg * SHARES + h) * 32 + (lane & 31)];
        f.x += w.x; f.y += w.y; f.z += w.z; f.w += w.w;
      }
    }
    const uint32_t mx[4] = {m.x, m.y, m.z, m.w};
    const float sum[4] = {f.x, f.y, f.z, f.w};
    bool few = false;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const uint32_t e = mx[c] >> 23;
      colm[c] = __uint_as_float((e == 255 ? 127u : min(268u - e, 254u)) << 23);
      // (less what d zeros add; a column of zeros alone has terms enough, one with an infinity or a NaN has not)
      if (col0 + c < a.n && mx[c]) few |= e == 255 || sum[c] - (float)a.d * kRoot0 < a.terms * root4(mx[c]);
    }
    if constexpr (HALF) {
      const bool wave_few = __any(few);
      if (lane == 0) vote[wave] = wave_few;
      __syncthreads();
      bool tile_few = false;
#pragma unroll
      for (int w = 0; w < NW; ++w) tile_few |= vote[w] != 0;
      if (bx == 0 && bz == 0 && tid == 0) a.few[by] = tile_few;
      if (tile_few) return;  // (uniform)
    }
    __syncthreads();  // (all of this lies where tiles of S will)
  }

  typedef uint32_t u4 __attribute__((ext_vector_type(4)));  // (an array of uint4 lands in scratch memory here)
  // S tiles on their way: SA stages are between the fetch of one and its place in LDS (tile t in sreg[t % SA])
  constexpr int SA = DEEP && sizeof(T) == 2 ? 2 : 1;
  u4 sreg[SA][PARTS * SREG];
  const int64_t s_first = ((int64_t)bx * a.total + t0) * (RW * KC) + tid * 8;
  auto s_fetch = [&](int t, u4 (&dst)[PARTS * SREG]) {
    if constexpr (DEEP) t = min(t, mine - 1);  // (behind the last tile, for zeros of A or not used)
#pragma unroll
    for (int pt = 0; pt < PARTS; ++pt)
#pragma unroll
      for (int i = 0; i < SREG; ++i)
        dst[pt * SREG + i] = *reinterpret_cast<const u4*>((pt == 0 ? a.S[0] : pt == 1 ? a.S[1] : a.S[2]) + s_first + (int64_t)t * (RW * KC) + i * NT * 8);
  };
  auto s_store = [&](int buf, u4 (&src)[PARTS * SREG]) {
#pragma unroll
    for (int pt = 0; pt < PARTS; ++pt)
#pragma unroll
      for (int i = 0; i < SREG; ++i) {
        const int e = tid + i * NT, row = e >> 3, c16 = e & 7;
        *reinterpret_cast<u4*>(s_tile + (buf * PARTS + pt) * TILE + row * PHI_LD + c16 * 8) = src[pt * SREG + i];
      }
  };
  auto lds_barrier = [&]() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
  };

  V ld[PFD][8];
  auto issue = [&](int kk, V (&dst)[8]) {
    if constexpr (DEEP) kk = min(kk, mine * KSTEPS);  // (16 rows behind the last one read zeros; offsets of more could wrap)
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const uint32_t soj = (uint32_t)((t0 * KSTEPS + kk) * 16 + j) * (uint32_t)row_bytes;
      if constexpr (sizeof(T) == 2)
        dst[j] = __builtin_bit_cast(V, __builtin_amdgcn_raw_buffer_load_b64(rs, voff, soj, 0));
      else
        dst[j] = __builtin_bit_cast(V, __builtin_amdgcn_raw_buffer_load_b128(rs, voff, soj, 0));
    }
  };

  // S operands of a k-step.  AHEAD: read one k-step before they are used (three pieces of a 128-row tile leave no registers for it).
  constexpr bool AHEAD = DEEP && PARTS <= 2;
  uint4 pa2[AHEAD ? 2 : 1][PARTS][MT];
  auto read_pa = [&](const uint16_t* tile, int ks, uint4 (&pa)[PARTS][MT]) {
#pragma unroll
    for (int pt = 0; pt < PARTS; ++pt)
#pragma unroll
      for (int mt = 0; mt < MT; ++mt)
        pa[pt][mt] = *reinterpret_cast<const uint4*>(
            tile + pt * TILE + ((rg * MT + mt) * 32 + (lane & 31)) * PHI_LD + ks * 16 + kg * 8);
  };

  // One stage; DEEP: t % 2 == PAR.  Tile t+1 is written behind its third k-step (DEEP) or its last into the buffer that held tile
  // t-1, and one barrier behind that, when this wave has read its last operands of tile t, gives it free.
  auto stage = [&](int t, auto par_tag, auto last_tag) {
    constexpr int PAR = decltype(par_tag)::value;
    constexpr bool LAST = decltype(last_tag)::value;
    const int buf = DEEP ? PAR : t & 1;
    const uint16_t* tile = s_tile + buf * PARTS * TILE;
    const uint16_t* next = s_tile + (1 - buf) * PARTS * TILE;
    if constexpr (!LAST && SA == 1) s_fetch(t + 1, sreg[0]);
#pragma unroll
    for (int ks = 0; ks < KSTEPS; ++ks) {
      uint4(&pa)[PARTS][MT] = pa2[AHEAD ? ks & 1 : 0];
      if constexpr (!AHEAD) read_pa(tile, ks, pa);
      else if (ks + 1 < KSTEPS) read_pa(tile, ks + 1, pa2[(ks + 1) & 1]);
      else if constexpr (!LAST) read_pa(next, 0, pa2[0]);
      V(&cur)[8] = ld[(PAR * KSTEPS + ks) % PFD];
      const bool fetch = !LAST || ks + PFD < KSTEPS;  // (behind the last row they read zeros)
      if constexpr (sizeof(T) == 2) {
        uint4 op[4];
        make_ops(cur, op);
        if (fetch) issue(t * KSTEPS + ks + PFD, cur);
#pragma unroll
        for (int c = 0; c < 4; ++c)
#pragma unroll
          for (int mt = 0; mt < MT; ++mt) acc[mt][c] = mfma<T>(pa[0][mt], op[c], acc[mt][c]);
      } else {
        // product by product over the row tiles: with MT = 4 an accumulator is reused only after three other MFMAs
        // (back-to-back dependent MFMAs stall the matrix pipe); smaller tiles of half pieces take two columns together
        constexpr int CG = HALF && MT < 4 ? 2 : 1;
#pragma unroll
        for (int c0 = 0; c0 < 4; c0 += CG) {
          uint4 x[CG][PARTS];
#pragma unroll
          for (int c = 0; c < CG; ++c) {
            uint32_t xs[8];
#pragma unroll
            for (int j = 0; j < 8; ++j)
              xs[j] = c0 + c == 0 ? cur[j].x : c0 + c == 1 ? cur[j].y : c0 + c == 2 ? cur[j].z : cur[j].w;
            if constexpr (REST) {  // exact, or far below what the column's largest entry leaves of fp32
#pragma unroll
              for (int j = 0; j < 8; ++j) xs[j] = __float_as_uint(__uint_as_float(xs[j]) * colm[c0 + c]);
            }
            if constexpr (HALF) split_half(xs, colm[c0 + c], x[c][0], x[c][1]);
            else split_ops(xs, x[c][0], x[c][1], x[c][PARTS - 1]);
          }
          auto product = [&](auto ps, auto px) {
#pragma unroll
            for (int c = 0; c < CG; ++c)
#pragma unroll
              for (int mt = 0; mt < MT; ++mt)
                acc[mt][c0 + c] = mfma<P>(pa[decltype(ps)::value][mt], x[c][decltype(px)::value], acc[mt][c0 + c]);
          };
          using I0 = std::integral_constant<int, 0>;
          using I1 = std::integral_constant<int, 1>;
          using I2 = std::integral_constant<int, PARTS - 1>;
          product(I0{}, I0{});
          product(I0{}, I1{});
          product(I1{}, I0{});
          if constexpr (!HALF) {
            product(I0{}, I2{});
            product(I2{}, I0{});
            product(I1{}, I1{});
          }
        }
        if (fetch) issue(t * KSTEPS + ks + PFD, cur);
      }
      if constexpr (!LAST) {
        if (ks == (DEEP ? KSTEPS - 2 : KSTEPS - 1)) {
          s_store(1 - buf, sreg[(1 - PAR) % SA]);
          if constexpr (SA == 2) s_fetch(t + 3, sreg[1 - PAR]);
        }
      }
      if constexpr (AHEAD) {  // one wave per SIMD: everything else between the MFMAs
        constexpr int NM = 4 * MT * (HALF ? 3 : 1);
#pragma unroll
        for (int i = 0; i < NM; ++i) {
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
          __builtin_amdgcn_sched_group_barrier(0x002, 3, 0);
          __builtin_amdgcn_sched_group_barrier(0x090, 1, 0);
        }
      }
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (!LAST) {
        if (ks == (AHEAD ? KSTEPS - 2 : KSTEPS - 1)) lds_barrier();
      }
    }
  };

#pragma unroll
  for (int i = 0; i < PFD; ++i) issue(i, ld[i]);
  s_fetch(0, sreg[0]);
  if constexpr (SA == 2) s_fetch(1, sreg[1]);
  s_store(0, sreg[0]);
  if constexpr (SA == 2) s_fetch(2, sreg[0]);
  lds_barrier();
  if constexpr (AHEAD) read_pa(s_tile, 0, pa2[0]);
  using P0 = std::integral_constant<int, 0>;
  using P1 = std::integral_constant<int, 1>;
  if constexpr (DEEP) {
    for (int t = 0; t + 2 < T_stages; t += 2) {
      stage(t, P0{}, std::false_type{});
      stage(t + 1, P1{}, std::false_type{});
    }
    if constexpr (ODD) {
      stage(T_stages - 1, P0{}, std::true_type{});
    } else {
      stage(T_stages - 2, P0{}, std::false_type{});
      stage(T_stages - 1, P1{}, std::true_type{});
    }
  } else {
    for (int t = 0; t + 1 < T_stages; ++t) stage(t, P0{}, std::false_type{});
    stage(T_stages - 1, P0{}, std::true_type{});
  }

  if (col0 >= a.n) return;
  int unscale[4];
  if constexpr (SCALE) {
#pragma unroll
    for (int c = 0; c < 4; ++c) unscale[c] = 127 - (int)(__float_as_uint(colm[c]) >> 23) - (HALF ? a.es : 0);
  }
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) {
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int64_t row = row_base + (rg * MT + mt) * 32 + 8 * (i >> 2) + 4 * kg + (i & 3);
      float v[4] = {acc[mt][0][i], acc[mt][1][i], acc[mt][2][i], acc[mt][3][i]};
      if constexpr (SCALE) {
#pragma unroll
        for (int c = 0; c < 4; ++c) v[c] = ldexpf(v[c], unscale[c]);
      }
      if (a.zsplit > 1) {  // a partial sum: plane bz (col0 + 3 < ldw)
        *reinterpret_cast<float4*>(a.ws + ((int64_t)bz * a.k + row) * a.ldw + col0) = make_float4(v[0], v[1], v[2], v[3]);
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

// half: fp32 on two half pieces; the maxima and sums of its columns, in up to 64 shares of the rows, and a word per column
// tile have kColmaxRoom bytes in front of the planes.
struct GaussPlan { int ncg = 4, zsplit = 1, stages = 1; bool half = false; double us = 0; };
constexpr size_t kColmaxRoom = (size_t)4 << 20;
int64_t colmax_parts(int64_t ldw) {
  const int64_t p = ((int64_t)kColmaxRoom - 4 * (ldw / 128 + 1)) / (ldw * 8);
  return p > 64 ? 64 : p;
}

// Terms from which on a column is summed as well from two half pieces as from three: three hold it exactly, so that what
// counts there is only how many of its additions are rounded; of a column of few terms hardly any.  A term counts by the
// fourth root of its share of the largest (2^-20 of it as 1/32: such terms are still rounded when they are added).  Error
// against 64 bits, two pieces / three, for m terms of random sign and place: of magnitude 1 1.77 (m = 2), 1.14 (16), 1.05 (128), 1.01
// (512) at 65536 x 512, k = 4096 with 8 splits of d, 1.10 (64), 1.05 (256), 1.03 (1024) at 32768 x 300, k = 512 with 64 splits, which are
// each summed apart; normal ones 1.08 (1), 0.94 (32), 0.80 (256) and 1.14, 1.04, 0.95; one term of magnitude 1 among 65536 of 2^-20 0.91, of
// 2^-26 1.00.  (A dense column of normal entries has 0.6 d.)
constexpr int gauss_terms(int zsplit) { return 256 + 16 * zsplit; }

// LDS of a work-group: two stages of the pieces of S.
size_t gauss_lds(fs_dtype dt, bool half) { return (size_t)2 * (half ? 2 : dt == FS_F32 ? 3 : 1) * 128 * PHI_LD * 2; }

// Columns per work-group (128, 256 or 512) and splits of the d/64 stages.  128-column waves that own all 128
// rows (512 columns per work-group) do the most matrix work per loaded element; fewer columns leave
// waves without any, so narrower work-groups divide the rows among the waves instead.  The smallest
// modelled time: rounds of resident work-groups (two on a CU take 1.7 times as long as one) times stages, plus the planes
// (written at 3.4, read at 6 TB/s, half that price while they stay in the Infinity Cache) and the reduction's launch.  The
// rates are a fit to the timed plans of 60 shapes (to 8 %; what it takes of the fp32 ones is slower than the best by 0.8 % in
// the geometric mean, 7 % at most).
GaussPlan gauss_plan(int64_t k, int64_t d, int64_t n, fs_dtype dt, size_t scratch, bool half) {
  GaussPlan pl;
  pl.half = half;
  const int total = (int)(d / KC);
  const double plane = (double)k * (double)((n + 3) & ~(int64_t)3) * 4.0;
  double best = 0;
  for (int ncg = 4; ncg >= 1; ncg /= 2) {
    const int64_t wgs = (k / 128) * ((n + 128 * ncg - 1) / (128 * ncg));
    // us per stage of a work-group that has its CU to itself
    const double stage_us = half           ? (ncg == 4 ? 3.8 : ncg == 2 ? 2.6 : 1.87)
                            : dt == FS_F32 ? (ncg == 4 ? 7.0 : ncg == 2 ? 4.4 : 3.28)
                                           : (ncg == 4 ? 1.75 : ncg == 2 ? 1.3 : 0.9);
    // (one wave per SIMD: one; else what the LDS holds, which with three pieces is one too: us per call of a handle without
    // half pieces, priced as two -> as one: 17664 x 52, k = 1280 52.2 -> 48.4; of 40 such calls 10 0.93 to 0.98 times, one 1.03)
    const int per_cu = ncg == 4 || (ncg == 2 && dt == FS_F32) || 2 * gauss_lds(dt, half) > kLdsMost ? 1 : 2;
    for (int z = 1, st; z <= total && z <= 128; z = st > 1 ? (total + st - 2) / (st - 1) : total + 1) {
      st = (total + z - 1) / z;
      if ((total + st - 1) / st != z) continue;
      if (z > 1 && plane * z > (double)scratch) break;
      const double w = (double)wgs * z, rounds = per_cu == 2 && w > 256 ? 1.7 * ceil(w / 512) : ceil(w / 256);
      double t = rounds * (st * stage_us + (dt == FS_F32 ? 4.4 : 3.0));
      if (z > 1) t += 4.0 + plane * z * (1 / 3.4e6 + 1 / 6e6) * (plane * z < 40e6 ? 0.5 : 1.0);
      if ((ncg == 4 && z == 1) || t < 0.98 * best) { best = t; pl.ncg = ncg; pl.zsplit = z; pl.stages = st; }
    }
  }
  pl.us = best + (half ? 10.0 + (double)d * (double)n * 4.0 / 4.5e6 : 0.0);
  return pl;
}

// fp32: two half pieces of both operands are three products where three bf16 pieces are six, behind a pass over A for what
// each column needs and before a launch that finds nothing to do unless a tile was left.  Small calls cannot win back the two
// launches and the read (us, six products against three: 4416 x 64, k = 3840 40.2 / 38.7; 12672 x 36, k = 1152 34.7 / 35.0; 4992 x 152,
// k = 2816 53.2 / 48.1; 57856 x 208, k = 640 117 / 94; 65536 x 1024, k = 4096 2283 / 1394).  Error against 64 bits: 4416 x 64 3.8e-7 / 2.8e-7,
// 57856 x 208 6.7e-7 / 4.4e-7, 65536 x 1024 2.7e-6 / 1.6e-6, 0.45 to 0.76 times in 60 random calls (half as many additions are
// rounded, each by more than the pieces leave out).
GaussPlan gauss_choose(int64_t k, int64_t d, int64_t n, fs_dtype dt, size_t scratch, bool pieces) {
  GaussPlan pl = gauss_plan(k, d, n, dt, scratch, false);
  if (dt == FS_F32 && pieces && colmax_parts((n + 3) & ~(int64_t)3) > 0) {
    const GaussPlan h = gauss_plan(k, d, n, dt, scratch, true);
    if (h.us < 0.95 * pl.us && d >= 4 * gauss_terms(h.zsplit)) pl = h;  // (where a dense column has the terms)
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
// The two half pieces and the room of the column maxima, behind them.
size_t gauss_half_bytes(int64_t k, int64_t d) { return (((size_t)k * (size_t)d * 4 + 255) & ~(size_t)255) + kColmaxRoom; }

namespace {
// S is scaled by 2^es before it is cut into half pieces: no entry is above 5.77 / sqrt(k) (24-bit Box-Muller), so the
// largest come to lie between 2^13 and 2^15.
int half_exponent(int64_t k) {
  int e = 0;
  while ((k >> (2 * e + 2)) > 0) ++e;  // floor(log2(k) / 2)
  return 12 + e;
}
}  // namespace

hipError_t gauss_fill(void* storage, bool half, int64_t k, int64_t d, uint32_t key1, hipStream_t st) {
  float* S32 = (float*)storage;
  uint16_t* b = (uint16_t*)(S32 + k * d);
  const int64_t blocks = (k * d + 255) / 256;
  if (blocks > 0x7fffffff) return hipErrorInvalidValue;
  const int tiled = d % KC == 0 && k % 128 == 0;
  f16* h = half ? (f16*)((char*)storage + gauss_bytes(k, d)) : nullptr;
  hipLaunchKernelGGL(gauss_fill_kernel, dim3((unsigned)blocks), dim3(256), 0, st, S32, b, b + k * d,
                     b + 2 * k * d, b + 3 * k * d, b + 4 * k * d, h, half ? h + k * d : nullptr, half_exponent(k), k, d,
                     key1, tiled, sqrt((double)k));
  return hipGetLastError();
}

bool gauss_supported(int64_t k, int64_t d, const void* A, int64_t lda, int64_t n, fs_dtype dt) {
  const int64_t esz = dt == FS_F32 ? 4 : 2;
  if (d % KC || k % 128 || n < 1) return false;
  if ((uintptr_t)A % (4 * esz) || lda % 4) return false;
  if (d * lda * esz >= ((int64_t)1 << 31)) return false;  // 32-bit buffer offsets over all of A
  return (n + 255) / 256 <= 65535;
}

hipError_t launch_gauss(void* storage, bool half, size_t scratch, int64_t k, int64_t d, const void* A, int64_t lda,
                        int64_t n, void* out, int64_t ldo, fs_dtype dt, hipStream_t st, EventPair ev, char* desc,
                        size_t desc_cap) {
  const float* S32 = (const float*)storage;
  const uint16_t* b = (const uint16_t*)(S32 + k * d);
  const size_t esz = dt == FS_F32 ? 4 : 2;
  const GaussPlan pl = gauss_choose(k, d, n, dt, scratch, half);
  if (desc && desc_cap)  // (a column tile with a column of few terms: by its counterpart on three pieces)
    snprintf(desc, desc_cap, "gauss_kernel<%s,%d,%d,%d,%s,%s>%s", dt == FS_F32 ? "f32" : dt == FS_BF16 ? "bf16" : "f16", pl.ncg,
             4 / pl.ncg, pl.ncg, pl.half ? "half" : "-", pl.ncg == 4 && pl.stages % 2 ? "odd" : "-",
             pl.zsplit > 1 ? "+reduce_planes" : "");
  GaussArgs a;
  a.A = A; a.out = out; a.k = k; a.d = d; a.lda = lda; a.ldo = ldo; a.n = (int)n;
  a.total = (int)(d / KC); a.stages = pl.stages; a.zsplit = pl.zsplit;
  a.ldw = (n + 3) & ~(int64_t)3;
  a.ws = (float*)((char*)storage + gauss_bytes(k, d) + (half ? gauss_half_bytes(k, d) : 0));
  a.out_vec = ((uintptr_t)out % (4 * esz) == 0 && (ldo * esz) % (4 * esz) == 0) ? 1 : 0;
  a.S[1] = a.S[2] = nullptr;
  a.colmax = nullptr; a.colsum = nullptr; a.few = nullptr; a.parts = 0; a.es = half_exponent(k);
  a.terms = (float)gauss_terms(pl.zsplit);
  if (ev.start) (void)hipEventRecord(ev.start, st);  // (both passes over A lie between the events)
  if (pl.half) {
    a.S[0] = (const uint16_t*)((char*)storage + gauss_bytes(k, d));
    a.S[1] = a.S[0] + k * d;
    const int sh = n > 512 ? 6 : n > 256 ? 5 : n > 128 ? 4 : 3;  // (three tiles or more: 64 work-groups do not read at the full rate)
    const int64_t tiles = (n + (4 << sh) - 1) / (4 << sh);
    int64_t parts = (256 + tiles - 1) / tiles;  // about 4096 waves
    parts = parts > colmax_parts(a.ldw) ? colmax_parts(a.ldw) : parts;
    uint32_t* maxima = (uint32_t*)((char*)a.ws - kColmaxRoom);
    a.colmax = maxima;
    const int64_t rows = (d + parts - 1) / parts;
    a.parts = (int)((d + rows - 1) / rows);
    float* sums = (float*)(maxima + a.parts * a.ldw);
    a.colsum = sums;
    a.few = (int*)(sums + a.parts * a.ldw);
    hipLaunchKernelGGL(gauss_colmax_kernel, dim3((unsigned)tiles, (unsigned)a.parts), dim3(1024), 0, st, (const float*)A, d,
                       lda, (int)n, rows, sh, maxima, sums, a.ldw);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  } else if (dt == FS_F32) { a.S[0] = b + k * d; a.S[1] = b + 2 * k * d; a.S[2] = b + 3 * k * d; }
  else a.S[0] = dt == FS_BF16 ? b : b + 4 * k * d;
  const dim3 grid((unsigned)(k / 128), (unsigned)((n + 128 * pl.ncg - 1) / (128 * pl.ncg)), (unsigned)pl.zsplit);
  a.cgroup = 1;
  while (2 * a.cgroup * 128 * pl.ncg <= 1024 && grid.y % (2 * a.cgroup) == 0) a.cgroup *= 2;
  hipError_t e;
#define FS_G(T, H, R)                                                                                               \
  (pl.ncg == 4   ? pl.stages % 2 ? go(gauss_kernel<T, 4, 1, 4, H, true, R>, grid, 256, gauss_lds(dt, H), st, a)     \
                                 : go(gauss_kernel<T, 4, 1, 4, H, false, R>, grid, 256, gauss_lds(dt, H), st, a)    \
   : pl.ncg == 2 ? go(gauss_kernel<T, 2, 2, 2, H, false, R>, grid, 256, gauss_lds(dt, H), st, a)                    \
                 : go(gauss_kernel<T, 1, 4, 1, H, false, R>, grid, 256, gauss_lds(dt, H), st, a))
  if (pl.half) {
    e = FS_G(float, true, false);
    if (e == hipSuccess) {  // the column tiles that it left, into the same planes
      a.S[0] = b + k * d; a.S[1] = b + 2 * k * d; a.S[2] = b + 3 * k * d;
      e = FS_G(float, false, true);
    }
  } else {
    e = dt == FS_F32    ? FS_G(float, false, false)
        : dt == FS_BF16 ? FS_G(uint16_t, false, false)
                        : FS_G(f16, false, false);
  }
#undef FS_G
  if (ev.stop) (void)hipEventRecord(ev.stop, st);
  if (e != hipSuccess || pl.zsplit == 1) return e;
#define FS_R(T) launch_reduce_planes<T>(a.ws, pl.zsplit, k, a.ldw, n, out, ldo, 1.0f, 1, nullptr, 1, 1, st)
  return dt == FS_F32 ? FS_R(float) : dt == FS_BF16 ? FS_R(uint16_t) : FS_R(f16);
#undef FS_R
}

}  // namespace fs
