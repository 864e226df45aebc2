// Shape-generic GEMM with the fused epilogues: any M, N, K (N even), fp32 or bf16 operands, fp32
// accumulation on the vector ALU.  It serves the fp32 configuration and every shape the MFMA
// family does not cover.
#include "pt_epilogue.h"

#define GG_BK 32

__device__ __forceinline__ void pair_columns(const pt_gemm_args& g, int p, int* n0, int* n1) {
  if (g.epi == EPI_SWIGLU) {
    *n0 = swiglu_gate_row(p);
    *n1 = *n0 + 32;
  } else if (g.epi == EPI_QKV) {
    const int half = g.hd >> 1, rot_pairs = (g.H + g.Hkv) * half;
    if (p < rot_pairs) {
      const int head = p / half, j = p - head * half;
      *n0 = head * g.hd + j;
      *n1 = *n0 + half;
    } else {
      *n0 = (g.H + g.Hkv) * g.hd + 2 * (p - rot_pairs);
      *n1 = *n0 + 1;
    }
  } else {
    *n0 = 2 * p;
    *n1 = 2 * p + 1;
  }
}

template <typename T>
__global__ void __launch_bounds__(256) gemm_generic_kernel(pt_gemm_args g) {
  __shared__ float As[16][GG_BK + 1];
  __shared__ float W0s[16][GG_BK + 1];
  __shared__ float W1s[16][GG_BK + 1];
  const int tx = threadIdx.x & 15, ty = threadIdx.x >> 4;
  const int b = blockIdx.z;
  const int m0 = blockIdx.y * 16, p0 = blockIdx.x * 16;
  const int npairs = g.N >> 1;
  const T* A = (const T*)g.A + b * g.a_bstride;
  const T* W = (const T*)g.W + b * g.w_bstride;
  if (g.blk_group) {   // grouped GEMM: weight matrix by 64-row block; blocks without rows are skipped
    const int group = g.blk_group[b * g.grp_bstride + (m0 >> 6)];
    if (group < 0) return;
    W += group * g.w_gstride;
  }
  // row of A behind tile row ty (a gather when a_rows is given)
  const int64_t arow = m0 + ty < g.M ? (g.a_rows ? g.a_rows[b * g.a_rows_bstride + m0 + ty] : m0 + ty) : 0;

  // the W rows this block needs, one pair per tile row
  int ln0 = 0, ln1 = 0;
  {
    const int p = p0 + ty;
    if (p < npairs) pair_columns(g, p, &ln0, &ln1);
  }
  float acc0 = 0.f, acc1 = 0.f;
  for (int k0 = 0; k0 < g.K; k0 += GG_BK) {
    for (int e = tx; e < GG_BK; e += 16) {
      const int k = k0 + e;
      const bool kin = k < g.K;
      As[ty][e] = (kin && m0 + ty < g.M) ? elem<T>::ld(A + arow * g.lda + k) : 0.f;
      const bool pin = kin && (p0 + ty) < npairs;
      W0s[ty][e] = pin ? elem<T>::ld(W + (int64_t)ln0 * g.ldb + k) : 0.f;
      W1s[ty][e] = pin ? elem<T>::ld(W + (int64_t)ln1 * g.ldb + k) : 0.f;
    }
    __syncthreads();
#pragma unroll
    for (int e = 0; e < GG_BK; ++e) {
      const float a = As[ty][e];
      acc0 = fmaf(a, W0s[tx][e], acc0);
      acc1 = fmaf(a, W1s[tx][e], acc1);
    }
    __syncthreads();
  }
  const int m = m0 + ty, p = p0 + tx;
  if (m >= g.M || p >= npairs) return;
  int n0, n1;
  pair_columns(g, p, &n0, &n1);
  switch (g.epi) {
    case EPI_STORE_F32:
      epi_store_f32<T>(g, b, m, n0, acc0);
      epi_store_f32<T>(g, b, m, n1, acc1);
      break;
    case EPI_RESIDUAL:
      epi_residual<T>(g, b, m, n0, acc0);
      epi_residual<T>(g, b, m, n1, acc1);
      break;
    case EPI_SWIGLU:
      epi_swiglu<T>(g, b, m, p, acc0, acc1);
      break;
    case EPI_QKV:
      if (n0 < (g.H + g.Hkv) * g.hd) {
        epi_rope_pair<T>(g, b, m, n0, acc0, acc1, epi_rope_entry(g, m, n0));
      } else {
        epi_v<T>(g, b, m, n0, acc0);
        epi_v<T>(g, b, m, n1, acc1);
      }
      break;
  }
}

// Sum over the 64 lanes, in every lane: prefix sums inside rows of 16 lanes, carried from row to row (no LDS).
__device__ __forceinline__ float wave_sum_dpp(float x) {
#define PT_DPP_ADD(ctrl, rows) \
  x += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), ctrl, rows, 0xf, false))
  PT_DPP_ADD(0x111, 0xf);   // row_shr:1
  PT_DPP_ADD(0x112, 0xf);   // row_shr:2
  PT_DPP_ADD(0x114, 0xf);   // row_shr:4
  PT_DPP_ADD(0x118, 0xf);   // row_shr:8
  PT_DPP_ADD(0x142, 0xa);   // row_bcast:15 into rows 1 and 3
  PT_DPP_ADD(0x143, 0xc);   // row_bcast:31 into rows 2 and 3
#undef PT_DPP_ADD
  return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, x), 63));
}

// fp32, few rows: one wavefront per pair of output columns and MR rows, lanes along K.  What bounds these launches is
// latency: the kernel above walks K in steps of 32 with two barriers each, about 1.1 us a step; here all loads of
// 256 elements of K are in flight at once and the lanes are folded at the end.  One row of the Tiny model, event to
// event with 6.3 us of overhead, K = 128 / 512: 9.5 / 24.5 us before, 6.4 / 6.4 now; fp32 at 4 tracks, width 1024: QKV, out,
// gate/up, down 63 / 52 / 84 / 188 us before, 15 / 8 / 27 / 18 now.
// NORM: the operand is RMSNorm(norm_src) * norm_gain, formed on the way (the row's 1/rms multiplies the finished sums),
// which saves the launch in front.  What the epilogue reads (residual values, rotary table) is loaded ahead of the sums.
template <int MR, bool NORM>
__global__ void __launch_bounds__(256) gemm_rows_kernel(pt_gemm_args g) {
  const int lane = threadIdx.x & 63;
  const int p = blockIdx.x * 4 + (threadIdx.x >> 6), m0 = blockIdx.y * MR, b = blockIdx.z;
  if (p >= g.N >> 1) return;
  int n0, n1;
  pair_columns(g, p, &n0, &n1);
  const float* w0p = (const float*)g.W + b * g.w_bstride + (int64_t)n0 * g.ldb;
  const float* w1p = (const float*)g.W + b * g.w_bstride + (int64_t)n1 * g.ldb;
  const float* a_first = NORM ? g.norm_src + b * g.norm_bstride : (const float*)g.A + b * g.a_bstride;
  const float* gain = NORM ? g.norm_gain + b * g.norm_gbstride : nullptr;
  const float* ap[MR];
#pragma unroll
  for (int r = 0; r < MR; ++r) ap[r] = a_first + (int64_t)min(m0 + r, g.M - 1) * g.lda;
  const int m = m0 + lane;                           // lane r finishes row m0 + r
  const bool mine = lane < MR && m < g.M;
  const bool rotated = g.epi == EPI_QKV && n0 < (g.H + g.Hkv) * g.hd;
  float2 ahead = make_float2(0.f, 0.f);
  if (mine) {
    if (g.epi == EPI_RESIDUAL) {                      // n1 = n0 + 1; single loads: nothing promises their alignment
      const float* r = g.res + b * g.res_bstride + (int64_t)m * g.ldo + n0;
      ahead = make_float2(r[0], r[1]);
    } else if (rotated) {
      ahead = epi_rope_entry(g, m, n0);
    }
  }
  float acc0[MR], acc1[MR], ss[MR];
#pragma unroll
  for (int r = 0; r < MR; ++r) acc0[r] = acc1[r] = ss[r] = 0.f;
#pragma unroll 2
  for (int k = lane * 4; k < g.K; k += 256) {
    const float4 w0 = *(const float4*)(w0p + k), w1 = *(const float4*)(w1p + k);
    float4 gn = make_float4(1.f, 1.f, 1.f, 1.f);
    if constexpr (NORM) gn = *(const float4*)(gain + k);
#pragma unroll
    for (int r = 0; r < MR; ++r) {
      float4 a = *(const float4*)(ap[r] + k);
      if constexpr (NORM) {
        ss[r] = fmaf(a.w, a.w, fmaf(a.z, a.z, fmaf(a.y, a.y, fmaf(a.x, a.x, ss[r]))));
        a.x *= gn.x; a.y *= gn.y; a.z *= gn.z; a.w *= gn.w;
      }
      acc0[r] = fmaf(a.w, w0.w, fmaf(a.z, w0.z, fmaf(a.y, w0.y, fmaf(a.x, w0.x, acc0[r]))));
      acc1[r] = fmaf(a.w, w1.w, fmaf(a.z, w1.z, fmaf(a.y, w1.y, fmaf(a.x, w1.x, acc1[r]))));
    }
  }
  float lo = 0.f, hi = 0.f;
#pragma unroll
  for (int r = 0; r < MR; ++r) {
    float s0 = wave_sum_dpp(acc0[r]), s1 = wave_sum_dpp(acc1[r]);
    if constexpr (NORM) {
      const float inv = 1.0f / sqrtf(wave_sum_dpp(ss[r]) / (float)g.K + g.norm_eps);
      s0 *= inv;
      s1 *= inv;
    }
    if (lane == r) { lo = s0; hi = s1; }
  }
  if (!mine) return;
  switch (g.epi) {
    case EPI_STORE_F32:
      epi_store_f32<float>(g, b, m, n0, lo);
      epi_store_f32<float>(g, b, m, n1, hi);
      break;
    case EPI_RESIDUAL:
      epi_store_f32<float>(g, b, m, n0, ahead.x + lo);
      epi_store_f32<float>(g, b, m, n1, ahead.y + hi);
      break;
    case EPI_SWIGLU:
      epi_swiglu<float>(g, b, m, p, lo, hi);
      break;
    case EPI_QKV:
      if (rotated) {
        epi_rope_pair<float>(g, b, m, n0, lo, hi, ahead);
      } else {
        epi_v<float>(g, b, m, n0, lo);
        epi_v<float>(g, b, m, n1, hi);
      }
      break;
  }
}

// Its work per workgroup (2 ns + K / 400 ns of the chip) grows with the rows, the other kernel's chain of K steps (44 ns
// per element of K) does not: Tiny with 192 rows (QKV, K = 128) 16.7 us against 11.4, with 32 rows 7.9 against 10.4;
// down (K = 512) with 192 rows 11 against 27.
static bool rows_covers(const pt_gemm_args& g) {
  const double wgs = (double)((g.N / 2 + 3) / 4) * ((g.M + 3) / 4) * g.batch;
  if (wgs * (2.0 + g.K / 400.0) >= 44.0 * g.K || g.M > 4 * 65535) return false;
  if (g.dtype != PT_F32 || g.blk_group || g.a_rows || ((g.K | g.lda | g.ldb) & 3) || (g.w_bstride & 3) || ((uintptr_t)g.W & 15)) return false;
  // the caller's hidden states may lie anywhere: rows of norm_src are read with loads that need 4-byte alignment only
  if (g.norm_src) return !(g.norm_gbstride & 3) && !((uintptr_t)g.norm_gain & 15);
  return !(g.a_bstride & 3) && !((uintptr_t)g.A & 15);
}

// The norm inside costs every wavefront of several rows about 0.3 ns of the chip, whatever K (sums of squares and their
// lane sums), the launch it saves 3.8 us.  QKV or gate/up, us with it / without: 4 tracks, width 1024, 4 rows QKV (6144
// wavefronts) 20.1 / 17.8, 8 rows (12288) 29.6 / 24.9, 4 rows gate/up (16384) 36.5 / 32.0; 1 x 1024, 8 rows gate/up (8192) 20.1 /
// 16.6; 2 x 2048, 8 rows QKV (12288) 46.3 / 42.0, 24 rows (36864) 95 / 82; a layer of the last 291 / 271.  One row: 27.5 / 27.1 at 16384.
bool pt_gemm_generic_fuses_norm(const pt_gemm_args& g) {
  return rows_covers(g) && g.epi != EPI_RESIDUAL && (g.M == 1 || (int64_t)(g.N / 2) * ((g.M + 3) / 4) * g.batch < 12288);
}

int pt_launch_gemm_generic(const pt_gemm_args& g, hipStream_t s) {
  if (g.M <= 0 || g.N <= 0 || g.batch <= 0) return PT_OK;
  if (g.N & 1) return pt_set_error(PT_ERR_INVALID_ARGUMENT, "generic GEMM needs an even N");
  if (rows_covers(g)) {
    const int mr = g.M == 1 ? 1 : 4;
    const dim3 rgrid((unsigned)((g.N / 2 + 3) / 4), (unsigned)((g.M + mr - 1) / mr), (unsigned)g.batch);
    if (mr == 1 && g.norm_src)
      hipLaunchKernelGGL((gemm_rows_kernel<1, true>), rgrid, dim3(256), 0, s, g);
    else if (mr == 1)
      hipLaunchKernelGGL((gemm_rows_kernel<1, false>), rgrid, dim3(256), 0, s, g);
    else if (g.norm_src)
      hipLaunchKernelGGL((gemm_rows_kernel<4, true>), rgrid, dim3(256), 0, s, g);
    else
      hipLaunchKernelGGL((gemm_rows_kernel<4, false>), rgrid, dim3(256), 0, s, g);
    PT_HIP_CHECK(hipGetLastError());
    return PT_OK;
  }
  if (g.norm_src) return pt_set_error(PT_ERR_HIP, "a GEMM that was to form its own normalised operand was not taken by that kernel");
  dim3 grid((unsigned)((g.N / 2 + 15) / 16), (unsigned)((g.M + 15) / 16), (unsigned)g.batch);
  if (grid.y > 65535u) return pt_set_error(PT_ERR_INVALID_ARGUMENT, "generic GEMM: M too large");
  if (g.dtype == PT_F32)
    hipLaunchKernelGGL(gemm_generic_kernel<float>, grid, dim3(256), 0, s, g);
  else
    hipLaunchKernelGGL(gemm_generic_kernel<bf16_t>, grid, dim3(256), 0, s, g);
  PT_HIP_CHECK(hipGetLastError());
  return PT_OK;
}
