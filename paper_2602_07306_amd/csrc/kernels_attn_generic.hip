// Shape-generic causal attention over the KV cache (prefill and decode), one wavefront per
// (query row, head): online softmax over chunks of 64 keys, fp32 arithmetic on the vector ALU.
// Serves the fp32 configuration and the shapes the tuned attention kernels do not cover.
#include "pt_device.h"

__device__ __forceinline__ float4 load4(const float* p) { return *(const float4*)p; }
__device__ __forceinline__ float4 load4(const bf16_t* p) {
  const uint2 v = *(const uint2*)p;
  return make_float4(__uint_as_float(v.x << 16), __uint_as_float(v.x & 0xffff0000u), __uint_as_float(v.y << 16), __uint_as_float(v.y & 0xffff0000u));
}

// VEC: four elements per load, the loads of a key row (and of 16 keys of V^T) in flight together, and two groups of
// keys side by side where a head is at most 32 wide (hd % 4 == 0, pointers aligned).  The loop of single loads waits
// for memory once per key: one row of the Tiny model (32 to 40 keys, head width 32) 8.6 us before, 5.3 now.
// NARROW (VEC, heads of at most 32; the number of loads of a key's row, 4 up to 16 elements, else 8): what bounds it is one
// load's latency after the other, so a chunk's keys, its values and q are requested together.  Eight loads also of narrower
// rows repeat the last one: two prompts of 1024 tokens, 8 tracks, 16 heads of 16, the whole pass in ms, no form of its own /
// eight loads / four: 12.0 / 12.7 / 10.8.
template <typename T, bool VEC, int NARROW>
__global__ void __launch_bounds__(64) attn_generic_kernel(pt_attn_args a) {
  __shared__ __attribute__((aligned(16))) float qs[256];
  const int lane = threadIdx.x;
  const int m = blockIdx.x, head = blockIdx.y, t = blockIdx.z;
  const int hd = a.hd;
  int seq, pos;
  if (a.row_map) {   // ragged batch: decode rows are indexed by sequence, prefill rows by packed row
    const int2 e = a.row_map[m];
    seq = e.x;
    pos = e.y;
  } else {
    seq = m / a.S;
    pos = a.pos0 + (m - seq * a.S);
  }
  const int nkeys = pos + 1;
  const int kvh = head / (a.H / a.Hkv);
  const int64_t hidx = t * a.kv_bstride + seq * a.kv_seq_stride + kvh;
  const T* K = (const T*)a.kc + hidx * a.kv_head_elems;
  const T* Vt = (const T*)a.vc + hidx * ((int64_t)hd * a.s_pad);
  const int64_t qoff = t * a.q_bstride + (int64_t)m * a.H * hd + head * hd;
  const T* q = (const T*)a.q + qoff;
  float q_mine = 0.f;
  if constexpr (NARROW) {
    if (lane < hd) q_mine = elem<T>::ld(q + lane);
  } else {
    for (int e = lane; e < hd; e += 64) qs[e] = elem<T>::ld(q + e);
    __syncthreads();
  }
  const float scale = 1.0f / sqrtf((float)hd);
  float mrun = -INFINITY, lsum = 0.f;
  float acc[4] = {0.f, 0.f, 0.f, 0.f};
  for (int base = 0; base < nkeys; base += 64) {
    const int key = base + lane;
    float s = -INFINITY;
    const int nk = min(64, nkeys - base);
    float4 kv[NARROW ? NARROW : 1], vv[NARROW ? 8 : 1];
    (void)kv; (void)vv;
    if constexpr (NARROW) {
      // lane: head-dim index lane % 32 of the values at positions 8 i + 4 * (lane / 32) .. + 3; the 64 positions of a chunk
      // lie inside the cache row.  Lanes past the last key or the head's width repeat the last one.
      const T* kr = K + (int64_t)min(key, nkeys - 1) * hd;
      const T* vr = Vt + (int64_t)min(lane & 31, hd - 1) * a.s_pad + base + 4 * (lane >> 5);
#pragma unroll
      for (int i = 0; i < NARROW; ++i) kv[i] = load4(kr + min(4 * i, hd - 4));
#pragma unroll
      for (int i = 0; i < 8; ++i)
        if (8 * i < nk) vv[i] = load4(vr + 8 * i);
      if (base == 0) {
        if (lane < hd) qs[lane] = q_mine;
        __syncthreads();
      }
      float4 d = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
      for (int i = 0; i < NARROW; ++i)
        if (4 * i < hd) {
          const float4 q4 = *(const float4*)(qs + 4 * i);
          d.x = fmaf(q4.x, kv[i].x, d.x); d.y = fmaf(q4.y, kv[i].y, d.y); d.z = fmaf(q4.z, kv[i].z, d.z); d.w = fmaf(q4.w, kv[i].w, d.w);
        }
      if (key < nkeys) s = ((d.x + d.y) + (d.z + d.w)) * scale;
    } else if (key < nkeys) {
      const T* kr = K + (int64_t)key * hd;
      float dot = 0.f;
      if constexpr (VEC) {
        float4 d = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll 8
        for (int e = 0; e < hd; e += 4) {
          const float4 k4 = load4(kr + e), q4 = *(const float4*)(qs + e);
          d.x = fmaf(q4.x, k4.x, d.x); d.y = fmaf(q4.y, k4.y, d.y); d.z = fmaf(q4.z, k4.z, d.z); d.w = fmaf(q4.w, k4.w, d.w);
        }
        dot = (d.x + d.y) + (d.z + d.w);
      } else {
        for (int e = 0; e < hd; ++e) dot = fmaf(qs[e], elem<T>::ld(kr + e), dot);
      }
      s = dot * scale;
    }
    const float mnew = fmaxf(mrun, wave_max(s));
    const float p = key < nkeys ? expf(s - mnew) : 0.f;
    const float corr = expf(mrun - mnew);   // 0 on the first chunk
    lsum = lsum * corr + wave_sum(p);
    mrun = mnew;
#pragma unroll
    for (int i = 0; i < 4; ++i) acc[i] *= corr;
    if constexpr (NARROW) {
#pragma unroll
      for (int i = 0; i < 8; ++i)
        if (8 * i < nk) {                               // wave-uniform
          const int kk = 8 * i + 4 * (lane >> 5);
          const float p0 = __shfl(p, kk, 64), p1 = __shfl(p, kk + 1, 64), p2 = __shfl(p, kk + 2, 64), p3 = __shfl(p, kk + 3, 64);
          // positions that no token has written may hold anything, and 0 * NaN is not 0
          acc[0] = fmaf(p0, kk < nk ? vv[i].x : 0.f, acc[0]);
          acc[0] = fmaf(p1, kk + 1 < nk ? vv[i].y : 0.f, acc[0]);
          acc[0] = fmaf(p2, kk + 2 < nk ? vv[i].z : 0.f, acc[0]);
          acc[0] = fmaf(p3, kk + 3 < nk ? vv[i].w : 0.f, acc[0]);
        }
    } else if constexpr (VEC) {
#pragma unroll 4
      for (int kk = 0; kk < nk; kk += 4) {            // at most 60: the 64 positions of a chunk lie inside the cache row
        const float p0 = __shfl(p, kk, 64), p1 = __shfl(p, kk + 1, 64), p2 = __shfl(p, kk + 2, 64), p3 = __shfl(p, kk + 3, 64);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int e = lane + 64 * i;
          if (e < hd) {
            const float4 v = load4(Vt + (int64_t)e * a.s_pad + base + kk);
            // positions that no token has written may hold anything, and 0 * NaN is not 0
            acc[i] = fmaf(p0, kk < nk ? v.x : 0.f, acc[i]);
            acc[i] = fmaf(p1, kk + 1 < nk ? v.y : 0.f, acc[i]);
            acc[i] = fmaf(p2, kk + 2 < nk ? v.z : 0.f, acc[i]);
            acc[i] = fmaf(p3, kk + 3 < nk ? v.w : 0.f, acc[i]);
          }
        }
      }
    } else
    for (int kk = 0; kk < nk; ++kk) {
      const float pk = __shfl(p, kk, 64);   // executed by the whole wavefront
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int e = lane + 64 * i;
        if (e < hd) acc[i] = fmaf(pk, elem<T>::ld(Vt + (int64_t)e * a.s_pad + base + kk), acc[i]);
      }
    }
  }
  T* o = (T*)a.o + qoff;
  const float inv = 1.0f / lsum;
  if (NARROW) acc[0] += __shfl_xor(acc[0], 32, 64);   // positions 0-3 and 4-7 of every eight
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int e = lane + 64 * i;
    if (e < hd) elem<T>::st(o + e, acc[i] * inv);
  }
}

int pt_launch_attn_generic(const pt_attn_args& a, hipStream_t s) {
  const int64_t rows = a.seq_info ? a.rows : (int64_t)a.B * a.S;
  if (rows <= 0) return PT_OK;
  if (a.hd > 256) return pt_set_error(PT_ERR_INVALID_ARGUMENT, "head_dim > 256");
  dim3 grid((unsigned)rows, (unsigned)a.H, (unsigned)a.n_tracks);
  const bool vec = !((a.hd | a.s_pad) & 3) && !(a.kv_head_elems & 3) && !(((uintptr_t)a.kc | (uintptr_t)a.vc) & 15);
  const int narrow = !vec || a.hd > 32 ? 0 : a.hd > 16 ? 8 : 4;
  auto launch = [&](auto kern) { hipLaunchKernelGGL(kern, grid, dim3(64), 0, s, a); };
  auto of_type = [&](auto t) {
    using T = decltype(t);
    if (narrow == 4) launch(attn_generic_kernel<T, true, 4>);
    else if (narrow == 8) launch(attn_generic_kernel<T, true, 8>);
    else if (vec) launch(attn_generic_kernel<T, true, 0>);
    else launch(attn_generic_kernel<T, false, 0>);
  };
  if (a.dtype == PT_F32) of_type(float{});
  else of_type(bf16_t{});
  PT_HIP_CHECK(hipGetLastError());
  return PT_OK;
}
