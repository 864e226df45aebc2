// The square tiles of the MFMA GEMM family (256 x 256 and 128 x 128, four wavefronts as 2 x 2): a persistent kernel body
// whose operand tiles go straight from global memory into LDS.  Included by gemm_mfma_impl.h.
//
// What bounds it and why it looks like this:
//  - On model data the chip is limited by power, so energy per operation is time.  A bare MFMA loop on N(0,1) x N(0,0.02)
//    operands reaches 1.77-1.85 PFLOP/s with 32x32x16 and 1.95-2.1 with 16x16x32 instructions (2.46 both on zeros): the
//    latter read and write half the accumulator bytes per operation.  Loads that go straight into LDS save the staging
//    registers and their LDS stores on top.
//  - The compiler does not keep 256 accumulators of 16x16 tiles in place (it copies them between registers around every
//    instruction), so the MFMAs are inline assembly with the accumulators tied to accumulation registers.
//  - Loads are spread evenly over the K step.  One every second MFMA takes 2090 us where one every sixth takes 1835
//    (4096 x 57344 x 8192, zeros).
//  - A workgroup takes tiles until none is left (one or two workgroups per compute unit).  The loads of the next tile's
//    first two K steps are issued in the last two K steps of this one, so the pipeline never empties: the epilogue has
//    LDS of its own and runs while they travel.
// SwiGLU GEMM on model data, us, before (32x32x16 MFMAs, tiles staged through registers, one workgroup per tile) and now:
// 4 tracks x 4096 x 8192, K = 1024: 253 -> 210; 8 x 16384 x 16384, K = 2048: 7170 -> 5910; 4096 x 57344, K = 8192: 2810 ->
// 2410.
//
// Operand order.  X is the operand whose rows become the rows of an accumulator tile, Y the other.  A lane of a 16x16
// tile holds Y row lane % 16 and, in element v, X row 4 * (lane / 16) + v.  X is the weight matrix, so a lane has four
// consecutive output columns of one row; only the V section of a QKV GEMM swaps the two (per wavefront, by its LDS
// offsets alone), so that a lane has four consecutive positions of one head-dim index, as V^T wants them.
#ifndef PT_GEMM_TILE_IMPL_H_
#define PT_GEMM_TILE_IMPL_H_

__device__ __forceinline__ void mfma_16x16x32(f32x4_t& c, const bf16x8_t& x, const bf16x8_t& y) {
  asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(c) : "v"(x), "v"(y));
}
__device__ __forceinline__ void mfma_16x16x32_first(f32x4_t& c, const bf16x8_t& x, const bf16x8_t& y) {
  asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, 0" : "=a"(c) : "v"(x), "v"(y));
}
__device__ __forceinline__ float acc_elem4(const f32x4_t& tile, int v) {
  float x;
  asm("v_accvgpr_read_b32 %0, %1" : "=v"(x) : "a"(tile[v]));
  return x;
}

// 8-byte LDS store.  Written as an ordinary one it waits for every load that is still on its way into LDS, the next
// tile's among them, because the compiler cannot tell that their places differ.
__device__ __forceinline__ void lds_write8(uint32_t addr, uint2 v) {
  asm volatile("ds_write_b64 %0, %1" ::"v"(addr), "v"(v) : "memory");
}

// 16 bytes from the accumulators, likewise.
__device__ __forceinline__ void lds_write_acc(uint32_t addr, const f32x4_t& v) {
  asm volatile("ds_write_b128 %0, %1" ::"v"(addr), "a"(v) : "memory");
}

// Sum over the N consecutive lanes (8 or 16 of an aligned group) in each of them.
template <int N>
__device__ __forceinline__ float lanes_sum(float x) {
  auto moved = [](float v, auto CTRL) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), decltype(CTRL)::value, 0xf, 0xf, false));
  };
  x += moved(x, std::integral_constant<int, 0xb1>{});    // quad_perm 1,0,3,2
  x += moved(x, std::integral_constant<int, 0x4e>{});    // quad_perm 2,3,0,1
  x += moved(x, std::integral_constant<int, 0x141>{});   // row_half_mirror
  if constexpr (N == 16) x += moved(x, std::integral_constant<int, 0x140>{});   // row_mirror
  return x;
}

// The kernel's arguments, loaded again wherever a phase of a tile begins: kept in registers from the start, their 80
// scalar registers and the K loop's own do not fit, and the compiler spills them around the loop.
typedef const __attribute__((address_space(4))) pt_gemm_args* gemm_kernarg_t;
__device__ __forceinline__ const pt_gemm_args& gemm_args_again() {
  gemm_kernarg_t p = (gemm_kernarg_t)__builtin_amdgcn_kernarg_segment_ptr();   // the arguments are the kernel's first parameter
  asm volatile("" : "+s"(p));
  return *(const pt_gemm_args*)p;
}

// Sizes of a square tile of BM rows and columns: T accumulator tiles per wavefront and direction, and its LDS.
// NB: K steps in LDS.  Two are enough where another workgroup on the compute unit, or the 2048 clocks of the large tile's
// K step, cover the loads; four for the small tile on a unit of its own (gemm_tile_deep_kernel).
template <int BM, int NB>
struct square_tile {
  static constexpr int BK = 64, T = BM / 32, TM = BM / 2;
  static constexpr int STG = 2 * BM * BK;                       // elements of one K step of both operands
  static constexpr int PATCH = 16 * TM * 2 + TM * 4;            // bytes per wavefront: 16 rows of bf16 (or half rows of fp32), and row factors
  static constexpr int LDS = NB * STG * 2 + 4 * PATCH;          // 146 KB (256) or 73 KB (128: two workgroups per unit)
  static constexpr int PER_CU = BM == 256 || NB > 2 ? 1 : 2;
};

// A wavefront's finished tile: acc[x][y], first row wave_m and column wave_n; `patch` is its private LDS.
template <int T, int EPI>
__device__ __forceinline__ void square_tile_epilogue(const pt_gemm_args& g, const f32x4_t (&acc)[T][T], bf16_t* patch, int b,
                                                     int wave_m, int wave_n, int lane, bool swapped, const float (&mine)[T / 4]) {
  constexpr int TM = 16 * T, CH = 2 * T;         // rows = columns of the wavefront's tile; 16-byte chunks of a patch row
  constexpr int RPI = 64 / CH;                   // patch rows that 64 lanes read at once, 16 bytes each
  const int lr = lane & 15, q = lane >> 4;
  const int rd_row = lane / CH, rd_ch = lane % CH;
  const uint32_t patch_lds = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)patch;
  // Patch rows are CH chunks; the chunk is XOR-ed with the row so that neither 16 rows written at one column nor whole
  // rows read meet in the same banks.
  auto swz = [](int row) { return T == 8 ? row : (row >> 1) & 7; };
  auto put4 = [&](int chunk, float x0, float x1, float x2, float x3) {     // 4 elements, half (q & 1) of a chunk of row lr
    uint2 pk;
    pk.x = pack_bf16x2(x0, x1);
    pk.y = pack_bf16x2(x2, x3);
    lds_write8(patch_lds + (lr * CH + (chunk ^ swz(lr))) * 16 + (q & 1) * 8, pk);
  };
  auto take8 = [&](int it) {
    const int r = it * RPI + rd_row;
    return *(const u32x4_t*)(patch + (r * CH + (rd_ch ^ swz(r))) * 8);
  };
  // the patch is private to the wavefront, whose LDS operations stay in order; this keeps the compiler from moving reads
  // of one type over writes of another
  auto in_order = [] { asm volatile("" ::: "memory"); };
  // At the end of a path whose loads are not all waited for on every branch: the compiler would otherwise wait for all
  // outstanding memory operations in front of the next tile, behind the other paths as well.
  auto settle = [] { __builtin_amdgcn_s_waitcnt(0x0f70); };   // vmcnt(0)
  (void)settle;
  // folded RMSNorm: one factor per row of the wavefront's tile (consumer) or one gain per column (producer)
  float* factors = (float*)(patch + 16 * TM);
  if constexpr (EPI != EPI_STORE_F32) {
#pragma unroll
    for (int i = 0; i < T / 4; ++i) factors[i * 64 + lane] = mine[i];
    in_order();
  }
  (void)take8; (void)put4; (void)factors; (void)patch_lds;

  if constexpr (EPI == EPI_STORE_F32 || EPI == EPI_RESIDUAL) {
    // 16 rows of G tiles at a time go through the patch, as fp32, so that consecutive lanes store consecutive pieces of a
    // row.  Straight from the accumulators consecutive lanes lie a row apart, and the memory pipe takes them 16 bytes at a
    // time: 29 clocks a row of a 128-column tile where this form waits for nothing.  us a launch, straight / now: four K
    // slices of 256, 4 tracks x 128 rows x 1024 9.2 / 8.2; residual with folded norm, K = 1024, 4 x 256 x 1024 15.8 / 14.2;
    // 2048 x 1536, K = 1536 23.0 / 21.6.
    constexpr int G = T / 2, RPF = 16 / G, NG = 2 * T;   // rows per instruction; groups in the wavefront's tile
    static_assert(64 / CH == RPF, "a patch row is CH chunks of 16 bytes here too");
    float* out = g.out + b * g.out_bstride;
    const float* res = EPI == EPI_RESIDUAL ? g.res + b * g.res_bstride : nullptr;
    const int m_l = wave_m + rd_row, n_l = wave_n + 4 * rd_ch;
    const int64_t off = (int64_t)m_l * g.ldo + n_l;
    auto park = [&](auto I_) {       // group I: tiles G * (I % 2) .. of rows 16 * (I / 2) ..
      static_for<G>([&](auto X_) {
        constexpr int x = decltype(X_)::value;
        lds_write_acc(patch_lds + (lr * CH + ((4 * x + q) ^ swz(lr))) * 16, acc[G * (decltype(I_)::value % 2) + x][decltype(I_)::value / 2]);
      });
    };
    auto run = [&](auto FULL_, auto FOLD_) {
      constexpr bool FULL = decltype(FULL_)::value, FOLD = decltype(FOLD_)::value;
      constexpr int DEPTH = T == 8 ? 3 : 4;        // groups whose residual values are in flight
      f32x4_t r[DEPTH + 1][G], val[G], gain[2];
      float ss[G];
      (void)r; (void)gain; (void)ss;
      auto load_res = [&](auto I_) {
        constexpr int i = decltype(I_)::value;
        static_for<G>([&](auto IT_) {
          constexpr int row = 16 * (i / 2) + RPF * decltype(IT_)::value, col = 16 * G * (i % 2);
          // past the edge: some value of the matrix, which is not used
          const int64_t at = FULL ? off + (int64_t)row * g.ldo + col : (int64_t)min(m_l + row, g.M - 1) * g.ldo + min(n_l + col, g.N - 4);
          r[i % (DEPTH + 1)][decltype(IT_)::value] = *(const f32x4_t*)(res + at);
        });
      };
      auto fetch = [&] {
        in_order();
        static_for<G>([&](auto IT_) {
          const int row = decltype(IT_)::value * RPF + rd_row;
          val[decltype(IT_)::value] = *(const f32x4_t*)(patch + (row * CH + (rd_ch ^ swz(row))) * 8);
        });
        in_order();
      };
      if constexpr (EPI == EPI_RESIDUAL) static_for<DEPTH>([&](auto I_) { load_res(I_); });
      if constexpr (FOLD)
        for (int k = 0; k < 2; ++k) gain[k] = *(const f32x4_t*)(factors + 16 * G * k + 4 * rd_ch);
      park(std::integral_constant<int, 0>{});
      fetch();
      static_for<NG>([&](auto I_) {
        constexpr int i = decltype(I_)::value, y = i / 2, col = 16 * G * (i % 2);
        if constexpr (EPI == EPI_RESIDUAL && i + DEPTH < NG) load_res(std::integral_constant<int, i + DEPTH>{});
        if constexpr (i + 1 < NG) park(std::integral_constant<int, i + 1>{});
        int m_i = m_l, n_i = n_l;   // opaque per group: the bounds tests of all groups together would fill the scalar registers
        if constexpr (!FULL) asm volatile("" : "+v"(m_i), "+v"(n_i));
        static_for<G>([&](auto IT_) {
          constexpr int it = decltype(IT_)::value, row = 16 * y + RPF * it;
          f32x4_t v = val[it];
          if constexpr (EPI == EPI_RESIDUAL) v += r[i % (DEPTH + 1)][it];
          const bool in = FULL || (m_i + row < g.M && n_i + col < g.N);
          if (in) *(f32x4_t*)(out + off + (int64_t)row * g.ldo + col) = v;
          if constexpr (FOLD) {   // folded RMSNorm, producer side: bf16(h * gain) and the row's sum of squares
            const float sq = v.x * v.x + v.y * v.y + v.z * v.z + v.w * v.w;
            ss[it] = i % 2 ? ss[it] + sq : sq;
            const f32x4_t& gn = gain[i % 2];
            uint2 pk;
            pk.x = pack_bf16x2(v.x * gn.x, v.y * gn.y);
            pk.y = pack_bf16x2(v.z * gn.z, v.w * gn.w);
            if (in) *(uint2*)((bf16_t*)g.nf_out + b * g.nf_out_bstride + (int64_t)(m_l + row) * g.N + n_l + col) = pk;
          }
        });
        if constexpr (i + 1 < NG) fetch();
        if constexpr (FOLD && i % 2) {
          float sum = 0.f;   // lane c of a row's CH lanes takes the c-th of the G sums
          static_for<G>([&](auto IT_) {
            constexpr int it = decltype(IT_)::value;
            const float t = lanes_sum<CH>(ss[it]);
            sum = rd_ch == it ? t : sum;
          });
          const int m = m_l + 16 * y + RPF * rd_ch;
          if (rd_ch < G && (FULL || m < g.M)) g.nf_ss[b * g.nf_ss_bstride + (int64_t)m * g.nf_parts + wave_n / TM] = sum;
        }
      });
      if constexpr (!FULL) settle();
    };
    const bool full = wave_m + TM <= g.M && wave_n + TM <= g.N;
    const bool fold = EPI == EPI_RESIDUAL && g.nf_out != nullptr;   // the columns are then whole wavefront tiles
    if constexpr (EPI == EPI_RESIDUAL) {
      if (fold) {
        if (full) run(std::true_type{}, std::true_type{});
        else if (wave_n < g.N) run(std::false_type{}, std::true_type{});
      } else {
        if (full) run(std::true_type{}, std::false_type{});
        else if (wave_n < g.N) run(std::false_type{}, std::false_type{});
      }
    } else {
      if (full) run(std::true_type{}, std::false_type{});
      else if (wave_n < g.N) run(std::false_type{}, std::false_type{});
    }
  } else if constexpr (EPI == EPI_SWIGLU) {
    // gate and up alternate in blocks of 32 columns (two tiles each): tiles 4p, 4p+1 are gates, 4p+2, 4p+3 the matching
    // ups.  32 rows of T * 8 products fill the patch: row lr of it holds rows lr and lr + 16 side by side.
    bf16_t* o = (bf16_t*)g.olp + b * g.olp_bstride;
    const int ldo = g.N >> 1;
    const bool full = wave_m + TM <= g.M && wave_n + TM <= g.N;
    static_for<T / 2>([&](auto B_) {
      constexpr int blk = decltype(B_)::value;
      static_for<2>([&](auto Y_) {
        constexpr int h = decltype(Y_)::value, y = 2 * blk + h;
        const float f = factors[16 * y + lr];
        static_for<T / 2>([&](auto P_) {
          constexpr int p = decltype(P_)::value, xg = (p >> 1) * 4 + (p & 1);
          float z[4];
          static_for<4>([&](auto V_) {
            constexpr int v = decltype(V_)::value;
            z[v] = silu_fast(f * acc_elem4(acc[xg][y], v)) * (f * acc_elem4(acc[xg + 2][y], v));
          });
          put4(h * T + p * 2 + (q >> 1), z[0], z[1], z[2], z[3]);
        });
        __builtin_amdgcn_sched_barrier(0);   // bounds the scheduler's window (register pressure)
      });
      in_order();
      const int j = (wave_n >> 1) + (rd_ch % T) * 8, row0 = wave_m + 32 * blk + 16 * (rd_ch / T) + rd_row;
      bf16_t* dst = o + (int64_t)row0 * ldo + j;
      u32x4_t val[16 / RPI];
      static_for<16 / RPI>([&](auto IT_) { val[decltype(IT_)::value] = take8(decltype(IT_)::value); });
      static_for<16 / RPI>([&](auto IT_) {
        constexpr int it = decltype(IT_)::value;
        if (full) *(u32x4_t*)(dst + (int64_t)(it * RPI) * ldo) = val[it];
      });
      if (!full)
        static_for<16 / RPI>([&](auto IT_) {
          constexpr int it = decltype(IT_)::value;
          if (row0 + it * RPI < g.M && 2 * j < g.N) *(u32x4_t*)(dst + (int64_t)(it * RPI) * ldo) = val[it];
        });
      in_order();
    });
  } else {   // EPI_QKV, EPI_QKV_ROWS
    const int hq = g.H * g.hd, hk = g.Hkv * g.hd;
    if (wave_n >= g.N) return;
    // the sequence and position of row m, the same for every lane (a scalar load where the row map has it)
    auto uniform_row = [&](int m) {
      if (g.row_map) {
        typedef const __attribute__((address_space(4))) int32_t* c_ptr;
        c_ptr e = (c_ptr)(const int32_t*)(g.row_map + m);
        return pt_rowpos{e[0], e[1]};
      }
      return gemm_row_pos(g, m);
    };
    auto part = [&](auto WIDE_, auto FULL_) {
      constexpr int HD = decltype(WIDE_)::value ? 128 : 64;
      constexpr int NH = HD / 32;                        // tiles of half a head
      constexpr bool FULL = decltype(FULL_)::value;      // all rows of the wavefront's tile lie inside the matrix
      if (!swapped) {
        // q or k: rotate (u_j, u_{j+hd/2}), both in the same lane and element; cosine and sine of the row's position from
        // the rotary table.  A wavefront's columns are whole heads.
        const bool is_q = wave_n < hq;
        const float* tab = g.rope + 8 * q;
        int seqs[T], poss[T];
        static_for<T>([&](auto Y_) {
          constexpr int y = decltype(Y_)::value;
          if constexpr (EPI == EPI_QKV) {                // 32-row blocks lie in one sequence
            if constexpr ((y & 1) == 0) {
              const pt_rowpos rp = uniform_row(FULL ? wave_m + 16 * y : min(wave_m + 16 * y, g.M - 32));
              seqs[y] = seqs[y + 1] = rp.seq;
              poss[y] = rp.pos;
              poss[y + 1] = rp.pos + 16;
            }
          } else {
            const pt_rowpos rp = gemm_row_pos(g, min(wave_m + 16 * y + lr, g.M - 1));
            seqs[y] = rp.seq;
            poss[y] = rp.pos;
          }
        });
        constexpr int AH = EPI == EPI_QKV ? 1 : 0;       // blocks of 16 rows that the table entries are loaded ahead
        f32x4_t cs[AH + 1][NH][2];
        auto load_cs = [&](auto Y_) {
          constexpr int y = decltype(Y_)::value;
          const float* p = tab + (int64_t)(EPI == EPI_QKV ? poss[y] + lr : poss[y]) * HD;
#pragma unroll
          for (int w = 0; w < NH; ++w) {
            cs[y & AH][w][0] = *(const f32x4_t*)(p + 32 * w);
            cs[y & AH][w][1] = *(const f32x4_t*)(p + 32 * w + 4);
          }
        };
        if constexpr (AH) load_cs(std::integral_constant<int, 0>{});
        const int c8 = (is_q ? wave_n : wave_n - hq) + rd_ch * 8;       // the lane's columns when it stores
        bf16_t* base = is_q ? (bf16_t*)g.olp + b * g.olp_bstride + c8
                            : (bf16_t*)g.kc + (b * g.kv_bstride + c8 / HD) * g.kv_head_elems + c8 % HD;
        const int64_t seq_pitch = is_q ? 0 : g.kv_seq_stride * g.kv_head_elems;   // q has rows, k sequences and positions
        const int pitch = is_q ? hq : HD;
        static_for<T>([&](auto Y_) {
          constexpr int y = decltype(Y_)::value;
          if constexpr (y + AH < T) load_cs(std::integral_constant<int, y + AH>{});
          const float f = factors[16 * y + lr];
          static_for<T / 2>([&](auto P_) {
            constexpr int p = decltype(P_)::value, w = p % NH, xl = (p / NH) * 2 * NH + w;
            float lo[4], hi[4];
            static_for<4>([&](auto V_) {
              constexpr int v = decltype(V_)::value;
              const f32x4_t& t = cs[y & AH][w][v >> 1];
              const float c = (v & 1) ? t.z : t.x, s = (v & 1) ? t.w : t.y;
              const float a = f * acc_elem4(acc[xl][y], v), e = f * acc_elem4(acc[xl + NH][y], v);
              lo[v] = a * c - e * s;
              hi[v] = e * c + a * s;
            });
            put4(xl * 2 + (q >> 1), lo[0], lo[1], lo[2], lo[3]);
            put4((xl + NH) * 2 + (q >> 1), hi[0], hi[1], hi[2], hi[3]);
          });
          in_order();
          static_for<16 / RPI>([&](auto IT_) {
            constexpr int it = decltype(IT_)::value;
            const int r = it * RPI + rd_row, m = wave_m + 16 * y + r;
            int64_t at;                                  // element offset of the row
            if constexpr (EPI == EPI_QKV) {
              at = seqs[y] * seq_pitch + (int64_t)((is_q ? wave_m + 16 * y : poss[y]) + r) * pitch;
            } else {
              const int seq = __shfl(seqs[y], r, 64), pos = __shfl(poss[y], r, 64);
              at = seq * seq_pitch + (int64_t)(is_q ? m : pos) * pitch;
            }
            if (FULL || m < g.M) {
              bf16_t* dst = base + at;
              *(u32x4_t*)dst = take8(it);
            }
          });
          in_order();
        });
      } else {
        // v: acc[x][y] holds head-dim index 16 y + lr at four consecutive rows from 16 x + 4 q on.  16 head-dim rows at a
        // time go through the patch and leave as pieces of 8 positions where a piece lies at an aligned place of one
        // sequence, which EPI_QKV promises.
        const int r8 = wave_m + rd_ch * 8;                // first row of the lane's piece
        const pt_rowpos rp8 = gemm_row_pos(g, FULL ? r8 : min(r8, EPI == EPI_QKV ? g.M - 8 : g.M - 1));
        const int colv = wave_n - hq - hk;                // heads follow one another in V^T: column = row of it
        const bool mine_ok = FULL || r8 < g.M;
        bool pieces = true;
        if constexpr (EPI == EPI_QKV_ROWS)
          pieces = !__any(mine_ok && (g.row_map || r8 + 8 > g.M || (rp8.pos & 7) || rp8.pos - g.pos0 + 8 > g.S));
        bf16_t* vt = (bf16_t*)g.vc + (b * g.kv_bstride + rp8.seq * g.kv_seq_stride) * ((int64_t)HD * g.s_pad) + rp8.pos;
        static_for<T>([&](auto Y_) {
          constexpr int y = decltype(Y_)::value;
          static_for<T>([&](auto X_) {
            constexpr int x = decltype(X_)::value;
            const f32x4_t f = *(const f32x4_t*)(factors + 16 * x + 4 * q);
            put4(x * 2 + (q >> 1), f.x * acc_elem4(acc[x][y], 0), f.y * acc_elem4(acc[x][y], 1), f.z * acc_elem4(acc[x][y], 2),
                 f.w * acc_elem4(acc[x][y], 3));
          });
          in_order();
          if (pieces) {
            static_for<16 / RPI>([&](auto IT_) {
              constexpr int it = decltype(IT_)::value;
              const u32x4_t val = take8(it);
              if (mine_ok) *(u32x4_t*)(vt + (int64_t)(colv + 16 * y + it * RPI + rd_row) * g.s_pad) = val;
            });
          } else if constexpr (EPI == EPI_QKV_ROWS) {
            // a lane per row: runs of consecutive positions, 2 bytes each
#pragma unroll
            for (int h = 0; h < T / 4; ++h) {
              const int r = h * 64 + lane;
              if (wave_m + r < g.M) {
                const pt_rowpos rp = gemm_row_pos(g, wave_m + r);
                bf16_t* dst = (bf16_t*)g.vc + (b * g.kv_bstride + rp.seq * g.kv_seq_stride) * ((int64_t)HD * g.s_pad) +
                              (int64_t)(colv + 16 * y) * g.s_pad + rp.pos;
#pragma unroll 8
                for (int n = 0; n < 16; ++n) dst[(int64_t)n * g.s_pad] = patch[(n * CH + ((r >> 3) ^ swz(n))) * 8 + (r & 7)];
              }
            }
          }
          in_order();
        });
      }
    };
    auto either = [&](auto WIDE_) {
      if constexpr (EPI == EPI_QKV) {
        if (wave_m + TM <= g.M) {
          part(WIDE_, std::true_type{});
          return;
        }
      }
      part(WIDE_, std::false_type{});
      settle();
    };
    if constexpr (T == 8) {
      if (g.hd == 128) { either(std::true_type{}); return; }
    }
    either(std::false_type{});   // a wavefront of the small tile has 64 columns: one head of 64
  }
}

template <int BM, int NB, int EPI>
__device__ __forceinline__ void square_tile_run(int tiles_m, int tiles_n) {
  using S = square_tile<BM, NB>;
  // more than two buffers take turns by an offset instead of in pairs of K steps; K is then at least NB steps
  constexpr bool DEEP = NB > 2;
  constexpr int BK = S::BK, T = S::T, TM = S::TM, STG = S::STG;
  // Schedule of a K step in MFMAs (2 T^2 of them, two sub-steps of 32 of K).  Sub-step 0 reads the fragments of sub-step 1
  // from the same LDS buffer, all of them in front of barrier 1 (MFMA P1); behind it the buffer is free and the loads of
  // the K step after next go into it, one every LSP MFMAs to the end of the K step.  Sub-step 1 reads the next K step's
  // first fragments from the other buffer behind barrier 2 (its MFMA P2), where the loads of one K step ago have landed.
  constexpr int NM = T * T, FR = 2 * T, LD = 2 * T, P1 = FR + (T == 8 ? 8 : 4), P2 = NM / 4, LSP = (2 * NM - P1) / LD;
  constexpr int AHEAD = (NM + P2 - P1 + LSP - 1) / LSP;   // loads of this K step in front of barrier 2
  static_assert(P1 + LSP * (LD - 1) < 2 * NM && P2 + FR <= NM && AHEAD <= LD, "schedule");
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  bf16_t* lds = (bf16_t*)smem;   // [NB][A rows then W rows][BK], then the wavefronts' patches
  typedef __attribute__((address_space(3))) void* lptr_t;
  // XOR swizzle of the 16-byte chunks, as in the register-staged kernel
  auto SWZ = [](int row) { return (row >> 1) & 7; };
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  const pt_gemm_args& g0 = gemm_args_again();
  // what the first tile's loads need, requested at once instead of one after the other on the way there
  asm volatile("" ::"s"(g0.A), "s"(g0.W), "s"(g0.a_bstride), "s"(g0.w_bstride), "s"(g0.lda), "s"(g0.ldb), "s"(g0.M), "s"(g0.N), "s"(g0.K),
               "s"(g0.batch), "s"(g0.blk_group), "s"(g0.a_rows), "s"(g0.k_tracks), "s"(tiles_m), "s"(tiles_n));
  const int total = tiles_m * tiles_n * g0.batch;
  const int KT = g0.K / BK;                               // K steps: even, >= 2

  // Loads: an instruction moves 8 rows of 128 bytes; this lane row lane / 8 and logical chunk (lane % 8) ^ swizzle.  Rows
  // and columns past the matrix are past the end of the buffer and read as zero.
  uint32_t a_voff[T], w_voff[T];
#pragma unroll
  for (int i = 0; i < T; ++i) {
    const int row = (wave * T + i) * 8 + (lane >> 3);
    const int ch = ((lane & 7) ^ SWZ(row)) * 8;
    a_voff[i] = (uint32_t)(row * g0.lda + ch) * 2;
    w_voff[i] = (uint32_t)(row * g0.ldb + ch) * 2;
  }
  struct place {
    int id, m0, n0, b, group;
  };
  // the first tile at or after `id` in this workgroup's sequence that has rows; id >= total: none
  auto locate = [&](const pt_gemm_args& g, int id) {
    place t = {id, 0, 0, 0, 0};
    for (; t.id < total; t.id += gridDim.x) {
      const tile_coord tc = map_tile(t.id, total, tiles_m, tiles_n);
      // the tile's coordinates are the same for every lane: kept in scalar registers
      t.m0 = __builtin_amdgcn_readfirstlane(tc.tm) * BM;
      t.n0 = __builtin_amdgcn_readfirstlane(tc.tn) * BM;
      t.b = __builtin_amdgcn_readfirstlane(tc.b);
      if constexpr (EPI == EPI_SWIGLU || EPI == EPI_STORE_F32) {   // grouped GEMM: blocks without rows have no group
        if (g.blk_group) {
          t.group = *(const __attribute__((address_space(4))) int32_t*)(g.blk_group + t.b * g.grp_bstride + (t.m0 >> 6));
          if (t.group < 0) continue;
        }
      }
      break;
    }
    return t;
  };
  __amdgpu_buffer_rsrc_t ra, rw;
  // the buffers of a tile's operand rows; empty for no tile (the last loads of a workgroup then read nothing)
  auto open = [&](const pt_gemm_args& g, const place& t) {
    int bt = t.b, k_off = 0;   // track and first element of the K slice
    if constexpr (EPI == EPI_STORE_F32) {
      if (g.k_tracks > 0) {
        const int slice = t.b / g.k_tracks;
        bt = t.b - slice * g.k_tracks;
        k_off = slice * g.K;
      }
    }
    const bool any = t.id < total;
    const bool gathered = (EPI == EPI_SWIGLU || EPI == EPI_STORE_F32) && g.a_rows;
    const bf16_t* a = (const bf16_t*)g.A + bt * g.a_bstride + k_off + (gathered ? 0 : (int64_t)t.m0 * g.lda);
    const bf16_t* w = (const bf16_t*)g.W + bt * g.w_bstride + k_off + t.group * g.w_gstride + (int64_t)t.n0 * g.ldb;
    // gathered rows are addressed from the track's first row: the host checks rows * lda * 2 < 2^32
    const uint32_t an = !any ? 0 : gathered ? 0xffffffffu : (uint32_t)((min(g.M - t.m0, BM) - 1) * g.lda + g.K) * 2;
    const uint32_t wn_bytes = !any ? 0 : (uint32_t)((min(g.N - t.n0, BM) - 1) * g.ldb + g.K) * 2;
    ra = __builtin_amdgcn_make_buffer_rsrc((void*)a, 0, an, 0x00020000);
    rw = __builtin_amdgcn_make_buffer_rsrc((void*)w, 0, wn_bytes, 0x00020000);
    if constexpr (EPI == EPI_SWIGLU || EPI == EPI_STORE_F32) {
      if (gathered && any) {
#pragma unroll
        for (int i = 0; i < T; ++i) {
          const int row = (wave * T + i) * 8 + (lane >> 3);
          a_voff[i] = ((uint32_t)g.a_rows[t.b * g.a_rows_bstride + t.m0 + row] * (uint32_t)g.lda + ((lane & 7) ^ SWZ(row)) * 8) * 2;
        }
      }
    }
  };
  // LDS byte address of the wavefront's first load.  Made opaque once a K step: the addresses of the single loads would
  // otherwise be kept in 32 scalar registers instead of being added up where they are used.
  const uint32_t lds_first = (uint32_t)(uintptr_t)(lptr_t)lds + wave * (T * 8 * BK * 2);
  uint32_t lds_wave = lds_first;
  auto issue_load = [&](auto I_, int koff, int stage) {
    constexpr int i = decltype(I_)::value;
    if constexpr (i < T)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(ra, (lptr_t)(uintptr_t)(lds_wave + (stage * STG + i * 8 * BK) * 2), 16, a_voff[i], koff, 0, 0);
    else
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rw, (lptr_t)(uintptr_t)(lds_wave + (stage * STG + BM * BK + (i - T) * 8 * BK) * 2), 16, w_voff[i - T], koff, 0, 0);
  };
  // Fragments: row = tile row + lane % 16, logical chunk 4 * sub-step + lane / 16.  x_fr / y_fr: element offset of the
  // wavefront's first tile for either sub-step.
  const int fr_a = (wm * TM + (lane & 15)) * BK, fr_w = BM * BK + (wn * TM + (lane & 15)) * BK;
  const int fr_ch0 = ((lane >> 4) ^ SWZ(lane & 15)) * 8, fr_ch1 = ((4 + (lane >> 4)) ^ SWZ(lane & 15)) * 8;
  auto is_swapped = [&](const pt_gemm_args& g, const place& t) {
    return (EPI == EPI_QKV || EPI == EPI_QKV_ROWS) && t.n0 + wn * TM >= (g.H + g.Hkv) * g.hd;
  };

  place cur = locate(g0, blockIdx.x);
  if (cur.id >= total) return;
  open(g0, cur);
  static_for<LD>([&](auto I_) { issue_load(I_, 0, 0); });
  static_for<LD>([&](auto I_) { issue_load(I_, BK * 2, 1); });
  if constexpr (DEEP) {
    static_assert(NB == 4 || !DEEP, "the fill issues two more K steps");
    static_for<LD>([&](auto I_) { issue_load(I_, 2 * BK * 2, 2); });
    static_for<LD>([&](auto I_) { issue_load(I_, 3 * BK * 2, 3); });
  }
  bool swapped = is_swapped(g0, cur);
  int x_fr0 = (swapped ? fr_a : fr_w) + fr_ch0, y_fr0 = (swapped ? fr_w : fr_a) + fr_ch0;
  int x_fr1 = (swapped ? fr_a : fr_w) + fr_ch1, y_fr1 = (swapped ? fr_w : fr_a) + fr_ch1;
  asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"((NB - 1) * LD) : "memory");
  f32x4_t acc[T][T];
  bf16x8_t xf[2][T], yf[2][T];
#pragma unroll
  for (int i = 0; i < T; ++i) xf[0][i] = *(const bf16x8_t*)(lds + x_fr0 + i * 16 * BK);
#pragma unroll
  for (int i = 0; i < T; ++i) yf[0][i] = *(const bf16x8_t*)(lds + y_fr0 + i * 16 * BK);
  int koff = NB * BK * 2;   // byte offset of the K step whose loads come next
  int turn = 0;   // DEEP: element offset of the buffer that is multiplied
  static_assert((NB & (NB - 1)) == 0, "buffers take turns by a mask");
  auto iteration = [&](auto PAR, auto FIRST_) {
    constexpr int buf = DEEP ? 0 : decltype(PAR)::value;
    constexpr bool FIRST = decltype(FIRST_)::value;
    asm volatile("" : "+s"(lds_wave));
    const bf16_t* C = lds + (DEEP ? turn : buf * STG);
    const bf16_t* N = lds + (DEEP ? (turn + STG) & (NB * STG - 1) : (buf ^ 1) * STG);
    static_for<2>([&](auto KK) {
      constexpr int kk = decltype(KK)::value, fb = kk ^ 1, R0 = kk == 0 ? 0 : P2;
      static_for<NM>([&](auto J) {
        constexpr int j = decltype(J)::value;
        constexpr int x = j / T, y = (x & 1) ? T - 1 - j % T : j % T;   // back and forth: one operand changes at a time
        if constexpr (kk == 0 && j == P1) asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        if constexpr (kk == 1 && j == P2) asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(AHEAD + (NB - 2) * LD) : "memory");
        if constexpr (FIRST && kk == 0) mfma_16x16x32_first(acc[x][y], xf[kk][x], yf[kk][y]);
        else mfma_16x16x32(acc[x][y], xf[kk][x], yf[kk][y]);
        if constexpr (j >= R0 && j - R0 < FR) {
          constexpr int r = j - R0;
          if constexpr (r < T) xf[fb][r] = *(const bf16x8_t*)((kk ? N + x_fr0 : C + x_fr1) + r * 16 * BK);
          else yf[fb][r - T] = *(const bf16x8_t*)((kk ? N + y_fr0 : C + y_fr1) + (r - T) * 16 * BK);
        }
        constexpr int s = kk * NM + j - P1;
        if constexpr (s >= 0 && s % LSP == 0 && s / LSP < LD) issue_load(std::integral_constant<int, s / LSP>{}, koff, buf);
        __builtin_amdgcn_sched_barrier(0);
      });
    });
    koff += BK * 2;
    if constexpr (DEEP) {
      turn = (turn + STG) & (NB * STG - 1);
      lds_wave = lds_first + turn * 2;
    }
  };
  for (;;) {
    PT_STAMP_TILE(cur.id, 6);
    PT_STAMP_TILE(cur.id, 0);
    // folded RMSNorm: 1/rms per row of the wavefront's tile (consumer, from pt_launch_row_inv_rms) or the gain per column
    // (producer); loaded here, parked in the patch after the K loop
    float mine[T / 4];
    {
      const pt_gemm_args& g = gemm_args_again();
#pragma unroll
      for (int i = 0; i < T / 4; ++i) {
        mine[i] = 1.0f;
        if constexpr (EPI == EPI_RESIDUAL) {
          if (g.nf_out) mine[i] = g.nf_gain[cur.b * g.nf_gain_bstride + min(cur.n0 + wn * TM + i * 64 + lane, g.N - 1)];
        } else if constexpr (EPI != EPI_STORE_F32) {
          if (g.rs_inv) mine[i] = g.rs_inv[cur.b * g.rs_bstride + min(cur.m0 + wm * TM + i * 64 + lane, g.M - 1)];
        }
      }
    }
    // ... or the row's partial sums of squares, from which the factor is formed here: requested behind the first K step and
    // added up behind the second, so that nothing waits for them and the epilogue's registers are not asked for
    constexpr bool SUMS = EPI == EPI_SWIGLU || EPI == EPI_QKV || (EPI == EPI_QKV_ROWS && T == 4);   // the large tile's row lookups leave no registers
    f32x4_t sums[SUMS ? T / 4 : 1][PT_NF_MAX_SUMS / 4];
    (void)sums;
    auto fetch_sums = [&] {
      if constexpr (SUMS) {
        const pt_gemm_args& g = gemm_args_again();
        if (g.nf_parts > 0) {
#pragma unroll
          for (int i = 0; i < T / 4; ++i) {
            const float* ss = g.nf_ss + cur.b * g.nf_ss_bstride + (int64_t)min(cur.m0 + wm * TM + i * 64 + lane, g.M - 1) * g.nf_parts;
#pragma unroll
            for (int p = 0; p < PT_NF_MAX_SUMS / 4; ++p) sums[i][p] = *(const f32x4_t*)(ss + min(4 * p, g.nf_parts - 4));
          }
        }
      }
    };
    auto add_sums = [&] {
      if constexpr (SUMS) {
        const pt_gemm_args& g = gemm_args_again();
        if (g.nf_parts > 0) {
#pragma unroll
          for (int i = 0; i < T / 4; ++i) {
            float acc_ss = 0.f;
#pragma unroll
            for (int p = 0; p < PT_NF_MAX_SUMS / 4; ++p)
              if (4 * p < g.nf_parts) acc_ss = (((acc_ss + sums[i][p].x) + sums[i][p].y) + sums[i][p].z) + sums[i][p].w;
            mine[i] = 1.0f / sqrtf(acc_ss * (1.0f / (float)g.K) + g.norm_eps);
          }
        }
      }
    };
    const pt_gemm_args& gn = gemm_args_again();
    const place nxt = locate(gn, cur.id + gridDim.x);
    const bool nxt_swapped = is_swapped(gn, nxt);
    PT_STAMP_TILE(cur.id, 1);
    auto next_fragments = [&] {   // from here on the first sub-step's fragments are the next tile's
      x_fr0 = (nxt_swapped ? fr_a : fr_w) + fr_ch0;
      y_fr0 = (nxt_swapped ? fr_w : fr_a) + fr_ch0;
    };
    if constexpr (DEEP) {
      auto step = [&](auto FIRST_, int kt) {
        if (kt + NB == KT) { open(gemm_args_again(), nxt); koff = 0; }
        if (kt + 1 == KT) next_fragments();
        iteration(std::integral_constant<int, 0>{}, FIRST_);
      };
      step(std::true_type{}, 0);
      fetch_sums();
      step(std::false_type{}, 1);
      add_sums();
      for (int kt = 2; kt < KT; ++kt) step(std::false_type{}, kt);
    } else {
      if (KT == 2) { open(gemm_args_again(), nxt); koff = 0; }
      iteration(std::integral_constant<int, 0>{}, std::true_type{});
      if (KT == 2) next_fragments();
      fetch_sums();
      iteration(std::integral_constant<int, 1>{}, std::false_type{});
      add_sums();
      for (int kt = 2; kt < KT; kt += 2) {
        if (kt + 2 == KT) { open(gemm_args_again(), nxt); koff = 0; }
        iteration(std::integral_constant<int, 0>{}, std::false_type{});
        if (kt + 2 == KT) next_fragments();
        iteration(std::integral_constant<int, 1>{}, std::false_type{});
      }
    }
    x_fr1 = (nxt_swapped ? fr_a : fr_w) + fr_ch1;
    y_fr1 = (nxt_swapped ? fr_w : fr_a) + fr_ch1;
    // The compiler does not see the MFMAs inside the assembly: their results take up to 18 cycles to arrive.  Every
    // accumulator passes through a statement behind the wait, so that nothing can read one in front of it.
    asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");
#pragma unroll
    for (int i = 0; i < T * T; ++i) asm volatile("" : "+a"(acc[i / T][i % T]));
    PT_STAMP_TILE(cur.id, 2);
    PT_STAMP_TILE(cur.id, 3);
    square_tile_epilogue<T, EPI>(gemm_args_again(), acc, (bf16_t*)(smem + NB * STG * 2 + wave * S::PATCH), cur.b, cur.m0 + wm * TM, cur.n0 + wn * TM,
                                 lane, swapped, mine);
    PT_STAMP_TILE(cur.id, 4);
    PT_STAMP_TILE(cur.id, 7);
    if (nxt.id >= total) break;
    cur = nxt;
    swapped = nxt_swapped;
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // no load may land in LDS after the workgroup has given it back
}

// The small tile with its loads issued four K steps ahead (a K step takes 512 clocks of MFMAs, far less than a load takes
// to arrive), one workgroup per compute unit.
template <int BM, int NB, int EPI>
__global__ void __launch_bounds__(256, 1) gemm_tile_deep_kernel(const pt_gemm_args g, int tiles_m, int tiles_n) {
#if defined(__HIP_DEVICE_COMPILE__)
  square_tile_run<BM, NB, EPI>(tiles_m, tiles_n);
#endif
}

#endif  // PT_GEMM_TILE_IMPL_H_
