// Tiled bf16 GEMM kernel for gfx950 (template) and its launcher; see gemm.hip for the overview.  Included by
// gemm.hip (dispatch) and by the gemm_inst_*.hip files, each of which instantiates some epilogue combinations so that
// they compile in parallel.
#pragma once

#include "gemm_route.h"
#include "pf_kernels.h"
#include "pf_device.h"

#include <type_traits>

namespace pf {
namespace gemm {


struct EpiDev {
  const void* bias;
  const void* resid;
  const void* dact_in;
  void* preact_out;
  int32_t gelu, accumulate;
  float scale;
};

// Epilogue for 4 consecutive columns n0..n0+3 of row m.  T = storage type of bias / resid / aux,
// OutT = type of C.  The vector form needs n0+3 < N and N % 4 == 0; the scalar form checks every
// element.
template <typename T, typename OutT>
__device__ __forceinline__ void epilogue4_vec(float v[4], int64_t m, int64_t n0, int64_t N, OutT* C,
                                              const EpiDev& ep) {
  const int64_t off = m * N + n0;
  const T* bias = (const T*)ep.bias;
  const T* resid = (const T*)ep.resid;
  const T* dact = (const T*)ep.dact_in;
  T* pre = (T*)ep.preact_out;
  float t[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) v[j] *= ep.scale;
  if (bias) {
    load4(bias + n0, t);
#pragma unroll
    for (int j = 0; j < 4; ++j) v[j] += t[j];
  }
  if (pre) store4(pre + off, v);
  if (ep.gelu) {
#pragma unroll
    for (int j = 0; j < 4; ++j) v[j] = gelu_as<T>(v[j]);
  }
  if (dact) {
    load4(dact + off, t);
#pragma unroll
    for (int j = 0; j < 4; ++j) v[j] *= gelu_grad_f(t[j]);
  }
  if (resid) {
    load4(resid + off, t);
#pragma unroll
    for (int j = 0; j < 4; ++j) v[j] += t[j];
  }
  if (ep.accumulate) {
    load4(C + off, t);
#pragma unroll
    for (int j = 0; j < 4; ++j) v[j] += t[j];
  }
  store4(C + off, v);
}

template <typename T, typename OutT>
__device__ __forceinline__ void epilogue4_scalar(float v[4], int64_t m, int64_t n0, int64_t M, int64_t N, OutT* C,
                                                 const EpiDev& ep) {
  if (m >= M) return;
  const int64_t off = m * N + n0;
  const T* bias = (const T*)ep.bias;
  const T* resid = (const T*)ep.resid;
  const T* dact = (const T*)ep.dact_in;
  T* pre = (T*)ep.preact_out;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    if (n0 + j < N) {
      float x = v[j] * ep.scale;
      if (bias) x += to_f32(bias[n0 + j]);
      if (pre) pre[off + j] = from_f32<T>(x);
      if (ep.gelu) x = gelu_as<T>(x);
      if (dact) x *= gelu_grad_f(to_f32(dact[off + j]));
      if (resid) x += to_f32(resid[off + j]);
      if (ep.accumulate) x += to_f32(C[off + j]);
      C[off + j] = from_f32<OutT>(x);
    }
  }
}

// Ring kernel (gemm_ring.hip).  Needs K a whole number of 16-byte chunks and 16-byte aligned X and W.
template <typename T, typename OutT>
hipError_t launch_ring_shape(Kernel shape, const void* X, const void* W, void* C, int64_t M, int64_t N, int64_t K,
                             const EpiDev& ep, hipStream_t stream);

// compile-time loop: f(integral_constant<int, I>) for I in [0, N)
template <int I, int N, class F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    static_for<I + 1, N>(f);
  }
}


// ------------------------------------------------------------------------------------------------
typedef __attribute__((address_space(3))) void* lds_ptr_t;

// The LDS tables of the staged epilogues, behind the two operand stages; every workgroup builds its copy before the
// K loop, whose barriers publish it.
// GELU for bf16 results by table: h(x) = gelu(x) - max(x, 0) is bounded and vanishes at both ends; 1024 segments
// of 1/64 on [-8, 8), value and slope per segment, linear interpolation (error below 2.5e-5, a hundredth of a bf16
// ulp at 1).  The same for GELU' (between -0.13 and 1.13, 0 and 1 beyond the ends), where the saved
// pre-activation is bf16.
template <int NW, typename OutT, int EPI>
__device__ __forceinline__ void build_epilogue_tables(float2* gelu_tab) {
  constexpr bool GELU_TAB = std::is_same<OutT, bf16_t>::value && (EPI & E_GELU) && !(EPI & E_ACC) && NW >= 8;
  if constexpr (GELU_TAB) {
    for (int e = threadIdx.x; e < 1024; e += 64 * NW) {
      const float x0 = -8.0f + (float)e * (1.0f / 64.0f), x1 = x0 + 1.0f / 64.0f;
      const float h0 = gelu_f(x0) - fmaxf(x0, 0.f), h1 = gelu_f(x1) - fmaxf(x1, 0.f);
      gelu_tab[e] = make_float2(h0, h1 - h0);
    }
  }
  constexpr bool GRAD_TAB = std::is_same<OutT, bf16_t>::value && EPI == E_DACT;
  if constexpr (GRAD_TAB) {
    for (int e = threadIdx.x; e < 1024; e += 64 * NW) {
      const float x0 = -8.0f + (float)e * (1.0f / 64.0f);
      const float d0 = gelu_grad_f(x0), d1 = gelu_grad_f(x0 + 1.0f / 64.0f);
      gelu_tab[e] = make_float2(d0, d1 - d0);
    }
  }
}

// The accumulators of a wave: TN x TM blocks of 32 x 32, W rows (columns of C) by X rows (rows of C), from MFMAs of either
// shape.  A lane has four quads of four consecutive columns in a block: quad q of block (a, b) lies in row row(b, q) and at
// column 4 * unit(a, q) of the wave's part of the tile.
//   32x32x16: D[i][j], lane holds j = lane % 32 (row of C) and i = 8 * q + 4 * (lane / 32) + r (column of C)
//   16x16x32: four 16x16 blocks, q = 2 * (column half) + row half; j = lane % 16, i = 4 * (lane / 16) + r
// slot, half: unit / 2 and unit % 2 (where the lane has no part in the slot, its swizzled place is one scalar expression per row:
// 15724 x 1728, K = 384 with GELU and copy 55.1 us by the unit, 52.6 this way).
// Indices must be compile-time constants or the accumulators leave the register file.
template <int SH, int TM, int TN>
struct Accumulators;
template <int TM, int TN>
struct Accumulators<32, TM, TN> {
  f32x16 v[TN][TM];
  template <class A, class B, class Q>
  __device__ __forceinline__ f32x4 quad(A a, B b, Q q) const {
    constexpr int o = decltype(q)::value * 4;
    const f32x16& t = v[decltype(a)::value][decltype(b)::value];
    return f32x4{t[o], t[o + 1], t[o + 2], t[o + 3]};
  }
  template <class A, class B, class Q>
  __device__ __forceinline__ void scale(A a, B b, Q q, f32x4 f) {
    constexpr int o = decltype(q)::value * 4;
#pragma unroll
    for (int r = 0; r < 4; ++r) v[decltype(a)::value][decltype(b)::value][o + r] *= f[r];
  }
  static __device__ __forceinline__ int row(int b, int, int lane) { return b * 32 + (lane & 31); }
  static __device__ __forceinline__ int unit(int a, int q, int lane) { return a * 8 + q * 2 + (lane >> 5); }
  static __device__ __forceinline__ int slot(int a, int q, int) { return a * 4 + q; }
  static __device__ __forceinline__ int half(int lane) { return lane >> 5; }
};
template <int TM, int TN>
struct Accumulators<16, TM, TN> {
  f32x4 v[2 * TN][2 * TM];
  template <class A, class B, class Q>
  __device__ __forceinline__ f32x4 quad(A a, B b, Q q) const {
    constexpr int qq = decltype(q)::value;
    return v[2 * decltype(a)::value + qq / 2][2 * decltype(b)::value + qq % 2];
  }
  template <class A, class B, class Q>
  __device__ __forceinline__ void scale(A a, B b, Q q, f32x4 f) {
    constexpr int qq = decltype(q)::value;
#pragma unroll
    for (int r = 0; r < 4; ++r) v[2 * decltype(a)::value + qq / 2][2 * decltype(b)::value + qq % 2][r] *= f[r];
  }
  static __device__ __forceinline__ int row(int b, int q, int lane) { return b * 32 + (q & 1) * 16 + (lane & 15); }
  static __device__ __forceinline__ int unit(int a, int q, int lane) { return a * 8 + (q >> 1) * 4 + (lane >> 4); }
  static __device__ __forceinline__ int slot(int a, int q, int lane) { return a * 4 + (q >> 1) * 2 + (lane >> 5); }
  static __device__ __forceinline__ int half(int lane) { return lane >> 4 & 1; }
};

// What a workgroup does with its finished accumulators: block (a, b) lies at rows (wm * TM + b) * 32, columns
// (wn * TN + a) * 32 of the BM x BN tile at (m0, n0).  smem: the two operand stages (free after the K loop)
// followed by the table of build_epilogue_tables.
template <int WGM, int WGN, int TM, int TN, typename OutT, int EPI, int NS = 2, int SH>
__device__ __forceinline__ void tile_epilogue(Accumulators<SH, TM, TN>& acc, uint4* smem, OutT* __restrict__ C, int64_t M,
                                              int64_t N, const EpiDev& ep, int64_t m0, int64_t n0) {
  typedef Accumulators<SH, TM, TN> Acc;
  constexpr int BM = WGM * TM * 32, BN = WGN * TN * 32, NW = WGM * WGN;
  constexpr int STAGE = (BM + BN) * 8;
  float2* gelu_tab = (float2*)(smem + NS * STAGE);
  auto gelu_grad_tab = [&](float x) {
    const float u = __builtin_amdgcn_fmed3f(fmaf(x, 64.0f, 512.0f), 0.0f, 1023.996f);
    const float2 e = gelu_tab[(int)u];
    return fmaf(e.y, __builtin_amdgcn_fractf(u), e.x);
  };
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave % WGM, wn = wave / WGM;
  const bool interior = (m0 + BM <= M) && (n0 + BN <= N) && ((N & 3) == 0);
  // Split K: the fp32 tile goes through LDS (row-major, 16-byte units XOR-swizzled by row) and is added to C with
  // hardware fp32 atomics, 64 consecutive columns of a row per wave instruction.  A lane-per-row atomic would touch 32
  // cache lines per instruction.  Only tiles whose fp32 image fits the two LDS stages split K (the launcher knows).
  if constexpr (std::is_same<OutT, float>::value && EPI == E_ACC && BM * BN * 4 <= 2 * STAGE * 16) {
    if (gridDim.y > 1) {
      float* stf = (float*)smem;
      constexpr int UNITS = BN / 4, NT = 64 * NW;
      static_for<0, TN>([&](auto a) {
        static_for<0, TM>([&](auto b) {
          static_for<0, 4>([&](auto q) {
            const int row = Acc::row(wm * TM + b, q, lane), unit = Acc::unit(wn * TN + a, q, lane);
            *(f32x4*)(stf + row * BN + ((unit ^ (row & (UNITS - 1))) * 4)) = acc.quad(a, b, q);
          });
        });
      });
      __builtin_amdgcn_s_waitcnt(0xc07f);
      __builtin_amdgcn_s_barrier();
#pragma unroll 8
      for (int i = 0; i < BM * BN / NT; ++i) {
        const int e = i * NT + tid, row = e / BN, col = e % BN;
        const float v = stf[row * BN + (((col >> 2) ^ (row & (UNITS - 1))) * 4) + (col & 3)];
        if (m0 + row < M && n0 + col < N) unsafeAtomicAdd((float*)C + (m0 + row) * N + n0 + col, v);
      }
      return;
    }
  }
  // Staged epilogue (bf16 output): bias and GELU are applied in registers, the bf16 tile goes through LDS (free
  // after the K loop; 16-byte slots XOR-swizzled by row) and leaves as 16-byte stores that cover whole rows of the
  // tile, the residual being added on the way out from equally coalesced loads.  The two training forms use the same
  // route: the pre-activation is a second tile staged and stored before the activated one, and the saved tensor whose
  // GELU' multiplies the result comes in the other way round, coalesced loads -> LDS -> the accumulator layout.
  // Not the residual of the kernels with three stages or more: the route by fp32 rows below rounds once and is no slower
  // (1659 x 768, K = 768 10.0 -> 9.8 us, 2048 x 2048, K = 2048 22 -> 21).
  constexpr bool STAGED = std::is_same<OutT, bf16_t>::value && !(EPI & E_ACC) && !((EPI & E_RESID) && NS > 2);
  if constexpr (STAGED) {
    static_assert(!(EPI & E_DACT) || EPI == E_DACT, "GELU' multiplies the plain product only");
    const bool aligned16 = ((N & 7) == 0) && ((((uintptr_t)C | (uintptr_t)ep.resid | (uintptr_t)ep.preact_out |
                                                 (uintptr_t)ep.dact_in) & 15) == 0);
    if (interior && aligned16 && N <= (1 << 21)) {
      constexpr int SLOTS = BN / 8, NT = 64 * NW, PER = BM * BN / 8 / NT;
      // 16-byte slot of a row, moved per row so that the lanes of a wave (32 rows, same column group) spread
      // over the banks: XOR when the slot count is a power of two, rotation otherwise
      auto swz = [](int slot, int row) {
        if constexpr ((SLOTS & (SLOTS - 1)) == 0) return slot ^ (row & (SLOTS - 1));
        else return (slot + row) % SLOTS;
      };
      uint2* st8 = (uint2*)smem;
      // Piece i of a thread on the way out (and of the residual on the way in): 16 bytes of row i * RP + r0 when the
      // threads of a workgroup cover whole rows.  The tile's corner is the base of a raw buffer, the thread's place a
      // 32-bit offset computed once, the rows of piece i a scalar offset (N <= 2^21 keeps all of it below 2^31): no
      // 64-bit vector arithmetic per piece, which is what a lone wave per SIMD has least of.
      typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
      constexpr bool ROWWISE = NT % SLOTS == 0;
      constexpr int RP = ROWWISE ? NT / SLOTS : 1;
      const int r0 = tid / SLOTS, slot0 = tid % SLOTS;
      const int voff = (int)((r0 * N + slot0 * 8) * 2);
      auto tile_rsrc = [&](const void* p) {
        return __builtin_amdgcn_make_buffer_rsrc((void*)((const bf16_t*)p + m0 * N + n0), 0, 0x7fffffff, 0x00020000);
      };
      auto lds_at = [&](int i) {
        if constexpr (ROWWISE) {
          const int row = i * RP + r0;
          return row * SLOTS + swz(slot0, row);
        } else {
          const int q = i * NT + tid, row = q / SLOTS, slot = q % SLOTS;
          return row * SLOTS + swz(slot, row);
        }
      };
      auto piece_load = [&](__amdgpu_buffer_rsrc_t rs, const void* p, int i) -> uint4 {
        if constexpr (ROWWISE) {
          const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(rs, voff, (int)(i * RP * N * 2), 0);
          return make_uint4(v[0], v[1], v[2], v[3]);
        } else {
          const int q = i * NT + tid, row = q / SLOTS, slot = q % SLOTS;
          return *(const uint4*)((const bf16_t*)p + (m0 + row) * N + n0 + slot * 8);
        }
      };
      auto piece_store = [&](__amdgpu_buffer_rsrc_t rs, void* p, int i, uint4 v) {
        if constexpr (ROWWISE) {
          const u32x4 w = {v.x, v.y, v.z, v.w};
          __builtin_amdgcn_raw_buffer_store_b128(w, rs, voff, (int)(i * RP * N * 2), 0);
        } else {
          const int q = i * NT + tid, row = q / SLOTS, slot = q % SLOTS;
          *(uint4*)((bf16_t*)p + (m0 + row) * N + n0 + slot * 8) = v;
        }
      };
      if constexpr (EPI & E_DACT) {
        // tile of the saved pre-activation: eight 16-byte pieces per thread at a time (more would not fit beside
        // the accumulators), then every lane picks up the values of its own accumulator elements
        constexpr int CH = PER < 8 ? PER : 8;
#pragma unroll
        for (int i0 = 0; i0 < PER; i0 += CH) {
          uint4 t[CH];
#pragma unroll
          for (int i = 0; i < CH; ++i) {
            if (i0 + i < PER) {
              const int q = (i0 + i) * NT + tid, row = q / SLOTS, slot = q % SLOTS;
              t[i] = *(const uint4*)((const bf16_t*)ep.dact_in + (m0 + row) * N + n0 + slot * 8);
            }
          }
#pragma unroll
          for (int i = 0; i < CH; ++i) {
            if (i0 + i < PER) {
              const int q = (i0 + i) * NT + tid, row = q / SLOTS, slot = q % SLOTS;
              smem[row * SLOTS + swz(slot, row)] = t[i];
            }
          }
        }
        __builtin_amdgcn_s_waitcnt(0xc07f);
        __builtin_amdgcn_s_barrier();
        static_for<0, TN>([&](auto a) {
          static_for<0, TM>([&](auto b) {
            static_for<0, 4>([&](auto q) {
              const int row = Acc::row(wm * TM + b, q, lane);
              const uint2 u = st8[row * (SLOTS * 2) + swz(Acc::slot(wn * TN + a, q, lane), row) * 2 + Acc::half(lane)];
              const f32x4 f = {gelu_grad_tab(bf16_bits_to_f32(u.x & 0xffffu)), gelu_grad_tab(bf16_bits_to_f32(u.x >> 16)),
                               gelu_grad_tab(bf16_bits_to_f32(u.y & 0xffffu)), gelu_grad_tab(bf16_bits_to_f32(u.y >> 16))};
              acc.scale(a, b, q, f);
            });
          });
        });
        __builtin_amdgcn_s_waitcnt(0xc07f);
        __builtin_amdgcn_s_barrier();   // everyone has its values: the tile's place in LDS is free again
      }
      // accumulators (+ bias) (-> GELU) -> bf16 -> LDS in the swizzled row-major layout
      auto stage_tile = [&](auto with_gelu) {
        static_for<0, TN>([&](auto a) {
          float bias4[4][4] = {};
          if constexpr (EPI & E_BIAS) {
#pragma unroll
            for (int q = 0; q < 4; ++q)
              if (SH == 32 || q % 2 == 0) load4((const bf16_t*)ep.bias + n0 + Acc::unit(wn * TN + a, q, lane) * 4, bias4[q]);
          }
          static_for<0, TM>([&](auto b) {
            static_for<0, 4>([&](auto q) {
              constexpr int bq = SH == 32 ? decltype(q)::value : decltype(q)::value & 2;   // quads of one column share the bias
              const int row = Acc::row(wm * TM + b, q, lane);
              const f32x4 t = acc.quad(a, b, q);
              float v[4] = {t[0], t[1], t[2], t[3]};
              if constexpr (EPI & E_BIAS) {
#pragma unroll
                for (int j = 0; j < 4; ++j) v[j] += bias4[bq][j];
              }
              if constexpr (decltype(with_gelu)::value) {
                // Eight waves: GELU from the table (9.5 VALU slots and one LDS gather per element; the second wave of
                // the SIMD covers the gather's latency).  Four waves, one per SIMD: nothing covers it, and the
                // arithmetic form (one exp2 and one reciprocal per element) is the faster one.
                if constexpr (NW >= 8) {
#pragma unroll
                  for (int j = 0; j < 4; ++j) {
                    const float u = __builtin_amdgcn_fmed3f(fmaf(v[j], 64.0f, 512.0f), 0.0f, 1023.996f);
                    const float2 e = gelu_tab[(int)u];
                    v[j] = fmaxf(v[j], 0.f) + fmaf(e.y, __builtin_amdgcn_fractf(u), e.x);
                  }
                } else {
#pragma unroll
                  for (int j = 0; j < 4; ++j) v[j] = gelu_bf16_f(v[j]);
                }
              }
              uint2 pk;
              pk.x = pack_bf16x2(v[0], v[1]);
              pk.y = pack_bf16x2(v[2], v[3]);
              st8[row * (SLOTS * 2) + swz(Acc::slot(wn * TN + a, q, lane), row) * 2 + Acc::half(lane)] = pk;
            });
          });
        });
      };
      if constexpr (EPI & E_PRE) {   // the value before the activation leaves first, the same way
        stage_tile(std::false_type{});
        __builtin_amdgcn_s_waitcnt(0xc07f);
        __builtin_amdgcn_s_barrier();
        const __amdgpu_buffer_rsrc_t prsrc = tile_rsrc(ep.preact_out);
#pragma unroll
        for (int i = 0; i < PER; ++i) piece_store(prsrc, ep.preact_out, i, smem[lds_at(i)]);
        __builtin_amdgcn_s_waitcnt(0xc07f);
        __builtin_amdgcn_s_barrier();
      }
      // the residual tile is requested first, in the layout of the final stores, so that it arrives while the
      // accumulators go through bias / GELU / LDS
      constexpr int EARLY = PER < 8 ? PER : 8;   // more would not fit beside the accumulators
      uint4 rres[(EPI & E_RESID) ? PER : 1];
      const __amdgpu_buffer_rsrc_t rrsrc = tile_rsrc((EPI & E_RESID) ? ep.resid : (const void*)C);
      if constexpr (EPI & E_RESID) {
#pragma unroll
        for (int i = 0; i < EARLY; ++i) rres[i] = piece_load(rrsrc, ep.resid, i);
      }
      stage_tile(std::integral_constant<bool, (EPI & E_GELU) != 0>{});
      if constexpr (EPI & E_RESID) {   // the accumulators are dead now: the rest of the residual tile
#pragma unroll
        for (int i = EARLY; i < PER; ++i) rres[i] = piece_load(rrsrc, ep.resid, i);
      }
      __builtin_amdgcn_s_waitcnt(0xc07f);
      __builtin_amdgcn_s_barrier();
      const __amdgpu_buffer_rsrc_t crsrc = tile_rsrc(C);
#pragma unroll
      for (int i = 0; i < PER; ++i) {
        uint4 v = smem[lds_at(i)];
        if constexpr (EPI & E_RESID) {
          const uint4 r = rres[i];
          const uint32_t vw[4] = {v.x, v.y, v.z, v.w}, rw[4] = {r.x, r.y, r.z, r.w};
          uint32_t ow[4];
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const float lo = bf16_bits_to_f32(vw[j] & 0xffffu) + bf16_bits_to_f32(rw[j] & 0xffffu);
            const float hi = bf16_bits_to_f32(vw[j] >> 16) + bf16_bits_to_f32(rw[j] >> 16);
            ow[j] = pack_bf16x2(lo, hi);
          }
          v = make_uint4(ow[0], ow[1], ow[2], ow[3]);
        }
        piece_store(crsrc, C, i, v);
      }
      return;
    }
  }
  // Everything else (fp32 results, bf16 tiles that stick out of C, operands or rows that are not aligned): the lanes of a
  // wave hold 32 rows, so going through memory from the registers would touch 32 rows in small pieces per instruction.
  // Instead each wave passes its 32-row blocks one by one, still in fp32, through a corner of LDS of its own (no barrier)
  // and goes through C and the other operands of the epilogue in whole rows of its tile.  A bf16 element takes the steps of
  // epilogue4_scalar: fp32, rounded once at the end, the formulas of GELU and GELU' (the staged route above rounds product +
  // bias before it adds the residual).
  //  * In pieces of 16 bytes (bf16 also 8) where rows and operands are aligned to them; what a block needs from memory is
  //    requested before it is staged.  Rows and columns past C's end are dropped by the buffers' bounds: loads deliver zeros,
  //    stores go nowhere.  8192 x 32768, K = 2048 accumulated into fp32: 1446 us from the registers, 1102 this way (1 GiB
  //    read, 1 GiB written).  From the registers a ragged bf16 result took 25 to 85 us longer than a whole one: 1659 x 768,
  //    K = 768 38 / 55 / 106 us with the 128- / 192- / 256-wide tiles, where 4096 x 768 took 14 / 20 / 21.
  //  * Otherwise element by element, what is read from memory for four groups of four columns at a time.
  constexpr bool F32 = std::is_same<OutT, float>::value;
  constexpr int UNITS = TN * 8;                             // 16-byte units of a row in LDS
  constexpr int XOR = UNITS % 16 == 0 ? 15 : 7;
  constexpr int OUTSIDE = 0x7fffff00;                       // past every buffer
  static_assert(32 * UNITS * NW <= 2 * STAGE, "a block per wave fits the operand stages");
  static_assert(!F32 || (EPI & ~E_ACC) == 0, "fp32 results have no epilogue but the sum");
  constexpr bool READS = (EPI & (E_ACC | E_RESID | E_DACT)) != 0;   // one operand of C's layout, at most
  const void* const read_from = (EPI & E_ACC) ? (const void*)C : (EPI & E_RESID) ? ep.resid : ep.dact_in;
  float4* st = (float4*)smem + wave * 32 * UNITS;
  const int wmu = __builtin_amdgcn_readfirstlane(wm), wnu = __builtin_amdgcn_readfirstlane(wn);   // scalar buffers
  const int64_t wm0 = m0 + wmu * TM * 32, wn0 = n0 + wnu * TN * 32;
  uintptr_t ptrs = (uintptr_t)C;
  if constexpr (EPI & E_BIAS) ptrs |= (uintptr_t)ep.bias;
  if constexpr (READS) ptrs |= (uintptr_t)read_from;
  if constexpr (EPI & E_PRE) ptrs |= (uintptr_t)ep.preact_out;
  // (the last barrier of the K loop comes after every wave's last read of the operand stages)
  auto stage_block = [&](auto b) {
    asm volatile("" ::: "memory");   // other lanes' values: a wave's LDS instructions execute in program order
    static_for<0, TN>([&](auto a) {
      static_for<0, 4>([&](auto q) {
        const int row = Acc::row(0, q, lane);
        f32x4 t = acc.quad(a, b, q);
        // (copied out one register each: as four-register operands of the LDS store, next to the staged route's reads, the
        // 256 accumulators of the four-wave kernel made the allocator spill 80 of them on every tile)
        float t0 = t[0], t1 = t[1], t2 = t[2], t3 = t[3];
        if constexpr (!F32) asm("" : "+v"(t0), "+v"(t1), "+v"(t2), "+v"(t3));
        st[row * UNITS + (Acc::unit(a, q, lane) ^ (row & XOR))] = make_float4(t0, t1, t2, t3);
      });
    });
    asm volatile("" ::: "memory");
  };
  // an element on its way out, given what was read for it
  auto finish = [&](float x, float read) {
    if constexpr (EPI & E_GELU) x = gelu_bf16_f(x);
    if constexpr (EPI & E_DACT) x *= gelu_grad_f(read);
    else if constexpr (READS) x += read;
    return x;
  };
  auto by_pieces = [&](auto words, auto keep) {
    constexpr int W = decltype(words)::value;                         // of a piece: 32-bit words,
    constexpr int CE = W * 4 / (int)sizeof(OutT), UP = CE / 4;        // columns, units in LDS
    constexpr int SLOTS = TN * 32 / CE, PIECES = SLOTS / 2;           // pieces of a row; wave instructions of a block
    typedef uint32_t piece_t __attribute__((ext_vector_type(W)));
    constexpr int AUX = decltype(keep)::value ? 0 : 2;                // 2: non-temporal
    auto load = [&](__amdgpu_buffer_rsrc_t rs, int off) -> piece_t {
      if constexpr (W == 4) return __builtin_amdgcn_raw_buffer_load_b128(rs, off, 0, AUX);
      else return __builtin_amdgcn_raw_buffer_load_b64(rs, off, 0, AUX);
    };
    auto store = [&](const float* v, __amdgpu_buffer_rsrc_t rs, int off) {
      piece_t w;
#pragma unroll
      for (int j = 0; j < W; ++j) {
        if constexpr (F32) w[j] = __float_as_uint(v[j]);
        else w[j] = pack_bf16x2(v[2 * j], v[2 * j + 1]);
      }
      if constexpr (W == 4) __builtin_amdgcn_raw_buffer_store_b128(w, rs, off, 0, AUX);
      else __builtin_amdgcn_raw_buffer_store_b64(w, rs, off, 0, AUX);
    };
    auto widen = [&](piece_t p, float* v) {
#pragma unroll
      for (int j = 0; j < W; ++j) {
        if constexpr (F32) v[j] = __uint_as_float(p[j]);
        else {
          v[2 * j] = bf16_bits_to_f32(p[j] & 0xffffu);
          v[2 * j + 1] = bf16_bits_to_f32(p[j] >> 16);
        }
      }
    };
    const int ncols = (int)(N - wn0 < TN * 32 ? (N > wn0 ? N - wn0 : 0) : TN * 32);
    const int nrows = (int)(M - wm0 < TM * 32 ? (M > wm0 ? M - wm0 : 0) : TM * 32);
    const int row_bytes = (int)N * (int)sizeof(OutT);
    // block b of the wave in an array of C's layout: a buffer from its first row to its last inside C
    auto block_rsrc = [&](const void* p, int b) {
      const int rows = nrows - b * 32 < 32 ? nrows - b * 32 : 32;
      const bool any = ncols > 0 && rows > 0;
      return __builtin_amdgcn_make_buffer_rsrc((void*)(any ? (const OutT*)p + (wm0 + b * 32) * N + wn0 : (const OutT*)p), 0,
                                               any ? (rows - 1) * row_bytes + ncols * (int)sizeof(OutT) : 0, 0x00020000);
    };
    int voff[PIECES], lds_at[PIECES];
#pragma unroll
    for (int i = 0; i < PIECES; ++i) {
      const int e = i * 64 + lane, row = e / SLOTS, slot = e % SLOTS;
      voff[i] = slot * CE < ncols ? row * row_bytes + slot * W * 4 : OUTSIDE;
      lds_at[i] = row * UNITS + ((slot * UP) ^ (row & XOR));   // second unit of a piece: this ^ 1
    }
    piece_t in[PIECES], bias[PIECES];
    if constexpr (EPI & E_BIAS) {
      const __amdgpu_buffer_rsrc_t brsrc = __builtin_amdgcn_make_buffer_rsrc(
          (void*)((const OutT*)ep.bias + (ncols > 0 ? wn0 : 0)), 0, ncols * (int)sizeof(OutT), 0x00020000);
#pragma unroll
      for (int i = 0; i < PIECES; ++i) bias[i] = load(brsrc, (i * 64 + lane) % SLOTS * W * 4);
    }
    static_for<0, TM>([&](auto b) {
      if constexpr (READS) {
        const __amdgpu_buffer_rsrc_t irsrc = block_rsrc(read_from, b);
#pragma unroll
        for (int i = 0; i < PIECES; ++i) in[i] = load(irsrc, voff[i]);
      }
      stage_block(b);
      const __amdgpu_buffer_rsrc_t crsrc = block_rsrc(C, b);
#pragma unroll
      for (int i = 0; i < PIECES; ++i) {
        float v[CE], t[CE] = {};
#pragma unroll
        for (int j = 0; j < UP; ++j) {
          const float4 u = st[lds_at[i] ^ j];
          v[4 * j] = u.x; v[4 * j + 1] = u.y; v[4 * j + 2] = u.z; v[4 * j + 3] = u.w;
        }
        if constexpr (EPI & E_BIAS) {
          widen(bias[i], t);
#pragma unroll
          for (int j = 0; j < CE; ++j) v[j] += t[j];
        }
        if constexpr (EPI & E_PRE) store(v, block_rsrc(ep.preact_out, b), voff[i]);
        if constexpr (READS) widen(in[i], t);
#pragma unroll
        for (int j = 0; j < CE; ++j) v[j] = finish(v[j], t[j]);
        store(v, crsrc, voff[i]);
      }
    });
  };
  if (N <= (1 << 23)) {   // 32 rows of C below 2^31 bytes
    if (N % (16 / (int)sizeof(OutT)) == 0 && (ptrs & 15) == 0) {
      // An accumulated C that no cache holds until it is read again (the memory-side cache has 256 MB) goes past them: 32768 x
      // 8192, K = 2048 (1 GB) 1115 -> 1030 us, 24576 x 8192 (805 MB) 829 -> 774; 8192 x 8192 (268 MB) loses, 292 -> 312.
      if constexpr ((EPI & E_ACC) != 0) {
        if (M * N >= (int64_t)96 << 20) {
          by_pieces(std::integral_constant<int, 4>{}, std::false_type{});
          return;
        }
      }
      by_pieces(std::integral_constant<int, 4>{}, std::true_type{});
      return;
    }
    if constexpr (!F32) {
      if (N % 4 == 0 && (ptrs & 7) == 0) {
        by_pieces(std::integral_constant<int, 2>{}, std::true_type{});
        return;
      }
    }
  }
  static_for<0, TM>([&](auto b) {
    stage_block(b);
#pragma unroll 1
    for (int i = 0; i < UNITS / 2; i += 4) {
      float t[4][4] = {};
      if constexpr (READS) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int e = (i + u) * 64 + lane;
          const int64_t m = wm0 + b * 32 + e / UNITS, n = wn0 + e % UNITS * 4;
#pragma unroll
          for (int j = 0; j < 4; ++j)
            if (m < M && n + j < N) t[u][j] = to_f32(((const OutT*)read_from)[m * N + n + j]);
        }
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int e = (i + u) * 64 + lane, row = e / UNITS, unit = e % UNITS;
        const int64_t m = wm0 + b * 32 + row, n = wn0 + unit * 4;
        const float4 s = st[row * UNITS + (unit ^ (row & XOR))];
        const float v[4] = {s.x, s.y, s.z, s.w};
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          if (m >= M || n + j >= N) continue;
          float x = v[j];
          if constexpr (EPI & E_BIAS) x += to_f32(((const OutT*)ep.bias)[n + j]);
          if constexpr (EPI & E_PRE) ((OutT*)ep.preact_out)[m * N + n + j] = from_f32<OutT>(x);
          C[m * N + n + j] = from_f32<OutT>(finish(x, t[u][j]));
        }
      }
    }
  });
}

__device__ __forceinline__ f32x16 mfma_bf16(bf16x8 w, bf16x8 x, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(w, x, c, 0, 0, 0);
}
__device__ __forceinline__ f32x4 mfma_bf16(bf16x8 w, bf16x8 x, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(w, x, c, 0, 0, 0);
}

// 256x192 tile on eight waves (4x2, wave tile 64x96, two per SIMD), 32x32x16 MFMAs (inside a 12-layer encoder pass 16384 x 768,
// K = 3072 takes 71.8 us with these and 74.1 with 16x16x32).
template <int WGM, int WGN, int TM, int TN, typename OutT, int EPI>
__global__ __launch_bounds__(64 * WGM * WGN) void gemm_bf16_nt_kernel(
    const bf16_t* __restrict__ X, const bf16_t* __restrict__ W, OutT* __restrict__ C, int64_t M, int64_t N,
    int64_t K, EpiDev ep, int32_t tiles_m, int32_t tiles_n, int32_t group_m) {
  constexpr int BM = WGM * TM * 32, BN = WGN * TN * 32, NW = WGM * WGN;
  constexpr int GX = BM / 8, G = (BM + BN) / 8, GPW = G / NW;   // 8-row groups of 1 KB; per wave
  constexpr int STAGE = (BM + BN) * 8;                          // uint4 per LDS stage
  static_assert(G % NW == 0 && GPW <= 32, "tile / wave mismatch");
  extern __shared__ uint4 smem[];
  build_epilogue_tables<NW, OutT, EPI>((float2*)(smem + 2 * STAGE));
  const int64_t tile = xcd_contiguous(blockIdx.x, (int64_t)tiles_m * tiles_n);
  const int64_t per_group = (int64_t)group_m * tiles_n;
  const int64_t grp = tile / per_group;
  const int32_t first_m = (int32_t)(grp * group_m);
  const int32_t rows_in_group = (tiles_m - first_m < group_m) ? tiles_m - first_m : group_m;
  const int32_t tm_i = first_m + (int32_t)((tile % per_group) % rows_in_group);
  const int32_t tn_i = (int32_t)((tile % per_group) / rows_in_group);
  const int64_t m0 = (int64_t)tm_i * BM, n0 = (int64_t)tn_i * BN;

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave % WGM, wn = wave / WGM;
  const int lr = lane & 31, lg = lane >> 5;

  // global source of this lane for each 1 KB group the wave moves per K step
  const bf16_t* src[GPW];
#pragma unroll
  for (int i = 0; i < GPW; ++i) {
    const int g = wave + i * NW;
    const bool isx = g < GX;
    const int r = (isx ? g : g - GX) * 8 + (lane >> 3);
    const int c = (lane & 7) ^ ((r >> 1) & 7);
    int64_t row = (isx ? m0 : n0) + r;
    const int64_t lim = isx ? M : N;
    if (row >= lim) row = lim - 1;
    src[i] = (isx ? X : W) + row * K + c * 8;
  }
  const uint32_t lds_base = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(lds_ptr_t)smem);
  // one 1 KB group of the stage at k0 straight into LDS stage `stage` (M0 carries the LDS address)
  auto issue1 = [&](auto ic, int stage, int64_t k0) {
    constexpr int i = decltype(ic)::value;
    const int g = wave + i * NW;
    const uint32_t dst = __builtin_amdgcn_readfirstlane(lds_base + (uint32_t)((stage * STAGE + g * 64) * 16));
    const bf16_t* p = src[i] + k0;
    lds_direct_load_1k(dst, p);
  };
  // A slice is 16 wide in k (one MFMA), a fragment 32 rows of it: the lane takes chunk 2 kk + lane / 32 of row lane % 32.
  // Fragments start at multiples of 32 rows, so all of a lane's have the same swizzle.
  const int sw = (lr >> 1) & 7;
  const int offW = BM * 8 + (wn * TN * 32 + lr) * 8, offX = (wm * TM * 32 + lr) * 8;
  Accumulators<32, TM, TN> acc;
#pragma unroll
  for (int a = 0; a < TN; ++a)
#pragma unroll
    for (int b = 0; b < TM; ++b)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc.v[a][b][r] = 0.f;
  bf16x8 fw[2][TN], fx[2][TM];
  auto load_frags = [&](int buf, const uint4* st, int kk) {
    const int c = (kk * 2 + lg) ^ sw;
#pragma unroll
    for (int a = 0; a < TN; ++a) fw[buf][a] = as_bf16x8(st[offW + a * 256 + c]);
#pragma unroll
    for (int b = 0; b < TM; ++b) fx[buf][b] = as_bf16x8(st[offX + b * 256 + c]);
  };
  // A burst of loads right after the barrier blocks every wave at the texture-address unit (1 KB per
  // instruction at 64 B/clk) while the MFMA pipe drains; instead one load is issued before every EVERY-th
  // MFMA of the block after the barrier (index 0) and of the blocks that follow, over three quarters of a K step.
  constexpr int MF = TM * TN, SPAN = 3 * MF, EVERY = SPAN / GPW;
  static_assert(EVERY >= 1 && EVERY * GPW <= SPAN, "load slots");
  auto mfma_block = [&](auto blkc, auto bufc, bool do_load, int stage, int64_t k0) {
    constexpr int blk = decltype(blkc)::value, buf = decltype(bufc)::value;
    static_for<0, MF>([&](auto mi) {
      constexpr int g = blk * MF + mi;
      if constexpr (g % EVERY == 0 && g / EVERY < GPW) {
        if (do_load) issue1(std::integral_constant<int, g / EVERY>{}, stage, k0);
      }
      constexpr int a = mi / TM, b = mi % TM;
      acc.v[a][b] = mfma_bf16(fw[buf][a], fx[buf][b], acc.v[a][b]);
    });
  };
  using I0 = std::integral_constant<int, 0>;
  using I1 = std::integral_constant<int, 1>;

  const int64_t nk = K / 64;
  // prologue: stage 0 completely; of stage 1 the share the block after a barrier issues
  static_for<0, GPW>([&](auto i) { issue1(i, 0, 0); });
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();
  if (nk > 1) {
    static_for<0, MF>([&](auto mi) {
      if constexpr (mi % EVERY == 0 && mi / EVERY < GPW) issue1(std::integral_constant<int, mi / EVERY>{}, 1, 64);
    });
  }
  load_frags(0, smem, 0);
  for (int64_t kt = 0; kt < nk; ++kt) {
    const int cur = (int)(kt & 1);
    const uint4* sc = smem + cur * STAGE;
    const uint4* sn = smem + (cur ^ 1) * STAGE;
    const bool more1 = kt + 1 < nk, more2 = kt + 2 < nk;
    const int64_t k1 = (kt + 1) * 64;
    __builtin_amdgcn_s_waitcnt(0xc07f);   // lgkmcnt(0): fragments fetched during the previous MFMA block
    static_for<1, 4>([&](auto sl) {
      load_frags(sl & 1, sc, sl);
      __builtin_amdgcn_sched_barrier(0);
      mfma_block(sl, std::integral_constant<int, (sl & 1) ^ 1>{}, more1, cur ^ 1, k1);
      __builtin_amdgcn_sched_barrier(0);
    });
    // every wave holds the last fragments of this stage in registers and the next stage has landed
    __builtin_amdgcn_s_waitcnt(0x0070);   // vmcnt(0) lgkmcnt(0)
    __builtin_amdgcn_s_barrier();
    if (kt + 1 < nk) load_frags(0, sn, 0);
    __builtin_amdgcn_sched_barrier(0);
    mfma_block(I0{}, I1{}, more2, cur, (kt + 2) * 64);   // stage `cur` is free: start refilling it
    __builtin_amdgcn_sched_barrier(0);
  }

  tile_epilogue<WGM, WGN, TM, TN, OutT, EPI>(acc, smem, C, M, N, ep, m0, n0);
}

// Four waves with room in the register file: the fragments of a WHOLE K step are double buffered.  While the MFMAs of step kt
// run on one set, they are interleaved with the LDS reads that fill the other set with step kt + 1 and with the copies of
// step kt + NS into the stage that step kt's reads have left.  One barrier a step, behind its first MFMAs (LAG), which cover
// the reads that are still on their way there.  No MFMA waits for an LDS read of its own step; with a slice's reads in flight
// at a time (the loop above, and what these tiles ran on before) a lone wave per SIMD waits for LDS at every slice, and that
// wait, not memory, bound these tiles (every operand out of L2 changes their times by 5 %).
//   128x128, four stages, a CU to itself (32x32x16 MFMAs): 0.61 -> 0.36 to 0.5 us a step, 333 x 6144, K = 2048 24.4 -> 16.3 us,
//     2048 x 2048, K = 2048 29 -> 20.5, 1659 x 2304, K = 768 13.5 -> 10.7
//   128x128, two stages, two workgroups per CU (16x16x32 MFMAs): 8192 x 1024, K = 4096 75 -> 59 us, 8192 x 4096, K = 1024 with
//     GELU' 96 -> 82, 1659 x 3072, K = 768 with GELU 19.2 -> 16.7
//   128x64 (wave tile 64x32), six stages (32x32x16), half as many products a step on twice the CUs: 1659 x 768, K = 3072 22.6 us on
//     128x128 tiles, 18.6 here
//   256x128 (wave tile 128x64), three stages (32x32x16): fewer operand bytes per product, for long K: 8192 x 1024, K = 50304
//     858 us on 128x128 tiles, 725 here
// Which MFMA: a full chip runs into the power limit, where 16x16x32 sustains more (2.1 against 1.82 PFLOP/s in a loop of
// nothing else on random operands: half the accumulator traffic per product); a lone wave per SIMD needs the longer MFMA to
// hide what it issues between two of them (333 x 6144, K = 2048 16.3 us on 32x32x16, 20.9 on 16x16x32).
template <int WGM, int WGN, int TM, int TN, typename OutT, int EPI, int NS, int SH>
__global__ __launch_bounds__(64 * WGM * WGN, TM * TN <= 4 && NS == 2 ? 2 : 1) void gemm_bf16_nt_step_kernel(
    const bf16_t* __restrict__ X, const bf16_t* __restrict__ W, OutT* __restrict__ C, int64_t M, int64_t N,
    int64_t K, EpiDev ep, int32_t tiles_m, int32_t tiles_n, int32_t group_m) {
  constexpr int BM = WGM * TM * 32, BN = WGN * TN * 32, NW = WGM * WGN;
  constexpr int GX = BM / 8, G = (BM + BN) / 8, GPW = G / NW;   // 8-row groups of 1 KB; per wave
  constexpr int STAGE = (BM + BN) * 8;                          // uint4 per LDS stage
  static_assert(G % NW == 0 && GX % NW == 0, "tile / wave mismatch");
  static_assert(GPW * (NS - 1) < 64, "vmcnt holds six bits");
  extern __shared__ uint4 smem[];
  build_epilogue_tables<NW, OutT, EPI>((float2*)(smem + NS * STAGE));
  const int64_t tile = xcd_contiguous(blockIdx.x, (int64_t)tiles_m * tiles_n);
  const int64_t per_group = (int64_t)group_m * tiles_n;
  const int64_t grp = tile / per_group;
  const int32_t first_m = (int32_t)(grp * group_m);
  const int32_t rows_in_group = (tiles_m - first_m < group_m) ? tiles_m - first_m : group_m;
  const int32_t tm_i = first_m + (int32_t)((tile % per_group) % rows_in_group);
  const int32_t tn_i = (int32_t)((tile % per_group) / rows_in_group);
  const int64_t m0 = (int64_t)tm_i * BM, n0 = (int64_t)tn_i * BN;

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave % WGM, wn = wave / WGM;
  const int lr = lane & (SH - 1), lg = lane / SH;

  // split K (accumulating fp32 epilogue only): workgroup y works on columns [y, y+1) * K / gridDim.y of both operands
  const int64_t k_len = K / gridDim.y;
  X += (int64_t)blockIdx.y * k_len;
  W += (int64_t)blockIdx.y * k_len;

  // Copies: the tile's first row is the base of a raw buffer, the lane's place a 32-bit offset (rows past the end repeat
  // the last one), the K step a scalar offset.
  uint32_t off[GPW];
#pragma unroll
  for (int i = 0; i < GPW; ++i) {
    const bool isx = i < GX / NW;
    const int g = wave + i * NW;
    const int r = (isx ? g : g - GX) * 8 + (lane >> 3);
    const int c = (lane & 7) ^ ((r >> 1) & 7);
    const int64_t last = (isx ? M - m0 : N - n0) - 1;
    const int64_t row = r <= last ? r : last;
    off[i] = (uint32_t)((row * K + c * 8) * 2);
  }
  lds_buffer_t xbuf = lds_buffer(X + m0 * K), wbuf = lds_buffer(W + n0 * K);
  const uint32_t lds_base = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(lds_ptr_t)smem) + (uint32_t)(wave * 1024);
  auto issue1 = [&](auto ic, uint32_t stage_at, int32_t k_bytes) {
    constexpr int i = decltype(ic)::value;
    lds_buffer_load_1k(stage_at + (uint32_t)(i * NW * 1024), i < GX / NW ? xbuf : wbuf, off[i], k_bytes);
  };
  // a slice is KS wide in k (one MFMA), a fragment SH rows of it: the lane takes chunk kk * KS / 8 + lane / SH of row lane % SH
  constexpr int KS = 512 / SH, SLICES = 64 / KS, FM = TM * 32 / SH, FN = TN * 32 / SH;
  const int sw = (lr >> 1) & 7;
  int at_x[SLICES], at_w[SLICES];   // chunk of slice kk in a stage
#pragma unroll
  for (int kk = 0; kk < SLICES; ++kk) {
    const int c = (kk * (KS / 8) + lg) ^ sw;
    at_x[kk] = (wm * TM * 32 + lr) * 8 + c;
    at_w[kk] = BM * 8 + (wn * TN * 32 + lr) * 8 + c;
  }
  Accumulators<SH, TM, TN> acc;
#pragma unroll
  for (int a = 0; a < FN; ++a)
#pragma unroll
    for (int b = 0; b < FM; ++b)
#pragma unroll
      for (int r = 0; r < SH * SH / 64; ++r) acc.v[a][b][r] = 0.f;
  bf16x8 fw[2][SLICES][FN], fx[2][SLICES][FM];
  constexpr int MF = SLICES * FM * FN, NR = SLICES * (FM + FN);   // MFMAs and fragment reads of a step
  constexpr int LAG = MF / 8;
  auto read1 = [&](auto setc, auto jc, const uint4* st) {
    constexpr int set = decltype(setc)::value, j = decltype(jc)::value, kk = j / (FM + FN), e = j % (FM + FN);
    if constexpr (e == 0) fw[set][kk][0] = as_bf16x8(st[at_w[kk]]);
    else if constexpr (e <= FM) fx[set][kk][e - 1] = as_bf16x8(st[at_x[kk] + (e - 1) * SH * 8]);
    else fw[set][kk][e - FM] = as_bf16x8(st[at_w[kk] + (e - FM) * SH * 8]);
  };
  // Past the last step there is nothing to fetch: the copies go to buffers of no length (zeros, no memory traffic) and the
  // last step reads the fragments of a stage nobody filled, so that one loop body serves every step and the counts of what
  // is on its way always hold.
  int32_t k_bytes = NS * 128;
  int cur = 0;
  const int64_t nk = k_len / 64;
  int32_t left = (int32_t)nk - NS;   // steps still to fetch
  auto step = [&](auto setc) {
    constexpr int set = decltype(setc)::value;
    const int nxt = cur + 1 == NS ? 0 : cur + 1;
    const uint4* sn = smem + nxt * STAGE;
    const uint32_t dst = lds_base + (uint32_t)(cur * STAGE * 16);
    xbuf[2] = wbuf[2] = left > 0 ? 0x7fffffffu : 0u;
    static_for<0, MF>([&](auto mi) {
      constexpr int m = decltype(mi)::value, r = m - LAG, RM = MF - LAG;
      if constexpr (r == 0) {
        // Before the barrier: this wave's fragments of the step are in registers (its stage may be overwritten) and its copies
        // of the next step have landed; the NS - 2 younger steps may stay on their way.
        __builtin_amdgcn_s_waitcnt(0x0070 | (GPW * (NS - 2) & 15) | (GPW * (NS - 2) >> 4 << 14));   // vmcnt, lgkmcnt(0)
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
      }
      if constexpr (r >= 0) {
        static_for<r * NR / RM, (r + 1) * NR / RM>([&](auto j) { read1(std::integral_constant<int, set ^ 1>{}, j, sn); });
        static_for<r * GPW / RM, (r + 1) * GPW / RM>([&](auto i) { issue1(i, dst, k_bytes); });
      }
      __builtin_amdgcn_sched_barrier(0);
      constexpr int kk = m / (FM * FN), a = m % (FM * FN) / FM, b = m % FM;
      acc.v[a][b] = mfma_bf16(fw[set][kk][a], fx[set][kk][b], acc.v[a][b]);
      __builtin_amdgcn_sched_barrier(0);
    });
    k_bytes += 128;
    --left;
    cur = nxt;
  };
  static_for<0, NS>([&](auto st) {
    if (st >= nk) xbuf[2] = wbuf[2] = 0;
    static_for<0, GPW>([&](auto i) { issue1(i, lds_base + (uint32_t)(st * STAGE * 16), st * 128); });
  });
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(GPW * (NS - 1)) : "memory");
  __builtin_amdgcn_s_barrier();
  static_for<0, NR>([&](auto j) { read1(std::integral_constant<int, 0>{}, j, smem); });
  const int32_t end = 1 - NS;   // of `left` in the last step
  for (;;) {
    step(std::integral_constant<int, 0>{});
    if (left < end) break;
    step(std::integral_constant<int, 1>{});
    if (left < end) break;
  }
  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");   // nothing writes to the stages any more,
  __builtin_amdgcn_s_barrier();                                  // nobody reads them: the epilogue may have them

  tile_epilogue<WGM, WGN, TM, TN, OutT, EPI, NS>(acc, smem, C, M, N, ep, m0, n0);
}

// The 256x256 tile on FOUR waves (one per SIMD, wave tile 128x128, accumulators in 256 registers): per K step the
// fragment reads take 128 KB out of LDS instead of the 192 KB the eight-wave form reads, and operands travel
// global -> registers -> LDS with every load in flight for a whole K step.  A wave moves sixteen 1 KB groups per step;
// slot i of a step writes the group that was loaded into register quad i one step earlier to the LDS stage that was
// freed by the previous barrier, and then reuses the quad for the load of the stage after next: sixty-four registers
// hold one stage in flight, the memory pipeline never drains, and the one barrier of a step (in the middle of the
// last MFMA block, so that queued MFMAs cover it) both publishes the next stage and frees the current one.
// Plain loads and stores: the compiler derives the vmcnt / lgkmcnt waits; the scheduling fences keep its order.
// SH = 32, 32x32x16 MFMAs, or 16, 16x16x32 ones: the power limit allows more of the latter, but they need an instruction slot
// twice as often and half as many fragment registers are reloaded at a time.  Which is faster where: gemm_route.cpp.
template <typename OutT, int EPI, int SH>
__global__ __launch_bounds__(256) void gemm_bf16_nt_w4_kernel(
    const bf16_t* __restrict__ X, const bf16_t* __restrict__ W, OutT* __restrict__ C, int64_t M, int64_t N,
    int64_t K, EpiDev ep, int32_t tiles_m, int32_t tiles_n, int32_t group_m) {
  constexpr int WGM = 2, WGN = 2, TM = 4, TN = 4, FM = TM * 32 / SH, FN = TN * 32 / SH;   // fragments of SH rows,
  constexpr int KS = 512 / SH, SLICES = 64 / KS;                                             // KS wide in k
  constexpr int BM = 256, BN = 256, NW = 4;
  constexpr int GX = BM / 8, G = (BM + BN) / 8, GPW = G / NW;   // 8-row groups of 1 KB; sixteen per wave
  constexpr int STAGE = (BM + BN) * 8;                          // uint4 per LDS stage
  extern __shared__ uint4 smem[];
  build_epilogue_tables<NW, OutT, EPI>((float2*)(smem + 2 * STAGE));

  const int64_t tile = xcd_contiguous(blockIdx.x, (int64_t)tiles_m * tiles_n);
  const int64_t per_group = (int64_t)group_m * tiles_n;
  const int64_t grp = tile / per_group;
  const int32_t first_m = (int32_t)(grp * group_m);
  const int32_t rows_in_group = (tiles_m - first_m < group_m) ? tiles_m - first_m : group_m;
  const int32_t tm_i = first_m + (int32_t)((tile % per_group) % rows_in_group);
  const int32_t tn_i = (int32_t)((tile % per_group) / rows_in_group);
  const int64_t m0 = (int64_t)tm_i * BM, n0 = (int64_t)tn_i * BN;

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave % WGM, wn = wave / WGM;
  const int lr = lane & (SH - 1), lg = lane / SH;

  typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));   // a first-class vector: a struct-typed quad would live in private memory
  // Global source of this lane for each group: a 32-bit byte offset from the tile's first row (rows past the end are
  // clamped: their products are never stored), added by the load instruction itself to a wave-uniform base that
  // advances by one K step; no vector arithmetic per load.  Groups 0..7 of a wave are rows of X, 8..15 rows of W.
  static_assert(GX == 8 * NW, "a wave's first eight groups are X rows");
  uint32_t off[GPW];
#pragma unroll
  for (int i = 0; i < GPW; ++i) {
    const int g = wave + i * NW;
    const bool isx = i < GPW / 2;
    const int r = (isx ? g : g - GX) * 8 + (lane >> 3);
    const int c = (lane & 7) ^ ((r >> 1) & 7);
    const int64_t last = (isx ? M - m0 : N - n0) - 1;   // last valid row of the tile
    const int64_t row = r <= last ? r : last;
    off[i] = (uint32_t)((row * K + c * 8) * 2);
  }
  // Buffer loads: the tile's first row is the base of a raw buffer (no stride, no bounds to speak of: every offset
  // stays below 2^31), the lane's offset a 32-bit register, the K step a scalar offset.
  const __amdgpu_buffer_rsrc_t xrsrc = __builtin_amdgcn_make_buffer_rsrc((void*)(X + m0 * K), 0, 0x7fffffff, 0x00020000);
  const __amdgpu_buffer_rsrc_t wrsrc = __builtin_amdgcn_make_buffer_rsrc((void*)(W + n0 * K), 0, 0x7fffffff, 0x00020000);
  auto gload = [&](auto ic, int64_t k0) {
    constexpr int i = decltype(ic)::value;
    return __builtin_amdgcn_raw_buffer_load_b128(i < GPW / 2 ? xrsrc : wrsrc, (int)off[i], (int)(k0 * 2), 0);
  };
  const int wro = wave * 64 + lane;   // group g of a stage starts at uint4 index g * 64: this lane's place in group `wave`
  // Fragment addresses without arithmetic in the loop.  Row r of a stage holds its 16-byte chunk c at position
  // c ^ (r / 2) % 8, and the rows a lane reads are SH apart, so every fragment of a lane has the same swizzle.  One
  // address per stage, operand and slice (16 or 8 registers); the blocks of rows go into the instructions' immediate offsets.
  const uint4* fx_at[2][SLICES];
  const uint4* fw_at[2][SLICES];
#pragma unroll
  for (int st = 0; st < 2; ++st)
#pragma unroll
    for (int kk = 0; kk < SLICES; ++kk) {
      const int chunk = (kk * (KS / 8) + lg) ^ ((lr >> 1) & 7);
      fx_at[st][kk] = smem + st * STAGE + (wm * TM * 32 + lr) * 8 + chunk;
      fw_at[st][kk] = smem + st * STAGE + BM * 8 + (wn * TN * 32 + lr) * 8 + chunk;
    }
  Accumulators<SH, TM, TN> acc;
#pragma unroll
  for (int a = 0; a < FN; ++a)
#pragma unroll
    for (int b = 0; b < FM; ++b)
#pragma unroll
      for (int r = 0; r < SH * SH / 64; ++r) acc.v[a][b][r] = 0.f;
  bf16x8 fw[SH == 32 ? 2 : 1][FN], fx[2][FM];
  using I0 = std::integral_constant<int, 0>;
  using I1 = std::integral_constant<int, 1>;
  using I2 = std::integral_constant<int, 2>;
  using I3 = std::integral_constant<int, 3>;
  auto load_w = [&](auto jc, auto stc, auto kkc) {
    constexpr int j = decltype(jc)::value, st = decltype(stc)::value, kk = decltype(kkc)::value;
    fw[SH == 32 ? kk & 1 : 0][j] = as_bf16x8(fw_at[st][kk][j * SH * 8]);
  };
  auto load_x = [&](auto jc, auto stc, auto kkc) {
    constexpr int j = decltype(jc)::value, st = decltype(stc)::value, kk = decltype(kkc)::value;
    fx[kk & 1][j] = as_bf16x8(fx_at[st][kk][j * SH * 8]);
  };
  u32x4 R[GPW];
  constexpr int MF = FM * FN;   // MFMAs per slice of the K step: 16 or 64
  // WR: stage kt + 1 exists (its groups wait in R); LD: stage kt + 2 exists.  Every memory instruction sits alone between two
  // MFMAs, so that none of them has to wait for an issue slot behind another (a wave issues in order, and with one wave per
  // SIMD whatever stalls it stalls the MFMA pipe).
  //
  // 32x32x16: slice KK, sixteen MFMAs on fragment set KK & 1, each preceded by one memory instruction.  Slices 0..2: eight
  // fragment reads for the next slice, in the order its MFMAs first need them (W block 0, the X blocks, W blocks 1..3), then
  // four times {write register quad q to the next stage, reload it for the stage after next}.  Slice 3: the last four
  // writes and reloads first, the barrier behind the eighth MFMA, then the first fragments of the next stage.
  auto load_both = [&](auto jc, auto stc, auto kkc) {
    constexpr int j = decltype(jc)::value;
    if constexpr (j == 0) load_w(I0{}, stc, kkc);
    else if constexpr (j <= 4) load_x(std::integral_constant<int, j - 1>{}, stc, kkc);
    else load_w(std::integral_constant<int, j - 4>{}, stc, kkc);
  };
  auto slice32 = [&](auto kkc, auto wrc, auto ldc, auto curc, int64_t k_next2) {
    constexpr int KK = decltype(kkc)::value, buf = KK & 1, CUR = decltype(curc)::value;
    uint4* const sn = smem + (CUR ^ 1) * STAGE;
    constexpr bool WR = decltype(wrc)::value, LD = decltype(ldc)::value;
    static_for<0, MF>([&](auto mi) {
      // One wait per group instead of one per use (the compiler, which still places every wait that is needed,
      // drops its own where these make them redundant): all eight fragments of this slice, read eight to sixteen
      // instructions ago with four LDS stores behind them, at the slice's first MFMA; the four register quads about
      // to be stored, loaded a K step ago with twelve younger loads behind them, at the first store.
      if constexpr (mi == 0 && KK > 0) __builtin_amdgcn_s_waitcnt(0xc47f);                                           // lgkmcnt(4)
      if constexpr (WR && LD && ((KK < 3 && mi == 8) || (KK == 3 && mi == 0))) __builtin_amdgcn_s_waitcnt(0x0f7c);   // vmcnt(12)
      if constexpr (KK < 3) {
        if constexpr (mi < 8) {
          load_both(mi, curc, std::integral_constant<int, (KK + 1) & 3>{});
        } else {
          constexpr int q = 4 * KK + (mi - 8) / 2;
          if constexpr ((mi & 1) == 0) {
            if constexpr (WR) *(u32x4*)(sn + wro + q * NW * 64) = R[q];
          } else {
            if constexpr (LD) R[q] = gload(std::integral_constant<int, q>{}, k_next2);
          }
        }
      } else {
        if constexpr (mi < 4) {
          if constexpr (WR) *(u32x4*)(sn + wro + (12 + mi) * NW * 64) = R[12 + mi];
        } else if constexpr (mi < 8) {
          if constexpr (LD) R[8 + mi] = gload(std::integral_constant<int, 8 + mi>{}, k_next2);
        } else {
          if constexpr (mi == 8) {
            __builtin_amdgcn_s_waitcnt(0xc07f);   // lgkmcnt(0): my LDS writes are done, my last fragments are in registers
            __builtin_amdgcn_s_barrier();
            __builtin_amdgcn_sched_barrier(0);
          }
          if constexpr (WR) load_both(std::integral_constant<int, mi - 8>{}, std::integral_constant<int, CUR ^ 1>{}, I0{});
        }
      }
      __builtin_amdgcn_sched_barrier(0);
      constexpr int a = mi / FM, b = mi % FM;
      acc.v[a][b] = mfma_bf16(fw[buf][a], fx[buf][b], acc.v[a][b]);
      __builtin_amdgcn_sched_barrier(0);
    });
  };
  // 16x16x32: slice KK, 64 MFMAs, every other one preceded by one memory instruction.  The MFMAs go through the W blocks one
  // after the other, so W needs one set of fragments: blocks 0..3 of the next slice replace this slice's once its first half
  // is through, blocks 4..7 arrive in the first slots of the slice that uses them.  X has two sets.
  // Slice 0, slots 0..31: W blocks 4..7; X of slice 1; two times {write register quad q to the next stage, reload it for
  // the stage after next}; W blocks 0..3 of slice 1; six more writes and reloads.
  // Slice 1: W blocks 4..7; the other eight writes; two reloads; the barrier; X and W blocks 0..3 of the next stage's slice
  // 0; six reloads.
  auto slice16 = [&](auto kkc, auto wrc, auto ldc, auto curc, int64_t k_next2) {
    constexpr int KK = decltype(kkc)::value, CUR = decltype(curc)::value;
    uint4* const sn = smem + (CUR ^ 1) * STAGE;
    constexpr bool WR = decltype(wrc)::value, LD = decltype(ldc)::value;
    using NEXT = std::integral_constant<int, CUR ^ 1>;
    auto put = [&](auto q) {
      if constexpr (WR) *(u32x4*)(sn + wro + q * NW * 64) = R[q];
    };
    auto get = [&](auto q) {
      if constexpr (LD) R[q] = gload(q, k_next2);
    };
    static_for<0, MF>([&](auto mi) {
      constexpr int slot = mi / 2;
      // One wait per group instead of one per use (the compiler, which still places every wait that is needed, drops its
      // own where these make them redundant): this slice's fragments at its first MFMA (behind them: six LDS stores in
      // slice 0's tail), the eight register quads about to be stored, loaded a K step ago with eight younger loads behind
      // them, at the first store.
      if constexpr (mi == 0) __builtin_amdgcn_s_waitcnt(KK == 0 ? 0xc07f : 0xc67f);                          // lgkmcnt(0 / 6)
      if constexpr (WR && LD && mi == (KK == 0 ? 24 : 8)) __builtin_amdgcn_s_waitcnt(0x0f78);                // vmcnt(8)
      if constexpr (mi % 2 == 0) {
        if constexpr (slot < 4) {
          load_w(std::integral_constant<int, 4 + slot>{}, curc, kkc);
        } else if constexpr (KK == 0) {
          if constexpr (slot < 12) load_x(std::integral_constant<int, slot - 4>{}, curc, I1{});
          else if constexpr (slot >= 16 && slot < 20) load_w(std::integral_constant<int, slot - 16>{}, curc, I1{});
          else {
            constexpr int i = slot < 16 ? slot - 12 : slot - 16;
            if constexpr (i % 2 == 0) put(std::integral_constant<int, i / 2>{});
            else get(std::integral_constant<int, i / 2>{});
          }
        } else {
          if constexpr (slot == 14) {
            __builtin_amdgcn_s_waitcnt(0xc07f);   // lgkmcnt(0): my LDS writes are done, my last fragments are in registers
            __builtin_amdgcn_s_barrier();
            __builtin_amdgcn_sched_barrier(0);
          }
          if constexpr (slot < 12) put(std::integral_constant<int, slot + 4>{});
          else if constexpr (slot < 14) get(std::integral_constant<int, slot - 4>{});
          else if constexpr (slot < 22) {
            if constexpr (WR) load_x(std::integral_constant<int, slot - 14>{}, NEXT{}, I0{});
          } else if constexpr (slot < 26) {
            if constexpr (WR) load_w(std::integral_constant<int, slot - 22>{}, NEXT{}, I0{});
          } else get(std::integral_constant<int, slot - 16>{});
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      constexpr int a = mi / FM, b = mi % FM;
      acc.v[a][b] = mfma_bf16(fw[0][a], fx[KK][b], acc.v[a][b]);
      __builtin_amdgcn_sched_barrier(0);
    });
  };
  // The stage is a compile-time constant (its addresses are picked from registers, not computed), so even and odd K
  // steps are separate instantiations.  Step kt works on stage (kt + nk) % 2: the last step is then always on stage
  // 1 and the one before it on stage 0 whatever nk is, and only the very first step of an odd nk stands alone.
  auto step = [&](auto wrc, auto ldc, auto curc, int64_t k_next2) {
    if constexpr (SH == 32) {
      slice32(I0{}, wrc, ldc, curc, k_next2);
      slice32(I1{}, wrc, ldc, curc, k_next2);
      slice32(I2{}, wrc, ldc, curc, k_next2);
      slice32(I3{}, wrc, ldc, curc, k_next2);
    } else {
      slice16(I0{}, wrc, ldc, curc, k_next2);
      slice16(I1{}, wrc, ldc, curc, k_next2);
    }
  };

  const int64_t nk = K / 64;
  const int s0 = (int)(nk & 1);
  // prologue: K step 0 through the registers into its stage, step 1 into the registers, the first fragments
  static_for<0, GPW>([&](auto i) { R[i] = gload(i, 0); });
  static_for<0, GPW>([&](auto i) { *(u32x4*)(smem + s0 * STAGE + wro + i * NW * 64) = R[i]; });
  if (nk > 1) static_for<0, GPW>([&](auto i) { R[i] = gload(i, 64); });
  __builtin_amdgcn_s_waitcnt(0xc07f);
  __builtin_amdgcn_s_barrier();
  auto first_frags = [&](auto stc) {
    if constexpr (SH == 32) {
      static_for<0, 8>([&](auto j) { load_both(j, stc, I0{}); });
    } else {
      static_for<0, 8>([&](auto j) { load_x(j, stc, I0{}); });
      static_for<0, 4>([&](auto j) { load_w(j, stc, I0{}); });
    }
  };
  if (s0) first_frags(I1{});
  else first_frags(I0{});
  int64_t kt = 0;
  if (nk >= 3 && s0) {
    step(std::true_type{}, std::true_type{}, I1{}, 2 * 64);
    kt = 1;
  }
  for (; kt + 2 < nk; kt += 2) {
    step(std::true_type{}, std::true_type{}, I0{}, (kt + 2) * 64);
    step(std::true_type{}, std::true_type{}, I1{}, (kt + 3) * 64);
  }
  if (nk >= 2) step(std::true_type{}, std::false_type{}, I0{}, 0);
  step(std::false_type{}, std::false_type{}, I1{}, 0);

  tile_epilogue<WGM, WGN, TM, TN, OutT, EPI>(acc, smem, C, M, N, ep, m0, n0);
}

template <typename OutT, typename Kern>
hipError_t launch_tiles(Kern kern, int BM, int BN, int threads, bool* attr_set, const void* X, const void* W, void* C,
                        int64_t M, int64_t N, int64_t K, const EpiDev& ep, int32_t splits, hipStream_t stream, int stages = 2) {
  const int64_t tiles_m = (M + BM - 1) / BM, tiles_n = (N + BN - 1) / BN;
  const size_t lds = (size_t)stages * (BM + BN) * 8 * sizeof(uint4) + 8192;   // operand stages + the GELU table
  if (!*attr_set) {   // raise the dynamic-LDS limit once per instantiation
    hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    *attr_set = true;
  }
  const int32_t group_m = 8;
  hipLaunchKernelGGL(kern, dim3((unsigned)(tiles_m * tiles_n), (unsigned)splits), dim3(threads), lds, stream, (const bf16_t*)X,
                     (const bf16_t*)W, (OutT*)C, M, N, K, ep,
                     (int32_t)tiles_m, (int32_t)tiles_n, group_m);
  return hipGetLastError();
}

// The tiled kernel of one epilogue combination that the route names (gemm_route.cpp says why).
template <typename OutT, int EPI>
hipError_t launch_fast(const Route& r, const void* X, const void* W, void* C, int64_t M, int64_t N, int64_t K,
                       const EpiDev& ep, hipStream_t stream) {
  static bool attr_big = false, attr_wide = false, attr_small = false, attr_deep = false, attr_tall = false, attr_slim = false, attr_16 = false;
  switch (r.kernel) {
    case TILE_256x256:
      return launch_tiles<OutT>(gemm_bf16_nt_w4_kernel<OutT, EPI, 32>, 256, 256, 256, &attr_big, X, W, C, M, N, K, ep, 1, stream);
    case TILE_256x256_16:
      return launch_tiles<OutT>(gemm_bf16_nt_w4_kernel<OutT, EPI, 16>, 256, 256, 256, &attr_16, X, W, C, M, N, K, ep, 1, stream);
    case TILE_256x192:
      return launch_tiles<OutT>(gemm_bf16_nt_kernel<4, 2, 2, 3, OutT, EPI>, 256, 192, 512, &attr_wide, X, W, C, M, N, K,
                                ep, 1, stream);
    case TILE_256x128:
      return launch_tiles<OutT>(gemm_bf16_nt_step_kernel<2, 2, 4, 2, OutT, EPI, 3, 32>, 256, 128, 256, &attr_tall, X, W, C, M, N, K,
                                ep, 1, stream, 3);
    case TILE_128x64:
      return launch_tiles<OutT>(gemm_bf16_nt_step_kernel<2, 2, 2, 1, OutT, EPI, 6, 32>, 128, 64, 256, &attr_slim, X, W, C, M, N, K,
                                ep, 1, stream, 6);
    case TILE_128x128_DEEP:
      return launch_tiles<OutT>(gemm_bf16_nt_step_kernel<2, 2, 2, 2, OutT, EPI, 4, 32>, 128, 128, 256, &attr_deep, X, W, C, M, N, K,
                                ep, r.splits, stream, 4);
    case TILE_128x128:
      return launch_tiles<OutT>(gemm_bf16_nt_step_kernel<2, 2, 2, 2, OutT, EPI, 2, 16>, 128, 128, 256, &attr_small, X, W, C,
                                M, N, K, ep, r.splits, stream);
    default:
      return hipErrorInvalidValue;
  }
}

}  // namespace gemm
}  // namespace pf
