// GEMM for launches that do not fill the chip:  C[M,N] = epilogue( X[M,K] * W[N,K]^T ), bf16 and fp32.
//
// What bounds such a launch is not the matrix cores but how many bytes are on their way: the tiled kernel keeps one
// K step in flight per workgroup and, with few workgroups, pays a memory latency per step (0.8 us at 128 x 768,
// K = 3072: 38.6 us for 48 steps on 6 of 256 CUs).  Here the waves of a workgroup share one small tile of C and
// divide K between them: wave w takes K steps w, w + WK, ... through a ring of DEPTH LDS stages of its own, so no wave
// waits for another (no barrier until the sums meet) and WK * DEPTH steps, 64 to 144 KB per workgroup, are in flight at once.
// A stage goes to registers whole and is refilled before its MFMAs run.  Two waves per SIMD with one stage each (the small
// tiles; the 32x32 one leaves room for two workgroups per CU) beat fewer waves with two stages, whose wait, LDS reads, copies
// and MFMAs follow one another, as long as a wave has few steps or its MFMAs are short: 128 x 2304, K = 768 6.0 -> 5.3 us, 333 x
// 2048, K = 2048 on 32x32 tiles 15.8 -> 12.3 us, 600 x 512, K = 2048 8.7 -> 7.6 us, 512 x 1536, K = 600 into fp32 7.6 -> 6.9 us.
// Where both forms of a tile exist, gemm_route.cpp says which runs.
// A K step is 128 bytes of every row (64 bf16 or 32 fp32 elements); stages hold eight 16-byte chunks per row,
// XOR-swizzled on the global side as in the tiled kernel.
//   bf16: 32x32x16 MFMA.  fp32: 32x32x2 fp32 MFMA, four per pair of chunks: lane half lk supplies element j of chunk
//   2 kk + lk in both operands, a permutation of the K order that both share.
// The partial tiles meet in LDS in the order of the waves (same bits every time) and leave as whole rows; residual,
// saved pre-activation input and bias were requested before the K loop.
// K need only be a whole number of 16-byte chunks: loads past the end repeat the last chunk and the operands of the
// last step are zeroed beyond K.
// Measured (MI355X, weights from the memory-side cache, launches back to back; before -> after): 128 x 768, K = 768
// 10.6 -> 3.9 us; 128 x 768, K = 3072 38.5 -> 7.3 us; 128 x 2304, K = 768 12.5 -> 5.3 us; 333 x 2048, K = 8192 122 -> 30 us
// (each of the 192 busy CUs takes in about 70 bytes per ns there, which is what now bounds it); 600-token weight gradient 2048 x 512
// 17.9 -> 8.6 us; fp32 512 x 256, K = 1024 115 -> 10 us.
#include "pf_kernels.h"
#include "gemm_tile.h"

namespace pf {
namespace gemm {
namespace {

template <typename T, typename OutT, int TM, int TN, int WK, int DEPTH>
__global__ __launch_bounds__(64 * WK) void gemm_ring_kernel(const T* __restrict__ X, const T* __restrict__ W, OutT* C,
                                                            int64_t M, int64_t N, int64_t K, EpiDev ep,
                                                            int32_t tiles_m, int32_t tiles_n, int32_t vec) {
  constexpr int BM = 32 * TM, BN = 32 * TN, NT = 64 * WK;
  constexpr int CE = 16 / (int)sizeof(T);               // elements per chunk
  constexpr int LPS = (TM + TN) * 4;                    // 1 KB copies per stage
  constexpr int STAGE = LPS * 64;                       // uint4 per stage
  constexpr int UNITS = BN / 4, ITEMS = BM * BN / 4, IT = (ITEMS + NT - 1) / NT;
  static_assert(LPS < 64, "vmcnt holds six bits: one stage may stay on its way");
  static_assert(BM * BN * 4 <= DEPTH * STAGE * 16, "the partial tiles fit the stages");
  extern __shared__ uint4 smem[];

  // row tiles of one column panel run on one XCD one after the other: its L2 fetches the panel of W once
  const int64_t tile = xcd_contiguous(blockIdx.x, (int64_t)tiles_m * tiles_n);
  const int64_t per_group = (int64_t)8 * tiles_n, grp = tile / per_group;
  const int32_t first_m = (int32_t)(grp * 8);
  const int32_t in_group = (tiles_m - first_m < 8) ? tiles_m - first_m : 8;
  const int64_t m0 = (int64_t)(first_m + (int32_t)((tile % per_group) % in_group)) * BM;
  const int64_t n0 = (int64_t)((tile % per_group) / in_group) * BN;

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lr = lane & 31, lk = lane >> 5;

  // copy i moves eight rows (X rows first, then W rows); rows past the end repeat the last one, their products are
  // never stored.  The chunk a lane fetches depends on the parity of i only.
  const T* row_at[LPS];
#pragma unroll
  for (int i = 0; i < LPS; ++i) {
    const bool isx = i < TM * 4;
    int64_t row = (isx ? m0 : n0) + (isx ? i : i - TM * 4) * 8 + (lane >> 3);
    const int64_t last = (isx ? M : N) - 1;
    if (row > last) row = last;
    row_at[i] = (isx ? X : W) + row * K;
  }
  const int c_even = (lane & 7) ^ (lane >> 4), c_odd = c_even ^ 4;
  const uint32_t lds_base =
      __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(lds_ptr_t)smem) + (uint32_t)(wave * DEPTH * STAGE * 16);
  auto issue = [&](int slot, int64_t step) {
    const int64_t k0 = step * 8 * CE;
    const int64_t ke = k0 + c_even * CE, ko = k0 + c_odd * CE;
    const int64_t off_e = ke < K ? ke : K - CE, off_o = ko < K ? ko : K - CE;
#pragma unroll
    for (int i = 0; i < LPS; ++i)
      lds_direct_load_1k(__builtin_amdgcn_readfirstlane(lds_base + (uint32_t)((slot * STAGE + i * 64) * 16)),
                         row_at[i] + ((i & 1) ? off_o : off_e));
  };

  const int64_t steps = (K + 8 * CE - 1) / (8 * CE);
  const int64_t mine = steps > wave ? (steps - wave + WK - 1) / WK : 0;

  // this thread's share of the output tile: item i is four columns of one row
  typedef typename std::conditional<std::is_same<T, float>::value, float4, uint2>::type raw4;
  auto item_row = [&](int i) { return (i * NT + tid) / UNITS; };
  auto item_unit = [&](int i) { return (i * NT + tid) % UNITS; };
  auto item_in = [&](int i) {
    return i * NT + tid < ITEMS && m0 + item_row(i) < M && n0 + item_unit(i) * 4 < N;
  };
  raw4 rbias[IT], raux[IT];
  const T* aux = (const T*)(ep.dact_in ? ep.dact_in : ep.resid);
  if (vec) {   // older than every copy, so the counts below stay right
    if (ep.bias) {
#pragma unroll
      for (int i = 0; i < IT; ++i)
        if (item_in(i)) rbias[i] = *(const raw4*)((const T*)ep.bias + n0 + item_unit(i) * 4);
    }
    if (aux) {
#pragma unroll
      for (int i = 0; i < IT; ++i)
        if (item_in(i)) raux[i] = *(const raw4*)(aux + (m0 + item_row(i)) * N + n0 + item_unit(i) * 4);
    }
  }

  f32x16 acc[TN][TM];
#pragma unroll
  for (int a = 0; a < TN; ++a)
#pragma unroll
    for (int b = 0; b < TM; ++b)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[a][b][r] = 0.f;

  for (int s = 0; s < DEPTH; ++s)
    if (s < mine) issue(s, wave + (int64_t)s * WK);
  const int sw = (lr >> 1) & 7;
  int slot = 0;
  for (int64_t s = 0; s < mine; ++s) {
    // the younger stage, if there is one, may stay on its way; the last step has none behind it.  (Written as s + DEPTH <= mine
    // the compiler makes two copies of the loop's body: 3709 x 320, K = 248 on 128x64 tiles 9.1 -> 9.4 us.)
    if (s + DEPTH - 1 < mine) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(LPS * (DEPTH - 1)) : "memory");
    else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    const uint4* st = smem + (wave * DEPTH + slot) * STAGE;
    uint4 fx[4][TM], fw[4][TN];
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
      const int c = (kk * 2 + lk) ^ sw;
#pragma unroll
      for (int b = 0; b < TM; ++b) fx[kk][b] = st[(b * 32 + lr) * 8 + c];
#pragma unroll
      for (int a = 0; a < TN; ++a) fw[kk][a] = st[((TM + a) * 32 + lr) * 8 + c];
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // the stage is in registers: refill it
    const int64_t step = wave + s * WK;
    if (s + DEPTH < mine) issue(slot, step + (int64_t)DEPTH * WK);
    slot = slot + 1 == DEPTH ? 0 : slot + 1;
    if ((step + 1) * 8 * CE > K) {
#pragma unroll
      for (int kk = 0; kk < 4; ++kk)
        if ((step * 8 + kk * 2 + lk) * CE >= K) {
#pragma unroll
          for (int b = 0; b < TM; ++b) fx[kk][b] = make_uint4(0, 0, 0, 0);
#pragma unroll
          for (int a = 0; a < TN; ++a) fw[kk][a] = make_uint4(0, 0, 0, 0);
        }
    }
#pragma unroll
    for (int kk = 0; kk < 4; ++kk)
#pragma unroll
      for (int a = 0; a < TN; ++a)
#pragma unroll
        for (int b = 0; b < TM; ++b) {
          if constexpr (std::is_same<T, float>::value) {
            const f32x4 vw = __builtin_bit_cast(f32x4, fw[kk][a]), vx = __builtin_bit_cast(f32x4, fx[kk][b]);
#pragma unroll
            for (int j = 0; j < 4; ++j)
              acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x2f32(vw[j], vx[j], acc[a][b], 0, 0, 0);
          } else {
            acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(fw[kk][a]), as_bf16x8(fx[kk][b]), acc[a][b],
                                                               0, 0, 0);
          }
        }
  }

  // partial tiles: fp32, row-major, 16-byte units XOR-swizzled by row
  __syncthreads();
  float4* red = (float4*)smem;
  static_for<0, TN>([&](auto a) {
    static_for<0, TM>([&](auto b) {
      const int row = b * 32 + lr;
      static_for<0, 4>([&](auto rg) {
        const int unit = a * 8 + rg * 2 + lk;
        red[wave * ITEMS + row * UNITS + (unit ^ (row & (UNITS - 1)))] =
            make_float4(acc[a][b][rg * 4 + 0], acc[a][b][rg * 4 + 1], acc[a][b][rg * 4 + 2], acc[a][b][rg * 4 + 3]);
      });
    });
  });
  __syncthreads();
#pragma unroll
  for (int i = 0; i < IT; ++i) {
    if (!item_in(i)) continue;
    const int row = item_row(i), unit = item_unit(i);
    float v[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < WK; ++w) {
      const float4 t = red[w * ITEMS + row * UNITS + (unit ^ (row & (UNITS - 1)))];
      v[0] += t.x; v[1] += t.y; v[2] += t.z; v[3] += t.w;
    }
    const int64_t m = m0 + row, n = n0 + unit * 4, off = m * N + n;
    if (!vec) {
      epilogue4_scalar<T, OutT>(v, m, n, M, N, C, ep);
      continue;
    }
    float t[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) v[j] *= ep.scale;
    if (ep.bias) {
      load4((const T*)&rbias[i], t);
#pragma unroll
      for (int j = 0; j < 4; ++j) v[j] += t[j];
    }
    if (ep.preact_out) store4((T*)ep.preact_out + off, v);
    if (ep.gelu) {
#pragma unroll
      for (int j = 0; j < 4; ++j) v[j] = gelu_as<T>(v[j]);
    }
    if (aux) load4((const T*)&raux[i], t);
    if (ep.dact_in) {
#pragma unroll
      for (int j = 0; j < 4; ++j) v[j] *= gelu_grad_f(t[j]);
      if (ep.resid) load4((const T*)ep.resid + off, t);
    }
    if (ep.resid) {
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
}

template <typename T, typename OutT, int TM, int TN, int WK, int DEPTH>
hipError_t launch_ring(const void* X, const void* W, void* C, int64_t M, int64_t N, int64_t K, const EpiDev& ep,
                       hipStream_t stream) {
  static bool attr = false;
  constexpr int lds = WK * DEPTH * (TM + TN) * 4096;
  auto kern = gemm_ring_kernel<T, OutT, TM, TN, WK, DEPTH>;
  if (!attr) {
    hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (e != hipSuccess) return e;
    attr = true;
  }
  const int64_t tiles_m = (M + 32 * TM - 1) / (32 * TM), tiles_n = (N + 32 * TN - 1) / (32 * TN);
  // four columns at a time: whole groups of four, operands of the epilogue aligned to them
  const uintptr_t p = (uintptr_t)ep.bias | (uintptr_t)ep.resid | (uintptr_t)ep.dact_in | (uintptr_t)ep.preact_out;
  const int32_t vec = (N & 3) == 0 && (p & (4 * sizeof(T) - 1)) == 0 && ((uintptr_t)C & (4 * sizeof(OutT) - 1)) == 0;
  hipLaunchKernelGGL(kern, dim3((unsigned)(tiles_m * tiles_n)), dim3(64 * WK), lds, stream, (const T*)X, (const T*)W,
                     (OutT*)C, M, N, K, ep, (int32_t)tiles_m, (int32_t)tiles_n, vec);
  return hipGetLastError();
}

}  // namespace

template <typename T, typename OutT>
hipError_t launch_ring_shape(Kernel shape, const void* X, const void* W, void* C, int64_t M, int64_t N, int64_t K,
                             const EpiDev& ep, hipStream_t stream) {
  switch (shape) {
    case RING_32x32: return launch_ring<T, OutT, 1, 1, 8, 1>(X, W, C, M, N, K, ep, stream);
    case RING_32x64: return launch_ring<T, OutT, 1, 2, 8, 1>(X, W, C, M, N, K, ep, stream);
    case RING_64x64: return launch_ring<T, OutT, 2, 2, 8, 1>(X, W, C, M, N, K, ep, stream);
    case RING_128x64: return launch_ring<T, OutT, 4, 2, 3, 2>(X, W, C, M, N, K, ep, stream);
    case RING_32x32_DEEP: return launch_ring<T, OutT, 1, 1, 8, 2>(X, W, C, M, N, K, ep, stream);
    case RING_32x64_DEEP:   // fp32 only
      if constexpr (std::is_same<T, float>::value) return launch_ring<T, OutT, 1, 2, 6, 2>(X, W, C, M, N, K, ep, stream);
      return hipErrorInvalidValue;
    case RING_64x64_DEEP: return launch_ring<T, OutT, 2, 2, 4, 2>(X, W, C, M, N, K, ep, stream);
    default: return hipErrorInvalidValue;
  }
}
template hipError_t launch_ring_shape<bf16_t, bf16_t>(Kernel, const void*, const void*, void*, int64_t, int64_t, int64_t, const EpiDev&, hipStream_t);
template hipError_t launch_ring_shape<bf16_t, float>(Kernel, const void*, const void*, void*, int64_t, int64_t, int64_t, const EpiDev&, hipStream_t);
template hipError_t launch_ring_shape<float, float>(Kernel, const void*, const void*, void*, int64_t, int64_t, int64_t, const EpiDev&, hipStream_t);

}  // namespace gemm
}  // namespace pf
