// Weight-gradient GEMM for bf16 training:  C[M][N] (fp32) += A^T B  with A [K][M] and B [K][N] row-major,
// i.e. both operands as the layer left them in memory (tokens are the slow index): dW = dY^T X needs no
// transposed copies.  Optionally colsum[m] += sum over k of A[k][m], which is the bias gradient of the same layer.
//
// 128x128 tiles, 4 waves (2x2, wave tile 64x64 in 16x16x32 MFMAs), K steps of 64, two LDS stages of 32 KB, two
// workgroups per CU.  Operand slabs go global -> LDS directly, 4 k-rows x 256 bytes per wave instruction, in the [k][m]
// order they have in memory; rows past the end of K are past the end of the buffer and arrive as zeros, so K need not be
// a multiple of 64 (it comes in eights).  MFMA wants, per lane, eight consecutive k of one m: ds_read_b64_tr_b16 delivers exactly that
// from a k-major image (a 16-lane group reads a 4 k x 16 m block and every lane receives the four k of its own m), two
// reads per fragment.  The 16-byte chunks of a k-row are XOR-swizzled by 4 * (k % 4) + 2 * (k / 8 % 2) (on the global
// side of the copy), so that the eight half rows the two groups of a half-wave read fall on disjoint banks.
// The fragments of a whole K step are double buffered in registers: while the MFMAs of one step run, its successor's 32
// reads and the copies of the step after that are issued between them, one barrier a step (behind its first MFMAs).  With a
// substep of reads in flight at a time and every copy of a step in one burst behind the barrier: 4096 x 1024, K = 8192 105 us,
// now 85; 50304 x 1024, K = 8192 1162 -> 960, 8192 x 8192, K = 2048 585 -> 448, 512 x 512, K = 640 20 -> 10.
// Split K: gridDim.y workgroups share a tile, each over a run of whole steps; the fp32 tile goes through LDS and is
// added to C with fp32 atomics in coalesced order (plain read-add-write when K is not split).  The column sum
// comes from one more MFMA per A fragment against a fragment of ones, on the waves of the first tile column.
// WIDE: M or N from 2^23 on, where 64 rows pass the 2^31 bytes of a raw buffer.  64-bit addresses per lane, whole K steps only.
#include <algorithm>
#include <type_traits>

#include "pf_device.h"
#include "pf_kernels.h"

namespace pf {
namespace {

typedef short v4s __attribute__((ext_vector_type(4)));
typedef short v8s __attribute__((ext_vector_type(8)));
typedef __attribute__((address_space(3))) v4s* lds_v4s_ptr;
typedef __attribute__((address_space(3))) void* lds_void_ptr;
typedef const __attribute__((address_space(3))) char* lds_char_ptr;

template <int I, int N, class F>
__device__ __forceinline__ void unrolled(F&& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    unrolled<I + 1, N>(f);
  }
}

template <bool COLSUM, bool WIDE>
__global__ __launch_bounds__(256, 2) void gemm_bf16_tn_acc_kernel(const bf16_t* __restrict__ A,
                                                                  const bf16_t* __restrict__ B, float* __restrict__ C,
                                                                  float* __restrict__ colsum, int64_t M, int64_t N,
                                                                  int64_t K, int32_t tiles_m, int32_t tiles_n) {
  constexpr int BM = 128, BN = 128, FM = 4, FN = 4, NW = 4, STAGE = 32768, BOFF = 16384;
  extern __shared__ char smem[];
  const int64_t tile = xcd_contiguous(blockIdx.x, (int64_t)tiles_m * tiles_n);
  const int32_t tn_i = (int32_t)(tile % tiles_n), tm_i = (int32_t)(tile / tiles_n);
  const int64_t m0 = (int64_t)tm_i * BM, n0 = (int64_t)tn_i * BN;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave & 1, wn = wave >> 1;
  const int li = lane & 15, lg = lane >> 4;
  const int32_t steps = (int32_t)((K + 63) / 64), share = (steps + (int32_t)gridDim.y - 1) / (int32_t)gridDim.y;
  const int32_t first = (int32_t)blockIdx.y * share;
  const int32_t nk = steps - first < share ? steps - first : share;   // the launcher leaves no slice empty

  // this lane's place in each of the 8 copies the wave issues per step (4 of A, 4 of B): copy q = wave + 4 i covers k-rows
  // 4 q .. 4 q + 3 of the step; the lane takes chunk (lane % 16) ^ swizzle of row lane / 16.  A tile that sticks out along M
  // or N takes any chunk of the row instead, the result is discarded.
  const int cglob = li ^ (4 * lg) ^ (2 * ((wave >> 1) & 1));
  const int64_t last_a = M - 8 - m0, last_b = N - 8 - n0;
  const int64_t ca = cglob * 8 < last_a ? cglob * 8 : last_a, cb = cglob * 8 < last_b ? cglob * 8 : last_b;
  uint32_t off[8];
  const bf16_t* const pa = A + ((int64_t)first * 64 + wave * 4 + lg) * M + m0 + ca;   // WIDE: copy 0 of the first step
  const bf16_t* const pb = B + ((int64_t)first * 64 + wave * 4 + lg) * N + n0 + cb;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int64_t r = (wave + 4 * i) * 4 + lg;
    off[i] = (uint32_t)((r * M + m0 + ca) * 2);
    off[4 + i] = (uint32_t)((r * N + n0 + cb) * 2);
  }
  // the rows of one K step are a raw buffer: rows past the end of K are outside it; a step past the slice has none
  const char* arow = (const char*)A + (int64_t)first * 128 * M;
  const char* brow = (const char*)B + (int64_t)first * 128 * N;
  int64_t rows_left = K - (int64_t)first * 64;
  int32_t left = nk;
  lds_buffer_t abuf, bbuf;
  int64_t row = 0;         // WIDE: of the slice, where the step that is copied next begins
  auto next_rows = [&] {   // of the step that is copied next
    if constexpr (WIDE) {   // a step past the slice is the last one again: nobody uses its fragments
      if (left < nk && left > 0) row += 64;
      --left;
      return;
    }
    const int32_t rows = left > 0 ? (int32_t)(rows_left < 64 ? rows_left : 64) : 0;
    abuf = lds_buffer(arow, (uint32_t)(rows * (int32_t)M * 2));
    bbuf = lds_buffer(brow, (uint32_t)(rows * (int32_t)N * 2));
    arow += 128 * M;
    brow += 128 * N;
    rows_left -= 64;
    --left;
  };
  const uint32_t lds_base = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(lds_void_ptr)smem) + (uint32_t)(wave * 1024);
  auto issue = [&](auto ic, auto stc) {
    constexpr int i = decltype(ic)::value, st = decltype(stc)::value;
    const uint32_t dst = lds_base + (uint32_t)(st * STAGE + (i < 4 ? 0 : BOFF) + (i & 3) * 4096);
    if constexpr (WIDE) lds_direct_load_1k(__builtin_amdgcn_readfirstlane(dst), (i < 4 ? pa : pb) + (row + (i & 3) * 16) * (i < 4 ? M : N));
    else lds_buffer_load_1k(dst, i < 4 ? abuf : bbuf, off[i], 0);
  };

  // fragment addressing: lane 16 g + i points at k-row 8 g + 4 r + i / 4 of the 32-row substep and at the four columns from
  // 4 * (i % 4) of its 16-column block, and receives column i with the four k of read r
  const int kq = li >> 2, swz = (4 * kq) ^ (2 * (lg & 1));
  int offA[FM], offB[FN];
#pragma unroll
  for (int f = 0; f < 4; ++f) {
    const int row = (8 * lg + kq) * 256 + 8 * (li & 1);
    offA[f] = row + (((wm * 8 + 2 * f + ((li & 3) >> 1)) ^ swz) << 4);
    offB[f] = BOFF + row + (((wn * 8 + 2 * f + ((li & 3) >> 1)) ^ swz) << 4);
  }
  v4s fa[2][2][FM][2], fb[2][2][FN][2];   // [set][substep][block][read]
  auto read1 = [&](auto setc, auto jc, auto stc) {   // order: the first A and B blocks of a substep first
    constexpr int set = decltype(setc)::value, j = decltype(jc)::value, st = decltype(stc)::value;
    constexpr int ks = j / 16, e = j % 16 / 2, r = j % 2;
    constexpr int at = st * STAGE + ks * 8192 + r * 1024;
    // e: B 0, A 0..3, B 1..3
    constexpr bool isa = e >= 1 && e <= 4;
    constexpr int f = e == 0 ? 0 : isa ? e - 1 : e - 4;
    lds_char_ptr p = (lds_char_ptr)(lds_void_ptr)smem + (isa ? offA[f] : offB[f]) + at;
    const v4s v = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s_ptr)p);
    if constexpr (isa) fa[set][ks][f][r] = v;
    else fb[set][ks][f][r] = v;
  };
  auto join = [](const v4s (&t)[2]) {
    const v8s o = {t[0][0], t[0][1], t[0][2], t[0][3], t[1][0], t[1][1], t[1][2], t[1][3]};
    return __builtin_bit_cast(bf16x8, o);
  };
  f32x4 acc[FN][FM], csum[FM];
#pragma unroll
  for (int a = 0; a < FN; ++a)
#pragma unroll
    for (int b = 0; b < FM; ++b)
#pragma unroll
      for (int r = 0; r < 4; ++r) acc[a][b][r] = 0.f;
#pragma unroll
  for (int b = 0; b < FM; ++b)
#pragma unroll
    for (int r = 0; r < 4; ++r) csum[b][r] = 0.f;
  v8s ones_s;
#pragma unroll
  for (int j = 0; j < 8; ++j) ones_s[j] = (short)0x3f80;   // bf16 1.0
  const bf16x8 ones = __builtin_bit_cast(bf16x8, ones_s);
  const bool do_sum = COLSUM && tn_i == 0 && wn == 0;

  constexpr int MF = 32, NR = 32, LAG = 4;
  auto step = [&](auto setc) {   // step kt works on stage kt % 2 and on fragment set kt % 2
    constexpr int set = decltype(setc)::value;
    using NEXT = std::integral_constant<int, set ^ 1>;
    next_rows();
    unrolled<0, MF>([&](auto mi) {
      constexpr int m = decltype(mi)::value, r = m - LAG, RM = MF - LAG;
      if constexpr (r == 0) {
        // this wave's fragments of the step are in registers (its stage may be overwritten), its copies of the next step
        // have landed
        __builtin_amdgcn_s_waitcnt(0x0070);   // vmcnt(0) lgkmcnt(0)
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
      }
      if constexpr (r >= 0) {
        unrolled<r * NR / RM, (r + 1) * NR / RM>([&](auto j) { read1(NEXT{}, j, NEXT{}); });
        unrolled<r * 8 / RM, (r + 1) * 8 / RM>([&](auto i) { issue(i, setc); });
      }
      __builtin_amdgcn_sched_barrier(0);
      constexpr int ks = m / 16, a = m % 16 / 4, b = m % 4;
      acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(join(fb[set][ks][a]), join(fa[set][ks][b]), acc[a][b], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    });
    if constexpr (COLSUM) {
      if (do_sum) {
#pragma unroll
        for (int ks = 0; ks < 2; ++ks)
#pragma unroll
          for (int b = 0; b < FM; ++b)
            csum[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones, join(fa[set][ks][b]), csum[b], 0, 0, 0);
      }
    }
  };
  using I0 = std::integral_constant<int, 0>;
  using I1 = std::integral_constant<int, 1>;
  next_rows();
  unrolled<0, 8>([&](auto i) { issue(i, I0{}); });
  next_rows();
  unrolled<0, 8>([&](auto i) { issue(i, I1{}); });
  asm volatile("s_waitcnt vmcnt(8)" ::: "memory");
  __builtin_amdgcn_s_barrier();
  unrolled<0, NR>([&](auto j) { read1(I0{}, j, I0{}); });
  // Past the last step nothing is fetched (empty buffers) and the fragments of a stage of zeros are read: one loop body.
  int32_t kt = 0;
  for (;;) {
    step(I0{});
    if (++kt >= nk) break;
    step(I1{});
    if (++kt >= nk) break;
  }
  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");   // nothing writes to the stages any more, nobody reads them
  __builtin_amdgcn_s_barrier();

  // D[i][j]: lane holds j = lane % 16 (row of C) and i = 4 * (lane / 16) + r (column of C).
  if constexpr (COLSUM) {
    // every row i of ones x A equals the column sums: row 0 sits in register 0 of lanes 0..15
    if (do_sum && lane < 16) {
#pragma unroll
      for (int b = 0; b < FM; ++b) {
        const int64_t m = m0 + wm * 64 + b * 16 + lane;
        if (m < M) unsafeAtomicAdd(colsum + m, csum[b][0]);
      }
    }
  }
  // the fp32 tile takes both LDS stages (row-major, 16-byte units XOR-swizzled by row) and leaves in rows
  float* stf = (float*)smem;
  constexpr int UNITS = BN / 4, NT = 64 * NW;
  unrolled<0, FN>([&](auto a) {
    unrolled<0, FM>([&](auto b) {
      const int row = wm * 64 + b * 16 + li, unit = wn * 16 + a * 4 + lg;
      *(f32x4*)(stf + row * BN + ((unit ^ (row & (UNITS - 1))) * 4)) = acc[a][b];
    });
  });
  __builtin_amdgcn_s_waitcnt(0xc07f);
  __builtin_amdgcn_s_barrier();
  const bool split = gridDim.y > 1;
  if (split || ((uintptr_t)C & 15) != 0) {
#pragma unroll 8
    for (int i = 0; i < BM * BN / NT; ++i) {
      const int e = i * NT + tid, row = e / BN, col = e % BN;
      const float v = stf[row * BN + (((col >> 2) ^ (row & (UNITS - 1))) * 4) + (col & 3)];
      if (m0 + row < M && n0 + col < N) {
        float* p = C + (m0 + row) * N + n0 + col;
        if (split) unsafeAtomicAdd(p, v);
        else *p += v;
      }
    }
    return;
  }
  // four columns at a time (N and the tile's columns come in eights), eight pieces requested before the first is used
#pragma unroll 1
  for (int i0 = 0; i0 < BM * UNITS / NT; i0 += 8) {
    f32x4 c[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int e = (i0 + i) * NT + tid, row = e / UNITS, unit = e % UNITS;
      if (m0 + row < M && n0 + unit * 4 < N) c[i] = *(const f32x4*)(C + (m0 + row) * N + n0 + unit * 4);
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int e = (i0 + i) * NT + tid, row = e / UNITS, unit = e % UNITS;
      if (m0 + row < M && n0 + unit * 4 < N)
        *(f32x4*)(C + (m0 + row) * N + n0 + unit * 4) = c[i] + *(const f32x4*)(stf + row * BN + (unit ^ (row & (UNITS - 1))) * 4);
    }
  }
}

}  // namespace

static bool wide(int64_t M, int64_t N) { return M >= (1 << 23) || N >= (1 << 23); }   // 64 rows in a raw buffer: below 2^31 bytes

bool gemm_tn_acc_supported(int32_t dtype, const void* A, const void* B, int64_t M, int64_t N, int64_t K) {
  // (K steps are counted in 32 bits; operands of 2^36 rows would take a terabyte)
  return dtype == PF_DTYPE_BF16_ && M >= 8 && N >= 8 && M % 8 == 0 && N % 8 == 0 && K >= 8 && K % (wide(M, N) ? 64 : 8) == 0 &&
         K < ((int64_t)1 << 36) && (((uintptr_t)A | (uintptr_t)B) & 15) == 0;
}

// The 128x128 tiles of this kernel reach 610 (8192 x 8192, K = 2048) to 810 TFLOP/s; the NT kernel's 256-wide tiles about 900 on
// results large enough to fill the chip with them, but it needs both operands transposed first (4 K (M + N) bytes at about
// 4 TB/s).  Equating the two at 650 gives M N / (M + N) = 1170 (8192 x 8192, K = 2048: 448 us here, 324 there): below that, or when 256x256 tiles would leave CUs idle,
// this kernel is the faster way to a weight gradient.
bool gemm_tn_acc_preferred(int64_t M, int64_t N, int64_t K) {
  // The NT kernel's tiled forms take whole K steps only.  Up to 192 tiles its ring kernel and two transposes are faster (600 tokens,
  // inside a training step: 2048 x 512 16.5 us in all, 19.6 here; 10048 x 512 50 and 23).  Otherwise K cancels out.
  if (K % 64 != 0) return ((M + 127) / 128) * ((N + 127) / 128) > 192;
  const int64_t big_tiles = ((M + 255) / 256) * ((N + 255) / 256);
  return big_tiles < 256 || M * N < 1170 * (M + N);
}

// Slices of K per tile.  Measured on MI355X (us, one / two / four / eight slices): 4096 x 1024, K = 8192 95 / 85 / 102 / 139;
// 3072 x 1024 104 / 76 / 95 / 121; 1024 x 1024 87 / 49 / 39 / 48, K = 2048 29.5 / 19.6 / 21.4 / 33; 1280 x 1280, K = 2048 31.2 / 23.7 /
// 30.3; 832 x 1472, K = 1152 21.2 / 15.4 / 22.4; 2304 x 768, K = 2048 29.8 / 23.7 / 31.1, K = 1024 16.5 / 17.7 / 27.3; 2048 x 2048, K =
// 4096 55 / 58 / 80 / 125.  A workgroup takes 6 us and 0.56 to 0.82 us a K step, by how many of them share the chip; one that keeps
// its whole K waits for C as well, and the longer its K the less of the operands is in L2 (up to 5.9 us); slices add their fp32
// tiles with atomics, 0.56 us per MiB while every workgroup has a CU, 0.83 beyond.  Fitted to 450 sizes timed with every number of
// slices: 0.7 % off the fastest on average.  Fewer than six steps stay together (4608 x 64, K = 256 8.7 / 9.6)
// unless the result is small (64 x 376, K = 256 8.3 / 7.5); more come in slices of two where few tiles make that the fastest (64 x 64,
// K = 704 8.1 us with four slices, 9.3 with two).
static int32_t tn_slices(int64_t M, int64_t N, int64_t K) {
  const int64_t tiles = ((M + 127) / 128) * ((N + 127) / 128), steps = (K + 63) / 64;
  const double mib = (double)M * (double)N * 4.0 / 1048576.0;
  int32_t best = 1;
  double best_t = -1.0;
  for (int32_t s = 1; s <= 16; s *= 2) {
    const int64_t share = (steps + s - 1) / s, wgs = tiles * s;
    if (s > 1 && ((steps < 6 && mib > 0.3) || share < 2 || share * (s - 1) >= steps || wgs > 512)) break;
    const double step = wgs <= 128 ? 0.56 : wgs <= 256 ? 0.65 : 0.82;
    const double unsplit = s == 1 ? std::min(5.9, 0.17 * (double)share) : 0.0;
    double t = (double)((wgs + 511) / 512) * (6.0 + unsplit + (double)share * step);
    if (s > 1) t += (wgs <= 256 ? 0.56 : 0.83) * mib * s;
    if (best_t < 0 || t < best_t) {
      best_t = t;
      best = s;
    }
  }
  return best;
}

hipError_t gemm_tn_acc(int32_t dtype, const void* A, const void* B, float* C, float* colsum, int64_t M, int64_t N,
                       int64_t K, hipStream_t stream) {
  if (!gemm_tn_acc_supported(dtype, A, B, M, N, K)) return hipErrorInvalidValue;
  const int64_t tiles_m = (M + 127) / 128, tiles_n = (N + 127) / 128, tiles = tiles_m * tiles_n;
  if (tiles > 0x7fffffff) return hipErrorInvalidValue;
  const int best = (int)tn_slices(M, N, K);
  static bool attr[4] = {false, false, false, false};
  auto launch = [&](auto kern, bool* attr_set) {
    if (!*attr_set) {
      hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, 65536);
      if (e != hipSuccess) return e;
      *attr_set = true;
    }
    hipLaunchKernelGGL(kern, dim3((unsigned)tiles, (unsigned)best), dim3(256), 65536, stream, (const bf16_t*)A,
                       (const bf16_t*)B, C, colsum, M, N, K, (int32_t)tiles_m, (int32_t)tiles_n);
    return hipGetLastError();
  };
  if (wide(M, N)) {
    if (colsum) return launch(gemm_bf16_tn_acc_kernel<true, true>, &attr[2]);
    return launch(gemm_bf16_tn_acc_kernel<false, true>, &attr[3]);
  }
  if (colsum) return launch(gemm_bf16_tn_acc_kernel<true, false>, &attr[0]);
  return launch(gemm_bf16_tn_acc_kernel<false, false>, &attr[1]);
}

}  // namespace pf

// For tests: K slices of a weight gradient.
extern "C" int32_t pf_gemm_tn_slices(int64_t M, int64_t N, int64_t K) { return pf::tn_slices(M, N, K); }
// For tests: the kernel itself, which takes K in eights (pf_op_gemm_tn: whole steps only); 0 or -1.
extern "C" int32_t pf_gemm_tn_eights(const void* A, const void* B, float* C, float* colsum, int64_t M, int64_t N, int64_t K,
                                     void* stream) {
  return pf::gemm_tn_acc(pf::PF_DTYPE_BF16_, A, B, C, colsum, M, N, K, (hipStream_t)stream) == hipSuccess ? 0 : -1;
}
