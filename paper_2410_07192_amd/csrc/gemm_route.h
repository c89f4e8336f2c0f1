// Which GEMM kernel runs a product: host rules only (gemm_route.cpp), no device code.
#pragma once

#include <cstdint>

namespace pf {
namespace gemm {

// Epilogue features the tiled kernels are specialised on (so that its loads carry no branches and the
// compiler can batch them); other combinations run on the ring and the generic kernel.
enum : int { E_BIAS = 1, E_GELU = 2, E_RESID = 4, E_DACT = 8, E_PRE = 16, E_ACC = 32 };

enum Kernel : int32_t {
  F32_FMA,                                        // gemm.hip
  BF16_GENERIC,
  RING_32x32, RING_32x64, RING_64x64, RING_128x64,   // gemm_ring.hip, bf16 and fp32: eight waves with one LDS stage each; 128x64: three, two
  TILE_256x256, TILE_256x192, TILE_128x128,       // gemm_tile.h; the last with two LDS stages,
  TILE_128x128_DEEP,                              // here with four
  TILE_256x128,                                   // with three
  TILE_128x64,                                    // with six
  RING_32x32_DEEP, RING_32x64_DEEP, RING_64x64_DEEP, // the first three with two LDS stages a wave, on eight, six and four waves
  TILE_256x256_16,                                // 256x256 with 16x16x32 MFMAs
};

inline bool is_ring(Kernel k) { return (k >= RING_32x32 && k <= RING_128x64) || (k >= RING_32x32_DEEP && k <= RING_64x64_DEEP); }

struct Product {
  bool bf16;           // else fp32
  int64_t M, N, K;
  bool aligned;        // X and W to 16 bytes
  bool out_f32;
  bool scaled;         // result multiplied by something other than 1
  int epi;             // E_*
};

struct Route {
  Kernel kernel;
  int32_t splits;      // workgroups that share a tile's K (their sums meet through fp32 atomics)
};

Route route(const Product& p);

}  // namespace gemm
}  // namespace pf

// For tests: kernel | splits << 8 of a product (flags: 1 misaligned operands, 2 fp32 result, 4 scaled).
extern "C" int32_t pf_gemm_route(int32_t dtype, int64_t M, int64_t N, int64_t K, int32_t epi, int32_t flags);
