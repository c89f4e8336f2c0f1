// Which GEMM kernel runs a product: estimated times, measured constants (MI355X).
#include "gemm_route.h"

#include "pf_internal.h"

#include <algorithm>

namespace pf {
namespace gemm {
namespace {

int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

// Ring kernel, tile shapes.  bf16: time of a round of up to 256 workgroups (one per CU) = fixed + per_byte x bytes of a row of
// X, in microseconds, measured on MI355X over K = 256 .. 8192.  The small tile moves twice the bytes of the 64x64 one per
// product but spreads them over four times the CUs; on few CUs its bytes come faster (one tile 0.00062 us each).
// odd: what a round costs more when columns don't come in fours and every thread goes through its share of C element by
// element (one group of four with the 32x32 tile, eleven with 128x64).  These are times with two LDS stages a wave; one stage
// (ring_form) is up to a third faster, which the choice between tiles does not see: over 846 products of small grids, bf16 and
// fp32, every tile and form timed, it is 0.4 % off the fastest on average, by more than a tenth in six (1536 x 1024, K = 512 in fp32
// 28.2 us on 64x64 tiles, 23.5 on 32x64).
struct RingShape { int bm, bn; double fixed, byte, odd; };
constexpr RingShape ring_shapes[] = {
    {32, 32, 2.6, 0.00098, 0.9}, {32, 64, 3.5, 0.0014, 2.2}, {64, 64, 4.6, 0.0017, 2.9}, {128, 64, 7.9, 0.0032, 9.4}};
// fp32: start + rounds x (fixed + per_k x K), K rounded up to the elements that all waves of the workgroup take in one step
// where few waves make that visible (64x64: of its four-wave form, ring_form).  Bound by the MFMAs (64 cycles for two K), which small tiles hide best: 2048 x 576,
// K = 512 25 / 28 / 28 / 33 us, K = 1024 on 2048 x 2048 124 / 127 / 87 / 105 us (32x32, 32x64, 64x64, 128x64).  The 128x64
// tile wins by up to a tenth where it saves a round and K fits two steps (2048 x 2048, K = 192: 32.3 us, 64x64 35.3).
struct RingShapeF32 { double start, fixed, per_k; int step; };
constexpr RingShapeF32 ring_shapes_f32[] = {{1.5, 2.0, 0.0055, 1}, {1.2, 2.9, 0.0125, 1}, {1.0, 4.1, 0.017, 128}, {0.5, 7.4, 0.0417, 96}};

double ring_estimate(const Product& p, Kernel* shape) {
  double best = 1e30;
  for (int i = 0; i < 4; ++i) {
    const RingShape& s = ring_shapes[i];
    const int64_t tiles = ceil_div(p.M, s.bm) * ceil_div(p.N, s.bn);
    const double rounds = (double)ceil_div(tiles, 256);
    const double byte = i == 0 ? 0.00062 + 0.00036 * (double)std::min<int64_t>(tiles, 256) / 256 : s.byte;
    const double odd = p.N % 4 ? s.odd : 0.0;
    double t = rounds * (s.fixed + odd + byte * (double)(p.K * 2));
    if (!p.bf16) {
      const RingShapeF32& f = ring_shapes_f32[i];
      t = f.start + rounds * (f.fixed + odd + f.per_k * (double)(ceil_div(p.K, f.step) * f.step));
    }
    if (t < best) {
      best = t;
      *shape = (Kernel)(RING_32x32 + i);
    }
  }
  return best;
}

// One LDS stage a wave, or two (deep)?  Measured on MI355X (us, one stage / two).  An fp32 step is 1024 cycles of MFMAs: a second
// stage hides the next step's wait behind them as soon as a wave has more than one step.  In bf16 the steps are short and the
// waves per SIMD, not their stages, hide the waits until a row is long.
//  * fp32 64x64: one step of every wave is 256 elements.  512 x 512, K = 256 8.8 / 9.9, K = 264 12.2 / 12.0, K = 320 14.0 / 12.0,
//    K = 1024 31.8 / 23.6, K = 4096 112 / 75; 2048 x 1024, K = 640 41.8 / 33.3.
//  * fp32 32x64: nine or ten steps are two for some waves, be they six or eight.  512 x 512, K = 256 6.1 / 7.2, K = 264 7.7 / 7.2,
//    K = 320 8.0 / 7.5, K = 352 8.1 / 8.5, K = 512 10.0 / 10.8.  Beyond one round of tiles one stage is no slower: 1024 x 1024,
//    K = 320 14.1 / 14.4.
//  * fp32 32x32: two workgroups per CU with one stage, one with two.  Alike on one round of tiles (512 x 512, K = 4096 29.4 / 29.5).
//    More: 600 x 512, K = 512 10.9 / 11.4, K = 1056 19.2 / 18.7, K = 2048 34.0 / 29.9, K = 8192 119 / 94; 1024 x 1024, K = 1024
//    32.8 / 33.8, K = 1568 48.2 / 47.7, K = 4096 119 / 102.  The last of three nearly full rounds leaves half of the CUs with two
//    workgroups and the others idle where two fit (704 x 1024, K = 228 10.3 / 11.8, K = 292 14.2 / 13.5, K = 932 29.6 / 26.8), the last
//    of five a little (1280 x 1024, K = 1060 46.2 / 45.7, K = 1572 64.2 / 60.4).
//  * bf16 64x64: 333 x 2048, K = 2048 10.7 / 11.2, K = 3136 14.0 / 14.3, K = 4096 17.1 / 16.5, K = 8192 29.9 / 29.0.
//  * bf16 32x32, one round of tiles, K from 1024 on: up to eight rows (nearly all operand bytes are W's) 1 x 208, K = 11392 15.1 /
//    13.7, 3 x 952, K = 4224 8.1 / 7.6, 8 x 1472, K = 4864 8.7 / 8.2; rows that don't start on a cache line 46 x 896, K = 1688 6.1 /
//    5.8, 43 x 2528, K = 3288 9.9 / 9.3; but 128 x 768, K = 1088 4.1 / 4.4, 512 x 512, K = 4096 8.9 / 9.3 and, with two workgroups
//    per CU, 1024 x 1024, K = 2048 14.6 / 19.4.
Kernel ring_form(const Product& p, Kernel shape) {
  const int64_t tiles_n64 = ceil_div(p.N, 64), t32 = ceil_div(p.M, 32) * ceil_div(p.N, 32);
  if (p.bf16) {
    if (shape == RING_64x64 && p.K > 2048) return RING_64x64_DEEP;
    if (shape == RING_32x32 && t32 <= 256 && p.K >= 1024 && (p.M <= 8 || p.K % 64 != 0)) return RING_32x32_DEEP;
    return shape;
  }
  if (shape == RING_64x64 && p.K > 256) return RING_64x64_DEEP;
  if (shape == RING_32x64 && p.K > 256 && p.K <= 320 && ceil_div(p.M, 32) * tiles_n64 <= 256) return RING_32x64_DEEP;
  if (shape == RING_32x32 && t32 > 256) {
    const int64_t rounds = ceil_div(t32, 256);
    const bool last_full = t32 > rounds * 256 - 128;
    const int64_t longest = rounds == 2 ? 1024 : rounds == 3 && last_full ? 256 : rounds == 5 && last_full ? 1056 : 1536;
    if (p.K > longest) return RING_32x32_DEEP;
  }
  return shape;
}

// Generic bf16 kernel on up to 256 whole tiles: a memory latency per K step, and C's layout read 32 rows at a time.
double generic_estimate(const Product& p) {
  return 5.8 + 0.98 * (double)ceil_div(p.K, 64) + (p.epi & (E_ACC | E_RESID | E_DACT) ? 5.7 : 0.0);
}

// fp32 FMA kernel (64x64 tiles, many workgroups per CU): one workgroup's own time, or the chip's rate.
double fma_estimate(const Product& p) {
  const double tiles = (double)(ceil_div(p.M, 64) * ceil_div(p.N, 64)), k = (double)p.K;
  return std::max(5.5 + 0.093 * k + 0.003 * tiles, 2.5 + tiles / 256 * (1.8 + 0.03 * k));
}

// 256x256 tiles with 16x16x32 MFMAs instead of 32x32x16: where the power limit sets the rate, i.e. on a chip that is full nearly
// all the time, and K is long enough for that to outweigh the slower start.  Measured on MI355X both alone (1660 pairs of results
// and epilogues, time with 16x16x32 by time with 32x32x16) and inside whole passes of 2 to 11 layers (146 passes, all such products
// of one by either form), which keep the chip at its power limit and decide where the two disagree:
//  * one round: alone, filled to 0.93 or more, K < 512 1.07, 512 .. 1000 1.04, 1400 .. 2000 0.98, 2048 0.98, from 4096 on 0.96; passes 0.96
//    to 1.00 from K = 1024 on (3840 x 4352, K = 1088 545 -> 523 us of three layers), 0.97 to 1.01 below; filled less 1.00 to 1.04 (160
//    to 225 tiles: 3804 x 2688, K = 10752 661 -> 689).
//  * more rounds, filled to 0.74 or more, K from 1024 on: passes 0.96 to 1.01, 0.985 on average (16384 x 4904, K = 1472 3217 -> 3095,
//    8192 x 6192, K = 1536 2162 -> 2097, 14720 x 4864, K = 1216 2132 -> 2157); alone 0.96 to 1.03 (4096 x 7168, K = 2112 108 -> 111).
//  * more rounds, K 512 .. 1000: passes 0.988 on average filled to 0.9 (17920 x 3384, K = 832 1697 -> 1652, 20480 x 3840, K = 960 1890 ->
//    1908), 1.00 below that (18 of them 0.98 to 1.01); alone 1.04.  K = 320 alone: 15632 x 7832 120 -> 137.
bool by_16(const Product& p) {
  const int64_t tiles = ceil_div(p.M, 256) * ceil_div(p.N, 256);
  const double filled = (double)tiles / (double)(256 * ceil_div(tiles, 256));
  if (tiles <= 256) return p.K >= 1024 && filled >= 0.93;
  return (p.K >= 1024 && filled >= 0.74) || (p.K >= 512 && filled >= 0.9);
}

// Tiled kernels, and the ring kernel where it is faster.
// Tile shapes: 256x256 (four waves, wave tile 128x128), 256x192 (8 waves as 4x2, wave tile 64x96) and 256x128 (four waves, wave
// tile 128x64), one workgroup per CU, and 128x128 (4 waves, two workgroups per CU).
// A 128x128 grid that leaves every workgroup a CU of its own gets four LDS stages instead of two; 128x64 tiles below.
// A launch takes ceil(workgroups / resident workgroups) rounds of start + step x (K steps of 64), in microseconds, measured
// on MI355X; the shape with the least estimate runs.  On 520 random products, every shape (and number of slices) timed: rows in
// eights and K from 512 on 0.8 % off the fastest on average, 3 of 211 by more than a tenth (774 x 9560, K = 1856: 256x192 tiles
// 45.5 us, 256x256 40.4); shorter K 1.9 %, 9 of 125 (5753 x 7744, K = 192 with GELU 53.9, 128x128 45.3).  Sums 4.6 %, 22 of 136, and
// other rows 5 %, 7 of 48: there the 128x64 tile, which is not among the candidates, would be the fastest (284 x 4096, K = 1408
// into fp32 18.3, 10.8).  E.g. N = 768 or 2304
// fills whole rounds with 192-wide tiles but wastes a quarter of the last round with 256-wide ones, and a 8192 x 1024
// result gives every CU work only with the small tile.  (A chip full of 256-wide tiles runs at 1.3 to 1.5 times these
// step times, every shape alike: the power limit.)  Partial tiles along N cost a shape nothing beyond the area they waste
// (4096 x 3456, K = 2048: 256x256 tiles 54 us, whole 128x128 ones 71).  Rows that do not come in fours go element by
// element, a fixed time per round that grows with the elements of a wave (odd; odd_read where an operand of C's layout is
// read as well).  So do GELU and the way of GELU' through LDS (dact: 8192 x 9648, K = 320 218 us on 256x256 tiles, 139 on
// 128x128 ones).
// Accumulating fp32 launches (weight gradients: small M x N, K = all tokens) may split K over up to 8 workgroups
// per 128x128 tile while that fills idle CUs and leaves each >= 8 K steps; the slices add into C with fp32 atomics
// (order-dependent in the last bits, like the other atomic reductions over tokens).  Those atomics go at about
// 1.5 TB/s on MI355X, far below plain stores, so the estimate charges every slice for its tile: two slices usually
// pay, eight rarely do.  Slices that leave some CUs with one workgroup are charged between the alone and the paired
// rate, fitted to the loop by slices of fragments.  With the present one, us: 1024 x 3072, K = 8192 unsplit 60.0, two slices 71.5 (which
// are chosen); 2048 x 1536 55.4 and 66.5; K = 4096 31.2 and 46.4; 768 x 1536, K = 8192 two slices 34.0, four 43.8 (chosen).  (256-wide tiles with split K were measured too: their atomic bursts at the end of the one
// round are not hidden by anything and they lose to the small tile on every weight-gradient shape tried.)
Route tiled_route(const Product& p) {
  struct Shape { Kernel kernel; int bm, bn, resident; double start, step, odd, odd_read, gelu, dact; };
  // 128x128 and 256x128: a whole K step of fragments in registers, timed for rows of whole 16-byte pieces, K from 512 on and
  // no sum into C (8192 x 1024, K = 4096 58.6 us with both; K = 50304 858 and 725).  Elsewhere a pair of 128x128 tiles (and for
  // sums and other rows a lone one) is taken with the times of its loop by slices of fragments, which it no longer runs: its own
  // start and step are shorter, and the choice is as far off as stated above.
  const bool timed = p.N % 8 == 0 && p.K >= 512 && !(p.epi & E_ACC);
  const Shape pair = timed ? Shape{TILE_128x128, 128, 128, 512, 3.8, 0.82, 11, 25, 1, 0} : Shape{TILE_128x128, 128, 128, 512, 4.1, 1.02, 11, 25, 1, 0};
  const Shape shapes[4] = {{TILE_256x256, 256, 256, 256, 8.0, 1.06, 44, 76, 5, 16}, {TILE_256x192, 256, 192, 256, 6.0, 1.1, 20, 42, 4, 4},
                           pair, {TILE_256x128, 256, 128, 256, 6.3, 0.69, 0, 0, 2.5, 2}};
  // a 128x128 workgroup that has its CU, and four stages, to itself; with nearly every CU busy a step takes longer
  // (K = 2048: 144 workgroups 16.3 us, 256 20.5)
  const double busy = std::min(1.0, std::max(0.0, ((double)(ceil_div(p.M, 128) * ceil_div(p.N, 128)) - 144) / 64));
  const bool whole = p.N % 8 == 0 && !(p.epi & E_ACC);   // any K: 1659 x 960 with residual K = 64 5.6 us, 512 8.2, 1024 10.8
  const double lone_start = whole ? 4.7 : 3.65, lone_step = timed ? 0.36 + 0.14 * busy : whole ? 0.36 : 0.608;
  const bool reads = (p.epi & (E_ACC | E_RESID | E_DACT)) != 0;
  Route best{TILE_256x256, 1};
  double best_time = 1e30;
  for (const Shape& sh : shapes) {
    const int64_t tiles = ceil_div(p.M, sh.bm) * ceil_div(p.N, sh.bn);
    const bool small = sh.kernel == TILE_128x128;
    if (sh.kernel == TILE_256x128 && !timed) continue;
    const int max_splits = p.out_f32 && p.epi == E_ACC && small ? 8 : 1;
    for (int splits = 1; splits <= max_splits; splits *= 2) {
      // a slice keeps >= 8 K steps, and splitting only fills CUs that would otherwise idle
      if (splits > 1 && (p.K % (128 * splits) != 0 || p.K / (128 * splits) < 8 || tiles * splits > sh.resident)) break;
      const int64_t wgs = tiles * splits;
      const bool alone = small && wgs <= 256;
      // share of the CUs that run two workgroups, as far as it shows in the time
      const double paired = alone ? 0.0 : splits > 1 && wgs < 512 ? std::max(0.55, (double)(wgs - 256) / 256) : 1.0;
      const double start = small ? lone_start + paired * (sh.start - lone_start) : sh.start;
      const double step = small ? lone_step + paired * (sh.step - lone_step) : sh.step;
      const double odd = p.N % 4 == 0 || splits > 1 ? 0.0 : reads ? sh.odd_read : sh.odd;
      double act = p.epi & E_DACT ? sh.dact : p.epi & E_GELU && !alone ? sh.gelu : 0.0;
      // (up to 32 rows, weights from memory, us on 128x128 / 32x64 ring tiles: GELU hides behind the other waves' waits, 32 x 19968, K =
      // 4992 49.7 / 51.3, with a copy 24 x 18856, K = 5760 55.8 / 56.9; GELU' costs more than a second round of a few ring tiles, 16 x
      // 17408, K = 4352 44.4 / 42.2, 8 x 16912, K = 5312 50.4 / 48.4, but no more than one of 40, 32 x 19968, K = 4992 50.9 / 51.5)
      if (alone && whole && p.M <= 32) act = p.epi & E_DACT && busy == 0.0 ? 2.5 : 0.0;
      else if (alone && whole) act = p.epi & E_DACT ? 2.5 : p.epi & E_PRE ? 1.6 : p.epi & E_GELU ? 0.9 : 0.0;
      double t = (double)ceil_div(wgs, sh.resident) * (start + odd + act + step * (double)(p.K / (64 * splits)));
      // every slice adds its whole fp32 tile with atomics: about 0.67 us per MiB, and 2.5 us whatever its size (128 x 128,
      // K = 4096: 25.9, 16.6 and 11.9 us with two, four and eight slices)
      if (splits > 1) t += (double)(p.M * p.N * splits) * 2.63e-6 + 2.5;
      if (t < best_time) {
        best_time = t;
        best = Route{alone ? TILE_128x128_DEEP : sh.kernel, splits};
      }
    }
  }
  // 128x64 tiles, six LDS stages, one workgroup per CU: where 128x128 ones leave half of the CUs idle (us, 128x128 deep / 128x64:
  // 1659 x 768, K = 64 5.4 / 4.8, K = 768 9.4 / 8.1, K = 3072 22.6 / 18.6; 1659 x 960, K = 768 9.6 / 8.2; 1659 x 1024, K = 4096 26.2 /
  // 21.9; 600 x 2048, K = 2048 15.4 / 12.1; 1000 x 2048, K = 8192 63.8 / 50.7, ring 53.3; 333 x 6144, K = 2048 16.4 / 23.9; with a
  // second result 1024 x 2048, K = 1024 13.3 / 15.3).
  if (whole) {
    const int64_t wgs = ceil_div(p.M, 128) * ceil_div(p.N, 64);
    const double step = 0.28 + 0.06 * std::min(1.0, std::max(0.0, (double)(wgs - 208) / 48));
    const double act = p.epi & E_PRE ? 3.0 : p.epi & E_DACT ? 1.6 : p.epi & E_GELU ? 0.3 : 0.0;
    const double t = (double)ceil_div(wgs, 256) * (4.4 + act + step * (double)(p.K / 64));
    if (t < best_time) {
      best_time = t;
      best = Route{TILE_128x64, 1};
    }
  }
  // The ring kernel takes what leaves the chip idle or waiting: 128 x 768, K = 3072 38.5 -> 7.5 us; 333 x 2048, K = 8192
  // 122 -> 30 us (four stages: 58).
  Kernel ring;
  if (ring_estimate(p, &ring) < best_time) return Route{ring_form(p, ring), 1};
  if (best.kernel == TILE_256x256 && by_16(p)) best.kernel = TILE_256x256_16;
  return best;
}

bool tiled(const Product& p) {
  if (p.K % 64 != 0 || !p.aligned || p.scaled) return false;
  if (p.K >= 1 << 22) return false;   // 256 rows of an operand are one raw buffer, below 2^31 bytes
  if (p.out_f32) return p.epi == 0 || p.epi == E_ACC;
  return p.epi == 0 || p.epi == E_BIAS || p.epi == (E_BIAS | E_GELU) || p.epi == (E_BIAS | E_RESID) ||
         p.epi == (E_BIAS | E_GELU | E_PRE) || p.epi == E_DACT;
}

}  // namespace

Route route(const Product& p) {
  Kernel ring;
  if (!p.bf16) {
    // The ring kernel takes 2048 x 512, K = 2048 from 297 to 41 us and 512 x 256, K = 1024 from 115 to 10, but one workgroup
    // a CU and rounds of 4 us lose where K is short and C large: 4096 x 2048, K = 64 45 us against 29, K = 128 60 against
    // 46, K = 192 61 against 61, K = 256 69 against 78; 2048 x 576, K = 32 12.1 against 9.6, K = 64 12.2 against 12.9.
    // (The FMA kernel's grid holds 65535 row tiles.)
    if (p.K % 4 != 0 || !p.aligned) return Route{F32_FMA, 1};
    if (fma_estimate(p) < ring_estimate(p, &ring) && ceil_div(p.M, 64) <= 65535) return Route{F32_FMA, 1};
    return Route{ring_form(p, ring), 1};
  }
  if (tiled(p)) return tiled_route(p);
  // The rest (K not a multiple of 64, scaled results, other combinations of epilogues).  Above 192 tiles of 128x128 the ring
  // kernel needs a round more (2048 x 1792, 224 tiles: K = 200 21.6 us against 15.5, K = 1000 34.3 against 28.2).  Up to there
  // the estimates decide, for C in whole tiles; a ragged C costs the generic kernel 7 us, and the ring kernel nothing.
  // Fitted to 32 .. 192 tiles, K = 40 .. 4104 (rows that don't start on a cache line cost the ring kernel 8 %); generic
  // against ring, us: 2048 x 1536 K = 200 9.6 / 14.5, K = 1000 20.1 / 23.2, K = 2008 38.3 / 33.9, accumulating into fp32
  // K = 600 21.2 / 22.1, K = 1000 27.6 / 26.8; 1024 x 2048 K = 40 6.8 / 8.3, K = 328 10.7 / 10.0; 512 x 512 K = 40 6.3 / 3.5.  (Ring
  // tiles with two LDS stages a wave.  With one, 2048 x 1536 takes 21.8 us at K = 1000 and, accumulating, 19.0 at K = 600, where the
  // generic kernel still runs.)
  if (p.aligned && ceil_div(p.M, 128) * ceil_div(p.N, 128) <= 192) {
    const double t = ring_estimate(p, &ring);
    const bool whole = p.M % 128 == 0 && p.N % 128 == 0;
    if (!whole || 1.08 * t < generic_estimate(p)) return Route{ring_form(p, ring), 1};
  }
  return Route{BF16_GENERIC, 1};
}

}  // namespace gemm
}  // namespace pf

extern "C" int32_t pf_gemm_route(int32_t dtype, int64_t M, int64_t N, int64_t K, int32_t epi, int32_t flags) {
  const pf::gemm::Route r = pf::gemm::route({dtype == PF_DTYPE_BF16, M, N, K, (flags & 1) == 0, (flags & 2) != 0, (flags & 4) != 0, epi});
  return r.kernel | r.splits << 8;
}
