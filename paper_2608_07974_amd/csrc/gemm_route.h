// Which kernel a bf16 GEMM takes: tile, splits of K and copy path, from its
// sizes alone.  Host arithmetic without HIP, so that it can be checked on the
// CPU.
#pragma once

#include <cstddef>
#include <cstdint>

namespace zl {

// What the choice depends on.  may_split: the epilogue allows a split and
// there is a workspace of part_elems floats.  heads: the RoPE or delta
// epilogue over heads of hd columns.
struct GemmShape {
  int M, N, K;
  bool ak, bk;  // A, B K-major
  bool may_split;
  size_t part_elems;
  bool heads;
  int hd;
};

// Tile size and splits of K below 240 large tiles, by an estimate of the launch's
// time from its sizes alone (microseconds; rates fitted to launches of the GPT-2,
// Llama-1B and 8B shapes at 128 to 16384 tokens, two and three stages deep):
//  - a 256 x 256 tile has a CU for itself and takes 0.027 per unit of K; its
//    prologue and epilogue about 12;
//  - a 128 x 128 tile shares its CU with a second one once there are more
//    than 256: 0.018 - 0.020 per unit of K by layout for 512 of them, 0.011 -
//    0.0125 up to 256, in proportion between; ends about 8;
//  - splitting K over nz blocks writes and reads nz fp32 partials (at about
//    4 TB/s) and adds the launch that sums them (5).
// It ranks the choices, no more: it counts the ends once per launch and knows
// neither the epilogue's kind nor the deeper pipeline of deep_stages.  No more
// splits than 256 of K each; split_k rounds their depth up to the k tile, so
// the last may be shorter and there may be fewer.  The partials stay within the
// workspace.  What it replaced - 128 x 128 tiles split to the next multiple above
// 256 blocks - took two waves of blocks where one does (48 tiles x 6 = 288
// blocks: 511 us; x 5: one wave), 192 large tiles as 768 small ones, and 256 x 256
// tiles always for the RoPE and delta epilogues (3 - 48 blocks).
struct GemmPlan {
  bool large;
  int nz;
};
inline GemmPlan plan_gemm(const GemmShape& g) {
  const long t256 = (long)((g.M + 255) / 256) * ((g.N + 255) / 256);
  const long t128 = (long)((g.M + 127) / 128) * ((g.N + 127) / 128);
  const double alone = g.ak ? 0.0125 : 0.011;
  const double two = g.ak && g.bk ? 0.020 : 0.018;
  const double mn = (double)g.M * g.N;
  long most = 1;  // splits allowed
  if (g.may_split) {
    most = g.K / 256;
    const long by_ws = (long)((double)g.part_elems / mn);
    if (most > by_ws) most = by_ws;
    if (most > 64) most = 64;
    if (most < 1) most = 1;
  }
  // From 240 large tiles up that are not mostly padding (an eighth at most; 80
  // rows of logits take 117 us as 1002 small tiles, 147 as 501 large ones) the
  // estimate decides nothing: large tiles, unless their last round would leave
  // three quarters of the chip idle, or half of it at a short K.  Measured at 64 to
  // 6144 of K in the three layouts, small over large is 0.83 - 0.95 at 288 and 320
  // tiles; at 376 and 384 0.89 - 1.01 to K 256, 1.04 - 1.14 from 768; at 564 to 640
  // 0.91 - 0.98 to K 768, 1.00 above and 1.05 - 1.10 at K 8192 - 16384; 1.08 - 1.24 at
  // 240 and 256 of K 256, 1.03 - 1.15 at 400 to 512 and from 672 up.
  if (t256 >= 240 && 2 * t128 >= 7 * t256) {
    const long last = (t256 - 1) % 256 + 1;
    const bool small = t256 > 256 && t256 <= 640 &&
                       ((t256 <= 512 && last <= 64) || (last <= 128 && g.K <= (t256 <= 512 ? 256 : 768)));
    return {!small, 1};
  }
  GemmPlan best = {true, 1};
  double tb = 0.;
  for (int large = 1; large >= 0; --large) {
    const long t = large ? t256 : t128;
    for (long nz = 1; nz <= most; ++nz) {
      // more blocks than two rounds need no further split
      if (nz > 1 && t * nz > 1024) break;
      const long b = t * nz;
      const double k = (double)g.K / nz;
      double c;
      if (large) {
        c = (double)((b + 255) / 256) * k * 0.027 + 12.;
      } else {
        const long full = b / 512, rem = b % 512;
        const double last = rem <= 256 ? alone : alone + (two - alone) * (rem - 256) / 256.;
        c = k * (full * two + (rem == 0 ? 0. : last)) + 8.;
      }
      if (nz > 1) c += 5. + nz * mn * 8. / 4e6;
      if (tb == 0. || c < tb) {
        tb = c;
        best = {large != 0, (int)nz};
      }
    }
  }
  return best;
}

// K per split, a multiple of the k tile, so every split but the last is
// whole; returns the number of splits.
inline int split_k(int K, int nz, int bk, int& ksplit) {
  ksplit = ((K + nz - 1) / nz + bk - 1) / bk * bk;
  if (nz <= 1 || ksplit >= K) { ksplit = K; return 1; }
  return (K + ksplit - 1) / ksplit;
}

// The direct-to-LDS path copies whole 16-byte chunks with 32-bit buffer
// offsets from the tile origin: every chunk it reads must be either fully
// valid or fully outside (K-major: valid k a multiple of 8; MN-major: the
// M or N extent a multiple of 8), rows 16-byte aligned, and the largest
// offset below 2^31.
inline bool dma_operand_ok(const void* p, int64_t ld, bool kmaj, int rows, int kvalid, int R) {
  if (reinterpret_cast<uintptr_t>(p) % 16 != 0 || ld % 8 != 0) return false;
  const int64_t lim = (int64_t)1 << 31;
  if (kmaj) return kvalid % 8 == 0 && ((int64_t)R * ld + kvalid + 64) * 2 < lim;
  return rows % 8 == 0 && ((int64_t)(kvalid + 64) * ld + R) * 2 < lim;
}

// Whether 128 x 128 tiles of 64-column wave tiles keep 256 of K in flight (128 KB of
// stages, one block per CU) instead of two or three k tiles (48 - 64 KB).  Both
// operands K-major: at any K (all forward GEMMs of a Llama-1B layer at 64 to 512
// tokens 214 - 325 us against 227 - 343).  With an MN-major operand the eight
// stages fill with as many copies of 32 k first, which pays where a block's K
// is long or the blocks together load the memory: data and weight gradients of a
// GPT-2 layer at 256 tokens 160 and 109 us against 150 and 104 with three
// stages, at 8192 tokens 522 and 524 against 534 and 571; at 2048 tokens (295000
// of K over all blocks) both are even.
inline bool deep_stages(bool ak, bool bk, long blocks, int k) {
  if (blocks > 256) return false;
  return (ak && bk) || k >= 8192 || (double)blocks * k > 3e5;
}

enum GemmTile {
  TILE_256,       // 256 x 256, 128-column wave tiles
  TILE_128,       // 128 x 128, 64-column wave tiles
  TILE_128_WIDE,  // 128 x 128, 128-column wave tiles (direct-to-LDS, A K-major)
};
inline int wave_columns(GemmTile t) { return t == TILE_128 ? 64 : 128; }

struct GemmRoute {
  GemmTile tile;
  bool dma;  // direct-to-LDS copies, else the register-staged kernel
  int nz;    // splits of K (of the direct-to-LDS kernels)
};

// dma_ok(R): the direct-to-LDS path can copy every operand in tiles of R rows.
// The RoPE and delta epilogues work on whole heads inside a wave tile: heads of
// 128 need 128 columns, which the register-staged kernel has in its large tile
// only.
template <typename F>
GemmRoute route_gemm(const GemmShape& g, F&& dma_ok) {
  const GemmPlan plan = plan_gemm(g);
  GemmRoute r = {plan.large ? TILE_256 : TILE_128, false, plan.nz};
  if (g.heads && !plan.large) {
    if (!g.ak) r = {TILE_256, false, 1};  // no projection of the chunk has an MN-major A
    else if (g.hd > 64) r.tile = TILE_128_WIDE;
  }
  r.dma = dma_ok(r.tile == TILE_256 ? 256 : 128);
  if (!r.dma) {
    if (r.tile == TILE_128_WIDE) r.tile = TILE_256;
    r.nz = 1;
  }
  return r;
}

// Products of few columns (N <= 64, np of them with the same M in one launch):
// whole rows per block (gemm_skinny.hip) or the tiles above, by estimates of
// both (microseconds) fitted to launches of 8 - 32768 rows, 8 - 64 columns and K
// 64 - 65536.  A row block takes 1.1 / 1.57 / 2.1 / 3.4 per 1024 of K at up to 8 /
// 16 / 32 / 64 columns, more in proportion past 256 blocks of 16 rows, and no
// less than reading A at 5.2 TB/s; tiles can split K where there is a
// workspace.  Near a tie (5 %) it is tiles, whose estimate is the closer one.
// (8192 x 64 x 14336 with a workspace: 126 us as rows against 47; 1024 x 8 x 2048:
// 5 against 13.)
inline bool skinny_better(const GemmShape* g, int np) {
  double lat = 0., all = 0., bytes = 0., tiles = 0.;
  for (int i = 0; i < np; ++i) {
    const int N = g[i].N;
    const double per = (N <= 8 ? 1.1 : N <= 16 ? 1.57 : N <= 32 ? 2.1 : 3.4) * (g[i].bk ? 1. : 0.9);
    const double one = g[i].K / 1024. * per;
    if (one > lat) lat = one;
    all += one * 1.15 * ((g[i].M + 15) / 16) / 256.;
    bytes += (double)g[i].M * g[i].K * 2. / 5.2e6;
    const int nz = plan_gemm(g[i]).nz;
    const double blocks = (double)((g[i].M + 127) / 128) * ((N + 127) / 128) * nz;
    tiles += 8.4 + (double)g[i].K / nz * (0.007 + 0.005 * blocks / 256.) +
             (nz > 1 ? nz * (0.062 + (double)g[i].M * N * 8. / 5.5e6) : 0.);
  }
  const double rows = 3.2 + (lat > all ? (lat > bytes ? lat : bytes) : (all > bytes ? all : bytes));
  return rows < 0.95 * tiles;
}

// fp32 GEMMs: 64 x 64 tiles on the vector ALUs, else 32 x 32 tiles on fp32 MFMA.
// The small tiles fill the chip and load 128 of K per round trip; the large ones
// read each operand half as often and do not pad K to 128, and win from this
// many tiles up (4096 x 4096 x 2048, both K-major: 1117 us against 2012; at
// 1024 x 768 x 2048: 317 against 107; crossings measured at K 8 to 1024).  Both
// operands MN-major the small tiles load without a transpose and win at any
// count where K fills its tiles (4096 x 4096 x 2048: 1041 against 809).
inline bool f32_large_tiles(int M, int N, int K, bool ak, bool bk) {
  const double tiles = (double)((M + 63) / 64) * ((N + 63) / 64);
  const double fill = K > 0 ? K / (double)((K + 127) / 128 * 128) : 1.;
  if (!ak && !bk) return fill < 0.8 && tiles > 1500. * fill;
  return tiles > (ak && bk ? 500. : 800.) * fill;
}

}  // namespace zl
