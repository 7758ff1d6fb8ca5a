// Output tiles of every contraction kind of the forward pipeline: the
// TileKinds<Prob> trait that the tile queues (tilequeue.hpp) build on, shared
// by the kernels that schedule (k_schedule, the sweep planner) and those
// that walk the queues.
#pragma once

#include "tilequeue.hpp"

namespace tebd {

// Sketch and power-iteration products (m x l, n x l): the sketch width l is
// a few dozen in a TEBD sweep, so 32-wide tiles halve the FP64 matrix-core
// work spent on padding (FP64 MFMA runs at the vector rate on this chip).
// 32 x 32 tiles (one 16 x 16 block per wavefront): the largest problems of a
// batch set the duration of the launch, and their K loop over the full
// contraction depth is the critical path, so smaller tiles spread it over
// more compute units.
constexpr int kSketchTileM = 32, kSketchTileN = 32;
// The split-depth variant: 16 x 16 tiles, each computed by the four
// wavefronts of a workgroup over a quarter of the contraction depth, so
// that a tile's chain of matrix-core steps is four times shorter and the
// largest problems spread over four times as many compute units.
constexpr int kSketchTileS = 16;

// Extent of the updated bond index that a TEBD update writes in Gamma^[k]
// (columns) and Gamma^[k+1] (rows): the new dimension chi' <= min(l, chi_max)
// and, cleared to zero, the old one chi_m; beyond both the arrays are
// already zero, so the padding up to the capacity is not rewritten.
__device__ __forceinline__ int updated_bond_extent(const Prob& P) {
  const int kept = P.l < P.kcap ? P.l : P.kcap;
  const int e = kept > P.chi_m ? kept : P.chi_m;
  return e < P.chi_cap ? e : P.chi_cap;
}

constexpr int kTileChunk = 32;

// Whether the Gram of a problem's sketches may be split into row chunks.
__device__ __forceinline__ bool gram_room(const Prob& P) {
  return P.Qc && !(P.chol & (kGramF32M | kGramF32N));
}

// Output shape of each contraction kind for problem P (0 x 0 when skipped).
template <>
struct TileKinds<Prob> {
  static constexpr int count = TK_COUNT;
  static constexpr bool small_tiles(int kind) {
    return kind == TK_SKM || kind == TK_SKN || kind == TK_FORMU || kind == TK_FORMV ||
           kind == TK_THETA || kind == TK_ACB || kind == TK_GRAM;
  }
  static constexpr int tile_m(int kind) {
    return kind == TK_GATE                      ? kGateTileM
           : kind == TK_SKM_S || kind == TK_SKN_S ? kSketchTileS
           : small_tiles(kind)                    ? kSketchTileM
                                                  : 64;
  }
  // TK_SKM_W / TK_SKN_W: the same products on 64 x 64 tiles
  static constexpr int tile_n(int kind) {
    return kind == TK_GATE                        ? kGateTileN
           : kind == TK_SKM_S || kind == TK_SKN_S ? kSketchTileS
           : small_tiles(kind)                    ? kSketchTileN
                                                  : 64;
  }
  // The gate product is short and wide (d_l d_r rows): the row tiles of a
  // column block run one after another, on one XCD, and share its Theta
  // columns in that XCD's L2; the whole gate matrix stays there too.
  static constexpr bool col_major(int kind) { return kind == TK_GATE; }
  // Whether the sketch products split the depth of their tiles between
  // wavefronts (k_sketch): launches of up to 400 32 x 32 tiles, which leave CUs
  // idle or with one tile each, whose chain over the whole depth is the
  // launch's time; and those of a sweep whose largest bond has over 2.5 times
  // the average's tiles, where such chains are its end, up to 1000 tiles.
  // Measured, the six products of a truncation, 32 x 32 / split: 96 x 80, l = 34
  // (9 tiles) 51 / 31 us; 1 x 2048^2, l = 74 (192 tiles) 894 / 549; 4 x 1024^2
  // (384) 622 / 526; 60 x 200^2, l = 30 (420) 159 / 168; 120 x 200^2 (840) 254 /
  // 290; 400 x 100^2 (1600) 257 / 271.  Sweeps of 16 chains whose front moves
  // through, split to 400 / 1000 tiles 45.8 / 41.9 ms (100 sites, 200 steps) and
  // 0.22 / 0.20 (60 sites); to 4000 tiles the first was 37.9, but a step of 16 x
  // 100 sites at chi = 19 went from 0.42 to 0.47.  The factor, 1.25 / 2.5 / 5: the
  // first 40.7 / 41.9 / 47.6 ms, the second 0.15 / 0.20 / 0.23, and 8 chains of 40
  // spins with equal bonds (chi = 33) 0.65 / 0.52 / 0.52.
  static constexpr int rule(int kind) { return kind == TK_SKM ? 0 : kind == TK_SKN ? 1 : -1; }
  static __host__ __device__ bool few(int total, int most, int nprob, int tebd) {
    return total <= 400 || (tebd && total <= 1000 && 2ll * most * nprob > 5ll * total);
  }
  // Tiles of caller matrices go to the XCDs in short runs: the queue starts
  // with the largest matrices, and one XCD must not get all their long tiles
  // (10 sizes from 300 to 2000 twice, l = 74: sketch products 3.65 ms with an
  // eighth of the queue per XCD, 2.52 ms so; runs of 96 2.91 ms; 256 matrices
  // up to 2048 46 and 35 ms).  A run still shares operands in the XCD's L2.
  static __device__ int chunk(int, int tebd) { return tebd ? 0 : kTileChunk; }
  __device__ static __forceinline__ void shape(int kind, const Prob& P, int tebd, int& M, int& N) {
    M = N = 0;
    if (kind == TK_GATE) {
      // the group's tiles belong to its first member, whatever its own state
      if (tebd && P.gn > 0 && P.gtot > 0) {
        M = P.dl * P.dr;
        N = P.gtot;
      }
      return;
    }
    if (P.l == 0) return;
    switch (kind) {
      case TK_THETA:
        if (tebd) {
          M = P.dl * P.chi_l;
          N = P.dr * P.chi_r;
        }
        break;
      case TK_SKM:
      case TK_SKM_W:
      case TK_SKM_S:
        M = P.m;
        N = P.l;
        break;
      case TK_SKN:
      case TK_SKN_W:
      case TK_SKN_S:
        M = P.n;
        N = P.l;
        break;
      case TK_FORMU:  // TEBD: the new bond's columns, and the old ones beyond it (cleared)
        M = P.m;
        N = tebd ? updated_bond_extent(P) : P.kcap;
        break;
      case TK_FORMV:
        M = tebd ? updated_bond_extent(P) : P.kcap;
        N = P.n;
        break;
      case TK_TAPEU:
        if (P.tape_u) {
          M = P.m;
          N = P.l;
        }
        break;
      case TK_TAPEV:
        if (P.tape_u) {
          M = P.l;
          N = P.n;
        }
        break;
      case TK_ACB:
        if (P.ac_r > 0) {
          M = P.m;
          N = P.ac_r;
        }
        break;
      case TK_GRAM:  // the chunks of either sketch side by side (FP32 products: one chunk)
        if (P.chol & (kGramF32M | kGramF32N)) {
          M = N = P.l;
        } else if (const int by = P.chol & 3) {
          M = P.l;
          const int rows = by == 1 ? P.m : by == 2 ? P.n : P.m > P.n ? P.m : P.n;
          N = gram_chunks(rows, P.l1, gram_room(P)) * gram_blocks(P.l) * kGramTile;
        }
        break;
      case TK_GQ_L:  // classes by the width the pass started with: it shrinks as QRs run
        M = N = gram_small(P.m, P.n, P.l1) ? 0 : 1;
        break;
      case TK_GQ_S:
        M = N = gram_small(P.m, P.n, P.l1) ? 1 : 0;
        break;
      case TK_GQ_F:
        M = N = P.chol & kGramFirst ? 1 : 0;
        break;
      case TK_QAPM:  // strips of 64 rows; FP32 products: a 64 x 64 tile here is a 32 x 32 one
        if (P.chol & kGramF32M) {
          M = 2 * P.m;
          N = 2 * P.l;
        } else if (P.chol & kGramTileM) {
          M = P.m;
          N = 1;
        }
        break;
      case TK_QAPN:
        if (P.chol & kGramF32N) {
          M = 2 * P.n;
          N = 2 * P.l;
        } else if (P.chol & kGramTileN) {
          M = P.n;
          N = 1;
        }
        break;
      default:
        break;
    }
  }
  // rows of the two sketches and the width of the pass (the QR size classes)
  __device__ static __forceinline__ bool dims(const Prob& P, int d[3]) {
    d[0] = P.m;
    d[1] = P.n;
    d[2] = P.l1;
    return P.l > 0;
  }
};

// Tiles of an M x N output of one kind.
template <int KIND>
constexpr int64_t tiles_of(int64_t M, int64_t N) {
  constexpr int TM = TileKinds<Prob>::tile_m(KIND), TN = TileKinds<Prob>::tile_n(KIND);
  return ((M + TM - 1) / TM) * ((N + TN - 1) / TN);
}

}  // namespace tebd
