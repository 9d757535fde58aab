// pair_plan.h -- how the two-step pass is laid out on a box: the tile rows and z
// chunks of the z-marching kernel and the tiles of the small-box kernel.  Host
// arithmetic on the box alone, done once per context: searched for at every
// launch it took 11 us of host time at 512 planes and 2 ms at 100000.
#pragma once

#include <stdint.h>

#include "../../include/lbm.h"

namespace lbm {

constexpr int kTB2MinChunk = 2;  // shortest z chunk (planes per block)
// The longest: blocks that march further drift apart and find less of their
// halos in L2 (640^3 FP16 with chunks of 640 planes 76.5k MLUPS, of 128 83k).
constexpr int kTB2MaxChunk = 128;
constexpr int kCUs = 256;

// Tile rows per block, the first the one that large grids take: 13 (16 waves,
// 1024 threads, one block per CU: the FP32 ring takes 127 KB of LDS) for 4- and
// 2-byte storage, which fit 128 VGPRs (forced FP32 along moving walls with two
// spilled); at 512^3 13 rows beat 12, 8, 6 and 5.  FP64 storage takes 5 (118 KB of
// LDS; 6 rows cap the 9 waves at 168 VGPRs, spill and ran 0.7% slower), and F32X
// (FP64 arithmetic) 8, whose 11 waves may use 168 VGPRs.  The others serve the
// sizes that the first leaves a last round nearly empty on (see plan_pairs);
// `cost` is the measured time of a plane against the first's (FP32 6.2 / 4.55 /
// 4.1 us, FP16 4.3 / 3.3 / 2.9, FP64 4.7 / 4.0).
struct Tb2Rows {
  int rows;
  double cost;
};
struct Tb2Table {
  int n;
  Tb2Rows choice[3];
};
constexpr Tb2Table tb2_table(int storage) {
  return storage == LBM_F64    ? Tb2Table{2, {{5, 1.0}, {4, 0.85}, {}}}
         : storage == LBM_F32X ? Tb2Table{1, {{8, 1.0}, {}, {}}}
                               : Tb2Table{3, {{13, 1.0}, {10, 0.74}, {8, 0.67}}};
}

// The z chunk of tiles of `rows` rows; *cost gets the pass's time in planes.  One
// block fills a CU, so the blocks run in rounds of kCUs, and a block's time is its
// planes plus the two it recomputes plus about two planes of start-up -- measured
// 6.1-6.6 us a plane and round in FP32 from 128^3 to 512^3, 4.1-4.3 in BF16 and
// 4.6-4.8 in FP64, whatever the z chunk.  So the chunk length is the one with the
// least rounds * (planes + 4), the longest of several.  (Against chunks of 128
// planes halved down to 16 until there were 1280 blocks: 128^3 FP32 103 -> 85 us a
// pass, 128 x 128 x 256 204 -> 155, 200^3 404 -> 329, 256^3 589 -> 541, 200^3 BF16
// 289 -> 225, 100^3 FP64 130 -> 84; 512^3 keeps its 128 planes.)
inline int z_chunk(int nx, int ny, int nz, int rows, int64_t* cost) {
  const int64_t tiles = int64_t((nx + 63) / 64) * ((ny + rows - 1) / rows);
  int best = nz;
  *cost = INT64_MAX;
  for (int zc = nz < kTB2MaxChunk ? nz : kTB2MaxChunk; zc >= kTB2MinChunk || zc == nz; --zc) {
    const int64_t rounds = (tiles * ((nz + zc - 1) / zc) + kCUs - 1) / kCUs;
    if (rounds * (zc + 4) < *cost) {
      *cost = rounds * (zc + 4);
      best = zc;
    }
  }
  return best;
}

struct TilePlan {
  int32_t tx, ty, tz, ntx, nty, nblocks;
  double cost;
};

// The tile of the small-box kernel: the least rounds of kCUs blocks times the
// waves of a block's two steps, the rows its pulls touch weighing a tenth of a
// wave each (32^3 FP32: 16 x 2 x 4 5.8 us a pass, 8 x 4 x 4 and 32 x 2 x 2 6.2,
// 8 x 4 x 2 6.8).
inline TilePlan plan_tiles(int nx, int ny, int nz) {
  constexpr int dims[][3] = {{8, 4, 2}, {16, 2, 4}, {8, 4, 4}, {8, 8, 4}, {12, 6, 6}};
  TilePlan best{};
  for (const auto& d : dims) {
    TilePlan t{d[0], d[1], d[2], (nx + d[0] - 1) / d[0], (ny + d[1] - 1) / d[1], 0, 0.0};
    t.nblocks = t.ntx * t.nty * ((nz + t.tz - 1) / t.tz);
    const int rows = (t.ty + 2) * (t.tz + 2), e = (t.tx + 2) * rows, o = t.tx * t.ty * t.tz;
    t.cost = ((t.nblocks + kCUs - 1) / kCUs) * ((e + 63) / 64 + (o + 63) / 64 + 0.1 * rows);
    if (!best.nblocks || t.cost < best.cost) best = t;
  }
  return best;
}

struct PairPlan {
  int32_t choice;  // tile rows of the z-marching kernel: index into tb2_table
  int32_t zc[3];   // z chunk with each of them
  bool tiles;      // the pass goes through the small-box kernel, with these tiles
  TilePlan tile;
  bool pays;       // two fused steps are faster than two single ones (the same bits)
};

inline PairPlan plan_pairs(int storage, int nx, int ny, int nz) {
  const Tb2Table table = tb2_table(storage);
  const int64_t cells = int64_t(nx) * ny * nz;
  PairPlan p{};
  // The choice of tile rows: the first unless another one's time, by the same
  // measure, is 6% less, in boxes of more than 2^23 cells 12% (the halo rows of
  // smaller tiles cost memory traffic that the measure leaves out, and the more so
  // the longer the pass runs: 640^3 with 10 rows, 7% less by the measure, FP16 78k
  // MLUPS against 84k with 13).  Measured, us a pass, 13 rows against the chosen:
  // FP32 64^3 18.6 / 15.6 (8 rows), 128^3 92 / 86 (8), 128 x 128 x 256 171 / 157 (8),
  // 160^3 183 / 160 (10); FP64 128^3 170 / 145 (4).
  double march = 0.0, least = 0.0;  // the choice's time, in planes of the first's
  for (int i = 0; i < table.n; ++i) {
    int64_t planes;
    p.zc[i] = z_chunk(nx, ny, nz, table.choice[i].rows, &planes);
    const double c = double(planes) * table.choice[i].cost;
    if (i == 0) least = (cells > (1 << 23) ? 0.88 : 0.94) * (march = c);
    else if (c < least) {
      least = march = c;
      p.choice = i;
    }
  }
  // The small-box kernel up to 2^17 cells (64^3 7.7 us a step against 7.1, FP64 10.8
  // against 10.8) unless the box is so flat that the other one's 64-wide tiles and
  // single plane cost less: their measures are compared, a unit of the tiles' being
  // worth a twelfth of a plane (F32X, with its 8 rows, an eighth, FP64 a seventh).
  // us a step, small-box / z-marching, FP32 48^3 4.9 / 6.3, 27 x 43 x 68 6.0 / 6.9, 1
  // x 206 x 82 3.8 / 4.6, 1 x 179 x 310 6.9 / 4.8, 1 x 341 x 299 11.2 / 5.2; F32X 1 x
  // 179 x 310 7.9 / 4.8; FP64 48^3 5.8 / 6.8, 24 x 76 x 64 porous 10.1 / 8.4, 1 x 341 x
  // 299 13.0 / 8.0.  (110 boxes x 5 storages: 0.4% behind the better one on average.)
  const double unit = storage == LBM_F64 ? 7.0 : storage == LBM_F32X ? 8.0 : 12.0;
  p.tile = plan_tiles(nx, ny, nz);
  p.tiles = cells <= (int64_t(1) << 17) && p.tile.cost < unit * march;
  // Single steps / pairs, us a step.  In the small-box kernel pairs win where one
  // round of blocks with tiles of at most 128 cells covers the box: FP32 24^3 3.4 /
  // 2.5, 32^3 3.6 / 3.2 (porous 4.2 / 3.9), FP16 32^3 3.2 / 2.5, FP64 5.3 / 3.5;
  // past that only some do (29 x 26 x 46 porous FP32 4.4 / 5.2, box F32X 3.6 / 3.8,
  // FP64 5.2 / 4.2), among them all rows of up to 8 cells, of which a wave of the
  // single step runs a lane each (3347 x 4 x 8 FP32 13.3 / 6.7, 4396 x 24 x 1 FP16 96
  // / 69).
  if (p.tiles) {
    p.pays = nx <= 8 || (p.tile.nblocks <= kCUs && p.tile.tx * p.tile.ty * p.tile.tz <= 128);
    return p;
  }
  // In the z-marching kernel a pass that is short of blocks leaves CUs idle, and one
  // of few planes per block fills the ring more than it uses it.  Both are in the
  // plan's measure, so pairs run from as many cells per plane of the pass's time as
  // single steps are worth.  Measured, us a step, single / pairs:
  //   FP32 62000: 64^3 (66k) 7.5 / 7.5, porous 8.7 / 8.1, 89 x 91 x 95 (88k) 20.6 /
  //     17.5, but 57 x 55 x 86 (52k) 9.2 / 9.8, 1 x 543 x 950 (38k) 13.3 / 18.6, 2020 x
  //     16 x 16 (39k) 23.5 / 31.4.
  //   FP64 24000: 4 x 175 x 328 (29k) 13.0 / 11.3, 4 x 121 x 477 (34k) 12.5 / 11.0, but
  //     1 x 804 x 336 (14k) 13.8 / 17.2; between solids pairs gain less, 8 x 250 x 135
  //     (26k) porous 15.1 / 17.8; in boxes above the memory-side cache 15000: 2 x 697 x
  //     717 (24k) 61.9 / 43.7, 1 x 1226 x 3328 (16k) 245.1 / 232.3.
  //   16 bits 62000: 3 x 204 x 603 (71k) 7.7 / 7.9, along a moving lid 17.4 / 12.2, 8 x
  //     288 x 239 (93k) 10.5 / 9.3, but 2 x 397 x 529 (52k) porous 11.0 / 12.1, 1 x 445
  //     x 1536 (37k) 11.0 / 18.0; above 2^20 cells 78000, as the halos of flat tiles
  //     then cost more: 3 x 381 x 1728 (76k) lid 37.0 / 52.3, 6 x 527 x 411 (97k) 19.1
  //     / 16.0.
  // F32X pays from 2^20 cells and 128 blocks: porous 96^3 24.5 / 25.7, 112^3 37 / 33.
  const int rows = table.choice[0].rows;
  const int64_t blocks = int64_t((nx + 63) / 64) * ((ny + rows - 1) / rows) * ((nz + p.zc[0] - 1) / p.zc[0]);
  const double each = double(cells) / march;
  p.pays = storage == LBM_F64    ? each >= (cells * 304 > (int64_t(256) << 20) ? 15000.0 : 24000.0)
           : storage == LBM_F32X ? cells >= (1 << 20) && blocks >= 128
           : storage == LBM_F32  ? cells >= (1 << 18) && blocks >= 128 && each >= 62000.0
                                 : each >= (cells > (1 << 20) ? 78000.0 : 62000.0);
  return p;
}

}  // namespace lbm
