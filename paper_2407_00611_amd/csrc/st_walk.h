// The walk of a query-stationary workgroup (256 rows of one head) over the 64-key tiles its rows see, as the hand-scheduled
// forward and dQ loops take it: a table in LDS, whole tiles first, masked ones last.
#pragma once

#include "st_internal.h"
#include "st_mfma.h"

namespace st {
namespace {

typedef __attribute__((__vector_size__(16 * sizeof(uint32_t)))) uint32_t u32x16;

// XOR swizzle of the LDS tiles (the f of swz<D> in st_mfma.h)
template <int D>
__device__ __forceinline__ int swz_f(int row) {
  return D == 128 ? (((row & 3) << 2) | ((row >> 2) & 3)) : ((((row >> 1) & 1) << 2) | ((row >> 2) & 3));
}

// every value passed through sgpr() is uniform over the wavefront by construction (kernel arguments, block index)
__device__ __forceinline__ uint32_t sgpr(uint32_t x) { return __builtin_amdgcn_readfirstlane(x); }
__device__ __forceinline__ uint32_t lo32(const void* p) { return (uint32_t)(uintptr_t)p; }
__device__ __forceinline__ uint32_t hi32(const void* p) { return (uint32_t)((uintptr_t)p >> 32); }
// sum over the lanes before this one; total = sum over all 64 (all of them active).  Data parallel primitives: a scan by
// shuffles waits for LDS six times, which is time no other wavefront of the workgroup has work for.
__device__ __forceinline__ int lane_scan(int x, int& total) {
  int sum = x;
  sum += __builtin_amdgcn_update_dpp(0, sum, 0x111, 0xf, 0xf, false);      // row_shr:1, inside the rows of 16
  sum += __builtin_amdgcn_update_dpp(0, sum, 0x112, 0xf, 0xf, false);
  sum += __builtin_amdgcn_update_dpp(0, sum, 0x114, 0xf, 0xf, false);
  sum += __builtin_amdgcn_update_dpp(0, sum, 0x118, 0xf, 0xf, false);
  sum += __builtin_amdgcn_update_dpp(0, sum, 0x142, 0xa, 0xf, false);      // row_bcast:15 into rows 1 and 3
  sum += __builtin_amdgcn_update_dpp(0, sum, 0x143, 0xc, 0xf, false);      // row_bcast:31 into rows 2 and 3
  total = __builtin_amdgcn_readlane(sum, 63);
  return sum - x;
}

// The shares of the key tiles of a head (see BwdArgs::kv_each).  `offsets`: a function that gives the position of chunk c.
struct KvPlace {
  int tile, share, n_share, slot;                    // slot: of the tile's share 1, within the head
};
// of share `w`, or (by_tile) the first one of tile w
template <typename F>
__device__ __forceinline__ KvPlace kv_place(const Shape& s, const KvSection (&sec)[kKvSections], int each, int n_kt, int w, bool by_tile, int lane, F offsets) {
  // the section that w is in, and the tiles and shares before it; picked by selects: an index that is only known at run time would
  // put the sections into scratch memory, a chain of stores and loads at the start of every workgroup
  int t0 = 0, i0 = 0, tiles = sec[0].tiles, items = sec[0].items, mixed = sec[0].mixed;
  int t1 = tiles, i1 = items;
#pragma unroll
  for (int x = 1; x < kKvSections; ++x) {
    const bool beyond = w >= (by_tile ? t1 : i1);
    t0 = beyond ? t1 : t0;
    i0 = beyond ? i1 : i0;
    tiles = beyond ? sec[x].tiles : tiles;
    items = beyond ? sec[x].items : items;
    mixed = beyond ? sec[x].mixed : mixed;
    t1 += sec[x].tiles;
    i1 += sec[x].items;
  }
  KvPlace p;
  if (!mixed) {
    p.n_share = items / max(tiles, 1);
    const int k = by_tile ? w - t0 : (w - i0) / p.n_share;
    p.tile = t0 + k;
    p.share = by_tile ? 0 : w - i0 - k * p.n_share;
    p.slot = i0 - t0 + k * (p.n_share - 1);
    return p;
  }
  p.tile = t0;
  p.share = p.slot = 0;
  p.n_share = 1;
  for (int at = t0; at < t0 + tiles; at += 64) {     // a lane per tile
    const int t = at + lane, n = t < t0 + tiles ? kv_shares(kv_blocks(s, offsets(min(t, t0 + tiles - 1) / n_kt), t % n_kt), each) : 0;
    int total;
    const int first = i0 + lane_scan(n, total);
    const uint64_t here = __ballot(by_tile ? t == w : w >= first && w < first + n);
    if (here) {
      const int l = (int)__builtin_ctzll(here), f = __builtin_amdgcn_readlane(first, l);
      p.tile = at + l;
      p.share = by_tile ? 0 : w - f;
      p.n_share = __builtin_amdgcn_readlane(n, l);
      p.slot = f - p.tile;
      break;
    }
    i0 += total;
  }
  return p;
}

// Block of a query-stationary launch -> query tile, head-and-batch index and share (see TileShares).  Where the tiles have
// numbers of their own, the shares of a head are numbered from its last tile down and handed out in that order, all heads'
// first ones first (qtile_block): the longest ones are the last tiles'.
__device__ __forceinline__ void share_block(const TileShares& t, int block_x, int grid_x, int block_y, int n_qt, int causal, int& qt, int& hb, int& split) {
  if (t.total <= 0) {
    qtile_block(block_x, grid_x, n_qt, causal, qt, hb);
    split = block_y;
    return;
  }
  qtile_block(block_x, grid_x, t.total, 0, split, hb);
  split = (int)sgpr(split);
  for (qt = n_qt - 1; qt > 0; --qt) {
    const int n = shares_of(t, qt);
    if (split < n) break;
    split -= n;
  }
}

constexpr int kRelMin = -(1 << 30);                  // relative position of a tile that no causal mask touches

// Position of row i relative to the workgroup's first row, as the mask routines compare it with a tile's: the sum of the two
// has to stay inside 32 bits.  Under a causal mask it does, as no tile has rows of two runs.  Without one the routines still run, for the
// ragged end of a chunk, and two runs of rows may lie any distance apart, so there a row has no position: all of them see
// every key of a tile at kRelMin.
__device__ __forceinline__ int walk_row_pos(const Shape& s, int i, int row0) {
  return s.causal ? (int)(q_pos(s, i) - q_pos(s, row0)) : 0;
}

// The tiles a workgroup walks, written to LDS by one wavefront, a lane per chunk of the table, while the others wait: a chain
// of latencies at the start of every workgroup (2.8 us of a 25 us launch with shuffles, 64-bit divisions and loads behind
// the table's length; 2.1 us so).  Entry (32 bytes): K and V
// addresses, tiles, position of the first key relative to q_base, first key of the (single) tile that counts, pad.
// Whole tiles of all chunks come first, then the masked ones.  In that order split y of n takes an equal share of the work,
// a masked tile counted as two whole ones: all of them are in the last splits, where they cost 0.5 to 1 us more each than a
// whole tile's 1.4 (in the mask routine and in the second copy of the loop, which is fetched for them).  Shares of equal
// tiles made the launch wait for the last split: 12 heads x 2 x 1000 rows in 3 splits 82 us, so 78.7 (dQ 105 and 102.5); 16 x
// 2 x 512 rows at head size 64 30.7 and 29.0 (31.8 and 30.5); three units for a masked tile are as far off on the other side
// (82.4, 107.5).  Returns the tiles of the split; n_masked of them, the last ones, are masked; their entries start at
// first_masked.
__device__ __forceinline__ int build_walk(const Shape& s, const ChunkTable& t, int splits, int row0, int row_end, int b, int hk, int split, ST_LDS uint32_t* tbl, int lane,
                                          int& n_masked, int& first_masked) {
  constexpr int BN = kQTileFastKeys;
  const int n64 = s.Sk / BN;
  static_assert(kMaxTable == 64, "a lane per chunk");
  // the whole table is read, so that the loads need not wait for its length (arguments come from host memory)
  const int64_t k0 = t.k_offset[lane];
  const char* kp = (const char*)t.k[lane] + ((int64_t)b * t.ksb + (int64_t)hk * t.ksh) * 2;
  const char* vp = (const char*)t.v[lane] + ((int64_t)b * t.vsb + (int64_t)hk * t.vsh) * 2;
  const int64_t q_base = q_pos(s, row0), q_last = q_pos(s, row_end - 1), rel0 = k0 - q_base;
  const int64_t nv = s.causal ? min(max(q_base - k0 + 1, (int64_t)0), (int64_t)s.Sk) : s.Sk;       // keys the first row sees
  const int64_t nv_last = s.causal ? min(max(q_last - k0 + 1, (int64_t)0), (int64_t)s.Sk) : s.Sk;  // and the last one
  const bool listed = lane < t.n;
  const int nf = listed ? (int)nv / BN : 0;                                                        // whole tiles
  const int nm = listed ? max(min(((int)nv_last + BN - 1) / BN, n64) - nf, 0) : 0;                 // masked tiles
  const int nr = listed && nv_last > (int64_t)n64 * BN;                                            // ragged end (0 or 1)
  int total_full, total_masked;
  const int pf = lane_scan(nf, total_full);
  const int pm = total_full + lane_scan(nm + nr, total_masked);
  int lo = 0, hi = total_full + total_masked;
  if (splits > 1) {
    const uint32_t units = (uint32_t)total_full + 2 * (uint32_t)total_masked, each = units / splits, rest = units % splits;
    auto edge = [&](uint32_t y) {                    // tiles before unit [units y / splits]
      const uint32_t u = each * y + rest * y / (uint32_t)splits;
      return (int)(u <= (uint32_t)total_full ? u : total_full + (u - total_full) / 2);
    };
    lo = edge(split), hi = edge(split + 1);
  }
  const int f0 = max(pf, lo), cf = max(min(pf + nf, hi) - f0, 0);
  const int m0 = max(pm, lo), cm = max(min(pm + nm, hi) - m0, 0);
  const int cr = nr && pm + nm >= lo && pm + nm < hi;
  const uint64_t before = ((uint64_t)1 << lane) - 1, has_f = __ballot(cf > 0), has_m = __ballot(cm > 0), has_r = __ballot(cr);
  auto put = [&](int entry, int key0, int tiles, int lo_key) {
    const char* k = kp + (int64_t)key0 * t.kss * 2;
    const char* v = vp + (int64_t)key0 * t.vss * 2;
    const int64_t rel = s.causal ? min(max(rel0 + key0, (int64_t)kRelMin), (int64_t)-kRelMin) : (int64_t)kRelMin;
    ST_LDS uint32_t* e = tbl + 8 * entry;
    e[0] = lo32(k); e[1] = hi32(k); e[2] = lo32(v); e[3] = hi32(v);
    e[4] = (uint32_t)tiles; e[5] = (uint32_t)(int32_t)rel; e[6] = (uint32_t)lo_key;
  };
  first_masked = __popcll(has_f);
  if (cf > 0) put(__popcll(has_f & before), (f0 - pf) * BN, cf, 0);
  const int em = first_masked + __popcll(has_m & before) + __popcll(has_r & before);
  if (cm > 0) put(em, (nf + m0 - pm) * BN, cm, 0);
  if (cr) put(em + (cm > 0), s.Sk - BN, 1, n64 * BN - (s.Sk - BN));   // the chunk's last 64 rows, those of the tile before masked
  n_masked = hi - max(lo, min(total_full, hi));
  return hi - lo;
}

// grid of a launch whose `total` query tiles, n_qt of each head, have these shares
inline dim3 share_grid(const TileShares& t, int64_t total, int n_qt) {
  if (t.total > 0) return dim3((unsigned)(total / n_qt * t.total));
  return dim3((unsigned)total, (unsigned)(t.n > 1 ? t.n : 1));
}

// what the loops keep in 32-bit registers fits them
inline bool walk_usable(const Shape& s, const ChunkTable& t) {
  if ((s.D != 128 && s.D != 64) || s.Sk < kQTileFastKeys || s.Sq < 1) return false;
  auto fits = [](int64_t x) { return x > 0 && x < (int64_t)1 << 30; };
  if (!(fits(kQTileFastKeys * t.kss * 2) && fits(kQTileFastKeys * t.vss * 2) && fits((int64_t)kQTileFastRows * s.Hq * s.D * 4)))
    return false;
  return true;
}

}  // namespace
}  // namespace st
