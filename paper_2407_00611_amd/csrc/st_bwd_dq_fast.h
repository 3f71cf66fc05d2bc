// The workgroup of the hand-scheduled bf16 dQ kernel, for the launches that hold it: dQ alone (st_bwd_dq_fast.hip) and
// dQ beside dK/dV (st_bwd_dkv_fast.hip).
#pragma once

#include "st_internal.h"
#include "st_mfma.h"
#include "st_walk.h"
#include "st_bwd_dq_asm.inc"
#include "st_bwd_dq64_asm.inc"

namespace st {
namespace {

typedef __attribute__((__vector_size__(4 * sizeof(uint32_t)))) uint32_t u32x4v;

constexpr float kLog2e = 1.4426950408889634f;

template <int D>
constexpr int dq_lds_bytes() { return D == 128 ? ST_DQ_FAST_LDS_BYTES : ST_DQ_FAST64_LDS_BYTES; }

// One workgroup: a share of a query tile's walk (share_block).
template <int D>
__device__ __forceinline__ void dq_fast_body(const BwdArgs& a, int block_x, int grid_x, int block_y, char* smem_raw) {
  constexpr int BM = kDqFastRows, BN = kDqFastKeys;
  constexpr int kLdsBytes = dq_lds_bytes<D>();
  constexpr int kQrel = kLdsBytes - 256 * 8;         // behind the tile ring: table, parameter block, row positions
  constexpr int kParams = kQrel - 64;
  constexpr int kTblOffset = kParams - 3 * 32 * kMaxTable;
  constexpr int ROW = 2 * D;                         // bytes of a K / V row in LDS
  constexpr int CPR = D / 8;                         // 16-byte chunks per row
  constexpr int RPI = 64 / CPR;                      // rows one direct-to-LDS load of a wavefront fills
  ST_LDS char* smem = (ST_LDS char*)smem_raw;
  const uint32_t lds_base = (uint32_t)(uintptr_t)smem;

  const Shape& s = a.s;
  const int tid = threadIdx.x, lane = tid & 63, wave = (int)sgpr(tid >> 6);
  const int g = lane >> 5, r = lane & 31;
  const QueryTiles tiles = query_tiles(s, BM);
  int qt, hb, split;
  share_block(a.shares, block_x, grid_x, block_y, tiles.count(), s.causal, qt, hb, split);
  const int n_split = max(shares_of(a.shares, qt), 1);
  // divisions run on the vector unit; their results are uniform, and so are the addresses made of them
  const int h = (int)sgpr(hb % s.Hq), b = (int)sgpr(hb / s.Hq), hk = (int)sgpr(h / (s.Hq / s.Hkv));
  const int row0 = (int)sgpr(tiles.row0(qt)), rows = (int)sgpr(tiles.rows_of(qt)), row_end = row0 + rows;

  const int q_row = row0 + 64 * wave + r;            // this lane's row of query block 0; block 1: + 32
  const int i0 = min(q_row, row_end - 1), i1 = min(q_row + 32, row_end - 1);
  ST_LDS uint32_t* params = (ST_LDS uint32_t*)(smem + kParams);
  {  // for the mask
    ST_LDS int32_t* qrel = (ST_LDS int32_t*)(smem + kQrel) + 2 * tid;
    qrel[0] = walk_row_pos(s, i0, row0) - 4 * g;
    qrel[1] = walk_row_pos(s, i1, row0) - 4 * g;
  }
  const bool part = n_split > 1 && split >= a.shares.own0;      // a sum of its own, not dq itself
  if (wave == 0) {
    int n_masked, first_masked;
    const int n = build_walk(s, a.t, n_split, row0, row_end, b, hk, split, (ST_LDS uint32_t*)(smem + kTblOffset), lane, n_masked, first_masked);
    if (lane == 0) {
      params[0] = (uint32_t)n_masked;
      params[1] = lds_base + kTblOffset + 32 * first_masked;
      params[2] = part ? 1 : 0;
      params[3] = (uint32_t)n;
    }
  }
  __syncthreads();
  const int total_tiles = (int)params[3];
  float* dq0 = (part ? dq_part(a.parts, s, tiles, a.shares, b, qt, split - a.shares.own0) : a.dq + ((int64_t)b * s.Sq + row0) * s.Hq * D) + h * D;
  if (total_tiles <= 0) {                            // uniform over the workgroup
    if (part)
      for (int p = tid; p < rows * (D / 4); p += 256)
        *reinterpret_cast<float4*>(dq0 + (int64_t)(p / (D / 4)) * s.Hq * D + p % (D / 4) * 4) = make_float4(0.f, 0.f, 0.f, 0.f);
    return;
  }

  const char* qbase = (const char*)a.q.ptr + ((int64_t)b * a.q.sb + (int64_t)h * a.q.sh) * 2;
  const char* dobase = (const char*)a.d_o.ptr + ((int64_t)b * a.d_o.sb + (int64_t)h * a.d_o.sh) * 2;
  const int64_t stat0 = ((int64_t)b * s.Hq + h) * s.Sq;

  uint32_t ss[11];   // scalar operands, pinned one by one (s32..s43)
  ss[0] = sgpr(lds_base);
  ss[1] = (uint32_t)__builtin_amdgcn_readfirstlane(wave);
  ss[2] = sgpr((uint32_t)total_tiles);
  ss[3] = sgpr((uint32_t)(4 * RPI * a.t.kss * 2));   // bytes between the rows of two consecutive loads of a wavefront
  ss[4] = sgpr((uint32_t)(4 * RPI * a.t.vss * 2));
  ss[5] = sgpr(__builtin_bit_cast(uint32_t, s.scale));
  ss[6] = sgpr(lo32(dq0));
  ss[7] = sgpr(hi32(dq0));
  ss[8] = sgpr((uint32_t)(32 * s.Hq * D * 4));       // bytes between the two 32-query blocks of a wavefront
  ss[9] = sgpr(lds_base + kTblOffset);
  ss[10] = sgpr((uint32_t)(BN * a.t.kss * 2));       // bytes per 64-key tile
  const uint32_t vtile = sgpr((uint32_t)(BN * a.t.vss * 2));

  u32x16 va;
  u32x4v vb;
  // Q / dO rows of this lane (B-operand fragments): elements 8 g .. + 7 of each 16; rows beyond the shard re-read its last one
  const char* qrow0 = qbase + (int64_t)i0 * a.q.ss * 2 + 16 * g;
  const char* qrow1 = qbase + (int64_t)i1 * a.q.ss * 2 + 16 * g;
  const char* dorow0 = dobase + (int64_t)i0 * a.d_o.ss * 2 + 16 * g;
  const char* dorow1 = dobase + (int64_t)i1 * a.d_o.ss * 2 + 16 * g;
  va[0] = lo32(qrow0);  va[1] = hi32(qrow0);  va[2] = lo32(qrow1);  va[3] = hi32(qrow1);
  va[4] = lo32(dorow0); va[5] = hi32(dorow0); va[6] = lo32(dorow1); va[7] = hi32(dorow1);
  // per-row statistics: exponent offset -lse * log2(e) (-inf for an empty row, whose P must be 0) and -Delta
  for (int qb = 0; qb < 2; ++qb) {
    const int64_t st = stat0 + (qb ? i1 : i0);
    const float l = a.lse[st];
    const float nl = l == -INFINITY ? -INFINITY : -l * kLog2e;
    va[8 + qb] = __builtin_bit_cast(uint32_t, nl);
    va[10 + qb] = __builtin_bit_cast(uint32_t, -a.delta[st]);
  }
  va[12] = lds_base + r * ROW;                                       // natural operand reads
  va[13] = (uint32_t)((g ^ swz_f<D>(r)) << 4);
  {                                                                  // transpose reads
    const int s16 = lane & 15, half = (lane >> 4) & 1;
    const int rowlo = 4 * g + (s16 >> 2), lc = 2 * half + ((s16 & 3) >> 1), sub = (s16 & 1) * 8;
    va[14] = lds_base + rowlo * ROW + sub;
    va[15] = (uint32_t)((lc ^ swz_f<D>(rowlo)) << 4);
  }
  // tile staging: instruction 4 j + wave fills rows RPI (4 j + wave) + lane / CPR, chunk position lane % CPR,
  // with source chunk (lane % CPR) ^ f(row)   (the XOR swizzle is applied on the global side)
  const int srow = RPI * wave + lane / CPR, spc = (lane % CPR) ^ swz_f<D>(srow);
  vb[0] = (uint32_t)(srow * a.t.kss * 2 + spc * 16);
  vb[1] = (uint32_t)(srow * a.t.vss * 2 + spc * 16);
  vb[2] = (uint32_t)((64 * wave + r) * s.Hq * D * 4 + g * 16);       // dQ row of this lane
  vb[3] = (q_row < row_end ? 1u : 0u) | (q_row + 32 < row_end ? 2u : 0u);

  if constexpr (D == 128) {
    asm volatile(ST_DQ_FAST_ASM
                 : "+{v[160:175]}"(va), "+{v[176:179]}"(vb)
                 : "{s32}"(ss[0]), "{s33}"(ss[1]), "{s34}"(ss[2]), "{s35}"(ss[3]), "{s36}"(ss[4]), "{s37}"(ss[5]),
                   "{s38}"(ss[6]), "{s39}"(ss[7]), "{s40}"(ss[8]), "{s41}"(ss[9]), "{s42}"(ss[10]), "{s43}"(vtile)
                 : ST_DQ_FAST_CLOBBERS);
  } else {
    asm volatile(ST_DQ_FAST64_ASM
                 : "+{v[160:175]}"(va), "+{v[176:179]}"(vb)
                 : "{s32}"(ss[0]), "{s33}"(ss[1]), "{s34}"(ss[2]), "{s35}"(ss[3]), "{s36}"(ss[4]), "{s37}"(ss[5]),
                   "{s38}"(ss[6]), "{s39}"(ss[7]), "{s40}"(ss[8]), "{s41}"(ss[9]), "{s42}"(ss[10]), "{s43}"(vtile)
                 : ST_DQ_FAST64_CLOBBERS);
  }
}

}  // namespace
}  // namespace st
