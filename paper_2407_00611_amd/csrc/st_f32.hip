// fp32 kernels: any D <= 256 (multiple of 8), any Sq / Sk, on the fp32 matrix instruction v_mfma_f32_32x32x2_f32
// (exact fp32 products and sums, 256 flop per clock and compute unit: twice what v_fma_f32 issues, and 64 cycles per
// instruction, under which operand loads and the softmax arithmetic hide).  Deterministic, no atomics: every
// accumulator element has one owning workgroup, whose wavefronts add up in a fixed order.
//
//   forward, dQ   a workgroup owns 32 query rows of one head; its wavefronts take the 32-key tiles of the walk in
//                 turn (a 512-row shard of 8 heads has only 128 such workgroups, so the keys have to be split inside
//                 one) and fold their states through LDS at the end.  Q and dO rows sit in LDS, shared by all.
//                     S^T = K Q^T, dP^T = V dO^T         lane = query column, registers = 16 keys
//                     O^T += V^T P^T, dQ^T += K^T dS^T   the S^T registers are the B operand as they stand
//   dK / dV       a workgroup owns 32 keys; its wavefronts take the (query head of the group, 32-row tile) pairs.
//                     S = Q K^T, dP = dO V^T             lane = key column, registers = 16 query rows
//                     dV^T += dO^T P, dK^T += Q^T dS
//
// Operand layouts (lane l: r = l % 32, g = l / 32): A holds row r at k = g, B holds column r at k = g, C holds column
// r at rows 8 (v / 4) + 4 g + v % 4, v = 0..15.  The k order is free as long as A and B agree, which gives
//   * contractions along D: one 16-byte load of elements 8 j + 4 g .. + 3 of row r feeds four instructions,
//   * contractions along a tile's rows: step v takes register v of a C tile as B and row 8 (v / 4) + 4 g + v % 4 as A.
//
// One wavefront per row with scalar fused multiply-adds, as these kernels were before, read K with every lane on a
// row of its own and one load per four multiply-adds: 8 heads x 512 rows x 8 chunks of 512 keys at D = 128 took 2460 us
// forward, 2640 us dQ, 3590 us dK / dV (3.2 TFLOP/s).  Now 102 us forward with the split launch (on one workgroup per query
// tile, 128 for 256 compute units: 181) and 312 to 322 us both backward passes in one launch (206 and 152 us, and a gap, in two).
// Long walks run at 100 TFLOP/s of the 154 of a large fp32 matrix product on this card.  Bursts of 60 to 130 us of nothing but
// this instruction on random data run at 129 to 136; of the forward's 103 us the loads cost 17 (without any 85), the exponential
// 4, masks, addresses and rescaling nothing that shows.  A tile's columns in one load a row in place of DB took 2 to 3 % off both.
#include <algorithm>
#include <type_traits>

#include "st_internal.h"
#include "st_mfma.h"
#include "st_walk.h"

namespace st {
namespace {

constexpr int kT = 32;             // rows of every tile

__device__ __forceinline__ f32x16 mfma_f32(float a, float b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
}

// wavefronts per workgroup: eight (two per SIMD, which hide each other's loads) as long as a wavefront's accumulators
// and operands fit 256 registers
template <int DP>
constexpr int waves() { return DP <= 128 ? 8 : 4; }

// number of leading keys of a chunk that query position qpos may see
__device__ __forceinline__ int visible_keys(const Shape& s, int64_t qpos, int64_t k0) {
  if (!s.causal) return s.Sk;
  int64_t n = qpos - k0 + 1;
  return n < 0 ? 0 : (n > s.Sk ? s.Sk : (int)n);
}

// row of a tile that register v of a C tile holds in half g
__device__ __forceinline__ int c_row(int v, int g) { return 8 * (v / 4) + 4 * g + v % 4; }

// ---- streamed operands, in pieces of N (32 or 16) registers.  While one piece is contracted (N instructions of 64
// cycles) the next one is on its way; two pieces and the accumulators are what fits beside a second wavefront.
// FULL: D == DP.  Otherwise the columns at or beyond D read as zero.
template <int N>
struct Piece {
  float x[N];
};
template <int DP, int N>
constexpr int row_pieces() { return (DP + 2 * N - 1) / (2 * N); }           // 2 N columns each
template <int DP, int N>
constexpr int piece_rows() {                                                // registers v of a C tile per column piece
  int n = 16;
  while (n * (DP / 32) > N) n /= 2;
  return n;
}
template <int DP, int N>
constexpr int col_pieces() { return 16 / piece_rows<DP, N>(); }

// Row r of a tile as the k-along-D operand: columns 2 N n + 8 j + 4 g .. + 3
template <int DP, bool FULL, int N>
__device__ __forceinline__ void load_rows(Piece<N>& f, const float* row, int n, int D, int g) {
#pragma unroll
  for (int j = 0; j < N / 4; ++j) {
    const int d = 2 * N * n + 8 * j;
    if (d >= DP) continue;
    float4 x = make_float4(0.f, 0.f, 0.f, 0.f);
    if (FULL || d < D) x = *reinterpret_cast<const float4*>(row + d + 4 * g);
    f.x[4 * j] = x.x; f.x[4 * j + 1] = x.y; f.x[4 * j + 2] = x.z; f.x[4 * j + 3] = x.w;
  }
}

// a pointer said to be global, where the compiler does not see it (it would load with flat loads, which wait for LDS too)
typedef const __attribute__((address_space(1))) float* GlobalFloats;
__device__ const __attribute__((aligned(16))) float zero_row[256] = {};
typedef float f32x2v __attribute__((ext_vector_type(2)));
typedef float f32x4v __attribute__((ext_vector_type(4)));
// The column that row m of accumulator db stands for, which is free as long as the results are stored so (acc_block).  A lane's
// columns are neighbours, one load of up to four floats a row, where their number is even.  Three would be three loads again, at
// strides of three floats: head size 96 has them 32 apart, a row's loads of a wavefront in one piece.
template <int DB>
__device__ __forceinline__ constexpr int column(int m, int db) { return DB % 2 == 0 ? DB * m + db : 32 * db + m; }
// The transposed operand of a tile X: lane r = columns column(r, 0 .. DB - 1), register v = row c_row(v, g).
// Rows at or beyond `limit` (tile-relative, >= 1) are zero: their weight is, but a row that exists, read in their place, may
// hold an infinity, and 0 * inf is NaN.
template <int DP, bool FULL, int N>
__device__ __forceinline__ void load_cols(Piece<N>& f, const float* tile, int64_t stride, int limit, int n, int D, int r, int g) {
  constexpr int DB = DP / 32;
  int mine = limit - 4 * g;
  asm volatile("" : "+v"(mine));                     // compared anew for every piece: kept, the masks of all rows spill
#pragma unroll
  for (int u = 0; u < piece_rows<DP, N>(); ++u) {
    const int v = n * piece_rows<DP, N>() + u, row = 8 * (v / 4) + v % 4;
    GlobalFloats p = (GlobalFloats)tile + (int64_t)(4 * g) * stride + (int64_t)row * stride;
    if (limit < kT) p = row < mine ? p : (GlobalFloats)zero_row;
    p += column<DB>(r, 0);
    float* x = f.x + DB * u;
    if constexpr (DB % 2 == 0) {
      constexpr int W = DB % 4 == 0 ? 4 : 2;
      typedef typename std::conditional<W == 4, f32x4v, f32x2v>::type Vec;
#pragma unroll
      for (int q = 0; q < DB; q += W) {
        Vec y = {};
        if (FULL || DB * r + q < D) y = *reinterpret_cast<const __attribute__((address_space(1))) Vec*>(p + q);   // D is a multiple of 8
#pragma unroll
        for (int e = 0; e < W; ++e) x[q + e] = y[e];
      }
    } else {
#pragma unroll
      for (int db = 0; db < DB; ++db) x[db] = FULL || column<DB>(r, db) < D ? p[32 * db] : 0.f;
    }
  }
}

// ---- resident tile in LDS: kT rows of D floats, rows padded by 4 floats so that 16-byte reads of one column by
// consecutive rows spread over the banks; rows at or beyond `limit` and columns at or beyond D are zero
template <int DP>
constexpr int lds_stride() { return DP + 4; }
template <int DP>
__device__ __forceinline__ void stage_tile(float* lds, const float* base, int64_t stride, int row0, int limit, int D, int tid) {
  for (int p = tid; p < kT * (DP / 4); p += waves<DP>() * 64) {
    const int row = p / (DP / 4), d = p % (DP / 4) * 4;
    float4 x = make_float4(0.f, 0.f, 0.f, 0.f);
    if (row0 + row < limit && d < D) x = *reinterpret_cast<const float4*>(base + (int64_t)(row0 + row) * stride + d);
    *reinterpret_cast<float4*>(lds + row * lds_stride<DP>() + d) = x;
  }
}

// C tile (rows: the streamed tile's, columns: the LDS tile's rows) += contraction along its row piece n
template <int DP, int N>
__device__ __forceinline__ void contract_d(f32x16& c, const Piece<N>& f, const float* lds, int n, int r, int g) {
#pragma unroll
  for (int j = 0; j < N / 4; ++j) {
    const int d = 2 * N * n + 8 * j;
    if (d >= DP) continue;
    const float4 y = *reinterpret_cast<const float4*>(lds + r * lds_stride<DP>() + d + 4 * g);
    c = mfma_f32(f.x[4 * j], y.x, c);
    c = mfma_f32(f.x[4 * j + 1], y.y, c);
    c = mfma_f32(f.x[4 * j + 2], y.z, c);
    c = mfma_f32(f.x[4 * j + 3], y.w, c);
  }
}

// acc^T[d][column] += sum over the rows of column piece n of X[row][d] w[row][column]
template <int DP, int N>
__device__ __forceinline__ void contract_rows(f32x16 (&acc)[DP / 32], const Piece<N>& f, const f32x16& w, int n) {
  constexpr int DB = DP / 32;
#pragma unroll
  for (int u = 0; u < piece_rows<DP, N>(); ++u)
#pragma unroll
    for (int db = 0; db < DB; ++db) acc[db] = mfma_f32(f.x[DB * u + db], w[n * piece_rows<DP, N>() + u], acc[db]);
}

// ---- infinities and NaN in a tile that a mask edge crosses.  The matrix instruction multiplies a row that a column
// does not see by a weight of zero, and 0 * inf is NaN; a row must not reach a column that it is masked from.  Such a
// tile ("dirty", found by reading it once more: only tiles on the edge are looked at) is contracted with those values
// taken as zero, and the workgroup adds them to the stored result of the columns that do see them.
__device__ __forceinline__ bool finite(float x) { return fabsf(x) <= 3.402823466e38f; }

__device__ __forceinline__ bool tile_dirty(const float* tile, int64_t stride, int limit, int D, int lane) {
  bool bad = false;
  for (int p = lane; p < limit * (D / 4); p += 64) {
    const float4 x = *reinterpret_cast<const float4*>(tile + (int64_t)(p / (D / 4)) * stride + p % (D / 4) * 4);
    bad = bad || !(finite(x.x) && finite(x.y) && finite(x.z) && finite(x.w));
  }
  return __any(bad);
}

template <int N>
__device__ __forceinline__ void scrub(Piece<N>& f) {
#pragma unroll
  for (int k = 0; k < N; ++k) f.x[k] = finite(f.x[k]) ? f.x[k] : 0.f;
}

// out[d] += X[t][d] wherever that is no finite number, for the rows t in [lo, hi); as_nan: their weight may have either sign
template <int DB>
__device__ __forceinline__ void add_nonfinite(float* out, float* out2, const float* x0, int64_t stride, int lo, int hi, int D, int g, bool as_nan) {
#pragma unroll 1
  for (int t = lo; t < hi; ++t)
#pragma unroll 1
    for (int d = 0; d < D; ++d) {
      const float x = x0[(int64_t)t * stride + d];
      if (((DB % 2 == 0 ? d / DB / 4 : d / 4) & 1) != g || finite(x)) continue;       // acc_block's half
      out[d] += as_nan ? __builtin_nanf("") : x;
      if (out2) out2[d] = out[d];
    }
}

template <int N>
__device__ __forceinline__ void zero_acc(f32x16 (&acc)[N]) {
#pragma unroll
  for (int i = 0; i < N; ++i)
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[i][v] = 0.f;
}

// Four neighbouring results of a lane, the columns from block_column on: number q of the DB that block j of its accumulators holds
template <int DB>
__device__ __forceinline__ int block_column(int j, int q, int g) { return DB % 2 == 0 ? 4 * (DB * (2 * j + g) + q) : 32 * q + 8 * j + 4 * g; }
template <int DB>
__device__ __forceinline__ float4 acc_block(const f32x16 (&acc)[DB], int j, int q, float c) {
  float x[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) x[e] = c * (DB % 2 == 0 ? acc[(4 * q + e) % DB][4 * j + (4 * q + e) / DB] : acc[q][4 * j + e]);
  return make_float4(x[0], x[1], x[2], x[3]);
}

__device__ __forceinline__ float4 add(float4 x, float4 y) { return make_float4(x.x + y.x, x.y + y.y, x.z + y.z, x.w + y.w); }

// One tree step of the fold of the wavefronts' accumulators: the upper half of `n` wavefronts puts its values down.
template <int N>
__device__ __forceinline__ void put_acc(float* slot, const f32x16 (&acc)[N], int lane) {
#pragma unroll
  for (int i = 0; i < N; ++i)
#pragma unroll
    for (int v = 0; v < 16; ++v) slot[(16 * i + v) * 64 + lane] = acc[i][v];
}
template <int N>
__device__ __forceinline__ void add_acc(const float* slot, f32x16 (&acc)[N], float own, float other, int lane) {
#pragma unroll
  for (int i = 0; i < N; ++i)
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[i][v] = own * acc[i][v] + other * slot[(16 * i + v) * 64 + lane];
}

// The 32-key tiles a query tile's workgroups walk, numbered through the chunks.  A share is a run of them, and the workgroup's
// wavefronts take the tiles of the run in turn: shares differ by one tile at most, whatever the mask and the chunks (dealt out
// in turns of eight, 104 tiles make four shares of 32 and 24: 4 heads x 400 rows x 8 chunks of 400 keys at head size 128 59 us,
// 51 so).  The table is in LDS because arguments come from host memory: a read of them is 0.7 us, and every chunk that the
// walk comes to would need some.
struct KeyTable {
  int32_t end[kMaxTable];                            // tiles up to and with this chunk that the workgroup's last row sees
  int64_t k_offset[kMaxTable];
  const float* k[kMaxTable];                         // of this head and batch entry
  const float* v[kMaxTable];
};
// by one wavefront, a lane per chunk; a barrier has to follow
__device__ __forceinline__ void build_key_table(KeyTable& tab, const Shape& s, const ChunkTable& t, int64_t last_pos, int b, int hk, int lane) {
  static_assert(kMaxTable == 64, "a lane per chunk");
  const int64_t k0 = t.k_offset[lane];               // the whole table is read: the loads need not wait for its length
  const float* k = (const float*)t.k[lane] + (int64_t)b * t.ksb + (int64_t)hk * t.ksh;
  const float* v = (const float*)t.v[lane] + (int64_t)b * t.vsb + (int64_t)hk * t.vsh;
  const int n = lane < t.n ? (visible_keys(s, last_pos, k0) + kT - 1) / kT : 0;
  int total;
  tab.end[lane] = lane_scan(n, total) + n;
  tab.k_offset[lane] = k0;
  tab.k[lane] = k;
  tab.v[lane] = v;
}
// tiles [lo, hi) of share y
__device__ __forceinline__ void key_share(int end, int n_split, int y, int& lo, int& hi) {
  const uint32_t total = (uint32_t)__builtin_amdgcn_readlane(end, 63), n = (uint32_t)max(n_split, 1), each = total / n, rest = total % n;
  lo = (int)(each * y + rest * y / n);
  hi = (int)(each * (y + 1) + rest * (y + 1) / n);
}
// Tile x of the walk, x below the last `end`; end = this lane's entry of the table
struct KeyTile {
  int key0;                                          // first key in its chunk
  int64_t k_offset;
  const float *k, *v;                                // at that key
};
__device__ __forceinline__ uint64_t uniform64(uint64_t x) { return (uint64_t)sgpr((uint32_t)x) | (uint64_t)sgpr((uint32_t)(x >> 32)) << 32; }
__device__ __forceinline__ const float* uniform_ptr(const float* p) { return (const float*)(GlobalFloats)uniform64((uint64_t)p); }
__device__ __forceinline__ KeyTile key_tile(const KeyTable& tab, const ChunkTable& t, int end, int x) {
  const int c = __popcll(__ballot(end <= x));
  const int first = c > 0 ? __builtin_amdgcn_readlane(end, c - 1) : 0;
  KeyTile y;
  y.key0 = (x - first) * kT;
  y.k_offset = (int64_t)uniform64((uint64_t)tab.k_offset[c]);
  y.k = uniform_ptr(tab.k[c]) + (int64_t)y.key0 * t.kss;
  y.v = uniform_ptr(tab.v[c]) + (int64_t)y.key0 * t.vss;
  return y;
}

// ---------------------------------------------------------------- forward
// Bounded by the matrix instructions: D per 32 x 32 tile pair and 64 cycles each.  Eight wavefronts share the 32 rows.  An
// under-filled launch gives a query tile several workgroups, each with a share of the walk (see KeyTable, TileShares).
template <int DP, bool FULL>
__global__ __launch_bounds__(waves<DP>() * 64) void fwd_f32_kernel(const FwdArgs a) {
  constexpr int NW = waves<DP>(), DB = DP / 32, N = 32, NR = row_pieces<DP, N>(), NC = col_pieces<DP, N>();
  __shared__ __attribute__((aligned(16))) float qs[kT * lds_stride<DP>()];
  __shared__ float fold[NW / 2 * DB * 16 * 64];
  __shared__ float fold_m[NW / 2 * 64], fold_l[NW / 2 * 64];
  __shared__ KeyTable tab;
  __shared__ int any_dirty;
  const Shape& s = a.s;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g = lane >> 5, r = lane & 31;
  const int n_qt = (s.Sq + kT - 1) / kT;
  int qt, hb, split;
  share_block(a.shares, blockIdx.x, gridDim.x, blockIdx.y, n_qt, s.causal, qt, hb, split);
  const int n_split = max(shares_of(a.shares, qt), 1);
  const int h = hb % s.Hq, b = hb / s.Hq, hk = h / (s.Hq / s.Hkv);
  const int row0 = qt * kT;
  const int64_t first_pos = q_pos(s, row0), last_pos = q_pos(s, min(row0 + kT, s.Sq) - 1);
  if (wave == 0) build_key_table(tab, s, a.t, last_pos, b, hk, lane);
  stage_tile<DP>(qs, (const float*)a.q.ptr + b * a.q.sb + h * a.q.sh, a.q.ss, row0, s.Sq, s.D, tid);
  if (tid == 0) any_dirty = 0;
  __syncthreads();

  const int i = min(row0 + r, s.Sq - 1);
  const int64_t qpos = q_pos(s, i);
  float m = -INFINITY, l = 0.f;
  f32x16 acc[DB];
  zero_acc(acc);
  const int end = tab.end[lane];
  int lo, hi;
  key_share(end, n_split, split, lo, hi);
  for (int x = lo + wave; x < hi; x += NW) {
    const KeyTile w = key_tile(tab, a.t, end, x);
    const float *kb = w.k, *vb = w.v;
    const int limit = min(kT, visible_keys(s, last_pos, w.k_offset) - w.key0);
    const int nv_first = visible_keys(s, first_pos, w.k_offset) - w.key0;                      // wave-uniform
    const int nv = nv_first < kT ? visible_keys(s, qpos, w.k_offset) - w.key0 : kT;
    const float* krow = kb + (int64_t)min(r, limit - 1) * a.t.kss;
    Piece<N> f[2];
    auto load = [&](int x) {
      if (x < NR) load_rows<DP, FULL>(f[x & 1], krow, x, s.D, g);
      else load_cols<DP, FULL>(f[x & 1], vb, a.t.vss, limit, x - NR, s.D, r, g);
      __builtin_amdgcn_sched_barrier(0);
    };
    f32x16 p;
#pragma unroll
    for (int v = 0; v < 16; ++v) p[v] = 0.f;
    load(0);
#pragma unroll
    for (int x = 0; x < NR; ++x) {
      load(x + 1);
      contract_d<DP>(p, f[x & 1], qs, x, r, g);
    }
    float mx = -INFINITY;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      p[v] = c_row(v, g) < nv ? s.scale * p[v] : -INFINITY;
      mx = fmaxf(mx, p[v]);
    }
    const float m_new = fmaxf(m, xhalf_max(mx));
    const float m_use = m_new == -INFINITY ? 0.f : m_new;      // no key of this row yet: every p below is exp(-inf) = 0
    float sum = 0.f;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      p[v] = expf(p[v] - m_use);
      sum += p[v];
    }
    const float alpha = expf(m - m_use);
    l = l * alpha + sum;
    m = m_new;
    if (__any(alpha != 1.f)) {
#pragma unroll
      for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[db][v] *= alpha;
    }
    const bool dirty = nv_first < limit && tile_dirty(vb, a.t.vss, limit, s.D, lane);          // wave-uniform
    if (dirty) any_dirty = 1;
#pragma unroll
    for (int x = NR; x < NR + NC; ++x) {
      if (x + 1 < NR + NC) load(x + 1);
      if (dirty) scrub(f[x & 1]);
      contract_rows<DP>(acc, f[x & 1], p, x - NR);
    }
  }

  // fold of the wavefronts' states (m, l, O), halving their number each time
  for (int n = NW / 2; n > 0; n /= 2) {
    if (wave >= n && wave < 2 * n) {
      put_acc(fold + (wave - n) * DB * 16 * 64, acc, lane);
      fold_m[(wave - n) * 64 + lane] = m;
      fold_l[(wave - n) * 64 + lane] = l;
    }
    __syncthreads();
    if (wave < n) {
      const float mo = fold_m[wave * 64 + lane], lo = fold_l[wave * 64 + lane];
      const float mn = fmaxf(m, mo), mu = mn == -INFINITY ? 0.f : mn;
      const float own = expf(m - mu), other = expf(mo - mu);
      add_acc(fold + wave * DB * 16 * 64, acc, own, other, lane);
      l = own * l + other * lo;
      m = mn;
    }
    __syncthreads();
  }
  if (wave != 0 || row0 + r >= s.Sq) return;
  l = xhalf_sum(l);
  const float inv = l > 0.f ? 1.f / l : 0.f;
  float* o = (n_split > 1 ? a.part_o + split * a.part_stride : a.o) + (((int64_t)b * s.Sq + row0 + r) * s.Hq + h) * s.D;
  float* ol = a.o_lowp && n_split <= 1 ? (float*)a.o_lowp + (((int64_t)b * s.Sq + row0 + r) * s.Hq + h) * s.D : nullptr;   // storage dtype is fp32 here
#pragma unroll
  for (int j = 0; j < 4; ++j)
#pragma unroll
    for (int q = 0; q < DB; ++q) {
      const int d = block_column<DB>(j, q, g);
      if (d >= s.D) continue;
      const float4 x = acc_block(acc, j, q, inv);
      *reinterpret_cast<float4*>(o + d) = x;
      if (ol) *reinterpret_cast<float4*>(ol + d) = x;
    }
  const int64_t stat = ((int64_t)b * s.Hq + h) * s.Sq + row0 + r;
  if (g == 0) (n_split > 1 ? a.part_lse + split * a.part_stride : a.lse)[stat] = l > 0.f ? m + logf(l) : -INFINITY;
  if (any_dirty)                                             // (a value that several shares add is the same infinity or NaN)
    for (int c = 0; c < a.t.n; ++c)
      add_nonfinite<DB>(o, ol, (const float*)a.t.v[c] + b * a.t.vsb + hk * a.t.vsh, a.t.vss,
                    visible_keys(s, first_pos, a.t.k_offset[c]) / kT * kT, visible_keys(s, qpos, a.t.k_offset[c]), s.D, g, false);
}

// ---------------------------------------------------------------- backward: dQ
// Three contractions per tile pair (S and dP are recomputed); otherwise the forward's layout and its shares.
template <int DP>
struct alignas(16) DqShared {
  float qs[kT * lds_stride<DP>()], dos[kT * lds_stride<DP>()];
  float fold[waves<DP>() / 2 * (DP / 32) * 16 * 64];
  KeyTable tab;
  int any_dirty;
};
template <int DP, bool FULL>
__device__ __forceinline__ void bwd_dq_f32(const BwdArgs& a, DqShared<DP>& sm, int block_x, int grid_x, int block_y) {
  constexpr int NW = waves<DP>(), DB = DP / 32, N = 32, NR = row_pieces<DP, N>(), NC = col_pieces<DP, N>();
  float *qs = sm.qs, *dos = sm.dos, *fold = sm.fold;
  KeyTable& tab = sm.tab;
  int& any_dirty = sm.any_dirty;
  const Shape& s = a.s;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g = lane >> 5, r = lane & 31;
  const int n_qt = (s.Sq + kT - 1) / kT;
  int qt, hb, split;
  share_block(a.shares, block_x, grid_x, block_y, n_qt, s.causal, qt, hb, split);
  const int n_split = max(shares_of(a.shares, qt), 1);
  const int h = hb % s.Hq, b = hb / s.Hq, hk = h / (s.Hq / s.Hkv);
  const int row0 = qt * kT;
  const int64_t first_pos = q_pos(s, row0), last_pos = q_pos(s, min(row0 + kT, s.Sq) - 1);
  if (wave == 0) build_key_table(tab, s, a.t, last_pos, b, hk, lane);
  stage_tile<DP>(qs, (const float*)a.q.ptr + b * a.q.sb + h * a.q.sh, a.q.ss, row0, s.Sq, s.D, tid);
  stage_tile<DP>(dos, (const float*)a.d_o.ptr + b * a.d_o.sb + h * a.d_o.sh, a.d_o.ss, row0, s.Sq, s.D, tid);
  if (tid == 0) any_dirty = 0;
  __syncthreads();

  const int i = min(row0 + r, s.Sq - 1);
  const int64_t stat = ((int64_t)b * s.Hq + h) * s.Sq + i;
  const float lse = a.lse[stat], dl = a.delta[stat];
  const bool empty = lse == -INFINITY;                       // empty row: no gradient
  const int64_t qpos = q_pos(s, i);
  f32x16 acc[DB];
  zero_acc(acc);
  const int end = tab.end[lane];
  int lo, hi;
  key_share(end, n_split, split, lo, hi);
  for (int x = lo + wave; x < hi; x += NW) {
    const KeyTile w = key_tile(tab, a.t, end, x);
    const float *kb = w.k, *vb = w.v;
    const int limit = min(kT, visible_keys(s, last_pos, w.k_offset) - w.key0);
    const int nv_first = visible_keys(s, first_pos, w.k_offset) - w.key0;                      // wave-uniform
    const int nv = empty ? 0 : nv_first < kT ? visible_keys(s, qpos, w.k_offset) - w.key0 : kT;
    const float* krow = kb + (int64_t)min(r, limit - 1) * a.t.kss;
    const float* vrow = vb + (int64_t)min(r, limit - 1) * a.t.vss;
    Piece<N> f[2];
    auto load = [&](int x) {
      if (x < 2 * NR) load_rows<DP, FULL>(f[x & 1], x < NR ? krow : vrow, x < NR ? x : x - NR, s.D, g);
      else load_cols<DP, FULL>(f[x & 1], kb, a.t.kss, limit, x - 2 * NR, s.D, r, g);
      __builtin_amdgcn_sched_barrier(0);
    };
    f32x16 p, ds;
#pragma unroll
    for (int v = 0; v < 16; ++v) p[v] = ds[v] = 0.f;
    load(0);
#pragma unroll
    for (int x = 0; x < 2 * NR; ++x) {
      load(x + 1);
      if (x < NR) contract_d<DP>(p, f[x & 1], qs, x, r, g);
      else contract_d<DP>(ds, f[x & 1], dos, x - NR, r, g);
    }
#pragma unroll
    for (int v = 0; v < 16; ++v) ds[v] = c_row(v, g) < nv ? expf(s.scale * p[v] - lse) * (ds[v] - dl) : 0.f;
    const bool dirty = nv_first < limit && tile_dirty(kb, a.t.kss, limit, s.D, lane);          // wave-uniform
    if (dirty) any_dirty = 1;
#pragma unroll
    for (int x = 2 * NR; x < 2 * NR + NC; ++x) {
      if (x + 1 < 2 * NR + NC) load(x + 1);
      if (dirty) scrub(f[x & 1]);
      contract_rows<DP>(acc, f[x & 1], ds, x - 2 * NR);
    }
  }
  for (int n = NW / 2; n > 0; n /= 2) {
    if (wave >= n && wave < 2 * n) put_acc(fold + (wave - n) * DB * 16 * 64, acc, lane);
    __syncthreads();
    if (wave < n) add_acc(fold + wave * DB * 16 * 64, acc, 1.f, 1.f, lane);
    __syncthreads();
  }
  if (wave != 0 || row0 + r >= s.Sq) return;
  const bool part = n_split > 1 && split >= a.shares.own0;   // a sum of its own (its memory holds nothing yet), not dq itself
  if (empty && !part) return;
  float* dq = (part ? dq_part(a.parts, s, query_tiles(s, kT), a.shares, b, qt, split - a.shares.own0) : a.dq + ((int64_t)b * s.Sq + row0) * s.Hq * s.D) + ((int64_t)r * s.Hq + h) * s.D;
#pragma unroll
  for (int j = 0; j < 4; ++j)
#pragma unroll
    for (int q = 0; q < DB; ++q) {
      const int d = block_column<DB>(j, q, g);
      if (d >= s.D) continue;
      float4 x = part ? make_float4(0.f, 0.f, 0.f, 0.f) : *reinterpret_cast<float4*>(dq + d);
      x = add(x, acc_block(acc, j, q, s.scale));
      *reinterpret_cast<float4*>(dq + d) = x;
    }
  if (any_dirty && !empty)
    for (int c = 0; c < a.t.n; ++c)
      add_nonfinite<DB>(dq, nullptr, (const float*)a.t.k[c] + b * a.t.ksb + hk * a.t.ksh, a.t.kss,
                    visible_keys(s, first_pos, a.t.k_offset[c]) / kT * kT, visible_keys(s, qpos, a.t.k_offset[c]), s.D, g, true);
}

// ---------------------------------------------------------------- backward: dK, dV
// block = key tile + ceil(Sk / 32) (KV head + Hkv (batch entry + B (chunk + n share))).  An under-filled launch gives every key
// tile kv_items workgroups, each with a run of its (head, row tile) pairs: 4/1 heads of 256 x 534 rows are 17 key tiles of up to
// 68 pairs, 379 us on 17 workgroups; with dQ (53 us) and the pass that adds up 91 + 7 now.
template <int DP>
struct alignas(16) DkvShared {
  float ks[kT * lds_stride<DP>()], vs[kT * lds_stride<DP>()];
  float stats[waves<DP>() * 64];
  float fold[waves<DP>() / 2 * (DP / 32) * 16 * 64];
  int any_dirty;
};
template <int DP, bool FULL>
__device__ __forceinline__ void bwd_dkv_f32(const BwdArgs& a, DkvShared<DP>& sm, int block) {
  constexpr int NW = waves<DP>(), DB = DP / 32, N = DP < 128 ? 32 : 16, NR = row_pieces<DP, N>(), NC = col_pieces<DP, N>();
  float *ks = sm.ks, *vs = sm.vs, *fold = sm.fold, *stats = sm.stats;
  int& any_dirty = sm.any_dirty;
  const Shape& s = a.s;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g = lane >> 5, r = lane & 31;
  const int n_kt = (s.Sk + kT - 1) / kT, outer = block / n_kt, bc = outer / s.Hkv, cs = bc / s.B;
  const int key0 = (int)sgpr((block - outer * n_kt) * kT), hk = (int)sgpr(outer - bc * s.Hkv), b = (int)sgpr(bc - cs * s.B);
  const int share = (int)sgpr(cs / a.t.n), c = (int)sgpr(cs - share * a.t.n);
  const int G = s.Hq / s.Hkv;
  const int64_t k0 = a.t.k_offset[c];
  // row i sees key t of the chunk iff i >= first_row(t)
  auto first_row = [&](int t) { return s.causal ? q_row_of(s, k0 + t) : 0; };
  const int wg_first = first_row(key0);
  if (wg_first >= s.Sq) return;                              // uniform over the workgroup
  const int wg_all = first_row(min(key0 + kT, s.Sk) - 1);    // from this row on every key is seen
  stage_tile<DP>(ks, (const float*)a.t.k[c] + b * a.t.ksb + hk * a.t.ksh, a.t.kss, key0, s.Sk, s.D, tid);
  stage_tile<DP>(vs, (const float*)a.t.v[c] + b * a.t.vsb + hk * a.t.vsh, a.t.vss, key0, s.Sk, s.D, tid);
  if (tid == 0) any_dirty = 0;
  __syncthreads();

  const int key_first = first_row(min(key0 + r, s.Sk - 1));
  const int t_lo = wg_first / kT, per_head = (s.Sq + kT - 1) / kT - t_lo;
  f32x16 acc_k[DB], acc_v[DB];
  zero_acc(acc_k);
  zero_acc(acc_v);
  const int pairs = G * per_head, n_share = max(a.kv_items, 1);
  for (int x = pairs * share / n_share + wave, x1 = pairs * (share + 1) / n_share; x < x1; x += NW) {
    const int h = hk * G + x / per_head, i0 = (t_lo + x % per_head) * kT;
    const float* qb = (const float*)a.q.ptr + b * a.q.sb + h * a.q.sh + (int64_t)i0 * a.q.ss;
    const float* db_ = (const float*)a.d_o.ptr + b * a.d_o.sb + h * a.d_o.sh + (int64_t)i0 * a.d_o.ss;
    const int64_t stat = ((int64_t)b * s.Hq + h) * s.Sq + i0;
    const int limit = min(kT, s.Sq - i0), lo = key_first - i0;
    const float* qrow = qb + (int64_t)min(r, limit - 1) * a.q.ss;
    const float* drow = db_ + (int64_t)min(r, limit - 1) * a.d_o.ss;
    Piece<N> f[2];
    auto load = [&](int x) {
      if (x < 2 * NR) load_rows<DP, FULL>(f[x & 1], x < NR ? qrow : drow, x < NR ? x : x - NR, s.D, g);
      else if (x < 2 * NR + NC) load_cols<DP, FULL>(f[x & 1], db_, a.d_o.ss, limit, x - 2 * NR, s.D, r, g);
      else load_cols<DP, FULL>(f[x & 1], qb, a.q.ss, limit, x - 2 * NR - NC, s.D, r, g);
      __builtin_amdgcn_sched_barrier(0);
    };
    f32x16 p, ds;
#pragma unroll
    for (int v = 0; v < 16; ++v) p[v] = ds[v] = 0.f;
    load(0);
#pragma unroll
    for (int x = 0; x < 2 * NR; ++x) {
      load(x + 1);
      if (x < NR) contract_d<DP>(p, f[x & 1], ks, x, r, g);
      else contract_d<DP>(ds, f[x & 1], vs, x - NR, r, g);
    }
    // the tile's row statistics pass through LDS: lse in the first 32 floats of this wavefront's slot, Delta behind
    stats[wave * 64 + lane] = (g ? a.delta : a.lse)[stat + min(r, limit - 1)];
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const float4 lse = *reinterpret_cast<const float4*>(stats + wave * 64 + 8 * j + 4 * g);
      const float4 dl = *reinterpret_cast<const float4*>(stats + wave * 64 + 32 + 8 * j + 4 * g);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int v = 4 * j + e, row = c_row(v, g);
        const float ls = e == 0 ? lse.x : e == 1 ? lse.y : e == 2 ? lse.z : lse.w, de = e == 0 ? dl.x : e == 1 ? dl.y : e == 2 ? dl.z : dl.w;
        const bool live = row >= lo && row < limit && ls != -INFINITY;
        p[v] = live ? expf(s.scale * p[v] - ls) : 0.f;
        ds[v] = live ? p[v] * (ds[v] - de) : 0.f;
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    __builtin_amdgcn_wave_barrier();
    const bool crossed = i0 < wg_all;                        // wave-uniform: some key does not see some row
    const bool dirty = crossed && (tile_dirty(db_, a.d_o.ss, limit, s.D, lane) || tile_dirty(qb, a.q.ss, limit, s.D, lane));
    if (dirty) any_dirty = 1;
#pragma unroll
    for (int x = 2 * NR; x < 2 * NR + 2 * NC; ++x) {
      if (x + 1 < 2 * NR + 2 * NC) load(x + 1);
      if (dirty) scrub(f[x & 1]);
      if (x < 2 * NR + NC) contract_rows<DP>(acc_v, f[x & 1], p, x - 2 * NR);
      else contract_rows<DP>(acc_k, f[x & 1], ds, x - 2 * NR - NC);
    }
  }
  for (int n = NW / 2; n > 0; n /= 2) {
    float* slot = fold + (wave - (wave >= n ? n : 0)) * DB * 16 * 64;
    if (wave >= n && wave < 2 * n) put_acc(slot, acc_k, lane);
    __syncthreads();
    if (wave < n) add_acc(slot, acc_k, 1.f, 1.f, lane);
    __syncthreads();
    if (wave >= n && wave < 2 * n) put_acc(slot, acc_v, lane);
    __syncthreads();
    if (wave < n) add_acc(slot, acc_v, 1.f, 1.f, lane);
    __syncthreads();
  }
  if (wave != 0 || key0 + r >= s.Sk || key_first >= s.Sq) return;
  const int64_t orow = (((int64_t)b * s.Sk + key0 + r) * s.Hkv + hk) * s.D;
  float* out_k = (share ? f32_kv_part(a.kv_parts, s, a.t.n, share, c, 0) : a.dk[c]) + orow;
  float* out_v = (share ? f32_kv_part(a.kv_parts, s, a.t.n, share, c, 1) : a.dv[c]) + orow;
#pragma unroll
  for (int j = 0; j < 4; ++j)
#pragma unroll
    for (int q = 0; q < DB; ++q) {
      const int d = block_column<DB>(j, q, g);
      if (d >= s.D) continue;
      float4* pk = reinterpret_cast<float4*>(out_k + d);
      float4* pv = reinterpret_cast<float4*>(out_v + d);
      float4 x = make_float4(0.f, 0.f, 0.f, 0.f), y = x;      // the memory of a partial sum holds nothing yet
      if (share == 0) x = *pk, y = *pv;
      x = add(x, acc_block(acc_k, j, q, s.scale));
      y = add(y, acc_block(acc_v, j, q, 1.f));
      *pk = x;
      *pv = y;
    }
  if (any_dirty)
    for (int h = hk * G; h < (hk + 1) * G; ++h) {
      const int hi = min(s.Sq, (wg_all + kT - 1) / kT * kT);
      add_nonfinite<DB>(out_k, nullptr, (const float*)a.q.ptr + b * a.q.sb + h * a.q.sh, a.q.ss, key_first, hi, s.D, g, true);
      add_nonfinite<DB>(out_v, nullptr, (const float*)a.d_o.ptr + b * a.d_o.sb + h * a.d_o.sh, a.d_o.ss, key_first, hi, s.D, g, false);
    }
}

// Both passes in one launch: the first n_kv workgroups are key tiles, the others the dQ launch's blocks.  Neither needs the other's
// results, each is a chain of latencies at its start and its end, and a causal shard's key tiles do unlike amounts of work:
// one head x 128 rows x 4 chunks of 128 keys 16 and 24 us apart and a gap between them, 8/2 heads x 512 rows x 8 chunks of
// 512 keys 206 and 152.  The workgroups are numbered through rows of `row`: a dimension of a grid holds fewer than 2^32 threads,
// and one that is wider loses the rest without an error.
template <int DP, bool FULL>
__global__ __launch_bounds__(waves<DP>() * 64) void bwd_f32_kernel(const BwdArgs a, uint32_t n_kv, int q_blocks, uint32_t row, uint32_t blocks) {
  __shared__ union Both {
    DqShared<DP> dq;
    DkvShared<DP> dkv;
  } sm;
  const uint32_t block = blockIdx.y * row + blockIdx.x;
  if (block >= blocks) return;
  if (block < n_kv) {
    bwd_dkv_f32<DP, FULL>(a, sm.dkv, (int)block);
  } else {
    const int x = (int)(block - n_kv);
    bwd_dq_f32<DP, FULL>(a, sm.dq, (int)sgpr(x % q_blocks), q_blocks, (int)sgpr(x / q_blocks));
  }
}

// f(integral constant, full): the kernels are built for these D, and for smaller ones with zero-filled columns
template <typename F>
hipError_t with_padded_d(int D, F f) {
  using std::integral_constant;
  constexpr integral_constant<bool, true> full;
  constexpr integral_constant<bool, false> padded;
  if (D == 64) return f(integral_constant<int, 64>(), full);
  if (D == 128) return f(integral_constant<int, 128>(), full);
  if (D == 256) return f(integral_constant<int, 256>(), full);
  if (D <= 32) return f(integral_constant<int, 32>(), padded);
  if (D <= 64) return f(integral_constant<int, 64>(), padded);
  if (D <= 96) return f(integral_constant<int, 96>(), padded);
  if (D <= 128) return f(integral_constant<int, 128>(), padded);
  if (D <= 192) return f(integral_constant<int, 192>(), padded);
  if (D <= 256) return f(integral_constant<int, 256>(), padded);
  return hipErrorInvalidValue;
}

}  // namespace

hipError_t launch_fwd_f32(const FwdArgs& a, hipStream_t stream) {
  const int64_t total = (int64_t)((a.s.Sq + kT - 1) / kT) * a.s.Hq * a.s.B;
  if (total <= 0) return hipSuccess;
  if (total > 0x7fffffff) return hipErrorInvalidValue;
  ProfScope prof("fwd_f32", stream);
  return with_padded_d(a.s.D, [&](auto dp, auto full) {
    constexpr int DP = decltype(dp)::value;
    constexpr bool FULL = decltype(full)::value;
    const dim3 grid = share_grid(a.shares, total, (a.s.Sq + kT - 1) / kT);
    hipLaunchKernelGGL((fwd_f32_kernel<DP, FULL>), grid, dim3(waves<DP>() * 64), 0, stream, a);
    return hipGetLastError();
  });
}

hipError_t launch_bwd_f32(const BwdArgs& a, hipStream_t stream) {
  const int n_qt = (a.s.Sq + kT - 1) / kT;
  const int64_t total = (int64_t)n_qt * a.s.Hq * a.s.B;
  if (total <= 0 || a.t.n == 0 || a.s.Sk == 0) return hipSuccess;
  const dim3 q_grid = share_grid(a.shares, total, n_qt);
  const int64_t n_kv = (int64_t)((a.s.Sk + kT - 1) / kT) * a.s.Hkv * a.s.B * a.t.n * std::max(a.kv_items, 1), blocks = n_kv + (int64_t)q_grid.x * q_grid.y;
  if (total > 0x7fffffff || blocks > 0x7fffffff) return hipErrorInvalidValue;
  hipError_t e = with_padded_d(a.s.D, [&](auto dp, auto full) {
    constexpr int DP = decltype(dp)::value;
    constexpr bool FULL = decltype(full)::value;
    ProfScope prof("bwd_f32", stream);
    const uint32_t row = (uint32_t)std::min<int64_t>(blocks, 1 << 22);
    hipLaunchKernelGGL((bwd_f32_kernel<DP, FULL>), dim3(row, (unsigned)((blocks + row - 1) / row)), dim3(waves<DP>() * 64), 0, stream, a, (uint32_t)n_kv,
                       (int)q_grid.x, row, (uint32_t)blocks);
    return hipGetLastError();
  });
  if (e == hipSuccess && a.kv_items > 1) e = launch_add_kv_parts_f32(a, stream);
  if (e == hipSuccess && a.shares.n > 1) e = launch_add_parts(a, kT, stream);
  return e;
}

}  // namespace st
