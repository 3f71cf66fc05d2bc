// HBM-bound passes: log-sum-exp merge of two partial states, combine of n partial states,
// Delta = rowsum(dO * O),
// fp32 -> storage-dtype casts and the (O = 0, lse = -inf) state fill.
// One 16-byte vector per lane, rows never straddle a lane; grid sized to the data.
#include <type_traits>

#include "st_internal.h"
#include "st_mfma.h"
#include "st_walk.h"

namespace st {
namespace {

__device__ __forceinline__ uint32_t f32_to_bf16_rne(float f) {
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7fffffffu) > 0x7f800000u) return (u >> 16) | 0x40u;   // NaN stays NaN
  return (u + 0x7fffu + ((u >> 16) & 1u)) >> 16;
}
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
  return f32_to_bf16_rne(lo) | (f32_to_bf16_rne(hi) << 16);
}
__device__ __forceinline__ float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }

// (b, i, h) of row (b * S + i) * H + h of `rows`.  Two 64-bit divisions are some 300 instructions per lane, which
// launches of a few megabytes do not hide; the rows of a tensor fit 32 bits but for the largest.
struct RowOf {
  int64_t b;
  int32_t i, h;
};
__device__ __forceinline__ RowOf row_of(int64_t row, int64_t rows, int32_t S, int32_t H) {
  if (rows <= 0x7fffffff) {
    const uint32_t x = (uint32_t)row, bi = x / (uint32_t)H, b = bi / (uint32_t)S;
    return RowOf{(int64_t)b, (int32_t)(bi - b * (uint32_t)S), (int32_t)(x - bi * (uint32_t)H)};
  }
  const int64_t bi = row / H;
  return RowOf{bi / S, (int32_t)(bi % S), (int32_t)(row % H)};
}

// ---- merge: thread = up to U float4 of one (b, i, h) row ---------------------------------------
// A row occupies a power-of-two group of lanes; lane `sub` of the group takes the vectors sub, sub + lanes, ...
// of the row, so consecutive lanes read consecutive 16-byte pieces (whole 128-byte lines once the group has
// eight lanes), the row's two lse are read once per U vectors and its weights are computed once.
// The group never straddles a wavefront: every lane of the row has read lse_acc before lane 0 overwrites it.
// Weights: w_acc = exp(lse_acc - lse'), w_part = exp(lse_part - lse'), lse' = max + log(sum).
// A side with lse = -inf gets weight 0 without ever forming (-inf) - (-inf), and its O is not read into the sum.
// U = vectors per thread (1, 2 or 4): all loads of a thread are in flight before its first store.
template <bool kLowp, int U>
__global__ __launch_bounds__(256) void merge_kernel(float* __restrict__ o_acc, float* __restrict__ lse_acc,
                                                    const float* __restrict__ o_part,
                                                    const float* __restrict__ lse_part, int64_t n_rows,
                                                    int32_t Sq, int32_t Hq, int32_t vec_per_row,
                                                    int32_t lane_shift, uint2* __restrict__ o_lowp) {
  const int64_t tid = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int64_t row = tid >> lane_shift;               // (b * Sq + i) * Hq + h
  const int32_t sub = (int32_t)(tid & ((1 << lane_shift) - 1));
  if (row >= n_rows) return;
  const RowOf at = row_of(row, n_rows, Sq, Hq);
  const int64_t sidx = (at.b * Hq + at.h) * Sq + at.i;
  const float la = lse_acc[sidx], lp = lse_part[sidx];
  int64_t v[U];
  bool live[U];
  float4 a[U], p[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int32_t vi = sub + (u << lane_shift);
    live[u] = vi < vec_per_row;
    v[u] = row * vec_per_row + (live[u] ? vi : 0);     // a slot beyond the row reads its first vector and stores nothing
    a[u] = reinterpret_cast<const float4*>(o_acc)[v[u]];
    typedef float f32x4_t __attribute__((ext_vector_type(4)));
    const f32x4_t t = __builtin_nontemporal_load(reinterpret_cast<const f32x4_t*>(o_part) + v[u]);   // read once
    p[u] = make_float4(t.x, t.y, t.z, t.w);
  }
  const float m = fmaxf(la, lp);
  float wa = 0.f, wp = 0.f, lnew = -INFINITY;
  if (m != -INFINITY) {
    const float ea = expf(la - m), ep = expf(lp - m);  // exp(-inf) = 0 for an empty side
    const float sum = ea + ep;
    lnew = m + logf(sum);
    const float inv = 1.f / sum;
    wa = ea * inv;
    wp = ep * inv;
  }
#pragma unroll
  for (int u = 0; u < U; ++u) {
    if (!live[u]) continue;
    // a side whose weight is exactly 0 (an empty state) is left out, so that a non-finite value in its O
    // (never written, or stale) cannot turn the result into NaN; the combine pass does the same
    const float4 za = wa != 0.f ? a[u] : make_float4(0.f, 0.f, 0.f, 0.f);
    const float4 zp = wp != 0.f ? p[u] : make_float4(0.f, 0.f, 0.f, 0.f);
    float4 r;
    r.x = wa * za.x + wp * zp.x;
    r.y = wa * za.y + wp * zp.y;
    r.z = wa * za.z + wp * zp.z;
    r.w = wa * za.w + wp * zp.w;
    reinterpret_cast<float4*>(o_acc)[v[u]] = r;
    if (kLowp) o_lowp[v[u]] = make_uint2(pack_bf16x2(r.x, r.y), pack_bf16x2(r.z, r.w));
  }
  if (sub == 0) lse_acc[sidx] = lnew;
}

// ---- combine: n partial states of the same rows -> one state, keeping a run of rows -----------
// Thread = one float4 of one kept (b, i, h) row, lanes per row as in the merge.  The weights are
// w_x = exp(lse_x - m) / sum_y exp(lse_y - m) with m the largest lse, so an empty state (lse = -inf)
// weighs 0 and (-inf) - (-inf) is never formed; a row empty in every state gives O = 0, lse = -inf.
// kFew: at most that many states, each lse of which is read once and kept (0: any number, lse read three times, one wait
// after the other).  O loads in flight together: all for up to 4 and 9 to 16 states, otherwise kCombineUnroll (8 states of
// 8 x 1024 rows of 128: 12.0 us, 12.4 with all eight at once).  16 states of 4 x 256 rows, the split of a short shard: 17.5
// us without their number known, 9.3 with it; of 8 x 1024 rows 21.7 and 18.5.
// kOwn: the states of a split forward whose tiles have numbers of their own.  Where all have the same it stays uniform: one head
// x 3000 rows 7.6 us, 7.9 with a number per lane.  (Numbers of their own: the last state read again in the place of the ones a
// row lacks, so that no load hangs on a mask, 8.0 for 7.5 us at 8 heads x 1024 rows; a uniform path for wavefronts whose rows
// agree 7.2 for 6.4 at 12 x 448: twice the code, and launches this short fetch all of it.)
constexpr int kCombineUnroll = 4;
template <bool kLowp, int kFew, bool kOwn = false>
__global__ __launch_bounds__(256) void combine_kernel(const CombineArgs a, int32_t vec_per_row, int32_t lane_shift) {
  const int64_t tid = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int64_t row = tid >> lane_shift;               // (b * Sq_out + i) * Hq + h
  const int32_t sub = (int32_t)(tid & ((1 << lane_shift) - 1));
  const int64_t n_rows = (int64_t)a.B * a.Sq_out * a.Hq;
  if (row >= n_rows || sub >= vec_per_row) return;
  const RowOf at = row_of(row, n_rows, a.Sq_out, a.Hq);
  const int64_t b = at.b;
  const int32_t i = at.i, h = at.h;
  const int64_t l_in = (b * a.Hq + h) * a.Sq_in + a.row0 + i;
  const int64_t v_in = ((b * a.Sq_in + a.row0 + i) * a.Hq + h) * vec_per_row + sub;

  typedef float f32x4_t __attribute__((ext_vector_type(4)));
  auto load_o = [&](int x) {
    const f32x4_t t = __builtin_nontemporal_load(reinterpret_cast<const f32x4_t*>(a.o[x]) + v_in);   // read once
    return make_float4(t.x, t.y, t.z, t.w);
  };
  // The O of an empty state may never have been written (the split forward leaves it out): it is loaded like the others, and a
  // weight of exactly 0 keeps it, NaN or not, out of the sum.
  auto add = [](float4& r, float w, const float4& p) {
    if (w != 0.f) {
      r.x = fmaf(w, p.x, r.x);
      r.y = fmaf(w, p.y, r.y);
      r.z = fmaf(w, p.z, r.z);
      r.w = fmaf(w, p.w, r.w);
    }
  };
  float4 r = make_float4(0.f, 0.f, 0.f, 0.f);
  float lnew = -INFINITY;
  if constexpr (kFew > 0) {
    // every lse is read once and kept, and the first O loads do not wait for them
    constexpr int N = kFew, U = N == 8 ? kCombineUnroll : N;
    int n = a.n;                                         // states that hold this row
    if constexpr (kOwn) {
      n = shares_of(a.shares, a.tiles.tile_of(i));
      if (n <= 1) return;
    }
    auto load_few = [&](int x) { return x < n ? load_o(x) : make_float4(0.f, 0.f, 0.f, 0.f); };
    float l[N];
    float4 p[U];
#pragma unroll
    for (int x = 0; x < N; ++x) l[x] = x < n ? a.lse[x][l_in] : -INFINITY;
#pragma unroll
    for (int u = 0; u < U; ++u) p[u] = load_few(u);
    float m = -INFINITY;
#pragma unroll
    for (int x = 0; x < N; ++x) m = fmaxf(m, l[x]);
    if (m != -INFINITY) {
      float sum = 0.f;
#pragma unroll
      for (int x = 0; x < N; ++x) {
        l[x] = expf(l[x] - m);                           // exp(-inf) = 0 for an empty state and for x >= n
        sum += l[x];
      }
      lnew = m + logf(sum);
      const float inv = 1.f / sum;
#pragma unroll
      for (int x0 = 0; x0 < N; x0 += U) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
          if (x0 > 0) p[u] = load_few(x0 + u);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) add(r, x0 + u < n ? l[x0 + u] * inv : 0.f, p[u]);
      }
    }
  } else {
    float m = -INFINITY;
    for (int x = 0; x < a.n; ++x) m = fmaxf(m, a.lse[x][l_in]);
    if (m != -INFINITY) {
      float sum = 0.f;
      for (int x = 0; x < a.n; ++x) sum += expf(a.lse[x][l_in] - m);
      lnew = m + logf(sum);
      const float inv = 1.f / sum;
      for (int x0 = 0; x0 < a.n; x0 += kCombineUnroll) {
        float4 p[kCombineUnroll];
        float w[kCombineUnroll];
#pragma unroll
        for (int u = 0; u < kCombineUnroll; ++u) {
          const int x = x0 + u < a.n ? x0 + u : a.n - 1;
          p[u] = load_o(x);
          w[u] = x0 + u < a.n ? expf(a.lse[x][l_in] - m) * inv : 0.f;
        }
#pragma unroll
        for (int u = 0; u < kCombineUnroll; ++u) add(r, w[u], p[u]);
      }
    }
  }
  const int64_t v_out = row * vec_per_row + sub;
  reinterpret_cast<float4*>(a.o_out)[v_out] = r;
  if (kLowp) reinterpret_cast<uint2*>(a.o_lowp)[v_out] = make_uint2(pack_bf16x2(r.x, r.y), pack_bf16x2(r.z, r.w));
  if (sub == 0) a.lse_out[(b * a.Hq + h) * a.Sq_out + i] = lnew;
}

// fp32 "lowp" copy for the fp32 storage dtype; the last n % 4 values one by one
__global__ __launch_bounds__(256) void copy_f32_kernel(const float4* src, float4* dst, int64_t n) {
  const int64_t v = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (4 * v + 4 <= n) dst[v] = src[v];
  else
    for (int64_t i = 4 * v; i < n; ++i) reinterpret_cast<float*>(dst)[i] = reinterpret_cast<const float*>(src)[i];
}

// ---- delta: 16 lanes per row, 16-byte loads, shuffle reduction inside the 16-lane group -------
template <bool kDoBf16, bool kOBf16>
__global__ __launch_bounds__(256) void delta_kernel(View d_o, View o, float* __restrict__ delta, int32_t B,
                                                    int32_t Sq, int32_t Hq, int32_t D) {
  const int64_t row = ((int64_t)blockIdx.x * 256 + threadIdx.x) >> 4;
  const int sub = threadIdx.x & 15;
  const int64_t n_rows = (int64_t)B * Sq * Hq;
  const RowOf at = row_of(row, n_rows, Sq, Hq);
  const int64_t b = at.b;
  const int32_t i = at.i, h = at.h;
  float acc = 0.f;
  if (row < n_rows) {
    const int64_t off_d = b * d_o.sb + (int64_t)i * d_o.ss + (int64_t)h * d_o.sh;
    const int64_t off_o = b * o.sb + (int64_t)i * o.ss + (int64_t)h * o.sh;
    for (int d = sub * 8; d < D; d += 128) {           // 8 elements per lane per step
      float x[8], y[8];
      if (kDoBf16) {
        const uint4 u = *reinterpret_cast<const uint4*>((const uint16_t*)d_o.ptr + off_d + d);
        x[0] = bf16_lo(u.x); x[1] = bf16_hi(u.x); x[2] = bf16_lo(u.y); x[3] = bf16_hi(u.y);
        x[4] = bf16_lo(u.z); x[5] = bf16_hi(u.z); x[6] = bf16_lo(u.w); x[7] = bf16_hi(u.w);
      } else {
        const float4 u0 = *reinterpret_cast<const float4*>((const float*)d_o.ptr + off_d + d);
        const float4 u1 = *reinterpret_cast<const float4*>((const float*)d_o.ptr + off_d + d + 4);
        x[0] = u0.x; x[1] = u0.y; x[2] = u0.z; x[3] = u0.w; x[4] = u1.x; x[5] = u1.y; x[6] = u1.z; x[7] = u1.w;
      }
      if (kOBf16) {
        const uint4 u = *reinterpret_cast<const uint4*>((const uint16_t*)o.ptr + off_o + d);
        y[0] = bf16_lo(u.x); y[1] = bf16_hi(u.x); y[2] = bf16_lo(u.y); y[3] = bf16_hi(u.y);
        y[4] = bf16_lo(u.z); y[5] = bf16_hi(u.z); y[6] = bf16_lo(u.w); y[7] = bf16_hi(u.w);
      } else {
        const float4 u0 = *reinterpret_cast<const float4*>((const float*)o.ptr + off_o + d);
        const float4 u1 = *reinterpret_cast<const float4*>((const float*)o.ptr + off_o + d + 4);
        y[0] = u0.x; y[1] = u0.y; y[2] = u0.z; y[3] = u0.w; y[4] = u1.x; y[5] = u1.y; y[6] = u1.z; y[7] = u1.w;
      }
#pragma unroll
      for (int e = 0; e < 8; ++e) acc = fmaf(x[e], y[e], acc);
    }
  }
#pragma unroll
  for (int s = 8; s > 0; s >>= 1) acc += __shfl_xor(acc, s);
  if (row < n_rows && sub == 0) delta[(b * Hq + h) * Sq + i] = acc;
}

// ---- backward preparation of a bf16 share in one pass: Delta, Q' = bf16(Q c), the tile counters of the dK/dV launch to zero.
// Lanes per row = D / 8, one 16-byte vector of each of dO, O (two of an fp32 O), Q per thread.  Bytes only; as three
// launches these were 4.5 (counters), 10 and 9 us for 2048 rows of 32 heads of 128, each with a gap to the next.
__device__ __forceinline__ void do_reset(const OneReset& r) {
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < r.n; i += (int64_t)gridDim.x * 256) r.zero[i] = make_uint4(i == r.plenty ? 0x7fffffffu : 0u, 0u, 0u, 0u);
}
__global__ __launch_bounds__(256) void one_reset_kernel(OneReset r) { do_reset(r); }

template <bool kOBf16, int LPR>
__global__ __launch_bounds__(256) void bwd_prep_kernel(View d_o, View o, View q, float* __restrict__ delta, u32x4* __restrict__ qs,
                                                       int32_t* __restrict__ queue, OneReset reset, int32_t B, int32_t Sq, int32_t Hq, float c) {
  if (blockIdx.x == 0 && threadIdx.x < kQueueInts) queue[threadIdx.x] = 0;
  do_reset(reset);
  const int64_t v = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int64_t row = v / LPR;
  const int d = (int)(v % LPR) * 8;
  const int64_t n_rows = (int64_t)B * Sq * Hq;
  const bool live = row < n_rows;
  const RowOf at = row_of(row, n_rows, Sq, Hq);
  const int64_t b = at.b;
  const int32_t i = at.i, h = at.h;
  float acc = 0.f;
  if (live) {
    const uint4 x = *reinterpret_cast<const uint4*>((const uint16_t*)d_o.ptr + b * d_o.sb + (int64_t)i * d_o.ss + (int64_t)h * d_o.sh + d);
    const u32x4 z = *reinterpret_cast<const u32x4*>((const uint16_t*)q.ptr + b * q.sb + (int64_t)i * q.ss + (int64_t)h * q.sh + d);
    const int64_t off_o = b * o.sb + (int64_t)i * o.ss + (int64_t)h * o.sh + d;
    float y[8];
    if (kOBf16) {
      const uint4 u = *reinterpret_cast<const uint4*>((const uint16_t*)o.ptr + off_o);
      y[0] = bf16_lo(u.x); y[1] = bf16_hi(u.x); y[2] = bf16_lo(u.y); y[3] = bf16_hi(u.y);
      y[4] = bf16_lo(u.z); y[5] = bf16_hi(u.z); y[6] = bf16_lo(u.w); y[7] = bf16_hi(u.w);
    } else {
      const float4 u0 = *reinterpret_cast<const float4*>((const float*)o.ptr + off_o);
      const float4 u1 = *reinterpret_cast<const float4*>((const float*)o.ptr + off_o + 4);
      y[0] = u0.x; y[1] = u0.y; y[2] = u0.z; y[3] = u0.w; y[4] = u1.x; y[5] = u1.y; y[6] = u1.z; y[7] = u1.w;
    }
    qs[v] = scale_bf16x8(z, c);
    acc = fmaf(bf16_lo(x.x), y[0], acc); acc = fmaf(bf16_hi(x.x), y[1], acc);
    acc = fmaf(bf16_lo(x.y), y[2], acc); acc = fmaf(bf16_hi(x.y), y[3], acc);
    acc = fmaf(bf16_lo(x.z), y[4], acc); acc = fmaf(bf16_hi(x.z), y[5], acc);
    acc = fmaf(bf16_lo(x.w), y[6], acc); acc = fmaf(bf16_hi(x.w), y[7], acc);
  }
#pragma unroll
  for (int s = LPR / 2; s > 0; s >>= 1) acc += __shfl_xor(acc, s);
  if (live && d == 0) delta[(b * Hq + h) * Sq + i] = acc;
}

__global__ __launch_bounds__(256) void cast_bf16_kernel(const float4* __restrict__ src, uint2* __restrict__ dst,
                                                        int64_t n_vec, const float* __restrict__ src_tail,
                                                        uint16_t* __restrict__ dst_tail, int tail) {
  const int64_t v = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (v < n_vec) {
    const float4 x = src[v];
    dst[v] = make_uint2(pack_bf16x2(x.x, x.y), pack_bf16x2(x.z, x.w));
  } else if (v - n_vec < tail) {
    dst_tail[v - n_vec] = (uint16_t)f32_to_bf16_rne(src_tail[v - n_vec]);
  }
}

// ---- Q' = bf16(Q * c): thread = 8 elements (16 bytes) of one (b, i, h) row; dense output -----------------
__global__ __launch_bounds__(256) void scale_q_kernel(View q, u32x4* __restrict__ dst, int32_t B, int32_t Sq,
                                                      int32_t Hq, int32_t D, float c) {
  const int64_t v = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int32_t per_row = D / 8;
  const int64_t n_rows = (int64_t)B * Sq * Hq;
  if (v >= n_rows * per_row) return;
  const int64_t row = n_rows * per_row <= 0x7fffffff ? (int64_t)((uint32_t)v / (uint32_t)per_row) : v / per_row;
  const int32_t chunk = (int32_t)(v - row * per_row);
  const RowOf at = row_of(row, n_rows, Sq, Hq);
  const int64_t off = at.b * q.sb + at.i * q.ss + at.h * q.sh + chunk * 8;
  dst[v] = scale_bf16x8(*reinterpret_cast<const u32x4*>((const uint16_t*)q.ptr + off), c);
}

// Partial sums of an under-filled launch: bytes only, (sums + 2) x 4 per element.  blockIdx.y is a query tile of a batch
// entry, whose rows are one run of memory in dq and in each sum.  Eight loads of a thread are in flight together; the order of
// the additions is fixed.
__global__ __launch_bounds__(256) void add_parts_kernel(float* dq, float* sums, Shape s, QueryTiles tiles, TileShares shares, int n_qt) {
  const int b = blockIdx.y / n_qt, qt = blockIdx.y % n_qt, n = shares_of(shares, qt) - shares.own0;
  if (n + shares.own0 <= 1) return;
  const int64_t n_vec = (int64_t)tiles.rows_of(qt) * s.Hq * s.D / 4, v = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (v >= n_vec) return;
  const float4* parts = reinterpret_cast<const float4*>(dq_part(sums, s, tiles, shares, b, qt, 0)) + v;
  float4* dst = reinterpret_cast<float4*>(dq + ((int64_t)b * s.Sq + tiles.row0(qt)) * s.Hq * s.D) + v;
  float4 x = *dst;
  for (int y0 = 0; y0 < n; y0 += 8) {
    float4 p[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) p[u] = parts[min(y0 + u, n - 1) * n_vec];
#pragma unroll
    for (int u = 0; u < 8; ++u)
      if (y0 + u < n) {
        x.x += p[u].x;
        x.y += p[u].y;
        x.z += p[u].z;
        x.w += p[u].w;
      }
  }
  *dst = x;
}

// The same for key tiles: blockIdx.y is a key tile of the table (kt fastest), blockIdx.z a head (kv_job's hb), the first half of
// the blocks in x dK and the other half dV.
__global__ __launch_bounds__(256) void add_kv_parts_kernel(const BwdArgs a) {
  const Shape& s = a.s;
  const int n_kt = (s.Sk + kDkvFastKeys - 1) / kDkvFastKeys, tile = blockIdx.y, c = tile / n_kt, kt = tile - c * n_kt;
  KvPlace place;
  if (a.kv_same > 0) {
    place.n_share = a.kv_same;
    place.slot = tile * (a.kv_same - 1);
  } else {
    place = kv_place(s, a.kv_sec, a.kv_each, n_kt, tile, true, threadIdx.x & 63, [&](int x) { return a.t.k_offset[x]; });
  }
  const int n = (int)sgpr(place.n_share), slot = blockIdx.z * (a.kv_items - n_kt * a.t.n) + (int)sgpr(place.slot);
  if (n <= 1) return;
  const int vec = s.D / 4, half = gridDim.x / 2, w = (int)blockIdx.x >= half, v = (blockIdx.x - w * half) * 256 + threadIdx.x, row = v / vec;
  if (row >= min(kDkvFastKeys, s.Sk - kt * kDkvFastKeys)) return;
  const int hk = blockIdx.z / s.B, b = blockIdx.z % s.B;
  const int64_t at = ((((int64_t)b * s.Sk + kt * kDkvFastKeys + row) * s.Hkv + hk) * s.D) / 4 + v % vec, slot_vec = kv_slot_floats(s) / 4;
  const float4* parts = reinterpret_cast<const float4*>(a.kv_parts) + slot * slot_vec + w * kDkvFastKeys * vec + v;
  float4* dst = reinterpret_cast<float4*>(w ? a.dv[c] : a.dk[c]) + at;
  float4 x = *dst;
  // eight loads in flight together, and no load twice: n is the same for the workgroup
  int y0 = 0;
  auto some = [&](auto count) {
    constexpr int N = decltype(count)::value;
    float4 p[N];
#pragma unroll
    for (int u = 0; u < N; ++u) p[u] = parts[(y0 + u) * slot_vec];
#pragma unroll
    for (int u = 0; u < N; ++u) {
      x.x += p[u].x;
      x.y += p[u].y;
      x.z += p[u].z;
      x.w += p[u].w;
    }
    y0 += N;
  };
  using std::integral_constant;
  while (n - 1 - y0 >= 8) some(integral_constant<int, 8>());
  switch (n - 1 - y0) {
    case 7: some(integral_constant<int, 7>()); break;
    case 6: some(integral_constant<int, 6>()); break;
    case 5: some(integral_constant<int, 5>()); break;
    case 4: some(integral_constant<int, 4>()); break;
    case 3: some(integral_constant<int, 3>()); break;
    case 2: some(integral_constant<int, 2>()); break;
    case 1: some(integral_constant<int, 1>()); break;
  }
  *dst = x;
  uint2* low = reinterpret_cast<uint2*>(w ? a.dv_lowp[c] : a.dk_lowp[c]);
  if (low) low[at] = make_uint2(pack_bf16x2(x.x, x.y), pack_bf16x2(x.z, x.w));
}

// fp32 key tiles: blockIdx.y is a chunk, dK and then dV.  Keys that no row sees have no sums.
__global__ __launch_bounds__(256) void add_kv_parts_f32_kernel(const BwdArgs a, int64_t n_vec) {
  const Shape& s = a.s;
  const int64_t v = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int c = blockIdx.y >> 1, w = blockIdx.y & 1, n = a.kv_items;
  if (v >= n_vec) return;
  const int64_t row = v / (s.Hkv * s.D / 4);
  if (s.causal && q_row_of(s, a.t.k_offset[c] + row % s.Sk) >= s.Sq) return;
  float4* dst = reinterpret_cast<float4*>(w ? a.dv[c] : a.dk[c]) + v;
  float4 x = *dst;
  for (int y0 = 1; y0 < n; y0 += 4) {
    float4 p[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) p[u] = reinterpret_cast<const float4*>(f32_kv_part(a.kv_parts, s, a.t.n, min(y0 + u, n - 1), c, w))[v];
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (y0 + u < n) {
        x.x += p[u].x;
        x.y += p[u].y;
        x.z += p[u].z;
        x.w += p[u].w;
      }
  }
  *dst = x;
}

__global__ __launch_bounds__(256) void fill_state_kernel(float* __restrict__ o, float* __restrict__ lse,
                                                         int64_t n_o, int64_t n_lse) {
  const int64_t v = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (v < n_o) o[v] = 0.f;
  if (v < n_lse) lse[v] = -INFINITY;
}

// blockIdx.y: a chunk, dK and then dV.  One launch instead of two fills and two casts per chunk: 2 heads x 832 rows, three hidden
// chunks, 91 us of them in a pass of 114.
__global__ __launch_bounds__(256) void hidden_kv_kernel(const KvTables t, int assign, int64_t n_vec) {
  const int64_t v = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int c = blockIdx.y >> 1, w = blockIdx.y & 1;
  if (v >= n_vec) return;
  float4* dst = reinterpret_cast<float4*>(w ? t.dv[c] : t.dk[c]) + v;
  float4 x = make_float4(0.f, 0.f, 0.f, 0.f);
  if (assign) *dst = x;
  else x = *dst;
  uint2* low = reinterpret_cast<uint2*>(w ? t.dv_lowp[c] : t.dk_lowp[c]);
  if (low) low[v] = make_uint2(pack_bf16x2(x.x, x.y), pack_bf16x2(x.z, x.w));
}

// n dwords to zero, four per lane (the tail lane by lane)
__global__ __launch_bounds__(256) void zero_kernel(uint32_t* __restrict__ dst, int64_t n) {
  const int64_t v = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 4;
  if (v + 4 <= n && (reinterpret_cast<uintptr_t>(dst) & 15) == 0) {
    *reinterpret_cast<uint4*>(dst + v) = make_uint4(0u, 0u, 0u, 0u);
  } else {
    for (int64_t i = v; i < n && i < v + 4; ++i) dst[i] = 0u;
  }
}

inline unsigned blocks_for(int64_t n) { return (unsigned)((n + 255) / 256); }

// In launches of at most 2^30 vectors: a dimension of a grid holds fewer than 2^32 threads, and one that is wider loses the rest
// without an error.
hipError_t copy_f32(const float* src, float* dst, int64_t n, hipStream_t s) {
  constexpr int64_t kMost = (int64_t)1 << 32;
  for (int64_t at = 0; at < n; at += kMost) {
    const int64_t here = n - at < kMost ? n - at : kMost;
    hipLaunchKernelGGL(copy_f32_kernel, dim3(blocks_for((here + 3) / 4)), dim3(256), 0, s, (const float4*)(src + at), (float4*)(dst + at), here);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace

hipError_t launch_merge(float* o_acc, float* lse_acc, const float* o_part, const float* lse_part, int32_t B,
                        int32_t Sq, int32_t Hq, int32_t D, void* o_lowp, int lowp_dtype, hipStream_t s) {
  const int64_t n_rows = (int64_t)B * Sq * Hq;
  const int64_t n_vec = n_rows * (D / 4);
  if (n_vec == 0) return hipSuccess;
  // lanes per row and vectors per lane: eight lanes where the row has that many vectors (a group then reads whole
  // 128-byte lines), up to four vectors each, more lanes for the longest rows (D <= 256: at most 16)
  const int vec = D / 4;
  int lane_shift = 0;
  while ((1 << lane_shift) < 8 && (1 << lane_shift) < vec) ++lane_shift;
  while ((4 << lane_shift) < vec) ++lane_shift;
  const int per_lane = (vec + (1 << lane_shift) - 1) >> lane_shift;      // 1 .. 4
  const unsigned blocks = blocks_for(n_rows << lane_shift);
  const bool lowp = o_lowp != nullptr && lowp_dtype == ST_BF16;
  ProfScope prof("merge", s);
#define ST_LAUNCH_MERGE(LOWP, U)                                                                                    \
  hipLaunchKernelGGL((merge_kernel<LOWP, U>), dim3(blocks), dim3(256), 0, s, o_acc, lse_acc, o_part, lse_part, n_rows, \
                     Sq, Hq, vec, lane_shift, (uint2*)(LOWP ? o_lowp : nullptr))
  if (lowp) {
    if (per_lane == 1) ST_LAUNCH_MERGE(true, 1);
    else if (per_lane == 2) ST_LAUNCH_MERGE(true, 2);
    else ST_LAUNCH_MERGE(true, 4);
    return hipGetLastError();
  }
  if (per_lane == 1) ST_LAUNCH_MERGE(false, 1);
  else if (per_lane == 2) ST_LAUNCH_MERGE(false, 2);
  else ST_LAUNCH_MERGE(false, 4);
#undef ST_LAUNCH_MERGE
  hipError_t e = hipGetLastError();
  if (e == hipSuccess && o_lowp != nullptr) e = copy_f32(o_acc, (float*)o_lowp, 4 * n_vec, s);
  return e;
}

hipError_t launch_combine(const CombineArgs& a, int lowp_dtype, hipStream_t s) {
  const int64_t n_rows = (int64_t)a.B * a.Sq_out * a.Hq;
  const int64_t n_vec = n_rows * (a.D / 4);
  if (n_vec == 0) return hipSuccess;
  int lane_shift = 0;
  while ((1 << lane_shift) < a.D / 4) ++lane_shift;
  const dim3 grid(blocks_for(n_rows << lane_shift)), block(256);
  const bool lowp = a.o_lowp != nullptr && lowp_dtype == ST_BF16;
  ProfScope prof("combine", s);
#define ST_LAUNCH_COMBINE(LOWP, FEW)                                                                                         \
  if (a.shares.n > 1 && a.shares.total > 0)                                                                                 \
    hipLaunchKernelGGL((combine_kernel<LOWP, FEW, (FEW > 0)>), grid, block, 0, s, a, a.D / 4, lane_shift);                   \
  else                                                                                                                      \
    hipLaunchKernelGGL((combine_kernel<LOWP, FEW>), grid, block, 0, s, a, a.D / 4, lane_shift)
  if (a.n <= 4) {
    if (lowp) {
      ST_LAUNCH_COMBINE(true, 4);
    } else {
      ST_LAUNCH_COMBINE(false, 4);
    }
  } else if (a.n <= 8) {
    if (lowp) {
      ST_LAUNCH_COMBINE(true, 8);
    } else {
      ST_LAUNCH_COMBINE(false, 8);
    }
  } else if (a.n <= 16) {                              // the most shares a tile can have
    if (lowp) {
      ST_LAUNCH_COMBINE(true, 16);
    } else {
      ST_LAUNCH_COMBINE(false, 16);
    }
  } else {
    if (lowp) {
      ST_LAUNCH_COMBINE(true, 0);
    } else {
      ST_LAUNCH_COMBINE(false, 0);
    }
  }
#undef ST_LAUNCH_COMBINE
  hipError_t e = hipGetLastError();
  if (e == hipSuccess && a.o_lowp != nullptr && !lowp) e = copy_f32(a.o_out, (float*)a.o_lowp, 4 * n_vec, s);
  return e;
}

hipError_t launch_delta(const View& d_o, int d_o_dtype, const View& o, int o_dtype, float* delta, int32_t B,
                        int32_t Sq, int32_t Hq, int32_t D, hipStream_t s) {
  const int64_t n_rows = (int64_t)B * Sq * Hq;
  if (n_rows == 0) return hipSuccess;
  const dim3 grid(blocks_for(n_rows * 16)), block(256);
  const bool db = d_o_dtype == ST_BF16, ob = o_dtype == ST_BF16;
  ProfScope prof("delta", s);
  if (db && ob) hipLaunchKernelGGL((delta_kernel<true, true>), grid, block, 0, s, d_o, o, delta, B, Sq, Hq, D);
  else if (db) hipLaunchKernelGGL((delta_kernel<true, false>), grid, block, 0, s, d_o, o, delta, B, Sq, Hq, D);
  else if (ob) hipLaunchKernelGGL((delta_kernel<false, true>), grid, block, 0, s, d_o, o, delta, B, Sq, Hq, D);
  else hipLaunchKernelGGL((delta_kernel<false, false>), grid, block, 0, s, d_o, o, delta, B, Sq, Hq, D);
  return hipGetLastError();
}

OneReset one_reset(void* room, const Shape& s, int n_chunks, int heads) {
  const OneRoom r(s, n_chunks, heads);
  return OneReset{(uint4*)room, (int32_t)(r.pairs / 16), (int32_t)(r.plenty / 16)};
}
hipError_t launch_one_reset(const OneReset& r, hipStream_t s) {
  ProfScope prof("one_reset", s);
  hipLaunchKernelGGL(one_reset_kernel, dim3((unsigned)((r.n + 255) / 256)), dim3(256), 0, s, r);
  return hipGetLastError();
}

hipError_t launch_bwd_prep(const View& d_o, const View& o, int o_dtype, const View& q, float* delta, void* qs, int32_t* queue,
                           const OneReset& reset, int32_t B, int32_t Sq, int32_t Hq, int32_t D, float scale, hipStream_t s) {
  const int64_t n_vec = (int64_t)B * Sq * Hq * (D / 8);
  if (n_vec == 0) return hipSuccess;
  const dim3 grid(blocks_for(n_vec)), block(256);
  const float c = scale * 1.4426950408889634f;
  ProfScope prof("bwd_prep", s);
#define ST_LAUNCH_PREP(OB, LPR) \
  hipLaunchKernelGGL((bwd_prep_kernel<OB, LPR>), grid, block, 0, s, d_o, o, q, delta, (u32x4*)qs, queue, reset, B, Sq, Hq, c)
  if (D == 128) {
    if (o_dtype == ST_BF16) ST_LAUNCH_PREP(true, 16);
    else ST_LAUNCH_PREP(false, 16);
  } else if (D == 64) {
    if (o_dtype == ST_BF16) ST_LAUNCH_PREP(true, 8);
    else ST_LAUNCH_PREP(false, 8);
  } else {
    return hipErrorInvalidValue;
  }
#undef ST_LAUNCH_PREP
  return hipGetLastError();
}

hipError_t launch_cast(const float* src, void* dst, int64_t n, int dst_dtype, hipStream_t s) {
  if (n == 0) return hipSuccess;
  const int64_t n_vec = n / 4;
  const int tail = (int)(n - n_vec * 4);
  ProfScope prof("cast", s);
  if (dst_dtype == ST_F32) return copy_f32(src, (float*)dst, n, s);      // as a copy of the runtime it held the stream for 5 us more
  hipLaunchKernelGGL(cast_bf16_kernel, dim3(blocks_for(n_vec + tail)), dim3(256), 0, s, (const float4*)src,
                     (uint2*)dst, n_vec, src + n_vec * 4, (uint16_t*)dst + n_vec * 4, tail);
  return hipGetLastError();
}

hipError_t launch_scale_q(const View& q, void* dst, int32_t B, int32_t Sq, int32_t Hq, int32_t D, float scale,
                          hipStream_t s) {
  const int64_t n_vec = (int64_t)B * Sq * Hq * (D / 8);
  if (n_vec == 0) return hipSuccess;
  ProfScope prof("scale_q", s);
  hipLaunchKernelGGL(scale_q_kernel, dim3(blocks_for(n_vec)), dim3(256), 0, s, q, (u32x4*)dst, B, Sq, Hq, D,
                     scale * 1.4426950408889634f);
  return hipGetLastError();
}

hipError_t launch_zero(void* dst, int64_t bytes, hipStream_t s) {
  if (bytes <= 0) return hipSuccess;
  const int64_t n = bytes / 4;
  ProfScope prof("zero", s);
  hipLaunchKernelGGL(zero_kernel, dim3(blocks_for((n + 3) / 4)), dim3(256), 0, s, (uint32_t*)dst, n);
  return hipGetLastError();
}

hipError_t launch_add_parts(const BwdArgs& a, int rows, hipStream_t s) {
  const QueryTiles tiles = query_tiles(a.s, rows);
  const int n_qt = tiles.count();
  if (n_qt <= 0 || a.s.B <= 0) return hipSuccess;
  if ((int64_t)n_qt * a.s.B > 65535) return hipErrorInvalidValue;     // split launches have fewer than 512 tiles
  ProfScope prof("add_parts", s);
  hipLaunchKernelGGL(add_parts_kernel, dim3(blocks_for((int64_t)min(rows, a.s.Sq) * a.s.Hq * a.s.D / 4), n_qt * a.s.B), dim3(256), 0, s, a.dq, a.parts, a.s, tiles, a.shares, n_qt);
  return hipGetLastError();
}

hipError_t launch_add_kv_parts(const BwdArgs& a_in, hipStream_t s) {
  BwdArgs a = a_in;
  kv_sections(a);
  const int tiles = (a.s.Sk + kDkvFastKeys - 1) / kDkvFastKeys * a.t.n, heads = a.s.Hkv * a.s.B;
  if (tiles <= 0 || heads <= 0) return hipSuccess;
  if (tiles > 65535 || heads > 65535) return hipErrorInvalidValue;    // split launches have fewer than 512 tiles that see rows
  ProfScope prof("add_kv_parts", s);
  hipLaunchKernelGGL(add_kv_parts_kernel, dim3(2 * blocks_for(kDkvFastKeys * a.s.D / 4), tiles, heads), dim3(256), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_add_kv_parts_f32(const BwdArgs& a, hipStream_t s) {
  const int64_t n_vec = (int64_t)a.s.B * a.s.Sk * a.s.Hkv * a.s.D / 4;
  if (n_vec <= 0 || a.t.n <= 0) return hipSuccess;
  ProfScope prof("add_kv_parts", s);
  hipLaunchKernelGGL(add_kv_parts_f32_kernel, dim3(blocks_for(n_vec), 2 * a.t.n), dim3(256), 0, s, a, n_vec);
  return hipGetLastError();
}

hipError_t launch_hidden_kv(const KvTables& t, int n, bool assign, int64_t n_kv, hipStream_t s) {
  if (n <= 0 || n_kv <= 0) return hipSuccess;
  ProfScope prof("hidden_kv", s);
  hipLaunchKernelGGL(hidden_kv_kernel, dim3(blocks_for(n_kv / 4), 2 * n), dim3(256), 0, s, t, assign ? 1 : 0, n_kv / 4);   // D % 8 == 0
  return hipGetLastError();
}

hipError_t launch_fill_state(float* o, float* lse, int64_t n_o, int64_t n_lse, hipStream_t s) {
  const int64_t n = n_o > n_lse ? n_o : n_lse;
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(fill_state_kernel, dim3(blocks_for(n)), dim3(256), 0, s, o, lse, n_o, n_lse);
  return hipGetLastError();
}

}  // namespace st
