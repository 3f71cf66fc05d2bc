// C-ABI layer: argument validation, dtype dispatch, the visit-order generator and the
// driver that walks a chunk-visit order.  No arithmetic of the method lives here; every
// step of the path runs in the HIP kernels behind the launch_* functions.
#include <algorithm>
#include <cstdarg>
#include <cstdio>
#include <cstring>

#include <mutex>
#include <vector>

#include "st_internal.h"
#include "st_testing.h"

namespace {

// ---- event profiler state ----
struct ProfRec {
  const char* name;
  hipEvent_t start, stop;
};
std::mutex g_prof_mu;
bool g_prof_on = false;
std::vector<ProfRec> g_prof;
constexpr size_t kProfMax = 4096;

thread_local char g_err[512] = "";

// ---- scratch of st_ring_bwd_noalloc: device memory every loaded GPU holds until the process ends ----
// In host code the array's name is only a handle: its device address differs from GPU to GPU and is looked up
// once per device with hipGetSymbolAddress (scratch_of_current_device); kernels only ever see that pointer.
// Partial sums of under-filled launches have an array of their own, as large as such a backward ever uses (kRoomMost): what a
// call gets beside it must not depend on how much of the 40 MiB its Delta and Q' leave.
constexpr size_t kScratchBytes = (size_t)40 << 20, kPartsMost = (size_t)64 << 20;
// What a ring backward ever uses beside its Delta and Q' (the sums of a walk of one, OneRoom, or partial sums, at most kPartsMost):
// shares that st_ring_bwd_noalloc takes, and larger ones (see room_most): backward of 32/8 heads x 16384 rows x 3 chunks in one walk 22.7
// ms, in two passes 26.4; 8 heads x 32768 x 2 14.1, 15.7.
constexpr size_t kRoomMost = (size_t)96 << 20, kRoomMostLarge = (size_t)320 << 20;
static __device__ __align__(256) unsigned char scratch[kScratchBytes];
static __device__ __align__(256) unsigned char scratch_parts[kRoomMost];
constexpr int kScratchDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kScratchDevices][2];

st_status fail(st_status s, const char* fmt, ...) {
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(g_err, sizeof(g_err), fmt, ap);
  va_end(ap);
  return s;
}

st_status hip_fail(hipError_t e, const char* what) {
  return fail(ST_ERR_HIP, "%s: %s", what, hipGetErrorString(e));
}

// Device addresses of `scratch` and `scratch_parts` on the current device (looked up on the first call per device, then cached).
st_status scratch_of_current_device(void** out, void** parts) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return hip_fail(e, "hipGetDevice");
  if (dev < 0 || dev >= kScratchDevices) return fail(ST_ERR_UNSUPPORTED, "device index %d beyond %d", dev, kScratchDevices - 1);
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  if (g_scratch_ptr[dev][0] == nullptr) {
    void *p = nullptr, *q = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e == hipSuccess) e = hipGetSymbolAddress(&q, HIP_SYMBOL(scratch_parts));
    if (e != hipSuccess) return hip_fail(e, "hipGetSymbolAddress(scratch)");
    for (void* x : {p, q})
      if (x == nullptr || reinterpret_cast<uintptr_t>(x) % 256) return fail(ST_ERR_HIP, "scratch symbol has no aligned device address");
    g_scratch_ptr[dev][0] = p;
    g_scratch_ptr[dev][1] = q;
  }
  *out = g_scratch_ptr[dev][0];
  *parts = g_scratch_ptr[dev][1];
  return ST_OK;
}

inline size_t elem_size(int dtype) { return dtype == ST_BF16 ? 2 : 4; }
inline size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

st_status check_scale(float scale) {
  if (!(scale > 0.f) || scale > 3.0e38f) return fail(ST_ERR_INVALID_ARG, "scale must be finite and positive");
  return ST_OK;
}

st_status check_shape(int dtype, int B, int Hq, int Hkv, int D, int Sq, int Sk) {
  if (dtype != ST_F32 && dtype != ST_BF16) return fail(ST_ERR_INVALID_ARG, "unknown dtype %d", dtype);
  if (B < 0 || Sq < 0 || Sk < 0) return fail(ST_ERR_INVALID_ARG, "negative size");
  if (Hq <= 0 || Hkv <= 0 || Hq % Hkv != 0) return fail(ST_ERR_INVALID_ARG, "need Hq %% Hkv == 0 (Hq=%d Hkv=%d)", Hq, Hkv);
  if (D <= 0) return fail(ST_ERR_INVALID_ARG, "D must be positive");
  if (dtype == ST_F32 && (D > 256 || D % 8 != 0)) return fail(ST_ERR_UNSUPPORTED, "fp32 path needs D <= 256 and D %% 8 == 0 (D=%d)", D);
  if (dtype == ST_BF16 && D != 128 && D != 64) return fail(ST_ERR_UNSUPPORTED, "bf16 path is built for D = 64 or 128 (D=%d)", D);
  if (B > 65535 || Hq > 65535) return fail(ST_ERR_UNSUPPORTED, "B and Hq must not exceed 65535");
  return ST_OK;
}

// a [B,S,heads,D] view whose rows must be 16-byte aligned
st_status check_view(const char* name, const void* ptr, int64_t sb, int64_t ss, int64_t sh, int dtype,
                     int64_t n_elems) {
  if (n_elems == 0) return ST_OK;
  if (ptr == nullptr) return fail(ST_ERR_INVALID_ARG, "%s: null pointer", name);
  const int64_t per16 = 16 / (int64_t)elem_size(dtype);
  if (reinterpret_cast<uintptr_t>(ptr) % 16 != 0) return fail(ST_ERR_ALIGNMENT, "%s: base pointer is not 16-byte aligned", name);
  if (sb % per16 || ss % per16 || sh % per16) return fail(ST_ERR_ALIGNMENT, "%s: strides must be multiples of %lld elements", name, (long long)per16);
  if (sb < 0 || ss < 0 || sh < 0) return fail(ST_ERR_INVALID_ARG, "%s: negative stride", name);
  return ST_OK;
}

st_status check_tensor(const char* name, const st_tensor* t, int dtype, int64_t n_elems) {
  if (t == nullptr) return fail(ST_ERR_INVALID_ARG, "%s: null st_tensor", name);
  return check_view(name, t->ptr, t->stride_b, t->stride_s, t->stride_h, dtype, n_elems);
}

st_status check_f32(const char* name, const void* p, int64_t n_elems) {
  if (n_elems == 0) return ST_OK;
  if (p == nullptr) return fail(ST_ERR_INVALID_ARG, "%s: null pointer", name);
  if (reinterpret_cast<uintptr_t>(p) % 16 != 0) return fail(ST_ERR_ALIGNMENT, "%s: not 16-byte aligned", name);
  return ST_OK;
}

st::View view_of(const st_tensor* t) { return st::View{t->ptr, t->stride_b, t->stride_s, t->stride_h}; }

st::Shape shape_of(const st_block_desc* d) {
  return st::Shape{d->B, d->Hq, d->Hkv, d->D, d->Sq, d->Sk, d->q_offset, d->causal ? 1 : 0, d->scale, d->q_seg, d->q_offset2};
}
st::Shape shape_of(const st_ring_desc* d) {
  return st::Shape{d->B, d->Hq, d->Hkv, d->D, d->Sq, d->Sk, d->q_offset, d->causal ? 1 : 0, d->scale, d->q_seg, d->q_offset2};
}

// two runs of query rows: the second must not start before the first ends (positions rise with the row index)
st_status check_segments(int32_t Sq, int64_t q_offset, int32_t q_seg, int64_t q_offset2) {
  if (q_seg == 0) return ST_OK;
  if (q_seg < 0 || q_seg >= Sq) return fail(ST_ERR_INVALID_ARG, "q_seg = %d must be 0 or inside the %d query rows", q_seg, Sq);
  if (q_offset2 < q_offset + q_seg) return fail(ST_ERR_INVALID_ARG, "second run of query rows starts before the first ends");
  return ST_OK;
}

#define ST_TRY(expr)                  \
  do {                                \
    st_status _s = (expr);            \
    if (_s != ST_OK) return _s;       \
  } while (0)
#define ST_HIP(expr, what)                        \
  do {                                            \
    hipError_t _e = (expr);                       \
    if (_e != hipSuccess) return hip_fail(_e, what); \
  } while (0)

hipError_t launch_fwd(int dtype, const st::FwdArgs& a, hipStream_t s) {
  return dtype == ST_BF16 ? st::launch_fwd_bf16(a, s) : st::launch_fwd_f32(a, s);
}
hipError_t launch_bwd(int dtype, const st::BwdArgs& a, hipStream_t s) {
  return dtype == ST_BF16 ? st::launch_bwd_bf16(a, s) : st::launch_bwd_f32(a, s);
}

// chunk lies entirely in the causal future of the shard: nothing to compute
inline bool chunk_invisible(const st_ring_desc* d, int j) {
  return d->Sk == 0 || (d->causal && d->k_offset[j] > st::q_pos(shape_of(d), d->Sq - 1));
}

st_status check_ring(const st_ring_desc* d, const st_tensor* q, const int32_t* order, int32_t n_visit) {
  if (d == nullptr) return fail(ST_ERR_INVALID_ARG, "null descriptor");
  ST_TRY(check_shape(d->dtype, d->B, d->Hq, d->Hkv, d->D, d->Sq, d->Sk));
  ST_TRY(check_scale(d->scale));
  ST_TRY(check_segments(d->Sq, d->q_offset, d->q_seg, d->q_offset2));
  if (d->n_chunks < 1 || d->n_chunks > ST_MAX_CHUNKS) return fail(ST_ERR_INVALID_ARG, "n_chunks must be in 1..%d", ST_MAX_CHUNKS);
  if (!d->k_ptr || !d->v_ptr || !d->k_offset) return fail(ST_ERR_INVALID_ARG, "null chunk table");
  if (n_visit < 0 || n_visit > d->n_chunks) return fail(ST_ERR_INVALID_ARG, "n_visit out of range");
  if (n_visit > 0 && order == nullptr) return fail(ST_ERR_INVALID_ARG, "null visit order");
  const int64_t n_kv = (int64_t)d->B * d->Sk * d->Hkv * d->D;
  bool seen[ST_MAX_CHUNKS] = {false};
  for (int x = 0; x < n_visit; ++x) {
    const int j = order[x];
    if (j < 0 || j >= d->n_chunks) return fail(ST_ERR_INVALID_ARG, "order[%d] = %d is not a chunk index", x, j);
    if (seen[j]) return fail(ST_ERR_INVALID_ARG, "chunk %d is visited twice", j);
    seen[j] = true;
    ST_TRY(check_view("k chunk", d->k_ptr[j], d->k_stride_b, d->k_stride_s, d->k_stride_h, d->dtype, n_kv));
    ST_TRY(check_view("v chunk", d->v_ptr[j], d->v_stride_b, d->v_stride_s, d->v_stride_h, d->dtype, n_kv));
  }
  return check_tensor("q", q, d->dtype, (int64_t)d->B * d->Sq * d->Hq * d->D);
}

constexpr int kMaxSplits = 16;
constexpr int kPlanCus = 256;

// fp32: the turns a query tile's workgroup takes over n chunks; in one its wavefronts (eight, four beyond head size 128) take
// a 32-key tile each
int64_t f32_turns(int D, int Sk, int64_t n) {
  const int waves = D <= 128 ? 8 : 4;
  return (n * ((Sk + 31) / 32) + waves - 1) / waves;
}

// What the query tiles of a launch have to walk, in the units their kernels deal out: 64-key tiles in bf16, a masked one
// counted twice (see build_walk), and turns in fp32.
struct QueryWalk {
  int64_t heads = 0;     // B Hq
  st::QueryTiles q = {};
  int tiles = 0;         // per head
  int n = 0;             // entries of units: one per tile, or a single one where all tiles have the same
  int units[st::kShareTiles];
  int64_t wgs() const { return heads * tiles; }
  int most() const { return *std::max_element(units, units + n); }
};
QueryWalk query_walk(const st::Shape& s, int dtype, const int64_t* k_offset, int n) {
  const bool bf16 = dtype == ST_BF16;
  QueryWalk w;
  w.q = st::query_tiles(s, bf16 ? st::kQTileFastRows : 32);
  w.tiles = w.q.count();
  w.heads = (int64_t)s.B * s.Hq;
  const bool apart = s.causal && k_offset && w.tiles >= 1 && w.tiles <= st::kShareTiles;
  w.n = apart ? w.tiles : 1;
  if (!apart) {
    w.units[0] = (int)std::min<int64_t>(bf16 ? (int64_t)n * ((s.Sk + st::kQTileFastKeys - 1) / st::kQTileFastKeys) : f32_turns(s.D, s.Sk, n), 1 << 28);
    return w;
  }
  const int n64 = s.Sk / st::kQTileFastKeys, waves = s.D <= 128 ? 8 : 4;
  for (int qt = 0; qt < w.tiles; ++qt) {
    const int64_t first = st::q_pos(s, w.q.row0(qt)), last = st::q_pos(s, w.q.row0(qt) + w.q.rows_of(qt) - 1);
    int64_t units = 0;
    for (int c = 0; c < n; ++c) {
      const int64_t nv_last = std::min<int64_t>(std::max<int64_t>(last - k_offset[c] + 1, 0), s.Sk);
      if (!bf16) {
        units += (nv_last + 31) / 32;
        continue;
      }
      const int64_t nf = std::min<int64_t>(std::max<int64_t>(first - k_offset[c] + 1, 0), s.Sk) / st::kQTileFastKeys;
      const int64_t seen = std::min<int64_t>((nv_last + st::kQTileFastKeys - 1) / st::kQTileFastKeys, n64);
      units += nf + 2 * (std::max<int64_t>(seen - nf, 0) + (nv_last > (int64_t)n64 * st::kQTileFastKeys));
    }
    w.units[qt] = (int)std::min<int64_t>(bf16 ? units : (units + waves - 1) / waves, 1 << 28);
  }
  return w;
}

// Time of a workgroup: what stands around its walk, and a unit of it.  Both grow with the workgroups that run beside it: they
// share the memory that results are written to, and the more of the chip works, the lower its clock.
struct Cost {
  double fixed_us, unit_us, fixed_full, unit_full;     // of one alone, and what is added on a full chip
  double us(double units, int64_t workgroups) const {
    const double f = (double)std::min<int64_t>(workgroups, kPlanCus) / kPlanCus;
    return fixed_us + f * fixed_full + units * (unit_us + f * unit_full);
  }
};
// Measured on 32 to 256 workgroups with walks of 4 to 128 units, kernels back to back.  Forward, a 256 x 64 tile; dQ, the same (three contractions
// instead of two); dK/dV, 256 keys x 32 rows of one head.  fp32: a turn (see f32_turns).
// The forward alone, launches of whole tiles in a graph, 1 / 64 / 128 / 192 / 256 workgroups: head size 128 4 tiles 15.3 / 16.7 / 19.4 / 21.8 / 24.2
// us, 16 tiles 26.8 / 29.8 / 33.0 / 36.3 / 42.9, 64 tiles 73 / 76 / 85 / 110 / 129; head size 64 16 tiles 19.2 / 20.5 / 22.8 / 24.4 / 27.5, 64 tiles
// 53 / 55 / 58 / 64 / 81; a masked tile is two.  In a share fewer workgroups cost somewhat more than that and splits somewhat less:
// constants that follow the table to the letter choose too few shares (100 under-filled shares 0.6 % slower than with these).
Cost fwd_cost(int dtype, int D) {
  if (dtype != ST_BF16) return Cost{5 + 0.035 * D, 2 + (D <= 128 ? 0.065 : 0.034) * D, 0, 0};
  return D == 128 ? Cost{13.5, 1.05, 2.5, 0.45} : Cost{9.5, 0.75, 1.5, 0.2};
}
Cost dq_cost(int dtype, int D) {
  if (dtype != ST_BF16) return Cost{10, 2 + (D <= 128 ? 0.11 : 0.055) * D, 0, 0};
  return D == 128 ? Cost{20, 1.45, 0, 0.35} : Cost{14, 0.95, 0, 0.25};
}
Cost dkv_cost(int D) { return D == 128 ? Cost{17, 0.9, 5, 0.25} : Cost{14, 0.68, 3, 0.2}; }

// Time of a launch of so many workgroups each: handed out in this order, each to the compute unit that is free first (one holds
// one).  Stops where it is beyond `most`.
struct Job {
  double us;
  int64_t n;
};
double jobs_us(const Job* job, int n, double most = 1e30) {
  struct Group { double us; int64_t n; };
  constexpr int kGroups = 64;
  Group cu[kGroups];                                  // free first, free last
  int groups = 1;
  cu[0] = Group{0, kPlanCus};
  double end = 0;
  for (int i = 0; i < n; ++i)
    for (int64_t left = job[i].n; left > 0;) {
      const int64_t take = std::min(left, cu[0].n);
      const double us = cu[0].us + job[i].us;
      end = std::max(end, us);
      if (end >= most) return end;
      left -= take;
      if (take == cu[0].n) std::copy(cu + 1, cu + groups--, cu);
      else cu[0].n -= take;
      int at = groups;
      while (at > 0 && cu[at - 1].us >= us) --at;
      if ((at < groups && cu[at].us < us + 0.5) || groups == kGroups) {
        cu[std::min(at, groups - 1)].n += take;       // as good as at the same time
        continue;
      }
      std::copy_backward(cu + at, cu + groups, cu + groups + 1);
      cu[at] = Group{us, take};
      ++groups;
    }
  return end;
}

// A way to split the tiles of a walk into shares of at most `each` units.
struct Split {
  const QueryWalk* w;
  int each;
  int n = 1;                    // most shares of a tile
  int total = 0;                // shares of a head
  int64_t rows = 0, rows_own0 = 0;   // rows of partial results per batch entry and head: all shares of split tiles, all but the first ones
  int shares(int i) const { return std::min(std::max((w->units[i] + each - 1) / each, 1), kMaxSplits); }
  Split(const QueryWalk& walk, int units) : w(&walk), each(std::max(units, 1)) {
    for (int i = 0; i < w->n; ++i) {
      const int x = shares(i), tiles = w->n == 1 ? w->tiles : 1;
      n = std::max(n, x);
      total += x * tiles;
      if (x == 1) continue;
      const int64_t rows_i = w->n == 1 ? w->q.Sq : w->q.rows_of(i);
      rows += x * rows_i;
      rows_own0 += (x - 1) * rows_i;
    }
  }
  int64_t workgroups() const { return w->heads * total; }
  int longest() const {         // units of the longest share
    int most = 0;
    for (int i = 0; i < w->n; ++i) most = std::max(most, (w->units[i] + shares(i) - 1) / shares(i));
    return most;
  }
  // its workgroups as jobs, longest first, beside `others`; returns their number
  int jobs(Job* to, const Cost& cost, int64_t others = 0) const {
    for (int i = 0; i < w->n; ++i)
      to[i] = Job{cost.us((w->units[i] + shares(i) - 1) / shares(i), others + workgroups()), w->heads * shares(i) * (w->n == 1 ? w->tiles : 1)};
    std::sort(to, to + w->n, [](const Job& x, const Job& y) { return x.us > y.us; });
    return w->n;
  }
  double longest_us(const Cost& cost, int64_t others = 0) const { return cost.us(longest(), others + workgroups()); }
  double launch_us(const Cost& cost) const {
    if (workgroups() <= kPlanCus) return longest_us(cost);
    Job job[st::kShareTiles];
    return jobs_us(job, jobs(job, cost));
  }
  st::TileShares table(bool own0) const {
    st::TileShares t;
    memset(&t, 0, sizeof(t));
    t.n = (int16_t)n;
    t.own0 = n > 1 && own0;
    bool same = true;
    for (int i = 1; i < w->n; ++i) same = same && shares(i) == shares(0);
    if (w->n == 1 || same) return t;
    t.total = (int16_t)total;
    for (int i = 0; i < w->n; ++i) t.less1[i >> 4] |= (uint64_t)(shares(i) - 1) << (4 * (i & 15));
    return t;
  }
};
// the passes that fold the shares have eight loads in flight; more are a second wait
double more_than_8_us(const Split& s) { return s.n > 8 ? 1.5 : 0; }
// f(split) for the splits that give the longest walk 2, 3, ... shares
template <typename F>
void each_split(const QueryWalk& w, int most, F f) {
  const int top = w.most();
  for (int k = 2, before = top; k <= most && k <= top; ++k) {
    const int each = (top + k - 1) / k;
    if (each == before) continue;
    before = each;
    const Split s(w, each);
    if (s.workgroups() > 8 * kPlanCus) return;
    f(s);
  }
}

// Workgroups per tile of a backward launch over n chunks, and the bytes of partial sums that
// takes (the two passes run one after the other and share them).
struct BwdSplit {
  st::TileShares dq = {};
  int kv_each = 0, kv_items = 0;
  bool pair = false;
  int one_heads = 0;
  size_t dq_bytes = 0, bytes = 0;
};
// dQ: the forward's model (the launch + the pass that adds up) with the constants of dq_cost.  fp32: the eight (four beyond head size 128) wavefronts of a workgroup take a
// 32-key tile each in 16 us at head size 128, 9 at 64, 5.5 at 32, and 16 at 256 (8 heads x 512 rows x 8 chunks of 512 keys at
// head size 128: 128 workgroups, 270 us; 157 us as two shares each and the adding pass); 10 us for the adding pass, as walks
// of two turns gain less than its launch takes.
// dK/dV: the key tiles that some row sees, by the query blocks they meet (under a causal mask the diagonal chunk's meet half of
// them, two runs of rows have chunks that only one run sees).  Few and long walks are split into shares of one size, so the
// launch does not wait for the longest; a tile that no row sees is written or skipped in 4 us.  24/3 heads x 1601 rows, first
// of two chunks: 21 tiles of up to 51 blocks x 8 heads, 130 us in equal numbers of shares and 61 of dQ; now 98 together.
// From 512 tiles on that some row sees, they go through the queue.
struct KeyWalk {
  int64_t heads = 0;     // B Hkv
  int tiles = 0;         // per head, over all chunks
  int G = 1, top = 0, seen = 0;     // heads per group, most blocks of a tile, tiles that meet some
  int n = 0;
  struct Class { int blocks, tiles; } c[512];   // tiles by the blocks they meet
};
void key_walk(KeyWalk& w, const st::Shape& s, const int64_t* k_offset, int n) {
  const int n_kt = (s.Sk + st::kDkvFastKeys - 1) / st::kDkvFastKeys, all = (s.Sq + st::kDkvFastRows - 1) / st::kDkvFastRows;
  w.heads = (int64_t)s.B * s.Hkv;
  w.tiles = n_kt * n;
  w.G = s.Hq / s.Hkv;
  w.n = 0;
  auto add = [&](int blocks, int tiles) {
    w.top = std::max(w.top, blocks);
    if (blocks > 0) w.seen += tiles;
    for (int i = 0; i < w.n; ++i)
      if (w.c[i].blocks == blocks) {
        w.c[i].tiles += tiles;
        return;
      }
    if (w.n < (int)(sizeof(w.c) / sizeof(w.c[0]))) w.c[w.n++] = KeyWalk::Class{blocks, tiles};
    else w.c[w.n - 1].tiles += tiles;
  };
  const int64_t first = st::q_pos(s, 0), last = st::q_pos(s, s.Sq - 1);
  for (int c = 0; c < n; ++c) {
    if (!s.causal || k_offset == nullptr || k_offset[c] + s.Sk - 1 <= first) add(all, n_kt);
    else if (k_offset[c] > last) add(0, n_kt);
    else
      for (int kt = 0; kt < n_kt; ++kt) add(st::kv_blocks(s, k_offset[c], kt), 1);
  }
  std::sort(w.c, w.c + w.n, [](const KeyWalk::Class& x, const KeyWalk::Class& y) { return x.blocks > y.blocks; });
}
// shares of at most `each` blocks (0: unsplit)
struct KeySplit {
  const KeyWalk* w;
  int each, longest = 0;        // blocks of the longest share
  int64_t items = 0, slots = 0, split_tiles = 0;   // of a head: shares, shares that store partial sums, tiles with some
  KeySplit(const KeyWalk& walk, int blocks) : w(&walk), each(blocks) {
    for (int i = 0; i < w->n; ++i) {
      const int x = st::kv_shares(w->c[i].blocks, each);
      items += (int64_t)x * w->c[i].tiles;
      slots += (int64_t)(x - 1) * w->c[i].tiles;
      if (x > 1) split_tiles += w->c[i].tiles;
      longest = std::max(longest, (w->c[i].blocks + x - 1) / x);
    }
  }
  int64_t workgroups() const { return w->heads * (items - (w->tiles - w->seen)); }       // that have something to do
  double longest_us(const Cost& cost, int64_t others = 0) const { return cost.us(longest * w->G, others + workgroups()); }
  int jobs(Job* to, const Cost& cost, int64_t others = 0) const {
    for (int i = 0; i < w->n; ++i) {
      const int x = st::kv_shares(w->c[i].blocks, each);
      to[i] = Job{w->c[i].blocks > 0 ? cost.us((w->c[i].blocks + x - 1) / x * w->G, others + workgroups()) : 4.0, w->heads * w->c[i].tiles * x};
    }
    return w->n;
  }
};
// fp32: both passes are always one launch.  A key tile is 32 keys, its wavefronts take a (head, 32-row tile) pair each in a turn of
// 23 us at head size 128, 12.6 at 64 and 21.5 at 256 (half the wavefronts), behind 15 us; dQ's are above.
void f32_bwd_split(BwdSplit& r, const st::Shape& s, const QueryWalk& walk, const int64_t* k_offset, int n, size_t room, bool split_dq) {
  const int n_kt = (s.Sk + 31) / 32, waves = s.D <= 128 ? 8 : 4, G = s.Hq / s.Hkv, rows = (s.Sq + 31) / 32;
  const Cost kv_cost{15, 3 + (s.D <= 128 ? 0.15 : 0.072) * s.D, 0, 0}, cost = dq_cost(ST_F32, s.D);
  // key tiles by the pairs they meet, at most 64 kinds
  struct Kind { int pairs; int64_t tiles; } kind[64];
  int kinds = 0;
  auto add = [&](int row_tiles, int64_t tiles) {
    const int pairs = row_tiles * G;
    for (int i = 0; i < kinds; ++i)
      if (kind[i].pairs == pairs || (kinds == 64 && i == 63)) {
        kind[i].tiles += tiles;
        return;
      }
    if (pairs > 0) kind[kinds++] = Kind{pairs, tiles};
  };
  const int64_t heads = (int64_t)s.B * s.Hkv, first = st::q_pos(s, 0);
  for (int c = 0; c < n; ++c) {
    if (!s.causal || k_offset == nullptr || k_offset[c] + s.Sk - 1 <= first) add(rows, heads * n_kt);
    else
      for (int kt = 0; kt < n_kt; ++kt) {
        const int row = st::q_row_of(s, k_offset[c] + kt * 32);
        add(row >= s.Sq ? 0 : rows - row / 32, heads);
      }
  }
  std::sort(kind, kind + kinds, [](const Kind& x, const Kind& y) { return x.pairs > y.pairs; });
  int64_t tiles = 0;
  for (int i = 0; i < kinds; ++i) tiles += kind[i].tiles;
  if (kinds == 0 || tiles >= 1024) return;
  const size_t kv_bytes = 2 * (size_t)n * st::f32_kv_floats(s) * sizeof(float), row_bytes = (size_t)s.B * s.Hq * s.D * sizeof(float);
  Job job[64 + st::kShareTiles];
  double best = 1e30;
  const BwdSplit none = {};
  auto look = [&](int x, const Split& q) {
    const size_t kv = (size_t)(x - 1) * kv_bytes;
    auto dq_bytes = [&](int64_t part_rows) { return q.n > 1 ? align_up((size_t)part_rows * row_bytes, 256) : 0; };
    if (kv + dq_bytes(q.rows_own0) > room) return;
    const double add = (x > 1 ? 7 + (double)kv_bytes * (x + 1) / 8e6 : 0) + (q.n > 1 ? 7 + (double)row_bytes * (q.rows + 2 * s.Sq) / 8e6 : 0);
    const double less = best < 1e30 ? (x > 1 || q.n > 1 ? 0.97 : 1) * best : best;
    for (int i = 0; i < kinds; ++i) job[i] = Job{kv_cost.us((kind[i].pairs + x * waves - 1) / (x * waves), 0), kind[i].tiles * x};
    if (job[0].us + add >= less || q.longest_us(cost) + add >= less) return;
    const double us = add + jobs_us(job, kinds + q.jobs(job + kinds, cost), less - add);
    if (us >= less) return;
    best = us;
    const bool own0 = kv + dq_bytes(q.rows) > room;
    r = none;
    r.dq = q.table(own0);
    r.dq_bytes = dq_bytes(own0 ? q.rows_own0 : q.rows);
    r.kv_items = x;
    r.pair = true;
    r.bytes = r.dq_bytes + kv;
  };
  const Split whole(walk, walk.most());
  for (int x = 1; x <= kMaxSplits && x <= (kind[0].pairs + waves - 1) / waves; x = x < 4 ? x + 1 : x + x / 2) {
    if (x > 1 && tiles * x > 4 * kPlanCus) break;
    look(x, whole);
    if (split_dq) each_split(walk, kMaxSplits, [&](const Split& q) { look(x, q); });
  }
}
// All three gradients in one walk over the key tiles (launch_bwd_one_fast), `batch` KV heads at a time on an XCD.  The XCD with the
// most batches sets the time: its 32 workgroups take the tiles in order, and a tile starts two blocks behind the one before.
// Measured (sums of a backward's launches, us; first the two passes, then one walk of batches of 1 / of all the heads of an XCD; last
// ranks of rings of 8): 8 heads x 1024 rows 129, 143; x 2048 389, 344; x 4096 1346, 1123; 32 heads x 512 158, 144 / 127; x 1024 420, 373 / 348; x
// 2048 1374, 1183 / 1178; 12 heads x 2048 582, 608; 24 heads x 2048 1072, 896; 8 x 4 heads x 1024 357, 343; x 2048 1300, 1134.  An XCD
// without a head, or with one less than the others, idles: 4 x 4 heads x 2048 679, 1109.  Head size 64, where a tile runs three blocks
// behind the one before: 8 heads x 1024 80, 134; x 2048 230, 251; x 4096 790, 650; 32 heads x 512 96, 83; x 1024 243, 198; x 4096 2867,
// 2506; 24 heads x 2048 625, 495; 12 heads x 2048 331, 341; 8 x 4 heads x 1024 208, 235; x 2048 751, 664; 4 x 4 heads x 2048 381, 576.
// What cannot come to less than less_us is given up as soon as that shows.  Every call of a ring backward plans, and it may have 50 us of
// work: the 512 jobs of 32 heads x 2048 rows x 16 chunks took 45 us as a search over 32 slots each, twice; so 2.
double one_walk_us(const st::Shape& s, const KeyWalk& keys, int batch, double less_us) {
  const int64_t rounds = (keys.heads / batch + 7) / 8;
  const double busy = (double)std::min<int64_t>(keys.heads, 8) / 8 * std::min(1.0, (double)keys.seen * rounds * batch / 32);
  const bool wide = s.D == 128;
  const double step = wide ? 1.5 + 0.45 * busy : 0.9 + 0.1 * busy, fixed = wide ? 20 : 12, unseen = 10, behind = wide ? step : 3 * step;
  const double around = 10 + (double)s.B * s.Hq * s.Sq * s.D * 12 / 5.5e6;      // the counts' start values, the pass that adds to dq
  double us = 0;
  for (int i = 0; i < keys.n; ++i) us += keys.c[i].tiles * (keys.c[i].blocks > 0 ? fixed + keys.c[i].blocks * keys.G * step : unseen);
  const double even = around + us * rounds * batch / 32;
  if (rounds * batch * keys.tiles > 512) return even + 31.0 / batch * behind;   // by the work alone
  if (even >= less_us) return even;
  // when the workgroups are free, rising, in a ring; the one that is free first takes a tile and falls back to where it ends.  A batch
  // that divides them moves in step: one of its heads stands for all.
  const bool in_step = 32 % batch == 0;
  const int m = in_step ? 32 / batch : 32, heads = in_step ? 1 : batch;
  double free[32] = {}, end = 0;
  int first = 0;
  for (int64_t r = 0; r < rounds; ++r) {
    double before[8] = {};
    for (int i = 0; i < keys.n; ++i)                    // most blocks first, as the tiles lie
      for (int t = 0; t < keys.c[i].tiles; ++t)
        for (int h = 0; h < heads; ++h) {
          double at = free[first];
          if (keys.c[i].blocks == 0) {
            at += unseen;
          } else {
            const double start = std::max(at + fixed / 2, before[h]);
            before[h] = start + behind;
            at = start + keys.c[i].blocks * keys.G * step + fixed / 2;
          }
          end = std::max(end, at);
          int slot = first;
          first = first + 1 < m ? first + 1 : 0;
          for (int ahead; slot != first && free[ahead = slot > 0 ? slot - 1 : m - 1] > at; slot = ahead) free[slot] = free[ahead];
          free[slot] = at;
        }
    if (around + end >= less_us) break;
  }
  return around + end;
}
// heads of a batch, 0: two passes
int one_walk(const st::Shape& s, const KeyWalk& keys, const int64_t* k_offset, int n, size_t room, double less_us) {
  if (s.Sk % st::kDkvFastKeys != 0 || keys.seen < 1 || st::knobs().one_walk == 0) return 0;
  if (st::knobs().one_walk != 1) less_us = 1e30;
  if (s.causal && k_offset != nullptr)
    for (int c = 1; c < n; ++c)                        // a tile sees the blocks of the ones behind it
      if (k_offset[c] < k_offset[c - 1] + s.Sk - st::kDkvFastKeys) return 0;
  int best = 0;
  const int64_t per_xcd = (keys.heads + 7) / 8;
  const int all = keys.heads % per_xcd == 0 && per_xcd <= 8 ? (int)per_xcd : 1, set = st::knobs().one_heads;
  const bool forced = set > 0 && keys.heads % set == 0;
  for (const int batch : {forced ? set : 1, forced ? set : all}) {
    if (batch == best || (size_t)st::OneRoom(s, n, batch).bytes > room) continue;
    const double us = one_walk_us(s, keys, batch, less_us);
    if (us >= less_us) continue;
    less_us = us;
    best = batch;
  }
  return best;
}
// Both passes in one launch: the compute units that have no key tile, or are done with theirs, take shares of the dQ pass
// meanwhile, and the launch ends with the last of them (jobs_us, key tiles first).  Forward and backward, apart and together:
// 4 heads x 700 rows x 4 chunks 99 and 77 us, 12 heads of 64 x 800 rows x 4 chunks 96 and 88 us, 6 heads x 1500 rows x 4
// chunks 146 and 116 us.
// `one`: the one walk may be taken.  `known`: for a caller who asks for the bytes only and has as many already (a plan with no more is
// any that has no more).
BwdSplit bwd_splits(const st::Shape& s, int dtype, const int64_t* k_offset, int n, size_t room, bool split_dq, bool one = false, size_t known = 0) {
  BwdSplit r;
  const bool bf16 = dtype == ST_BF16;
  const size_t one_room = room;
  room = std::min(room, kPartsMost);
  if ((bf16 && s.D != 128 && s.D != 64) || n < 1 || n > st::kMaxTable || s.B < 1 || s.Sq < 1 || s.Sk < 1 || s.Hq < 1 || s.Hkv < 1) return r;
  int64_t sorted[st::kMaxTable];                       // the plan does not depend on the order of the table
  if (s.causal && k_offset != nullptr) {
    std::copy(k_offset, k_offset + n, sorted);
    std::sort(sorted, sorted + n);
    k_offset = sorted;
  }
  QueryWalk walk;
  const int64_t wgs = (int64_t)s.B * s.Hq * st::query_tiles(s, bf16 ? st::kQTileFastRows : 32).count();
  const bool plan_dq = wgs < 1024 && (!bf16 || s.Sk >= st::kQTileFastKeys);
  split_dq = split_dq && wgs < 512;
  const Cost cost = dq_cost(dtype, s.D);
  const double add_us = bf16 ? 6 : 10;
  const size_t row_bytes = (size_t)s.B * s.Hq * s.D * sizeof(float);
  auto part_us = [&](int64_t rows) { return (double)(row_bytes * rows) / 8e6; };
  auto fits = [&](const Split& x) { return (size_t)x.rows_own0 * row_bytes <= room; };
  auto set_dq = [&](const Split& x) {
    const bool own0 = (size_t)x.rows * row_bytes > room;
    r.dq = x.table(own0);
    r.bytes = (size_t)(own0 ? x.rows_own0 : x.rows) * row_bytes;
  };
  double dq_us = 0;
  int dq_units = 0;
  if (plan_dq) {
    walk = query_walk(s, dtype, k_offset, n);
    dq_units = walk.most();
    double best = Split(walk, dq_units).launch_us(cost);
    if (split_dq) each_split(walk, kMaxSplits, [&](const Split& x) {
      if (!fits(x)) return;
      const double add = add_us + more_than_8_us(x) + part_us(x.rows + 2 * s.Sq);
      if (x.longest_us(cost) + add >= 0.95 * best) return;
      const double t = x.launch_us(cost) + add;
      if (t < 0.95 * best) {
        best = t;
        set_dq(x);
      }
    });
    dq_us = best;
  }
  if (!bf16) {
    if (plan_dq) f32_bwd_split(r, s, walk, k_offset, n, room, split_dq);
    return r;
  }
  KeyWalk keys;
  key_walk(keys, s, k_offset, n);
  const Cost kv_cost = dkv_cost(s.D);
  // the one walk instead, if it is faster than the two passes: over 108 shares its model is right to 6 % on average, that of the passes
  // says 0.87 of what they take (a walk of some hundred blocks on a full chip runs at the power limit).  Head size 64, 81 shares: right to
  // 8 %, the passes' 1.1 of what short ones take; at this bar none of them lost, and three that would have gained 3 to 8 % stay with them
  auto or_one = [&](const BwdSplit& two, double us) {
    if (two.bytes <= known && (size_t)st::OneRoom(s, n, 1).bytes <= known) return two;      // (larger batches need less)
    const int heads = one ? one_walk(s, keys, k_offset, n, one_room, (s.D == 128 ? 1.07 : 0.87) * us) : 0;
    if (heads == 0) return two;
    BwdSplit one;
    one.one_heads = heads;
    one.bytes = (size_t)st::OneRoom(s, n, heads).bytes;
    return one;
  };
  if (keys.seen < 1 || keys.tiles > 32767) return r;
  if (keys.heads * keys.seen >= 512) {
    double us = 0;                                     // through the queue, and dQ in many workgroups: by the work alone
    for (int i = 0; i < keys.n; ++i) us += keys.heads * keys.c[i].tiles * (keys.c[i].blocks > 0 ? kv_cost.us(keys.c[i].blocks * keys.G, kPlanCus) : 8) / kPlanCus;
    if (!plan_dq) {
      walk = query_walk(s, dtype, k_offset, n);
      for (int i = 0; i < walk.n; ++i) dq_us += cost.us(walk.units[i], kPlanCus) * walk.heads * (walk.n == 1 ? walk.tiles : 1) / kPlanCus;
    }
    return or_one(r, us + dq_us);
  }
  auto slot_bytes = [&](const KeySplit& x) { return (size_t)(keys.heads * x.slots * st::kv_slot_floats(s)) * sizeof(float); };
  // the adding pass reads the sums and reads and writes the gradients; only the keys a tile has are there, of the last tile of a
  // chunk often few.  What fits the L2 caches comes at some 16 TB/s, the rest at 5.
  const double tile_bytes = (double)keys.heads * 2 * s.Sk / ((s.Sk + st::kDkvFastKeys - 1) / st::kDkvFastKeys) * s.D * sizeof(float);
  auto add_kv_us = [&](const KeySplit& x) {
    const double bytes = tile_bytes * (x.slots + 2 * x.split_tiles), in_l2 = std::min(bytes, 16e6);
    return x.slots > 0 ? 6 + in_l2 / 16e6 + (bytes - in_l2) / 5e6 : 0.0;
  };
  Job job[512 + st::kShareTiles];
  int each_of[st::kKvSharesMost], ways = 1;            // unsplit, and the splits that have room
  each_of[0] = 0;
  for (int k = 2, before = keys.top; k <= st::kKvSharesMost && k <= keys.top; ++k) {
    const int each = (keys.top + k - 1) / k;
    if (each == before) continue;
    before = each;
    const KeySplit x(keys, each);
    if (slot_bytes(x) > room || keys.heads * x.items > 4 * kPlanCus) break;
    each_of[ways++] = each;
  }
  KeySplit kv(keys, 0);
  double kv_us = jobs_us(job, kv.jobs(job, kv_cost));
  for (int i = 1; i < ways; ++i) {
    const KeySplit x(keys, each_of[i]);
    const double add = add_kv_us(x), less = 0.95 * kv_us;     // more workgroups have to be worth it
    if (x.longest_us(kv_cost) + add >= less) continue;
    const double us = add + jobs_us(job, x.jobs(job, kv_cost), less - add);
    if (us < less) {
      kv_us = us;
      kv = x;
    }
  }
  size_t dq_bytes = r.bytes;
  double two_us = kv_us + 4 + dq_us;
  if (plan_dq && !st::dq_few(s, n)) {
    // Whole key tiles and the split that is best by itself first; any other one has to be better by 10 %, as the model does not know
    // that a share with the blocks of the diagonal takes longer (12/3 heads x 1408 rows: shares of 9 blocks a few per cent
    // better than of 4 in the model, 81 and 74 us).  Where the one that is best by itself fills the chip, few workgroups beside
    // dQ's may be far better: 2 x 8/4 heads x 1728 rows x 573 keys, three blocks 172 us and 224 in launches of their own.
    double &least = two_us, dq_work = 0, kv_work = 0;
    for (int i = 0; i < walk.n; ++i) dq_work += (double)walk.heads * (walk.n == 1 ? walk.tiles : 1) * walk.units[i];
    for (int i = 0; i < keys.n; ++i) kv_work += (double)keys.heads * keys.G * keys.c[i].tiles * keys.c[i].blocks;
    const int by_itself = kv.each;
    auto together = [&](const KeySplit& y, const Split& x) {
      const size_t left = room - slot_bytes(y);
      if (x.n > 1 && (size_t)x.rows_own0 * row_bytes > left) return;
      const double less = (y.each == 0 || y.each == by_itself ? 1 : 0.9) * least, add = (x.n > 1 ? add_us + more_than_8_us(x) + part_us(x.rows + 2 * s.Sq) : 0) + add_kv_us(y);
      if (x.longest_us(cost, y.workgroups()) + add >= less || y.longest_us(kv_cost, x.workgroups()) + add >= less) return;
      // not before all of the work is done, evenly spread
      const int64_t beside = x.workgroups() + y.workgroups();
      const double fixed = x.workgroups() * cost.us(0, beside) + y.workgroups() * kv_cost.us(0, beside);
      const double work = dq_work * (cost.us(1, beside) - cost.us(0, beside)) + kv_work * (kv_cost.us(1, beside) - kv_cost.us(0, beside));
      if ((fixed + work) / kPlanCus + add >= less) return;
      const int m = y.jobs(job, kv_cost, x.workgroups());
      const double us = add + jobs_us(job, m + x.jobs(job + m, cost, y.workgroups()), less - add);
      if (us >= less) return;
      least = us;
      const bool own0 = x.n > 1 && (size_t)x.rows * row_bytes > left;
      r.dq = x.table(own0);
      dq_bytes = x.n > 1 ? (size_t)(own0 ? x.rows_own0 : x.rows) * row_bytes : 0;
      r.pair = true;
      kv = y;
    };
    for (const bool others : {false, true})
      for (int i = 0; i < ways; ++i) {
        if (others == (i == 0 || each_of[i] == by_itself)) continue;
        const KeySplit y(keys, each_of[i]);
        together(y, Split(walk, dq_units));
        if (split_dq) each_split(walk, kMaxSplits, [&](const Split& x) { together(y, x); });
      }
  }
  r.kv_each = kv.each;
  r.kv_items = (int)kv.items;
  r.dq_bytes = dq_bytes;                               // whole rows of 64 or 128 floats: kv_parts stays on its boundary
  r.bytes = r.pair ? dq_bytes + slot_bytes(kv) : std::max(dq_bytes, slot_bytes(kv));
  return or_one(r, two_us);
}
void set_splits(st::BwdArgs& a, const BwdSplit& x, void* parts) {
  a.shares = x.dq;
  a.kv_each = x.kv_each;
  a.kv_items = x.kv_items;
  a.pair = x.pair;
  a.one_heads = x.one_heads;
  a.parts = (float*)parts;
  a.kv_parts = (float*)((char*)parts + (x.pair ? x.dq_bytes : 0));
}
void set_table_strides(st::ChunkTable& t, const st_ring_desc* d) {
  t.ksb = d->k_stride_b; t.kss = d->k_stride_s; t.ksh = d->k_stride_h;
  t.vsb = d->v_stride_b; t.vss = d->v_stride_s; t.vsh = d->v_stride_h;
}

}  // namespace

namespace st {

ProfScope::ProfScope(const char* name, hipStream_t s) : slot(-1), stream(s) {
  std::lock_guard<std::mutex> lk(g_prof_mu);
  if (!g_prof_on || g_prof.size() >= kProfMax) return;
  ProfRec r{name, nullptr, nullptr};
  if (hipEventCreate(&r.start) != hipSuccess) return;
  if (hipEventCreate(&r.stop) != hipSuccess) {
    (void)hipEventDestroy(r.start);
    return;
  }
  (void)hipEventRecord(r.start, s);
  g_prof.push_back(r);
  slot = (int)g_prof.size() - 1;
}

ProfScope::~ProfScope() {
  if (slot < 0) return;
  std::lock_guard<std::mutex> lk(g_prof_mu);
  if (slot < (int)g_prof.size()) (void)hipEventRecord(g_prof[slot].stop, stream);
}

}  // namespace st

extern "C" {

st_status st_profile_begin(void) {
  std::lock_guard<std::mutex> lk(g_prof_mu);
  for (auto& r : g_prof) {
    (void)hipEventDestroy(r.start);
    (void)hipEventDestroy(r.stop);
  }
  g_prof.clear();
  g_prof_on = true;
  return ST_OK;
}

st_status st_profile_end(st_profile_entry* out, int32_t max_entries, int32_t* n_entries) {
  if (!out || !n_entries || max_entries < 0) return fail(ST_ERR_INVALID_ARG, "null output");
  std::lock_guard<std::mutex> lk(g_prof_mu);
  g_prof_on = false;
  int32_t n = 0;
  st_status status = ST_OK;
  for (auto& r : g_prof) {
    float ms = 0.f;
    hipError_t e = hipEventSynchronize(r.stop);
    if (e == hipSuccess) e = hipEventElapsedTime(&ms, r.start, r.stop);
    if (e != hipSuccess) status = hip_fail(e, "st_profile_end");
    int32_t k = 0;
    while (k < n && strncmp(out[k].name, r.name, sizeof(out[k].name) - 1) != 0) ++k;
    if (k == n) {
      if (n >= max_entries) continue;
      memset(&out[n], 0, sizeof(out[n]));
      strncpy(out[n].name, r.name, sizeof(out[n].name) - 1);
      ++n;
    }
    out[k].launches += 1;
    out[k].total_ms += ms;
    (void)hipEventDestroy(r.start);
    (void)hipEventDestroy(r.stop);
  }
  g_prof.clear();
  *n_entries = n;
  return status;
}

st_status st_mfma_probe(const void* operands, int64_t operand_bytes, int32_t mix, int32_t iters, float* sink,
                        int64_t sink_floats, double* flop, void* hip_stream) {
  if (operands == nullptr || sink == nullptr) return fail(ST_ERR_INVALID_ARG, "null pointer");
  if (reinterpret_cast<uintptr_t>(operands) % 16) return fail(ST_ERR_ALIGNMENT, "operands: not 16-byte aligned");
  if (operand_bytes < 65536) return fail(ST_ERR_INVALID_ARG, "operands: at least 65536 bytes are needed");
  if (iters < 1 || iters > (1 << 24)) return fail(ST_ERR_INVALID_ARG, "iters must be in 1 .. 2^24");
  if (mix < 0 || mix > st::mfma_probe_mixes()) return fail(ST_ERR_INVALID_ARG, "mix must be in 0 .. %d", st::mfma_probe_mixes());
  const int blocks = st::mfma_probe_blocks();
  if (sink_floats < (int64_t)blocks * 256) return fail(ST_ERR_INVALID_ARG, "sink: %lld floats are needed", (long long)blocks * 256);
  ST_HIP(st::launch_mfma_probe(operands, operand_bytes, mix, iters, sink, blocks, (hipStream_t)hip_stream), "st_mfma_probe launch");
  if (flop) *flop = st::mfma_probe_flop(blocks, mix, iters);
  return ST_OK;
}

int32_t st_mfma_probe_mixes(void) { return st::mfma_probe_mixes(); }
const char* st_mfma_probe_mix_name(int32_t mix) { return st::mfma_probe_mix_name(mix); }

st_status st_device_facts(st_device_report* out) {
  if (out == nullptr) return fail(ST_ERR_INVALID_ARG, "null output");
  memset(out, 0, sizeof(*out));
  int dev = 0;
  ST_HIP(hipGetDevice(&dev), "hipGetDevice");
  hipDeviceProp_t prop;
  ST_HIP(hipGetDeviceProperties(&prop, dev), "hipGetDeviceProperties");
  const st::DeviceInfo& info = st::device_info();
  out->compute_units = info.cus > 0 ? info.cus : prop.multiProcessorCount;
  out->xcds = info.xcds;
  out->max_clock_mhz = prop.clockRate / 1000;
  out->memory_clock_mhz = prop.memoryClockRate / 1000;
  out->memory_bus_bits = prop.memoryBusWidth;
  out->hbm_bytes = (int64_t)prop.totalGlobalMem;
  strncpy(out->name, prop.name, sizeof(out->name) - 1);
  strncpy(out->arch, prop.gcnArchName, sizeof(out->arch) - 1);
  return ST_OK;
}

const char* st_status_str(st_status s) {
  switch (s) {
    case ST_OK: return "ok";
    case ST_ERR_INVALID_ARG: return "invalid argument";
    case ST_ERR_UNSUPPORTED: return "unsupported dtype / head_dim / size";
    case ST_ERR_ALIGNMENT: return "misaligned pointer or stride";
    case ST_ERR_HIP: return "HIP error";
    case ST_ERR_WORKSPACE: return "workspace missing or too small";
  }
  return "unknown status";
}

const char* st_last_error(void) { return g_err; }
int32_t st_version(void) { return 100; }

st_status st_attn_block_fwd(const st_block_desc* d, const st_tensor* q, const st_tensor* k, const st_tensor* v,
                            float* o_part, float* lse_part, void* hip_stream) {
  if (d == nullptr) return fail(ST_ERR_INVALID_ARG, "null descriptor");
  ST_TRY(check_shape(d->dtype, d->B, d->Hq, d->Hkv, d->D, d->Sq, d->Sk));
  ST_TRY(check_scale(d->scale));
  ST_TRY(check_segments(d->Sq, d->q_offset, d->q_seg, d->q_offset2));
  const int64_t n_q = (int64_t)d->B * d->Sq * d->Hq * d->D, n_kv = (int64_t)d->B * d->Sk * d->Hkv * d->D;
  ST_TRY(check_tensor("q", q, d->dtype, n_q));
  ST_TRY(check_tensor("k", k, d->dtype, n_kv));
  ST_TRY(check_tensor("v", v, d->dtype, n_kv));
  ST_TRY(check_f32("o_part", o_part, n_q));
  ST_TRY(check_f32("lse_part", lse_part, n_q));
  if (n_q == 0) return ST_OK;
  st::FwdArgs a;
  memset(&a, 0, sizeof(a));
  a.s = shape_of(d);
  a.q = view_of(q);
  a.t.n = n_kv > 0 ? 1 : 0;
  a.t.k[0] = k->ptr; a.t.v[0] = v->ptr; a.t.k_offset[0] = d->k_offset;
  a.t.ksb = k->stride_b; a.t.kss = k->stride_s; a.t.ksh = k->stride_h;
  a.t.vsb = v->stride_b; a.t.vss = v->stride_s; a.t.vsh = v->stride_h;
  a.o = o_part; a.lse = lse_part; a.o_lowp = nullptr;
  ST_HIP(launch_fwd(d->dtype, a, (hipStream_t)hip_stream), "st_attn_block_fwd launch");
  return ST_OK;
}

st_status st_attn_merge(float* o_acc, float* lse_acc, const float* o_part, const float* lse_part, int32_t B,
                        int32_t Sq, int32_t Hq, int32_t D, int32_t out_dtype, void* o_out_lowp, void* hip_stream) {
  if (B < 0 || Sq < 0 || Hq <= 0 || D <= 0) return fail(ST_ERR_INVALID_ARG, "bad sizes");
  if (D > 256 || D % 8 != 0) return fail(ST_ERR_UNSUPPORTED, "merge needs D <= 256 and D %% 8 == 0");
  if (out_dtype != ST_F32 && out_dtype != ST_BF16) return fail(ST_ERR_INVALID_ARG, "unknown out_dtype");
  const int64_t n = (int64_t)B * Sq * Hq * D;
  ST_TRY(check_f32("o_acc", o_acc, n));
  ST_TRY(check_f32("lse_acc", lse_acc, n));
  ST_TRY(check_f32("o_part", o_part, n));
  ST_TRY(check_f32("lse_part", lse_part, n));
  if (o_out_lowp && reinterpret_cast<uintptr_t>(o_out_lowp) % 16) return fail(ST_ERR_ALIGNMENT, "o_out_lowp: not 16-byte aligned");
  if (n > 0 && o_acc == o_part) return fail(ST_ERR_INVALID_ARG, "o_part aliases o_acc");
  ST_HIP(st::launch_merge(o_acc, lse_acc, o_part, lse_part, B, Sq, Hq, D, o_out_lowp, out_dtype,
                          (hipStream_t)hip_stream), "st_attn_merge launch");
  return ST_OK;
}

st_status st_attn_combine(const float* const* o_parts, const float* const* lse_parts, int32_t n_states, int32_t B,
                          int32_t Sq_in, int32_t Hq, int32_t D, int32_t row0, int32_t Sq_out, float* o_out,
                          float* lse_out, int32_t out_dtype, void* o_out_lowp, void* hip_stream) {
  if (!o_parts || !lse_parts) return fail(ST_ERR_INVALID_ARG, "null state tables");
  if (n_states < 1 || n_states > st::kMaxTable) return fail(ST_ERR_INVALID_ARG, "n_states must be 1..%d", st::kMaxTable);
  if (B < 0 || Sq_in < 0 || Sq_out < 0 || Hq <= 0 || D <= 0) return fail(ST_ERR_INVALID_ARG, "bad sizes");
  if (row0 < 0 || (int64_t)row0 + Sq_out > Sq_in) return fail(ST_ERR_INVALID_ARG, "rows [%d, %d + %d) are not inside the %d rows of the states", row0, row0, Sq_out, Sq_in);
  if (D > 256 || D % 8 != 0) return fail(ST_ERR_UNSUPPORTED, "combine needs D <= 256 and D %% 8 == 0");
  if (out_dtype != ST_F32 && out_dtype != ST_BF16) return fail(ST_ERR_INVALID_ARG, "unknown out_dtype");
  const int64_t n_in = (int64_t)B * Sq_in * Hq * D, n_out = (int64_t)B * Sq_out * Hq * D;
  ST_TRY(check_f32("o_out", o_out, n_out));
  ST_TRY(check_f32("lse_out", lse_out, n_out));
  if (o_out_lowp && reinterpret_cast<uintptr_t>(o_out_lowp) % 16) return fail(ST_ERR_ALIGNMENT, "o_out_lowp: not 16-byte aligned");
  st::CombineArgs a;
  memset(&a, 0, sizeof(a));
  for (int x = 0; x < n_states; ++x) {
    ST_TRY(check_f32("o_parts[x]", o_parts[x], n_in));
    ST_TRY(check_f32("lse_parts[x]", lse_parts[x], n_in));
    if (n_out > 0 && (o_parts[x] == o_out || lse_parts[x] == lse_out)) return fail(ST_ERR_INVALID_ARG, "an output aliases state %d", x);
    a.o[x] = o_parts[x];
    a.lse[x] = lse_parts[x];
  }
  if (n_out == 0) return ST_OK;
  a.n = n_states;
  a.B = B; a.Sq_in = Sq_in; a.Hq = Hq; a.D = D; a.row0 = row0; a.Sq_out = Sq_out;
  a.o_out = o_out; a.lse_out = lse_out; a.o_lowp = o_out_lowp;
  ST_HIP(st::launch_combine(a, out_dtype, (hipStream_t)hip_stream), "st_attn_combine launch");
  return ST_OK;
}

st_status st_attn_delta(const st_block_desc* d, const st_tensor* d_o, const st_tensor* o, int32_t o_dtype,
                        float* delta, void* hip_stream) {
  if (d == nullptr) return fail(ST_ERR_INVALID_ARG, "null descriptor");
  ST_TRY(check_shape(d->dtype, d->B, d->Hq, d->Hkv, d->D, d->Sq, 0));
  if (o_dtype != ST_F32 && o_dtype != d->dtype) return fail(ST_ERR_INVALID_ARG, "o_dtype must be ST_F32 or the storage dtype");
  const int64_t n = (int64_t)d->B * d->Sq * d->Hq * d->D;
  ST_TRY(check_tensor("d_o", d_o, d->dtype, n));
  ST_TRY(check_tensor("o", o, o_dtype, n));
  ST_TRY(check_f32("delta", delta, n));
  if (n == 0) return ST_OK;
  ST_HIP(st::launch_delta(view_of(d_o), d->dtype, view_of(o), o_dtype, delta, d->B, d->Sq, d->Hq, d->D,
                          (hipStream_t)hip_stream), "st_attn_delta launch");
  return ST_OK;
}

// Q' = bf16(Q scale log2 e), then room for the partial sums of an under-filled dK/dV launch (which runs unsplit without it).
// The dQ of this call is the same with and without a workspace, bit for bit, so that pass is never split here.
static size_t block_base_bytes(const st_block_desc* d) { return align_up((size_t)d->B * d->Sq * d->Hq * d->D * 2, 256); }

// as with a ring's (ring_plan): one plan whatever the room, unless that is short
static BwdSplit block_plan(const st::Shape& s, int dtype, int64_t k_offset, size_t room) {
  const BwdSplit r = bwd_splits(s, dtype, &k_offset, 1, kPartsMost, false);
  return r.bytes <= room ? r : bwd_splits(s, dtype, &k_offset, 1, room, false);
}

size_t st_attn_block_bwd_workspace_bytes(const st_block_desc* d) {
  if (d == nullptr || d->dtype != ST_BF16 || d->B <= 0 || d->Sq <= 0 || d->Hq <= 0 || d->D <= 0) return 0;
  const st::Shape s = shape_of(d);
  size_t most = bwd_splits(s, d->dtype, nullptr, 1, kPartsMost, false).bytes;
  if (d->causal)
    // one workspace serves every chunk of a ring, and under a mask the plan depends on where the chunk lies: seen whole (above),
    // here, on the diagonal of either run of rows, and seen by the second run only
    for (const int64_t k_offset : {d->k_offset, d->q_offset, d->q_offset2, d->q_offset + d->q_seg})
      most = std::max(most, bwd_splits(s, d->dtype, &k_offset, 1, kPartsMost, false).bytes);
  return block_base_bytes(d) + most;
}

st_status st_attn_block_bwd(const st_block_desc* d, const st_tensor* q, const st_tensor* k, const st_tensor* v,
                            const st_tensor* d_o, const float* lse_final, const float* delta, float* dq_acc,
                            float* dk_acc, float* dv_acc, void* workspace, size_t workspace_bytes, void* hip_stream) {
  if (d == nullptr) return fail(ST_ERR_INVALID_ARG, "null descriptor");
  ST_TRY(check_shape(d->dtype, d->B, d->Hq, d->Hkv, d->D, d->Sq, d->Sk));
  ST_TRY(check_scale(d->scale));
  ST_TRY(check_segments(d->Sq, d->q_offset, d->q_seg, d->q_offset2));
  const int64_t n_q = (int64_t)d->B * d->Sq * d->Hq * d->D, n_kv = (int64_t)d->B * d->Sk * d->Hkv * d->D;
  ST_TRY(check_tensor("q", q, d->dtype, n_q));
  ST_TRY(check_tensor("d_o", d_o, d->dtype, n_q));
  ST_TRY(check_tensor("k", k, d->dtype, n_kv));
  ST_TRY(check_tensor("v", v, d->dtype, n_kv));
  ST_TRY(check_f32("lse_final", lse_final, n_q));
  ST_TRY(check_f32("delta", delta, n_q));
  ST_TRY(check_f32("dq_acc", dq_acc, n_q));
  ST_TRY(check_f32("dk_acc", dk_acc, n_kv));
  ST_TRY(check_f32("dv_acc", dv_acc, n_kv));
  if (n_q == 0 || n_kv == 0) return ST_OK;
  if (d->causal && d->k_offset > st::q_pos(shape_of(d), d->Sq - 1)) return ST_OK;   // chunk entirely in the future
  st::BwdArgs a;
  memset(&a, 0, sizeof(a));
  a.s = shape_of(d);
  a.q = view_of(q);
  a.d_o = view_of(d_o);
  a.t.n = 1;
  a.t.k[0] = k->ptr; a.t.v[0] = v->ptr; a.t.k_offset[0] = d->k_offset;
  a.t.ksb = k->stride_b; a.t.kss = k->stride_s; a.t.ksh = k->stride_h;
  a.t.vsb = v->stride_b; a.t.vss = v->stride_s; a.t.vsh = v->stride_h;
  a.lse = lse_final; a.delta = delta; a.dq = dq_acc; a.dk[0] = dk_acc; a.dv[0] = dv_acc;
  if (d->dtype == ST_BF16 && workspace != nullptr) {
    if (workspace_bytes < block_base_bytes(d)) return fail(ST_ERR_WORKSPACE, "block backward workspace needs %zu bytes", st_attn_block_bwd_workspace_bytes(d));
    if (reinterpret_cast<uintptr_t>(workspace) % 256) return fail(ST_ERR_ALIGNMENT, "workspace: not 256-byte aligned");
    ST_HIP(st::launch_scale_q(a.q, workspace, d->B, d->Sq, d->Hq, d->D, d->scale, (hipStream_t)hip_stream), "scaled-Q launch");
    a.qs = workspace;
    const size_t left = workspace_bytes - block_base_bytes(d);
    set_splits(a, block_plan(a.s, d->dtype, d->k_offset, std::min(left, kPartsMost)), (char*)workspace + block_base_bytes(d));
  }
  ST_HIP(launch_bwd(d->dtype, a, (hipStream_t)hip_stream), "st_attn_block_bwd launch");
  return ST_OK;
}

st_status st_cast_from_f32(const float* src, void* dst, int64_t n, int32_t dst_dtype, void* hip_stream) {
  if (n < 0) return fail(ST_ERR_INVALID_ARG, "negative n");
  if (dst_dtype != ST_F32 && dst_dtype != ST_BF16) return fail(ST_ERR_INVALID_ARG, "unknown dst_dtype");
  ST_TRY(check_f32("src", src, n));
  if (n > 0 && (dst == nullptr || reinterpret_cast<uintptr_t>(dst) % 16)) return fail(dst ? ST_ERR_ALIGNMENT : ST_ERR_INVALID_ARG, "dst: null or misaligned");
  ST_HIP(st::launch_cast(src, dst, n, dst_dtype, (hipStream_t)hip_stream), "st_cast_from_f32 launch");
  return ST_OK;
}

// Closed form of the schedule.  With S = P / C^2 teams per team group, the initial dispatch
// leaves GPU (team t, member a) holding the gathered KV of team (t mod S) * C + a, and every
// sub-ring step hands a buffer to the next team of the group, so at iteration i the GPU works on
// team buffer ((t - i) mod S) * C + a, i.e. sequence shards [buffer * C, buffer * C + C).
st_status st_visit_order(int32_t P, int32_t C, int32_t rank, int32_t* shard_idx, int32_t* member_of) {
  if (P < 1 || C < 1 || P % C != 0 || (P / C) % C != 0) return fail(ST_ERR_INVALID_ARG, "layout needs C >= 1 and C*C | P (P=%d C=%d)", P, C);
  if (rank < 0 || rank >= P) return fail(ST_ERR_INVALID_ARG, "rank %d outside 0..%d", rank, P - 1);
  if (!shard_idx || !member_of) return fail(ST_ERR_INVALID_ARG, "null output");
  const int32_t S = P / (C * C);
  const int32_t t = rank / C;
  int32_t n = 0;
  for (int32_t a = 0; a < C; ++a)
    for (int32_t i = 0; i < S; ++i) {
      const int32_t pos = ((t - i) % S + S) % S;
      const int32_t buffer = pos * C + a;
      for (int32_t c = 0; c < C; ++c, ++n) {
        shard_idx[n] = buffer * C + c;
        member_of[n] = a;
      }
    }
  return ST_OK;
}

// Iteration i of GPU (team t, member a) works on the gathered buffer of team ((t - i) mod S) * C + a,
// S = P / C^2 GPUs per sub-ring (closed form of the initial placement followed by i sub-ring passes).
st_status st_team_visit_order(int32_t P, int32_t C, int32_t rank, int32_t* team_buffer) {
  if (!team_buffer) return fail(ST_ERR_INVALID_ARG, "null output");
  if (P < 1 || C < 1 || P % C != 0 || (P / C) % C != 0) return fail(ST_ERR_INVALID_ARG, "layout needs C >= 1 and C*C | P (P=%d C=%d)", P, C);
  if (rank < 0 || rank >= P) return fail(ST_ERR_INVALID_ARG, "rank %d outside 0..%d", rank, P - 1);
  const int32_t S = P / (C * C), t = rank / C, a = rank % C;
  for (int32_t i = 0; i < S; ++i) {
    const int32_t pos = ((t - i) % S + S) % S;
    team_buffer[i] = pos * C + a;
  }
  return ST_OK;
}

// Iteration counts and exchanged bytes of plain ring attention and of the concentric layout for one
// attention block forward on one GPU (Section 3.2, "Theoretical Analysis", its three communication
// expressions with bandwidth W and latency L).  A ring step hands on one K and one V shard of N/P tokens; a sub-ring step hands on
// the C shards a team gathered; the team all-gather of Q, K, V and the reduce-scatter of O move
// (C - 1) / C of 4 tensors of C N / P tokens.
st_status st_schedule_report(int32_t P, int32_t C, int64_t B, int64_t N, int64_t H, int32_t e, double W, double L,
                             st_comm_report* out) {
  if (!out) return fail(ST_ERR_INVALID_ARG, "null output");
  if (P < 1 || C < 1 || P % C != 0 || (P / C) % C != 0) return fail(ST_ERR_INVALID_ARG, "layout needs C >= 1 and C*C | P (P=%d C=%d)", P, C);
  if (B < 1 || N < 1 || H < 1 || e < 1 || N % P != 0) return fail(ST_ERR_INVALID_ARG, "sizes must be positive and P must divide N");
  if (!(W > 0.0) || !(L >= 0.0)) return fail(ST_ERR_INVALID_ARG, "bandwidth must be positive and latency non-negative");
  const __int128 shard = (__int128)B * (N / P) * H * e;            // bytes of one tensor's shard on one GPU
  const __int128 limit = ((__int128)1 << 62);
  if (shard * 4 * P > limit) return fail(ST_ERR_INVALID_ARG, "sizes overflow 64-bit byte counts");
  out->ring_iterations = P - 1;
  out->startrail_iterations = P / (C * C) - 1;
  out->ring_p2p_bytes_per_iter = (int64_t)(2 * shard);
  out->startrail_p2p_bytes_per_iter = (int64_t)(2 * shard * C);
  out->ring_p2p_bytes = out->ring_p2p_bytes_per_iter * out->ring_iterations;
  out->startrail_p2p_bytes = out->startrail_p2p_bytes_per_iter * out->startrail_iterations;
  out->startrail_collective_bytes = (int64_t)(4 * shard * (C - 1));
  out->ring_p2p_seconds = out->ring_iterations * ((double)out->ring_p2p_bytes_per_iter / W + L);
  out->startrail_p2p_seconds = out->startrail_iterations * ((double)out->startrail_p2p_bytes_per_iter / W + L);
  out->startrail_collective_seconds = (double)out->startrail_collective_bytes / W;
  return ST_OK;
}

// A fused forward whose query tiles alone would leave part of the chip idle (a workgroup per 256 rows and head in bf16, per
// 32 rows in fp32, on 256 compute units) is split over the keys: a query tile gets several workgroups, each with a share of
// the walk and a partial state of its own, and one combine pass folds the states (the tiles of a ring are independent
// until the fold, Algorithm 1).  The split is the one for which launch + combine is least (Split::launch_us) with the
// constants of fwd_cost, 5 us for the combine pass and what its bytes take, 8 TB/s from the caches; fp32 8 us, as a caller that
// waits for launches loses some by one more.  To be split at all has to be worth 5 %; a split of more workgroups 3 % (100
// under-filled shares 0.7 % faster than with 5; with 1 some that are 3 to 10 % slower, and more states).
// Under a causal mask the tiles differ, and shares of one size are what fills the chip: 48 heads x two runs of 736 rows,
// walks of 230 and 610 tiles, 885 us with one number of shares for all tiles and 674 so (dQ 1254 and 1024); 3 heads x two
// runs of 2112 rows 254 and 185 (342 and 253).
static bool fwd_splittable(const st_ring_desc* d, int n_visible) {
  const bool bf16 = d->dtype == ST_BF16;
  if (n_visible < 1 || n_visible > st::kMaxTable || d->B < 1 || d->Sq < 1 || d->Hq < 1) return false;
  if (bf16 && ((d->D != 128 && d->D != 64) || d->Sk < st::kQTileFastKeys)) return false;
  return (int64_t)d->B * d->Hq * st::query_tiles(shape_of(d), bf16 ? st::kQTileFastRows : 32).count() < 512;
}
// k_offset of the visible chunks; nullptr: of chunks that every row sees
static st::TileShares fwd_shares(const st_ring_desc* d, const int64_t* k_offset, int n_visible, int most = kMaxSplits) {
  st::TileShares r = {};
  if (!fwd_splittable(d, n_visible)) return r;
  const bool bf16 = d->dtype == ST_BF16;
  const QueryWalk walk = query_walk(shape_of(d), d->dtype, k_offset, n_visible);
  const Cost cost = fwd_cost(d->dtype, d->D);
  const double combine_us = bf16 ? 5 : 8;
  const double row_us = (double)d->B * d->Hq * d->D * sizeof(float) / 8e6;
  double best = Split(walk, walk.most()).launch_us(cost);
  each_split(walk, most, [&](const Split& x) {
    const double add = combine_us + more_than_8_us(x) + (x.rows + 1.5 * d->Sq) * row_us;
    const double less = (r.n > 1 ? 0.97 : 0.95) * best;      // to be split at all has to be worth it; of two splits the better one
    if (x.longest_us(cost) + add >= less) return;
    const double t = x.launch_us(cost) + add;
    if (t < less) {
      best = t;
      r = x.table(false);
    }
  });
  return r;
}
// A share whose full 256-row tiles fill less than half of the chip: its workspace has always held a state per chunk (up to
// 256 workgroups) and one more, and its forward has always been refused without one.  Both are part of the interface.
static int fwd_states_small(const st_ring_desc* d, int n_visible) {
  if (d->dtype != ST_BF16 || (d->D != 128 && d->D != 64) || n_visible < 2 || n_visible > st::kMaxTable) return 1;
  if (d->Sq < st::kQTileFastRows || d->Sk < st::kQTileFastKeys) return 1;
  const int64_t wgs = (int64_t)d->B * d->Hq * (d->Sq / st::kQTileFastRows);
  if (wgs < 1 || wgs >= 128) return 1;
  int64_t n = 256 / wgs;
  if (n > n_visible) n = n_visible;
  if (n > kMaxSplits) n = kMaxSplits;
  return (int)n + 1;
}
// States to provide for: any subset of the chunks may be visited.  Under a causal mask the tiles with the longest walks may
// be split where one number for all of them would not be, as the chunks that this shard sees lie; they have about twice the
// average, so more than twice the chip's workgroups are not provided for.
static int fwd_states_most(const st_ring_desc* d) {
  const int n_most = d->n_chunks < st::kMaxTable ? d->n_chunks : st::kMaxTable;
  int most = fwd_states_small(d, n_most);
  for (int n = 1; n <= n_most; ++n) most = std::max(most, (int)fwd_shares(d, nullptr, n).n);
  if (!d->causal || d->k_offset == nullptr || !fwd_splittable(d, n_most)) return most;
  int64_t k_offset[st::kMaxTable];
  int n = 0;
  for (int j = 0; j < std::min(d->n_chunks, ST_MAX_CHUNKS) && n <= st::kMaxTable; ++j)
    if (!chunk_invisible(d, j) && n++ < st::kMaxTable) k_offset[n - 1] = d->k_offset[j];
  if (n > st::kMaxTable) return most;                  // are never split
  const int64_t wgs = query_walk(shape_of(d), d->dtype, nullptr, n_most).wgs();
  const int provided = (int)std::min<int64_t>(kMaxSplits, (2 * kPlanCus + wgs - 1) / wgs);
  return std::max(most, (int)fwd_shares(d, k_offset, n, std::max(most, provided)).n);
}

// Workspace layout (each block 256-byte aligned):
//   forward, stepwise: partial O, partial lse, member O, member lse
//   forward, fused:    partial O and partial lse, once (when more than one launch is needed) or once per
//                      split of an under-filled launch: [O_0, lse_0, O_1, ...]
//   backward:          Delta, the tile counters of the dK/dV launch (kQueueInts ints), for the bf16 dtype
//                      Q' = bf16(Q scale log2 e), dense [B,Sq,Hq,D], and the partial sums of
//                      under-filled dQ and dK/dV launches (at most kPartsMost)
static size_t bwd_base_bytes(const st_ring_desc* d) {
  const size_t n_o = align_up((size_t)d->B * d->Sq * d->Hq * d->D * sizeof(float), 256);
  return align_up((size_t)d->B * d->Sq * d->Hq * sizeof(float), 256) + align_up(st::kQueueInts * sizeof(int32_t), 256) +
         (d->dtype == ST_BF16 ? align_up(n_o / 2, 256) : 0);
}

// What a workspace has beyond the rest, for the sums of a ring backward, and the most of it that is ever used
static size_t room_most(const st_ring_desc* d) { return bwd_base_bytes(d) > kScratchBytes ? kRoomMostLarge : kRoomMost; }
static size_t ring_room(const st_ring_desc* d, size_t workspace_bytes) {
  const size_t base = bwd_base_bytes(d);
  return workspace_bytes > base ? std::min(workspace_bytes - base, room_most(d)) : 0;
}

// Whether the one walk takes this share's K and V rows: as far as the descriptor tells (the launcher has the last word, one_fast_usable)
static bool one_strides(const st_ring_desc* d) {
  return std::max(d->k_stride_s, d->v_stride_s) < ((int64_t)1 << 30) / (2 * st::kDkvFastKeys);
}

// Partial sums to provide for.  Under a causal mask the plan depends on where the chunks lie: as a caller visits them who lists
// all of them, in one launch or a launch each, and where every row sees them, so that what was sized for one shard does for
// its neighbours.  Without one it depends on their number, and any subset may be visited.
// `enough`: what more than that is not of interest.
static size_t ring_parts_bytes(const st_ring_desc* d, int mode, size_t enough = SIZE_MAX) {
  const st::Shape s = shape_of(d);
  const bool fused = mode == ST_RING_FUSED;
  const int n_chunks = std::min(d->n_chunks, ST_MAX_CHUNKS), per_launch = std::min(n_chunks, fused ? st::kMaxTable : 1);
  size_t most = 0;
  auto look = [&](const int64_t* k_offset, int n) {
    if (most < enough) most = std::max(most, bwd_splits(s, d->dtype, k_offset, n, room_most(d), true, one_strides(d), most).bytes);
  };
  if (!d->causal || d->k_offset == nullptr) {
    look(nullptr, per_launch);                         // the sums of one walk grow with the chunks; the plans of few are made quickly
    for (int n = 1; n < per_launch; ++n) look(nullptr, n);
    return most;
  }
  look(nullptr, per_launch);
  for (int hidden = 0; hidden <= (fused && d->dtype == ST_BF16); ++hidden) {       // without and with the chunks that nobody sees
    int64_t k_offset[st::kMaxTable];
    int n = 0;
    bool whole = false;                                // one that every row sees has been looked at
    for (int j = 0; j < n_chunks; ++j) {
      if (!hidden && chunk_invisible(d, j)) continue;
      if (!fused && d->k_offset[j] + d->Sk - 1 <= d->q_offset) {
        if (whole) continue;
        whole = true;
      }
      k_offset[n++] = d->k_offset[j];
      if (n == per_launch) {
        look(k_offset, n);
        n = 0;
      }
    }
    if (n > 0) look(k_offset, n);
  }
  return most;
}

// The chunks of a backward launch and whether ring_parts_bytes has looked at such a one
struct RingVisit {
  int chunk[ST_MAX_CHUNKS], n = 0, hidden = 0;
  void add(const st_ring_desc* d, int j) {
    chunk[n++] = j;
    hidden += chunk_invisible(d, j);
  }
  bool provided(const st_ring_desc* d, int mode) const {
    if (mode != ST_RING_FUSED || !d->causal) return true;
    if (n > st::kMaxTable) return false;
    int seen = 0;
    for (int j = 0; j < d->n_chunks; ++j) seen += !chunk_invisible(d, j);
    return n - hidden == seen && (hidden == 0 || n == d->n_chunks);
  }
};

// The plan of a launch over n chunks.  It does not depend on the room beyond what st_ring_workspace_bytes provides for, so that
// st_ring_bwd with that much and st_ring_bwd_noalloc compute the same sums; with less it is the best one that fits.  `one`: the one walk
// takes these tensors.
static BwdSplit ring_plan(const st_ring_desc* d, int mode, const int64_t* k_offset, int n, bool provided, size_t room, bool one) {
  const st::Shape s = shape_of(d);
  BwdSplit r = bwd_splits(s, d->dtype, k_offset, n, room_most(d), true, one);
  provided = provided && one == one_strides(d);
  if (!provided && r.bytes > 0) room = std::min(room, ring_parts_bytes(d, mode, r.bytes));
  return r.bytes <= room ? r : bwd_splits(s, d->dtype, k_offset, n, room, true, one);
}

size_t st_ring_workspace_bytes(const st_ring_desc* d, int32_t mode, int32_t backward) {
  if (d == nullptr) return 0;
  const size_t n_o = align_up((size_t)d->B * d->Sq * d->Hq * d->D * sizeof(float), 256);
  const size_t n_l = align_up((size_t)d->B * d->Sq * d->Hq * sizeof(float), 256);
  if (backward) return bwd_base_bytes(d) + ring_parts_bytes(d, mode);
  if (mode == ST_RING_STEPWISE) return 2 * (n_o + n_l);
  return (size_t)fwd_states_most(d) * (n_o + n_l);
}

st_status st_ring_fwd(const st_ring_desc* d, const st_tensor* q, const int32_t* order, const int32_t* member_of,
                      int32_t n_visit, int32_t mode, float* o_acc, float* lse, void* o_lowp, void* workspace,
                      size_t workspace_bytes, void* hip_stream) {
  ST_TRY(check_ring(d, q, order, n_visit));
  if (mode != ST_RING_STEPWISE && mode != ST_RING_FUSED) return fail(ST_ERR_INVALID_ARG, "unknown mode %d", mode);
  const int64_t n_o = (int64_t)d->B * d->Sq * d->Hq * d->D, n_l = (int64_t)d->B * d->Sq * d->Hq;
  ST_TRY(check_f32("o_acc", o_acc, n_o));
  ST_TRY(check_f32("lse", lse, n_o));
  if (o_lowp && reinterpret_cast<uintptr_t>(o_lowp) % 16) return fail(ST_ERR_ALIGNMENT, "o_lowp: not 16-byte aligned");
  if (n_o == 0) return ST_OK;
  hipStream_t stream = (hipStream_t)hip_stream;

  // visible chunks in visit order
  int vis[ST_MAX_CHUNKS], mem[ST_MAX_CHUNKS], n = 0;
  for (int x = 0; x < n_visit; ++x)
    if (!chunk_invisible(d, order[x])) {
      vis[n] = order[x];
      mem[n] = member_of ? member_of[x] : 0;
      ++n;
    }

  const size_t b_o = align_up((size_t)n_o * sizeof(float), 256), b_l = align_up((size_t)n_l * sizeof(float), 256);
  st::FwdArgs a;
  memset(&a, 0, sizeof(a));
  a.s = shape_of(d);
  a.q = view_of(q);
  set_table_strides(a.t, d);
  const bool fused = mode == ST_RING_FUSED, fast = d->dtype == ST_BF16 && st::fwd_fast_usable(a);
  const size_t state = b_o + b_l;
  // The step-wise walk, more chunks than one launch takes and small shares need a workspace: the least of it is what they
  // have always asked for.  What is there beyond that, or for any other share, only decides how many states a split may have:
  // one that is missing, short or off the boundary costs workgroups, not the call.
  const int n_most = d->n_chunks < st::kMaxTable ? d->n_chunks : st::kMaxTable;
  const bool small = fused && fast && fwd_states_small(d, n) > 1;
  const size_t least = !fused ? 2 * state : small || n > st::kMaxTable ? fwd_states_small(d, n_most) * state : 0;
  const bool on_boundary = reinterpret_cast<uintptr_t>(workspace) % 256 == 0;
  if (least > 0) {
    if (workspace == nullptr || workspace_bytes < least) return fail(ST_ERR_WORKSPACE, "forward workspace needs %zu bytes", st_ring_workspace_bytes(d, mode, 0));
    if (!on_boundary) return fail(ST_ERR_ALIGNMENT, "workspace: not 256-byte aligned");
  }
  const size_t room = fused && workspace != nullptr && on_boundary ? workspace_bytes / state : 0;
  st::TileShares shares = {};
  if (room > 1 && n > 0 && n <= st::kMaxTable && (fast || d->dtype != ST_BF16)) {        // only the hand-scheduled kernel walks a split table
    int64_t k_offset[st::kMaxTable];
    for (int x = 0; x < n; ++x) k_offset[x] = d->k_offset[vis[x]];
    shares = fwd_shares(d, k_offset, n, room < (size_t)kMaxSplits ? (int)room : kMaxSplits);
  }
  char* ws = (char*)workspace;
  float* part_o = (float*)ws;
  float* part_l = (float*)(ws + b_o);

  if (shares.n > 1) {
    a.t.n = n;
    for (int x = 0; x < n; ++x) {
      a.t.k[x] = d->k_ptr[vis[x]];
      a.t.v[x] = d->v_ptr[vis[x]];
      a.t.k_offset[x] = d->k_offset[vis[x]];
    }
    a.o = o_acc;
    a.lse = lse;
    a.o_lowp = o_lowp;
    a.shares = shares;
    a.part_o = part_o;
    a.part_lse = part_l;
    a.part_stride = (int64_t)(state / sizeof(float));
    ST_HIP(launch_fwd(d->dtype, a, stream), "split forward launch");
    st::CombineArgs c;
    memset(&c, 0, sizeof(c));
    c.n = shares.n;
    c.shares = shares;
    c.tiles = st::query_tiles(a.s, d->dtype == ST_BF16 ? st::kQTileFastRows : 32);
    for (int y = 0; y < c.n; ++y) {
      c.o[y] = part_o + y * a.part_stride;
      c.lse[y] = part_l + y * a.part_stride;
    }
    c.B = d->B; c.Sq_in = d->Sq; c.Hq = d->Hq; c.D = d->D; c.row0 = 0; c.Sq_out = d->Sq;
    c.o_out = o_acc; c.lse_out = lse; c.o_lowp = o_lowp;
    ST_HIP(st::launch_combine(c, d->dtype, stream), "combine launch");
    return ST_OK;
  }

  if (mode == ST_RING_FUSED) {
    // one launch per kMaxTable visible chunks; further launches go through a partial state + merge
    if (n == 0) {
      ST_HIP(st::launch_fill_state(o_acc, lse, n_o, n_l, stream), "state fill");
      if (o_lowp) ST_HIP(st::launch_cast(o_acc, o_lowp, n_o, d->dtype, stream), "cast");
      return ST_OK;
    }
    for (int x0 = 0; x0 < n; x0 += st::kMaxTable) {
      const int cnt = n - x0 < st::kMaxTable ? n - x0 : st::kMaxTable;
      a.t.n = cnt;
      for (int x = 0; x < cnt; ++x) {
        a.t.k[x] = d->k_ptr[vis[x0 + x]];
        a.t.v[x] = d->v_ptr[vis[x0 + x]];
        a.t.k_offset[x] = d->k_offset[vis[x0 + x]];
      }
      const bool single = n <= st::kMaxTable;
      a.o = x0 == 0 ? o_acc : part_o;
      a.lse = x0 == 0 ? lse : part_l;
      a.o_lowp = single ? o_lowp : nullptr;
      ST_HIP(launch_fwd(d->dtype, a, stream), "fused forward launch");
      if (x0 > 0) {
        const bool last = x0 + cnt >= n;
        ST_HIP(st::launch_merge(o_acc, lse, part_o, part_l, d->B, d->Sq, d->Hq, d->D, last ? o_lowp : nullptr,
                                d->dtype, stream), "merge launch");
      }
    }
    return ST_OK;
  }

  // stepwise: per member a running state (Algorithm 1 loop), then the combine of the member states.  A fold into an empty state
  // is that state, bit for bit: the first block of a member starts its state, and the first member's state is the result's
  // (24/12 heads x 2 x 838 rows, one visible chunk: 76 us with the fills and folds of empty states, 35 without).
  if (n == 0) {
    ST_HIP(st::launch_fill_state(o_acc, lse, n_o, n_l, stream), "state fill");
    if (o_lowp) ST_HIP(st::launch_cast(o_acc, o_lowp, n_o, d->dtype, stream), "cast");
    return ST_OK;
  }
  float* mem_o = (float*)(ws + b_o + b_l);
  float* mem_l = (float*)(ws + 2 * b_o + b_l);
  a.t.n = 1;
  for (int x = 0; x < n;) {
    const int member = mem[x], first = x;
    float *to = first == 0 ? o_acc : mem_o, *to_l = first == 0 ? lse : mem_l;
    for (; x < n && mem[x] == member; ++x) {
      a.t.k[0] = d->k_ptr[vis[x]];
      a.t.v[0] = d->v_ptr[vis[x]];
      a.t.k_offset[0] = d->k_offset[vis[x]];
      a.o = x == first ? to : part_o;
      a.lse = x == first ? to_l : part_l;
      a.o_lowp = n == 1 ? o_lowp : nullptr;          // the last write of the result rounds it
      ST_HIP(launch_fwd(d->dtype, a, stream), "block forward launch");
      if (x > first)
        ST_HIP(st::launch_merge(to, to_l, part_o, part_l, d->B, d->Sq, d->Hq, d->D, first == 0 && x == n - 1 ? o_lowp : nullptr, d->dtype, stream), "merge launch");
    }
    if (first > 0)
      ST_HIP(st::launch_merge(o_acc, lse, mem_o, mem_l, d->B, d->Sq, d->Hq, d->D, x == n ? o_lowp : nullptr, d->dtype, stream), "combine launch");
  }
  return ST_OK;
}

// partial sums in parts_bytes bytes at `parts`
static st_status ring_bwd(const st_ring_desc* d, const st_tensor* q, const st_tensor* d_o, const st_tensor* o, int32_t o_dtype,
                          const float* lse_final, const int32_t* order, int32_t n_visit, int32_t mode, float* dq_acc, float* const* dk_acc,
                          float* const* dv_acc, int32_t kv_flags, void* const* dk_lowp, void* const* dv_lowp, void* workspace,
                          size_t workspace_bytes, void* parts, size_t parts_bytes, void* hip_stream);

st_status st_ring_bwd(const st_ring_desc* d, const st_tensor* q, const st_tensor* d_o, const st_tensor* o,
                      int32_t o_dtype, const float* lse_final, const int32_t* order, int32_t n_visit, int32_t mode,
                      float* dq_acc, float* const* dk_acc, float* const* dv_acc, void* workspace,
                      size_t workspace_bytes, void* hip_stream) {
  return st_ring_bwd_last(d, q, d_o, o, o_dtype, lse_final, order, n_visit, mode, dq_acc, dk_acc, dv_acc, 0, nullptr,
                          nullptr, workspace, workspace_bytes, hip_stream);
}

st_status st_ring_bwd_noalloc(const st_ring_desc* d, const st_tensor* q, const st_tensor* d_o, const st_tensor* o,
                              int32_t o_dtype, const float* lse_final, const int32_t* order, int32_t n_visit,
                              int32_t mode, float* dq_acc, float* const* dk_acc, float* const* dv_acc, void* hip_stream) {
  if (d == nullptr) return fail(ST_ERR_INVALID_ARG, "null descriptor");
  ST_TRY(check_shape(d->dtype, d->B, d->Hq, d->Hkv, d->D, d->Sq, d->Sk));
  const size_t need = bwd_base_bytes(d);               // partial sums have their own array
  if (need > kScratchBytes)
    return fail(ST_ERR_WORKSPACE, "st_ring_bwd_noalloc: this share needs %zu bytes of scratch, the library's static scratch holds %zu; use st_ring_bwd with a workspace", need, kScratchBytes);
  void *ws = nullptr, *parts = nullptr;
  ST_TRY(scratch_of_current_device(&ws, &parts));
  return ring_bwd(d, q, d_o, o, o_dtype, lse_final, order, n_visit, mode, dq_acc, dk_acc, dv_acc, 0, nullptr, nullptr, ws, kScratchBytes,
                  parts, kRoomMost, hip_stream);
}

size_t st_ring_bwd_noalloc_max_bytes(void) { return kScratchBytes; }

st_status st_ring_bwd_last(const st_ring_desc* d, const st_tensor* q, const st_tensor* d_o, const st_tensor* o,
                           int32_t o_dtype, const float* lse_final, const int32_t* order, int32_t n_visit,
                           int32_t mode, float* dq_acc, float* const* dk_acc, float* const* dv_acc, int32_t kv_flags,
                           void* const* dk_lowp, void* const* dv_lowp, void* workspace, size_t workspace_bytes,
                           void* hip_stream) {
  // partial sums: what the workspace has beyond the rest
  const size_t room = d == nullptr || workspace == nullptr ? 0 : ring_room(d, workspace_bytes);
  return ring_bwd(d, q, d_o, o, o_dtype, lse_final, order, n_visit, mode, dq_acc, dk_acc, dv_acc, kv_flags, dk_lowp, dv_lowp, workspace,
                  workspace_bytes, room > 0 ? (char*)workspace + bwd_base_bytes(d) : nullptr, room, hip_stream);
}

}  // extern "C"

static st_status ring_bwd(const st_ring_desc* d, const st_tensor* q, const st_tensor* d_o, const st_tensor* o, int32_t o_dtype,
                          const float* lse_final, const int32_t* order, int32_t n_visit, int32_t mode, float* dq_acc, float* const* dk_acc,
                          float* const* dv_acc, int32_t kv_flags, void* const* dk_lowp, void* const* dv_lowp, void* workspace,
                          size_t workspace_bytes, void* parts, size_t parts_bytes, void* hip_stream) {
  ST_TRY(check_ring(d, q, order, n_visit));
  if (mode != ST_RING_STEPWISE && mode != ST_RING_FUSED) return fail(ST_ERR_INVALID_ARG, "unknown mode %d", mode);
  if (o_dtype != ST_F32 && o_dtype != d->dtype) return fail(ST_ERR_INVALID_ARG, "o_dtype must be ST_F32 or the storage dtype");
  const int64_t n_o = (int64_t)d->B * d->Sq * d->Hq * d->D, n_kv = (int64_t)d->B * d->Sk * d->Hkv * d->D;
  ST_TRY(check_tensor("d_o", d_o, d->dtype, n_o));
  ST_TRY(check_tensor("o", o, o_dtype, n_o));
  ST_TRY(check_f32("lse_final", lse_final, n_o));
  ST_TRY(check_f32("dq_acc", dq_acc, n_o));
  if (n_visit > 0 && (!dk_acc || !dv_acc)) return fail(ST_ERR_INVALID_ARG, "null gradient tables");
  if (kv_flags & ~ST_KV_ASSIGN) return fail(ST_ERR_INVALID_ARG, "unknown kv_flags %d", kv_flags);
  if ((dk_lowp == nullptr) != (dv_lowp == nullptr)) return fail(ST_ERR_INVALID_ARG, "dk_lowp and dv_lowp: both or neither");
  if (dk_lowp && d->dtype != ST_BF16) return fail(ST_ERR_UNSUPPORTED, "bf16 copies of dK / dV need an ST_BF16 descriptor");
  const bool assign = (kv_flags & ST_KV_ASSIGN) != 0;
  const bool no_rows = n_o == 0;                     // no query rows: every contribution is zero
  if (no_rows && !assign && !dk_lowp) return ST_OK;
  if (!no_rows) {
    // without room for the partial sums of the dQ pass it runs on fewer workgroups
    if (workspace == nullptr || workspace_bytes < bwd_base_bytes(d)) return fail(ST_ERR_WORKSPACE, "backward workspace needs %zu bytes", st_ring_workspace_bytes(d, mode, 1));
    if (reinterpret_cast<uintptr_t>(workspace) % 256) return fail(ST_ERR_ALIGNMENT, "workspace: not 256-byte aligned");
  }
  hipStream_t stream = (hipStream_t)hip_stream;
  auto unseen = [&](int j) { return no_rows || chunk_invisible(d, j); };

  // Listed chunks that nobody sees contribute zero, but may have to be assigned or rounded: in one launch with the others
  // (their key tiles find no query block), or by launches of their own where every chunk has its own (step-wise), and where
  // there are no query rows at all.
  const bool hidden_too = mode == ST_RING_FUSED && d->dtype == ST_BF16 && !no_rows && n_kv > 0;
  RingVisit vis;
  for (int x = 0; x < n_visit; ++x) {
    const int j = order[x];
    void* lk = dk_lowp ? dk_lowp[j] : nullptr;
    void* lv = dk_lowp ? dv_lowp[j] : nullptr;
    if ((lk == nullptr) != (lv == nullptr)) return fail(ST_ERR_INVALID_ARG, "dk_lowp[%d] and dv_lowp[%d]: both or neither", j, j);
    if (lk && (reinterpret_cast<uintptr_t>(lk) % 16 || reinterpret_cast<uintptr_t>(lv) % 16))
      return fail(ST_ERR_ALIGNMENT, "dk_lowp[%d] / dv_lowp[%d]: not 16-byte aligned", j, j);
    const bool hidden = unseen(j);
    if (!hidden || assign || lk) {
      ST_TRY(check_f32("dk_acc[j]", dk_acc[j], n_kv));
      ST_TRY(check_f32("dv_acc[j]", dv_acc[j], n_kv));
    }
    if (!hidden || (hidden_too && (assign || lk))) vis.add(d, j);
  }
  if (!hidden_too && n_kv > 0 && (assign || dk_lowp)) {
    st::KvTables h;                                  // of the hidden chunks, as many as one launch takes
    int cnt = 0;
    for (int x = 0; x <= n_visit; ++x) {
      if (cnt == st::kMaxTable || (x == n_visit && cnt > 0)) {
        ST_HIP(st::launch_hidden_kv(h, cnt, assign, n_kv, stream), "hidden chunks");
        cnt = 0;
      }
      if (x == n_visit || !unseen(order[x])) continue;
      const int j = order[x];
      void *lk = dk_lowp ? dk_lowp[j] : nullptr, *lv = dk_lowp ? dv_lowp[j] : nullptr;
      if (!assign && !lk) continue;
      h.dk[cnt] = dk_acc[j]; h.dv[cnt] = dv_acc[j]; h.dk_lowp[cnt] = lk; h.dv_lowp[cnt] = lv;
      ++cnt;
    }
  }
  if (no_rows) return ST_OK;

  float* delta = (float*)workspace;
  st::BwdArgs a;
  memset(&a, 0, sizeof(a));
  a.s = shape_of(d);
  a.q = view_of(q);
  a.d_o = view_of(d_o);
  set_table_strides(a.t, d);
  a.lse = lse_final; a.delta = delta; a.dq = dq_acc;
  a.queue = (int32_t*)((char*)workspace + align_up((size_t)d->B * d->Sq * d->Hq * sizeof(float), 256));
  const int per_launch = mode == ST_RING_FUSED ? st::kMaxTable : 1;
  const bool provided = vis.provided(d, mode);
  void* const qs = (char*)a.queue + align_up(st::kQueueInts * sizeof(int32_t), 256);
  a.qs = d->dtype == ST_BF16 ? qs : nullptr;
  const bool one = d->dtype == ST_BF16 && one_strides(d) && st::one_fast_usable(a);
  for (int x0 = 0; x0 == 0 || x0 < vis.n; x0 += per_launch) {
    const int cnt = std::min(vis.n - x0, per_launch);
    a.t.n = cnt;
    a.queue_clean = d->dtype == ST_BF16 && x0 == 0;
    for (int x = 0; x < cnt; ++x) {
      const int j = vis.chunk[x0 + x];
      a.t.k[x] = d->k_ptr[j]; a.t.v[x] = d->v_ptr[j]; a.t.k_offset[x] = d->k_offset[j];
      a.dk[x] = dk_acc[j]; a.dv[x] = dv_acc[j];
      a.dk_lowp[x] = dk_lowp ? dk_lowp[j] : nullptr;
      a.dv_lowp[x] = dk_lowp ? dv_lowp[j] : nullptr;
    }
    if (cnt > 0) set_splits(a, ring_plan(d, mode, a.t.k_offset, cnt, provided, parts_bytes, one), parts);
    if (x0 == 0) {
      if (d->dtype == ST_BF16) {
        const st::OneReset reset = a.one_heads > 0 ? st::one_reset(a.parts, a.s, cnt, a.one_heads) : st::OneReset();
        ST_HIP(st::launch_bwd_prep(a.d_o, view_of(o), o_dtype, a.q, delta, qs, a.queue, reset, d->B, d->Sq, d->Hq, d->D, d->scale, stream), "backward preparation launch");
      } else {
        ST_HIP(st::launch_delta(a.d_o, d->dtype, view_of(o), o_dtype, delta, d->B, d->Sq, d->Hq, d->D, stream), "delta launch");
      }
      if (cnt <= 0) break;
    }
    a.kv_assign = assign ? ~0ull : 0ull;
    if (d->dtype != ST_BF16 && assign)              // the fp32 kernels only add
      for (int x = 0; x < cnt; ++x) {
        ST_HIP(st::launch_zero(a.dk[x], n_kv * (int64_t)sizeof(float), stream), "dk_acc fill");
        ST_HIP(st::launch_zero(a.dv[x], n_kv * (int64_t)sizeof(float), stream), "dv_acc fill");
      }
    ST_HIP(launch_bwd(d->dtype, a, stream), "backward launch");
  }
  return ST_OK;
}

extern "C" int st_testing_bwd_plan(const st_ring_desc* d, const int32_t* order, int32_t n_visit, int32_t mode, int32_t assign,
                                   int64_t workspace_bytes, int64_t* out, int32_t max_out) {
  if (check_shape(d->dtype, d->B, d->Hq, d->Hkv, d->D, d->Sq, d->Sk) != ST_OK || d->n_chunks < 1 || d->n_chunks > ST_MAX_CHUNKS) return -1;
  RingVisit vis;
  for (int x = 0; x < n_visit; ++x)
    if (!chunk_invisible(d, order[x]) || (assign && mode == ST_RING_FUSED && d->dtype == ST_BF16)) vis.add(d, order[x]);
  const size_t base = mode < 0 ? align_up((size_t)d->B * d->Sq * d->Hq * d->D * 2, 256) : bwd_base_bytes(d);
  const size_t most = mode < 0 ? kPartsMost : room_most(d), room = workspace_bytes < 0 ? most : (size_t)workspace_bytes > base ? std::min((size_t)workspace_bytes - base, most) : 0;
  const int per_launch = mode == ST_RING_FUSED ? st::kMaxTable : 1;
  int written = 0;
  for (int x0 = 0; x0 < vis.n; x0 += per_launch) {
    int64_t k_offset[st::kMaxTable];
    const int cnt = std::min(vis.n - x0, per_launch);
    for (int x = 0; x < cnt; ++x) k_offset[x] = d->k_offset[vis.chunk[x0 + x]];
    const BwdSplit p = mode < 0 ? block_plan(shape_of(d), d->dtype, k_offset[0], room) : ring_plan(d, mode, k_offset, cnt, vis.provided(d, mode), room, one_strides(d));
    const int64_t v[] = {cnt, p.dq.n, p.dq.total, p.dq.own0, (int64_t)p.dq.less1[0], (int64_t)p.dq.less1[1], (int64_t)p.dq.less1[2],
                         (int64_t)p.dq.less1[3], p.kv_each, p.one_heads > 0 ? -p.one_heads : p.kv_items, p.pair, (int64_t)p.bytes};
    for (int64_t y : v) {
      if (written >= max_out) return -1;
      out[written++] = y;
    }
  }
  return written;
}
