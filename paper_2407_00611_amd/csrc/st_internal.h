// Internal launch interface between the C-ABI layer (st_api.cpp) and the HIP kernels.
// Plain structs passed BY VALUE as kernel arguments: no device-side tables to allocate or copy.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/startrail.h"

namespace st {

constexpr int kMaxTable = 64;   // chunks one kernel launch can walk (fits the 4 KiB kernel-argument space)

struct View {                   // [B, S, heads, D] view, element strides, D contiguous
  const void* ptr;
  int64_t sb, ss, sh;
};

struct Shape {
  int32_t B, Hq, Hkv, D, Sq, Sk;
  int64_t q_offset;   // global position of query row 0
  int32_t causal;
  float scale;
  int32_t q_seg;      // 0: one run of rows; > 0: rows [q_seg, Sq) are a second run that starts at q_offset2
  int64_t q_offset2;  //    (two half-shards of a load-balanced causal placement); positions rise with the row
};

// Global position of query row i.
__host__ __device__ inline int64_t q_pos(const Shape& s, int i) {
  return (s.q_seg > 0 && i >= s.q_seg) ? s.q_offset2 + (i - s.q_seg) : s.q_offset + i;
}
// Smallest row index whose position is >= p: under a causal mask row i sees a key at p iff i >= q_row_of(p).
// Sq if no row does.
__host__ __device__ inline int q_row_of(const Shape& s, int64_t p) {
  const int n0 = s.q_seg > 0 ? s.q_seg : s.Sq;
  int64_t i = p - s.q_offset;
  if (i < n0) return i < 0 ? 0 : (int)i;
  if (s.q_seg <= 0) return s.Sq;
  i = p - s.q_offset2;
  if (i < 0) i = 0;
  return i >= s.Sq - n0 ? s.Sq : n0 + (int)i;
}

// Chunks in visit order.  k/v are base pointers of [B,Sk,Hkv,D] views that share one stride set.
struct ChunkTable {
  int32_t n;
  const void* k[kMaxTable];
  const void* v[kMaxTable];
  int64_t k_offset[kMaxTable];
  int64_t ksb, kss, ksh, vsb, vss, vsh;
};

// The query tiles of a head, `rows` rows each but for the last one; where n_lo > 0 the two runs of rows have tiles of their own,
// n_lo of them the first run.
struct QueryTiles {
  int32_t rows, Sq, seg, n_lo;
  __host__ __device__ int count() const { return n_lo > 0 ? n_lo + (Sq - seg + rows - 1) / rows : (Sq + rows - 1) / rows; }
  __host__ __device__ int row0(int qt) const { return n_lo > 0 && qt >= n_lo ? seg + (qt - n_lo) * rows : qt * rows; }
  __host__ __device__ int rows_of(int qt) const {
    const int left = (n_lo > 0 && qt < n_lo ? seg : Sq) - row0(qt);
    return left < rows ? left : rows;
  }
  __host__ __device__ int tile_of(int row) const {     // rows is a power of two
    const int shift = 31 - __builtin_clz((unsigned)rows);
    return n_lo > 0 && row >= seg ? n_lo + ((row - seg) >> shift) : row >> shift;
  }
};
// of the hand-scheduled kernels (kQTileFastRows) and the fp32 ones (32 rows).  Under a causal mask a 256-row tile with rows of
// both runs would walk what the second run sees with masks all the way: a masked tile takes 1.4 (dQ) to 2 times a whole one (64
// workgroups of 128 tiles, head size 128: forward 142 us whole and 266 masked, dQ 198 and 275).
constexpr int kQTileFastRows = 256;
__host__ __device__ inline QueryTiles query_tiles(const Shape& s, int rows) {
  return QueryTiles{rows, s.Sq, s.q_seg, s.causal && s.q_seg % rows && rows == kQTileFastRows ? (s.q_seg + rows - 1) / rows : 0};
}

// Under-filled launches of the query-stationary kernels: workgroups per query tile, each with a share of the tile's walk.
// Every tile has n of them (total == 0; grid (tiles, n)), or, where a causal mask makes the walks of the tiles differ, tile qt
// has its own number, at most n (total > 0: their sum over the tiles of a head; grid (heads * total)).  n <= 1: no tile is split.
constexpr int kShareTiles = 64;      // tiles per head such a table has room for
struct TileShares {
  int16_t n, total;
  int16_t own0;        // dQ only, 1: the first share of a split tile adds to dq itself instead of storing a partial sum
  uint64_t less1[kShareTiles / 16];   // shares less one of tile qt: bits 4 (qt % 16) of word qt / 16
};
// (the words are picked by selects, so that a kernel reads all of them at once with its other arguments, which come from host
// memory, and not one after the other)
__host__ __device__ inline int shares_of(const TileShares& t, int qt) {
  if (t.total <= 0) return t.n;
  uint64_t w = t.less1[0];
  for (int x = 1; x < kShareTiles / 16; ++x) w = (qt >> 4) == x ? t.less1[x] : w;
  return (int)(w >> (4 * (qt & 15)) & 15) + 1;
}
// partial sums the tiles before qt store (see BwdArgs::shares): n - own0 each for n > 1 shares
__host__ __device__ inline int parts_before(const TileShares& t, int qt) {
  if (t.n <= 1) return 0;
  if (t.total <= 0) return qt * (t.n - t.own0);
  int sum = 0;
  for (int x = 0; x < kShareTiles / 16; ++x) {
    const int k = qt - 16 * x;                         // tiles of this word
    const uint64_t m = k <= 0 ? 0 : k >= 16 ? t.less1[x] : t.less1[x] & (((uint64_t)1 << (4 * k)) - 1);
    const uint64_t low = 0x0f0f0f0f0f0f0f0full, pairs = (m & low) + (m >> 4 & low);      // at most 8 x 30 together
    const uint64_t split = (m | m >> 1 | m >> 2 | m >> 3) & 0x1111111111111111ull;
    sum += (int)(pairs * 0x0101010101010101ull >> 56) + (1 - t.own0) * __builtin_popcountll(split);
  }
  return sum;
}

struct FwdArgs {
  Shape s;
  View q;
  ChunkTable t;
  float* o;        // fp32 [B,Sq,Hq,D]
  float* lse;      // fp32 [B,Hq,Sq]
  void* o_lowp;    // nullable, [B,Sq,Hq,D] in the storage dtype
  // A split launch (shares.n > 1): share y of a split tile writes a partial state of its own at part_o + y * part_stride,
  // part_lse + y * part_stride (floats), the states are combined afterwards; tiles with one share write o, lse and o_lowp.
  TileShares shares;
  float *part_o, *part_lse;
  int64_t part_stride;
  float sum_limit;   // fast kernel: sum over a block's probabilities beyond which the lazy exponent reference moves (set by its launcher)
};

// Tile of the hand-scheduled dK/dV kernel
constexpr int kDkvFastKeys = 256;
constexpr int kDkvFastRows = 32;
// 32-row query blocks with a row that sees some key of key tile kt of a chunk at position k0: the last so many of the shard
__host__ __device__ inline int kv_blocks(const Shape& s, int64_t k0, int kt) {
  const int all = (s.Sq + kDkvFastRows - 1) / kDkvFastRows;
  const int first = s.causal ? q_row_of(s, k0 + (int64_t)kt * kDkvFastKeys) : 0;
  return first >= s.Sq ? 0 : all - first / kDkvFastRows;
}
constexpr int kKvSharesMost = 16;
// shares of a key tile that meets so many blocks (see BwdArgs::kv_each)
__host__ __device__ inline int kv_shares(int blocks, int each) {
  const int n = each > 0 ? (blocks + each - 1) / each : 1;
  return n < 1 ? 1 : n > kKvSharesMost ? kKvSharesMost : n;
}

// Runs of key tiles, in table order, that a workgroup finds its tile through without reading the chunks' positions (arguments are
// in host memory, and a load of them per lane takes 2 us of a launch that may be 20): all tiles of a run have the same
// number of shares, unless it is `mixed`.  The last run may hold anything.
struct KvSection {
  int32_t tiles, items;        // items: shares
  int32_t mixed;
};
constexpr int kKvSections = 5;

struct BwdArgs {
  Shape s;
  View q, d_o;
  const void* qs;      // bf16 path: Q' = bf16(Q * scale * log2 e), the exponent operand (see scale_bf16x8), dense
                       // [B,Sq,Hq,D], made by launch_scale_q; nullable: without it the key-stationary pass stays in
                       // the general kernel, which converts the rows it stages itself
  ChunkTable t;
  const float* lse;    // final
  const float* delta;
  float* dq;           // fp32 [B,Sq,Hq,D], +=
  float* dk[kMaxTable];  // fp32 [B,Sk,Hkv,D] per table entry, +=
  float* dv[kMaxTable];
  // Under-filled dQ launches of the hand-scheduled and of the fp32 kernel: a share of a split tile stores its sum, and the
  // launcher then adds the sums to dq in order.  Sum y of tile qt holds the tile's rows, dense as dq has them, behind those of
  // the tiles before it and of the shares before it (see dq_part).  Where the workspace has no room for all of them
  // (shares.own0) the first share adds to dq itself, and its reads end the launch 2 us later.
  TileShares shares;
  // Under-filled dK/dV launches likewise: kv_each > 0 splits the query blocks a key tile meets into shares of at most that many
  // (kv_shares).  The first share writes dk[c] / dv[c]; each other one stores its sums, dK and then dV of kDkvFastKeys rows of D
  // floats, in a slot of kv_parts: slots are numbered through the tiles of a head (kt fastest), a head's behind another's; the
  // launcher adds them up (and rounds) in order.  kv_items: shares of a head, kv_sec: where they are (both set by the launcher).
  // The fp32 kernels: kv_items shares of every key tile (0: one), sums as f32_kv_part says.
  int32_t kv_each, kv_items;
  KvSection kv_sec[kKvSections];
  int32_t kv_same;     // shares of every tile where all have the same number (then nothing is looked up), else 0; set by the launcher
  int32_t pair;        // 1: both passes in one launch, where the hand-scheduled kernels take both
  int32_t one_heads;   // > 0: all gradients in one walk (see OneRoom), batches of so many KV heads; parts is its room
  int32_t one_polls;   // most polls of a wait there; set by the launcher
  float *parts, *kv_parts;   // of launches that run one after the other they may be the same memory
  // dK / dV work of a chunk's last visit folded into the launch (bf16 path): the hand-scheduled kernel's epilogue does it,
  // beside the general kernel the launcher runs fill and cast launches
  uint64_t kv_assign;          // bit c: dk[c] / dv[c] are overwritten, not added to
  void* dk_lowp[kMaxTable];    // nullable per entry: the final dk[c] / dv[c] rounded to bf16, dense [B,Sk,Hkv,D]
  void* dv_lowp[kMaxTable];
  int32_t* queue;      // nullable, kQueueInts ints of device memory: the fast dK/dV kernel hands its key tiles out
                       // through it (one counter per XCD), so that XCDs that run faster take more of them
  int16_t queue_clean; // 1: the counters are zero already, and the room of a walk of one is reset (the first launch behind launch_bwd_prep)
  int16_t queue_xcds;  // counters in use (the device's XCD count, 1 .. 8); set by the launcher
};
// Partial sum y of query tile qt of batch entry b: [row, head, element] floats from here on.  The sums of a batch entry lie one
// behind the other; dq_part_rows are the rows before that of tile qt.
__host__ __device__ inline int64_t dq_part_rows(const QueryTiles& q, const TileShares& t, int qt) {
  // every tile before qt as a full one, less what the last tile of the first run lacks
  int64_t rows = (int64_t)parts_before(t, qt) * q.rows;
  if (q.n_lo > 0 && qt >= q.n_lo) {
    const int n = shares_of(t, q.n_lo - 1);
    rows -= (int64_t)(n > 1 ? n - t.own0 : 0) * (q.n_lo * q.rows - q.seg);
  }
  return rows;
}
__host__ __device__ inline int64_t dq_part_rows_all(const QueryTiles& q, const TileShares& t) {
  const int last = q.count() - 1, n = shares_of(t, last);
  return dq_part_rows(q, t, last) + (int64_t)(t.n > 1 && n > 1 ? n - t.own0 : 0) * q.rows_of(last);
}
__host__ __device__ inline float* dq_part(float* parts, const Shape& s, const QueryTiles& q, const TileShares& t, int b, int qt, int y) {
  return parts + (b * dq_part_rows_all(q, t) + dq_part_rows(q, t, qt) + (int64_t)y * q.rows_of(qt)) * s.Hq * s.D;
}
// fp32: sum of share `y` >= 1 of chunk c, laid out as dk[c] (w = 0) and dv[c] (1)
__host__ __device__ inline int64_t f32_kv_floats(const Shape& s) { return ((int64_t)s.B * s.Sk * s.Hkv * s.D + 63) / 64 * 64; }
__host__ __device__ inline float* f32_kv_part(float* parts, const Shape& s, int n_chunks, int y, int c, int w) {
  return parts + ((int64_t)(y - 1) * n_chunks + c) * 2 * f32_kv_floats(s) + w * f32_kv_floats(s);
}
// bf16: a slot of a key tile's sums, dk behind dv (not a multiple of a large power of two: workgroups in step would write to the
// same memory channels)
__host__ __device__ inline int64_t kv_slot_floats(const Shape& s) { return (int64_t)2 * kDkvFastKeys * s.D + 17 * 64; }
// Room of a backward in one walk (gen_bwd_one_asm.py), byte offsets: what hands out the tiles (tickets of 16 XCDs and the next batch, 128
// bytes apart, claims), a count that is never too low, a word that is set when a wait gives up, the tiles' counts (one per wavefront), a
// pair of zeros, and the pairs of each (KV head, batch entry) in the order of the walk behind two that do not exist.
__host__ __device__ constexpr int one_pair_bytes(int d) { return 32 * d * 4; }
struct OneRoom {
  int64_t plenty, gave_up, claims, counts, zeros, pairs, group_bytes, bytes;
  int32_t claims_each, tiles;
  __host__ __device__ OneRoom(const Shape& s, int n_chunks, int heads) {
    const int64_t groups = (int64_t)s.B * s.Hkv, blocks = (s.Sq + 31) / 32;
    tiles = (s.Sk + kDkvFastKeys - 1) / kDkvFastKeys * n_chunks;
    plenty = 17 * 128;
    gave_up = plenty + 64;                             // (GAVE_UP in gen_bwd_one_asm.py)
    claims = 18 * 128;
    claims_each = (int32_t)((groups / heads + 256 + 31) / 32 * 32);      // (a workgroup that finds no batch left has taken a ticket too)
    counts = claims + (int64_t)16 * claims_each * 4;
    zeros = counts + (groups * tiles * 4 * 4 + 255) / 256 * 256;
    pairs = zeros + one_pair_bytes(s.D);
    group_bytes = (s.Hq / s.Hkv * blocks + 2) * one_pair_bytes(s.D);
    bytes = pairs + groups * group_bytes;
  }
};
constexpr int kQueueInts = 8 * 32;   // at most 8 counters, 128 bytes apart
// passed by value: a kernel takes 4096 bytes of arguments
static_assert(sizeof(BwdArgs) <= 4096 - 64 && sizeof(FwdArgs) <= 4096 - 64, "argument structs must fit the kernel arguments");

// n partial states of the same query rows (each O fp32 [B,Sq_in,Hq,D], lse fp32 [B,Hq,Sq_in]) and the run of
// rows [row0, row0 + Sq_out) the combined state keeps.
struct CombineArgs {
  int32_t n;
  const float* o[kMaxTable];
  const float* lse[kMaxTable];
  int32_t B, Sq_in, Hq, D, row0, Sq_out;
  float* o_out;      // fp32 [B,Sq_out,Hq,D]
  float* lse_out;    // fp32 [B,Hq,Sq_out]
  void* o_lowp;      // nullable, [B,Sq_out,Hq,D]
  // The states of a split forward (shares.n > 1; row0 = 0, Sq_out = Sq_in): only the first shares_of(tile) of them hold rows of
  // a tile, and the rows of a tile with one share are not combined.
  TileShares shares;
  QueryTiles tiles;
};

// Tuning and testing switches of the launchers.  The defaults are the product.  They are read from the
// environment ONCE, when the library is loaded (ST_FWD_FAST, ST_DQ_FAST, ST_DKV_FAST, ST_DKV_QUEUE, ST_ONE_WALK, ST_FWD_WQ,
// ST_FWD_PIPE, ST_FWD_GAP); afterwards only st_testing_set() changes them, an exported entry point for the
// library's own tests that the public header does not declare.  No launcher reads the environment.
struct Knobs {
  int fwd_fast = 1;    // 0: the forward stays in the general kernels
  int dq_fast = 1;     // 0: the dQ pass stays in the general kernel
  int dkv_fast = 1;    // 0: the dK/dV pass stays in the general kernel
  int dkv_queue = 1;   // 0: every dK/dV key tile is a workgroup of its own (no tile queue)
  int one_polls = 1 << 21;   // ring backward in one walk: most polls of a wait (about a microsecond each)
  int one_walk = 1;    // ring backward, all gradients in one walk: 0 never, 1 where it is the faster plan, 2 wherever the kernel takes it
  int one_heads = 0;   // KV heads of its batches: 0 as planned, 1 .. 8 so many where they divide the heads
  int fwd_wq = 32;     // general forward without the fast path: queries per wavefront (32 or 64)
  int fwd_pipe = 1;    // general forward without the fast path, head size 128: the pipelined variant
  float fwd_gap = 8.f; // fast forward: log2 units every block maximum may exceed the lazy exponent reference by (0 .. 64)
};
Knobs& knobs();

// Facts about a device that the launchers need, queried once per device and cached.
constexpr int kMaxXcds = 8;
struct DeviceInfo {
  int cus = 0;         // compute units
  int xcds = kMaxXcds; // accelerator complex dies (each with its own L2); kMaxXcds when the runtime does not tell
};
const DeviceInfo& device_info();   // of the current device

// Optional per-kernel timing (st_profile_begin / st_profile_end): while enabled, a ProfScope
// records a HIP event on the launch stream before and after the kernel it brackets.
struct ProfScope {
  ProfScope(const char* name, hipStream_t s);
  ~ProfScope();
  int slot;
  hipStream_t stream;
};

// Keys of a tile of the hand-scheduled query-stationary kernels (forward, dQ); its rows are kQTileFastRows
constexpr int kQTileFastKeys = 64;
constexpr int kDqFastRows = kQTileFastRows;
constexpr int kDqFastKeys = kQTileFastKeys;

// A dQ walk of a few tiles ends before the hand-scheduled loop has made up for its prologue (head size 128: one 64-key tile
// 14.1 against 10.5 us on the general kernel, five 26.9 against 20.9, eight 23.2 against 23.7, 64 tiles 106 against 137;
// head size 64: 11.2 against 8.7, 17.7 against 15.3, 15.6 against 17.7, 61 against 94): unless it is split it stays there, and
// out of the launch that holds both passes.
inline bool dq_few(const Shape& s, int n) { return (int64_t)n * ((s.Sk + kDqFastKeys - 1) / kDqFastKeys) <= 6; }

// ---- launchers (each returns hipGetLastError() after the launch) ----
hipError_t launch_fwd_f32(const FwdArgs& a, hipStream_t s);
hipError_t launch_bwd_f32(const BwdArgs& a, hipStream_t s);
hipError_t launch_fwd_bf16(const FwdArgs& a, hipStream_t s);
bool fwd_fast_usable(const FwdArgs& a);
hipError_t launch_fwd_fast(const FwdArgs& a, hipStream_t s);
hipError_t launch_bwd_bf16(const BwdArgs& a, hipStream_t s);
bool dkv_fast_usable(const BwdArgs& a);
void kv_sections(BwdArgs& a);    // sets kv_items and kv_sec from the table and kv_each
hipError_t launch_bwd_dkv_fast(const BwdArgs& a, hipStream_t s);
hipError_t launch_bwd_pair_fast(const BwdArgs& a, hipStream_t s);   // both
hipError_t launch_bwd_one_fast(const BwdArgs& a, hipStream_t s);    // all three gradients in one walk
bool dq_fast_usable(const BwdArgs& a);
hipError_t launch_bwd_dq_fast(const BwdArgs& a, hipStream_t s);

hipError_t launch_merge(float* o_acc, float* lse_acc, const float* o_part, const float* lse_part,
                        int32_t B, int32_t Sq, int32_t Hq, int32_t D, void* o_lowp, int lowp_dtype,
                        hipStream_t s);
hipError_t launch_combine(const CombineArgs& a, int lowp_dtype, hipStream_t s);
hipError_t launch_delta(const View& d_o, int d_o_dtype, const View& o, int o_dtype, float* delta,
                        int32_t B, int32_t Sq, int32_t Hq, int32_t D, hipStream_t s);
// What a walk of one finds in its room when it starts (OneRoom): zeros up to the pairs, and the count that is never too low
struct OneReset {
  uint4* zero = nullptr;
  int32_t n = 0;             // 16-byte units
  int32_t plenty = 0;        // the unit whose first word is that count
};
OneReset one_reset(void* room, const Shape& s, int n_chunks, int heads);
hipError_t launch_one_reset(const OneReset& r, hipStream_t s);
bool one_fast_usable(const BwdArgs& a);
// bf16 backward, head size 64 or 128: delta = rowsum(dO o O), qs as launch_scale_q, queue (kQueueInts ints) to zero, reset done
hipError_t launch_bwd_prep(const View& d_o, const View& o, int o_dtype, const View& q, float* delta, void* qs, int32_t* queue,
                           const OneReset& reset, int32_t B, int32_t Sq, int32_t Hq, int32_t D, float scale, hipStream_t s);
hipError_t launch_cast(const float* src, void* dst, int64_t n, int dst_dtype, hipStream_t s);
// dst (dense bf16 [B,Sq,Hq,D]) = bf16(q * scale * log2 e) of a bf16 view q
hipError_t launch_scale_q(const View& q, void* dst, int32_t B, int32_t Sq, int32_t Hq, int32_t D, float scale, hipStream_t s);
// dk[c] += its partial sums (see BwdArgs::kv_each) in order, likewise dv[c]; rounded to dk_lowp[c] / dv_lowp[c] where given
hipError_t launch_add_kv_parts(const BwdArgs& a, hipStream_t s);
hipError_t launch_add_kv_parts_f32(const BwdArgs& a, hipStream_t s);
// dq += its partial sums (see BwdArgs::shares) in order; `rows` rows per query tile
hipError_t launch_add_parts(const BwdArgs& a, int rows, hipStream_t s);
// gradients of chunks that no row sees: set to zero (assign), and rounded to bf16 where a copy is asked for
struct KvTables {
  float *dk[kMaxTable], *dv[kMaxTable];
  void *dk_lowp[kMaxTable], *dv_lowp[kMaxTable];
};
hipError_t launch_hidden_kv(const KvTables& t, int n, bool assign, int64_t n_kv, hipStream_t s);
hipError_t launch_fill_state(float* o, float* lse, int64_t n_o, int64_t n_lse, hipStream_t s);
hipError_t launch_zero(void* dst, int64_t bytes, hipStream_t s);   // bytes % 4 == 0, dst 4-byte aligned
// benchmark aid: MFMA-only loop, one workgroup per compute unit (see st_probe.hip)
int mfma_probe_blocks();
int mfma_probe_mixes();                              // side-instruction mixes 1 .. mfma_probe_mixes(); 0 = MFMAs only
const char* mfma_probe_mix_name(int mix);
double mfma_probe_flop(int blocks, int mix, int32_t iters);
hipError_t launch_mfma_probe(const void* operands, int64_t operand_bytes, int mix, int32_t iters, float* sink, int blocks,
                             hipStream_t s);

}  // namespace st
