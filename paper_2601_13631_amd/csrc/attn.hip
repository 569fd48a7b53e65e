// attn.hip -- Re-Prefill sparse attention (Def. 2.1) for gfx950, bf16.
//
// For query t of head h (KV head g = h / G) the keys are the tokens of the k
// kept chunks (compact positions 0 .. k*c-1; rows past n of a short last chunk
// are masked) followed by the suffix tokens 0..t (causal).
//
// Rows of one KV head are r = t*G + i (query t, head g*G + i), so the G query
// heads that share a KV head share every K/V tile.  A workgroup owns 128 rows
// (4 waves x 32) and one contiguous slice ("split") of the key positions.  At
// its start it resolves the slice in units of min(c, 32) keys to source rows
// (the prefix K/V source or the suffix) in LDS.  Per 64-key stage, in two halves
// of 32 keys:
//   S^T = K Q^T   bf16 MFMA 32x32x16, A = K rows from LDS, B = Q^T in
//                 registers: every lane owns one query row and 16 keys;
//   numerators    exp2 in fp32 (sm_scale*log2 e folded in) against a fixed
//                 reference per row: the maximum over the slice's first 32
//                 keys (64 where it is the row's only slice).  A slice whose
//                 sums or outputs then leave a guard (or that had no
//                 reference) is done again against its own maximum, so that
//                 the guess decides no more than roundings;
//   O^T += V^T P^T  A = V^T read from LDS with the transposing
//                 ds_read_b64_tr_b16, B = P^T straight from the softmax
//                 registers.
// The K operand rows are loaded in a permuted order so that the registers a
// lane holds after the first product are exactly the 8 consecutive keys the
// second product needs from it -- no register shuffles between the two.
// Splits write their partial output O in half precision with an exponent per row,
// and (reference, l) in fp32; a combine kernel merges them in split order
// (deterministic).
//
// What bounds it: the matrix cores (32 MFMAs of 32 cycles per wave and stage at
// D = 128), the numerators' VALU work (112 instructions, the exponentials 8.6
// cycles each) and the LDS reads (32 KB per wave and stage, 128 bytes a cycle
// per CU) would each take about half of a stage's time, so they have to run side
// by side.  Hence the runs of the stage loop below, K/V rows that go straight
// from memory to LDS, and no running maximum (a chain from the MFMAs through the
// maximum to the exponentials).  Measured against a loop with the running
// maximum, register staging and operands read right before their MFMA, at 1.85
// GHz (what the chip holds under this load): 32K layer 27 -> 24 us, 64K layer
// 154 -> 119 us, 128K layer 367 -> 286 us, 8,000 of 16,000 tokens with 512
// queries and 32 heads, with their combine, 103 -> 75 us (920 TFLOP/s).  Not
// faster: 64 rows per wave (half the LDS reads, one wave per SIMD: 3,350 cycles per
// stage and 64 rows, two waves of 32 rows 3,440), and a loop that spreads the
// numerators over all 32 MFMAs by running a product of the next stage early (128K
// 295 against 302 us of the loop below, small grids 10% slower for its longer
// prologue).
//
// A slice that is done again costs its workgroup a pass over its K rows and a second
// pass of everything.  With every slice done again (in each 64 keys one 130 log2
// units above the others): 32K layer 31 -> 48 us, 64K 113 -> 262, 8K 11.5 -> 19.2,
// 8,000 tokens x 32 heads 79 -> 173; a running maximum took 32, 139, 12.0 and 100 us
// on these inputs.  It takes a logit 120 log2 units (83 nats) above all of the slice's
// first keys, or outputs past fp32; up to there a low reference costs nothing.

#include <atomic>
#include <type_traits>
#include <utility>

#include "ckv_internal.h"

namespace ckv {
namespace {

std::atomic<int> g_force_wide{0};  // ckv_debug_attn_wide_addressing

constexpr int kWaves = 4;
constexpr int kWaveRows = 32;
constexpr int kBlockRows = kWaves * kWaveRows;  // 128
constexpr int kTile = 64;                       // keys per LDS stage
constexpr int kSub = 32;                        // keys per MFMA product
// A slice is done again when its sum of numerators passes kGuard (1 / sum stays a normal
// number below it), or lies below kGuardLow without a reference.
constexpr float kGuard = 0x1p120f, kGuardLow = 0x1p-64f;
// Unit tables: a slice's keys in units of min(c, 32) keys, each inside one chunk
// or inside the suffix (kc is a multiple of c).  base: the unit's first row in
// its source (a byte offset when every row of both sources lies below 4 GiB);
// valid: how many of its rows exist (fewer at the end of a short last chunk
// and of the suffix, none for an index that names no chunk).
constexpr int kMaxSliceUnits = 1536;  // 12 KiB of tables: two workgroups still share a CU's LDS
constexpr int kMaxSliceStages = 512;

// MFMA row p of the K operand holds key kappa(p); afterwards register v of a
// lane in half h holds key 16*(v/8) + 8*h + v%8.
__device__ __forceinline__ int kappa(int p) {
  const int i = p >> 3, h = (p >> 2) & 1, j = p & 3;
  return 16 * (i >> 1) + 8 * h + 4 * (i & 1) + j;
}

// LDS stages hold kTile rows of D bf16, unpadded (the direct-to-LDS loads write
// lane i's 16 bytes at base + 16 i), with the 16-byte segments of a row
// permuted by an XOR that depends on the row: segment s of row r sits at
// position s ^ swz(r).  K: any 16 consecutive MFMA rows (kappa) then read one
// segment column from all 64 banks.
template <int D>
__device__ __forceinline__ int k_swz(int row) {
  return D == 128 ? (row & 15) : ((row >> 1) & 7);
}

// V: conflict-free for the transposing reads.
template <int D>
__device__ __forceinline__ int v_swz(int row) {
  if constexpr (D == 128)
    return ((row & 1) ? 4 : 0) ^ ((row & 2) ? 10 : 0);
  else
    return ((row & 1) ? 2 : 0) ^ ((row & 2) ? 4 : 0);
}
template <int D>
__device__ __forceinline__ int v_off(int row, int seg) { return row * D + ((seg ^ v_swz<D>(row)) << 3); }

__device__ __forceinline__ float partner_f(float x) {
  int v = __float_as_int(x);
  auto r = __builtin_amdgcn_permlane32_swap(v, v, false, false);
  return __int_as_float(threadIdx.x & 32 ? r[0] : r[1]);
}

struct AttnArgs {
  const uint16_t* q;       // [S][Hq][D]
  const uint16_t* kbase;   // prefix chunks (see ChunkSource)
  const uint16_t* vbase;
  const int32_t* chunk_off;
  int32_t direct;
  int rows_per_slot;       // chunk slot stride of the source in rows of Hkv*D elements
  const int32_t* sel;      // [k]
  int kc;                  // k * c prefix positions (< 2^31)
  int64_t n, m;
  int c;
  int log2c;               // log2(c) when c is a power of two, else -1
  int log2u;               // log2 of the keys per unit: min(c, 32)
  const uint16_t* ks;      // [S][Hkv][D]
  const uint16_t* vs;
  uint16_t* out;           // [S][Hq][D]
  uint16_t* o_part;        // [splits][Hkv][R][D]: 2^-E O, fp16
  float2* ml_part;         // [splits][Hkv][R]: (reference, sum)
  int S, Hq, Hkv, G, R, n_splits, tiles_per_split, n_row_blocks;
  int partial;             // write split partials for a combine (else the output itself)
  int with_suffix;         // the keys end with the causal suffix (else prefix chunks only)
  float c1;
  uint32_t nblocks, nblocks_padded;
  uint32_t row_bytes;      // Hkv * D * 2: bytes between consecutive rows of a source
  int off32;               // every row of both sources lies below 4 GiB from its base
  uint32_t pre_bytes, suf_bytes;  // bytes of the prefix and suffix sources (when off32)
};

// Buffer resource over `bytes` bytes from p (raw loads; offsets past the end read 0).
__device__ __forceinline__ __amdgpu_buffer_rsrc_t raw_rsrc(const void* p, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), (short)0, (int)bytes, 0x00020000);
}

// Chunk of compact prefix position pos.
__device__ __forceinline__ int chunk_of(const AttnArgs& a, int pos) {
  return a.log2c >= 0 ? (pos >> a.log2c) : (int)((uint32_t)pos / (uint32_t)a.c);
}

// The unit that starts at compact position pos, in two steps so that a thread
// can issue its index loads before using any: unit_chunk fetches sel[u] (and the
// slot table entry) of its chunk u, unit_entry finishes.  Kept chunk u begins at
// source row slot*rows_per_slot, slot = chunk_off[u] (slot table), sel[u]
// (spans read in place) or u (compact copy).
__device__ __forceinline__ void unit_chunk(const AttnArgs& a, int pos, int& j, int& slot) {
  j = 0;
  slot = 0;
  if (pos < a.kc) {
    const int u = chunk_of(a, pos);
    j = a.sel[u];
    if (a.chunk_off) slot = a.chunk_off[u];
  }
}

__device__ __forceinline__ void unit_entry(const AttnArgs& a, int pos, int j, int slot_tab, int& row,
                                           int& valid) {
  const int size = 1 << a.log2u;
  row = 0;
  valid = 0;
  if (pos < a.kc) {
    const int u = chunk_of(a, pos);
    const int off = pos - u * a.c;
    if (j < 0 || (int64_t)j >= a.m) return;
    const int64_t left = a.n - ((int64_t)j * a.c + off);  // <= 0: past n in a short last chunk
    if (left <= 0) return;
    valid = (int)min<int64_t>(left, size);
    const int slot = a.chunk_off ? slot_tab : (a.direct ? j : u);
    row = slot * a.rows_per_slot + off;
  } else if (a.with_suffix && pos - a.kc < a.S) {
    row = pos - a.kc;
    valid = min(a.S - row, size);
  }
}

// Flags of a stage: bit 0, some row of the block must not see some of its keys;
// bits 1-2, its keys are 64 rows of the prefix source, 64 rows of the suffix
// source, or anything else.
constexpr int kStageMask = 1, kStagePrefix = 1 << 1, kStageSuffix = 2 << 1, kStageMixed = 3 << 1;

// The direct-to-LDS loads of one 64-key stage: instruction p of wave w moves
// the K (or V) rows of keys p*kKeyStep + w*kRowsPerLoad .. +kRowsPerLoad-1,
// kSegs lanes per row.
template <int D>
struct Stage {
  static constexpr int kSegs = D / 8;
  static constexpr int kRowsPerLoad = 64 / kSegs;
  static constexpr int kKeyStep = kWaves * kRowsPerLoad;
  static constexpr int kPer = kTile / kKeyStep;
};

using LdsPtr = __attribute__((address_space(3))) void*;

// 16 bytes per lane from memory to lds + 16 * lane (lds is uniform).  Buffer
// loads only: a global load to LDS counts as a FLAT access, after which the
// compiler no longer counts the LDS reads in flight and waits for all of them.
__device__ __forceinline__ void buffer_to_lds(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff,
                                              uint16_t* lds) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (LdsPtr)lds, 16, voff, soff, 0, 0);
}

// What the stage loads of one lane need: its first key of a stage, and the byte
// column of a K and of a V row it moves (which undoes the LDS permutation) plus
// the key's offset inside its unit.
struct LoadLane {
  int key0, kcol, vcol;
};

// Loads the K rows of the stage at position pos0 into dk and (kV) its V rows into
// dv.  base: the unit table entries of this lane's keys; bases/valids: the stage's
// unit tables.
// A stage of 64 rows of one source (the common case) goes through one buffer
// resource per tensor with 32-bit byte offsets.  Any other takes the lanes of
// the two sources in turn (a key without a row reads its unit's last, or suffix
// row 0; its weight is forced to 0), and with a source past 4 GiB a resource per
// group of 4 keys, which share a unit.
template <int D, bool kV = true>
__device__ __forceinline__ void stage_load(const AttnArgs& a, int flags, const int* base,
                                           const int* bases, const int* valids, int pos0, int wave,
                                           const LoadLane& ll, uint16_t* dk, uint16_t* dv) {
  using St = Stage<D>;
  const int umask = (1 << a.log2u) - 1;
  dk += wave * St::kRowsPerLoad * D;
  dv += wave * St::kRowsPerLoad * D;
  if (a.off32 && (flags & kStageMixed) != kStageMixed) {  // uniform
    const bool pre = flags & kStagePrefix;
    const uint32_t bytes = pre ? a.pre_bytes : a.suf_bytes;
    const __amdgpu_buffer_rsrc_t kr = raw_rsrc(pre ? a.kbase : a.ks, bytes);
    const __amdgpu_buffer_rsrc_t vr = raw_rsrc(pre ? a.vbase : a.vs, bytes);
#pragma unroll
    for (int p = 0; p < St::kPer; ++p) {
      const uint32_t soff = (p * St::kKeyStep & umask) * a.row_bytes;
      buffer_to_lds(kr, (uint32_t)base[p] + (uint32_t)ll.kcol, soff, dk + p * St::kKeyStep * D);
      if constexpr (kV)
        buffer_to_lds(vr, (uint32_t)base[p] + (uint32_t)ll.vcol, soff, dv + p * St::kKeyStep * D);
    }
    return;
  }
  int key0 = ll.key0, kcol = ll.kcol, vcol = ll.vcol;
  asm volatile("" : "+v"(kcol), "+v"(vcol), "+v"(key0), "+s"(wave));  // nothing is kept across stages
  // the columns alone: they hold the key's offset inside its unit as well
  kcol -= (key0 & umask) * (int)a.row_bytes;
  vcol -= (key0 & umask) * (int)a.row_bytes;
  if (a.off32) {
    const __amdgpu_buffer_rsrc_t kp = raw_rsrc(a.kbase, a.pre_bytes), vp = raw_rsrc(a.vbase, a.pre_bytes);
    const __amdgpu_buffer_rsrc_t ks = raw_rsrc(a.ks, a.suf_bytes), vs = raw_rsrc(a.vs, a.suf_bytes);
    int valid[St::kPer];
#pragma unroll
    for (int p = 0; p < St::kPer; ++p) valid[p] = valids[(key0 + p * St::kKeyStep) >> a.log2u];
#pragma unroll
    for (int p = 0; p < St::kPer; ++p) {
      const int key = key0 + p * St::kKeyStep;
      const uint32_t off = valid[p] > 0 ? (uint32_t)base[p] +
                                              (uint32_t)min(key & umask, valid[p] - 1) * a.row_bytes
                                        : 0u;
      if (valid[p] > 0 && pos0 + key < a.kc) {
        buffer_to_lds(kp, off + (uint32_t)kcol, 0, dk + p * St::kKeyStep * D);
        if constexpr (kV)
          buffer_to_lds(vp, off + (uint32_t)vcol, 0, dv + p * St::kKeyStep * D);
      } else {
        buffer_to_lds(ks, off + (uint32_t)kcol, 0, dk + p * St::kKeyStep * D);
        if constexpr (kV)
          buffer_to_lds(vs, off + (uint32_t)vcol, 0, dv + p * St::kKeyStep * D);
      }
    }
    return;
  }
  constexpr int kGroups = St::kRowsPerLoad / 4, kN = St::kPer * kGroups;
#pragma unroll 1
  for (int i = 0; i < kN; ++i) {
    const int p = i / kGroups, q = i % kGroups;
    const int gkey = p * St::kKeyStep + wave * St::kRowsPerLoad + 4 * q;  // uniform
    const int valid = __builtin_amdgcn_readfirstlane(valids[gkey >> a.log2u]);
    const uint32_t row = (uint32_t)__builtin_amdgcn_readfirstlane(bases[gkey >> a.log2u]);
    const bool pre = valid > 0 && pos0 + gkey < a.kc;
    const uint64_t off = valid > 0 ? (uint64_t)row * a.row_bytes : 0;
    const uint32_t in_unit = (uint32_t)min((key0 + p * St::kKeyStep) & umask, max(valid - 1, 0)) * a.row_bytes;
    const char* kp = reinterpret_cast<const char*>(pre ? a.kbase : a.ks) + off;
    const char* vp = reinterpret_cast<const char*>(pre ? a.vbase : a.vs) + off;
    // (the offsets stay inside one unit: no bound is needed beyond it)
    if (kGroups == 1 || (int)((threadIdx.x & 63) / (64 / kGroups)) == q) {
      buffer_to_lds(raw_rsrc(kp, 0xffffffffu), (uint32_t)kcol + in_unit, 0, dk + p * St::kKeyStep * D);
      if constexpr (kV)
        buffer_to_lds(raw_rsrc(vp, 0xffffffffu), (uint32_t)vcol + in_unit, 0, dv + p * St::kKeyStep * D);
    }
  }
}

// Every wave's stage loads have landed in LDS (and the LDS reads before this
// are done): each wave waits for its own, then for the others.
__device__ __forceinline__ void stage_barrier() {
  __builtin_amdgcn_s_waitcnt(0x0070);  // vmcnt(0) lgkmcnt(0)
  __syncthreads();
}

// K operand fragment ks of 32 keys: kfo is this lane's byte offset of segment
// `half` of its row; segment 2 ks + half sits at that offset ^ 32 ks.
template <int D>
__device__ __forceinline__ bf16x8 read_k(const uint16_t* lk, uint32_t kfo, int sub, int ks) {
  return *reinterpret_cast<const bf16x8*>(reinterpret_cast<const char*>(lk) + (kfo ^ (32u * ks)) +
                                          sub * kSub * D * 2);
}

// V^T operand fragment (kb, db) of 32 keys: voff is the byte offset for db = 0,
// that of db is voff ^ 64 db, and (sub, kb, rd) add whole rows.
template <int D>
__device__ __forceinline__ bf16x8 read_v(const uint16_t* lv, uint32_t voff, int sub, int kb, int db) {
  bf16x8 vf;
#pragma unroll
  for (int rd = 0; rd < 2; ++rd)
    *(reinterpret_cast<s16x4*>(&vf) + rd) = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
        (__attribute__((address_space(3))) s16x4*)(reinterpret_cast<const char*>(lv) +
                                                   (voff ^ (64u * db)) +
                                                   (sub * kSub + 16 * kb + 4 * rd) * D * 2));
  return vf;
}

// The numerators exp2(c1 s - m) of 32 keys in 16 / E + 2 steps, which are
// issued between MFMAs: step i scales the E logits of group i, takes the
// exponentials of group i - 1, and adds those of group i - 2 to the row's sums
// and packs them to bf16 pairs (P^T).  The empty asm keeps a step in its place.
template <int E, int i>
__device__ __forceinline__ void numerator_step(f32x16& s, float c1, float m, float (&l)[2],
                                               u32x4 (&pb)[2]) {
  constexpr int kGroups = 16 / E;
  if constexpr (i < 0 || i > kGroups + 1) return;
#pragma unroll
  for (int e = 0; e < E; ++e) {
    if (i < kGroups) s[E * i + e] = fmaf(s[E * i + e], c1, -m);
    if (i >= 1 && i <= kGroups) s[E * (i - 1) + e] = __builtin_amdgcn_exp2f(s[E * (i - 1) + e]);
    const int v = E * (i - 2) + e;
    if (i < 2 || i > kGroups + 1) continue;
    l[v & 1] += s[v];
    asm volatile("" : "+v"(l[v & 1]));
    if (v & 1) {
      const bf16x2 b = {(__bf16)s[v - 1], (__bf16)s[v]};
      uint32_t w = __builtin_bit_cast(uint32_t, b);
      asm volatile("" : "+v"(w));
      pb[v >> 3][(v & 7) >> 1] = w;
    }
  }
}

// -inf for the keys of product `sub` of the stage at position pos0 that this
// lane's query t must not see.  Register v holds key 32*sub + 16*(v/8) + 8*half +
// v%8.
__device__ __forceinline__ void mask_logits(const AttnArgs& a, const int* valids, int pos0, int sub,
                                            int t, f32x16& s) {
  int key_lane = kSub * sub + ((threadIdx.x >> 2) & 8);  // + 8 * half
  asm volatile("" : "+v"(key_lane));  // nothing of this (rare) path is kept across stages
#pragma unroll
  for (int q = 0; q < 4; ++q) {  // 4 keys, inside one unit
    const int key = key_lane + 16 * (q >> 1) + 4 * (q & 1);
    int seen = valids[key >> a.log2u] - (key & ((1 << a.log2u) - 1));
    const int p = pos0 + key - a.kc;  // suffix position
    if (p >= 0) seen = min(seen, t - p + 1);
#pragma unroll
    for (int e = 0; e < 4; ++e) s[4 * q + e] = e < seen ? s[4 * q + e] : -INFINITY;
  }
}

__device__ __forceinline__ float max16(const f32x16& s) {
  float mx = s[0];
#pragma unroll
  for (int v = 1; v < 16; ++v) mx = fmaxf(mx, s[v]);
  return mx;
}

// f(0), f(1), ... with compile-time arguments.
template <class F, int... I>
__device__ __forceinline__ void for_each_of(std::integer_sequence<int, I...>, F&& f) {
  (f(std::integral_constant<int, I>{}), ...);
}
template <int N, class F>
__device__ __forceinline__ void static_for(F&& f) {
  for_each_of(std::make_integer_sequence<int, N>{}, f);
}

// kPartial: the slice is one of several of its rows (AttnArgs::o_part, ml_part).
template <int D, bool kPartial>
__global__ __launch_bounds__(kWaves * 64, 2) void attn_kernel(AttnArgs a) {
  using St = Stage<D>;
  // two stage buffers, as arrays of their own: loads into one are then known
  // not to touch the other
  __shared__ __attribute__((aligned(16))) uint16_t k0[kTile * D], k1[kTile * D];
  __shared__ __attribute__((aligned(16))) uint16_t v0[kTile * D], v1[kTile * D];
  // unit tables of the slice (base, valid), then one flags word per stage
  // (dynamic: attn_slice_bytes)
  extern __shared__ int slice_lds[];
  const int upst = kTile >> a.log2u;  // units per stage
  int* bases = slice_lds;
  int* valids = slice_lds + a.tiles_per_split * upst;
  int* stage_flags = slice_lds + 2 * a.tiles_per_split * upst;

  // logical order (g, split, row block): blocks reading the same K/V tiles are
  // adjacent, hence on the same XCD and its L2
  const uint32_t L = xcd_remap(blockIdx.x, a.nblocks_padded);
  if (L >= a.nblocks) return;
  const int rb = (int)(L % a.n_row_blocks);
  const int split = (int)((L / a.n_row_blocks) % a.n_splits);
  const int g = (int)(L / ((uint32_t)a.n_splits * a.n_row_blocks));
  const int lane = threadIdx.x & 63, half = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);

  const int row = rb * kBlockRows + wave * kWaveRows + (lane & 31);
  const bool row_ok = row < a.R;
  const int t = row_ok ? row / a.G : -1;
  const int hi = row_ok ? row % a.G : 0;

  // keys the block's last query can see; the block's first query sees every
  // suffix key up to its own position (both in scalar registers: left to itself the
  // compiler keeps them, and every branch on them, in vector ones, 0.4 us a launch)
  const int first_t = __builtin_amdgcn_readfirstlane((rb * kBlockRows) / a.G);
  const int last_row = min(a.R - 1, rb * kBlockRows + kBlockRows - 1);
  const int np_block = a.kc + (a.with_suffix ? last_row / a.G + 1 : 0);
  const int ntiles = (np_block + kTile - 1) / kTile;
  const int tile0 = split * a.tiles_per_split;
  const int nt = __builtin_amdgcn_readfirstlane(max(0, min(ntiles, tile0 + a.tiles_per_split) - tile0));

  // the first units' index loads, then Q: loads return in order, so the tables
  // (on the critical path to the first K/V loads) do not wait for Q
  const int pos00 = tile0 * kTile, n_units = nt * upst;
  int j0, slot0;
  unit_chunk(a, (int)threadIdx.x < n_units ? pos00 + ((int)threadIdx.x << a.log2u) : a.kc, j0, slot0);
  bf16x8 qf[D / 16];
  {
    const uint16_t* src = a.q + ((int64_t)(row_ok ? t : 0) * a.Hq + (int64_t)g * a.G + hi) * D + 8 * half;
#pragma unroll
    for (int ks = 0; ks < D / 16; ++ks)
      qf[ks] = *reinterpret_cast<const bf16x8*>(src + 16 * ks);
  }
  // the units of a stage are neighbouring lanes of one wave, the first of which
  // writes the stage's flags: a unit short of rows makes it mixed and masked
  for (int i0 = 0; i0 < n_units; i0 += kWaves * 64) {
    const int i = i0 + (int)threadIdx.x, pos = pos00 + (i << a.log2u);
    int urow = 0, valid = 0;
    if (i0 > 0) unit_chunk(a, i < n_units ? pos : a.kc, j0, slot0);
    if (i < n_units) unit_entry(a, pos, j0, slot0, urow, valid);
    const uint64_t shortfall = __ballot(valid < (1 << a.log2u)) >> (lane & -upst);
    if (i < n_units) {
      // the row's byte offset from its source's base when every one fits in 32 bits
      bases[i] = a.off32 ? (int)((uint32_t)urow * a.row_bytes) : urow;
      valids[i] = valid;
      if ((i & (upst - 1)) == 0) {
        const int end = pos + kTile - a.kc;  // keys of the stage's end past the prefix
        int f = (pos < a.kc ? kStagePrefix : 0) | (end > 0 ? kStageSuffix : 0);
        if (end > 0 && end - 1 > first_t) f |= kStageMask;
        if (shortfall & ((1ull << upst) - 1)) f |= kStageMixed | kStageMask;
        stage_flags[(uint32_t)i / (uint32_t)upst] = f;
      }
    }
  }
  if (!row_ok) {
#pragma unroll
    for (int ks = 0; ks < D / 16; ++ks) qf[ks] = __builtin_bit_cast(bf16x8, u32x4{0u, 0u, 0u, 0u});
  }
  __syncthreads();

  // this lane's keys and byte columns of the stage loads
  LoadLane ll;
  {
    ll.key0 = wave * St::kRowsPerLoad + lane / St::kSegs;
    const int seg = lane % St::kSegs, in_unit = (ll.key0 & ((1 << a.log2u) - 1)) * (int)a.row_bytes;
    ll.kcol = 2 * (g * D + ((seg ^ k_swz<D>(ll.key0)) << 3)) + in_unit;
    ll.vcol = 2 * (g * D + ((seg ^ v_swz<D>(ll.key0)) << 3)) + in_unit;
  }
  const int* lane_bases = bases + (ll.key0 >> a.log2u);
  // byte offsets of the operand reads (the same for every stage)
  const int kr = kappa(lane & 31);
  const uint32_t kfo = 2 * (kr * D + ((half ^ k_swz<D>(kr)) << 3));
  // V^T fragment pieces: lane (group g4 = (lane/16)%2, s16 = lane%16) supplies
  // row 16*kb + 8*half + 4*rd + s16/4, columns 32*db + 16*g4 + 4*(s16%4) .. +3.
  // The swizzle depends on the row modulo 4 only.
  const int s16 = lane & 15, g4 = (lane >> 4) & 1;
  const uint32_t voff = 2 * (v_off<D>(8 * half + (s16 >> 2), 2 * g4 + ((s16 & 3) >> 1)) + 4 * (s16 & 1));

  constexpr int kG = D / 16;  // MFMAs of one 32-key product, and of one O update
  constexpr int kE = 256 / D; // logits per numerator step: kG + 2 steps per half
  f32x16 o[D / 32];
  float l[2];
  float ref = 0.f;  // reference of this lane's row (scaled log2 units)
  auto flags_of = [&](int st) { return __builtin_amdgcn_readfirstlane(stage_flags[st]); };
  // the unit table entries of this lane's keys of a stage
  auto read_bases = [&](int st, int* r) {
#pragma unroll
    for (int p = 0; p < St::kPer; ++p) r[p] = lane_bases[st * upst + (p * St::kKeyStep >> a.log2u)];
  };
  auto load_stage = [&](int st, int f, const int* r, uint16_t* dk, uint16_t* dv) {
    stage_load<D>(a, f, r, bases + st * upst, valids + st * upst, pos00 + st * kTile, wave, ll, dk, dv);
  };
  auto mask = [&](int st, int sub, f32x16& s) {
    mask_logits(a, valids + st * upst, pos00 + st * kTile, sub, t, s);
  };

  // whether this lane's query sees a key of the slice
  auto sees_key = [&]() {
    for (int i = 0; i < n_units; ++i) {
      const int pos = pos00 + (i << a.log2u);
      if (valids[i] > 0) return pos < a.kc || t >= pos - a.kc;  // later units: later positions
    }
    return false;
  };

  bool no_ref = false;  // the reference had to be taken from no key at all
  for (int attempt = 0;; ++attempt) {
#pragma unroll
    for (int db = 0; db < D / 32; ++db)
#pragma unroll
      for (int v = 0; v < 16; ++v) o[db][v] = 0.f;
    l[0] = l[1] = 0.f;
    if (nt > 0) {
      int r[St::kPer];
      read_bases(0, r);
      int fl = flags_of(0);  // of the current stage
      load_stage(0, fl, r, k0, v0);
      stage_barrier();
      bf16x8 ka[kG];  // K fragments of the current stage's first 32 keys
#pragma unroll
      for (int i = 0; i < kG; ++i) ka[i] = read_k<D>(k0, kfo, 0, i);

      // One stage (K in lk, V in lv), with the next one's rows loading into nk and
      // nv, as four runs of kG MFMAs: the first half's product, the second half's
      // product beside the first half's numerators, the first half's O update
      // beside the second half's numerators, and the second half's O update; each
      // run reads the operands of the next.  The order inside a run is fixed by
      // scheduling barriers: left to itself the compiler reads each operand right
      // before its MFMA, which then waits for it.
      auto stage = [&](int st, uint16_t* lk, uint16_t* lv, uint16_t* nk, uint16_t* nv)
          __attribute__((always_inline)) {
        // the operand offsets stay opaque here, so that each buffer's address is
        // an immediate of the read and not a register of its own
        uint32_t ko = kfo, vo = voff;
        asm volatile("" : "+v"(ko), "+v"(vo));
        int fn = 0;
        if (st + 1 < nt) {
          read_bases(st + 1, r);
          fn = flags_of(st + 1);
          load_stage(st + 1, fn, r, nk, nv);
        }
        bf16x8 kb[kG], va[2][D / 32], vb[2][D / 32];
        f32x16 s0, s1;
        u32x4 p0[2], p1[2];
#pragma unroll
        for (int v = 0; v < 16; ++v) s0[v] = s1[v] = 0.f;
        __builtin_amdgcn_sched_barrier(0);
        static_for<kG>([&](auto i) __attribute__((always_inline)) {
          kb[i] = read_k<D>(lk, ko, 1, i);
          s0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka[i], qf[i], s0, 0, 0, 0);
          __builtin_amdgcn_sched_barrier(0);
        });
        if (fl & kStageMask) mask(st, 0, s0);
        if (st == 0 && attempt == 0) {  // the reference: the first 32 keys' largest logit
          float mx = max16(s0);
          if constexpr (!kPartial) {
            // A row's only slice takes it from 64 keys: the largest weight is then exactly
            // 1 as often as with a running maximum over whole stages, and no partial's
            // rounding is saved that would pay for less (280 keys: 2.31e-3 -> 2.29e-3 off
            // fp64; 0.1 us of 8.7, 0.3 where the first stage is masked).
#pragma unroll
            for (int i = 0; i < kG; ++i)
              s1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kb[i], qf[i], s1, 0, 0, 0);
            if (fl & kStageMask) mask(st, 1, s1);
            mx = fmaxf(mx, max16(s1));
#pragma unroll
            for (int v = 0; v < 16; ++v) s1[v] = 0.f;
          }
          mx = fmaxf(mx, partner_f(mx));
          no_ref = mx == -INFINITY;
          ref = no_ref ? 0.f : mx * a.c1;
        }
        __builtin_amdgcn_sched_barrier(0);
        static_for<kG>([&](auto i) __attribute__((always_inline)) {
          constexpr int kk = i / (D / 32), db = i % (D / 32);
          va[kk][db] = read_v<D>(lv, vo, 0, kk, db);
          s1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kb[i], qf[i], s1, 0, 0, 0);
          numerator_step<kE, i>(s0, a.c1, ref, l, p0);
          __builtin_amdgcn_sched_barrier(0);
        });
        if (fl & kStageMask) mask(st, 1, s1);
        __builtin_amdgcn_sched_barrier(0);
        static_for<kG>([&](auto i) __attribute__((always_inline)) {
          constexpr int kk = i / (D / 32), db = i % (D / 32);
          vb[kk][db] = read_v<D>(lv, vo, 1, kk, db);
          if constexpr (i < 2) numerator_step<kE, kG + i>(s0, a.c1, ref, l, p0);
          o[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va[kk][db], __builtin_bit_cast(bf16x8, p0[kk]),
                                                          o[db], 0, 0, 0);
          numerator_step<kE, i>(s1, a.c1, ref, l, p1);
          __builtin_amdgcn_sched_barrier(0);
        });
        stage_barrier();  // the next stage has landed; this one's buffers are read
        __builtin_amdgcn_sched_barrier(0);
        static_for<kG>([&](auto i) __attribute__((always_inline)) {
          constexpr int kk = i / (D / 32), db = i % (D / 32);
          ka[i] = read_k<D>(nk, ko, 0, i);  // (after the last stage: read and not used)
          if constexpr (i < 2) numerator_step<kE, kG + i>(s1, a.c1, ref, l, p1);
          o[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vb[kk][db], __builtin_bit_cast(bf16x8, p1[kk]),
                                                          o[db], 0, 0, 0);
          __builtin_amdgcn_sched_barrier(0);
        });
        fl = fn;
      };
      for (int st = 0; st < nt; st += 2) {
        stage(st, k0, v0, k1, v1);
        if (st + 1 >= nt) break;
        stage(st + 1, k1, v1, k0, v0);
      }
    }
    l[0] += l[1];
    l[0] += partner_f(l[0]);
    // The reference is the first keys' maximum: a later logit far above it can
    // push the sum past the guard or an output past fp32, and a row whose first
    // keys are all hidden has none.  Then once more, against the slice's own
    // maximum.  (A row that sees no key of the slice, as those before a slice that
    // begins inside their block's part of the suffix, has nothing to do again.)
    if (attempt) break;
    // (a sum over the outputs is inf or NaN if one of them is)
    float any[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int db = 0; db < D / 32; ++db)
#pragma unroll
      for (int v = 0; v < 16; ++v) any[v & 3] += o[db][v];
    const uint32_t total = __float_as_uint((any[0] + any[1]) + (any[2] + any[3]));
    const bool bad = (total & 0x7f800000u) == 0x7f800000u ||
                     (__float_as_uint(l[0]) & 0x7fffffffu) > __float_as_uint(kGuard) ||
                     (no_ref && l[0] < kGuardLow && sees_key());
    if (!__syncthreads_or(bad)) break;
    float mx = -INFINITY;
    for (int st = 0; st < nt; ++st) {
      int r[St::kPer];
      read_bases(st, r);
      const int f = flags_of(st);
      stage_load<D, false>(a, f, r, bases + st * upst, valids + st * upst, pos00 + st * kTile, wave, ll,
                           k0, v0);
      stage_barrier();
#pragma unroll
      for (int sub = 0; sub < 2; ++sub) {
        f32x16 s;
#pragma unroll
        for (int v = 0; v < 16; ++v) s[v] = 0.f;
#pragma unroll
        for (int i = 0; i < kG; ++i)
          s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(read_k<D>(k0, kfo, sub, i), qf[i], s, 0, 0, 0);
        mask(st, sub, s);
        mx = fmaxf(mx, max16(s));
      }
      __syncthreads();
    }
    mx = fmaxf(mx, partner_f(mx));
    ref = mx == -INFINITY ? 0.f : mx * a.c1;
  }

  // Output rows through LDS, so that every global store is a whole 16-byte
  // piece of a row and 16 lanes cover a row: the wave's 32 rows go to a stage
  // buffer of its own, which every wave has finished reading (the barrier above).
  float2 ml = make_float2(ref, 0.f);  // (reference 0 and no sum while no key was seen)
  {
    constexpr int kRow = D + 8;
    uint16_t* tile = wave == 0 ? k0 : wave == 1 ? k1 : wave == 2 ? v0 : v1;
    // o[db][v] holds d = 32*db + 8*(v/4) + 4*half + v%4 of this lane's row
    auto put_rows = [&](auto type, float scale) __attribute__((always_inline)) {
      using T = decltype(type);
#pragma unroll
      for (int db = 0; db < D / 32; ++db)
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4) {
          T b[4];
#pragma unroll
          for (int j = 0; j < 4; ++j) b[j] = (T)(o[db][4 * q4 + j] * scale);
          *reinterpret_cast<uint2*>(tile + (lane & 31) * kRow + 32 * db + 8 * q4 + 4 * half) =
              *reinterpret_cast<uint2*>(b);
        }
    };
    if constexpr (kPartial) {
      // A partial is stored as outputs 2^-E O in half precision, E the row's own (its
      // largest output lies in [2^14, 2^15)), and as the pair of ref + e and of l 2^-e
      // in [1, 2) with E - e for its exponent: against the reference ref + e the merge
      // takes the sum from that mantissa and the outputs' power from that exponent.
      // With e in the reference both are of V's size at most: a reference far below
      // the slice's maximum leaves a sum up to kGuard, by which the merge would
      // otherwise multiply outputs as large as V.  Halves in place of bf16 cost no
      // bytes and 0.05 us, and take the partials' rounding, which was a third of the
      // output's squared error, to a 64th (1,648 keys in 7 splits: 2.93e-3 -> 2.37e-3
      // off fp64 in the 2-norm).
      float om = 0.f;
#pragma unroll
      for (int db = 0; db < D / 32; ++db)
#pragma unroll
        for (int v = 0; v < 16; ++v) om = fmaxf(om, fabsf(o[db][v]));
      om = fmaxf(om, partner_f(om));
      const uint32_t lb = __float_as_uint(l[0]);
      const int e = (int)(lb >> 23) - 127;
      // (E - e and E no lower than -110, so that both powers stay in fp32's range)
      const int E = max((int)(__float_as_uint(om) >> 23) - 127 - 14, max(e, 0) - 110);
      put_rows(_Float16{}, __uint_as_float((uint32_t)(127 - E) << 23));
      if (l[0] > 0.f)
        ml = make_float2(ref + (float)e,
                         __uint_as_float((lb & 0x007fffffu) | (uint32_t)(E - e + 127) << 23));
    } else {
      put_rows(__bf16{}, l[0] > 0.f ? 1.f / l[0] : 0.f);
    }
    // 64 lanes = 64 / (D/8) rows x D/8 segments of 8
    constexpr int kSegs = D / 8, kRowsPerPass = 64 / kSegs;
    const int seg = lane % kSegs;
    const int row_base = rb * kBlockRows + wave * kWaveRows;
    // output row of this lane's query row; row rr's is lane rr's
    const int out_row = kPartial ? row : (row_ok ? t : 0) * a.Hq + g * a.G + hi;
    uint16_t* obase = kPartial ? a.o_part + ((int64_t)split * a.Hkv + g) * a.R * D : a.out;
#pragma unroll
    for (int r0 = 0; r0 < kWaveRows; r0 += kRowsPerPass) {
      const int rr = r0 + lane / kSegs;
      const uint4 v = *reinterpret_cast<const uint4*>(tile + rr * kRow + seg * 8);
      const int orow = __shfl(out_row, rr);
      if (row_base + rr < a.R) *reinterpret_cast<uint4*>(obase + (int64_t)orow * D + seg * 8) = v;
    }
  }
  if (kPartial && row_ok && half == 0) a.ml_part[((int64_t)split * a.Hkv + g) * a.R + row] = ml;
}

// Merges the splits of each row in split order: out = sum_s w_s O_s / sum_s w_s l_s,
// w_s = exp2(m_s - max m), from what a partial stores (see there), as a running
// merge over batches of kCombineBatch splits whose loads are in flight together.
// One thread per (row, 8 columns).
constexpr int kCombineBatch = 8;

template <int D>
__global__ __launch_bounds__(256) void combine_kernel(const uint16_t* __restrict__ o_part,
                                                      const float2* __restrict__ ml_part,
                                                      uint16_t* __restrict__ out, int n_splits,
                                                      int Hkv, int R, int G, int Hq) {
  const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int64_t rows = (int64_t)Hkv * R;
  if (idx >= rows * (D / 8)) return;
  const int64_t grow = idx / (D / 8);
  const int c8 = (int)(idx % (D / 8)) * 8;
  float M = -INFINITY, Lsum = 0.f;
  float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  for (int s0 = 0; s0 < n_splits; s0 += kCombineBatch) {
    // unconditional loads (a split past the last re-reads the last one and is
    // then ignored), so the whole batch is in flight together
    float2 ml[kCombineBatch];
    uint4 raw[kCombineBatch];
#pragma unroll
    for (int i = 0; i < kCombineBatch; ++i) {
      const int64_t sp = min(s0 + i, n_splits - 1);
      ml[i] = ml_part[sp * rows + grow];
      raw[i] = *reinterpret_cast<const uint4*>(o_part + (sp * rows + grow) * D + c8);
    }
#pragma unroll
    for (int i = 0; i < kCombineBatch; ++i)
      if (s0 + i >= n_splits) ml[i] = make_float2(0.f, 0.f);
#pragma unroll
    for (int i = 0; i < kCombineBatch; ++i) {
      if (!(ml[i].y > 0.f)) continue;  // absent, or the split saw no key of this row
      if (ml[i].x > M) {
        const float scale = M == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(M - ml[i].x);
        Lsum *= scale;
#pragma unroll
        for (int j = 0; j < 8; ++j) acc[j] *= scale;
        M = ml[i].x;
      }
      const uint32_t y = __float_as_uint(ml[i].y);
      const float w = __builtin_amdgcn_exp2f(ml[i].x - M), wgt = w * __uint_as_float(y & 0x7f800000u);
      Lsum += w * __uint_as_float((y & 0x007fffffu) | 0x3f800000u);
      const _Float16* h = reinterpret_cast<const _Float16*>(&raw[i]);
#pragma unroll
      for (int j = 0; j < 8; ++j) acc[j] += wgt * (float)h[j];
    }
  }
  const int g = (int)(grow / R), row = (int)(grow % R);
  const int t = row / G, i = row % G;
  const float inv = 1.f / Lsum;
  __bf16 b[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) b[j] = (__bf16)(acc[j] * inv);
  *reinterpret_cast<uint4*>(out + ((int64_t)t * Hq + (int64_t)g * G + i) * D + c8) =
      *reinterpret_cast<uint4*>(b);
}

// ---------------------------------------------------------------------------
// fp32 path: one workgroup per (query t, head h).  Four lanes share a key of the
// row's sequence (16 elements each of its K and V rows), the workgroup's 128 lane
// groups visit keys i, i + 128, ..., two of them in flight, with an online softmax
// per group (fp32, exp2 with the scale folded in); the groups' states merge by
// shuffles in a wave and through LDS between waves.
//
// Bound by the chain of one key (its index, then its K and V rows) and the merge:
// one wave per row with a key per lane, whose 64 rows are 64 cache lines per load
// and whose states merge through LDS, took 9.9 us at 32 queries x 4 heads over 256
// keys, this 6.4.
// ---------------------------------------------------------------------------
constexpr int kF32Waves = 8;
constexpr int kF32Lanes = 4;  // lanes per key
struct AttnArgsF32 {
  const float* q;
  const float* kbase;
  const float* vbase;
  int64_t chunk_stride;
  const int32_t* chunk_off;
  int32_t direct;
  const int32_t* sel;
  int64_t kc, n;
  int c;
  const float* ks;
  const float* vs;
  float* out;
  int S, Hq, Hkv, G;
  float c1;
};

template <int D>
__global__ __launch_bounds__(64 * kF32Waves) void attn_f32_kernel(AttnArgsF32 a) {
  constexpr int kKeys = 64 * kF32Waves / kF32Lanes;  // keys per step
  constexpr int kVec = D / (4 * kF32Lanes);          // 16-byte pieces of a row per lane
  const int64_t rid = blockIdx.x;  // t * Hq + h
  const int t = (int)(rid / a.Hq), h = (int)(rid % a.Hq), g = h / a.G;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int e0 = 4 * (threadIdx.x % kF32Lanes);  // element of piece 0; piece j at + 4 * kF32Lanes * j
  f32x4 q[kVec], o[kVec];
#pragma unroll
  for (int j = 0; j < kVec; ++j) {
    q[j] = *reinterpret_cast<const f32x4*>(a.q + rid * D + e0 + 4 * kF32Lanes * j);
    o[j] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  float m = -INFINITY, l = 0.f;
  const int64_t np = a.kc + t + 1;
  for (int64_t p0 = threadIdx.x / kF32Lanes; p0 < np; p0 += 2 * kKeys) {
    f32x4 kv[2][kVec], vv[2][kVec];
    bool valid[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int64_t pos = p0 + i * kKeys;
      valid[i] = pos < np;
      const float* kr = a.ks;  // a hidden key reads the suffix's first row
      const float* vr = a.vs;
      if (pos < a.kc) {
        const int64_t u = pos / a.c;
        const int off = (int)(pos - u * a.c);
        const int64_t j = a.sel[u];
        valid[i] = j >= 0 && off < min<int64_t>(a.c, a.n - j * a.c);
        if (valid[i]) {
          const int64_t slot = a.chunk_off ? (int64_t)a.chunk_off[u] : (a.direct ? j : u);
          const int64_t e = slot * a.chunk_stride + ((int64_t)off * a.Hkv + g) * D;
          kr = a.kbase + e;
          vr = a.vbase + e;
        }
      } else if (valid[i]) {
        const int64_t e = ((pos - a.kc) * a.Hkv + g) * D;
        kr = a.ks + e;
        vr = a.vs + e;
      }
#pragma unroll
      for (int j = 0; j < kVec; ++j) {
        kv[i][j] = *reinterpret_cast<const f32x4*>(kr + e0 + 4 * kF32Lanes * j);
        vv[i][j] = *reinterpret_cast<const f32x4*>(vr + e0 + 4 * kF32Lanes * j);
      }
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      float dot = 0.f;
#pragma unroll
      for (int j = 0; j < kVec; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) dot = fmaf(q[j][e], kv[i][j][e], dot);
#pragma unroll
      for (int x = 1; x < kF32Lanes; x <<= 1) dot += __shfl_xor(dot, x);
      if (!valid[i]) continue;  // the same for the four lanes of a key
      const float s = dot * a.c1;
      const float mn = fmaxf(m, s);
      const float alpha = __builtin_amdgcn_exp2f(m - mn);
      const float p = __builtin_amdgcn_exp2f(s - mn);
      l = l * alpha + p;
#pragma unroll
      for (int j = 0; j < kVec; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) o[j][e] = fmaf(p, vv[i][j][e], o[j][e] * alpha);
      m = mn;
    }
  }
  // merge in the wave against its maximum reference, then over the waves
  __shared__ f32x4 wo[kF32Waves][D / 4];
  __shared__ float wm[kF32Waves], wl[kF32Waves];
  float M = m;
#pragma unroll
  for (int x = kF32Lanes; x < 64; x <<= 1) M = fmaxf(M, __shfl_xor(M, x));
  const float scale = m == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m - M);
  float L = l * scale;
#pragma unroll
  for (int x = kF32Lanes; x < 64; x <<= 1) L += __shfl_xor(L, x);
#pragma unroll
  for (int j = 0; j < kVec; ++j) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      float y = o[j][e] * scale;
#pragma unroll
      for (int x = kF32Lanes; x < 64; x <<= 1) y += __shfl_xor(y, x);
      o[j][e] = y;
    }
    if (lane < kF32Lanes) wo[wave][lane + kF32Lanes * j] = o[j];
  }
  if (lane == 0) {
    wm[wave] = M;
    wl[wave] = L;
  }
  __syncthreads();
  M = -INFINITY;
#pragma unroll
  for (int w = 0; w < kF32Waves; ++w) M = fmaxf(M, wm[w]);
  float f[kF32Waves];
  L = 0.f;
#pragma unroll
  for (int w = 0; w < kF32Waves; ++w) {
    f[w] = wm[w] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(wm[w] - M);
    L = fmaf(wl[w], f[w], L);
  }
  const float inv = L > 0.f ? 1.f / L : 0.f;
  for (int e = threadIdx.x; e < D; e += 64 * kF32Waves) {
    float acc = 0.f;
#pragma unroll
    for (int w = 0; w < kF32Waves; ++w)
      acc = fmaf(reinterpret_cast<const float*>(wo[w])[e], f[w], acc);
    a.out[rid * D + e] = acc * inv;
  }
}

}  // namespace

namespace {

// Keys of a unit (see kMaxSliceUnits), as a power of two: c is 4, 8, 16 or a
// multiple of 32.
int log2_unit(int c) { return c < 32 ? __builtin_ctz(c) : 5; }

// Stages whose tables fit a workgroup's share of the LDS.
int64_t max_slice_stages(int c) {
  return std::min<int64_t>(kMaxSliceStages, kMaxSliceUnits / (kTile >> log2_unit(c)));
}

// 64-key stages of an attention over k chunks (no keys: one empty stage).
int64_t attn_stages(const ckv_dims* d, int64_t k, bool with_suffix) {
  return std::max<int64_t>(1, ceil_div(k * d->chunk_size + (with_suffix ? d->n_suffix : 0), kTile));
}

// Workgroups of one split.
int64_t attn_blocks(const ckv_dims* d) {
  return (int64_t)d->n_kv_heads * ceil_div((int64_t)(d->n_q_heads / d->n_kv_heads) * d->n_suffix, kBlockRows);
}

// The most splits that make_attn_plan may take: those that give 512 workgroups of 4
// stages or more, or that hold a slice to 16 stages.  They bound the partials'
// workspace.  The smallest launches would gain from shorter slices (15 stages of 2
// workgroups: 8.3 us in 8 splits, 10.5 in the 3 taken; 20 of 16: 13.6 in 7, 14.9 in
// 5), others not (48 of 8, which the model below expects to gain 14% from 24 splits:
// 14.7 us, 14.5 in the 12 taken).
int64_t attn_most_splits(const ckv_dims* d, int64_t ntiles) {
  return std::max(std::max<int64_t>(1, std::min(512 / attn_blocks(d), ntiles / 4)), ceil_div(ntiles, 16));
}

}  // namespace

AttnPlan make_attn_plan(const ckv_dims* d, int64_t k, bool with_suffix) {
  AttnPlan p{};
  const int G = d->n_q_heads / d->n_kv_heads;
  p.rows = G * d->n_suffix;
  if (d->dtype == CKV_DTYPE_F32) {  // one workgroup per row, no splits
    p.n_splits = 1;
    return p;
  }
  const int64_t ntiles = attn_stages(d, k, with_suffix), base = attn_blocks(d);
  // The splits that cost least by a model of the launch, in cycles at 1.85 GHz:
  // 512 workgroups run at once, two per CU, each for its stages (two of them
  // take 3,440 cycles per stage, one alone on its CU 2,100) and a fixed part
  // (tables, first loads, output); and every split's partials are merged (14
  // splits of 40,960 rows took 25 us, 3 of them 8).  The constants are of head_dim
  // 128; at 64, where a stage has half the MFMAs and three workgroups fit a CU, five
  // of six plans were within 8% of the best of nine split counts (the sixth is the
  // launch of 2 workgroups above).
  constexpr double kFixed = 15000, kStage = 3440, kFixedAlone = 12500, kStageAlone = 2100;
  constexpr double kCombine = 5500, kMergeBytes = 5000;
  const double merge = (double)d->n_kv_heads * p.rows * d->head_dim * 2 / kMergeBytes;
  const int64_t n_min = ceil_div(ntiles, max_slice_stages(d->chunk_size));
  const int64_t n_max = attn_most_splits(d, ntiles);
  int64_t splits = 0;
  double best = 0;
  // (past sqrt(ntiles) many counts give the same stages per split: on to the next that
  // does not; below, the divisions of a count do not wait for those of the last)
  for (int64_t n0 = n_min, per = 0; n0 <= n_max;
       n0 = n0 * n0 < ntiles || per == 1 ? n0 + 1 : ceil_div(ntiles, per - 1)) {
    per = ceil_div(ntiles, n0);
    const int64_t n = ceil_div(ntiles, per), wgs = base * n, rem = wgs % 512;
    double cost = (double)(wgs / 512) * (kFixed + kStage * (double)per);
    if (rem > 0)
      cost += rem <= 256 ? kFixedAlone + kStageAlone * (double)per : kFixed + kStage * (double)per;
    if (n > 1) cost += kCombine + merge * (double)n;
    if (!splits || cost < best) {
      best = cost;
      splits = n;
    }
  }
  p.n_splits = (int32_t)splits;
  size_t off = 0;
  if (splits > 1) {
    const size_t rows = (size_t)d->n_kv_heads * p.rows;
    p.off_o = off;
    off = align_up(off + (size_t)splits * rows * d->head_dim * sizeof(uint16_t), 256);
    p.off_ml = off;
    off = align_up(off + (size_t)splits * rows * sizeof(float2), 256);
  }
  p.bytes = off;
  return p;
}

namespace {

// Arguments of one bf16 attention launch over the kept chunks sel[0..k) of
// src (and the suffix when with_suffix) in n_splits key splits.
ckv_status attn_args(const ckv_dims* d, const void* q, const ChunkSource& src, const int32_t* sel,
                     int64_t k, const void* k_suffix, const void* v_suffix, bool with_suffix,
                     int32_t n_splits, AttnArgs& a) {
  a.q = static_cast<const uint16_t*>(q);
  a.kbase = static_cast<const uint16_t*>(src.k_base);
  a.vbase = static_cast<const uint16_t*>(src.v_base);
  a.chunk_off = src.chunk_off;
  a.direct = src.direct;
  {
    const int64_t hd = (int64_t)d->n_kv_heads * d->head_dim;
    if (src.chunk_stride % hd != 0) CKV_FAIL(CKV_EINVAL, "chunk stride is not a whole number of rows");
    const int64_t rps = src.chunk_stride / hd;
    // largest source row a key can name: every slot index is below n_slots
    if (src.n_slots < 0 || src.n_slots * rps >= (int64_t(1) << 31))
      CKV_FAIL(CKV_EUNSUPPORTED, "chunk source too large");
    a.rows_per_slot = (int)rps;
    // 32-bit byte offsets reach every row of both sources
    const int64_t rb = hd * (int64_t)sizeof(uint16_t);
    a.row_bytes = (uint32_t)rb;
    // (strictly below 4 GiB, so each source's byte count is a buffer size)
    const int64_t pre = src.n_slots * rps * rb, suf = (int64_t)d->n_suffix * rb;
    a.off32 = pre < (int64_t(1) << 32) && suf < (int64_t(1) << 32) &&
              g_force_wide.load(std::memory_order_relaxed) == 0;
    a.pre_bytes = (uint32_t)std::min<int64_t>(pre, UINT32_MAX);
    a.suf_bytes = (uint32_t)std::min<int64_t>(suf, UINT32_MAX);
  }
  a.sel = sel;
  a.kc = (int)(k * d->chunk_size);
  a.n = d->n_prefix;
  a.m = ceil_div(d->n_prefix, d->chunk_size);
  a.c = d->chunk_size;
  a.log2c = (d->chunk_size & (d->chunk_size - 1)) == 0 ? __builtin_ctz(d->chunk_size) : -1;
  a.log2u = log2_unit(d->chunk_size);
  a.ks = static_cast<const uint16_t*>(k_suffix);
  a.vs = static_cast<const uint16_t*>(v_suffix);
  a.S = d->n_suffix; a.Hq = d->n_q_heads; a.Hkv = d->n_kv_heads;
  a.G = d->n_q_heads / d->n_kv_heads; a.R = a.G * d->n_suffix;
  a.n_splits = n_splits;
  a.with_suffix = with_suffix ? 1 : 0;
  const int64_t ntiles = ceil_div(a.kc + (with_suffix ? a.S : 0), kTile);
  a.tiles_per_split = (int)ceil_div(ntiles, n_splits);  // <= max_slice_stages
  a.n_row_blocks = (int)ceil_div(a.R, kBlockRows);
  a.c1 = resolve_scale(d) * 1.4426950408889634f;
  a.nblocks = (uint32_t)((int64_t)a.Hkv * a.n_row_blocks * a.n_splits);
  a.nblocks_padded = (uint32_t)align_up(a.nblocks, 8);
  return CKV_OK;
}

ckv_status launch_attn_kernel(const ckv_dims* d, const AttnArgs& a, hipStream_t st) {
  const size_t slice_bytes = (size_t)a.tiles_per_split * (2 * (kTile >> a.log2u) + 1) * sizeof(int);
  const auto kernel = d->head_dim == 128 ? (a.partial ? attn_kernel<128, true> : attn_kernel<128, false>)
                                         : (a.partial ? attn_kernel<64, true> : attn_kernel<64, false>);
  hipLaunchKernelGGL(kernel, dim3(a.nblocks_padded), dim3(kWaves * 64), slice_bytes, st, a);
  CKV_HIP(hipGetLastError());
  return CKV_OK;
}

ckv_status launch_combine(const ckv_dims* d, const uint16_t* o_part, const float2* ml_part,
                          int32_t n_splits, void* out, hipStream_t st) {
  const int G = d->n_q_heads / d->n_kv_heads, R = G * d->n_suffix;
  const int64_t work = (int64_t)d->n_kv_heads * R * (d->head_dim / 8);
  uint16_t* o = static_cast<uint16_t*>(out);
  if (d->head_dim == 128)
    hipLaunchKernelGGL(combine_kernel<128>, dim3((unsigned)ceil_div(work, 256)), dim3(256), 0, st,
                       o_part, ml_part, o, n_splits, d->n_kv_heads, R, G, d->n_q_heads);
  else
    hipLaunchKernelGGL(combine_kernel<64>, dim3((unsigned)ceil_div(work, 256)), dim3(256), 0, st,
                       o_part, ml_part, o, n_splits, d->n_kv_heads, R, G, d->n_q_heads);
  CKV_HIP(hipGetLastError());
  return CKV_OK;
}

// Split partials of a parted attention: splits [0, max_splits) of o_part
// ([split][Hkv][R][D] fp16) then of ml_part ([split][Hkv][R] float2).
size_t part_o_bytes(const ckv_dims* d, int64_t max_splits) {
  const int G = d->n_q_heads / d->n_kv_heads;
  return align_up((size_t)max_splits * d->n_kv_heads * G * d->n_suffix * d->head_dim *
                      sizeof(uint16_t), 256);
}

}  // namespace

ckv_status launch_attn(const ckv_dims* d, const void* q, const ChunkSource& src, const int32_t* sel,
                       int64_t k, const void* k_suffix, const void* v_suffix, void* out, void* ws,
                       size_t ws_bytes, hipStream_t st) {
  if (d->dtype == CKV_DTYPE_F32) {
    AttnArgsF32 a;
    a.q = static_cast<const float*>(q);
    a.kbase = static_cast<const float*>(src.k_base);
    a.vbase = static_cast<const float*>(src.v_base);
    a.chunk_stride = src.chunk_stride;
    a.chunk_off = src.chunk_off;
    a.direct = src.direct;
    a.sel = sel;
    a.kc = k * d->chunk_size;
    a.n = d->n_prefix;
    a.c = d->chunk_size;
    a.ks = static_cast<const float*>(k_suffix);
    a.vs = static_cast<const float*>(v_suffix);
    a.out = static_cast<float*>(out);
    a.S = d->n_suffix; a.Hq = d->n_q_heads; a.Hkv = d->n_kv_heads;
    a.G = d->n_q_heads / d->n_kv_heads;
    a.c1 = resolve_scale(d) * 1.4426950408889634f;
    hipLaunchKernelGGL(attn_f32_kernel<64>, dim3((unsigned)((int64_t)a.S * a.Hq)),
                       dim3(64 * kF32Waves), 0, st, a);
    CKV_HIP(hipGetLastError());
    return CKV_OK;
  }
  const AttnPlan p = make_attn_plan(d, k);
  if (ws_bytes < p.bytes) CKV_FAIL(CKV_EINVAL, "attention workspace too small: %zu < %zu", ws_bytes, p.bytes);
  AttnArgs a;
  ckv_status s = attn_args(d, q, src, sel, k, k_suffix, v_suffix, true, p.n_splits, a);
  if (s != CKV_OK) return s;
  a.out = static_cast<uint16_t*>(out);
  a.partial = p.n_splits > 1 ? 1 : 0;
  a.o_part = a.partial ? reinterpret_cast<uint16_t*>(static_cast<char*>(ws) + p.off_o) : nullptr;
  a.ml_part = a.partial ? reinterpret_cast<float2*>(static_cast<char*>(ws) + p.off_ml) : nullptr;
  if ((s = launch_attn_kernel(d, a, st)) != CKV_OK) return s;
  if (a.partial) return launch_combine(d, a.o_part, a.ml_part, a.n_splits, out, st);
  return CKV_OK;
}

// Every share holds one chunk plus a part of the rest that shrinks
// geometrically, share j weighing kShareA^j kShareB^(parts-1-j), so that the
// last share -- whose attention is all that follows the last copy -- is the
// smallest and no share is empty (integer arithmetic: the same shares on every
// host).  1 <= parts <= n_late.
constexpr int64_t kShareA = 1, kShareB = 2;

int64_t attn_late_part_begin(int64_t n_late, int parts, int i) {
  int64_t cum = 0, total = 0;
  for (int j = 0; j < parts; ++j) {
    int64_t w = 1;
    for (int e = 0; e < j; ++e) w *= kShareA;
    for (int e = 0; e < parts - 1 - j; ++e) w *= kShareB;
    if (j < i) cum += w;
    total += w;
  }
  return i + (n_late - parts) * cum / total;
}

// (from the closed bound, since it goes over every ka: with the plan itself, a search, a
// context of 8,192 kept chunks took 8.8 ms here instead of 0.9, one of 32,768 126
// instead of 3.7)
int64_t attn_parted_splits(const ckv_dims* d, int64_t k, int max_late_parts) {
  auto bound = [&](int64_t kept, bool with_suffix) {
    const int64_t ntiles = attn_stages(d, kept, with_suffix);
    return ceil_div(ntiles, ceil_div(ntiles, attn_most_splits(d, ntiles)));
  };
  int64_t most = 0;
  for (int64_t ka = 0; ka <= k; ++ka) {
    const int64_t nl = k - ka;
    const int parts = (int)std::min<int64_t>(max_late_parts, nl);
    int64_t n = bound(ka, true);
    for (int i = 0; i < parts; ++i)
      n += bound(attn_late_part_begin(nl, parts, i + 1) - attn_late_part_begin(nl, parts, i), false);
    most = std::max(most, n);
  }
  return most;
}

size_t attn_parted_bytes(const ckv_dims* d, int64_t max_splits) {
  const int G = d->n_q_heads / d->n_kv_heads;
  return align_up(part_o_bytes(d, max_splits) +
                      (size_t)max_splits * d->n_kv_heads * G * d->n_suffix * sizeof(float2),
                  256);
}

ckv_status launch_attn_part(const ckv_dims* d, const void* q, const ChunkSource& src,
                            const int32_t* sel, int64_t k, const void* k_suffix,
                            const void* v_suffix, bool with_suffix, void* ws, int64_t max_splits,
                            int32_t split_base, int32_t* n_splits, hipStream_t st) {
  if (d->dtype != CKV_DTYPE_BF16) CKV_FAIL(CKV_EUNSUPPORTED, "parted attention is bf16 only");
  if (k == 0 && !with_suffix) CKV_FAIL(CKV_EINVAL, "an attention part without the suffix needs chunks");
  const AttnPlan p = make_attn_plan(d, k, with_suffix);
  if (split_base < 0 || split_base + (int64_t)p.n_splits > max_splits)
    CKV_FAIL(CKV_EINVAL, "attention splits %d + %d exceed the workspace's %lld", split_base,
             p.n_splits, (long long)max_splits);
  AttnArgs a;
  ckv_status s = attn_args(d, q, src, sel, k, k_suffix, v_suffix, with_suffix, p.n_splits, a);
  if (s != CKV_OK) return s;
  const size_t rows = (size_t)d->n_kv_heads * a.R;
  a.out = nullptr;
  a.partial = 1;
  a.o_part = static_cast<uint16_t*>(ws) + (size_t)split_base * rows * d->head_dim;
  a.ml_part = reinterpret_cast<float2*>(static_cast<char*>(ws) + part_o_bytes(d, max_splits)) +
              (size_t)split_base * rows;
  *n_splits = p.n_splits;
  return launch_attn_kernel(d, a, st);
}

ckv_status launch_attn_combine(const ckv_dims* d, const void* ws, int64_t max_splits,
                               int32_t n_splits, void* out, hipStream_t st) {
  if (n_splits < 1 || n_splits > max_splits)
    CKV_FAIL(CKV_EINVAL, "combine of %d splits (workspace holds %lld)", n_splits,
             (long long)max_splits);
  return launch_combine(d, static_cast<const uint16_t*>(ws),
                        reinterpret_cast<const float2*>(static_cast<const char*>(ws) +
                                                        part_o_bytes(d, max_splits)),
                        n_splits, out, st);
}

}  // namespace ckv

extern "C" ckv_status ckv_debug_attn_wide_addressing(int32_t force_wide) {
  ckv::clear_error();
  if (force_wide != 0 && force_wide != 1) CKV_FAIL(CKV_EINVAL, "force_wide must be 0 or 1");
  ckv::g_force_wide.store(force_wide, std::memory_order_relaxed);
  return CKV_OK;
}
