// attend.hip -- temporal-causal attention forward with per-query log-sum-exp, gfx950.
//
// Computes, for one frame and one layer (Sec. 3.1 Eq. 2-3 and the LSE equation of
// Sec. 3.3), for every head h and query i of the frame:
//   z_ic = q_i . k_c / 8 over the context c = [memory rows of h ; the frame's keys],
//   LSE_i = log sum_c exp(z_ic),  o_i = sum_c exp(z_ic - LSE_i) v_c.
//
// Design (CDNA4):
// * Work unit = (head, 128-query tile); 4 wave64s, 32 queries each.  Key/value tiles of
//   64 rows go straight from global memory into LDS (global_load_lds_dwordx4), row-major
//   with an XOR swizzle, through a 4-stage ring whose stage offsets are compile-time
//   constants: two tiles are computed per barrier while the next two stream in.
// * Scores are formed transposed, S^T = K Q^T (v_mfma_f32_32x32x16_bf16), so each lane
//   owns one query column: softmax max/sum are in-lane plus one exchange between the
//   two 32-lane halves sharing a query.  The output is accumulated transposed too,
//   O^T += V^T P^T: P^T is the score accumulator itself (its 16 rows per lane are the
//   8+8 keys the B operand wants), and V^T comes straight from the row-major V tile
//   through ds_read_b64_tr_b16 transposing reads.
// * Online softmax in base 2 with 1/sqrt(64) folded into one FMA.  Probabilities are
//   taken against a running reference that is only raised when a tile could overflow
//   (tile sums >= 2^64), so neither tile maxima nor accumulator rescales are computed in
//   the common case (exact either way: the LSE uses the reference the sums were taken
//   against).
// * Scheduling: 1041 queries x 16 heads is only 144 units, too few for 256 CUs, so each
//   unit's key range is split.  Units are dealt to one queue per XCD (whole heads where
//   possible); each queue's (unit, key tile) iterations, laid out with a stride of U
//   tiles per unit, are cut into chunks, one per workgroup.  With U = T (the unit's
//   tile count) this is stream-K: chunks may straddle units, and the first n_first
//   chunks of a queue (served by the workgroups dispatched first on their CUs, which
//   run faster) hold E tiles against E1 for the rest.  With
//   U = k E >= T every unit is cut into k aligned pieces, so the workgroups holding the
//   query tiles of one head walk the same key tiles at the same time and share them in
//   L2.  A chunk that covers a whole unit writes its output directly; otherwise it
//   writes a partial result (its output normalised by its own row sum, in bf16, with
//   its reference m and row sum l) to its slot and a second launch merges each split
//   unit's partials in chunk order (deterministic; the kernel boundary is the only
//   synchronisation, so results do not depend on where the hardware places the
//   workgroups; the merge workgroups follow the queues' XCD mapping only so that the
//   partials are likely still in that XCD's L2).
#include <type_traits>

#include "rv_internal.h"

namespace rv {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef short i16x4 __attribute__((ext_vector_type(4)));
typedef short i16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int BQ = kAttnBQ;
constexpr int BK = kAttnBK;
constexpr int D = kHeadDim;
constexpr int TILE = BK * D;                    // one K or V tile: 64 rows x 128 bytes
constexpr int STAGE = 2 * TILE;                 // K tile then V tile
constexpr int NSTAGE = 4;                       // LDS ring: two tiles computed, two in flight
constexpr float kLn2 = 0.69314718055994531f;
constexpr float kLog2e = 1.44269504088896341f;
constexpr float kScaleLog2 = 1.44269504088896341f * 0.125f;  // log2(e) / sqrt(64)
constexpr float kOverflowGuard = 18446744073709551616.0f;  // 2^64
constexpr float kNegBig = -1.0e30f;

typedef __attribute__((address_space(3))) i16x4 lds_i16x4;

template <int P>
struct StageConst {
  static constexpr int value = P;
};

__device__ __forceinline__ f32x16 mfma32(bf16x8 a, bf16x8 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ uint2 to_bf16x4(float a, float b, float c, float d) {
  typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
  bf16x4 v = {(__bf16)a, (__bf16)b, (__bf16)c, (__bf16)d};
  return __builtin_bit_cast(uint2, v);
}

__device__ __forceinline__ int hw_xcc_id() { return __builtin_amdgcn_s_getreg((3 << 11) | 20) & 15; }

// Partner value of the other 32-lane half (lane l <-> l ^ 32): v_permlane32_swap returns
// the two halves exchanged between its operands, so the pair holds {own, partner} in
// some order on every lane; sums and maxima over the pair need no lane test.
__device__ __forceinline__ float half_max(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float half_sum(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

__device__ __forceinline__ int uniform(int x) { return __builtin_amdgcn_readfirstlane(x); }

// LDS tile layout: 64 rows of 128 bytes, no padding.  The 16-byte chunk c of row r is
// stored at chunk c ^ sw(r), sw(r) = (2 (r & 3) | (r >> 2) & 1) ^ 2 ((r >> 3) & 1), which
// takes 8 distinct values on every 8 aligned rows and, with the row's parity, 16 distinct
// (parity, chunk) pairs on every 16: the 16-byte K reads (one row per lane, 8 or 16
// lanes a cycle) and the transposing V reads (4 rows x 32 bytes per 16 lanes, the rows'
// 32-byte pieces on disjoint chunk pairs) are free of bank conflicts whether the LDS
// serves 128 or 256 bytes a cycle.
__device__ __forceinline__ int sw(int row) { return attn_tile_swizzle(row); }
__device__ __forceinline__ int swz(int row, int chunk) { return row * D + ((chunk ^ sw(row)) << 3); }

// Key/value rows of one head: the memory segment (row stride 64) followed by the frame
// (row stride H*64).  Tiles go straight from global memory to LDS
// (global_load_lds_dwordx4: lane l of a wave writes 16 bytes at the wave's LDS base +
// 16 l), so each thread fetches the global chunk that belongs at its LDS slot: thread
// tid fills physical chunk tid % 8 of rows tid / 8 and tid / 8 + 32, i.e. the global
// chunk (tid % 8) ^ sw(row) of those rows.  Addresses are a wave-uniform base
// plus a 32-bit per-thread byte offset fixed for the whole segment; the last tile of
// each part re-reads its last row in place of the rows past the end (always in
// bounds; their scores are masked).
struct TileCursor {
  const char* km;          // memory K / V rows of this head
  const char* vm;
  const char* kc;          // the frame's K / V rows of this head
  const char* vc;
  int64_t cur_tile;        // bytes between consecutive frame tiles: 64 * H * 64 * 2
  uint32_t off_m0, off_m1;     // thread byte offsets inside a full memory tile
  uint32_t off_c0, off_c1;     // ... inside a full frame tile
  uint32_t dt_m0, dt_m1;   // added for the last memory tile (rows clamped)
  uint32_t dt_c0, dt_c1;   // added for the last frame tile
  int nt_mem;              // memory tiles
  int t_last;              // index of the unit's last tile
  int mem_tail;            // valid rows of the last memory tile
  int tok_tail;            // valid rows of the last frame tile
};

__device__ __forceinline__ int tile_valid(const TileCursor& tc, int t) {
  int v = BK;
  if (t == tc.t_last) v = tc.tok_tail;
  if (t == tc.nt_mem - 1) v = tc.mem_tail;
  return v;
}

typedef __attribute__((address_space(3))) void lds_void;

__device__ __forceinline__ void lds_load16(const char* g, uint16_t* lds_wave_base) {
  __builtin_amdgcn_global_load_lds((const void*)g, (lds_void*)lds_wave_base, 16, 0, 0);
}

// Issue tile t's K and V loads into ring stage S (completion: vmcnt + barrier).
// `ldsw` is the LDS ring plus this wave's row block (rows 8w .. 8w+7 of a tile; the
// second load of each operand fills rows 32 + 8w ..).
template <int S>
__device__ __forceinline__ void load_tile(const TileCursor& tc, int t, uint16_t* ldsw) {
  const char *kb, *vb;
  uint32_t o0, o1;
  if (t < tc.nt_mem) {  // uniform branches
    kb = tc.km + (int64_t)t * (BK * D * 2);
    vb = tc.vm + (int64_t)t * (BK * D * 2);
    o0 = tc.off_m0;
    o1 = tc.off_m1;
    if (t == tc.nt_mem - 1) {  // (additive, so no select between two fields' addresses)
      o0 += tc.dt_m0;
      o1 += tc.dt_m1;
    }
  } else {
    const int tc_i = t - tc.nt_mem;
    kb = tc.kc + tc_i * tc.cur_tile;
    vb = tc.vc + tc_i * tc.cur_tile;
    o0 = tc.off_c0;
    o1 = tc.off_c1;
    if (t == tc.t_last) {
      o0 += tc.dt_c0;
      o1 += tc.dt_c1;
    }
  }
  uint16_t* st = ldsw + S * STAGE;
  lds_load16(kb + o0, st);
  lds_load16(kb + o1, st + 32 * D);
  lds_load16(vb + o0, st + TILE);
  lds_load16(vb + o1, st + TILE + 32 * D);
}

struct SoftmaxState {
  float m;      // running max of z * log2(e) / 8
  float l;      // this lane's share of the row sum
  f32x16 o0;    // O^T rows d = 0..31 for this lane's query (accumulator layout)
  f32x16 o1;    // d = 32..63
};

// One 64-key tile for this wave's 32 queries.  kFirst: the segment's first tile, whose
// running reference is still unset, so its maximum is taken directly (the exact path of
// a later tile, without the rescale of an empty state).
template <bool kFirst>
__device__ __forceinline__ void tile_compute(const uint16_t* stage, const bf16x8 (&qf)[4], int lane, int valid,
                                             SoftmaxState& sm) {
  const int l32 = lane & 31, half = lane >> 5;
  // Wave priority 1 from the score MFMAs through the softmax, 0 for the value product: of
  // the two waves sharing a SIMD, the one in the first part of its tile issues first, which
  // keeps the pair out of step so that one's MFMAs run under the other's vector work
  // (about +1 % per stream over a uniform priority).  Priority changes no result.
  __builtin_amdgcn_s_setprio(1);
  f32x16 s0 = {}, s1 = {};
#pragma unroll
  for (int ds = 0; ds < 4; ++ds) {
    const bf16x8 ka = *reinterpret_cast<const bf16x8*>(&stage[swz(l32, ds * 2 + half)]);
    const bf16x8 kb = *reinterpret_cast<const bf16x8*>(&stage[swz(32 + l32, ds * 2 + half)]);
    s0 = mfma32(ka, qf[ds], s0);
    s1 = mfma32(kb, qf[ds], s1);
  }
  // accumulator entry r of this lane: key 8*(r/4) + 4*half + r%4 (+32 in s1)
  if (__builtin_expect(valid < BK, 0)) {
    // keys >= valid get -1e30: sat(key + 1 - valid) is 1 exactly for them, 0 otherwise
    // (arithmetic masking keeps the 32 lane masks out of scalar registers)
    const float fv = (float)(valid - 4 * half - 1);
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const float key = (float)(8 * (r >> 2) + (r & 3));
      s0[r] = fmaf(__saturatef(key - fv), kNegBig, s0[r]);
      s1[r] = fmaf(__saturatef(key + 32.0f - fv), kNegBig, s1[r]);
    }
  }
  // P = 2^(z*log2e/8 - m) against the running reference m.  Softmax does not depend on
  // the reference, so the tile maximum is only needed when some p could overflow: a
  // lane whose tile sum reaches 2^64 (or inf; every p starts as inf while m is unset)
  // makes the wave take the exact path -- raise m to the tile maximum, rescale the
  // accumulators, recompute P.  Terms far below the reference underflow to 0, exactly
  // as they would relative to the true maximum.
  bf16x8 p[4];
  float rsum = -0.f;  // -0 + x == x: the first add folds away
  auto exact = [&]() {
    float mx = fmaxf(s0[0], s1[0]);
#pragma unroll
    for (int r = 1; r < 16; ++r) mx = fmaxf(mx, fmaxf(s0[r], s1[r]));
    const float m_new = fmaxf(sm.m, half_max(mx) * kScaleLog2);
    if (!kFirst) {
      const float alpha = __builtin_amdgcn_exp2f(sm.m - m_new);
      sm.l *= alpha;
      sm.o0 *= alpha;
      sm.o1 *= alpha;
    }
    sm.m = m_new;
    rsum = -0.f;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const float e0 = __builtin_amdgcn_exp2f(fmaf(s0[r], kScaleLog2, -sm.m));
      const float e1 = __builtin_amdgcn_exp2f(fmaf(s1[r], kScaleLog2, -sm.m));
      rsum += e0 + e1;
      p[r >> 3][r & 7] = (__bf16)e0;
      p[2 + (r >> 3)][r & 7] = (__bf16)e1;
    }
  };
  if (kFirst) {
    exact();
  } else {
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const float e0 = __builtin_amdgcn_exp2f(fmaf(s0[r], kScaleLog2, -sm.m));
      const float e1 = __builtin_amdgcn_exp2f(fmaf(s1[r], kScaleLog2, -sm.m));
      rsum += e0 + e1;
      p[r >> 3][r & 7] = (__bf16)e0;
      p[2 + (r >> 3)][r & 7] = (__bf16)e1;
    }
    if (__any(!(rsum < kOverflowGuard))) exact();
  }
  sm.l += rsum;
  __builtin_amdgcn_s_setprio(0);

  // V^T operand through transposing LDS reads.  Within each 16-lane group, lane i
  // receives element i%4 of the 8-byte chunk addressed by lane 4r + i/4 (r = 0..3), so
  // lane 4r + j points at row (key) r, columns d0 + 4j .. +3: lane i then holds
  // V[key r][d0 + i] for the 4 keys.  Keys follow the P^T slot order: for k-step ks and
  // lane half hh, slots 0..3 are keys ks*16 + 4hh + r, slots 4..7 keys ks*16 + 8 + 4hh + r.
  const uint16_t* vt = stage + TILE;
  const int g = lane >> 4, i16 = lane & 15, rr = i16 >> 2, jj = i16 & 3, hh = g >> 1;
  const int col = 16 * (g & 1) + 4 * jj;  // logical column (elements) within a 32-dim block
#pragma unroll
  for (int ks = 0; ks < 4; ++ks) {
    const int row = ks * 16 + 4 * hh + rr;
#pragma unroll
    for (int db = 0; db < 2; ++db) {
      const int lcol = db * 32 + col;
      const i16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
          (lds_i16x4*)(vt + swz(row, lcol >> 3) + (lcol & 7)));
      const i16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
          (lds_i16x4*)(vt + swz(row + 8, lcol >> 3) + (lcol & 7)));
      const i16x8 w = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
      const bf16x8 va = __builtin_bit_cast(bf16x8, w);
      if (db == 0)
        sm.o0 = mfma32(va, p[ks], sm.o0);
      else
        sm.o1 = mfma32(va, p[ks], sm.o1);
    }
  }
}

// Partial slots: chunk c's segment of a unit writes its output rows normalised by its
// own row sum, in bf16 ([BQ][64]), then its reference m[BQ] and row sum l[BQ] (fp32).
constexpr int kSlotStatsFloat = BQ * D / 2;
constexpr int kMergeRows = 32;   // output rows per merge workgroup (8 threads per row)
constexpr int kMergeMax = 8;     // partials whose loads are in flight together

// First iteration of chunk c of a queue (chunk arithmetic: rv_plan.h).
__device__ __forceinline__ int64_t chunk_start(const AttnArgs& a, int c) { return chunk_cut(a, c); }

// Partial slot of chunk c's segment of unit ui: slot 0 if the chunk starts inside the
// unit, slot 1 if it began in an earlier unit.
__device__ __forceinline__ const float* slot_ptr(const AttnArgs& a, int q, int c, int ui) {
  const int slot = 2 * (a.chunk_base[q] + c) + (chunk_start(a, c) >= (int64_t)ui * a.U ? 0 : 1);
  return a.part + (int64_t)slot * kAttnSlotFloats;
}

// Merge the partials of chunks c_first..c_last (in chunk order) for rows
// rb*32 .. rb*32+31 of `unit` and write the final output rows and LSE.  Partial j is
// weighted by 2^(m_j - M) l_j (M the largest m).  Thread -> (row, 8 dims); up to eight
// partials' statistics and rows are loaded in one round trip (indices clamped, surplus
// weights zero).
__device__ void merge_rows(const AttnArgs& a, int q, int unit, int ui, int rb, int c_first, int c_last) {
  const int tid = threadIdx.x;
  const int h = unit / a.q_tiles, qt = unit % a.q_tiles;
  const int row = rb * kMergeRows + (tid >> 3), d8 = (tid & 7) * 8;
  const int qi = qt * BQ + row;
  if (qi >= a.n_tokens) return;
  float mmax = kNegBig, L = 0.f;
  float acc[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) acc[e] = 0.f;
  for (int c0 = c_first; c0 <= c_last; c0 += kMergeMax) {
    const int n = min(kMergeMax, c_last - c0 + 1);
    float mv[kMergeMax], lv[kMergeMax];
    uint4 v[kMergeMax];
#pragma unroll
    for (int j = 0; j < kMergeMax; ++j) {
      const float* ps = slot_ptr(a, q, min(c0 + j, c_last), ui);
      mv[j] = ps[kSlotStatsFloat + row];
      lv[j] = ps[kSlotStatsFloat + BQ + row];
      v[j] = *reinterpret_cast<const uint4*>(reinterpret_cast<const uint16_t*>(ps) + row * D + d8);
    }
    float m_new = mmax;
#pragma unroll
    for (int j = 0; j < kMergeMax; ++j) m_new = fmaxf(m_new, mv[j]);  // clamped copies repeat a real one
    const float scale = __builtin_amdgcn_exp2f(mmax - m_new);
    L *= scale;
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[e] *= scale;
    mmax = m_new;
#pragma unroll
    for (int j = 0; j < kMergeMax; ++j) {
      const float w = j < n ? __builtin_amdgcn_exp2f(mv[j] - mmax) * lv[j] : 0.f;
      L += w;
      const uint32_t wd[4] = {v[j].x, v[j].y, v[j].z, v[j].w};
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        acc[2 * i] = fmaf(w, __uint_as_float(wd[i] << 16), acc[2 * i]);
        acc[2 * i + 1] = fmaf(w, __uint_as_float(wd[i] & 0xFFFF0000u), acc[2 * i + 1]);
      }
    }
  }
  const float inv = 1.f / L;
  uint16_t* op = a.out + ((int64_t)qi * a.n_heads + h) * D + d8;
  const uint2 lo = to_bf16x4(acc[0] * inv, acc[1] * inv, acc[2] * inv, acc[3] * inv);
  const uint2 hi = to_bf16x4(acc[4] * inv, acc[5] * inv, acc[6] * inv, acc[7] * inv);
  *reinterpret_cast<uint4*>(op) = make_uint4(lo.x, lo.y, hi.x, hi.y);
  if (d8 == 0) a.lse[(int64_t)h * a.n_tokens + qi] = (mmax + __log2f(L)) * kLn2;
}

// Key tiles t0..t1-1 of `unit` (queue-local index ui) as part of chunk c of queue q.
__device__ void process_segment(const AttnArgs& a, int q, int c, int unit, int ui, int t0, int t1, uint16_t* lds) {
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = uniform(tid >> 6);
  const int l32 = lane & 31, half = lane >> 5;
  unit = uniform(unit);
  t0 = uniform(t0);
  t1 = uniform(t1);
  const int h = uniform(unit / a.q_tiles), qt = uniform(unit % a.q_tiles);
  const int q0 = qt * BQ + wave * 32;
  const int qi = q0 + l32;
  const bool wave_active = q0 < a.n_tokens;

  TileCursor tc;
  {
    const int r = tid >> 3, c8 = (tid & 7) * 8, rs = a.n_heads * D;
    tc.km = reinterpret_cast<const char*>(a.memK + (int64_t)h * a.head_stride * D);
    tc.vm = reinterpret_cast<const char*>(a.memV + (int64_t)h * a.head_stride * D);
    tc.kc = reinterpret_cast<const char*>(a.K + (int64_t)h * D);
    tc.vc = reinterpret_cast<const char*>(a.V + (int64_t)h * D);
    tc.cur_tile = (int64_t)BK * rs * 2;
    tc.nt_mem = a.nt_mem;
    tc.t_last = a.T - 1;
    tc.mem_tail = a.nt_mem > 0 ? (int)(a.mem_len - (int64_t)(a.nt_mem - 1) * BK) : BK;
    tc.tok_tail = a.T > a.nt_mem ? a.n_fkeys - (a.T - 1 - a.nt_mem) * BK : BK;
    const int r1 = r + 32;
    const int g0 = c8 ^ (sw(r) << 3), g1 = c8 ^ (sw(r1) << 3);
    tc.off_m0 = 2u * (uint32_t)(r * D + g0);
    tc.off_m1 = 2u * (uint32_t)(r1 * D + g1);
    tc.off_c0 = 2u * (uint32_t)(r * rs + g0);
    tc.off_c1 = 2u * (uint32_t)(r1 * rs + g1);
    tc.dt_m0 = 2u * (uint32_t)(min(r, tc.mem_tail - 1) * D + g0) - tc.off_m0;
    tc.dt_m1 = 2u * (uint32_t)(min(r1, tc.mem_tail - 1) * D + g1) - tc.off_m1;
    tc.dt_c0 = 2u * (uint32_t)(min(r, tc.tok_tail - 1) * rs + g0) - tc.off_c0;
    tc.dt_c1 = 2u * (uint32_t)(min(r1, tc.tok_tail - 1) * rs + g1) - tc.off_c1;
  }
  uint16_t* const ldsw = lds + wave * 8 * D;

  // B operand of S^T = K Q^T: this lane's query, head dims ds*16 + half*8 .. +7.
  bf16x8 qf[4];
  {
    const uint16_t* qp = a.Q + ((int64_t)min(qi, a.n_tokens - 1) * a.n_heads + h) * D + half * 8;
#pragma unroll
    for (int ds = 0; ds < 4; ++ds) qf[ds] = *reinterpret_cast<const bf16x8*>(qp + ds * 16);
  }
  SoftmaxState sm;
  sm.m = kNegBig;
  sm.l = 0.f;
  sm.o0 = f32x16{};
  sm.o1 = f32x16{};

  // Ring of NSTAGE (4) tiles, two computed per barrier: tile t0 + j lives in stage j % 4,
  // so every stage offset is a compile-time constant of the unrolled loop.  The next
  // pair streams into the two stages the previous pair used (freed at the last barrier)
  // while this pair is computed.  The first step is peeled off: its first tile sets the
  // running reference.
  auto step = [&](auto phase, auto first, int t) {
    constexpr int P = decltype(phase)::value;
    if (t + 2 < t1) load_tile<(P + 2) % NSTAGE>(tc, t + 2, ldsw);
    if (t + 3 < t1) load_tile<(P + 3) % NSTAGE>(tc, t + 3, ldsw);
    if (wave_active) {
      tile_compute<decltype(first)::value>(lds + P * STAGE, qf, lane, tile_valid(tc, t), sm);
      if (t + 1 < t1) tile_compute<false>(lds + (P + 1) * STAGE, qf, lane, tile_valid(tc, t + 1), sm);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
  };
  load_tile<0>(tc, t0, ldsw);
  if (t0 + 1 < t1) load_tile<1>(tc, t0 + 1, ldsw);
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  step(StageConst<0>{}, std::true_type{}, t0);
  for (int t = t0 + 2; t < t1; t = uniform(t + 4)) {
    step(StageConst<2>{}, std::false_type{}, t);
    if (t + 2 >= t1) break;
    step(StageConst<0>{}, std::false_type{}, t + 2);
  }

  const float l_tot = half_sum(sm.l);
  // The output rows (normalised by the row sum, bf16) go out through LDS: each wave stages
  // its 32 rows (row stride kOutStageRow elements, so that the 32 rows' 8-byte pieces spread
  // over the banks), then writes whole 128-byte rows, 8 lanes a row (before: each store
  // wrote 16 bytes into each of 32 rows; 2 % per stream).  The ring is free: the last
  // step ended with a barrier.
  constexpr int kOutStageRow = D + 8;
  uint16_t* const st = lds + wave * 32 * kOutStageRow;
  if (wave_active) {
    const float inv = 1.f / l_tot;
    uint16_t* sp = st + l32 * kOutStageRow + 4 * half;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      *reinterpret_cast<uint2*>(sp + 8 * j) =
          to_bf16x4(sm.o0[4 * j] * inv, sm.o0[4 * j + 1] * inv, sm.o0[4 * j + 2] * inv, sm.o0[4 * j + 3] * inv);
      *reinterpret_cast<uint2*>(sp + 32 + 8 * j) =
          to_bf16x4(sm.o1[4 * j] * inv, sm.o1[4 * j + 1] * inv, sm.o1[4 * j + 2] * inv, sm.o1[4 * j + 3] * inv);
    }
  }
  __syncthreads();
  const int r8 = lane >> 3, c8 = (lane & 7) * 8;
  if (t0 == 0 && t1 == a.T) {
    // the whole unit in this chunk: final output rows and LSE
    if (wave_active) {
      if (half == 0 && qi < a.n_tokens) a.lse[(int64_t)h * a.n_tokens + qi] = (sm.m + __log2f(l_tot)) * kLn2;
#pragma unroll
      for (int pass = 0; pass < 4; ++pass) {
        const int r = pass * 8 + r8, qr = q0 + r;
        if (qr < a.n_tokens)
          *reinterpret_cast<uint4*>(a.out + ((int64_t)qr * a.n_heads + h) * D + c8) =
              *reinterpret_cast<const uint4*>(st + r * kOutStageRow + c8);
      }
    }
  } else {
    // partial result, merged by the second launch: the normalised output rows in bf16
    // (the merge weights them by 2^(m - M) l), then m and l in fp32
    const int seg = chunk_start(a, c) >= (int64_t)ui * a.U ? 0 : 1;
    float* ps = a.part + (int64_t)(2 * (a.chunk_base[q] + c) + seg) * kAttnSlotFloats;
    if (wave_active) {
      if (half == 0) {
        const int row = wave * 32 + l32;
        ps[kSlotStatsFloat + row] = sm.m;
        ps[kSlotStatsFloat + BQ + row] = l_tot;
      }
      uint16_t* po = reinterpret_cast<uint16_t*>(ps) + wave * 32 * D;
#pragma unroll
      for (int pass = 0; pass < 4; ++pass) {
        const int r = pass * 8 + r8;
        *reinterpret_cast<uint4*>(po + r * D + c8) = *reinterpret_cast<const uint4*>(st + r * kOutStageRow + c8);
      }
    }
  }
  __syncthreads();  // (the ring is the next segment's)
}

// ---- long chunks --------------------------------------------------------------------
//
// The forward launch where a workgroup has many tiles (plan_long_chunks).  The same units,
// chunks, tiles and partial results; another split of a workgroup's work over its waves.
// Wave (wq, kh) takes queries 64 wq .. + 63 of the unit as two 32-query blocks and keys 32 kh
// .. + 31 of every tile, so that each K and V fragment read from LDS serves two blocks (half
// the LDS reads: 5.5 M instead of 10.5 M wave instructions at 52,000 rows), and the work is
// pipelined by half a tile: the score MFMAs of the next block and the value MFMAs of the one
// before run under each block's exponentials.  The two key halves meet in LDS at a segment's
// end.
//
// The matrix core is busy 44 % of the cycles, the vector ALU 58 %; waves wait for 21 % of theirs
// and hold an instruction that does not issue for 29 %; and the clock is at about 2.1 GHz with
// data like the streams' (2.4 with zeros).  Against attn_fwd_kernel (53,300 keys, 1041 tokens, 16
// heads) the launch takes 4.20 M cycles over the XCDs instead of 4.45 M, and 245 us instead of
// 254.  On stream-K plans of 90 tiles a chunk or more the step takes 0 to 7 % less (16 heads, 1041
// tokens: 20,000 rows 106 -> 106 us, 52,000 rows 253 -> 249-251; 1374 tokens: 20,000 rows 136 ->
// 133, 52,000 rows 326 -> 305; 12 heads, 1041 tokens, 52,000 rows 206 -> 194), the same at 40 to
// 60, and up to 2.5 us more below: the longer prologue, the exchange at the end and odd tiles
// (1041 tokens, empty memory: 15.3 -> 17.5).
// Added to the scores of keys past a tile's end.  Scaled, it lies below kNegBig, the lowest
// softmax reference here as in attn_fwd_kernel, so that a wave whose 32 keys are all masked
// gets p = 0 for each.
constexpr float kLongMask = -1.0e31f;
static_assert(kLongMask * kScaleLog2 < kNegBig, "masked keys lie below every reference");

__device__ __forceinline__ const char* uniform_ptr(const char* p) {
  const uint64_t x = reinterpret_cast<uint64_t>(p);
  const uint32_t lo = (uint32_t)uniform((int)(uint32_t)x), hi = (uint32_t)uniform((int)(uint32_t)(x >> 32));
  return reinterpret_cast<const char*>((uint64_t)hi << 32 | lo);
}

// As TileCursor, with the byte offsets formed from the thread's row and the tile's row stride.
struct LongCursor {
  const char* km;          // memory K / V rows of this head
  const char* vm;
  const char* kc;          // the frame's K / V rows of this head
  const char* vc;
  uint32_t cur_row;        // bytes between consecutive frame rows: H * 64 * 2
  uint32_t r, g0, g1;      // this thread's row (and row + 32), and byte offsets in the rows
  int nt_mem;              // memory tiles
  int t_last;              // index of the unit's last tile
  int mem_tail;            // valid rows of the last memory tile
  int tok_tail;            // valid rows of the last frame tile
};

__device__ __forceinline__ int long_tile_valid(const LongCursor& tc, int t) {
  int v = BK;
  if (t == tc.t_last) v = tc.tok_tail;
  if (t == tc.nt_mem - 1) v = tc.mem_tail;
  return v;
}

// Lane l's 16 bytes at base + off go to LDS byte lds + 16 l.  (Assembly: the compiler would
// wait for every such load in flight before the transposing LDS reads, whichever slots they
// read; the pipeline below waits for them itself, at the end of a step.  No register is
// written.  The wait states are those a scalar that a vector instruction wrote needs before a
// load reads it: the compiler does not look for such hazards here.)
__device__ __forceinline__ void lds_load16_asm(const char* base, uint32_t off, uint32_t lds) {
  asm volatile("s_nop 4\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(off), "s"(base), "{m0}"(lds));
}

// Global addresses of tile t: the K and V bases and this thread's byte offsets of its two
// 16-byte pieces (selects, no branches: they are computed in the middle of a tile's MFMAs).
struct LongSrc {
  const char *k, *v;
  uint32_t o0, o1;
};
__device__ __forceinline__ LongSrc long_src(const LongCursor& tc, int t) {
  const bool mem = t < tc.nt_mem;  // uniform
  const uint32_t row = mem ? D * 2 : tc.cur_row;
  const int64_t at = (int64_t)(mem ? t : t - tc.nt_mem) * BK * row;
  const uint32_t last = (uint32_t)long_tile_valid(tc, t) - 1;
  LongSrc ts;
  ts.k = uniform_ptr((mem ? tc.km : tc.kc) + at);
  ts.v = uniform_ptr((mem ? tc.vm : tc.vc) + at);
  ts.o0 = min(tc.r, last) * row + tc.g0;
  ts.o1 = min(tc.r + 32, last) * row + tc.g1;
  return ts;
}

// Issue one tile's loads into an LDS slot (completion: vmcnt + barrier).  `slot` is the byte
// address of the tile plus this wave's row block (rows 8w .. 8w+7; the second load fills rows
// 32 + 8w ..).
__device__ __forceinline__ void load_rows(const char* base, const LongSrc& ts, uint32_t slot) {
  lds_load16_asm(base, ts.o0, slot);
  lds_load16_asm(base, ts.o1, slot + 32 * D * 2);
}

// One 32-query block of a wave: its softmax state over the wave's keys.
struct QueryBlock {
  float m;      // reference of the exponentials (z * log2(e) / 8)
  float l;      // this lane's share of the row sum
  f32x16 o0;    // O^T rows d = 0..31 for this lane's query (accumulator layout)
  f32x16 o1;    // d = 32..63
};

// Scores of keys >= valid (of the wave's 32) fall by 1e31: sat(key + 1 - valid) is 1 exactly
// for them, 0 otherwise (arithmetic masking keeps 16 lane masks out of scalar registers).
// Accumulator entry r of a lane is key 8*(r/4) + 4*half + r%4.
__device__ __forceinline__ void mask_keys(f32x16& s, int half, int valid) {
  const float fv = (float)(valid - 4 * half - 1);
#pragma unroll
  for (int r = 0; r < 16; ++r) s[r] = fmaf(__saturatef((float)(8 * (r >> 2) + (r & 3)) - fv), kLongMask, s[r]);
}

// Maximum of the 32 keys' scaled scores of each query, at least kNegBig.
__device__ __forceinline__ float tile_ref(const f32x16& s) {
  float mx = s[0];
#pragma unroll
  for (int r = 1; r < 16; ++r) mx = fmaxf(mx, s[r]);
  return fmaxf(half_max(mx) * kScaleLog2, kNegBig);
}

// p = 2^(z log2(e) / 8 - m) of one query block's 32 keys, as the value product's operand;
// returns this lane's share of their sum.
__device__ __forceinline__ float exponentials(const f32x16& s, float m, bf16x8 (&p)[2]) {
  float rsum = -0.f;  // -0 + x == x: the first add folds away
#pragma unroll
  for (int r = 0; r < 16; r += 2) {
    const float e0 = __builtin_amdgcn_exp2f(fmaf(s[r], kScaleLog2, -m));
    const float e1 = __builtin_amdgcn_exp2f(fmaf(s[r + 1], kScaleLog2, -m));
    rsum += e0 + e1;
    p[r >> 3][r & 7] = (__bf16)e0;
    p[r >> 3][(r & 7) + 1] = (__bf16)e1;
  }
  return rsum;
}

// The end of a block's softmax: adds the row sum, or, where some lane's sum reaches 2^64 (or
// inf), takes the exact path -- raise the reference to the keys' maximum, rescale the
// accumulators, recompute p.  Terms far below the reference underflow to 0, exactly as they
// would relative to the true maximum, so nothing else depends on the reference.
__device__ __forceinline__ void add_row_sum(const f32x16& s, QueryBlock& b, bf16x8 (&p)[2], float rsum) {
  asm volatile("" : "+v"(p[0]), "+v"(p[1]));  // (p is formed before the branch, among the MFMAs)
  if (__builtin_expect(__any(!(rsum < kOverflowGuard)), 0)) {
    const float m_new = fmaxf(b.m, tile_ref(s));
    const float alpha = __builtin_amdgcn_exp2f(b.m - m_new);
    b.l *= alpha;
    b.o0 *= alpha;
    b.o1 *= alpha;
    b.m = m_new;
    rsum = exponentials(s, m_new, p);
  }
  b.l += rsum;
}

// The tile a segment starts at, `done` iterations into chunk c.  The chunks of a head cover
// different key ranges, but the sums over a segment's keys take any order: with chunks of E
// tiles, the chunk that has worked for i iterations takes the tile that is i modulo E where its
// segment holds one, so that a head's chunks are at the same few tiles at a time (one for each E
// tiles of the context) and find them in their XCD's L2.  In key order the chunks of plans that
// are not aligned with the units drift apart and fetch the keys from beyond L2 once for each
// query tile (700 tokens, 16 heads: 30,000 rows 113 -> 104 us, 52,000 rows 188 -> 167; 1041
// tokens, 12 heads, 52,000 rows 202 -> 192; aligned plans within 1 %).
__device__ __forceinline__ int first_tile(const AttnArgs& a, int c, int done, int t0, int t1) {
  const int E = (c < a.n_first ? a.E : a.E1) / kCutScale;
  if (E <= 1) return t0;
  const int ahead = (done - t0) % E;
  const int ts = t0 + (ahead < 0 ? ahead + E : ahead);
  return ts < t1 ? ts : t0;
}

// Key tiles t0..t1-1 of `unit` (queue-local index ui) as part of chunk c of queue q, in the
// order ts..t1-1, t0..ts-1.
__device__ __forceinline__ void process_long_segment(const AttnArgs& a, int q, int c, int unit, int ui, int t0,
                                                     int t1, int ts, uint16_t* lds) {
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = uniform(tid >> 6);
  const int l32 = lane & 31, half = lane >> 5;
  unit = uniform(unit);
  t0 = uniform(t0);
  t1 = uniform(t1);
  ts = uniform(ts);
  const int n = t1 - t0;              // tiles, taken in the order of index 0 .. n - 1
  const int n_up = t1 - ts;           // indices before the order wraps to t0
  const int wrap = n_up < n ? n : 0;  // subtracted from ts + i for i >= n_up
  auto tile_at = [&](int i) { return ts + i - (i >= n_up ? wrap : 0); };
  const int h = uniform(unit / a.q_tiles), qt = uniform(unit % a.q_tiles);
  const int q0 = qt * BQ + wave * 32;
  const int qi = q0 + l32;
  const bool wave_active = q0 < a.n_tokens;

  LongCursor tc;
  {
    tc.km = reinterpret_cast<const char*>(a.memK + (int64_t)h * a.head_stride * D);
    tc.vm = reinterpret_cast<const char*>(a.memV + (int64_t)h * a.head_stride * D);
    tc.kc = reinterpret_cast<const char*>(a.K + (int64_t)h * D);
    tc.vc = reinterpret_cast<const char*>(a.V + (int64_t)h * D);
    tc.cur_row = 2u * (uint32_t)(a.n_heads * D);
    tc.r = tid >> 3;
    tc.g0 = 16u * ((tid & 7) ^ sw(tid >> 3));
    tc.g1 = 16u * ((tid & 7) ^ sw((tid >> 3) + 32));
    tc.nt_mem = a.nt_mem;
    tc.t_last = a.T - 1;
    tc.mem_tail = a.nt_mem > 0 ? (int)(a.mem_len - (int64_t)(a.nt_mem - 1) * BK) : BK;
    tc.tok_tail = a.T > a.nt_mem ? a.n_fkeys - (a.T - 1 - a.nt_mem) * BK : BK;
  }
  // Wave (wq, kh): query blocks 64 wq + 0..31 and + 32..63 of the unit, and keys 32 kh ..
  // + 31 of every tile.
  const int wq = wave >> 1, kh = wave & 1;
  const bool computes = qt * BQ + 64 * wq < a.n_tokens;

  // B operand of S^T = K Q^T: this lane's two queries, head dims ds*16 + half*8 .. +7.
  bf16x8 qf[2][4];
#pragma unroll
  for (int qb = 0; qb < 2; ++qb) {
    const int qr = min(qt * BQ + 64 * wq + 32 * qb + l32, a.n_tokens - 1);
    const uint16_t* qp = a.Q + ((int64_t)qr * a.n_heads + h) * D + half * 8;
#pragma unroll
    for (int ds = 0; ds < 4; ++ds) qf[qb][ds] = *reinterpret_cast<const bf16x8*>(qp + ds * 16);
  }
  QueryBlock b0, b1;
  b0.l = b1.l = 0.f;
  b0.o0 = b0.o1 = b1.o0 = b1.o1 = f32x16{};

  constexpr uint32_t kSlot = TILE * 2, kVRing = 4 * kSlot;
  // This lane's byte offsets in a tile.  K (A operand of S^T): row 32 kh + l32, chunk
  // 2 ds + half.  V^T operand through transposing LDS reads: within each 16-lane group, lane
  // i receives element i%4 of the 8-byte chunk addressed by lane 4r + i/4 (r = 0..3), so lane
  // 4r + j points at row (key) r, columns d0 + 4j .. +3: lane i then holds V[key r][d0 + i]
  // for the 4 keys.  Keys follow the P^T slot order: for k-step ks and lane half hh, slots
  // 0..3 are keys ks*16 + 4hh + r, slots 4..7 keys ks*16 + 8 + 4hh + r.
  uint32_t ko[4], vo[2][2];   // byte offsets in the ring, of the half the next step reads
  {
    const int g = lane >> 4, i16 = lane & 15, rr = i16 >> 2, jj = i16 & 3;
    const int col = 16 * (g & 1) + 4 * jj;
#pragma unroll
    for (int ds = 0; ds < 4; ++ds) ko[ds] = 2 * swz(32 * kh + l32, 2 * ds + half);
#pragma unroll
    for (int hi = 0; hi < 2; ++hi)
#pragma unroll
      for (int db = 0; db < 2; ++db)
        vo[hi][db] = 2 * (swz(32 * kh + 8 * hi + 4 * (g >> 1) + rr, (db * 32 + col) >> 3) + (col & 7));
  }
  bf16x8 kf[4], vf[2][2];
  f32x16 s0, s1;
  bf16x8 p0[2], p1[2];
  typedef __attribute__((address_space(3))) const char lds_char;
  typedef __attribute__((address_space(3))) const bf16x8 lds_bf16x8;
  lds_char* const ldsb = (lds_char*)(lds_void*)lds;
  auto read_k = [&](int slot) {
#pragma unroll
    for (int ds = 0; ds < 4; ++ds) kf[ds] = *(lds_bf16x8*)(ldsb + ko[ds] + slot * kSlot);
  };
  auto read_v = [&](int slot) {
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int db = 0; db < 2; ++db) {
        const int at = kVRing + slot * kSlot + ks * 16 * D * 2;
        const i16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4*)(ldsb + vo[0][db] + at));
        const i16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4*)(ldsb + vo[1][db] + at));
        vf[ks][db] = __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
      }
  };
  auto scores = [&](const bf16x8 (&q)[4], f32x16& s) {
    s = f32x16{};
#pragma unroll
    for (int ds = 0; ds < 4; ++ds) s = mfma32(kf[ds], q[ds], s);
  };
  auto values = [&](const bf16x8 (&p)[2], QueryBlock& b) {
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      b.o0 = mfma32(vf[ks][0], p[ks], b.o0);
      b.o1 = mfma32(vf[ks][1], p[ks], b.o1);
    }
  };

  // The ring: four K slots, then four V slots; `ring` is K slot 0 plus this wave's row block.
  const uint32_t ring = (uint32_t)(uintptr_t)(lds_void*)lds + wave * 8 * D * 2;
  auto flip = [&](auto& off) {  // to the other half of the ring
#pragma unroll
    for (auto& x : off) x ^= 2 * kSlot;
  };
  auto tile_keys = [&](int t) { return long_tile_valid(tc, tile_at(t)) - 32 * kh; };  // valid, of the wave's 32
  // Running addresses of the loads of a step at index t: K of index t + 3 and V of t + 2, while
  // those tiles and that of t + 4 follow one another in one part (memory or frame) and are full
  // (t + 4 < run_end).
  const char *k3 = tc.km, *v2 = tc.vm;
  uint32_t step_bytes = 0;
  LongSrc off{};
  int run_end = 0;
  auto set_run = [&](int t) {
    const int at = tile_at(t + 2);
    const bool mem = at < tc.nt_mem;
    const uint32_t row = mem ? D * 2 : tc.cur_row;
    step_bytes = BK * row;
    const int64_t i = at - (mem ? 0 : tc.nt_mem);
    k3 = uniform_ptr((mem ? tc.km : tc.kc) + (i + 1) * step_bytes);
    v2 = uniform_ptr((mem ? tc.vm : tc.vc) + i * step_bytes);
    off.o0 = tc.r * row + tc.g0;
    off.o1 = (tc.r + 32) * row + tc.g1;
    const int full = mem ? tc.nt_mem - (tc.mem_tail < BK) : tc.t_last + 1 - (tc.tok_tail < BK);
    run_end = uniform(t + 2 + min(full - at, (t + 2 < n_up ? n_up : n) - (t + 2)));
  };
  // What this wave does at each point of the ring's schedule (long_ring).  A step's loads of
  // full tiles of one part go by running addresses, others by long_src.
  bool run = false;
  auto ops = ring_ops(
      [&](RingLoadPair x) __attribute__((always_inline)) {
        const LongSrc src = long_src(tc, tile_at(x.i));
        load_rows(src.k, src, ring + x.slot * kSlot);
        load_rows(src.v, src, ring + kVRing + x.slot * kSlot);
      },
      [&](RingLoadK x) __attribute__((always_inline)) {
        const LongSrc src = long_src(tc, tile_at(x.i));
        load_rows(src.k, src, ring + x.slot * kSlot);
      },
      // (the query fragments pass through the first wait: the compiler's own wait for them
      // belongs there, not in the loop, where it would be a wait for the tiles in flight)
      [&](RingFirstArrived) __attribute__((always_inline)) {
        asm volatile("s_waitcnt vmcnt(0)"
                     : "+v"(qf[0][0]), "+v"(qf[0][1]), "+v"(qf[0][2]), "+v"(qf[0][3]), "+v"(qf[1][0]),
                       "+v"(qf[1][1]), "+v"(qf[1][2]), "+v"(qf[1][3])::"memory");
        __syncthreads();
      },
      [&](RingArrived) __attribute__((always_inline)) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
      },
      [&](RingBarrier) __attribute__((always_inline)) { __syncthreads(); },
      [&](RingReadFirstK) __attribute__((always_inline)) { read_k(0); },
      // The first tile's maxima are the references; its second block's scores are formed again
      // in the pipeline, and the pipeline's first value product multiplies zeros.
      [&](RingFirstScores) __attribute__((always_inline)) {
        const int valid = tile_keys(0);
        scores(qf[1], s1);
        scores(qf[0], s0);
        if (valid < 32) mask_keys(s1, half, valid);
        b1.m = tile_ref(s1);
        f32x16 sm = s0;
        if (valid < 32) mask_keys(sm, half, valid);
        b0.m = tile_ref(sm);
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          p1[i] = bf16x8{};
          vf[i][0] = vf[i][1] = bf16x8{};
        }
      },
      [&](RingStep x) __attribute__((always_inline)) {
        if (x.t + 2 >= run_end && x.t + 2 < n) set_run(x.t);
        run = x.t + 4 < run_end;
      },
      [&](RingLoads x) __attribute__((always_inline)) {
        if (run) {
          const uint32_t at = x.second ? step_bytes : 0;
          load_rows(v2 + at, off, ring + kVRing + x.v_slot * kSlot);
          load_rows(k3 + at, off, ring + x.k_slot * kSlot);
        } else {
          if (x.v < n) {
            const LongSrc src = long_src(tc, tile_at(x.v));
            load_rows(src.v, src, ring + kVRing + x.v_slot * kSlot);
          }
          if (x.k < n) {
            const LongSrc src = long_src(tc, tile_at(x.k));
            load_rows(src.k, src, ring + x.k_slot * kSlot);
          }
        }
        if (x.second) {
          k3 += 2 * step_bytes;
          v2 += 2 * step_bytes;
        }
      },
      [&](RingTileA x) __attribute__((always_inline)) {
        const int valid = tile_keys(x.t);
        if (__builtin_expect(valid < 32, 0)) mask_keys(s0, half, valid);
        scores(qf[1], s1);
        const float r0 = exponentials(s0, b0.m, p0);
        read_k(x.slot);
        values(p1, b1);
        add_row_sum(s0, b0, p0, r0);
      },
      [&](RingTileB x) __attribute__((always_inline)) {
        const int valid = tile_keys(x.t);
        if (__builtin_expect(valid < 32, 0)) mask_keys(s1, half, valid);
        read_v(x.slot);
        scores(qf[0], s0);
        const float r1 = exponentials(s1, b1.m, p1);
        values(p0, b0);
        add_row_sum(s1, b1, p1, r1);
      },
      [&](RingFlipK) __attribute__((always_inline)) { flip(ko); },
      [&](RingFlipV) __attribute__((always_inline)) {
        flip(vo[0]);
        flip(vo[1]);
      });
  long_ring(n, computes, ops);
  if (computes) values(p1, b1);

  // Each wave keeps one of its query blocks (block kh: rows 32 wave .. + 31 of the unit), takes
  // the other key half's sums of it from the wave beside it, and hands over the other block.
  float l_tot, m_tot;
  f32x16 o0, o1;
  {
    const bool hi = kh != 0;
    f32x16 g0, g1;  // handed over
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      g0[r] = hi ? b0.o0[r] : b1.o0[r];
      g1[r] = hi ? b0.o1[r] : b1.o1[r];
      o0[r] = hi ? b1.o0[r] : b0.o0[r];
      o1[r] = hi ? b1.o1[r] : b0.o1[r];
    }
    const float mg = hi ? b0.m : b1.m, lg = half_sum(hi ? b0.l : b1.l);
    const float mk = hi ? b1.m : b0.m, lk = half_sum(hi ? b1.l : b0.l);
    static_assert(TILE * 2 == 8 * 64 * 16, "a wave's 32 accumulator entries fill one K slot");
    float* const xs = reinterpret_cast<float*>(lds + 4 * TILE);  // [wave][2][64 lanes]
    if (computes) {
      float4* po = reinterpret_cast<float4*>(lds + wave * TILE) + lane;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        po[j * 64] = make_float4(g0[4 * j], g0[4 * j + 1], g0[4 * j + 2], g0[4 * j + 3]);
        po[(4 + j) * 64] = make_float4(g1[4 * j], g1[4 * j + 1], g1[4 * j + 2], g1[4 * j + 3]);
      }
      xs[wave * 128 + lane] = mg;
      xs[wave * 128 + 64 + lane] = lg;
    }
    __syncthreads();
    if (computes) {
      const int w = wave ^ 1;
      const float mo = xs[w * 128 + lane], lo = xs[w * 128 + 64 + lane];
      m_tot = fmaxf(mk, mo);
      const float ak = __builtin_amdgcn_exp2f(mk - m_tot), ao = __builtin_amdgcn_exp2f(mo - m_tot);
      l_tot = lk * ak + lo * ao;
      const float4* po = reinterpret_cast<const float4*>(lds + w * TILE) + lane;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const float4 x = po[j * 64], y = po[(4 + j) * 64];
        const float xv[4] = {x.x, x.y, x.z, x.w}, yv[4] = {y.x, y.y, y.z, y.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          o0[4 * j + i] = fmaf(xv[i], ao, o0[4 * j + i] * ak);
          o1[4 * j + i] = fmaf(yv[i], ao, o1[4 * j + i] * ak);
        }
      }
    }
    __syncthreads();
  }
  // The output rows (normalised by the row sum, bf16) go out through LDS: each wave stages
  // its 32 rows, then writes whole 128-byte rows, as process_segment does.
  constexpr int kOutStageRow = D + 8;
  static_assert(32 * kOutStageRow <= TILE, "a wave's rows fit one V slot");
  uint16_t* const st = lds + (4 + wave) * TILE;
  if (wave_active) {
    const float inv = 1.f / l_tot;
    uint16_t* sp = st + l32 * kOutStageRow + 4 * half;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      *reinterpret_cast<uint2*>(sp + 8 * j) =
          to_bf16x4(o0[4 * j] * inv, o0[4 * j + 1] * inv, o0[4 * j + 2] * inv, o0[4 * j + 3] * inv);
      *reinterpret_cast<uint2*>(sp + 32 + 8 * j) =
          to_bf16x4(o1[4 * j] * inv, o1[4 * j + 1] * inv, o1[4 * j + 2] * inv, o1[4 * j + 3] * inv);
    }
  }
  __syncthreads();
  const int r8 = lane >> 3, c8 = (lane & 7) * 8;
  if (t0 == 0 && t1 == a.T) {
    // the whole unit in this chunk: final output rows and LSE
    if (wave_active) {
      if (half == 0 && qi < a.n_tokens) a.lse[(int64_t)h * a.n_tokens + qi] = (m_tot + __log2f(l_tot)) * kLn2;
#pragma unroll
      for (int pass = 0; pass < 4; ++pass) {
        const int r = pass * 8 + r8, qr = q0 + r;
        if (qr < a.n_tokens)
          *reinterpret_cast<uint4*>(a.out + ((int64_t)qr * a.n_heads + h) * D + c8) =
              *reinterpret_cast<const uint4*>(st + r * kOutStageRow + c8);
      }
    }
  } else {
    // partial result, merged by the second launch: the normalised output rows in bf16
    // (the merge weights them by 2^(m - M) l), then m and l in fp32
    const int seg = chunk_start(a, c) >= (int64_t)ui * a.U ? 0 : 1;
    float* ps = a.part + (int64_t)(2 * (a.chunk_base[q] + c) + seg) * kAttnSlotFloats;
    if (wave_active) {
      if (half == 0) {
        const int row = wave * 32 + l32;
        ps[kSlotStatsFloat + row] = m_tot;
        ps[kSlotStatsFloat + BQ + row] = l_tot;
      }
      uint16_t* po = reinterpret_cast<uint16_t*>(ps) + wave * 32 * D;
#pragma unroll
      for (int pass = 0; pass < 4; ++pass) {
        const int r = pass * 8 + r8;
        *reinterpret_cast<uint4*>(po + r * D + c8) = *reinterpret_cast<const uint4*>(st + r * kOutStageRow + c8);
      }
    }
  }
  __syncthreads();  // (the ring is the next segment's)
}

// Requests a field from every 64-byte line of the argument block at once: the reads that
// follow (some of them through indices that other arguments give) then hit the scalar
// cache, instead of each line's first read costing a round trip of its own.
// (The scalars before the tables lie in the lines of Q, lse and unit_base[0]; each table
// spans at most two lines, holding its first and last entries.)
static_assert(offsetof(AttnArgs, lse) / 64 == 1 && offsetof(AttnArgs, unit_base) / 64 == 2 &&
                  offsetof(AttnArgs, chunk_base) + 4 * kMaxQueues + 8 > sizeof(AttnArgs) && kMaxQueues <= 16,
              "touch_args names a field in every line of the argument block");
__device__ __forceinline__ void touch_args(const AttnArgs& a) {
  asm volatile("" ::"s"(a.Q), "s"(a.lse), "s"(a.unit_base[0]), "s"(a.unit_base[kMaxQueues]), "s"(a.n_chunks[0]),
               "s"(a.n_chunks[kMaxQueues - 1]), "s"(a.chunk_base[0]), "s"(a.chunk_base[kMaxQueues - 1]));
}

__global__ __launch_bounds__(kAttnThreads, kAttnWgPerCu) void attn_fwd_kernel(AttnArgs a) {
  __shared__ __attribute__((aligned(16))) uint16_t lds[NSTAGE * STAGE];
  // Workgroup b serves queue b % n_queues, chunk b / n_queues.  Queues are per XCD (the
  // hardware deals workgroup ids round-robin over the XCDs), which keeps the query
  // tiles of a head under one L2; placement only affects speed, never results.
  touch_args(a);
  const int q = (int)(blockIdx.x % (unsigned)a.n_queues);
  const int c = (int)(blockIdx.x / (unsigned)a.n_queues);
  if (c >= a.n_chunks[q]) return;
  const int ub = a.unit_base[q];
  int64_t first, end;
  chunk_iters(a, c, (int64_t)(a.unit_base[q + 1] - ub) * a.U, &first, &end);
  int it = (int)first;
  const int it_end = (int)end;
  while (it < it_end) {
    const int ui = it / a.U;
    const int t0 = it - ui * a.U;
    if (t0 >= a.T) {  // padding after the unit's last tile (split mode)
      it = (ui + 1) * a.U;
      continue;
    }
    const int seg_end = min(it_end, ui * a.U + a.T);
    process_segment(a, q, c, ub + ui, ui, t0, t0 + (seg_end - it), lds);
    it = (seg_end == ui * a.U + a.T) ? (ui + 1) * a.U : seg_end;
  }
}

__global__ __launch_bounds__(kAttnThreads, kAttnWgPerCu) void attn_long_kernel(AttnArgs a) {
  __shared__ __attribute__((aligned(16))) uint16_t lds[8 * TILE];
  touch_args(a);
  const int q = (int)(blockIdx.x % (unsigned)a.n_queues);
  const int c = (int)(blockIdx.x / (unsigned)a.n_queues);
  if (c >= a.n_chunks[q]) return;
  const int ub = a.unit_base[q];
  int64_t first, end;
  chunk_iters(a, c, (int64_t)(a.unit_base[q + 1] - ub) * a.U, &first, &end);
  int it = (int)first;
  const int it_end = (int)end;
  while (it < it_end) {
    const int ui = it / a.U;
    const int t0 = it - ui * a.U;
    if (t0 >= a.T) {  // padding after the unit's last tile (split mode)
      it = (ui + 1) * a.U;
      continue;
    }
    const int seg_end = min(it_end, ui * a.U + a.T);
    const int t1 = t0 + (seg_end - it);
    process_long_segment(a, q, c, ub + ui, ui, t0, t1, first_tile(a, c, it - (int)first, t0, t1), lds);
    it = (seg_end == ui * a.U + a.T) ? (ui + 1) * a.U : seg_end;
  }
}

// Second launch: for every unit whose key range was split over several chunks, four
// workgroups (32 rows each) merge the partial results (the kernel boundary makes them
// visible on every XCD).
__global__ __launch_bounds__(kAttnThreads) void attn_merge_kernel(AttnArgs a) {
  // Workgroup b merges for queue b % n_queues, like the forward workgroups that wrote
  // the partials (a locality heuristic: the partials may still be in that XCD's L2).
  touch_args(a);
  const int q = (int)(blockIdx.x % (unsigned)a.n_queues);
  const int j = (int)(blockIdx.x / (unsigned)a.n_queues);
  const int ui = j / (BQ / kMergeRows), rb = j % (BQ / kMergeRows);
  if (ui >= a.unit_base[q + 1] - a.unit_base[q]) return;
  const int unit = a.unit_base[q] + ui;
  const int c_first = chunk_holding(a, (int64_t)ui * a.U);
  const int c_last = chunk_holding(a, (int64_t)ui * a.U + a.T - 1);
  if (c_first == c_last) return;  // written whole by its only chunk
  merge_rows(a, q, unit, ui, rb, c_first, c_last);
}

// Merge launch with the saliency in its epilogue (Sec. 3.3: the saliency reuses the LSE,
// so it can only start once a query's LSE is final).  kEpiGroups workgroups per unit
// (head h, 128-query block qt); workgroup g
// * merges output rows 32 g .. 32 g + 31 of a split unit exactly as the merge launch does
//   (a unit whose key range one chunk covered was written by the forward launch);
// * forms the final LSE (log2 units) of all 128 rows -- from the partials' m and l with
//   merge_rows' arithmetic, or read back for a whole unit -- and lists the block's sampled
//   queries (the window rule of SalEpi) in row order, staging their rows in LDS;
// * sums, for the keys of its quarter of the frame's 32-key blocks, exp2(z log2(e) / 8 -
//   LSE log2(e)) over the sampled queries with v_mfma_f32_32x32x16_bf16 (Z = Q~ K^T, one
//   lane per key), in a fixed order -- in-lane over the accumulator rows, over 32-query
//   blocks, then across the lane halves -- into tiles[h][qt][j].
// What bounds it is latency: the merge's round trips (4.8 us alone), then each wave's chain of
// (key block, query block) steps.  So the key and query rows are requested ahead of the
// merge's partials and the wave's key blocks go through each query block two at a time (1041
// tokens, 16 heads, 5,000 rows remembered: 11.2 -> 9.3 us a launch; three at a time 10.0, and
// where a wave has four blocks, three and one took longer than before: 2000 tokens, 8 heads,
// 10.2 -> 10.8 and, by two, 9.6).  That takes more than 128 registers, so three workgroups fit a
// CU.  A launch that four to a CU would carry in fewer rounds keeps the form with fewer registers
// (attn_merge_sal_late_kernel: rows requested when they are needed, one block at a time): 2000
// tokens, 16 heads, 1,024 workgroups: 17.1 us, and 20.2 with the rows requested early.
constexpr int kEpiGroups = 4;
constexpr int kEpiQStride = kHeadDim + 8;   // staged query rows, 144 bytes
constexpr int kEpiEarlyPerCu = 3, kEpiLatePerCu = 4;   // workgroups that fit a CU

// Final LSE (log2 units) of row `row` of a split unit, with merge_rows' arithmetic.
__device__ float merged_lse2(const AttnArgs& a, int q, int ui, int row, int c_first, int c_last) {
  float mmax = kNegBig, L = 0.f;
  for (int c0 = c_first; c0 <= c_last; c0 += kMergeMax) {
    const int n = min(kMergeMax, c_last - c0 + 1);
    float mv[kMergeMax], lv[kMergeMax];
#pragma unroll
    for (int j = 0; j < kMergeMax; ++j) {
      const float* ps = slot_ptr(a, q, min(c0 + j, c_last), ui);
      mv[j] = ps[kSlotStatsFloat + row];
      lv[j] = ps[kSlotStatsFloat + BQ + row];
    }
    float m_new = mmax;
#pragma unroll
    for (int j = 0; j < kMergeMax; ++j) m_new = fmaxf(m_new, mv[j]);
    L *= __builtin_amdgcn_exp2f(mmax - m_new);
    mmax = m_new;
#pragma unroll
    for (int j = 0; j < kMergeMax; ++j) L += j < n ? __builtin_amdgcn_exp2f(mv[j] - mmax) * lv[j] : 0.f;
  }
  return mmax + __log2f(L);
}

template <bool kEarly>
__device__ __forceinline__ void merge_sal_body(const AttnArgs& a, const SalEpi& e) {
  __shared__ float s_lse2[BQ];                        // by row
  __shared__ float s_lsec[BQ];                        // by sampled position (padding: +inf)
  __shared__ int s_list[BQ];
  __shared__ int s_count[2];
  __shared__ __attribute__((aligned(16))) uint16_t s_q[BQ * kEpiQStride];
  touch_args(a);
  const int tid = threadIdx.x, lane = tid & 63, wave = uniform(tid >> 6);
  const int q = (int)(blockIdx.x % (unsigned)a.n_queues);
  const int jg = (int)(blockIdx.x / (unsigned)a.n_queues);
  const int ui = jg / kEpiGroups, g = jg % kEpiGroups;
  if (ui >= a.unit_base[q + 1] - a.unit_base[q]) return;  // uniform
  const int unit = a.unit_base[q] + ui;
  const int h = unit / a.q_tiles, qt = unit % a.q_tiles;
  const int N = a.n_tokens;
  const int c_first = chunk_holding(a, (int64_t)ui * a.U);
  const int c_last = chunk_holding(a, (int64_t)ui * a.U + a.T - 1);

  // ---- this group's output rows, and the LSE of all the block's rows ----
  auto merge = [&]() __attribute__((always_inline)) {
    if (c_first != c_last) merge_rows(a, q, unit, ui, g, c_first, c_last);
    if (tid < BQ) {
      const int qi = qt * BQ + tid;
      float l2 = 0.f;
      if (qi < N) l2 = c_first == c_last ? a.lse[(int64_t)h * N + qi] * kLog2e : merged_lse2(a, q, ui, tid, c_first, c_last);
      s_lse2[tid] = l2;
    }
  };
  if (!kEarly) merge();

  // ---- the block's sampled queries, in row order (waves 0 and 1 hold rows 0 .. 127) ----
  const int srow = wave * 64 + lane;
  bool sampled = false;
  int before = 0;
  if (wave < 2) {
    const int r = qt * BQ + srow - e.q_base;
    sampled = r >= 0 && r < e.grid_cells && (r / e.grid_w) % e.stride == 0 && (r % e.grid_w) % e.stride == 0;
    const uint64_t bal = __ballot(sampled);
    before = __builtin_popcountll(bal & ((1ull << lane) - 1ull));
    if (lane == 0) s_count[wave] = __builtin_popcountll(bal);
  }
  __syncthreads();
  if (sampled) s_list[(wave == 1 ? s_count[0] : 0) + before] = srow;
  __syncthreads();
  const int n_s = s_count[0] + s_count[1];
  const int ns_pad = (n_s + 31) & ~31;
  const int l32 = lane & 31, half = lane >> 5;
  const uint16_t* Kh = e.K + (int64_t)h * e.kv_head;
  float* tile_h = e.tiles + ((int64_t)h * a.q_tiles + qt) * N;
  const int n_blocks = (N + 31) / 32;
  const int per_group = (n_blocks + kEpiGroups - 1) / kEpiGroups;
  const int blk0 = g * per_group, blk1 = min(n_blocks, blk0 + per_group);

  constexpr int kWaves = kAttnThreads / 64;
  // ---- kEarly: everything the saliency reads, requested before the merge's partials: the key
  // rows of the wave's first blocks and the sampled query rows (clamped, valid addresses) ----
  constexpr int kKeyBatch = kEarly ? 2 : 4;  // 32-key blocks whose K rows a wave loads together
  bf16x8 kf[kKeyBatch][4];
  auto load_k = [&](int kb0) {
#pragma unroll
    for (int bb = 0; bb < kKeyBatch; ++bb) {
      const int j = min((kb0 + bb * kWaves) * 32 + l32, N - 1);  // past the range: result unused
      const uint16_t* kp = Kh + (int64_t)j * e.kv_row + half * 8;
#pragma unroll
      for (int ds = 0; ds < 4; ++ds) kf[bb][ds] = *reinterpret_cast<const bf16x8*>(kp + ds * 16);
    }
  };
  constexpr int kRowLoads = BQ * 8 / kAttnThreads;
  auto q_row = [&](int x) {  // 16-byte chunk x % 8 of the x / 8-th sampled query
    const int row = s_list[min(x >> 3, n_s - 1)];
    return *reinterpret_cast<const uint4*>(a.Q + ((int64_t)(qt * BQ + row) * a.n_heads + h) * D + (x & 7) * 8);
  };
  uint4 qv[kRowLoads];
  if (kEarly && n_s > 0) {
    load_k(blk0 + wave);
#pragma unroll
    for (int i = 0; i < kRowLoads; ++i) qv[i] = q_row(tid + i * kAttnThreads);
  }

  if (kEarly) merge();
  if (n_s == 0) {  // no sampled query in this block: its saliency row is the empty sum
    for (int j = blk0 * 32 + tid; j < min(N, blk1 * 32); j += kAttnThreads) tile_h[j] = 0.f;
    return;
  }
  // sampled query rows and their LSE (padding rows: zero rows, +inf -> weight 0)
  auto stage = [&](int x, const uint4& v) {
    *reinterpret_cast<uint4*>(&s_q[(x >> 3) * kEpiQStride + (x & 7) * 8]) = (x >> 3) < n_s ? v : uint4{0u, 0u, 0u, 0u};
  };
  if constexpr (kEarly) {
#pragma unroll
    for (int i = 0; i < kRowLoads; ++i)
      if (tid + i * kAttnThreads < ns_pad * 8) stage(tid + i * kAttnThreads, qv[i]);
  } else {
    for (int x = tid; x < ns_pad * 8; x += kAttnThreads) stage(x, q_row(x));
  }
  __syncthreads();
  for (int s = tid; s < ns_pad; s += kAttnThreads) s_lsec[s] = s < n_s ? s_lse2[s_list[s]] : __builtin_inff();
  __syncthreads();

  // ---- this group's key blocks, kKeyBatch per wave at a time; kEarly: the two go through each
  // sampled query block together, its rows and LSE read once for both, their MFMA and
  // exponential chains independent ----
  for (int kb0 = blk0 + wave; kb0 < blk1; kb0 += kKeyBatch * kWaves) {
    if (!kEarly || kb0 != blk0 + wave) load_k(kb0);
    auto sweep = [&](auto first_c, auto nb_c) {  // blocks first .. first + NB - 1 of the batch
      constexpr int F = decltype(first_c)::value, NB = decltype(nb_c)::value;
      float acc[NB] = {};
      for (int qb = 0; qb < ns_pad; qb += 32) {
        bf16x8 qf[4];
#pragma unroll
        for (int ds = 0; ds < 4; ++ds)
          qf[ds] = *reinterpret_cast<const bf16x8*>(&s_q[(qb + l32) * kEpiQStride + ds * 16 + half * 8]);
        // accumulator entry r: sampled query qb + 8 (r / 4) + 4 half + r % 4, key kb * 32 + l32
        float ls[16];
#pragma unroll
        for (int r = 0; r < 16; ++r) ls[r] = s_lsec[qb + 8 * (r >> 2) + 4 * half + (r & 3)];
        f32x16 z[NB] = {};
#pragma unroll
        for (int ds = 0; ds < 4; ++ds)
#pragma unroll
          for (int bb = 0; bb < NB; ++bb) z[bb] = mfma32(qf[ds], kf[F + bb][ds], z[bb]);
#pragma unroll
        for (int bb = 0; bb < NB; ++bb) {
          float s0 = 0.f, s1 = 0.f;
#pragma unroll
          for (int r = 0; r < 16; r += 2) {
            s0 += __builtin_amdgcn_exp2f(fmaf(z[bb][r], kScaleLog2, -ls[r]));
            s1 += __builtin_amdgcn_exp2f(fmaf(z[bb][r + 1], kScaleLog2, -ls[r + 1]));
          }
          acc[bb] += s0 + s1;
        }
      }
#pragma unroll
      for (int bb = 0; bb < NB; ++bb) {
        const float tot = acc[bb] + __shfl_xor(acc[bb], 32);
        const int j = (kb0 + (F + bb) * kWaves) * 32 + l32;
        if (half == 0 && j < N) tile_h[j] = tot;
      }
    };
    using std::integral_constant;
    if constexpr (kEarly) {
      if (kb0 + kWaves < blk1)  // uniform
        sweep(integral_constant<int, 0>{}, integral_constant<int, 2>{});
      else
        sweep(integral_constant<int, 0>{}, integral_constant<int, 1>{});
    } else {
      sweep(integral_constant<int, 0>{}, integral_constant<int, 1>{});
      if (kb0 + kWaves < blk1) sweep(integral_constant<int, 1>{}, integral_constant<int, 1>{});  // uniform
      if (kb0 + 2 * kWaves < blk1) sweep(integral_constant<int, 2>{}, integral_constant<int, 1>{});
      if (kb0 + 3 * kWaves < blk1) sweep(integral_constant<int, 3>{}, integral_constant<int, 1>{});
    }
  }
}

__global__ __launch_bounds__(kAttnThreads, kEpiEarlyPerCu) void attn_merge_sal_kernel(AttnArgs a, SalEpi e) {
  merge_sal_body<true>(a, e);
}
__global__ __launch_bounds__(kAttnThreads, kEpiLatePerCu) void attn_merge_sal_late_kernel(AttnArgs a, SalEpi e) {
  merge_sal_body<false>(a, e);
}

__global__ void xcc_probe_kernel(int* ids) {
  if (threadIdx.x == 0) ids[blockIdx.x] = hw_xcc_id();
}

// Split-KV partial slots of the allocation-free entry point: every GPU the library runs
// on holds one copy, from the library's load until the process ends.
static __device__ __align__(256) float scratch[(size_t)kStaticScratchSlots * kAttnSlotFloats];

}  // namespace

hipError_t static_scratch_address(float** ptr) {
  // host code may not use `scratch` itself as a device address: take the current
  // device's copy of the array through the runtime
  return hipGetSymbolAddress(reinterpret_cast<void**>(ptr), HIP_SYMBOL(scratch));
}

namespace {
hipError_t launch_forward(const AttnArgs& a, int grid, bool long_chunks, hipStream_t s) {
  hipLaunchKernelGGL(long_chunks ? attn_long_kernel : attn_fwd_kernel, dim3(grid), dim3(kAttnThreads), 0, s, a);
  return hipGetLastError();
}
}  // namespace

hipError_t launch_attention(const AttnArgs& a, int grid, bool merge, bool long_chunks, hipStream_t s) {
  hipError_t e = launch_forward(a, grid, long_chunks, s);
  if (e != hipSuccess || !merge) return e;
  int max_units = 0;
  for (int q = 0; q < a.n_queues; ++q) max_units = max(max_units, a.unit_base[q + 1] - a.unit_base[q]);
  hipLaunchKernelGGL(attn_merge_kernel, dim3(a.n_queues * max_units * (BQ / kMergeRows)), dim3(kAttnThreads), 0,
                     s, a);
  return hipGetLastError();
}

hipError_t launch_attention_saliency(const AttnArgs& a, const SalEpi& e, int grid, bool long_chunks, int n_cus,
                                     hipStream_t s) {
  hipError_t err = launch_forward(a, grid, long_chunks, s);
  if (err != hipSuccess) return err;
  int max_units = 0;
  for (int q = 0; q < a.n_queues; ++q) max_units = max(max_units, a.unit_base[q + 1] - a.unit_base[q]);
  // (rounds of an XCD's workgroups on its CUs)
  const int n_wg = max_units * kEpiGroups, cus = max(1, n_cus / a.n_queues);
  const bool late = (n_wg + kEpiLatePerCu * cus - 1) / (kEpiLatePerCu * cus) <
                    (n_wg + kEpiEarlyPerCu * cus - 1) / (kEpiEarlyPerCu * cus);
  hipLaunchKernelGGL(late ? attn_merge_sal_late_kernel : attn_merge_sal_kernel, dim3(a.n_queues * n_wg),
                     dim3(kAttnThreads), 0, s, a, e);
  return hipGetLastError();
}

hipError_t launch_xcc_probe(int* ids, int n_blocks, hipStream_t s) {
  hipLaunchKernelGGL(xcc_probe_kernel, dim3(n_blocks), dim3(64), 0, s, ids);
  return hipGetLastError();
}

}  // namespace rv
