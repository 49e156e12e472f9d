// admit.hip -- LSE-saliency, per-head top-k and memory append, gfx950.
//
// Two launches per call, each spread over the whole chip:
//
// sal_kernel (Sec. 3.3, saliency score and the A_ij equation): for key j of the frame,
//   S_j = sum over sampled queries i of exp(q_i . k_j / 8 - LSE_i),
// with the LSE the attention pass saved, so every term is an exact attention
// probability and no score matrix is stored.  A (layer, head) is split over
// `sal_groups` workgroups of 4 wave64s (about three per CU over the launch), each taking
// a contiguous range of 32-key blocks.  The sampled query rows and their LSE are staged
// in LDS once per workgroup; each wave then takes its blocks two at a time, or its only one (K
// rows in registers) and sweeps the sampled queries in blocks of 32 with
// v_mfma_f32_32x32x16_bf16 (Z = Q~ K^T, each lane owning one key column), each block's
// accumulator seeded with -8 LSE of its rows so that the MFMAs leave 8 (z - LSE).  The
// exponentials are summed in fp32 in a fixed order -- pairwise in-lane, over query
// blocks, then across the two lane halves -- so S is bit-reproducible with no atomics.
// The vector-ALU work is one multiply, one exp and one add per (query, key).
//
// select_kernel (Sec. 3.3 Eq. 6, head-specific retention): one workgroup per
// (layer, head) takes the `budget` largest S_j, equal values ordered by lower index.
// The order is that of the 64-bit key (bits of S, ~j): fp32 bit patterns order like
// the values for S >= 0.  Small budgets (takes_ranked): a lower bound of the budget-th largest
// value, from the threads' own maxima, leaves a few candidates, which are ranked by counting.
// Others, and frames whose largest values lie on so few threads that too many candidates are
// left: an MSB-first radix select over the bit patterns finds the threshold value and
// how many of its ties to take, and block scans emit the indices.  Either way the indices
// come out ascending and the chosen K/V rows are copied to the memory arena at rows
// mem_len.. with their provenance.
#include <type_traits>

#include "rv_internal.h"

namespace rv {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int D = kHeadDim;
constexpr int NT = kAdmitThreads;  // 256
constexpr int NW = NT / 64;
constexpr int kBlocksPerStep = 2;  // 32-key blocks a saliency wave holds at once (sal_one_kernel: 1)
static_assert(kBlocksPerStep == 2, "a range's last step holds one block or two");
constexpr int QS_STRIDE = kSalQStride;  // staged sampled-query rows, 144 bytes
constexpr int kPrefetchQBlock = 4;  // query block of a step at which the next step's K rows are requested
constexpr int kStageBatch = 9;     // 16-byte query-row loads in flight per thread (one pass of 288 rows)
constexpr float kLog2e = 1.44269504088896341f;
constexpr float kScaleLog2 = kLog2e * 0.125f;

static_assert(NT == 256, "the radix histogram has one bin per thread");

// ---- saliency -----------------------------------------------------------------------

// The two query-row sources are separate instantiations, so that neither path's
// memory waits are merged into the other's loop.
template <bool kStaged, int kStep>
__device__ __forceinline__ void sal_body(const AdmitArgs& a, unsigned char* smem) {
  const int H = a.n_heads, N = a.n_tokens, tid = threadIdx.x;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, half = lane >> 5;
  const int groups = a.sal_groups;
  // Workgroup b runs on XCD b % X (ids are dealt round-robin over the XCDs): group g of
  // (layer, head) lh = l_x X + x is id (g HX + l_x) X + x (HX = pairs per XCD), all of a
  // head's groups on XCD x, so the head's sampled query rows and LSE that every group
  // stages are read once from memory and then from that XCD's L2.  The first groups of
  // all heads come first, so a head's groups are dispatched in different rounds and the
  // later ones find the head's rows in L2.  Placement only affects speed.
  const int X = a.sal_xcds > 0 ? a.sal_xcds : 1;
  const int HX = (a.n_layers * H + X - 1) / X;
  const int xcd = blockIdx.x % X, rr = blockIdx.x / X;
  const int g = rr / HX, lh = (rr - g * HX) * X + xcd;
  if (g >= groups || lh >= a.n_layers * H) return;  // uniform: ids past the last (layer, head)
  // (uniform: the layer's operand addresses then live in scalar registers)
  const int layer = __builtin_amdgcn_readfirstlane(lh / H), h = __builtin_amdgcn_readfirstlane(lh - layer * H);
  const int n_blocks = (N + 31) / 32;
  int blk0, blk1;
  sal_group_blocks(a, g, n_blocks, &blk0, &blk1);
  if (blk0 >= blk1) return;  // uniform over the workgroup
  // The layer's operands, read once: this head's frame keys, query rows, LSE and
  // saliency row.
  const AdmitLayer& L = a.layer[layer];
  const int64_t kv_row = L.kv_row;
  const uint16_t* Kh = L.K + (int64_t)h * L.kv_head;
  const uint16_t* Qh = L.Q + (int64_t)h * D;
  const float* lse_h = L.lse + (int64_t)h * N;
  float* sal_h = L.sal + (int64_t)h * N;
  const int nq_pad = (a.n_q + 31) & ~31;
  if (nq_pad == 0) {  // no sampled queries: every key's saliency is the empty sum
    for (int j = blk0 * 32 + tid; j < min(N, blk1 * 32); j += NT) sal_h[j] = 0.f;
    return;
  }
  float* s_nlse8 = reinterpret_cast<float*>(smem);
  uint16_t* s_q = reinterpret_cast<uint16_t*>(smem + (size_t)nq_pad * 4);

  // -8 LSE of the sampled queries (the initial value of the score accumulators, so that
  // an accumulator ends as q.k - 8 LSE = 8 (z - LSE); padding rows: -inf -> weight 0)
  // and, when they fit, the sampled query rows (padding rows zero), a pass of q_pass
  // rows at a time.  Every load reads a clamped, valid address and padding is selected
  // afterwards, so no load sits behind a branch with a wait of its own: the LSE loads go
  // out together, then each batch of kStageBatch row loads per thread, and the K rows of
  // the wave's first step are requested after the staged data, so that the staging
  // does not wait for them.
  auto q_token = [&](int i) {
    const int qi = i / a.q_cols;
    return a.q_base + qi * a.q_row_stride + (i - qi * a.q_cols) * a.q_col_stride;
  };
  // K rows (B operands, K^T) of a step's blocks: lane's key, dims ds*16 + half*8 ..;
  // a pass's first step's rows are requested after its staging, each next step's rows
  // while the current step computes.
  auto load_k = [&](int bb, bf16x8 (&kf)[kStep][4]) {
#pragma unroll
    for (int b = 0; b < kStep; ++b) {
      const int j = min((bb + b) * 32 + l32, N - 1);  // past the frame or the range: result unused
      const uint16_t* kp = Kh + (int64_t)j * kv_row + half * 8;
#pragma unroll
      for (int ds = 0; ds < 4; ++ds) kf[b][ds] = *reinterpret_cast<const bf16x8*>(kp + ds * 16);
    }
  };
  auto lse_load = [&](int i0, float (&v)[4]) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int i = i0 + u * NT + tid;
      const float x = lse_h[q_token(min(i, a.n_q - 1))];
      v[u] = i < a.n_q ? x : __builtin_inff();
    }
  };
  auto lse_store = [&](int i0, const float (&v)[4]) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int i = i0 + u * NT + tid;
      if (i < nq_pad) s_nlse8[i] = -8.0f * v[u];
    }
  };
  // 16-byte chunk c (row p0 + c/8) of a pass's query rows
  auto rows_load = [&](int p0, int c0, uint4 (&v)[kStageBatch]) {
#pragma unroll
    for (int u = 0; u < kStageBatch; ++u) {
      const int c = c0 + u * NT + tid, i = p0 + (c >> 3), ch = c & 7;
      const uint4 x = *reinterpret_cast<const uint4*>(Qh + (int64_t)q_token(min(i, a.n_q - 1)) * H * D + ch * 8);
      v[u] = i < a.n_q ? x : uint4{0u, 0u, 0u, 0u};
    }
  };
  auto rows_store = [&](int rows, int c0, const uint4 (&v)[kStageBatch]) {
#pragma unroll
    for (int u = 0; u < kStageBatch; ++u) {
      const int c = c0 + u * NT + tid, ch = c & 7;
      if (c < rows * 8) *reinterpret_cast<uint4*>(&s_q[(c >> 3) * QS_STRIDE + ch * 8]) = v[u];
    }
  };
  bf16x8 kf[kStep][4], kn[kStep][4];
  // With one block a step the first LSE values are stored once the first batch of rows is in
  // flight too (one round trip less; with two there are no registers for it).
  constexpr bool kLateLse = kStaged && kStep == 1;
  float lse0[4];
  if (kLateLse) lse_load(0, lse0);
  for (int i0 = kLateLse ? NT * 4 : 0; i0 < nq_pad; i0 += NT * 4) {
    float lv[4];
    lse_load(i0, lv);
    lse_store(i0, lv);
  }

  // Passes over the sampled queries; each key's sum is carried from pass to pass by the
  // lane that owns it (fixed order).
  const int q_pass = kStaged ? a.q_pass : nq_pad;
  for (int p0 = 0; p0 < nq_pad; p0 += q_pass) {
    const int p1 = min(nq_pad, p0 + q_pass), rows = p1 - p0;
    if (kStaged) {
      for (int c0 = 0; c0 < rows * 8; c0 += NT * kStageBatch) {
        uint4 qv[kStageBatch];
        rows_load(p0, c0, qv);
        if (kLateLse && p0 + c0 == 0) lse_store(0, lse0);
        rows_store(rows, c0, qv);
      }
    }
    load_k(blk0 + wave * kStep, kf);  // (a wave without blocks loads rows it never uses)
    __syncthreads();

    for (int bb = blk0 + wave * kStep; bb < blk1; bb += NW * kStep) {
      // The next step's K rows are requested a few query blocks into this step, not at
      // its start: every workgroup of the launch stages at once, and the workgroups
      // served first would otherwise queue their next step's rows ahead of the staging
      // loads of those served last.
      const bool prefetch = bb + NW * kStep < blk1;
      const int q_prefetch = p0 + 32 * min(kPrefetchQBlock, (p1 - p0) / 32 - 1);
      // NB blocks held (the range's last step may hold fewer than kStep).
      auto sweep = [&](auto nb_c) {
        constexpr int NB = decltype(nb_c)::value;
        float acc[NB] = {};
        // A operand (query rows qb + l32) of a query block, from LDS or memory.
        auto load_q = [&](int qb, bf16x8 (&qf)[4]) {
          if (kStaged) {
#pragma unroll
            for (int ds = 0; ds < 4; ++ds)
              qf[ds] = *reinterpret_cast<const bf16x8*>(&s_q[(qb - p0 + l32) * QS_STRIDE + ds * 16 + half * 8]);
          } else {
            const uint16_t* qp = Qh + (int64_t)q_token(min(qb + l32, a.n_q - 1)) * H * D + half * 8;
#pragma unroll
            for (int ds = 0; ds < 4; ++ds) qf[ds] = *reinterpret_cast<const bf16x8*>(qp + ds * 16);
          }
        };
        bf16x8 qf[4];
        load_q(p0, qf);
        for (int qb = p0; qb < p1; qb += 32) {
          if (prefetch && qb == q_prefetch) load_k(bb + NW * kStep, kn);
          // Wave priority 0 for the MFMAs, 1 from the next block's row reads through the
          // exponentials: of the waves sharing a SIMD, those in their vector work issue
          // first, so the MFMAs of the others run under it (about -2 % per launch against a
          // uniform priority; priority changes no result).
          __builtin_amdgcn_s_setprio(0);
          // Each block's accumulator starts at -8 LSE of its 16 rows (queries
          // qb + 8*(r/4) + 4*half + r%4), so the MFMAs leave 8 (z - LSE) in it and the
          // two blocks' chains are independent.
          f32x16 z[NB];
#pragma unroll
          for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int r4 = 0; r4 < 4; ++r4) {
              const float4 v = *reinterpret_cast<const float4*>(&s_nlse8[qb + 8 * r4 + 4 * half]);
              z[b][4 * r4] = v.x;
              z[b][4 * r4 + 1] = v.y;
              z[b][4 * r4 + 2] = v.z;
              z[b][4 * r4 + 3] = v.w;
            }
#pragma unroll
          for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int ds = 0; ds < 4; ++ds) z[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(qf[ds], kf[b][ds], z[b], 0, 0, 0);
          __builtin_amdgcn_s_setprio(1);
          if (qb + 32 < p1) load_q(qb + 32, qf);  // the next block's rows, under this block's exponentials
#pragma unroll
          for (int b = 0; b < NB; ++b) {
            // exp(z - LSE) = 2^(8 (z - LSE) log2(e) / 8), all 16 independent, then a fixed
            // pairwise sum.
            float e[16];
#pragma unroll
            for (int r = 0; r < 16; ++r) e[r] = __builtin_amdgcn_exp2f(z[b][r] * kScaleLog2);
#pragma unroll
            for (int w = 8; w >= 1; w >>= 1)
#pragma unroll
              for (int r = 0; r < w; ++r) e[r] = e[r] + e[r + w];
            acc[b] += e[0];
          }
        }
        __builtin_amdgcn_s_setprio(0);
#pragma unroll
        for (int b = 0; b < NB; ++b) {
          const float tot = acc[b] + __shfl_xor(acc[b], 32);
          const int j = (bb + b) * 32 + l32;
          if (half == 0 && j < N) {
            if (p0 == 0)  // uniform
              sal_h[j] = tot;
            else
              sal_h[j] += tot;
          }
        }
      };
      if (bb + kStep <= blk1)  // uniform
        sweep(std::integral_constant<int, kStep>{});
      else if (kStep > 1)
        sweep(std::integral_constant<int, 1>{});
#pragma unroll
      for (int b = 0; b < kStep; ++b)
#pragma unroll
        for (int ds = 0; ds < 4; ++ds) kf[b][ds] = kn[b][ds];
    }
    if (p1 < nq_pad) __syncthreads();  // the staged rows are replaced by the next pass
  }
}

// Blocks a wave takes at a time: two, or one (sal_one_kernel) where no range holds more than a
// block a wave (launches of few layers: the wave's chain of query blocks is what the launch waits for,
// and half as long with one).  Saliency alone, two -> one: one layer of 1041 tokens, 16 heads
// 10.4 -> 8.0 us, 4 layers 12.6 -> 11.6; with every patch sampled one layer 29.0 -> 21.4, 4 layers
// 34.6 -> 30.9.  (One instantiation for both made the launch of 24 layers 0.9 % longer.)
__global__ __launch_bounds__(NT, 3) void sal_kernel(AdmitArgs a) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  if (a.stage_queries)
    sal_body<true, kBlocksPerStep>(a, smem);
  else
    sal_body<false, kBlocksPerStep>(a, smem);
}

__global__ __launch_bounds__(NT, 3) void sal_one_kernel(AdmitArgs a) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  if (a.stage_queries)
    sal_body<true, 1>(a, smem);
  else
    sal_body<false, 1>(a, smem);
}

// ---- selection and append -----------------------------------------------------------

// Exclusive prefix sum over the workgroup's threads (every thread must call it).
__device__ int block_exclusive_scan(int v, int* s_wave) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int x = v;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const int u = __shfl_up(x, off);
    if (lane >= off) x += u;
  }
  if (lane == 63) s_wave[wave] = x;
  __syncthreads();
  int base = 0;
#pragma unroll
  for (int w = 0; w < NW; ++w) base += w < wave ? s_wave[w] : 0;
  __syncthreads();
  return base + x - v;
}

// Top-`budget` of sal[0..N) (ties -> lower index), ascending, into s_idx[0..budget).
__device__ void select_topk(const float* sal, int N, int budget, int32_t* s_idx) {
  __shared__ unsigned int hist[256];
  __shared__ int s_wave[NW];
  __shared__ int s_bin, s_need;
  const int tid = threadIdx.x, lane = tid & 63;

  if (budget >= N) {
    for (int j = tid; j < N; j += NT) s_idx[j] = j;
    __syncthreads();
    return;
  }
  // Radix select, 8 bits per pass from the top: candidates share the prefix found so
  // far; the bin whose upper-tail count first reaches `need` holds the threshold.
  unsigned int prefix = 0u, mask = 0u;
  int need = budget;
  for (int shift = 24; shift >= 0; shift -= 8) {
    hist[tid] = 0u;  // NT == 256 bins
    __syncthreads();
    for (int j = tid; j < N; j += NT) {
      const unsigned int kj = __float_as_uint(sal[j]);
      if ((kj & mask) == prefix) atomicAdd(&hist[(kj >> shift) & 255u], 1u);
    }
    __syncthreads();
    if (tid < 64) {
      // lane i holds bins 255-4i .. 252-4i (descending); suffix counts by a wave scan
      unsigned int c[4];
#pragma unroll
      for (int m = 0; m < 4; ++m) c[m] = hist[255 - 4 * lane - m];
      const unsigned int tot = c[0] + c[1] + c[2] + c[3];
      unsigned int x = tot;
#pragma unroll
      for (int off = 1; off < 64; off <<= 1) {
        const unsigned int u = __shfl_up(x, off);
        if (lane >= off) x += u;
      }
      unsigned int ge = x - tot;  // elements in bins above this lane's first bin
#pragma unroll
      for (int m = 0; m < 4; ++m) {
        const unsigned int gt = ge;
        ge += c[m];
        if (gt < (unsigned int)need && (unsigned int)need <= ge) {
          s_bin = 255 - 4 * lane - m;
          s_need = need - (int)gt;
        }
      }
    }
    __syncthreads();
    prefix |= (unsigned int)s_bin << shift;
    mask |= 255u << shift;
    need = s_need;
  }
  const unsigned int tau = prefix;  // the budget-th largest value; take `need` of its ties

  // Each thread owns a contiguous run of indices; two scans give the tie ranks and the
  // output positions in index order.
  const int E = (N + NT - 1) / NT;
  const int j0 = min(N, tid * E), j1 = min(N, j0 + E);
  int n_gt = 0, n_eq = 0;
  for (int j = j0; j < j1; ++j) {
    const unsigned int kj = __float_as_uint(sal[j]);
    n_gt += kj > tau;
    n_eq += kj == tau;
  }
  const int eq_before = block_exclusive_scan(n_eq, s_wave);
  const int take_eq = max(0, min(n_eq, need - eq_before));
  const int n_sel = n_gt + take_eq;
  int pos = block_exclusive_scan(n_sel, s_wave);
  int eq_seen = eq_before;
  for (int j = j0; j < j1; ++j) {
    const unsigned int kj = __float_as_uint(sal[j]);
    bool sel = kj > tau;
    if (kj == tau) {
      sel = eq_seen < need;
      ++eq_seen;
    }
    if (sel && pos < budget) s_idx[pos++] = j;
  }
  __syncthreads();
}

// Order key of token j: saliency bits above, ~j below, so larger keys are larger
// saliencies and, among equal ones, lower indices.  0 marks "no candidate".
__device__ __forceinline__ uint64_t rank_key(float v, int j) {
  return ((uint64_t)__float_as_uint(v) << 32) | (uint32_t)~(uint32_t)j;
}

template <int CTRL>
__device__ __forceinline__ uint32_t dpp(uint32_t x) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, 0xF, 0xF, false);
}

// x of lane l ^ 16, and of lane l ^ 32: a v_permlane*_swap of x with itself leaves the two
// lanes' values in some order on every lane.
__device__ __forceinline__ uint32_t from_xor16(uint32_t x) {
  const auto r = __builtin_amdgcn_permlane16_swap(x, x, false, false);
  return (uint32_t)r[0] ^ (uint32_t)r[1] ^ x;
}
__device__ __forceinline__ uint32_t from_xor32(uint32_t x) {
  const auto r = __builtin_amdgcn_permlane32_swap(x, x, false, false);
  return (uint32_t)r[0] ^ (uint32_t)r[1] ^ x;
}

// x of lane l ^ MASK.
template <int MASK>
__device__ __forceinline__ uint32_t from_lane_xor(uint32_t x) {
  if constexpr ((MASK & 32) != 0) x = from_xor32(x);
  if constexpr ((MASK & 16) != 0) x = from_xor16(x);
  constexpr int m = MASK & 15;
  if constexpr (m == 1) return dpp<0xB1>(x);          // quad_perm [1,0,3,2]
  if constexpr (m == 2) return dpp<0x4E>(x);          // quad_perm [2,3,0,1]
  if constexpr (m == 3) return dpp<0x1B>(x);          // quad_perm [3,2,1,0]
  if constexpr (m == 4) return dpp<0x1B>(dpp<0x141>(x));  // row_half_mirror (l ^ 7), then l ^ 3
  if constexpr (m == 7) return dpp<0x141>(x);
  if constexpr (m == 8) return dpp<0x128>(x);         // row_ror:8
  if constexpr (m == 15) return dpp<0x140>(x);        // row_mirror
  static_assert(m == 0 || m == 1 || m == 2 || m == 3 || m == 4 || m == 7 || m == 8 || m == 15, "lane mask");
  return x;
}

// One compare-exchange of a descending sort: of lanes l and l ^ MASK, the one whose bit BIT is
// clear keeps the larger value.
template <int MASK, int BIT>
__device__ __forceinline__ uint32_t exchange(uint32_t x, int lane) {
  const uint32_t y = from_lane_xor<MASK>(x);
  return (lane & BIT) ? min(x, y) : max(x, y);
}

// The wave's 64 values sorted, largest on lane 0 (bitonic; the first step of each merge pairs
// mirrored lanes, so that every run descends).
__device__ __forceinline__ uint32_t wave_sort(uint32_t x, int lane) {
  x = exchange<1, 1>(x, lane);
  x = exchange<3, 2>(x, lane);
  x = exchange<1, 1>(x, lane);
  x = exchange<7, 4>(x, lane);
  x = exchange<2, 2>(x, lane);
  x = exchange<1, 1>(x, lane);
  x = exchange<15, 8>(x, lane);
  x = exchange<4, 4>(x, lane);
  x = exchange<2, 2>(x, lane);
  x = exchange<1, 1>(x, lane);
  x = exchange<31, 16>(x, lane);
  x = exchange<8, 8>(x, lane);
  x = exchange<4, 4>(x, lane);
  x = exchange<2, 2>(x, lane);
  x = exchange<1, 1>(x, lane);
  x = exchange<63, 32>(x, lane);
  x = exchange<16, 16>(x, lane);
  x = exchange<8, 8>(x, lane);
  x = exchange<4, 4>(x, lane);
  x = exchange<2, 2>(x, lane);
  return exchange<1, 1>(x, lane);
}

// Whether the selection ranks its candidates (select_ranked) or takes the radix way.  The lines:
// kLaneSlots values in registers, and a budget up to which the counts take less than the radix
// way (selection alone, 256 heads, budgets 64 / 96 / 128: 257 tokens 8.7 / 10.6 / 13.5 us ranked,
// 8.6 / 9.4 / 10.4 radix; 1041 tokens 9.1 / 11.3 / 13.8 and 10.6 / 11.0 / 12.0; 2048 tokens 9.1 /
// 11.5 / 13.6 and 11.8 / 12.8 / 13.9); of few tokens, no more than half, which is the room for
// candidates.
constexpr int kLaneSlots = 8;
constexpr int kRankedTokens = NT * kLaneSlots;
constexpr int kRankedBudget = 128;
__device__ __forceinline__ bool takes_ranked(int N, int budget) {
  return N <= kRankedTokens && 2 * budget <= N && budget <= 40 + N / 24;
}
static_assert(40 + kRankedTokens / 24 <= kRankedBudget && kRankedBudget <= NT, "one thread a winner");

// Candidates that are ranked, at most: one a thread.  (More would take a second round of counts:
// 256 candidates at budget 10 take 11 us, 320 take 16, as long as the radix way after the attempt.)
constexpr int kMaxCandidates = NT;
// Candidates past twice the budget from which the equal ones among them are looked at, and equal
// ones past those needed from which they are cut.  (The cut takes about 2.5 us, as long as counting
// over 100 more candidates.  All tokens equal, 1041 tokens: 8.6 us at budget 1, 9.2 at 10; without
// the cut, through the radix way, 15.5 and 15.2.)
constexpr int kManyMore = 64;

// Top-`budget` (takes_ranked), ascending, into s_idx; v[m] is the value of token tid + NT m.  The
// budget-th largest of the 256 threads' maxima is no larger than the budget-th largest value, so
// the tokens at or above it hold the selection: budget threads' tokens at most, and those equal
// to the bound.  Where the latter are many, the tokens above the bound are counted exactly and
// only the first equal ones that the budget still needs are candidates.  The candidates are
// gathered into s_cand (in any order: the keys are distinct), each one's rank is the number of
// larger keys, and the place of a winner is the number of winners with a lower index.  False, on
// every thread, if there are more than `cap` candidates.
// What bounds it is the chain of dependent steps, one wave per SIMD.  (Before: `budget`
// rounds of wave-wide maxima in each wave and again over their winners, or, above 32, the
// radix select.  The selection launch for 24 layers of 1041 tokens: 8.8 -> 5.2 us at budget
// 10, 12.6 -> 6.1 at 20, 13.0 -> 8.4 at 52; one layer 7.4 -> 5.2; an empty launch takes 2.4.
// Reading eight keys a step in the counts was slower by a tenth.)
__device__ __forceinline__ bool select_ranked(const float (&v)[kLaneSlots], int N, int budget, int32_t* s_idx,
                                              uint64_t* s_cand, int cap) {
  __shared__ uint64_t s_equal[kLaneSlots * NW];  // tokens equal to the bound, a bit each, in order
  __shared__ uint32_t s_sorted[NT];
  __shared__ int32_t s_win[kRankedBudget];
  __shared__ uint32_t s_bound;
  __shared__ int s_count[3];  // tokens at or above the bound; above it; candidates
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  uint32_t best = 0u;  // (threads without tokens rank last: budget < N)
#pragma unroll
  for (int m = 0; m < kLaneSlots; ++m)
    if (tid + NT * m < N) best = max(best, __float_as_uint(v[m]));
  const uint32_t x = wave_sort(best, lane);
  s_sorted[tid] = x;
  if (tid < 3) s_count[tid] = 0;
  __syncthreads();
  // Rank of x among all 256, equal values in the order of waves then lanes.
  int rank = lane;
#pragma unroll
  for (int o = 1; o < NW; ++o) {
    const int w = (wave + o) & (NW - 1);
    // first position of wave w's descending list whose value is below x (w earlier: equal
    // values come before), or not above x (w later)
    const uint32_t limit = x - (w < wave ? 1u : 0u);  // values > limit come before; x = 0 wraps: none are below 0
    int lo = 0;
#pragma unroll
    for (int step = 32; step > 0; step >>= 1)
      if (s_sorted[w * 64 + lo + step - 1] > limit || (w < wave && x == 0u)) lo += step;
    if (s_sorted[w * 64 + lo] > limit || (w < wave && x == 0u)) ++lo;
    rank += lo;
  }
  if (rank == budget - 1) s_bound = x;
  __syncthreads();
  const uint32_t bound = s_bound;
  uint32_t in = 0u;  // the thread's tokens at or above the bound, a bit each
#pragma unroll
  for (int m = 0; m < kLaneSlots; ++m)
    in |= (uint32_t)(tid + NT * m < N && __float_as_uint(v[m]) >= bound) << m;
  auto gather = [&](int* count) {
    if (in == 0u) return;
    int at = atomicAdd(count, __popc(in));
#pragma unroll
    for (int m = 0; m < kLaneSlots; ++m)
      if (in >> m & 1u) {
        if (at < cap) s_cand[at] = rank_key(v[m], tid + NT * m);
        ++at;
      }
  };
  gather(&s_count[0]);
  __syncthreads();
  int nc = s_count[0];
  if (nc > 2 * budget + kManyMore) {  // uniform
    int n_above = 0;
#pragma unroll
    for (int m = 0; m < kLaneSlots; ++m) {
      const bool eq = (in >> m & 1u) && __float_as_uint(v[m]) == bound;
      const uint64_t word = __ballot(eq);
      n_above += __popcll(__ballot(in >> m & 1u)) - __popcll(word);
      if (lane == 0) s_equal[m * NW + wave] = word;  // tokens NT m + 64 wave ..
    }
    if (lane == 0 && n_above) atomicAdd(&s_count[1], n_above);
    __syncthreads();
    const int above = s_count[1], need = max(0, budget - above);
    if (nc - above > need + kManyMore) {  // uniform
      // Equal tokens before word l, on lane l.
      const int own = lane < kLaneSlots * NW ? __popcll(s_equal[lane]) : 0;
      int before = own;
#pragma unroll
      for (int off = 1; off < kLaneSlots * NW; off <<= 1) {
        const int u = __shfl_up(before, off);
        if (lane >= off) before += u;
      }
      before -= own;
#pragma unroll
      for (int m = 0; m < kLaneSlots; ++m) {
        const int first = __shfl(before, m * NW + wave);
        const uint64_t word = s_equal[m * NW + wave];
        if ((word >> lane & 1u) && first + __popcll(word & ((1ull << lane) - 1)) >= need) in &= ~(1u << m);
      }
      gather(&s_count[2]);
      __syncthreads();
      nc = s_count[2];
    }
  }
  if (nc > cap) {  // uniform
    __syncthreads();  // (s_cand is the caller's again)
    return false;
  }
  for (int i = tid; i < nc; i += NT) {
    const uint64_t key = s_cand[i];
    int r = 0;
    for (int u = 0; u < nc; ++u) r += s_cand[u] > key;
    if (r < budget) s_win[r] = (int32_t)~(uint32_t)key;
  }
  __syncthreads();
  if (tid < budget) {
    const int32_t j = s_win[tid];
    int pos = 0;
    for (int u = 0; u < budget; ++u) pos += s_win[u] < j;
    s_idx[pos] = j;
  }
  __syncthreads();
  return true;
}

// Head-specific retention (the paper's rule, Sec. 3.3): one workgroup per (layer, head)
// ranks that head's saliency.  Shared selection (the arm without head-specific
// retention in the ablation of Sec. 4.5, Table 4): every head's workgroup ranks the sum
// over heads of the saliencies (summed in head order, so every workgroup of a layer
// reaches the same selection; it orders tokens as the mean does) and appends those
// tokens to its own head.
__global__ __launch_bounds__(NT) void select_kernel(AdmitArgs a) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int H = a.n_heads, N = a.n_tokens, k = a.budget, tid = threadIdx.x;
  const int layer = blockIdx.x / H, h_own = blockIdx.x - layer * H;
  const AdmitLayer& L = a.layer[layer];
  float* s_sal = reinterpret_cast<float*>(smem);
  int32_t* s_idx = reinterpret_cast<int32_t*>(smem + (((size_t)N * 4 + 15) & ~(size_t)15));

  // The saliency that is ranked: the sum, in order, of n_rows rows of N values -- the head's
  // row; its per-block rows (computed in the attention epilogue: the sum is the saliency,
  // written out when asked for); or all heads' rows.  Tokens j0 + NT m, with kLaneSlots *
  // kRowBatch loads in flight (token by token, eight rows at a time, the nine per-block rows of
  // 1041 tokens took the launch of 7 layers 10.8 us instead of 6.9).
  const int n_rows = a.shared_select ? H : a.sal_tiles > 0 ? a.sal_tiles : 1;
  const float* const rows = a.shared_select ? L.sal : L.sal + (int64_t)h_own * n_rows * N;
  auto values = [&](int j0, float (&acc)[kLaneSlots]) {
    constexpr int M = kLaneSlots, kRowBatch = 4;
#pragma unroll
    for (int m = 0; m < M; ++m) acc[m] = 0.f;
    for (int r0 = 0; r0 < n_rows; r0 += kRowBatch) {
      float x[kRowBatch][M];
#pragma unroll
      for (int u = 0; u < kRowBatch; ++u)
        if (r0 + u < n_rows)  // uniform
#pragma unroll
          for (int m = 0; m < M; ++m) x[u][m] = rows[(int64_t)(r0 + u) * N + min(j0 + NT * m, N - 1)];
#pragma unroll
      for (int u = 0; u < kRowBatch; ++u)
        if (r0 + u < n_rows)
#pragma unroll
          for (int m = 0; m < M; ++m) acc[m] += x[u][m];
    }
    if (a.sal_tiles > 0 && L.sal_out)
#pragma unroll
      for (int m = 0; m < M; ++m)
        if (j0 + NT * m < N) L.sal_out[(int64_t)h_own * N + j0 + NT * m] = acc[m];
  };
  bool ranked = false;
  float v[kLaneSlots];
  const bool few = takes_ranked(N, k);  // uniform
  if (few) {
    values(tid, v);
    // (the candidates lie where the values would)
    ranked = select_ranked(v, N, k, s_idx, reinterpret_cast<uint64_t*>(s_sal), min(kMaxCandidates, N / 2));
  }
  if (!ranked) {  // uniform
    if (few) {
#pragma unroll
      for (int m = 0; m < kLaneSlots; ++m)
        if (tid + NT * m < N) s_sal[tid + NT * m] = v[m];
    } else if (a.shared_select || a.sal_tiles > 0) {
      for (int j0 = tid; j0 < N; j0 += NT * kLaneSlots) {
        values(j0, v);
#pragma unroll
        for (int m = 0; m < kLaneSlots; ++m)
          if (j0 + NT * m < N) s_sal[j0 + NT * m] = v[m];
      }
    } else if ((N & 3) == 0) {  // (+ 0: as the sums, -0 ranks as 0)
      for (int j = tid; j < N / 4; j += NT) {
        const float4 x = reinterpret_cast<const float4*>(rows)[j];
        reinterpret_cast<float4*>(s_sal)[j] = make_float4(x.x + 0.f, x.y + 0.f, x.z + 0.f, x.w + 0.f);
      }
    } else {
      for (int j = tid; j < N; j += NT) s_sal[j] = rows[j] + 0.f;
    }
    __syncthreads();
    select_topk(s_sal, N, k, s_idx);
  }
  {
    const int h = h_own;
    if (L.idx)
      for (int r = tid; r < k; r += NT) L.idx[(int64_t)h * k + r] = s_idx[r];
    // 16-byte chunks: 8 per K row, 8 per V row.
    if (!a.in_place) {
      for (int c = tid; c < k * 16; c += NT) {
        const int r = c >> 4, part = c & 15, chunk = part & 7;
        const int j = s_idx[r];
        if (j < 0 || j >= N) continue;  // unreachable: the selection emits exactly k indices < N
        const int64_t src = (int64_t)j * L.kv_row + (int64_t)h * L.kv_head + chunk * 8;
        const int64_t dst = ((int64_t)h * L.head_stride + L.mem_len + r) * D + chunk * 8;
        if (part < 8)
          *reinterpret_cast<uint4*>(L.memK + dst) = *reinterpret_cast<const uint4*>(L.K + src);
        else
          *reinterpret_cast<uint4*>(L.memV + dst) = *reinterpret_cast<const uint4*>(L.V + src);
      }
    } else {
      // Compaction inside the arena: the staged row idx[r] moves to row mem_len + r.
      // Indices ascend, so idx[r] >= r: passes of NT / 16 rows in ascending order read
      // all of a pass's sources before writing its destinations, and no later pass reads
      // a row an earlier one wrote (its sources lie at or past its own destinations).
      for (int r0 = 0; r0 < k; r0 += NT / 16) {
        const int r = r0 + (tid >> 4), part = tid & 15, chunk = part & 7;
        uint4 v = make_uint4(0, 0, 0, 0);
        int64_t dst = -1;
        if (r < k) {
          const int j = s_idx[r];
          if (j >= 0 && j < N) {  // always: the selection emits exactly k indices < N
            const int64_t src = (int64_t)j * L.kv_row + (int64_t)h * L.kv_head + chunk * 8;
            v = *reinterpret_cast<const uint4*>((part < 8 ? L.K : L.V) + src);
            dst = ((int64_t)h * L.head_stride + L.mem_len + r) * D + chunk * 8;
          }
        }
        __syncthreads();
        if (dst >= 0) *reinterpret_cast<uint4*>((part < 8 ? L.memK : L.memV) + dst) = v;
        __syncthreads();
      }
    }
    for (int r = tid; r < k; r += NT) {
      int32_t* pv = L.prov + ((int64_t)h * L.head_stride + L.mem_len + r) * 2;
      pv[0] = a.frame_id;
      pv[1] = s_idx[r];
    }
  }
}

hipError_t set_lds_limit(const void* kernel, int* cached, int limit) {
  if (*cached == limit) return hipSuccess;
  const hipError_t e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, limit);
  if (e == hipSuccess) *cached = limit;
  return e;
}

}  // namespace

hipError_t launch_admit(const AdmitArgs& a, int max_lds, hipStream_t s) {
  static int sal_attr = 0, sal_one_attr = 0, sel_attr = 0;
  const int limit = admit_max_dynamic_lds(max_lds);
  if (a.mode & kModeSaliency) {
    int b0, b1;
    sal_group_blocks(a, 0, (a.n_tokens + 31) / 32, &b0, &b1);  // (no later group holds more)
    const bool one = b1 - b0 <= NW;
    auto* const kernel = one ? sal_one_kernel : sal_kernel;
    hipError_t e = set_lds_limit((const void*)sal_kernel, &sal_attr, limit);
    if (e == hipSuccess) e = set_lds_limit((const void*)sal_one_kernel, &sal_one_attr, limit);
    if (e != hipSuccess) return e;
    const unsigned X = (unsigned)(a.sal_xcds > 0 ? a.sal_xcds : 1);
    const unsigned n_lh = (unsigned)(a.n_layers * a.n_heads);
    const unsigned grid = (n_lh + X - 1) / X * X * (unsigned)a.sal_groups;
    hipLaunchKernelGGL(kernel, dim3(grid), dim3(NT), sal_lds_bytes(a), s, a);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  if ((a.mode & kModeSelect) && a.budget > 0) {
    hipError_t e = set_lds_limit((const void*)select_kernel, &sel_attr, limit);
    if (e != hipSuccess) return e;
    const unsigned grid = (unsigned)(a.n_layers * a.n_heads);
    hipLaunchKernelGGL(select_kernel, dim3(grid), dim3(NT), select_lds_bytes(a), s, a);
    return hipGetLastError();
  }
  return hipSuccess;
}

namespace {

// One thread per 16-byte chunk of the frame (8 per row of 64 bf16), in the frame's order.
__global__ __launch_bounds__(256) void stage_kernel(uint16_t* dK, uint16_t* dV, int64_t head_stride,
                                                    const uint16_t* K, const uint16_t* V, int n, int H) {
  const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= (int64_t)n * H * 8) return;
  const int chunk = (int)(c & 7);
  const int64_t row = c >> 3;  // token * H + head
  const int h = (int)(row % H);
  const int64_t j = row / H;
  const int64_t d = ((int64_t)h * head_stride + j) * D + chunk * 8;
  *reinterpret_cast<uint4*>(dK + d) = reinterpret_cast<const uint4*>(K)[c];
  *reinterpret_cast<uint4*>(dV + d) = reinterpret_cast<const uint4*>(V)[c];
}

// Several layers' frames in one launch: blockIdx.y is the layer.
__global__ __launch_bounds__(256) void stage_layers_kernel(StageArgs a) {
  const StageLayer& L = a.layer[blockIdx.y];
  const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= (int64_t)a.n_tokens * a.n_heads * 8) return;
  const int chunk = (int)(c & 7);
  const int64_t row = c >> 3;  // token * H + head
  const int h = (int)(row % a.n_heads);
  const int64_t j = row / a.n_heads;
  const int64_t d = ((int64_t)h * L.head_stride + j) * D + chunk * 8;
  *reinterpret_cast<uint4*>(L.dK + d) = reinterpret_cast<const uint4*>(L.K)[c];
  *reinterpret_cast<uint4*>(L.dV + d) = reinterpret_cast<const uint4*>(L.V)[c];
}

}  // namespace

hipError_t launch_stage(uint16_t* dK, uint16_t* dV, int64_t head_stride, const uint16_t* K, const uint16_t* V,
                        int n, int H, hipStream_t s) {
  const int64_t chunks = (int64_t)n * H * 8;
  hipLaunchKernelGGL(stage_kernel, dim3((unsigned)((chunks + 255) / 256)), dim3(256), 0, s, dK, dV, head_stride,
                     K, V, n, H);
  return hipGetLastError();
}

hipError_t launch_stage_layers(const StageArgs& a, hipStream_t s) {
  const int64_t chunks = (int64_t)a.n_tokens * a.n_heads * 8;
  hipLaunchKernelGGL(stage_layers_kernel, dim3((unsigned)((chunks + 255) / 256), (unsigned)a.n_layers), dim3(256), 0,
                     s, a);
  return hipGetLastError();
}

}  // namespace rv
