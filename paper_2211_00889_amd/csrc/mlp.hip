// End-to-end workload for gfx950: per-mini-batch gradients of a two-layer MLP
// (d_in -> hidden, ReLU -> classes, softmax cross-entropy, mean over a
// 32-sample mini-batch) written into G[i][j] of the Non-blocking step, and the
// mean loss of a parameter vector on a sample list (evaluation).
//
// Every GEMM input is rounded to bf16 (round to nearest even, the hardware
// conversion) and multiplied with fp32 accumulation:
//   k_mlp_fwd    partial Z1 = A W1 over one slice of d_in, per 128-row x
//                128-unit tile, on MFMA 16x16x32 (both operands staged in LDS)
//   k_mlp_back   per mini-batch: Z1 = sum of the slices (in an order that does not
//                depend on their number) + b1, H =
//                bf16(relu(Z1)), logits = H W2 + b2 (MFMA, classes padded to
//                16), softmax-CE, the loss; and for gradients dZ2, dZ1 = (dZ2
//                W2^T) * [Z1 > 0], db1, dW2 = H^T dZ2, db2 and dW1 = A^T dZ1
//                (MFMA, K = batch = 32)
// MFMA 16x16x32 bf16 operand layout (lane l, t = 0..7): A[l % 16][8 (l / 16) + t],
// B[8 (l / 16) + t][l % 16]; result D[4 (l / 16) + t][l % 16], t = 0..3.
//
// Flat parameter layout of a replica: W1[d_in][hidden], b1[hidden],
// W2[hidden][classes], b2[classes], then zeros up to a multiple of 4 floats,
// so every replica row and every G row starts 16-byte aligned (rows are ld
// floats apart, ld >= P a multiple of 4; ld = P unless the caller pads them).
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>
#include <string.h>

#include <algorithm>
#include <mutex>
#include <vector>

#include "internal.h"
#include "mlp_plan.h"
#include "mlp_shape.h"

using namespace nbsgd;

namespace {

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x8 __attribute__((ext_vector_type(8)));

// kBatch, kMaxHidden, kMaxClasses, kFeatBlock, kSkMaxSlices and Dims: mlp_shape.h
constexpr int kMaxList = 896;    // mini-batches per launch group (kernel-argument list)
constexpr int kMaxEval = 512;    // batches of 32 per nbsgd_mlp_loss call

// One launch group's mini-batches, word e = learner << 24 | slot << 12,
// sorted by learner.  A slot indexes the caller's sample list (slot * 32 ..),
// the G rows and the loss output; the workspace rows of entry e are
// e * 32 .. e * 32 + 31.  Read as 32-bit words only.
struct List {
  int32_t count;
  uint32_t w[kMaxList];
};

// Sample indices of list entries first .. first + n_slots - 1, 32 per entry:
// two to a word (16 bits each) when `wide` is 0, one to a word otherwise.
constexpr int kUpSlots = 60;
struct IdxChunk {
  int32_t first, n_slots, wide;
  uint32_t v[kUpSlots * kBatch / 2];
};

// Sample indices of a whole launch group carried in the forward kernel's
// arguments (groups of at most kInline mini-batches whose indices all fit 16
// bits): row e * 32 + r in the 16-bit half r % 2 of word (e * 32 + r) / 2.
constexpr int kInline = 56;
template <int N>
struct Idx16 {
  uint32_t v[N];
};
using InlineIdx = Idx16<kInline * kBatch / 2>;

// kernel arguments are limited to 4 KiB: the list, the shapes and at most
// ten pointers or 64-bit scalars
static_assert(sizeof(List) + sizeof(Dims) + 10 * 8 <= 4096, "kernel arguments exceed 4 KiB");
static_assert(sizeof(IdxChunk) + 32 <= 4096, "kernel arguments exceed 4 KiB");
static_assert(kMaxList <= 4096 && kMaxEval <= 4096, "slots are packed in 16 bits");

__host__ __device__ __forceinline__ int item_learner(uint32_t w) { return (int)(w >> 24); }
__device__ __forceinline__ int item_slot(uint32_t w) { return (int)((w >> 12) & 0xfffu); }

// Two (eight) floats to bf16 as one vector conversion: one v_cvt_pk_bf16_f32 a
// pair.  Converted one by one and combined by hand they took seven instructions a
// pair, and the conversions, not the matrix cores or the loads, filled the VALUs of
// the forward (70% busy on 4,096 samples).
__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi) {
  return __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2){lo, hi}, bf16x2));
}
__device__ __forceinline__ bf16x8 to_bf16(f32x4 lo, f32x4 hi) {
  return __builtin_convertvector((f32x8){lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]},
                                 bf16x8);
}

// Orders the wave's LDS writes before its later LDS accesses (other lanes' data).
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Swizzle of row r of a 16-row tile of the forward's LDS: within rows 0-7 and
// within 8-15 all eight values differ (writes), and so they do within the even and
// the odd rows, in pairs 2 v, 2 v + 1 for rows 0-3 and 12-15 (reads).
__device__ __forceinline__ int fwd_swizzle(int r) {
  return ((r & 4) | (r & 1) << 1 | ((r >> 1) & 1)) ^ (r & 8 ? 6 : 0);
}

// W1 of the present learners in bf16, as the forward's LDS holds it: tile (learner
// k, unit block, chunk), chunks fastest, is the image [unit row][64 k] of 128 units.
constexpr int kFwUnits = 128, kFwTile = kFwUnits * kFwKc;
struct Pack {
  const float* X;
  __bf16* w1;
  int64_t ld;
  int32_t hidden, chunks, ub;
  int32_t idx_blocks;    // workgroups before the first tile's
  uint32_t learner[4];   // as SkMap's
};
static_assert(sizeof(IdxChunk) + sizeof(Pack) + 32 <= 4096, "kernel arguments exceed 4 KiB");

// Writes the sample index of every row of the chunk's list entries (used when a
// group's indices do not fit the forward kernel's arguments); workgroups from
// p.idx_blocks on write one tile of the packed W1 each, a thread 8 k x 4 units.
__global__ void __launch_bounds__(256) k_put_idx(int32_t* __restrict__ dst, IdxChunk c, Pack p) {
  if ((int)blockIdx.x >= p.idx_blocks) {  // uniform
    const int tile = blockIdx.x - p.idx_blocks;
    const int chunk = tile % p.chunks, ubk = tile / p.chunks % p.ub, li = tile / p.chunks / p.ub;
    const int learner = (int)((p.learner[li >> 2] >> (8 * (li & 3))) & 0xffu);
    const int wq = threadIdx.x & 31, o = threadIdx.x >> 5, H = p.hidden, u0 = kFwUnits * ubk;
    // unit quads past the block read its first units; nothing stores what they give
    const float* src = p.X + (int64_t)learner * p.ld + (int64_t)(kFwKc * chunk + 8 * o) * H + u0 +
                       (u0 + 4 * wq < H ? 4 * wq : 0);
    f32x4 v[8];
#pragma unroll
    for (int r = 0; r < 8; ++r) v[r] = *reinterpret_cast<const f32x4*>(src + (int64_t)r * H);
    __bf16* out = p.w1 + (int64_t)tile * kFwTile + (64 * (wq >> 4) + (wq & 15)) * kFwKc +
                  8 * (o ^ fwd_swizzle(wq & 15));
#pragma unroll
    for (int t = 0; t < 4; ++t)
      *reinterpret_cast<bf16x8*>(out + 16 * t * kFwKc) = to_bf16(
          (f32x4){v[0][t], v[1][t], v[2][t], v[3][t]}, (f32x4){v[4][t], v[5][t], v[6][t], v[7][t]});
    return;
  }
  const int t = blockIdx.x * 256 + threadIdx.x;
  if (t >= c.n_slots * kBatch) return;
  const int32_t v = c.wide ? (int32_t)c.v[t] : (int32_t)((c.v[t >> 1] >> (16 * (t & 1))) & 0xffffu);
  dst[c.first * kBatch + t] = v;
}

// Forward, split over d_in.  Work item: a quad (up to four mini-batches of one
// learner, 128 rows), a block of 128 hidden units and one of S slices of d_in (parts
// and their order: mlp_plan.h).  Eight waves: wave w takes all 128 units for
// mini-batch w % 4 over side w / 4 of the slice (2 x 8 accumulators, twice that where
// a side has two leaves), so that a W1 fragment read from LDS
// feeds two MFMAs and four waves share its staging.  Per chunk of 64 k:
//   W1  [side][unit][k] in bf16, staged by all waves for all (each thread
//       transposes a 4 k x 4 unit cell of either side), two buffers, one barrier
//       a chunk; loaded one chunk ahead of its staging
//   A   the wave's own 32 rows, loaded one chunk ahead with four lanes on 64
//       contiguous bytes of a row, converted into the wave's own LDS rows and read
//       back as fragments: no other wave needs them, so no barrier.  (Loading the
//       fragments straight from memory puts the 16 rows of a tile on consecutive
//       lanes, and the L1 then serves 16 bytes an access: 36.6 against 28.7 us.)
// Rows are 64 bf16 (128 bytes); octet o of a row is stored at o ^ swizzle(row),
// which leaves the 8-byte writes (16 lanes a cycle) and the 16-byte fragment reads
// free of bank conflicts; a 64-unit group's unit 4 q + t is LDS row 16 t + q, so
// that lane q of a result holds four consecutive units.  The two sides are added
// through LDS at the end of a pair of parts and the sum goes to slice s of the partial
// buffer; k_mlp_back adds the slices.
// What bounds it: with samples and W1 cold (8 x 8 workload, 73 MB) their fetch, 25-29 us;
// with 4,096 samples of one learner the chunk's chain of staging, LDS reads and
// MFMAs and the partial sums' write, 26.6 us (45.8 with 32-row x 64-unit waves,
// both operands staged for all waves and 1/4 slices: twice the partial sums).
// The work items are split into eight equal ranges, one per XCD (workgroup b runs
// on XCD b % 8), so the items of one learner share an L2; the unit blocks of a
// quad's slice follow each other, so that they read its sample rows at the same
// time (4,096 samples: 200 MB of reads past the L2s with the unit blocks a round
// apart, 75 MB so).  INLINE: the sample indices come from the kernel arguments
// and the workgroups of slice 0 and unit block 0 copy them to the workspace for
// the later kernels; otherwise they are read from the workspace.  PACKED: W1 comes
// from the workspace in bf16, tile by tile as LDS holds it (k_put_idx packed it), and
// is staged as it is: half the bytes through the L2s and L1s, which deliver 128 KiB
// a chunk step to every CU without it, and no conversion in each of the quads
// (4,096 samples 31.3 us without it in the trace; a second chunk of samples loaded
// ahead on top changed nothing).
constexpr int kFwWaves = 8, kFwMb = 4;
struct SkMap {
  int32_t n;              // learners present
  int32_t S;              // K slices
  int32_t ub;             // unit blocks
  uint32_t learner[4];    // learner id of present learner k in byte k % 4 of word k / 4
  int32_t off[17];        // first work item of each learner (off[n] = total)
  int32_t first[17];      // first list entry of each learner (first[n] = count)
};
static_assert(NBSGD_MAX_LEARNERS <= 16, "SkMap holds at most 16 learners");
static_assert(sizeof(InlineIdx) + sizeof(Dims) + sizeof(SkMap) + 6 * 8 <= 4096,
              "kernel arguments exceed 4 KiB");

template <bool INLINE, bool PACKED, int PAIRS>
__global__ void __launch_bounds__(64 * kFwWaves, 2)
    k_mlp_fwd(const float* __restrict__ X, const __bf16* __restrict__ w1,
              const float* __restrict__ data, int32_t* __restrict__ idx, float* __restrict__ Zpart, int64_t part_stride, Dims d,
              SkMap M, Idx16<INLINE ? kInline * kBatch / 2 : 1> I) {
  constexpr int UB = kFwUnits, KC = kFwKc;
  __shared__ __attribute__((aligned(16))) __bf16 Ws[2][2][UB * KC];
  __shared__ __attribute__((aligned(16))) __bf16 As[kFwWaves][kBatch * KC];
  // the exchange of sums: W1's buffers, which nothing reads after a slice's last step,
  // but a slice's first of two pairs ends with the second's first chunk staged
  __shared__ __attribute__((aligned(16))) float Sums[PAIRS == 2 ? kFwWaves * 16 * UB : 1];
  float* Ex = PAIRS == 2 ? Sums : reinterpret_cast<float*>(Ws);
  static_assert(sizeof(Ws) == kFwWaves * 16 * UB * sizeof(float), "an exchange takes W1's buffers");
  const int xcd = blockIdx.x & 7;
  const int64_t total = M.off[M.n];
  const int item = (int)(xcd * total / 8) + (int)(blockIdx.x >> 3);
  if (item >= (int)((xcd + 1) * total / 8)) return;  // uniform
  int li = 0;
  while (li + 1 < M.n && M.off[li + 1] <= item) ++li;
  const int cnt = M.first[li + 1] - M.first[li];
  const int quads = (cnt + kFwMb - 1) / kFwMb;
  int local = item - M.off[li];
  const int ubk = local % M.ub;
  local /= M.ub;
  const int quad = local % quads, s = local / quads;
  const int e0 = M.first[li] + kFwMb * quad;  // first list entry of the quad
  const int nmb = min(kFwMb, cnt - kFwMb * quad);
  const int H = d.hidden, u0 = UB * ubk;
  const int units = min(UB, H - u0);
  const FwdChunks chunks = {d.d_in / KC};
  const int per = chunks.parts() / M.S;  // parts of a slice
  const int learner = (int)((M.learner[li >> 2] >> (8 * (li & 3))) & 0xffu);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int mb = wave & 3, kh = wave >> 2;
  const int i = lane & 15, g = lane >> 4;
  const bool live = mb < nmb;
  // Mini-batches past the quad's read its first one and unit quads past the block
  // its first units (both in bounds); nothing stores what they give.
  // A: rows 16 f + ar, floats 4 p .. +3 of every 16
  const int p = lane & 3, ar = ((lane >> 2) & 1) | ((lane >> 3) & 3) << 2 | (lane >> 5) << 1;
  const float* ap[2];
#pragma unroll
  for (int f = 0; f < 2; ++f) {
    const int t = (e0 + (live ? mb : 0)) * kBatch + 16 * f + ar;
    int32_t v;
    if constexpr (INLINE) {
      v = (int32_t)((I.v[t >> 1] >> (16 * (t & 1))) & 0xffffu);
      if (live && kh == 0 && s == 0 && ubk == 0 && p == 0) idx[t] = v;
    } else {
      v = idx[t];
    }
    ap[f] = data + (int64_t)v * d.d_in + 4 * p;
  }
  // W1: k 8 wave + 4 half .. +3 of either half's chunk, units 4 wq .. +3; four
  // lanes read 64 contiguous bytes, a load two whole 512-byte row pieces
  const int wq = 4 * (lane >> 3) + (lane & 3);
  const int half = (lane >> 2) & 1;
  const float* wp = X + (int64_t)learner * d.ld + (int64_t)(8 * wave + 4 * half) * H + u0 +
                    (4 * wq < units ? 4 * wq : 0);
  const int wofs = (64 * (wq >> 4) + (wq & 15)) * KC + 8 * (wave ^ fwd_swizzle(wq & 15)) + 4 * half;

  // packed W1: 16 bytes of each 8 KiB of a tile
  const __bf16* pp = w1 + (int64_t)(li * M.ub + ubk) * chunks.T * kFwTile + 8 * tid;

  f32x4 a[2][KC / 16], w[2][4];
  u32x4 wb[2][2];
  auto load_a = [&](int c) {
#pragma unroll
    for (int f = 0; f < 2; ++f)
#pragma unroll
      for (int q = 0; q < KC / 16; ++q) a[f][q] = *reinterpret_cast<const f32x4*>(ap[f] + c * KC + 16 * q);
  };
  auto load_w = [&](int k0, int k1) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int k = h ? k1 : k0;
      if constexpr (PACKED) {
#pragma unroll
        for (int r = 0; r < 2; ++r)
          wb[h][r] = *reinterpret_cast<const u32x4*>(pp + (int64_t)k * kFwTile + r * (kFwTile / 2));
      } else {
#pragma unroll
        for (int r = 0; r < 4; ++r) w[h][r] = *reinterpret_cast<const f32x4*>(wp + (int64_t)(k * KC + r) * H);
      }
    }
  };
  auto stage_w = [&](int buf) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      if constexpr (PACKED) {
#pragma unroll
        for (int r = 0; r < 2; ++r)
          *reinterpret_cast<u32x4*>(&Ws[buf][h][r * (kFwTile / 2) + 8 * tid]) = wb[h][r];
      } else {
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          const uint2 v = {pack_bf16(w[h][0][t], w[h][1][t]), pack_bf16(w[h][2][t], w[h][3][t])};
          *reinterpret_cast<uint2*>(&Ws[buf][h][wofs + 16 * t * KC]) = v;
        }
      }
    }
  };
  __bf16* aw = As[wave];
  auto stage_a = [&]() {
#pragma unroll
    for (int f = 0; f < 2; ++f)
#pragma unroll
      for (int q = 0; q < KC / 16; ++q) {
        const uint2 v = {pack_bf16(a[f][q][0], a[f][q][1]), pack_bf16(a[f][q][2], a[f][q][3])};
        *reinterpret_cast<uint2*>(aw + (16 * f + ar) * KC + 8 * ((2 * q + (p >> 1)) ^ fwd_swizzle(ar)) + 4 * (p & 1)) = v;
      }
    wave_lds_fence();
  };
  f32x4 acc0[2][UB / 16], acc[2][UB / 16];  // of a side's first of two leaves, and of the other or only one
  auto clear = [&]() {
#pragma unroll
    for (int f = 0; f < 2; ++f)
#pragma unroll
      for (int u = 0; u < UB / 16; ++u) acc0[f][u] = acc[f][u] = f32x4{0.f, 0.f, 0.f, 0.f};
  };
  clear();
  auto multiply = [&](int buf, f32x4 (&acc)[2][UB / 16]) {
#pragma unroll
    for (int ks = 0; ks < KC / 32; ++ks) {
      const int o = 8 * ((4 * ks + g) ^ fwd_swizzle(i));
      const bf16x8 a0 = *reinterpret_cast<const bf16x8*>(aw + i * KC + o);
      const bf16x8 a1 = *reinterpret_cast<const bf16x8*>(aw + (16 + i) * KC + o);
#pragma unroll
      for (int u = 0; u < UB / 16; ++u) {
        const bf16x8 b = *reinterpret_cast<const bf16x8*>(
            &Ws[buf][kh][(64 * (u >> 2) + 16 * (u & 3) + i) * KC + o]);
        acc[0][u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a0, b, acc[0][u], 0, 0, 0);
        acc[1][u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a1, b, acc[1][u], 0, 0, 0);
      }
    }
    wave_lds_fence();
  };
  // Ends a pair: wave w < 4 keeps row tile 0 and gives row tile 1 to wave w + 4, through
  // Ex, which the partner reads after a barrier and which is written again a step's
  // barrier later at the earliest.  The sum of a slice's first pair waits for the
  // second where this wave read the partner's share of it.
  f32x4 sum[UB / 64][4];
  auto add = [&](bool first, bool last) {
    if constexpr (PAIRS > 0) {
#pragma unroll
      for (int f = 0; f < 2; ++f)
#pragma unroll
        for (int u = 0; u < UB / 16; ++u) acc[f][u] += acc0[f][u];
    }
    f32x4* give = reinterpret_cast<f32x4*>(Ex + wave * (16 * UB)) + lane;
    f32x4* take = reinterpret_cast<f32x4*>(Ex + (wave ^ 4) * (16 * UB)) + lane;
    if (PAIRS == 2 && !first) {
#pragma unroll
      for (int q = 0; q < UB / 64; ++q)
#pragma unroll
        for (int t = 0; t < 4; ++t) sum[q][t] = take[64 * (4 * q + t)];
      __syncthreads();
    }
#pragma unroll
    for (int q = 0; q < UB / 64; ++q)
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        f32x4 v;
#pragma unroll
        for (int o = 0; o < 4; ++o) {
          const float lo = acc[0][4 * q + o][t], hi = acc[1][4 * q + o][t];
          v[o] = kh ? lo : hi;
        }
        give[64 * (4 * q + t)] = v;
      }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < UB / 64; ++q)
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        f32x4 v = take[64 * (4 * q + t)];
#pragma unroll
        for (int o = 0; o < 4; ++o) {
          const float lo = acc[0][4 * q + o][t], hi = acc[1][4 * q + o][t];
          v[o] += kh ? hi : lo;
        }
        sum[q][t] = PAIRS < 2 || first ? v : sum[q][t] + v;
      }
    if (PAIRS == 2 && !last) {
#pragma unroll
      for (int q = 0; q < UB / 64; ++q)
#pragma unroll
        for (int t = 0; t < 4; ++t) take[64 * (4 * q + t)] = sum[q][t];
      clear();
    }
  };
  fwd_walk<PAIRS, PACKED>(
      chunks, s * per, (s + 1) * per, kh, load_w, load_a, stage_w, stage_a,
      [&](int buf) { multiply(buf, acc0); }, [&](int buf) { multiply(buf, acc); },
      [] { __syncthreads(); }, add);
  if (!live) return;
  float* out = Zpart + (int64_t)s * part_stride + ((int64_t)(e0 + mb) * kBatch + 16 * kh) * H + u0 + 4 * i;
#pragma unroll
  for (int q = 0; q < UB / 64; ++q) {
    if (64 * q >= units) break;
#pragma unroll
    for (int t = 0; t < 4; ++t) *reinterpret_cast<f32x4*>(out + (int64_t)(4 * g + t) * H + 64 * q) = sum[q][t];
  }
}

// Per list entry e = blockIdx.x (workspace rows e * 32 ..; G row and loss of its
// slot) and, when BACKWARD, every gridDim.y-th block of 128 features from
// blockIdx.y.  Eight waves, 32 rows, all hidden units:
//   Z1 = the S partial slices (in the order of mlp_plan.h) + b1; kept in LDS as bf16
//   relu(Z1), with -0 where Z1 is not above zero, which is the ReLU's mask
//   logits = relu(Z1) bf16(W2) + b2 on the matrix cores (classes zero-padded to
//   16; wave w takes the 32-unit K steps w and w + 8, the waves' sums are added in
//   wave order), softmax cross-entropy by one thread per (row, class), the loss
//   and dZ2 = (softmax - onehot) / 32
//   dZ1 = (bf16(dZ2) bf16(W2)^T) * [Z1 > 0], which stays in registers: a result's
//   rows 4 g + t and 16 + 4 g + t (g = lane / 16) are the K order of the dW1 product,
//   kk(g, t), so the two row tiles of a unit are its B fragment as they are
//   (unit 4 i + j of a 64-unit group in lane i of tile j)
//   dW1[f][h] = sum_r bf16(A[s_r][f]) bf16(dZ1[r][h]): A fragments (16 features, the
//   rows in kk order) from the sample columns staged in LDS, two buffers; a wave
//   takes two groups of units, swaps half rows between their results
//   (v_permlane16_swap) and stores 512 contiguous bytes of two G rows at a time
//   workgroups blockIdx.y == 0 write db1 (row sums by lane shuffles), dW2 =
//   relu(Z1)^T dZ2 (the mask's registers are its A fragment), db2, the padding of
//   G and the loss
// Bound by the 299 MB of G that the 8 x 8 workload writes (48 us at the 6.2 TB/s of
// a large copy; 58-60 us here) after 10 us to the first store.  It replaces a head
// kernel, one 1024-thread workgroup per mini-batch (15.8 us, 209 CUs idle), that
// passed dZ1 through memory to a dW1 kernel (53.2 us): recomputing the head in
// every workgroup costs less than its launch on few CUs.  The features are taken
// in turns, so that all workgroups write G in increasing column order and the
// step, which reads from the last column, finds the newest in the memory-side
// cache (a contiguous range per workgroup: 97.1 against 95.9 us, and a slower step).
constexpr int kBackThreads = 512, kBackWaves = kBackThreads / 64;

template <bool BACKWARD>
__global__ void __launch_bounds__(kBackThreads, 4)
    k_mlp_back(const float* __restrict__ X, const float* __restrict__ data,
               const int32_t* __restrict__ idx, const int32_t* __restrict__ labels,
               const float* __restrict__ Zpart, int64_t part_stride, int S, float* __restrict__ G,
               float* __restrict__ losses, Dims d, List L) {
  constexpr int kLdh = kMaxHidden + 8;  // bf16 per row of Hs
  __shared__ __attribute__((aligned(16))) __bf16 Hs[kBatch * kLdh];
  __shared__ __attribute__((aligned(16))) __bf16 W2s[kMaxHidden * kMaxClasses];  // [unit][16]
  __shared__ float Zs[kBatch * kMaxClasses];                     // dZ2
  __shared__ __attribute__((aligned(16))) __bf16 Zb[kBatch * kMaxClasses];  // bf16(dZ2)
  __shared__ float row_loss[kBatch];
  __shared__ int ys[kBatch];
  // each wave's partial logits, then the sample columns of two feature blocks
  __shared__ __attribute__((aligned(16))) float Lp[kBackWaves * kBatch * 16];
  static_assert(sizeof(Lp) == 2 * kFeatBlock * kBatch * sizeof(__bf16), "two buffers");
  __bf16* At = reinterpret_cast<__bf16*>(Lp);
  const int e = blockIdx.x;
  if (e >= L.count) return;  // uniform
  const uint32_t item = L.w[e];
  const int slot = item_slot(item);
  const float* prm = X + (int64_t)item_learner(item) * d.ld;
  const int H = d.hidden, C = d.classes;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int i = lane & 15, g = lane >> 4;
  const int64_t row0 = (int64_t)e * kBatch;
  const int nb = d.d_in / kFeatBlock;
  const int blk0 = blockIdx.y, step = gridDim.y;  // blocks blk0, blk0 + step, ..
  const bool first = BACKWARD && blockIdx.y == 0;  // writes what is not dW1

  const int32_t sample = idx[row0 + (tid & (kBatch - 1))];
  // samples: rows 2 pr, 2 pr + 1, features fq .. +3 of a block
  const int pr = tid >> 5, fq = 4 * (tid & 31);
  const float* s0 = data + (int64_t)idx[row0 + 2 * pr] * d.d_in + fq;
  const float* s1 = data + (int64_t)idx[row0 + 2 * pr + 1] * d.d_in + fq;
  f32x4 x0, x1;

  float b2v;
  {
    // Z1: row r, units uq + 64 j; every load of a half is issued before any is
    // used, and the rest of the phase's with the first half's
    const int r = tid >> 4, uq = 4 * (tid & 15);
    const float* src = Zpart + (row0 + r) * H + uq;
    const float* pb = prm + d.off_b1 + uq;
    const float* pw = prm + d.off_w2 + (int64_t)min(tid, H - 1) * C;
    float w2[kMaxClasses];
    int32_t y;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      if (256 * h >= H) break;
      f32x4 p[kSkMaxSlices][4], b[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int u = 64 * (4 * h + j);
        if (u < H) {  // uniform, as every condition on j and q here
#pragma unroll
          for (int q = 0; q < kSkMaxSlices; ++q)
            if (q < S) p[q][j] = *reinterpret_cast<const f32x4*>(src + (int64_t)q * part_stride + u);
          b[j] = *reinterpret_cast<const f32x4*>(pb + u);
        }
      }
      if (h == 0) {
        y = labels[sample];
        b2v = prm[d.off_b2 + min(tid & 15, C - 1)];
        if (BACKWARD) {
          x0 = *reinterpret_cast<const f32x4*>(s0 + blk0 * kFeatBlock);
          x1 = *reinterpret_cast<const f32x4*>(s1 + blk0 * kFeatBlock);
        }
      }
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int u = 64 * (4 * h + j);
        if (u < H) {
          f32x4 z = p[0][j];
          if (S > 1) z += p[1][j];
          if (S == 3) z += p[2][j];
          if (S == 4) z += p[2][j] + p[3][j];
          z += b[j];
          // relu(z) in bf16; -0 where z is not above zero
#pragma unroll
          for (int t = 0; t < 4; ++t) z[t] = z[t] > 0.0f ? z[t] : -0.0f;
          const uint2 v = {pack_bf16(z[0], z[1]), pack_bf16(z[2], z[3])};
          *reinterpret_cast<uint2*>(Hs + r * kLdh + uq + u) = v;
        }
      }
      if (h == 0) {
#pragma unroll
        for (int k = 0; k < kMaxClasses; ++k)
          if (k < C) w2[k] = pw[k];
      }
    }
    uint32_t wv[kMaxClasses / 2];
#pragma unroll
    for (int k = 0; k < kMaxClasses / 2; ++k)
      wv[k] = pack_bf16(2 * k < C ? w2[2 * k] : 0.0f, 2 * k + 1 < C ? w2[2 * k + 1] : 0.0f);
    if (tid < H) {
      *reinterpret_cast<uint4*>(W2s + tid * kMaxClasses) = (uint4){wv[0], wv[1], wv[2], wv[3]};
      *reinterpret_cast<uint4*>(W2s + tid * kMaxClasses + 8) = (uint4){wv[4], wv[5], wv[6], wv[7]};
    }
    if (tid < kBatch) ys[tid] = y < 0 ? 0 : (y >= C ? C - 1 : y);
  }
  // position of row 2 pr of a sample column: rows 4 g + t and 16 + 4 g + t at 8 g + t and 8 g + 4 + t
  const int rr = 2 * pr, opos = (rr & 15) >> 2, wpos = (rr & 3) + 4 * (rr >> 4);
  // octet of a sample column's 32 rows: in the 16 columns of a fragment read, equal
  // bank groups (columns four apart) get four values, {0, 1} and {2, 3} for the two
  // halves of the hardware's 16-lane passes
  auto aswz = [](int f) { const int q = (f >> 2) & 3; return (((q ^ (q >> 1)) & 1) << 1) | (q >> 1); };
  auto stage_x = [&](int buf) {
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const int f = fq + c;
      *reinterpret_cast<uint32_t*>(&At[buf * kFeatBlock * kBatch + f * kBatch + 8 * (opos ^ aswz(f)) + wpos]) = pack_bf16(x0[c], x1[c]);
    }
  };
  __syncthreads();
  {
    f32x4 acc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
    for (int ks = wave; ks < H / 32; ks += kBackWaves) {
      const int u0 = 32 * ks + 8 * g;
      bf16x8 fb;
#pragma unroll
      for (int t = 0; t < 8; ++t) fb[t] = W2s[(u0 + t) * kMaxClasses + i];
#pragma unroll
      for (int rt = 0; rt < 2; ++rt) {
        const bf16x8 fa = *reinterpret_cast<const bf16x8*>(Hs + (16 * rt + i) * kLdh + u0);
        acc[rt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa, fb, acc[rt], 0, 0, 0);
      }
    }
#pragma unroll
    for (int rt = 0; rt < 2; ++rt)
#pragma unroll
      for (int t = 0; t < 4; ++t) Lp[(wave * kBatch + 16 * rt + 4 * g + t) * 16 + i] = acc[rt][t];
  }
  __syncthreads();
  {
    const int r = tid >> 4, c = tid & 15;
    const bool live = c < C;
    float z = 0.0f;
#pragma unroll
    for (int w = 0; w < kBackWaves; ++w) z += Lp[(w * kBatch + r) * 16 + c];
    z += b2v;
    float zmax = live ? z : -INFINITY;
#pragma unroll
    for (int o = 8; o; o >>= 1) zmax = fmaxf(zmax, __shfl_xor(zmax, o, 16));
    float sum = live ? expf(z - zmax) : 0.0f;
#pragma unroll
    for (int o = 8; o; o >>= 1) sum += __shfl_xor(sum, o, 16);
    const float lse = zmax + logf(sum);
    const int yr = ys[r];
    if (c == yr) row_loss[r] = lse - z;
    if (BACKWARD) {
      const float gz = live ? (expf(z - lse) - (c == yr ? 1.0f : 0.0f)) * (1.0f / kBatch) : 0.0f;
      Zs[r * kMaxClasses + c] = gz;
      Zb[r * kMaxClasses + c] = (__bf16)gz;
    }
  }
  __syncthreads();
  if ((!BACKWARD || first) && tid == 0) {
    float s = 0.0f;
    for (int r = 0; r < kBatch; ++r) s += row_loss[r];
    losses[slot] = s * (1.0f / kBatch);
  }
  if (!BACKWARD) return;
  stage_x(0);
  float* gr = G + (int64_t)slot * d.ld;
  if (first) {
    if (tid < C) {
      float s = 0.0f;
      for (int r = 0; r < kBatch; ++r) s += Zs[r * kMaxClasses + tid];
      gr[d.off_b2 + tid] = s;
    }
    if (tid < d.P - d.off_pad) gr[d.off_pad + tid] = 0.0f;
  }
  // the wave's units: two neighbouring groups of 64 (the last may be alone), and
  // its share of the feature tiles
  const int ng = H / 64, np = (ng + 1) / 2, parts = kBackWaves / np;
  const int pair = wave % np, part = wave / np;
  const bool busy = part < parts, two = 2 * pair + 1 < ng;  // uniform
  bf16x8 dz[2][4];
  if (busy) {
    bf16x8 fz[2];
#pragma unroll
    for (int rt = 0; rt < 2; ++rt) {
      fz[rt] = *reinterpret_cast<const bf16x8*>(Zb + (16 * rt + i) * kMaxClasses + 8 * (g & 1));
      if (g > 1) fz[rt] = (bf16x8)((__bf16)0.0f);
    }
    bf16x8 fd;  // B[row kk][class]
#pragma unroll
    for (int t = 0; t < 8; ++t) fd[t] = Zb[(4 * g + (t & 3) + 16 * (t >> 2)) * kMaxClasses + i];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const int ub = 64 * (2 * pair + (two ? q : 0)) + 4 * i;  // units ub + j, j = tile
      uint2 h[8];  // H of rows kk(g, t), units ub .. ub + 3
#pragma unroll
      for (int t = 0; t < 8; ++t)
        h[t] = *reinterpret_cast<const uint2*>(Hs + (4 * g + (t & 3) + 16 * (t >> 2)) * kLdh + ub);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        // B[class][unit]; classes 16-31 are zero on both sides (a zero of fz alone
        // would make an infinite weight NaN)
        bf16x8 fw = *reinterpret_cast<const bf16x8*>(W2s + (ub + j) * kMaxClasses + 8 * (g & 1));
        if (g > 1) fw = (bf16x8)((__bf16)0.0f);
        f32x4 v[2];
        float db1 = 0.0f;
#pragma unroll
        for (int rt = 0; rt < 2; ++rt) {
          v[rt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fz[rt], fw, (f32x4){0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
#pragma unroll
          for (int t = 0; t < 4; ++t) {
            const uint2 hh = h[4 * rt + t];
            const uint32_t bits = j < 2 ? hh.x : hh.y;
            v[rt][t] = (bits >> (j & 1 ? 31 : 15)) & 1 ? 0.0f : v[rt][t];
            db1 += v[rt][t];
          }
        }
        dz[q][j] = to_bf16(v[0], v[1]);
        if (first && part == 0 && (q == 0 || two)) {
          db1 += __shfl_xor(db1, 16);
          db1 += __shfl_xor(db1, 32);
          if (lane < 16) gr[d.off_b1 + ub + j] = db1;
          uint32_t hw[4];
#pragma unroll
          for (int o = 0; o < 4; ++o) {
            const uint32_t a = j < 2 ? h[2 * o].x : h[2 * o].y, b = j < 2 ? h[2 * o + 1].x : h[2 * o + 1].y;
            hw[o] = j & 1 ? (a >> 16) | (b & 0xffff0000u) : (a & 0xffffu) | (b << 16);
          }
          const bf16x8 fh = __builtin_bit_cast(bf16x8, (uint4){hw[0], hw[1], hw[2], hw[3]});
          const f32x4 acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fh, fd, (f32x4){0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
          if (i < C) {
#pragma unroll
            for (int t = 0; t < 4; ++t)  // unit of M index 4 g + t
              gr[d.off_w2 + (int64_t)(64 * (2 * pair + q) + 4 * (4 * g + t) + j) * C + i] = acc[t];
          }
        }
      }
    }
  }
  __syncthreads();
  int buf = 0;
  for (int blk = blk0; blk < nb; blk += step, buf ^= 1) {
    if (blk + step < nb) {
      x0 = *reinterpret_cast<const f32x4*>(s0 + (blk + step) * kFeatBlock);
      x1 = *reinterpret_cast<const f32x4*>(s1 + (blk + step) * kFeatBlock);
    }
    if (busy) {
      // group 2 pair of feature 4 g + t, and once swapped both groups of two features
      float* o = gr + (int64_t)blk * kFeatBlock * H + 128 * pair + 4 * i;
#pragma unroll 1
      for (int ft = part; ft < kFeatBlock / 16; ft += parts) {
        const int f = 16 * ft + i;
        const bf16x8 a = *reinterpret_cast<const bf16x8*>(&At[buf * kFeatBlock * kBatch + f * kBatch + 8 * (g ^ aswz(f))]);
        f32x4 acc[2][4];
#pragma unroll
        for (int q = 0; q < 2; ++q) {
#pragma unroll
          for (int j = 0; j < 4; ++j)
            acc[q][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, dz[q][j], (f32x4){0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
        }
        if (two) {
          float* o2 = o + 64 * (g & 1);
#pragma unroll
          for (int t = 0; t < 4; ++t) {
            f32x4 lo, hi;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
              const float a0 = acc[0][j][t], a1 = acc[1][j][t];
              const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a0), __float_as_uint(a1), false, false);
              const uint32_t r0 = r[0], r1 = r[1];
              lo[j] = __uint_as_float(r0);
              hi[j] = __uint_as_float(r1);
            }
            const int fl = 16 * ft + 4 * (g & 2) + t;  // lanes 0-31: features t, 32-63: 8 + t
            *reinterpret_cast<f32x4*>(o2 + (int64_t)fl * H) = lo;
            *reinterpret_cast<f32x4*>(o2 + (int64_t)(fl + 4) * H) = hi;
          }
        } else {
#pragma unroll
          for (int t = 0; t < 4; ++t)
            *reinterpret_cast<f32x4*>(o + (int64_t)(16 * ft + 4 * g + t) * H) =
                (f32x4){acc[0][0][t], acc[0][1][t], acc[0][2][t], acc[0][3][t]};
        }
      }
    }
    if (blk + step < nb) {
      stage_x(buf ^ 1);
      __syncthreads();
    }
  }
}

// ------------------------------------------------------------------ host

struct Workspace {
  int32_t* idx;
  __bf16* w1;         // packed W1, where it fits
  size_t w1_bytes;
  float* part;        // partial Z1 of each d_in slice
  int64_t part_stride;
};

Workspace carve(void* ws, const Dims& d, int64_t rows) {
  char* p = static_cast<char*>(ws);
  Workspace w;
  w.idx = reinterpret_cast<int32_t*>(p);
  p += up256((size_t)rows * 4);
  w.w1 = reinterpret_cast<__bf16*>(p);
  w.w1_bytes = up256((size_t)rows * d.hidden * 2);
  p += w.w1_bytes;
  w.part = reinterpret_cast<float*>(p);
  w.part_stride = (int64_t)(up256((size_t)rows * d.hidden * 4) / 4);
  return w;
}

// Checks every sample index of the mini-batches `slots` (host idx[slot*32 ..]).
nbsgd_status check_idx(const int32_t* host, const int32_t* slots, int n_slots, int64_t n_samples) {
  for (int k = 0; k < n_slots; ++k)
    for (int r = 0; r < kBatch; ++r) {
      const int64_t pos = (int64_t)slots[k] * kBatch + r;
      if (host[pos] < 0 || host[pos] >= n_samples)
        return fail(NBSGD_E_ARG, "sample index %d at position %lld is outside [0, %lld)", host[pos],
                    (long long)pos, (long long)n_samples);
    }
  return NBSGD_OK;
}

// Copies the sample indices of list entries 0 .. count-1 (host idx[slot*32 ..]
// of entry e's slot mb[e].second) to the workspace rows e*32 .. through the
// kernel arguments of k_put_idx; its first launch also packs `tiles` tiles of W1.
void put_idx(const int32_t* host, const std::pair<int, int>* mb, int count, bool wide,
             const Workspace& w, Pack pack, int tiles, hipStream_t s) {
  const int per = wide ? kUpSlots / 2 : kUpSlots;
  for (int k0 = 0; k0 < count; k0 += per) {
    IdxChunk c;
    memset(&c, 0, sizeof(c));
    c.first = k0;
    c.n_slots = std::min(per, count - k0);
    c.wide = wide ? 1 : 0;
    for (int k = 0; k < c.n_slots; ++k) {
      const int32_t* src = host + (int64_t)mb[k0 + k].second * kBatch;
      for (int r = 0; r < kBatch; ++r) {
        const int t = k * kBatch + r;
        if (wide) c.v[t] = (uint32_t)src[r];
        else c.v[t >> 1] |= (uint32_t)src[r] << (16 * (t & 1));
      }
    }
    pack.idx_blocks = (c.n_slots * kBatch + 255) / 256;
    hipLaunchKernelGGL(k_put_idx, dim3(pack.idx_blocks + (k0 ? 0 : tiles)), dim3(256), 0, s, w.idx, c,
                       pack);
  }
}

nbsgd_status launch_err(const char* what) {
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(NBSGD_E_HIP, "%s launch failed: %s", what, hipGetErrorString(e));
  return NBSGD_OK;
}

uint32_t item(int learner, int slot) { return ((uint32_t)learner << 24) | ((uint32_t)slot << 12); }

// Chunk steps of a CU from which the forward reads W1 packed: a step saves 0.2-0.4
// us, packing adds 1-1.5 us to a launch that is there anyway (a group whose indices
// go inline has none and is never packed).  mlp_loss, 32-sample batches x d_in x
// hidden, packed against not: 512 x 3072x512 (48 steps) 129.6 and 148.1 us, 256 x
// 3072x512 (24) 69.9 and 77.3, 128 x 3072x512 (12) 41.2 and 43.0, 256 x 896x512 (7) 38.8
// and 39.5, 70 x 1152x512 (5) 24.7 and 25.5, 128 x 1024x512 (4) 27.7 and 28.6, 40 x
// 1152x512 (3) 19.3 and 19.3; gradients of 8 x 16 mini-batches 384x512 (3) 52.7 and 52.5.
constexpr int kPackSteps = 4;

// Tiles of W1 that the forward of this group reads packed; 0 where it does not, or
// where they would not fit their part of the workspace.
int pack_tiles(const SkMap& K, const Dims& d, int steps, const Workspace& w) {
  const int tiles = K.n * K.ub * (d.d_in / kFwKc);
  return steps >= kPackSteps && (size_t)tiles * kFwTile * sizeof(__bf16) <= w.w1_bytes ? tiles : 0;
}

// Launches the kernels over mini-batches `mb` (learner, slot), sorted by
// learner, of one group (at most kMaxList): the sample indices host_idx[slot
// * 32 ..] (checked) go to the workspace in the forward kernel's arguments
// when the group has at most kInline mini-batches and they fit 16 bits
// (`wide` false), otherwise through k_put_idx first, which also packs W1 for long
// forwards.
template <bool BACKWARD>
void launch_group(const std::pair<int, int>* mb, int count, const int32_t* host_idx, bool wide,
                  const float* X, const float* data, const int32_t* labels, const Workspace& w,
                  float* G, float* losses, const Dims& d, hipStream_t st) {
  List items;
  items.count = count;
  for (int k = 0; k < count; ++k) items.w[k] = item(mb[k].first, mb[k].second);
  // forward over quads of each learner's mini-batches, slices of d_in
  SkMap K;
  memset(&K, 0, sizeof K);
  K.ub = (d.hidden + kFwUnits - 1) / kFwUnits;
  int sk_total = 0;
  for (int k = 0; k < items.count; ++k) {
    if (k == 0 || item_learner(items.w[k]) != item_learner(items.w[k - 1])) {
      K.first[K.n] = k;
      K.learner[K.n >> 2] |= (uint32_t)item_learner(items.w[k]) << (8 * (K.n & 3));
      ++K.n;
    }
  }
  K.first[K.n] = items.count;
  int tiles = 0;
  for (int k = 0; k < K.n; ++k) tiles += K.ub * ((K.first[k + 1] - K.first[k] + kFwMb - 1) / kFwMb);
  int steps = 0;
  K.S = fwd_slices(d.d_in, tiles, &steps);
  for (int k = 0; k < K.n; ++k) {
    K.off[k] = sk_total;
    sk_total += K.S * K.ub * ((K.first[k + 1] - K.first[k] + kFwMb - 1) / kFwMb);
  }
  K.off[K.n] = sk_total;
  const dim3 fgrid(8 * ((sk_total + 7) / 8));
  const int pairs = fwd_pairs(FwdChunks{d.d_in / kFwKc}.parts() / K.S);
  if (!wide && count <= kInline) {
    InlineIdx I;
    memset(&I, 0, sizeof I);
    for (int e = 0; e < count; ++e) {
      const int32_t* src = host_idx + (int64_t)mb[e].second * kBatch;
      for (int r = 0; r < kBatch; ++r) {
        const int t = e * kBatch + r;
        I.v[t >> 1] |= (uint32_t)src[r] << (16 * (t & 1));
      }
    }
    const auto kernel = pairs == 0 ? k_mlp_fwd<true, false, 0> : pairs == 1 ? k_mlp_fwd<true, false, 1> : k_mlp_fwd<true, false, 2>;
    hipLaunchKernelGGL(kernel, fgrid, dim3(64 * kFwWaves), 0, st, X, w.w1, data, w.idx, w.part, w.part_stride, d,
                       K, I);
  } else {
    const int pk = pack_tiles(K, d, steps, w);
    Pack pack;
    memset(&pack, 0, sizeof pack);
    pack.X = X;
    pack.w1 = w.w1;
    pack.ld = d.ld;
    pack.hidden = d.hidden;
    pack.chunks = d.d_in / kFwKc;
    pack.ub = K.ub;
    memcpy(pack.learner, K.learner, sizeof pack.learner);
    put_idx(host_idx, mb, count, wide, w, pack, pk, st);
    const Idx16<1> none = {{0u}};
    const auto kernel = pk ? (pairs == 0 ? k_mlp_fwd<false, true, 0> : pairs == 1 ? k_mlp_fwd<false, true, 1> : k_mlp_fwd<false, true, 2>)
                           : (pairs == 0 ? k_mlp_fwd<false, false, 0> : pairs == 1 ? k_mlp_fwd<false, false, 1> : k_mlp_fwd<false, false, 2>);
    hipLaunchKernelGGL(kernel, fgrid, dim3(64 * kFwWaves), 0, st, X, w.w1, data, w.idx, w.part, w.part_stride, d,
                       K, none);
  }
  const int entries = back_entries(count), blocks = d.d_in / kFeatBlock;
  const int each = back_blocks(blocks, entries);
  hipLaunchKernelGGL(k_mlp_back<BACKWARD>, dim3(entries, BACKWARD ? (blocks + each - 1) / each : 1),
                     dim3(kBackThreads), 0, st, X, data, w.idx, labels, w.part, w.part_stride, K.S, G,
                     losses, d, items);
}

}  // namespace

namespace {

// Argument checks shared by the gradient entry points, before the workspace
// and the sample indices (checked by the caller, in that order): shapes, row
// stride, pointers and alignment.  On success *d holds the shape with d->ld
// set and *finished the finished (learner * m + mini-batch) entries in order.
nbsgd_status mlp_grad_check(const float* X, int64_t ld, int32_t n, int32_t m,
                            const nbsgd_mlp_shape* s, const float* data, const int32_t* labels,
                            int64_t n_samples, const int32_t* idx, const uint8_t* mask, float* G,
                            float* losses, Dims* d, std::vector<int32_t>* finished) {
  if (nbsgd_status st = check_nm(n, m)) return st;
  if (nbsgd_status st = check_shape(s, d)) return st;
  if (ld == 0) ld = d->P;
  if (ld < d->P || ld % 4)
    return fail(NBSGD_E_SHAPE, "row stride %lld must be a multiple of 4 and at least P=%lld",
                (long long)ld, (long long)d->P);
  d->ld = ld;
  if (!X || !data || !labels || !idx || !mask || !G || !losses)
    return fail(NBSGD_E_ARG, "null pointer argument");
  if (((uintptr_t)X | (uintptr_t)data | (uintptr_t)G) & 15)
    return fail(NBSGD_E_ALIGN, "X, data and G must be 16-byte aligned");
  if (n_samples < 1) return fail(NBSGD_E_SHAPE, "n_samples must be >= 1");
  finished->clear();
  for (int32_t k = 0; k < n * m; ++k)
    if (mask[k]) finished->push_back(k);
  return NBSGD_OK;
}

// Launches the gradient kernels of the finished mini-batches in groups of at
// most kMaxList, each group's workspace rows starting at entry 0 of `w`.
nbsgd_status mlp_grad_launch(const float* X, int32_t m, const Dims& d, const float* data,
                             const int32_t* labels, int64_t n_samples, const int32_t* idx,
                             const std::vector<int32_t>& finished, float* G, float* losses,
                             const Workspace& w, hipStream_t st) {
  const bool wide = n_samples > 65536;
  std::pair<int, int> mb[kMaxList];
  int count = 0;
  for (int32_t k : finished) {
    mb[count++] = {k / m, k};
    if (count == kMaxList) {
      launch_group<true>(mb, count, idx, wide, X, data, labels, w, G, losses, d, st);
      count = 0;
    }
  }
  if (count) launch_group<true>(mb, count, idx, wide, X, data, labels, w, G, losses, d, st);
  return launch_err("nbsgd_mlp_grad");
}

nbsgd_status mlp_grad_impl(const float* X, int64_t ld, int32_t n, int32_t m,
                           const nbsgd_mlp_shape* s, const float* data, const int32_t* labels,
                           int64_t n_samples, const int32_t* idx, const uint8_t* mask, float* G,
                           float* losses, void* workspace, size_t workspace_bytes, void* stream) {
  Dims d;
  std::vector<int32_t> finished;
  if (nbsgd_status st = mlp_grad_check(X, ld, n, m, s, data, labels, n_samples, idx, mask, G,
                                       losses, &d, &finished))
    return st;
  if (!workspace) return fail(NBSGD_E_ARG, "null pointer argument");
  if ((uintptr_t)workspace & 15) return fail(NBSGD_E_ALIGN, "workspace must be 16-byte aligned");
  const int64_t rows = (int64_t)n * m * kBatch;
  if (workspace_bytes < workspace_for(d, rows))
    return fail(NBSGD_E_ARG, "workspace of %zu bytes is below the %zu needed", workspace_bytes,
                workspace_for(d, rows));
  if (nbsgd_status r = check_idx(idx, finished.data(), (int)finished.size(), n_samples)) return r;
  return mlp_grad_launch(X, m, d, data, labels, n_samples, idx, finished, G, losses,
                         carve(workspace, d, rows), reinterpret_cast<hipStream_t>(stream));
}

// ------------------------------------------------ allocation-free variant
// The workspace of nbsgd_mlp_grad_noalloc: a static device array, one copy
// per GPU the library is loaded on, held until the process ends.  Host code
// never passes `scratch` itself to a kernel (on the host the name is only a
// stand-in for the symbol): the device address of each GPU's copy comes from
// hipGetSymbolAddress with that GPU current, and is kept per device.
static __device__ __align__(256) unsigned char scratch[NBSGD_MLP_SCRATCH_BYTES];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices] = {};

// Device address of the current device's scratch, looked up once per device.
nbsgd_status scratch_address(hipStream_t stream, void** out) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return fail(NBSGD_E_HIP, "hipGetDevice: %s", hipGetErrorString(e));
  if (stream) {
    hipDevice_t sdev = -1;
    e = hipStreamGetDevice(stream, &sdev);
    if (e != hipSuccess) return fail(NBSGD_E_HIP, "hipStreamGetDevice: %s", hipGetErrorString(e));
    if (sdev != dev)
      return fail(NBSGD_E_ARG, "stream belongs to device %d but device %d is current", (int)sdev,
                  dev);
  }
  if (dev < 0 || dev >= kMaxDevices)
    return fail(NBSGD_E_UNSUPPORTED, "device %d is beyond the %d devices supported", dev,
                kMaxDevices);
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !p)
      return fail(NBSGD_E_HIP, "hipGetSymbolAddress(scratch) on device %d: %s", dev,
                  hipGetErrorString(e));
    g_scratch_ptr[dev] = p;
  }
  *out = g_scratch_ptr[dev];
  return NBSGD_OK;
}

}  // namespace

extern "C" nbsgd_status nbsgd_mlp_grad(const float* X, int32_t n, int32_t m, const nbsgd_mlp_shape* s,
                                       const float* data, const int32_t* labels, int64_t n_samples,
                                       const int32_t* idx, const uint8_t* mask, float* G,
                                       float* losses, void* workspace, size_t workspace_bytes,
                                       void* stream) {
  clear_error();
  return mlp_grad_impl(X, 0, n, m, s, data, labels, n_samples, idx, mask, G, losses, workspace,
                       workspace_bytes, stream);
}

extern "C" nbsgd_status nbsgd_mlp_grad_strided(const float* X, int64_t ld, int32_t n, int32_t m,
                                               const nbsgd_mlp_shape* s, const float* data,
                                               const int32_t* labels, int64_t n_samples,
                                               const int32_t* idx, const uint8_t* mask, float* G,
                                               float* losses, void* workspace,
                                               size_t workspace_bytes, void* stream) {
  clear_error();
  if (ld <= 0) return fail(NBSGD_E_SHAPE, "row stride %lld must be positive", (long long)ld);
  return mlp_grad_impl(X, ld, n, m, s, data, labels, n_samples, idx, mask, G, losses, workspace,
                       workspace_bytes, stream);
}

extern "C" nbsgd_status nbsgd_mlp_grad_noalloc(const float* X, int64_t ld, int32_t n, int32_t m,
                                               const nbsgd_mlp_shape* s, const float* data,
                                               const int32_t* labels, int64_t n_samples,
                                               const int32_t* idx, const uint8_t* mask, float* G,
                                               float* losses, void* stream) {
  clear_error();
  if (ld <= 0) return fail(NBSGD_E_SHAPE, "row stride %lld must be positive", (long long)ld);
  Dims d;
  std::vector<int32_t> finished;
  if (nbsgd_status st = mlp_grad_check(X, ld, n, m, s, data, labels, n_samples, idx, mask, G,
                                       losses, &d, &finished))
    return st;
  // workspace rows for one launch group: the kernels index them by the
  // group's list entries, so the largest group sets the size
  const int64_t rows = (int64_t)std::min<size_t>(finished.size(), kMaxList) * kBatch;
  const size_t need = workspace_for(d, rows);
  if (need > (size_t)NBSGD_MLP_SCRATCH_BYTES)
    return fail(NBSGD_E_UNSUPPORTED,
                "%zu finished mini-batches of this shape need %zu bytes of workspace, above the "
                "%zu-byte static scratch buffer (use nbsgd_mlp_grad_strided with a workspace)",
                finished.size(), need, (size_t)NBSGD_MLP_SCRATCH_BYTES);
  if (nbsgd_status r = check_idx(idx, finished.data(), (int)finished.size(), n_samples)) return r;
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  void* ws = nullptr;
  if (nbsgd_status r = scratch_address(st, &ws)) return r;
  return mlp_grad_launch(X, m, d, data, labels, n_samples, idx, finished, G, losses,
                         carve(ws, d, rows), st);
}

extern "C" nbsgd_status nbsgd_mlp_loss(const float* params, const nbsgd_mlp_shape* s,
                                       const float* data, const int32_t* labels, int64_t n_samples,
                                       const int32_t* idx, int32_t count, float* losses,
                                       void* workspace, size_t workspace_bytes, void* stream) {
  clear_error();
  Dims d;
  if (nbsgd_status st = check_shape(s, &d)) return st;
  if (!params || !data || !labels || !idx || !losses || !workspace)
    return fail(NBSGD_E_ARG, "null pointer argument");
  if (((uintptr_t)params | (uintptr_t)data | (uintptr_t)workspace) & 15)
    return fail(NBSGD_E_ALIGN, "params, data and workspace must be 16-byte aligned");
  if (n_samples < 1) return fail(NBSGD_E_SHAPE, "n_samples must be >= 1");
  if (count < kBatch || count % kBatch || count / kBatch > kMaxEval)
    return fail(NBSGD_E_SHAPE, "count=%d must be a multiple of %d, at most %d", count, kBatch,
                kBatch * kMaxEval);
  if (workspace_bytes < workspace_for(d, count))
    return fail(NBSGD_E_ARG, "workspace of %zu bytes is below the %zu needed", workspace_bytes,
                workspace_for(d, count));
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  const Workspace w = carve(workspace, d, count);
  std::pair<int, int> mb[kMaxEval];
  int32_t slots[kMaxEval];
  for (int32_t k = 0; k < count / kBatch; ++k) {
    mb[k] = {0, k};
    slots[k] = k;
  }
  if (nbsgd_status r = check_idx(idx, slots, count / kBatch, n_samples)) return r;
  launch_group<false>(mb, count / kBatch, idx, n_samples > 65536, params, data, labels, w, nullptr,
                      losses, d, st);
  return launch_err("nbsgd_mlp_loss");
}
