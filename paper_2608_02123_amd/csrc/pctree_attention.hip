// Tree-masked verification attention of one target layer (paper Sec. 4.2
// and App. A, "Tensor implementation"): the emitted tree is checked in one
// target forward, in which tree node i may attend to the verified prefix, to
// itself and to its ancestors.  Cache slot prefix_len + j holds tree node j,
// so the admitted slots of node i are [0, prefix_len) and prefix_len + j for
// every set bit j < count of its ancestor-mask row.
//
// Layout (bf16): q [R][N][Hq][D], k and v [R][Hkv][C][D], out [R][N][Hq][D];
// query head h reads key/value head h / g, g = Hq / Hkv.
//
// One workgroup takes 128 query rows of one key/value head, row rho = node * g
// + (h mod g), and a run of key slots (the whole admitted range, or one split
// of it when there are too few workgroups to fill the chip).  Its eight waves
// are two groups of four (32 rows each) that take the run's 64-slot chunks in
// turn and join their results at the end, so that two waves share a SIMD and a
// long request's chain of chunks is half as long.  Short runs, and layers of
// many workgroups, have one group: no join, and two workgroups to a compute
// unit (plan_attention).  K and V of a chunk go from
// memory straight into LDS (no registers, no staging instructions), one chunk
// ahead, both row-major with their 16-byte units permuted so that the fragment
// reads touch all banks; V's fragments are read with the transposing LDS read.
// Each wave owns two 16-row column tiles and computes, on bf16 MFMA 16x16x32
// with fp32 accumulation (every K and V fragment read from LDS serves both
// tiles),
//   S^T = K Q^T   (a 32-key x 16-row tile pair, contraction over D), then
//   O^T += V^T P^T (D x 16 rows, contraction over the 32 keys),
// with an online softmax in base 2 (one update per chunk).  The two K tiles of
// a pair take keys {8c..8c+3} and {8c+4..8c+7} on row group c, so that every
// lane ends up with the scores of 8 consecutive keys of its query row: exactly
// the B operand of the second product, with no data movement between lanes.
//
// With few workgroups and a cache of at most kDirectChunks chunks, a second
// kernel gives each of a workgroup's eight waves its own chunks for 16 or 32
// rows, and joins them in LDS; longer caches are split over workgroups, whose
// runs leave (max, sum, unnormalised output) per row in the workspace for a
// merging kernel.  plan_attention chooses.
//
// What bounds the first is instruction issue: staging through registers
// (zeroing, transposing V by 16-bit stores) and the softmax took 460 vector
// instructions per 64 MFMAs, now 250.
#include "pctree.h"

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "pctree_attention.h"
#include "pctree_lds.h"

namespace pctree {
namespace {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

constexpr int kGroupThreads = 256;  // a slot group: 4 waves
constexpr int kColTiles = 2;       // 16-row MFMA column tiles per wave
constexpr int kRowsPerWave = 16 * kColTiles;
constexpr int kRowsPerBlock = 4 * kRowsPerWave;  // query rows of one workgroup
constexpr int kChunk = 64;         // key slots per LDS stage (two 32-slot halves)
constexpr int kMaxSplits = 32;     // slot runs of a layer at most
constexpr int kXcds = 8;           // L2 domains the dispatcher deals workgroups over
constexpr int kMergeThreads = 256;
constexpr int kMergeBatch = 8;     // slot runs whose loads one merge thread issues together
constexpr float kNegInf = -__builtin_inff();

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ float exp2_hw(float x) { return __builtin_amdgcn_exp2f(x); }

// Two floats to packed bf16 (round to nearest even), the low half first.
__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi) {
  bf16x2 v;
  v[0] = (__bf16)lo;
  v[1] = (__bf16)hi;
  return __builtin_bit_cast(uint32_t, v);
}

__device__ __forceinline__ f32x4 mfma_bf16(u32x4 a, u32x4 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a),
                                                  __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

// Permutation of the 16-byte units of a K or V row in LDS (an XOR of the unit
// index).  A K fragment read takes one unit of the 16 rows {0..3, 8..11,
// 16..19, 24..27} (+ 4, + 32); with 256-byte rows all of them start in one
// bank, so the four row bits that vary choose among the 16 units (rows of 128
// bytes alternate between two halves of the banks: three bits choose among
// 8).  A V fragment read takes 32 bytes (two units) of four consecutive keys
// per lane group: pairs of units are permuted by the key's low two bits and
// its bit 3, all that fits the 8 pairs (or two of the three, D = 64).
template <int D>
__device__ __forceinline__ int k_unit(int row) {
  return D == 128 ? (row & 3) | ((row >> 1) & 12) : ((row >> 1) & 1) | ((row >> 2) & 6);
}
template <int D>
__device__ __forceinline__ int v_unit(int row) {
  return D == 128 ? ((row & 3) << 1) | (row & 8) : (row & 2) | ((row >> 1) & 4);
}

// Every vector-memory load of the wave has landed, those into LDS among them.
__device__ __forceinline__ void wait_loads() {
  __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
  __atomic_signal_fence(__ATOMIC_SEQ_CST);
}
// A workgroup barrier for LDS traffic.
__device__ __forceinline__ void lds_barrier() {
  __atomic_signal_fence(__ATOMIC_SEQ_CST);
  __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
  __builtin_amdgcn_s_barrier();
  __atomic_signal_fence(__ATOMIC_SEQ_CST);
}

// Transposing LDS read: in each 16 lanes, lanes 4 i .. 4 i + 3 address row i (16
// consecutive 16-bit values), and lane l receives column l of rows 0 .. 3.
typedef short s16x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ u32x2 read_tr(const uint16_t* src) {
  return __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16(
      (__attribute__((address_space(3))) s16x4*)src));
}

// Low `n` bits set, n in [0, 64].
__device__ __forceinline__ uint64_t low_bits(int n) {
  return n >= 64 ? ~0ull : ((1ull << n) - 1ull);
}

// Admitted key range of request r: [0, prefix + count) clamped to the cache.
struct ReqRange {
  int prefix, cnt, end;
};

__device__ __forceinline__ ReqRange req_range(const AttnArgs& a, int r) {
  ReqRange q;
  q.cnt = min(max(a.count[r], 0), a.N);
  q.prefix = min(max(a.prefix_len[r], 0), a.C);
  q.end = min(q.prefix + q.cnt, a.C);
  return q;
}

// Workgroups are dealt round-robin over the XCDs, each with its own L2.  The
// query blocks of one (request, kv head, slot run) read the same K and V, so
// they are given block ids that land on one XCD: block b serves group
// (b / 8 / qblocks) * 8 + b % 8, query block (b / 8) % qblocks.  Ids past the
// last group return at once.
struct Work {
  int r, kvh, split, qb;
  bool ok;
};

__device__ __forceinline__ Work work_of(const AttnArgs& a, int qblocks, int nsplit) {
  const int b = blockIdx.x;
  const int j = b / kXcds;
  const int grp = (j / qblocks) * kXcds + b % kXcds;
  Work w;
  w.ok = grp < a.R * a.Hkv * nsplit;
  w.qb = j % qblocks;
  w.split = grp % nsplit;
  w.kvh = grp / nsplit % a.Hkv;
  w.r = grp / nsplit / a.Hkv;
  // Longest requests first (up to 64 requests, one per lane): the workgroups
  // that start last, on the compute units that are free first, are then the
  // shortest ones.  (Not where all start at once: the lengths come from memory,
  // and the K and V loads wait for them.)
  if (a.order && w.ok) {
    const int lane = threadIdx.x & 63;
    const int len = lane < a.R ? req_range(a, min(lane, a.R - 1)).end : -1;
    int rank = 0;
    for (int i = 0; i < a.R; ++i) {
      const int o = __builtin_amdgcn_readlane(len, i);
      rank += o > len || (o == len && i < lane);
    }
    w.r = __builtin_ctzll(__ballot(rank == w.r));
  }
  return w;
}

// Maximum over the four lanes that hold one query row (lanes l, l ^ 16,
// l ^ 32, l ^ 48), exchanged on the VALU (v_permlane{16,32}_swap return the
// lane's own value and its partner's, in a lane-dependent order that a
// maximum does not care about).
__device__ __forceinline__ float row_max4(float v) {
  const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false,
                                                   false);
  v = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
  const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false,
                                                   false);
  return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}

// Online softmax of one 16-row column tile over a 64-slot chunk.  s[h][t]
// holds the raw scores q.k of half h, tile t (slots 32 h + 8 grp + 4 t + e);
// `adm` has bit 8 h + i set when slot 32 h + 8 grp + i is admitted (ignored
// when `all`).  The running maximum m is kept in raw units, which
// needs scale > 0: the weights are 2^(scale log2(e) (s - m)).  Writes the
// weights as bf16 B operands bp[h] and returns the factor the accumulated
// output must be scaled by.
__device__ __forceinline__ float softmax_chunk(const f32x4 (&s)[2][2], uint32_t adm, bool all,
                                               float c, float& m, float& l, u32x4 (&bp)[2]) {
  float v[16];
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      v[8 * h + e] = s[h][0][e];
      v[8 * h + 4 + e] = s[h][1][e];
    }
  if (!all) {
#pragma unroll
    for (int i = 0; i < 16; ++i) v[i] = ((adm >> i) & 1u) ? v[i] : kNegInf;
  }
  float cmax = v[0];
#pragma unroll
  for (int i = 1; i < 16; ++i) cmax = fmaxf(cmax, v[i]);
  const float mx = row_max4(cmax);
  float alpha = 1.0f;
  if (__any(mx > m)) {
    const float mn = fmaxf(m, mx);
    alpha = mn == m ? 1.0f : exp2_hw((m - mn) * c);  // m = -inf: 0
    m = mn;
    l *= alpha;
  }
  const float off = m == kNegInf ? 0.0f : m * c;  // nothing admitted yet: every weight 0
  float ps = 0.0f;
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    v[i] = exp2_hw(__builtin_fmaf(v[i], c, -off));
    ps += v[i];
  }
  l += ps;
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int i = 0; i < 4; ++i) bp[h][i] = pack_bf16(v[8 * h + 2 * i], v[8 * h + 2 * i + 1]);
  return alpha;
}

// Admitted slots of the 64-slot chunk at c0 for a node with mask words mw (in
// LDS), as the 16 bits of lane group grp: bits 8 h + i for slot 32 h + 8 grp + i.
__device__ __forceinline__ uint32_t admitted(const AttnArgs& a, const ReqRange& rr,
                                             const uint32_t* mw, int c0, int kend, int grp) {
  const int j0 = c0 - rr.prefix;
  const int wb = j0 >> 5, sh = j0 & 31;  // (floor)
  const uint32_t w0 = wb >= 0 && wb < a.NW ? mw[wb] : 0u;
  const uint32_t w1 = wb + 1 >= 0 && wb + 1 < a.NW ? mw[wb + 1] : 0u;
  const uint32_t w2 = wb + 2 >= 0 && wb + 2 < a.NW ? mw[wb + 2] : 0u;
  const uint64_t lo64 = ((uint64_t)w1 << 32) | w0;
  const uint64_t tree = sh ? (lo64 >> sh) | ((uint64_t)w2 << (64 - sh)) : lo64;
  const int np = min(max(-j0, 0), kChunk);
  const uint64_t win =
      (low_bits(np) | (tree & ~low_bits(np))) & low_bits(min(max(kend - c0, 0), kChunk));
  return ((uint32_t)(win >> (8 * grp)) & 0xffu) | ((uint32_t)(win >> (32 + 8 * grp)) & 0xffu) << 8;
}

template <int D, int G>
__global__ __launch_bounds__(G * kGroupThreads) __attribute__((amdgpu_waves_per_eu(2))) void attn_kernel(AttnArgs a) {
  constexpr int KS = D / 32;   // contraction steps of S = K Q^T
  constexpr int DT = D / 16;   // 16-wide d tiles of O
  constexpr int UPR = D / 8;   // 16-byte units of a K or V row
  constexpr int CT = kColTiles;
  constexpr int TILE = kChunk * D;            // bf16 of a chunk's K (or V)
  constexpr int IPW = kChunk * UPR / 64 / 4;  // load instructions per wave, chunk and tensor
  // [group][buffer][K, V]
  __shared__ __attribute__((aligned(16))) uint16_t sKV[G][2][2][TILE];
  extern __shared__ uint32_t sMask[];     // the nodes' mask rows (mask_bytes)
  __shared__ float2 sML[kRowsPerBlock];  // (two groups) the second group's row statistics
  static_assert(G == 1 || (G == 2 && sizeof(sKV) >= kRowsPerBlock * D * sizeof(float)),
                "the second group's output fits the tiles");

  const Work wk = work_of(a, a.qblocks, a.nsplit);
  if (!wk.ok) return;
  const int r = wk.r, kvh = wk.kvh, split = wk.split;
  const int group = __builtin_amdgcn_readfirstlane(threadIdx.x / kGroupThreads);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x % kGroupThreads / 64);
  const int lane = threadIdx.x & 63;
  const int col = lane & 15, grp = lane >> 4;

  // this lane's query rows (MFMA column col of each tile): rho = node * g + (h mod g)
  const int rows_kv = a.N * a.g;
  const int n0 = wk.qb * kRowsPerBlock / a.g;  // first node of the block
  const int nn = min((wk.qb * kRowsPerBlock + kRowsPerBlock - 1) / a.g - n0 + 1, a.N - n0);
  bool row_in[CT];
  int node[CT], hq[CT];
#pragma unroll
  for (int c = 0; c < CT; ++c) {
    const int rho = wk.qb * kRowsPerBlock + wave * kRowsPerWave + 16 * c + col;
    row_in[c] = rho < rows_kv;
    node[c] = row_in[c] ? rho / a.g : 0;
    hq[c] = kvh * a.g + (row_in[c] ? rho % a.g : 0);
  }

  // Q^T fragments (8 consecutive d of the row per contraction step), issued
  // before the request's lengths are known
  u32x4 bq[CT][KS];
#pragma unroll
  for (int c = 0; c < CT; ++c) {
    const uint16_t* qrow = a.q + (((size_t)r * a.N + node[c]) * a.Hq + hq[c]) * D + grp * 8;
#pragma unroll
    for (int s = 0; s < KS; ++s) bq[c][s] = *(const u32x4*)(qrow + s * 32);
  }

  const ReqRange rr = req_range(a, r);
  // the groups take the run's chunks in turn
  const int kbeg = split * a.split_keys;
  const int kend = min(kbeg + a.split_keys, rr.end);
  if (a.nsplit > 1 && kbeg >= rr.end) return;  // empty run: the merge skips it

  // A chunk's K and V into a buffer: instruction i of the wave fills LDS units
  // 64 (IPW wave + i) ..; the slot's row and the unit it holds there.  Slots
  // past the run repeat its last one (a finite value that weight 0 drops).
  const size_t kvbase = ((size_t)r * a.Hkv + kvh) * a.C * D;
  auto fetch = [&](int c0, int buf) __attribute__((always_inline)) {
    const uint16_t* kb = a.k + kvbase + (size_t)c0 * D;
    const uint16_t* vb = a.v + kvbase + (size_t)c0 * D;
    const int last = kend - 1 - c0;
#pragma unroll
    for (int i = 0; i < IPW; ++i) {
      const int u = (wave * IPW + i) * 64 + lane;
      const int row = u / UPR, pos = u % UPR;
      const uint32_t ro = (uint32_t)min(row, last) * (D * 2);
      load_lds16(kb, ro + (uint32_t)(pos ^ k_unit<D>(row)) * 16,
                 &sKV[group][buf][0][(wave * IPW + i) * 512]);
      load_lds16(vb, ro + (uint32_t)(pos ^ v_unit<D>(row)) * 16,
                 &sKV[group][buf][1][(wave * IPW + i) * 512]);
    }
  };
  const int kfirst = kbeg + group * kChunk;
  if (kfirst < kend) fetch(kfirst, 0);

  // the mask rows of the block's nodes (bit j of a row is tree node j, at slot
  // prefix + j)
  const uint32_t* mrow_g = a.mask + ((size_t)r * a.N + n0) * a.NW;
  for (int i = threadIdx.x; i < nn * a.NW; i += G * kGroupThreads) sMask[i] = mrow_g[i];

  bool row_live[CT];
#pragma unroll
  for (int c = 0; c < CT; ++c) {
    row_live[c] = row_in[c] && node[c] < rr.cnt;
    if (!row_live[c]) {
#pragma unroll
      for (int s = 0; s < KS; ++s) bq[c][s] = u32x4{0u, 0u, 0u, 0u};
    }
  }

  f32x4 o[CT][DT];
  float m[CT], l[CT];
#pragma unroll
  for (int c = 0; c < CT; ++c) {
    m[c] = kNegInf;
    l[c] = 0.0f;
#pragma unroll
    for (int t = 0; t < DT; ++t) o[c][t] = f32x4{0.f, 0.f, 0.f, 0.f};
  }

  // A-operand rows of an S^T tile pair: tile 0 holds keys 8c + e, tile 1 keys
  // 8c + 4 + e, for MFMA row 4c + e (c = col / 4, e = col % 4)
  const int krow0 = 8 * (col >> 2) + (col & 3);

  // (the step's base chunk is the first group's; the second may have one less)
  int buf = 0;
  for (int cb = kbeg; cb < kend; cb += G * kChunk, buf ^= 1) {
    const int c0 = cb + group * kChunk;
    wait_loads();
    lds_barrier();  // the chunk is complete; the other buffer is no longer read
    if (c0 >= kend) break;  // (the last step: no barrier of the loop follows)
    if (c0 + G * kChunk < kend) fetch(c0 + G * kChunk, buf ^ 1);
    const uint16_t* sK = sKV[group][buf][0];
    const uint16_t* sV = sKV[group][buf][1];
    // every slot of the chunk admitted for every live row: no masking (rows
    // past the tree then take weights like the rest and are written as zeros)
    const bool full = c0 + kChunk <= min(kend, rr.prefix);

    // S^T for both halves and both column tiles: 8 independent chains
    f32x4 sacc[CT][2][2];
#pragma unroll
    for (int c = 0; c < CT; ++c)
#pragma unroll
      for (int h = 0; h < 2; ++h) sacc[c][h][0] = sacc[c][h][1] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int k = 0; k < KS; ++k) {
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        // (rows 4 and 32 apart share their permutation)
        const uint16_t* kr = sK + (32 * h + krow0) * D + ((4 * k + grp) ^ k_unit<D>(krow0)) * 8;
        const u32x4 a0 = *(const u32x4*)kr;
        const u32x4 a1 = *(const u32x4*)(kr + 4 * D);
#pragma unroll
        for (int c = 0; c < CT; ++c) {
          sacc[c][h][0] = mfma_bf16(a0, bq[c][k], sacc[c][h][0]);
          sacc[c][h][1] = mfma_bf16(a1, bq[c][k], sacc[c][h][1]);
        }
      }
    }
    u32x4 bp[CT][2];
#pragma unroll
    for (int c = 0; c < CT; ++c) {
      const uint32_t adm =
          !full && row_live[c]
              ? admitted(a, rr, sMask + (node[c] - n0) * a.NW, c0, kend, grp)
              : 0u;
      const float alpha =
          softmax_chunk(sacc[c], adm, full, a.scale_log2, m[c], l[c], bp[c]);
      if (__any(alpha != 1.0f)) {
#pragma unroll
        for (int t = 0; t < DT; ++t) o[c][t] *= alpha;
      }
    }
    // O^T += V^T P^T: lane (d = col, keys 8 grp .. + 7 of the half) from two
    // transposing reads of four keys each
    const int vkey = 8 * grp + (col >> 2);  // the key this lane addresses (of the first four)
#pragma unroll
    for (int t = 0; t < DT; ++t) {
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const uint16_t* vr = sV + (32 * h + vkey) * D +
                             ((2 * t + ((col >> 1) & 1)) ^ v_unit<D>(vkey)) * 8 + (col & 1) * 4;
        const u32x2 lo = read_tr(vr), hi = read_tr(vr + 4 * D);
        const u32x4 av = {lo[0], lo[1], hi[0], hi[1]};
#pragma unroll
        for (int c = 0; c < CT; ++c) o[c][t] = mfma_bf16(av, bp[c][h], o[c][t]);
      }
    }
  }

  // the row's sum over its four lane groups
#pragma unroll
  for (int c = 0; c < CT; ++c) {
    l[c] += __shfl_xor(l[c], 16, 64);
    l[c] += __shfl_xor(l[c], 32, 64);
  }
  // the second group's (max, sum, output) joins the first's, through the
  // tiles' place in LDS
  f32x4* sO = (f32x4*)sKV;
  if constexpr (G == 2) {
    lds_barrier();
    if (group == 1) {
#pragma unroll
      for (int c = 0; c < CT; ++c) {
#pragma unroll
        for (int t = 0; t < DT; ++t) sO[((wave * CT + c) * DT + t) * 64 + lane] = o[c][t];
        if (grp == 0) sML[wave * kRowsPerWave + 16 * c + col] = make_float2(m[c], l[c]);
      }
    }
    lds_barrier();
    if (group == 1) return;
  }
#pragma unroll
  for (int c = 0; c < CT; ++c) {
    float lc = l[c];
    if constexpr (G == 2) {
      const float2 ml = sML[wave * kRowsPerWave + 16 * c + col];
      const float mn = fmaxf(m[c], ml.x);
      const float w0 = m[c] == mn ? 1.0f : exp2_hw((m[c] - mn) * a.scale_log2);
      const float w1 = ml.x == mn ? 1.0f : exp2_hw((ml.x - mn) * a.scale_log2);
      m[c] = mn;  // (both -inf, no admitted slot: weights 1 on zeros)
      lc = l[c] * w0 + ml.y * w1;
#pragma unroll
      for (int t = 0; t < DT; ++t)
        o[c][t] = o[c][t] * w0 + sO[((wave * CT + c) * DT + t) * 64 + lane] * w1;
    }
    if (!row_in[c]) continue;
    const size_t qidx = ((size_t)r * a.N + node[c]) * a.Hq + hq[c];  // (request, node, head)
    if (a.nsplit == 1) {
      const float inv = row_live[c] && lc > 0.0f ? 1.0f / lc : 0.0f;
      uint16_t* orow = a.out + qidx * D;
#pragma unroll
      for (int t = 0; t < DT; ++t) {
        const f32x4 v = o[c][t] * inv;
        u32x2 w;
        w[0] = pack_bf16(v[0], v[1]);
        w[1] = pack_bf16(v[2], v[3]);
        *(u32x2*)(orow + t * 16 + 4 * grp) = w;
      }
    } else {
      const size_t prow = (size_t)split * a.R * a.N * a.Hq + qidx;
      float* po = a.part_o + prow * D;
#pragma unroll
      for (int t = 0; t < DT; ++t) *(f32x4*)(po + t * 16 + 4 * grp) = o[c][t];
      if (grp == 0) {
        a.part_ml[2 * prow] = row_live[c] ? m[c] : kNegInf;
        a.part_ml[2 * prow + 1] = row_live[c] ? lc : 0.0f;
      }
    }
  }
}

// Few workgroups, short caches: 16 CT rows of one (request, kv head) per
// workgroup; wave w takes the chunks w, w + 8, ... on its own (K fragments
// straight from memory into registers, V through its own LDS tile) and the
// eight waves' results are joined in LDS, so that nothing goes through the
// workspace and no second launch follows (which took 4 of the 15 us of a
// one-request layer; its partials were twice the layer's own bytes).
constexpr int kDirectWaves = 8;
constexpr int kDirectChunks = 24;  // (three chunks per wave)

template <int D, int CT>
__global__ __launch_bounds__(kDirectWaves * 64) void attn_direct_kernel(AttnArgs a, int qblocks) {
  constexpr int KS = D / 32, DT = D / 16, UPR = D / 8;
  constexpr int ROWS = 16 * CT;
  constexpr int TILE = kChunk * D;              // bf16 of a chunk's V
  constexpr int INS = kChunk * UPR / 64;        // load instructions of a chunk's V
  constexpr int PART = CT * DT * 64;            // f32x4 of a wave's output
  __shared__ __attribute__((aligned(16))) uint16_t sV[kDirectWaves][TILE];
  __shared__ uint32_t sMask[ROWS * (PCTREE_MAX_MASK_BUDGET / 32)];
  __shared__ float2 sML[kDirectWaves][ROWS];
  static_assert(sizeof(uint16_t) * TILE >= PART * sizeof(f32x4), "a wave's output fits its V tile");

  const Work wk = work_of(a, qblocks, 1);
  if (!wk.ok) return;
  const int r = wk.r, kvh = wk.kvh;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64), lane = threadIdx.x & 63;
  const int col = lane & 15, grp = lane >> 4;
  const int rows_kv = a.N * a.g;
  const int n0 = wk.qb * ROWS / a.g;
  const int nn = min((wk.qb * ROWS + ROWS - 1) / a.g - n0 + 1, a.N - n0);
  bool row_in[CT];
  int node[CT], hq[CT];
  u32x4 bq[CT][KS];
#pragma unroll
  for (int c = 0; c < CT; ++c) {
    const int rho = wk.qb * ROWS + 16 * c + col;
    row_in[c] = rho < rows_kv;
    node[c] = row_in[c] ? rho / a.g : 0;
    hq[c] = kvh * a.g + (row_in[c] ? rho % a.g : 0);
    const uint16_t* qrow = a.q + (((size_t)r * a.N + node[c]) * a.Hq + hq[c]) * D + grp * 8;
#pragma unroll
    for (int s = 0; s < KS; ++s) bq[c][s] = *(const u32x4*)(qrow + s * 32);
  }
  const ReqRange rr = req_range(a, r);
  const int kend = rr.end;
  const size_t kvbase = ((size_t)r * a.Hkv + kvh) * a.C * D;
  const uint32_t* mrow_g = a.mask + ((size_t)r * a.N + n0) * a.NW;
  for (int i = threadIdx.x; i < nn * a.NW; i += kDirectWaves * 64) sMask[i] = mrow_g[i];
  bool row_live[CT];
  f32x4 o[CT][DT];
  float m[CT], l[CT];
#pragma unroll
  for (int c = 0; c < CT; ++c) {
    row_live[c] = row_in[c] && node[c] < rr.cnt;
    if (!row_live[c]) {
#pragma unroll
      for (int s = 0; s < KS; ++s) bq[c][s] = u32x4{0u, 0u, 0u, 0u};
    }
    m[c] = kNegInf;
    l[c] = 0.0f;
#pragma unroll
    for (int t = 0; t < DT; ++t) o[c][t] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  lds_barrier();  // the mask rows
  const int krow0 = 8 * (col >> 2) + (col & 3);
  const int vkey = 8 * grp + (col >> 2);
  for (int c0 = wave * kChunk; c0 < kend; c0 += kDirectWaves * kChunk) {
    // (slots past the range repeat its last one, which weight 0 drops)
    const int last = kend - 1 - c0;
    const uint16_t* kb = a.k + kvbase + (size_t)c0 * D;
    const uint16_t* vb = a.v + kvbase + (size_t)c0 * D;
#pragma unroll
    for (int i = 0; i < INS; ++i) {
      const int u = i * 64 + lane, row = u / UPR, pos = u % UPR;
      load_lds16(vb, (uint32_t)min(row, last) * (D * 2) + (uint32_t)(pos ^ v_unit<D>(row)) * 16,
                 &sV[wave][i * 512]);
    }
    u32x4 kf[2][2][KS];
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        const uint16_t* kr = kb + (size_t)min(32 * h + krow0 + 4 * t, last) * D + grp * 8;
#pragma unroll
        for (int k = 0; k < KS; ++k) kf[h][t][k] = *(const u32x4*)(kr + 32 * k);
      }
    f32x4 sacc[CT][2][2];
#pragma unroll
    for (int c = 0; c < CT; ++c)
#pragma unroll
      for (int h = 0; h < 2; ++h) sacc[c][h][0] = sacc[c][h][1] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int k = 0; k < KS; ++k)
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int c = 0; c < CT; ++c) {
          sacc[c][h][0] = mfma_bf16(kf[h][0][k], bq[c][k], sacc[c][h][0]);
          sacc[c][h][1] = mfma_bf16(kf[h][1][k], bq[c][k], sacc[c][h][1]);
        }
    const bool full = c0 + kChunk <= min(kend, rr.prefix);
    u32x4 bp[CT][2];
#pragma unroll
    for (int c = 0; c < CT; ++c) {
      const uint32_t adm = !full && row_live[c]
                               ? admitted(a, rr, sMask + (node[c] - n0) * a.NW, c0, kend, grp)
                               : 0u;
      const float alpha = softmax_chunk(sacc[c], adm, full, a.scale_log2, m[c], l[c], bp[c]);
      if (__any(alpha != 1.0f)) {
#pragma unroll
        for (int t = 0; t < DT; ++t) o[c][t] *= alpha;
      }
    }
    wait_loads();
#pragma unroll
    for (int t = 0; t < DT; ++t)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const uint16_t* vr = sV[wave] + (32 * h + vkey) * D +
                             ((2 * t + ((col >> 1) & 1)) ^ v_unit<D>(vkey)) * 8 + (col & 1) * 4;
        const u32x2 lo = read_tr(vr), hi = read_tr(vr + 4 * D);
        const u32x4 av = {lo[0], lo[1], hi[0], hi[1]};
#pragma unroll
        for (int c = 0; c < CT; ++c) o[c][t] = mfma_bf16(av, bp[c][h], o[c][t]);
      }
    // (the tile's reads are back before the next chunk's loads overwrite it)
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
    __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
  }
  // the waves' results, each in its own V tile's place
  f32x4* sO = (f32x4*)sV[wave];
#pragma unroll
  for (int c = 0; c < CT; ++c) {
    l[c] += __shfl_xor(l[c], 16, 64);
    l[c] += __shfl_xor(l[c], 32, 64);
    if (grp == 0) sML[wave][16 * c + col] = make_float2(m[c], l[c]);
#pragma unroll
    for (int t = 0; t < DT; ++t) sO[(c * DT + t) * 64 + lane] = o[c][t];
  }
  lds_barrier();
  for (int e = threadIdx.x; e < PART; e += kDirectWaves * 64) {
    const int ct = e / 64, c = ct / DT, t = ct % DT;  // (e % 64 == lane)
    const int rho = wk.qb * ROWS + 16 * c + col;
    if (rho >= rows_kv) continue;
    float M = kNegInf;
    float2 ml[kDirectWaves];
#pragma unroll
    for (int w = 0; w < kDirectWaves; ++w) {
      ml[w] = sML[w][16 * c + col];
      M = fmaxf(M, ml[w].x);
    }
    float L = 0.0f;
    f32x4 O = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < kDirectWaves; ++w) {
      const float wt = ml[w].x == kNegInf ? 0.0f : exp2_hw((ml[w].x - M) * a.scale_log2);
      L += wt * ml[w].y;
      O += ((const f32x4*)sV[w])[e] * wt;
    }
    const int nd = rho / a.g;
    const float inv = nd < rr.cnt && L > 0.0f ? 1.0f / L : 0.0f;
    u32x2 wv;
    wv[0] = pack_bf16(O[0] * inv, O[1] * inv);
    wv[1] = pack_bf16(O[2] * inv, O[3] * inv);
    *(u32x2*)(a.out + (((size_t)r * a.N + nd) * a.Hq + kvh * a.g + rho % a.g) * D + t * 16 +
              4 * grp) = wv;
  }
}

// Merge of the slot runs: D / 4 threads per row of (request, node, head), 4
// consecutive d each.  Only the runs that hold admitted slots were written.
// The runs are read in batches of kMergeBatch whose loads are all issued
// before any is used (clamped to a written run), folded into a running
// (max, sum, output) per batch.
template <int D>
__global__ __launch_bounds__(kMergeThreads) void attn_merge_kernel(AttnArgs a) {
  constexpr int TPR = D / 4;                // threads per row
  constexpr int RPB = kMergeThreads / TPR;  // rows per workgroup
  const size_t rows = (size_t)a.R * a.N * a.Hq;
  const size_t qidx = (size_t)blockIdx.x * RPB + threadIdx.x / TPR;
  const int d = (threadIdx.x % TPR) * 4;
  if (qidx >= rows) return;
  const int r = (int)(qidx / ((size_t)a.N * a.Hq));
  const int node = (int)(qidx / a.Hq % a.N);
  const ReqRange rr = req_range(a, r);
  const int ns = node < rr.cnt ? min(a.nsplit, (rr.end + a.split_keys - 1) / a.split_keys) : 0;
  float M = kNegInf, L = 0.0f;
  f32x4 O = {0.f, 0.f, 0.f, 0.f};
  for (int s0 = 0; s0 < ns; s0 += kMergeBatch) {
    float ms[kMergeBatch], ls[kMergeBatch];
    f32x4 os[kMergeBatch];
#pragma unroll
    for (int i = 0; i < kMergeBatch; ++i) {
      const size_t prow = (size_t)min(s0 + i, ns - 1) * rows + qidx;
      ms[i] = a.part_ml[2 * prow];
      ls[i] = a.part_ml[2 * prow + 1];
      os[i] = *(const f32x4*)(a.part_o + prow * D + d);
    }
    float bm = kNegInf;
#pragma unroll
    for (int i = 0; i < kMergeBatch; ++i)
      if (s0 + i < ns) bm = fmaxf(bm, ms[i]);
    const float Mn = fmaxf(M, bm);
    if (Mn == kNegInf) continue;  // no admitted slot so far
    const float sc = M == kNegInf ? 0.0f : exp2_hw((M - Mn) * a.scale_log2);
    L *= sc;
    O *= sc;
#pragma unroll
    for (int i = 0; i < kMergeBatch; ++i) {
      // a run with no admitted slot of this row (max -inf) adds nothing
      if (s0 + i < ns && ms[i] != kNegInf) {
        const float w = exp2_hw((ms[i] - Mn) * a.scale_log2);  // maxima in raw units
        L += w * ls[i];
        O += os[i] * w;
      }
    }
    M = Mn;
  }
  const float inv = L > 0.0f ? 1.0f / L : 0.0f;
  u32x2 w;
  w[0] = pack_bf16(O[0] * inv, O[1] * inv);
  w[1] = pack_bf16(O[2] * inv, O[3] * inv);
  *(u32x2*)(a.out + qidx * D + d) = w;
}

}  // namespace

AttnPlan plan_attention(int R, int N, int Hq, int Hkv, int D, int C, int cus) {
  AttnPlan p;
  const int g = Hq / Hkv;
  p.qblocks = (N * g + kRowsPerBlock - 1) / kRowsPerBlock;
  const long long base = (long long)R * Hkv * p.qblocks;
  const int chunks = (C + kChunk - 1) / kChunk;
  // enough workgroups for one per two compute units (more runs cost more in
  // the merge pass than they save here)
  int ns = 1;
  const int target = cus / 2;
  if (base < target) ns = (int)((target + base - 1) / base);
  ns = ns < chunks ? ns : chunks;
  ns = ns < kMaxSplits ? ns : kMaxSplits;
  ns = ns < 1 ? 1 : ns;
  const int per = (chunks + ns - 1) / ns;  // chunks per run
  p.split_keys = per * kChunk;
  p.nsplit = (chunks + per - 1) / per;
  const size_t rows = (size_t)R * N * Hq;
  p.ws_bytes = p.nsplit > 1 ? (size_t)p.nsplit * rows * (D + 2) * sizeof(float) + 256 : 0;

  // The kernel, by measurements over 1400 shapes (heads of 64 and 128, 16 to 128
  // nodes, 1 to 8 requests, caches of 80 to 1628 slots); times in us, heads of
  // 128 unless said otherwise.
  //  * Direct: layers that would be split (fewer than 128 workgroups of 128
  //    rows) while each wave has at most three chunks and all workgroups fit one
  //    to a compute unit, with 16 rows each or else 32; with one chunk per wave
  //    also at more.  Direct / split: up to 8 chunks 9.5 / 14, 9 to 16 10.4 /
  //    15.5, 17 to 20 12.6 / 17.  Past 20 chunks runs of at most 4 chunks are
  //    faster (17.8 / 16.4 at 96 workgroups of 16 rows, 24 chunks), but not with
  //    heads of 64 (11 / 13.5).
  //  * One group: runs of at most three chunks (10.2 / 10.6 at two, 11.7 / 12.3
  //    at three, 14.1 / 13.6 at four: a second group then mostly adds the join).
  //    Also with more workgroups than compute units, two of which fit a unit:
  //    up to twice as many, the second group's shorter chains win from 12 to 18
  //    chunks on (320 workgroups: 19.8 / 26.9 at 5 chunks, 28.2 / 31.9 at 12,
  //    36.5 / 36.9 at 18, 58 / 50 at 34; heads of 64: 20.5 / 21.9 at 12, 26.5 /
  //    25.2 at 18); beyond that one group always does (640: 49.8 / 57.8 at 18,
  //    121 / 122 at 66).
  const int q16 = (N * g + 15) / 16, q32 = (N * g + 31) / 32;
  const long long heads = (long long)R * Hkv;
  const bool short_runs = D == 128 && chunks > 20 && per <= 4;
  if (p.nsplit > 1 && chunks <= kDirectChunks && !short_runs && heads * q16 <= cus)
    p.kernel = kAttnDirect16;
  else if (p.nsplit > 1 && chunks <= kDirectChunks && !short_runs &&
           (heads * q32 <= cus || chunks <= kDirectWaves))
    p.kernel = kAttnDirect32;
  else
    p.kernel = per <= 3 || (base > cus && chunks <= 12) || base > 2 * cus ? kAttnOneGroup
                                                                       : kAttnTwoGroups;

  // blocks: groups of workgroups that share K and V, padded to whole XCD rounds
  const bool direct = p.kernel == kAttnDirect16 || p.kernel == kAttnDirect32;
  const int qb = p.kernel == kAttnDirect16 ? q16 : (p.kernel == kAttnDirect32 ? q32 : p.qblocks);
  const long long groups = heads * (direct ? 1 : p.nsplit);
  p.blocks = (int)(((groups + kXcds - 1) / kXcds) * kXcds * qb);
  // (an XCD has an eighth of the units and the padded blocks)
  p.order = R > 1 && R <= 64 && p.blocks > cus;
  return p;
}

namespace {

// The mask rows of a workgroup's nodes: 128 rows touch at most 127 / g + 2 nodes.
unsigned mask_bytes(const AttnArgs& a) {
  const int nodes = (kRowsPerBlock - 1) / a.g + 2;
  return (unsigned)((nodes < a.N ? nodes : a.N) * a.NW * sizeof(uint32_t));
}

template <int D>
hipError_t launch(const AttnArgs& a, const AttnPlan& p, hipStream_t stream) {
  const int rows = a.N * a.g;
  switch (p.kernel) {
    case kAttnDirect16:
      attn_direct_kernel<D, 1><<<p.blocks, kDirectWaves * 64, 0, stream>>>(a, (rows + 15) / 16);
      return hipGetLastError();
    case kAttnDirect32:
      attn_direct_kernel<D, 2><<<p.blocks, kDirectWaves * 64, 0, stream>>>(a, (rows + 31) / 32);
      return hipGetLastError();
    case kAttnOneGroup:
      attn_kernel<D, 1><<<p.blocks, kGroupThreads, mask_bytes(a), stream>>>(a);
      break;
    case kAttnTwoGroups:
      attn_kernel<D, 2><<<p.blocks, 2 * kGroupThreads, mask_bytes(a), stream>>>(a);
      break;
  }
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess || a.nsplit == 1) return e;
  const size_t out_rows = (size_t)a.R * a.N * a.Hq;
  const int rpb = kMergeThreads / (D / 4);
  attn_merge_kernel<D><<<(unsigned)((out_rows + rpb - 1) / rpb), kMergeThreads, 0, stream>>>(a);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_attention(const AttnArgs& a, const AttnPlan& plan, int D, hipStream_t stream) {
  return D == 128 ? launch<128>(a, plan, stream) : launch<64>(a, plan, stream);
}

}  // namespace pctree
