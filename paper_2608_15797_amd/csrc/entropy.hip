// Full-vocabulary token entropy (Eq. (4)) with the moving-average
// degeneration detector (Sec. 3.2, implementation details), gfx950.
//
// One pass over the logits. Each thread keeps an online triple in the log2
// domain: m = running max of y = inv_temp * x * log2(e), Z = sum 2^(y - m) and
// S = sum (y - m) 2^(y - m), rescaled when m grows. Since the natural-log
// entropy is H = ln Z - (sum (x' - m') e^(x' - m')) / Z with x' the scaled
// logits, in log2 units H = ln2 * (log2 Z - S / Z). Triples merge
// associatively, first across a wave with shuffles, then across the
// workgroup's waves. When a row is split over several workgroups (so that a
// few long rows still fill the chip), each writes its triple to the workspace
// and a second, tiny kernel merges them per row and runs the detector. A
// kernel boundary orders the two: merging inside the first kernel would need
// device-scope fences, which on this chip write back and invalidate the
// per-XCD L2 caches in every workgroup.
//
// Loads are buffer loads from a per-split resource (16 bytes per lane; lanes
// past the split's range return zero without touching memory), issued U at a
// time before any arithmetic, with invalid values masked by selects rather
// than branches.
//
// Fused sampler (temperature, top-k, top-p; Sec. 4.1 decoding setup) in the
// same pass. Candidates are 64-bit keys (an order-preserving map of the raw
// logit's bits above the complemented token id, so a larger key is a larger
// logit and, among equal logits, a lower id). A split that fits in registers
// takes its threshold from its lanes' maxima (sample_split). A longer one
// streams with a candidate buffer per wave: a candidate must beat the wave's
// threshold, the k-th best key at its last compaction (seeded, in the first
// round, with the k-th largest of the lanes' maxima, which bounds the wave's
// k-th best logit from below); when the buffer would overflow, the wave keeps
// at most 128 of its best and raises the threshold. Thresholds are found bit
// by bit from the top with ballot counts only (compare, ballot, popcount; no
// cross-lane data movement), stopping as soon as the kept count fits. Each
// split ends with its k best keys in the workspace; the per-row merge takes
// the k best of all splits, forms the temperature softmax over them, cuts the
// nucleus at top_p and draws with a Philox4x64-10 uniform (counter (step, row,
// 0, 0), key (seed, 0), top 24 bits of the first word).
#include <hip/hip_runtime.h>

#include <atomic>

#include "entropy_common.h"
#include "sampler_common.h"
#include "kvr_device.h"
#include "kvr_internal.h"

namespace kvr {

// Split partials of the allocation-free entropy entry point: one file-scope
// device array per GPU, held until the process ends. Host code never uses
// its name as an address; it uses the per-device pointer from
// entropy_scratch() below.
__device__ __align__(256) unsigned char scratch[kEntropyScratchBytes];

namespace {

constexpr int kThreads = 256;
constexpr int kU = 10;                      // 8-logit vectors per thread per round (entropy alone)
constexpr int kRoundVecs = kU * kThreads;   // vectors per workgroup per round
// Whole-row workgroups: when a call has at least one row per CU and long
// rows, each row gets one workgroup of kRowThreads threads that reduces it
// completely (entropy and detector in the same kernel, no split partials
// and no merge launch).
constexpr int kRowThreads = 1024;
constexpr int kRowMinRows = 256;
constexpr int kRowMinVecs = 8 * kRowThreads;

// One workgroup of NT threads per (split, global row of the batch).
// VEC = true: 16-byte loads of 8 elements (row starts 16-byte aligned).
// SAMPLE = true: also collect the split's top_k candidates (always writes
// the split's partials, even unsplit rows, for the sampling merge).
template <typename T, bool VEC, bool SAMPLE, int NT = kThreads>
__global__ __launch_bounds__(NT) void entropy_kernel(EntropyBatch b) {
  __shared__ Tri part[NT / kWave];
  __shared__ uint64_t cand[SAMPLE ? (NT / kWave) * kCandCap : 1];
  __shared__ int cand_n[NT / kWave];
  const int bset = batch_set(b, blockIdx.y);
  const EntropyParams &p = b.set[bset];
  const int row = blockIdx.y - b.row0[bset];
  const int split = blockIdx.x;
  const int splits = gridDim.x;
  const int tid = threadIdx.x;
  const int lane = tid % kWave;
  const int wave = tid / kWave;
  const T *x = static_cast<const T *>(p.logits) + (size_t)row * p.ld;
  const float c = p.inv_temp * kLog2e;
  Cands cs{cand + (SAMPLE ? wave * kCandCap : 0), 0, 1, kNegInf};

  Tri t{kNegInf, 0.f, 0.f};
  if constexpr (VEC) {
    // U vectors of 8 logits per thread per round, all loads issued first and
    // each vector folded as soon as it has arrived, so the arithmetic of the
    // round overlaps its later loads. Entropy alone: 10, so that a split of
    // the 7B / 1.5B vocabularies over 8 workgroups per row is one round. With
    // the sampler: 8, whose lower register count keeps 4 waves per SIMD.
    // Whole-row workgroups keep 10 (20, one round over a 152k bf16 row,
    // measured 3% slower).
    constexpr int U = SAMPLE ? 8 : kU;
    const int nvec = p.V / 8;
    const int per = (nvec + splits - 1) / splits;
    const int v0 = split * per;
    const int v1 = min(v0 + per, nvec);
    // The resource ends where this split's vectors end, so the lanes of a
    // partly used round load nothing instead of fetching the next split.
    const rsrc_t rr = row_rsrc(x, (uint32_t)v1 * 8u * (uint32_t)sizeof(T));
    // The loop bound is the same for every thread (lanes past the end load
    // zeros and skip them), so waves offer sampler candidates in lockstep.
    for (int b0 = v0; b0 < v1; b0 += U * NT) {
      const int base = b0 + tid;
      const bool full = b0 + U * NT <= v1;
      // The loads are issued in vector order (the scheduling barriers keep
      // the compiler from reordering them), so that each fold below waits
      // only for its own vector; the asm statement keeps a load whose value
      // is used under a branch from sinking into it.
      Vec8<T> w[U];
#pragma unroll
      for (int u = 0; u < U; u++) {
        w[u].load(rr, base + u * NT);
        __builtin_amdgcn_sched_barrier(0);
      }
      asm volatile("" ::: "memory");
      if constexpr (SAMPLE) {
        if (b0 == v0) {
          // First round: seed the thresholds from the lanes' maxima.
          float mx = kNegInf;
#pragma unroll
          for (int u = 0; u < U; u++) {
            float a[8];
            w[u].get(a);
            if (base + u * NT < v1)
#pragma unroll
              for (int e = 0; e < 8; e++) mx = vmax(mx, a[e]);
          }
          cand_seed(cs, mx, p.top_k);
        }
      }
#pragma unroll
      for (int u = 0; u < U; u++) {
        float a[8];
        w[u].get(a);
        const int v = base + u * NT;
        const bool ok = full || v < v1;
        if constexpr (SAMPLE) cand_offer(cs, p.top_k, lane, a, (uint32_t)v * 8u, ok ? 8 : 0);
        if (ok) tri_fold8(t, a, c);
      }
    }
    if (split == splits - 1) {
      // The V % 8 trailing logits (one per thread of the first wave).
      const int e = nvec * 8 + tid;
      float a[8] = {kNegInf, kNegInf, kNegInf, kNegInf, kNegInf, kNegInf, kNegInf, kNegInf};
      const bool has = e < p.V;
      if (has) a[0] = load1(x + e);
      if constexpr (SAMPLE) {
        if (wave == 0) cand_offer(cs, p.top_k, lane, a, (uint32_t)e, has ? 1 : 0);
      }
      if (has) {
        float b[1] = {a[0] * c};
        tri_add<1>(t, b);
      }
    }
  } else {
    const int per = (p.V + splits - 1) / splits;
    const int e0 = split * per;
    const int e1 = min(e0 + per, p.V);
    // Every thread runs the same number of iterations so that whole waves
    // offer candidates together.
    for (int eb = e0; eb < e1; eb += NT) {
      const int e = eb + tid;
      const bool has = e < e1;
      float a[8] = {kNegInf, kNegInf, kNegInf, kNegInf, kNegInf, kNegInf, kNegInf, kNegInf};
      if (has) a[0] = load1(x + e);
      if constexpr (SAMPLE) cand_offer(cs, p.top_k, lane, a, (uint32_t)e, has ? 1 : 0);
      if (has) {
        float b[1] = {a[0] * c};
        tri_add<1>(t, b);
      }
    }
  }

  t = wave_merge(t);
  if (lane == 0) part[wave] = t;
  if constexpr (SAMPLE) {
    if (cs.cnt > p.top_k) cand_reduce_any(cs, p.top_k, p.top_k, lane);  // exactly the k best
    if (lane == 0) cand_n[wave] = cs.cnt;
  }
  __syncthreads();
  if constexpr (SAMPLE) {
    // First wave: the k best of the waves' lists go to the workspace.
    if (wave != 0) return;
    constexpr int NW = NT / kWave;
    int off[NW + 1];
    off[0] = 0;
#pragma unroll
    for (int w = 0; w < NW; w++) off[w + 1] = off[w] + cand_n[w];
    uint64_t *keys = reinterpret_cast<uint64_t *>(static_cast<float *>(p.ws) + (size_t)p.R * splits * 4) +
                     ((size_t)row * splits + split) * p.top_k;
    int nw;
    if (off[NW] <= kWave) nw = gather_select<1, NW>(cand, off, p.top_k, lane, keys);
    else if (off[NW] <= 2 * kWave) nw = gather_select<2, NW>(cand, off, p.top_k, lane, keys);
    else nw = gather_select<NW * kTopKMax / kWave, NW>(cand, off, p.top_k, lane, keys);
    for (int q = nw + lane; q < p.top_k; q += kWave) keys[q] = 0;
    if (lane == 0) {
      Tri r = part[0];
#pragma unroll
      for (int w = 1; w < NW; w++) r = tri_merge(r, part[w]);
      reinterpret_cast<float4 *>(p.ws)[(size_t)row * splits + split] = make_float4(r.m, r.z, r.s, 0.f);
    }
    return;
  } else {
    if (wave != 0) return;
    Tri r = part[0];
#pragma unroll
    for (int w = 1; w < NT / kWave; w++) r = tri_merge(r, part[w]);
    if (splits == 1) {
      const float H = finish_entropy(r);
      if (lane == 0) p.H[row] = H;
      detector_push(p, row, H, lane);
      return;
    }
    if (lane == 0)
      reinterpret_cast<float4 *>(p.ws)[(size_t)row * splits + split] = make_float4(r.m, r.z, r.s, 0.f);
  }
}

// The merged triple of a row's split partials ([splits] float4 (m, Z, S, -)
// in the workspace), by one whole wave: each lane loads every 64th partial,
// so the row costs one memory round trip.
__device__ __forceinline__ Tri wave_merge_splits(const EntropyParams &p, int row, int lane) {
  const float4 *q = reinterpret_cast<const float4 *>(p.ws) + (size_t)row * p.splits;
  Tri acc{kNegInf, 0.f, 0.f};
  for (int k = lane; k < p.splits; k += kWave) {
    const float4 v = q[k];
    acc = tri_merge(acc, Tri{v.x, v.y, v.z});
  }
  return wave_merge(acc);
}

// Per-row merge of the split partials, then the detector; one wave per
// global row of the batch.
__global__ __launch_bounds__(kWave) void entropy_merge(EntropyBatch b) {
  const int bset = batch_set(b, blockIdx.x);
  const EntropyParams &p = b.set[bset];
  const int row = blockIdx.x - b.row0[bset];
  const int lane = threadIdx.x;
  const float H = finish_entropy(wave_merge_splits(p, row, lane));
  if (lane == 0) p.H[row] = H;
  detector_push(p, row, H, lane);
}

// One split of a row with the sampler, all of its logits in registers at once
// (at most kRoundVecs vectors; sample_splits gives at least that many splits
// where the merge can take their candidates). A workgroup folds its vectors
// as they arrive, keeping each one's largest logit; the k-th largest of the
// 256 lanes' maxima (16 leading bits of it) then bounds the split's k-th best
// from below, so about k logits of the whole workgroup are candidates and most
// vectors are passed over by one compare. The candidates (in any order) are
// ranked by counting and the k best stored sorted. Rows with more than a
// candidate per thread (many equal logits, say) take the per-wave buffers of
// entropy_kernel, from the same registers.
// Bound by the entropy's arithmetic and the latency of the steps after the
// loads. 128 rows of 152064 bf16 logits: 16.4 us, against 27.2 us with
// entropy_kernel's per-wave buffers; four waves per SIMD (all 1024 workgroups
// at once) against three take 4 us off.
template <typename T>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(4))) void sample_split(EntropyParams p) {
  constexpr int U = kU, NT = kThreads, NW = NT / kWave;
  __shared__ Tri part[NW];
  __shared__ uint32_t lane_max[NT];
  __shared__ __align__(16) uint64_t cand[NW * kCandCap];
  __shared__ int count, cand_n[NW];
  static_assert(NW * kCandCap >= NT && NT % 8 == 0, "a candidate per thread, ranked in eights");
  const int row = blockIdx.y, split = blockIdx.x, splits = gridDim.x;
  const int tid = threadIdx.x, lane = tid % kWave, wave = tid / kWave;
  const int K = p.top_k;
  const T *x = static_cast<const T *>(p.logits) + (size_t)row * p.ld;
  const float c = p.inv_temp * kLog2e;
  // Vectors from the row's first 16-byte boundary, element `skip`; the logits
  // before it and the last few one per thread.
  const int skip = min((int)((0 - reinterpret_cast<uintptr_t>(x)) % 16 / sizeof(T)), p.V);
  const int nvec = (p.V - skip) / 8;
  const int per = (nvec + splits - 1) / splits;
  const int v0 = split * per;
  const int v1 = min(v0 + per, nvec);
  const rsrc_t rr = row_rsrc(x + skip, (uint32_t)max(v1, 0) * 8u * (uint32_t)sizeof(T));
  Vec8<T> w[U];
#pragma unroll
  for (int u = 0; u < U; u++) {
    w[u].load(rr, v0 + tid + u * NT);
    __builtin_amdgcn_sched_barrier(0);
  }
  asm volatile("" ::: "memory");
  if (tid == 0) count = 0;
  Tri t{kNegInf, 0.f, 0.f};
  float lm[U], mx = kNegInf;
#pragma unroll
  for (int u = 0; u < U; u++) {
    float a[8];
    w[u].get(a);
    lm[u] = kNegInf;
    if (v0 + tid + u * NT < v1) {
      lm[u] = max8(a);
      tri_fold8(t, a, lm[u], c);
    }
    mx = vmax(mx, lm[u]);
  }
  // The logits outside the vectors (fewer than 16), one per thread of the last split's first wave.
  const int et = tid < skip ? tid : nvec * 8 + tid;
  const bool has_tail = split == splits - 1 && et < p.V && tid < kWave;
  float tail = kNegInf;
  if (has_tail) {
    tail = load1(x + et);
    float y[1] = {tail * c};
    tri_add<1>(t, y);
    mx = vmax(mx, tail);
  }
  lane_max[tid] = order_bits(mx);
  cand[tid] = 0;
  __syncthreads();

  const float vmin = group_bound<NW>(lane_max, lane, K);  // nothing below it is among the split's k best
  // With fewer than K finite lane maxima every logit would qualify: straight
  // to the buffers. A lane stops once the candidates outnumber the threads.
  bool over = vmin == kNegInf;
  if (over) count = NT + 1;
  auto offer = [&](float v, uint32_t id) {
    const int at = atomicAdd(&count, 1);
    if (at < NT) cand[at] = cand_key(v, id);
    over = at >= NT;
  };
#pragma unroll
  for (int u = 0; u < U; u++) {
    const int v = v0 + tid + u * NT;
    if (v < v1 && !over && lm[u] >= vmin) {
      float a[8];
      w[u].get(a);
#pragma unroll
      for (int e = 0; e < 8; e++)
        if (!over && a[e] >= vmin) offer(a[e], (uint32_t)(skip + v * 8 + e));
    }
  }
  if (has_tail && !over && tail >= vmin) offer(tail, (uint32_t)et);
  t = wave_merge(t);
  if (lane == 0) part[wave] = t;
  __syncthreads();

  if (tid == NT - 1) {
    Tri r = part[0];
#pragma unroll
    for (int q = 1; q < NW; q++) r = tri_merge(r, part[q]);
    reinterpret_cast<float4 *>(p.ws)[(size_t)row * splits + split] = make_float4(r.m, r.z, r.s, 0.f);
  }
  uint64_t *keys = reinterpret_cast<uint64_t *>(static_cast<float *>(p.ws) + (size_t)p.R * splits * 4) +
                   ((size_t)row * splits + split) * K;
  const int n = count;
  if (n <= NT) {
    const uint64_t key = tid < n ? cand[tid] : 0;
    int rank = 0;
    for (int j = 0; j < n; j += 8)
#pragma unroll
      for (int q = 0; q < 8; q++) rank += cand[j + q] > key;  // zeros past the last
    if (tid < n) {
      if (rank < K) keys[rank] = key;
    } else if (tid < K) {
      keys[tid] = 0;
    }
    return;
  }
  // Every thread is past its read of the count, which stays; a wave's buffer
  // below holds nothing that is read again.
  Cands cs{cand + wave * kCandCap, 0, 1, kNegInf};
  cand_seed(cs, mx, K);
#pragma unroll 1
  for (int u = 0; u < U; u++) {
    float a[8];
    Vec8<T> wu = w[0];
#pragma unroll
    for (int q = 1; q < U; q++)
      if (q == u) wu = w[q];
    wu.get(a);
    const int v = v0 + tid + u * NT;
    cand_offer(cs, K, lane, a, (uint32_t)(skip + v * 8), v < v1 ? 8 : 0);
  }
  float a[8] = {tail, kNegInf, kNegInf, kNegInf, kNegInf, kNegInf, kNegInf, kNegInf};
  if (wave == 0) cand_offer(cs, K, lane, a, (uint32_t)et, has_tail ? 1 : 0);
  if (cs.cnt > K) cand_reduce_any(cs, K, K, lane);
  if (lane == 0) cand_n[wave] = cs.cnt;
  __syncthreads();
  if (wave != 0) return;
  int off[NW + 1];
  off[0] = 0;
#pragma unroll
  for (int q = 0; q < NW; q++) off[q + 1] = off[q] + cand_n[q];
  const int nw = gather_select<NW * kTopKMax / kWave, NW>(cand, off, K, lane, keys);
  for (int q = nw + lane; q < K; q += kWave) keys[q] = 0;
}

constexpr int kMergeEntries = 1024;  // splits * top_k bound of the sampling merge
constexpr int kMergeThreads = 1024;

// Per-row sampling merge, one workgroup per row: the splits' keys go to LDS
// and are ranked by counting, a quarter of the comparisons per group of 256
// threads (unique keys, so the ranks are the sorted order); meanwhile one
// wave merges the entropies and runs the detector and another draws the
// uniform. The first wave then has the softmax, the nucleus and the token. One wave
// doing all of it in turn (a bit-by-bit threshold, then the sort) took 9.5 us
// for 128 rows of 8 splits x 20 keys, this 4.7.
// The comparisons grow with the square of the keys (1024 of them 30 us). More
// than 256 are first cut to those that reach the leading bits of the top_k-th
// largest of 256 groups' maxima, about top_k of them; all are ranked where more
// than 256 do (many equal logits).
__global__ __launch_bounds__(kMergeThreads) void sample_merge(EntropyParams p) {
  constexpr int PARTS = 4, PT = kMergeThreads / PARTS;
  __shared__ __align__(16) uint64_t all[kMergeEntries + PT];  // the splits' keys, then those that may win
  __shared__ int rank[kMergeEntries];
  __shared__ uint64_t sorted[kTopKMax];
  __shared__ uint32_t group_max[PT];
  __shared__ int count;
  __shared__ float uniform;
  static_assert(kMergeEntries == PARTS * PT, "four keys per group");
  const int row = blockIdx.x;
  const int tid = threadIdx.x, lane = tid % kWave, wave = tid / kWave;
  const int S = p.splits, K = p.top_k;
  const int E = S * K;
  const uint64_t *src = reinterpret_cast<const uint64_t *>(static_cast<const float *>(p.ws) + (size_t)p.R * S * 4) +
                        (size_t)row * E;
  const uint64_t mine = tid < E ? src[tid] : 0;
  all[tid] = mine;
  rank[tid] = 0;
  if (tid < kTopKMax) sorted[tid] = 0;
  if (tid == 0) count = 0;
  __syncthreads();
  int n = E, base = 0;  // keys to rank: all[base ..), n of them
  if (E > PT) {
    if (tid < PT) {
      uint32_t m = 0;
#pragma unroll
      for (int q = 0; q < PARTS; q++) m = max(m, (uint32_t)(all[tid + q * PT] >> 32));
      group_max[tid] = m;
    }
    __syncthreads();
    const uint32_t bound = kth_bits<PT / kWave>(group_max, lane, K);
    if (mine != 0 && (uint32_t)(mine >> 32) >= bound) {
      const int at = atomicAdd(&count, 1);
      if (at < PT) all[kMergeEntries + at] = mine;
    }
    __syncthreads();
    if (count <= PT) {
      n = count;
      base = kMergeEntries;
    }
  }
  const uint64_t *keys = all + base;
  const int part = tid / PT;
  const int j0 = n * part / PARTS, j1 = n * (part + 1) / PARTS;
  for (int i = tid % PT; i < n; i += PT) {
    const uint64_t key = keys[i];
    int r = 0;
#pragma unroll 8
    for (int j = j0; j < j1; j++) r += keys[j] > key;
    if (key != 0) atomicAdd(&rank[i], r);
  }
  constexpr int NW = kMergeThreads / kWave;
  if (wave == NW - 1) {
    const float H = finish_entropy(wave_merge_splits(p, row, lane));
    if (lane == 0) p.H[row] = H;
    detector_push(p, row, H, lane);
  }
  if (wave == NW - 2) {
    const float u = row_uniform(p, row);
    if (lane == 0) uniform = u;
  }
  __syncthreads();
  if (tid < n && keys[tid] != 0 && rank[tid] < K) sorted[rank[tid]] = keys[tid];
  __syncthreads();
  if (wave == 0) sample_pick(p, row, lane, lane < K ? sorted[lane] : 0, uniform);
}

}  // namespace

static bool row_groups(int R, int V) { return R >= kRowMinRows && V / 8 >= kRowMinVecs; }

static int split_rule(int R, int V) {
  // Enough workgroups to cover the chip (~1024), but at least 1024 vectors of
  // 8 logits per workgroup; and, when the rows alone fill the chip, still no
  // more than one round of the vector loop per workgroup (measured: 256 rows
  // of 152k logits in 8 splits, 2048 workgroups, beat 4 splits by 6%).
  const long nvec = V / 8;
  long s = (1024 + R - 1) / R;
  const long maxs = nvec / 1024 > 0 ? nvec / 1024 : 1;
  if (s > maxs) s = maxs;
  const long one_round = (nvec + kRoundVecs - 1) / kRoundVecs;
  if (s < one_round) s = one_round;
  if (s < 1) s = 1;
  if (s > 1024) s = 1024;
  return (int)s;
}

int entropy_splits(int R, int V) { return row_groups(R, V) ? 1 : split_rule(R, V); }

size_t entropy_workspace_bytes(int R, int V) {
  const int s = entropy_splits(R, V);
  if (s == 1) return 0;
  return (size_t)R * s * 4 * sizeof(float);
}

// The splits of a sampling call, at least one round each where the merge takes
// that many candidates (splits * top_k).
int sample_splits(int R, int V, int top_k) {
  int s = split_rule(R, V);
  const int maxs = kMergeEntries / (top_k > 0 ? top_k : 1);
  return s < maxs ? s : maxs;
}

size_t sample_workspace_bytes(int R, int V, int top_k) {
  const int s = sample_splits(R, V, top_k);
  return (size_t)R * s * 4 * sizeof(float) + (size_t)R * s * top_k * sizeof(uint64_t);
}

template <typename T, bool VEC>
static void launch_split(const EntropyBatch &b, bool sample, bool rows, dim3 grid, hipStream_t stream) {
  if (sample) hipLaunchKernelGGL((entropy_kernel<T, VEC, true>), grid, dim3(kThreads), 0, stream, b);
  else if (rows) hipLaunchKernelGGL((entropy_kernel<T, VEC, false, kRowThreads>), grid, dim3(kRowThreads), 0, stream, b);
  else hipLaunchKernelGGL((entropy_kernel<T, VEC, false>), grid, dim3(kThreads), 0, stream, b);
}

// The split pass over every row of the batch (one launch), with 16-byte
// loads when every set's rows start 16-byte aligned.
static hipError_t launch_partials(const EntropyBatch &b, bool sample, hipStream_t stream) {
  const EntropyParams &p0 = b.set[0];
  const size_t esz = p0.dtype == 0 ? 4 : 2;
  bool vec = true;
  int vmin = p0.V;
  for (int k = 0; k < b.nsets; k++) {
    vec = vec && ((uintptr_t)b.set[k].logits % 16 == 0) && ((size_t)b.set[k].ld * esz % 16 == 0);
    vmin = b.set[k].V < vmin ? b.set[k].V : vmin;
  }
  const int R = b.row0[b.nsets];
  const bool rows = p0.splits == 1 && row_groups(R, vmin);
  const dim3 grid(p0.splits, R);
  if (p0.dtype == 0) {
    if (vec) launch_split<float, true>(b, sample, rows, grid, stream);
    else launch_split<float, false>(b, sample, rows, grid, stream);
  } else {
    if (vec) launch_split<bf16_t, true>(b, sample, rows, grid, stream);
    else launch_split<bf16_t, false>(b, sample, rows, grid, stream);
  }
  return hipGetLastError();
}

hipError_t entropy_scratch(void **ptr) {
  // Device address of `scratch` on the current device, looked up once per
  // device with that device current (each GPU holds its own copy).
  constexpr int kMaxDevices = 64;
  static std::atomic<void *> cache[kMaxDevices];
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  void *p = cache[dev].load(std::memory_order_acquire);
  if (p == nullptr) {
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (p == nullptr) return hipErrorInvalidSymbol;
    cache[dev].store(p, std::memory_order_release);
  }
  *ptr = p;
  return hipSuccess;
}

hipError_t launch_logit_entropy_batch(const EntropyBatch &b, hipStream_t stream) {
  hipError_t e = launch_partials(b, false, stream);
  if (e != hipSuccess || b.set[0].splits == 1) return e;
  hipLaunchKernelGGL(entropy_merge, dim3(b.row0[b.nsets]), dim3(kWave), 0, stream, b);
  return hipGetLastError();
}

hipError_t launch_logit_entropy(const EntropyParams &p, hipStream_t stream) {
  EntropyBatch b{};
  b.set[0] = p;
  b.row0[0] = 0;
  b.row0[1] = p.R;
  b.nsets = 1;
  if (p.top_k <= 0) return launch_logit_entropy_batch(b, stream);
  // Splits of one round; longer ones stream (entropy_kernel): rows beyond 327,680
  // logits with top_k 64, beyond a million with top_k 20. So do rows of fewer
  // than top_k vectors, too few lanes for a bound: one row of 100 logits with
  // top_k 13 14.7 us here and 8.8 there, 64 rows 18.6 and 12.2.
  const int nvec = p.V / 8;
  hipError_t e;
  if ((nvec + p.splits - 1) / p.splits <= kRoundVecs && nvec >= p.top_k) {
    const dim3 grid(p.splits, p.R);
    if (p.dtype == 0) hipLaunchKernelGGL(sample_split<float>, grid, dim3(kThreads), 0, stream, p);
    else hipLaunchKernelGGL(sample_split<bf16_t>, grid, dim3(kThreads), 0, stream, p);
    e = hipGetLastError();
  } else {
    e = launch_partials(b, true, stream);
  }
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(sample_merge, dim3(p.R), dim3(kMergeThreads), 0, stream, p);
  return hipGetLastError();
}

}  // namespace kvr
