// Window re-computation of the accumulated-attention importance score
// (Sec. 2.1): for the last nq tokens of every sequence, window row r attends
// causally over len - (nq-1-r) cache entries; each entry's score is the
// probability mass it receives, summed over the window rows and over the G
// query heads of its KV head. This runs when a whole step's tokens are encoded
// in one pass (a committed helper step, a one-shot prompt), not per decoded
// token.
//
// bf16 caches: the R = G * nq window rows of one (sequence, layer, KV head)
// form a dense [R x D] x [D x n] contraction, done on MFMA 16x16x32 bf16, one
// workgroup of eight waves per head. What bounds it is vector issue and the
// products, which overlap little (77% and 37% of the cycles over 42 commit and 6
// prompt calls); so each exp and each vector instruction counts:
//   - Heads of up to 768 keys (8 waves x 6 tiles of 16 keys in registers) take
//     one pass: every product and every exp is formed once, and the waves
//     exchange their rows' partial normalisers through LDS. On the commit
//     shape (16 x 28 x 4 heads, 896 rows, 641-768 keys) 0.44 ms, against 1.03
//     for two passes over keys streamed through LDS.
//   - Longer heads take two passes, the first with the window rows in
//     registers and the keys streaming (normalisers), the second with the keys
//     in registers and the rows streaming (column sums): 3.5 ms against 6.4
//     on 4096 keys.
//   - No running maximum: a row's exps need no reference as long as its
//     normaliser stays within 2^-80 .. 2^100, which is tested once per row. In
//     one pass a head with a row outside is done again with the rows' maxima
//     taken first; in two passes a group of rows with one outside is redone with
//     references that trail each lane's maximum. Measured with queries of
//     standard deviation 1 and 8 / 16 to 256 / 64 in one query head of 7: commit
//     shape 0.45 / 0.67-0.82 / 0.98 ms, 4096 keys 3.5 / 5.5-5.9 / 4.9; two passes
//     with an online maximum throughout take 1.04-1.16 and 6.3-6.8. There a NaN
//     logit counts as no probability, and a row with an infinite logit (or
//     none finite) adds nothing, so neither reaches another key's or row's score.
// Column sums are float32 over at most 32 rows (8 a lane, then a quad of
// lanes), then float64 in a fixed order over all of a head's rows, so the
// scores are bitwise reproducible and as exact as their float32 result (commit
// shape 2.7e-8 in the 2-norm against float64; 2.9e-8, but 1-2% less time, with
// 64 rows).
// Measured and not kept: products interleaved one by one with the exps, 32x32
// products, two or three independent workgroups per CU, four waves per SIMD
// (all 3.4 to 4.0 ms on 4096 keys).
//
// float32 caches take a plain one-wave-per-head kernel (one key per lane).
#include <hip/hip_runtime.h>

#include "kvr_device.h"
#include "kvr_internal.h"

namespace kvr {

namespace {

template <typename T>
__device__ __forceinline__ float ld(const T *p, size_t i);
template <>
__device__ __forceinline__ float ld<float>(const float *p, size_t i) { return p[i]; }
template <>
__device__ __forceinline__ float ld<bf16_t>(const bf16_t *p, size_t i) { return bf16_to_f32(p[i]); }

template <typename T>
__global__ __launch_bounds__(64) void window_scores_kernel(ScoreParams p) {
  extern __shared__ float smem[];
  const int unit = blockIdx.x;
  const int h = unit % p.Hkv;
  const int sl = unit / p.Hkv;
  const int l = sl % p.L;
  const int s = sl / p.L;
  const int lane = threadIdx.x;
  const int D = p.D, G = p.G;
  int n = p.len[s];
  n = n < 0 ? 0 : (n > p.cap ? p.cap : n);
  const T *K = static_cast<const T *>(p.k) + (size_t)unit * p.cap * D;
  float *qs = smem;          // [D]
  float *xs = smem + D;      // [cap]
  float *acc = xs + p.cap;   // [cap]
  for (int j = lane; j < n; j += kWave) acc[j] = 0.f;
  const float sl2 = p.scale * kLog2e;
  for (int r = 0; r < p.nq; r++) {
    const int nr = n - (p.nq - 1 - r);
    if (nr <= 0) continue;
    for (int g = 0; g < G; g++) {
      const size_t qoff = ((((size_t)s * p.L + l) * p.Hq + h * G + g) * p.nq + r) * D;
      __syncthreads();
      for (int d = lane; d < D; d += kWave) qs[d] = ld<T>(static_cast<const T *>(p.q_win), qoff + d);
      __syncthreads();
      float mloc = -__builtin_huge_valf();
      for (int j = lane; j < nr; j += kWave) {
        float dot = 0.f;
        for (int d = 0; d < D; d++) dot = fmaf(qs[d], ld<T>(K, (size_t)j * D + d), dot);
        xs[j] = dot * sl2;
        mloc = fmaxf(mloc, xs[j]);
      }
      const float m = wave_max(mloc);
      float zloc = 0.f;
      for (int j = lane; j < nr; j += kWave) zloc += fast_exp2(xs[j] - m);
      const float iz = 1.0f / wave_sum(zloc);
      for (int j = lane; j < nr; j += kWave) acc[j] += fast_exp2(xs[j] - m) * iz;
    }
  }
  float *sc = p.scores + (size_t)unit * p.cap;
  for (int j = lane; j < n; j += kWave) sc[j] = p.accumulate ? sc[j] + acc[j] : acc[j];
}


typedef __amdgpu_buffer_rsrc_t rsrc_t;
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ rsrc_t make_rsrc(const void *ptr, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(ptr), (short)0, (int)bytes, 0x00020000);
}

constexpr float kNegInf = -__builtin_huge_valf();

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef __attribute__((address_space(3))) void lds_void_t;

// s_waitcnt vmcnt(n), other counters unconstrained.
template <int N>
__device__ __forceinline__ void wait_vm() {
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (15 << 8));
}

__device__ __forceinline__ float4_t mfma(u32x4 a, u32x4 b, float4_t c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, a), __builtin_bit_cast(bf16x8_t, b), c,
                                                 0, 0, 0);
}

__device__ __forceinline__ float recip(float z) {
  const float r = __builtin_amdgcn_rcpf(z);
  return fmaf(fmaf(-z, r, 1.0f), r, r);
}

template <int CTRL>
__device__ __forceinline__ float dpp(float x) {
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), CTRL, 0xF, 0xF, true));
}
constexpr int kXor1 = 0xB1, kXor2 = 0x4E;  // quad_perm [1,0,3,2] and [2,3,0,1]
constexpr int kHalfMirror = 0x141, kMirror = 0x140;

// Sum (or maximum) over the 16 lanes of a row of lanes, in every one of them.
template <bool MAX>
__device__ __forceinline__ float reduce16(float v) {
  auto op = [](float a, float b) { return MAX ? fmaxf(a, b) : a + b; };
  v = op(v, dpp<kXor1>(v));
  v = op(v, dpp<kXor2>(v));
  v = op(v, dpp<kHalfMirror>(v));
  return op(v, dpp<kMirror>(v));
}

// Sum (or maximum) of the lanes l, l^16, l^32, l^48, in every one of them.
template <bool MAX>
__device__ __forceinline__ float reduce_groups(float v) {
  auto op = [](uint32_t a, uint32_t b) {
    return MAX ? fmaxf(__uint_as_float(a), __uint_as_float(b)) : __uint_as_float(a) + __uint_as_float(b);
  };
  const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = op(a[0], a[1]);
  const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return op(b[0], b[1]);
}
constexpr int kNW = 8;           // waves per workgroup
constexpr int kKeyTiles = 6;     // 16-key tiles a wave holds at once
constexpr int kRowTiles = 7;     // 16-row tiles a wave holds at once (pass 1 of two)
constexpr int kRG = kNW * kRowTiles * 16;  // window rows per group (two passes)
constexpr int kFlush = 4;        // blocks of 32 rows between the float32 column sums' flushes
// A row's exponentials are taken without a reference while its normaliser
// lies in this range: its largest logit is then between about -92 and 100
// (log2), nothing overflows, and the terms that underflow (below 2^-126) are
// less than 2^-33 of the normaliser together. What a logit's own rounding
// costs is the matrix product's error again: at logits of standard deviation 8
// the scores' error in the 2-norm is 2.8e-7 so, 2.6e-7 relative to maxima.
constexpr float kZLow = 0x1p-80f, kZHigh = 0x1p100f;
constexpr int kProbe = 8;  // blocks of 32 keys after which a group of rows that already left the range stops
// Exponent of an exp relative to a row's maximum: NaN (a NaN logit, or an
// infinite one less an infinite maximum) and anything as small become 2^-256 = 0.
// A row that adds nothing takes +inf for its maximum.
__device__ __forceinline__ float rel_exp2(float x) { return fast_exp2(fmaxf(x, -256.0f)); }

template <int D>
struct WLds {
  static constexpr int RU = D / 8;              // 16-byte units per row
  static constexpr int SLOT = 32 * D * 2;       // bytes per ring slot
  char ring[2][SLOT];
  double sum[kKeyTiles][kNW * kWave];  // the lanes' column sums
  union {
    float z[2][32][36];                // one pass: per row, the partial normalisers of 8 waves x 4 lanes
    struct {
      int nr[kRG];                     // two passes, per row of the group: the keys it sees,
      float f[kRG], m[kRG];            // 1 / normaliser and reference
    } g;
  };
  int bad;
};

// The window scores of one (sequence, layer, KV head) of n keys and R window
// rows by kNW waves. One operand of the products stays in a wave's registers
// (16-row tiles wave + kNW * k, the M dimension), the other streams through an
// LDS ring in blocks of 32, shared by the waves (halves of 16, the N
// dimension). A lane then holds N index lane & 15 and M index 4 * (lane >> 4)
// + i of each tile.
template <int D>
struct Window {
  static constexpr int KS = D / 32;  // MFMA k-steps
  static constexpr int RU = WLds<D>::RU;
  static constexpr int NI = WLds<D>::SLOT / 1024;  // 1 KiB loads per ring slot

  const ScoreParams &p;
  WLds<D> &lds;
  rsrc_t qr, kr;
  int n, R, wave, lane;
  float c;
  float *sc;

  // A copy whose lane number the compiler cannot follow, so that the address
  // arithmetic of one variant is not kept in registers through the others.
  __device__ __forceinline__ Window fresh() const {
    Window w = *this;
#if defined(__HIP_DEVICE_COMPILE__)
    asm volatile("" : "+v"(w.lane));
#endif
    return w;
  }

  // Workgroup barrier without the fence of __syncthreads (whose release
  // would also wait for the ring loads in flight): this wave's LDS
  // operations are complete, its ring loads are waited for explicitly, and
  // the memory clobber keeps the compiler from moving accesses across it.
  __device__ __forceinline__ void bar() const {
    __builtin_amdgcn_s_waitcnt(15 | (7 << 4) | (0 << 8) | (3 << 14));  // lgkmcnt(0)
    asm volatile("s_barrier" ::: "memory");
  }

  // Rows row0 .. row0 + 31 of r's array into a ring slot, 16-byte unit u of
  // row r at u ^ (r mod RU), spread over the waves; zeros past the array.
  __device__ __forceinline__ void issue(rsrc_t r, int row0, int slot) const {
#if defined(__HIP_DEVICE_COMPILE__)
    if (NI >= kNW || wave < NI) {
      const int row = wave * (1024 / (D * 2)) + lane / RU;
      const int u = (lane % RU) ^ (row % RU);
      const uint32_t off = ((uint32_t)(row0 + row) * RU + (uint32_t)u) * 16u;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_void_t *)(lds.ring[slot] + wave * 1024), 16, off, 0, 0, 0);
    }
#else
    (void)r;  // the host pass has no buffer-to-LDS loads
    (void)row0;
    (void)slot;
    (void)RU;
    (void)NI;
#endif
  }

  // The wave's M tiles k0 .. k0 + T - 1 of r's array from row base.
  template <int T>
  __device__ __forceinline__ void load_tiles(u32x4 (&mf)[T][KS], rsrc_t r, int base, int k0) const {
#pragma unroll
    for (int k = 0; k < T; k++) {
      const uint32_t off = (uint32_t)(base + (wave + kNW * (k0 + k)) * 16 + (lane & 15)) * (D * 2) +
                           (uint32_t)(lane >> 4) * 16u;
#pragma unroll
      for (int t = 0; t < KS; t++) mf[k][t] = __builtin_amdgcn_raw_buffer_load_b128(r, off + 64u * t, 0, 0);
    }
  }

  // Products of half b of a ring slot with the wave's tiles.
  template <int T>
  __device__ __forceinline__ void products(const u32x4 (&mf)[T][KS], int slot, int b, float4_t (&a)[T]) const {
    const int row = 16 * b + (lane & 15);
    u32x4 q[KS];
#pragma unroll
    for (int t = 0; t < KS; t++)
      q[t] = *reinterpret_cast<const u32x4 *>(lds.ring[slot] + (row * RU + ((4 * t + (lane >> 4)) ^ (row % RU))) * 16);
#pragma unroll
    for (int k = 0; k < T; k++) {
      a[k] = float4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int t = 0; t < KS; t++) a[k] = mfma(mf[k][t], q[t], a[k]);
    }
  }

  // Column sums: a lane's float32 sums of 4 T keys, each over at most 2 kFlush
  // rows, are summed over quads of lanes (lane l of a quad keeps key l of each
  // tile's four) and added in float64.
  template <int T>
  __device__ __forceinline__ void flush(float4_t (&acc)[T]) const {
    const bool b0 = lane & 1, b1 = lane & 2;
#pragma unroll
    for (int k = 0; k < T; k++) {
      const float s01 = (b0 ? acc[k][1] : acc[k][0]) + dpp<kXor1>(b0 ? acc[k][0] : acc[k][1]);
      const float s23 = (b0 ? acc[k][3] : acc[k][2]) + dpp<kXor1>(b0 ? acc[k][2] : acc[k][3]);
      lds.sum[k][threadIdx.x] += (double)((b1 ? s23 : s01) + dpp<kXor2>(b1 ? s01 : s23));
      acc[k] = float4_t{0.f, 0.f, 0.f, 0.f};
    }
  }

  template <int T>
  __device__ __forceinline__ void clear(float4_t (&acc)[T]) const {
#pragma unroll
    for (int k = 0; k < T; k++) {
      acc[k] = float4_t{0.f, 0.f, 0.f, 0.f};
      lds.sum[k][threadIdx.x] = 0.0;
    }
  }

  // The quads' sums, written by the first quad's lanes. With several groups of
  // window rows (two passes) a key's sum is carried in float64 from the first
  // group (`begin`) to the last (`end`), by the same lane in each.
  template <int T>
  __device__ __forceinline__ void put(int k0, bool begin, bool end) const {
    extern __shared__ double carried[];  // [cap], with several groups only
#pragma unroll
    for (int k = 0; k < T; k++) {
      double v = lds.sum[k][threadIdx.x];
      v += shfl_xor(v, 4);
      v += shfl_xor(v, 8);
      const int j = (wave + kNW * (k0 + k)) * 16 + 4 * (lane >> 4) + (lane & 15);
      if ((lane & 15) < 4 && j < n) {
        if (!begin) v += carried[j];
        if (!end) carried[j] = v;
        else sc[j] = p.accumulate ? sc[j] + (float)v : (float)v;
      }
    }
  }

  // Keys that window row rho sees (0 past the last row).
  __device__ __forceinline__ int visible(int rho) const {
    const int late = p.nq - 1 - (int)((uint32_t)rho % (uint32_t)p.nq);
    return rho < R ? n - late : 0;
  }

  // A row's value from the 32 partial ones that the waves left in lds.z[buf]:
  // this lane takes 8 of them, then the four groups of lanes meet.
  template <bool MAX>
  __device__ __forceinline__ float exchange(int buf, int row) const {
    const float *zr = lds.z[buf][row] + 8 * (lane >> 4);
    const float4_t a = *reinterpret_cast<const float4_t *>(zr), b = *reinterpret_cast<const float4_t *>(zr + 4);
    auto op = [](float x, float y) { return MAX ? fmaxf(x, y) : x + y; };
    return reduce_groups<MAX>(op(op(op(a[0], a[1]), op(a[2], a[3])), op(op(b[0], b[1]), op(b[2], b[3]))));
  }

  // One pass: every key of the head in the waves' registers, the window rows
  // streaming. Per block of 32 rows the waves exchange their partial
  // normalisers through LDS and add the probabilities, each formed once, to
  // the column sums. The last MS tiles may hold keys a row does not see.
  // A head with a row outside the range of the reference-free form is done
  // again with the rows' maxima taken before the exps (one barrier and a
  // maximum per logit more). The test comes after 4, 16, 64 ... blocks: after
  // every one, or with the flush, it costs each head 3 to 5%.
  template <int T, int MS>
  __device__ __forceinline__ void one_pass() const {
    const int gq = lane >> 4, r16 = lane & 15;
    u32x4 kf[T][KS];
    load_tiles<T>(kf, kr, 0, 0);
    float4_t acc[T];
    clear<T>(acc);
    const int blocks = (R + 31) / 32;
    auto sees = [&](int k, int i, int nr) { return k < T - MS || (wave + kNW * k) * 16 + 4 * gq + i < nr; };
    auto add = [&](const float4_t (&v)[2][T], const float (&f)[2]) {
#pragma unroll
      for (int b = 0; b < 2; b++)
#pragma unroll
        for (int k = 0; k < T; k++)
#pragma unroll
          for (int i = 0; i < 4; i++) acc[k][i] = fmaf(v[b][k][i], f[b], acc[k][i]);
    };
    issue(qr, 0, 0);
    wait_vm<0>();
    bar();
    bool bad = false;
    int blk = 0;
#pragma unroll 1
    for (int stop = blocks < kFlush ? blocks : kFlush;; stop = 4 * stop < blocks ? 4 * stop : blocks) {
#pragma unroll 1
      for (; blk < stop; blk++) {
        issue(qr, (blk + 1) * 32, (blk + 1) & 1);  // past the last row: zeros, no memory traffic
        float4_t x[2][T];
        int nr[2];
#pragma unroll
        for (int b = 0; b < 2; b++) {
          nr[b] = visible(blk * 32 + 16 * b + r16);
          products<T>(kf, blk & 1, b, x[b]);
        }
#pragma unroll
        for (int b = 0; b < 2; b++) {
          float4_t z = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int k = 0; k < T; k++)
#pragma unroll
            for (int i = 0; i < 4; i++) {
              const float v = fast_exp2(x[b][k][i] * c);
              x[b][k][i] = sees(k, i, nr[b]) ? v : 0.f;
              z[i] += x[b][k][i];
            }
          lds.z[blk & 1][16 * b + r16][4 * wave + gq] = (z[0] + z[1]) + (z[2] + z[3]);
        }
        wait_vm<0>();
        bar();
        float f[2];
#pragma unroll
        for (int b = 0; b < 2; b++) {
          const float Z = exchange<false>(blk & 1, 16 * b + r16);
          bad |= nr[b] > 0 && !(Z >= kZLow && Z <= kZHigh);
          f[b] = nr[b] > 0 ? recip(Z) : 0.f;
        }
        add(x, f);
        if (blk % kFlush == kFlush - 1) flush<T>(acc);
      }
      // The waves hold the same normalisers, so they agree.
      if (__builtin_amdgcn_ballot_w64(bad) != 0 || stop == blocks) break;
    }
    if (__builtin_amdgcn_ballot_w64(bad) != 0) {
      blk = 0;
      clear<T>(acc);
      bar();  // every wave's reads of the ring and the normalisers are done
      issue(qr, blk * 32, blk & 1);
      wait_vm<0>();
      bar();
#pragma unroll 1
      for (; blk < blocks; blk++) {
        issue(qr, (blk + 1) * 32, (blk + 1) & 1);
        float4_t x[2][T];
        int nr[2];
#pragma unroll
        for (int b = 0; b < 2; b++) {
          nr[b] = visible(blk * 32 + 16 * b + r16);
          products<T>(kf, blk & 1, b, x[b]);
          float m = kNegInf;
#pragma unroll
          for (int k = 0; k < T; k++)
#pragma unroll
            for (int i = 0; i < 4; i++) m = fmaxf(m, sees(k, i, nr[b]) ? x[b][k][i] * c : kNegInf);
          lds.z[1][16 * b + r16][4 * wave + gq] = m;
        }
        wait_vm<0>();
        bar();
#pragma unroll
        for (int b = 0; b < 2; b++) {
          float m = exchange<true>(1, 16 * b + r16);
          m = m > kNegInf ? m : -kNegInf;
          float4_t z = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int k = 0; k < T; k++)
#pragma unroll
            for (int i = 0; i < 4; i++) {
              const float v = rel_exp2(fmaf(x[b][k][i], c, -m));
              x[b][k][i] = sees(k, i, nr[b]) ? v : 0.f;
              z[i] += x[b][k][i];
            }
          lds.z[0][16 * b + r16][4 * wave + gq] = (z[0] + z[1]) + (z[2] + z[3]);
        }
        bar();
        float f[2];
#pragma unroll
        for (int b = 0; b < 2; b++) {
          const float Z = exchange<false>(0, 16 * b + r16);
          f[b] = nr[b] > 0 && Z > 0.f ? recip(Z) : 0.f;
        }
        add(x, f);
        if (blk % kFlush == kFlush - 1) flush<T>(acc);
      }
    }
    flush<T>(acc);
    put<T>(0, true, true);
  }

  // Two passes: `blocks` blocks of 32 rows of r's array from row0 through the
  // ring, eat(h, a) for the products of each half h (unscaled). Block i + 1 is
  // loaded while block i is read; the rows past the array are zeros.
  template <int T, typename Eat>
  __device__ __forceinline__ void stream(const u32x4 (&mf)[T][KS], rsrc_t r, int row0, int blocks, Eat eat) const {
    issue(r, row0, 0);
#pragma unroll 1
    for (int i = 0; i < blocks; i++) {
      wait_vm<0>();
      bar();
      issue(r, row0 + (i + 1) * 32, (i + 1) & 1);
      float4_t a[2][T];
#pragma unroll
      for (int b = 0; b < 2; b++) products<T>(mf, i & 1, b, a[b]);
#pragma unroll
      for (int b = 0; b < 2; b++) eat(2 * i + b, a[b]);
    }
    wait_vm<0>();
    bar();  // every wave's reads of the ring are done
  }

  // Pass 1 over the keys, with the group's row tiles t0 + wave + kNW * k in
  // the waves' registers: each row's normaliser, without a reference, or (REF)
  // relative to one that trails the lane's maximum by up to 2^kSlack, so that
  // it hardly ever moves; the row's goes to lds.g.m.
  template <int T, bool REF>
  __device__ __forceinline__ void normalisers(int row0, int t0) const {
    constexpr float kSlack = 64.0f;
    const int gq = lane >> 4, r16 = lane & 15;
    u32x4 qf[T][KS];
    load_tiles<T>(qf, qr, row0 + 16 * t0, 0);
    auto at = [&](int k) { return (t0 + wave + kNW * k) * 16 + 4 * gq; };
    float4_t z[T], m[REF ? T : 1];
#pragma unroll
    for (int k = 0; k < T; k++) {
      z[k] = float4_t{0.f, 0.f, 0.f, 0.f};
      if (REF) m[k] = float4_t{kNegInf, kNegInf, kNegInf, kNegInf};
    }
    auto fold = [&](const float4_t (&a)[T], auto sees) {
      if constexpr (!REF) {
#pragma unroll
        for (int k = 0; k < T; k++)
#pragma unroll
          for (int i = 0; i < 4; i++) z[k][i] += fast_exp2(sees(k, i) ? a[k][i] * c : kNegInf);
      } else {
        bool up = false;
#pragma unroll
        for (int k = 0; k < T; k++)
#pragma unroll
          for (int i = 0; i < 4; i++) up |= sees(k, i) && a[k][i] * c > m[k][i] + kSlack;
        if (__builtin_amdgcn_ballot_w64(up) != 0) {
#pragma unroll
          for (int k = 0; k < T; k++)
#pragma unroll
            for (int i = 0; i < 4; i++) {
              const float x = a[k][i] * c;
              if (sees(k, i) && x > m[k][i] + kSlack) {
                z[k][i] = z[k][i] > 0.f ? z[k][i] * fast_exp2(m[k][i] - x) : 0.f;
                m[k][i] = x;
              }
            }
        }
#pragma unroll
        for (int k = 0; k < T; k++)
#pragma unroll
          for (int i = 0; i < 4; i++) z[k][i] += rel_exp2(sees(k, i) ? fmaf(a[k][i], c, -m[k][i]) : kNegInf);
      }
    };
    // Blocks of keys that every row sees, then the others with the mask.
    const int seen = n - p.nq + 1;
    const int plain = seen > 0 ? seen / 32 : 0, all = (n + 31) / 32;
    auto fold_all = [&](int, const float4_t (&a)[T]) { fold(a, [](int, int) { return true; }); };
    int from = 0;
    if (!REF && plain > kProbe) {
      stream<T>(qf, kr, 0, kProbe, fold_all);
      bool over = false;
#pragma unroll
      for (int k = 0; k < T; k++)
#pragma unroll
        for (int i = 0; i < 4; i++) over |= !(z[k][i] <= kZHigh);
      if (over) lds.bad = 1;
      bar();
      if (lds.bad) return;  // every wave: it is written again after a barrier of the next blocks only
      from = kProbe;
    }
    if (plain > from) stream<T>(qf, kr, from * 32, plain - from, fold_all);
    if (all > plain)
      stream<T>(qf, kr, plain * 32, all - plain, [&](int h, const float4_t (&a)[T]) {
        const int key = (plain * 2 + h) * 16 + r16;
        fold(a, [&](int k, int i) { return key < lds.g.nr[at(k) + i]; });
      });
    bool bad = false;
#pragma unroll
    for (int k = 0; k < T; k++) {
      float4_t f, M;
#pragma unroll
      for (int i = 0; i < 4; i++) {
        const bool live = lds.g.nr[at(k) + i] > 0;
        float Z = z[k][i];
        if (REF) {
          const float ml = m[REF ? k : 0][i];
          M[i] = reduce16<true>(ml);
          Z = Z > 0.f ? Z * fast_exp2(ml - M[i]) : 0.f;
        }
        Z = reduce16<false>(Z);
        if (!REF) bad |= live && !(Z >= kZLow && Z <= kZHigh);
        f[i] = live && Z > 0.f ? recip(Z) : 0.f;
        if (REF && f[i] == 0.f) M[i] = -kNegInf;
      }
      if (r16 == 0) {
        *reinterpret_cast<float4_t *>(lds.g.f + at(k)) = f;
        if (REF) *reinterpret_cast<float4_t *>(lds.g.m + at(k)) = M;
      }
    }
    if (bad) lds.bad = 1;
  }

  template <bool REF>
  __device__ __forceinline__ void normalise(int row0, int tiles) const {
    const int slots = (tiles + kNW - 1) / kNW;  // per wave, at most kRowTiles
    // Few rows wait for the keys' stream more than for their products, so one
    // tile has a form of its own: 112 heads of 800 keys and 128 rows 121 -> 110 us.
    if (slots <= 1) fresh().template normalisers<1, REF>(row0, 0);
    else if (slots <= 2) fresh().template normalisers<2, REF>(row0, 0);
    else if (slots <= 4) fresh().template normalisers<4, REF>(row0, 0);
    else if constexpr (!REF) fresh().template normalisers<kRowTiles, REF>(row0, 0);
    else {
      // References take registers: two passes over the keys.
      fresh().template normalisers<4, REF>(row0, 0);
      fresh().template normalisers<kRowTiles - 4, REF>(row0, 4 * kNW);
    }
    bar();
  }

  // Pass 2, over the group's rows with tiles k0 .. k0 + T - 1 of the keys in
  // the waves' registers: their column sums. REF: relative to the rows' references.
  template <int T, bool MASK, bool REF>
  __device__ __forceinline__ void columns(int row0, int blocks, int k0, bool last) const {
    const int gq = lane >> 4, r16 = lane & 15;
    u32x4 kf[T][KS];
    load_tiles<T>(kf, kr, 0, k0);
    float4_t acc[T];
    clear<T>(acc);
    stream<T>(kf, qr, row0, blocks, [&](int h, const float4_t (&a)[T]) {
      const float f = lds.g.f[16 * h + r16], m = lds.g.m[16 * h + r16];
      const int nr = MASK ? lds.g.nr[16 * h + r16] : 0;
#pragma unroll
      for (int k = 0; k < T; k++)
#pragma unroll
        for (int i = 0; i < 4; i++) {
          float x = fmaf(a[k][i], c, -m);
          if (MASK) x = (wave + kNW * (k0 + k)) * 16 + 4 * gq + i < nr ? x : kNegInf;
          acc[k][i] = fmaf(REF ? rel_exp2(x) : fast_exp2(x), f, acc[k][i]);
        }
      if (h % (2 * kFlush) == 2 * kFlush - 1) flush<T>(acc);
    });
    flush<T>(acc);
    put<T>(k0, row0 == 0, last);
  }

  template <bool REF>
  __device__ __forceinline__ void columns_of(int row0, int blocks, int slots, int seen, bool last) const {
#pragma unroll 1
    for (int k0 = 0; k0 < slots; k0 += kKeyTiles) {
      const int kt = slots - k0;
      // Uniform over the workgroup (every wave meets the barriers inside).
      const bool mask = kNW * (k0 + kKeyTiles) * 16 > seen;
      if (kt <= 2) fresh().template columns<2, true, REF>(row0, blocks, k0, last);
      else if (kt <= 4) fresh().template columns<4, true, REF>(row0, blocks, k0, last);
      else if (mask) fresh().template columns<kKeyTiles, true, REF>(row0, blocks, k0, last);
      else fresh().template columns<kKeyTiles, false, REF>(row0, blocks, k0, last);
    }
  }

  __device__ __forceinline__ void two_pass(int slots) const {
    const int groups = (R + kRG - 1) / kRG;
    const int per = ((R + groups - 1) / groups + 31) / 32 * 32;  // rows per group, at most kRG
    const int seen = n - p.nq + 1;  // keys below this are visible to every row
#pragma unroll 1
    for (int row0 = 0; row0 < R; row0 += per) {
      const int rows = R - row0 < per ? R - row0 : per;
      const int blocks = (rows + 31) / 32;
      if (threadIdx.x == 0) lds.bad = 0;
      for (int at = threadIdx.x; at < kRG; at += kNW * kWave) {
        lds.g.nr[at] = at < rows ? visible(row0 + at) : 0;
        lds.g.f[at] = lds.g.m[at] = 0.f;
      }
      bar();
      normalise<false>(row0, 2 * blocks);
      if (lds.bad) {
        normalise<true>(row0, 2 * blocks);
        columns_of<true>(row0, blocks, slots, seen, row0 + rows == R);
      } else {
        columns_of<false>(row0, blocks, slots, seen, row0 + rows == R);
      }
    }
  }
};

template <int D>
__global__ __launch_bounds__(kNW * 64) __attribute__((amdgpu_waves_per_eu(2))) void window_scores_bf16(ScoreParams p) {
  __shared__ __align__(16) WLds<D> lds;
  const int unit = blockIdx.x;
  const int h = unit % p.Hkv;
  const int sl = unit / p.Hkv;
  const int l = sl % p.L;
  const int s = sl / p.L;
  int n = p.len[s];
  n = n < 0 ? 0 : (n > p.cap ? p.cap : n);
  if (n == 0) return;
  const int R = p.G * p.nq;
  const bf16_t *Q = static_cast<const bf16_t *>(p.q_win) + (((size_t)s * p.L + l) * p.Hq + (size_t)h * p.G) * p.nq * D;
  const bf16_t *K = static_cast<const bf16_t *>(p.k) + (size_t)unit * p.cap * D;
  const Window<D> w{p, lds, make_rsrc(Q, (uint32_t)R * D * 2u), make_rsrc(K, (uint32_t)n * D * 2u), n, R,
                    __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), (int)(threadIdx.x % kWave),
                    p.scale * kLog2e, p.scores + (size_t)unit * p.cap};
  const int slots = ((n + 15) / 16 + kNW - 1) / kNW;  // 16-key tiles per wave
  if (slots <= 2) w.fresh().template one_pass<2, 2>();
  else if (slots <= 4) w.fresh().template one_pass<4, 4>();
  else if (slots <= kKeyTiles) {
    // The causal mask reaches the last two tiles of a wave only, or all.
    if (n >= p.nq && (n - p.nq + 1) / (16 * kNW) >= kKeyTiles - 2) w.fresh().template one_pass<6, 2>();
    else w.fresh().template one_pass<6, 6>();
  } else {
    w.two_pass(slots);
  }
}

}  // namespace

hipError_t launch_accumulate_scores(const ScoreParams &p, hipStream_t stream) {
  const dim3 grid(p.S * p.L * p.Hkv);
  if (p.dtype == 0) {
    const size_t lds = ((size_t)p.D + 2 * (size_t)p.cap) * sizeof(float);
    hipLaunchKernelGGL(window_scores_kernel<float>, grid, dim3(64), lds, stream, p);
  } else {
    // Sums carried between groups of window rows (two passes): 64 KiB at the
    // longest cache, 8192 slots, beside 51 KiB of the kernel's own, of the
    // 160 KiB of a CU, whose registers hold one workgroup.
    const size_t lds = p.G * p.nq > kRG && p.cap > kNW * kKeyTiles * 16 ? (size_t)p.cap * sizeof(double) : 0;
    if (p.D == 128) hipLaunchKernelGGL(window_scores_bf16<128>, grid, dim3(kNW * kWave), lds, stream, p);
    else hipLaunchKernelGGL(window_scores_bf16<64>, grid, dim3(kNW * kWave), lds, stream, p);
  }
  return hipGetLastError();
}

}  // namespace kvr
