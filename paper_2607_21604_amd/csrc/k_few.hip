// Projection GEMMs over few rows: C = A . B^T (A [M][K] activations, B [N][K] weights) where
// M is so small that the weights' stream from HBM and the latency of each k-step count, not
// the matrix cores (probe layers at small refresh ratios, caching one memory unit, the query
// rows of the last layer).
//
// Blocks of 4 waves on small BM x BN tiles, so that even a few rows make enough blocks to
// stream the weights without cutting K. Operand tiles of BK columns go from global memory
// straight into LDS (buffer loads to LDS, no registers), NST tiles deep: with 128 KB in
// flight per CU a k-step waits for loads issued NST - 1 steps earlier. A wave holds the
// fragments of two k-tiles in registers: while it multiplies one, the next is read from LDS,
// so a k-step has one wait and one barrier and no LDS latency on its critical path.
//   step t: fragments of t in registers, tile t + 1 landed -> barrier -> request tile t + NST
//           into t's buffer (every wave has read it), read the fragments of t + 1, multiply t.
// 16-byte chunk c of a row sits at position c ^ (row % chunks), which keeps fragment reads
// free of bank conflicts. The product is formed transposed (the weights are the MFMA's row
// operand), so a lane holds four neighbouring output columns of one row and the epilogues
// work from the registers: a tile's columns are pairs (gate / up, the two rotary halves)
// stacked so that a wave holds both members.
// What bounds it: below about 150 rows the weights' stream and the launch, from there the
// k-steps, whose operands pass from L2 to the CUs at 12 to 16 TB/s (the tiles' (BM + BN) x 128
// bytes per 64 columns); whether that rate is the limit or the LDS traffic at one wave per SIMD
// has not been told apart.
// us of the 3B QKV, output, gate/up and down projections, 8-wave tiles with their K split -> the
// picks of launch_gemm (tile, K slices), weights from HBM:
//    64 rows  21.8, 18.7, 38.2, 27.2 -> 15.8 (32x64), 13.0 (64x64, 4), 27.2 (64x64), 22.0 (64x64, 4)
//   173 rows  22.9, 20.3, 41.2, 28.4 -> 19.4 (64x64), 17.9 (96x128, 5), 37.5 (96x128), 27.5 (96x128, 5)
// and with the weights in cache, as in a repeated call, at 173 rows 20.9, 19.6, 38.4, 28.4 ->
// 15.6, 16.2, 25.1, 22.0 (the output projection on 64x64 without slices 13.8, but 18.7 from HBM). At
// 475 rows only the output projection is taken: 26.7 -> 23.4 (96x64).
// Stages: 64 x 64 tiles of 64 columns three deep took 22.1 us for the 173-row QKV, eight deep
// 17.2, and with the fragments of two tiles in registers 16.4; 128 columns four deep 15.7.
#include <algorithm>

#include "gemm_dev.h"
#include "kernels.h"

namespace akvs {

namespace {

template <int BM, int BN, int BK>
struct Few {
  static constexpr int WM = BM / 2, WN = BN / 2, MI = WM / 16, NJ = WN / 16;
  static constexpr int CPR = BK / 8, RPI = 64 / CPR;       // chunks per row, rows per request
  static constexpr int IC = (BM + BN) / (4 * RPI), IA = BM / (4 * RPI);  // requests per wave
  static constexpr int KS = BK / 32;
  static constexpr int STAGE = (BM + BN) * BK;             // bf16 elements
  static_assert(BM % (4 * RPI) == 0 && BN % (4 * RPI) == 0 && NJ % 2 == 0, "tile shape");
};

// s_waitcnt with vmcnt(n) alone (n < 64), and lgkmcnt(0) alone
#define AKVS_WAIT_VM(n) __builtin_amdgcn_s_waitcnt(0x0f70 | ((n) & 15) | (((n) >> 4) << 14))
#define AKVS_WAIT_LGKM() __builtin_amdgcn_s_waitcnt(0xc07f)

// MODE: EPI_RESID, EPI_SWIGLU or EPI_QKV. splits > 1 (EPI_RESID only): block takes k-slice
// bid / tiles of tile bid % tiles and writes its fp32 sums to part [splits][M][N].
template <int BM, int BN, int BK, int NST, int MODE>
__device__ __forceinline__ void few_body(bf16_t *const (&st)[6], const bf16_t *__restrict__ A,
                                         int lda, const bf16_t *__restrict__ B, int ldb, int M,
                                         int M_eff, int N, int K, int b_rows, const Epi &e,
                                         int splits, float *__restrict__ part) {
  using S = Few<BM, BN, BK>;
  constexpr bool swiglu = MODE == EPI_SWIGLU, pairs = swiglu || MODE == EPI_QKV;
  static_assert(NST % 2 == 0 && NST <= 6, "stages");
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1, lr = lane & 15, lg = lane >> 4;
  constexpr int bn_out = swiglu ? BN / 2 : BN;
  const int n_tiles = (N + bn_out - 1) / bn_out, m_tiles = (M_eff + BM - 1) / BM;
  int split = 0, bid = blockIdx.x;
  if (splits > 1) {
    const int tiles = max(1, m_tiles * n_tiles);
    split = bid / tiles;
    bid -= split * tiles;
    if (split >= splits) return;
  }
  int mt, nt;
  if (!grouped_tile<8>(bid, m_tiles, n_tiles, mt, nt)) return;
  const int m0 = mt * BM, n0 = nt * bn_out;
  const int half = e.hd >> 1, half_shift = e.hd == 128 ? 6 : 5;
  const __amdgpu_buffer_rsrc_t ra = gemm_rsrc(A, (uint32_t)((size_t)M_eff * lda * 2));
  const __amdgpu_buffer_rsrc_t rb = gemm_rsrc(B, (uint32_t)b_rows * (uint32_t)ldb * 2u);

  // request i of a wave fills rows (4 i + wave) RPI .. of the stacked [A tile; B tile]; rows
  // past M / N read a valid row, whose results are discarded
  int voff[S::IC];
#pragma unroll
  for (int i = 0; i < S::IC; ++i) {
    const int r = (i * 4 + wave) * S::RPI + lane / S::CPR;
    const int ch = ((lane % S::CPR) ^ (r % S::CPR)) * 8;
    if (i < S::IA) {
      voff[i] = (min(m0 + r, M_eff - 1) * lda + ch) * 2;
    } else {
      const int j = r - BM;
      int gn;
      if (pairs) {  // a wave's columns: WN / 2 first members, then their second members
        const int w = j / S::WN, jj = j - w * S::WN, second = jj >= S::WN / 2;
        const int p = nt * (BN / 2) + w * (S::WN / 2) + jj - second * (S::WN / 2);
        if (swiglu) {
          gn = min(p, N - 1) + second * N;
        } else {
          const int pp = min(p, N / 2 - 1);
          gn = (pp >> half_shift) * e.hd + (pp & (half - 1)) + second * half;
        }
      } else {
        gn = min(n0 + j, N - 1);
      }
      voff[i] = (gn * ldb + ch) * 2;
    }
  }
  const int nk_all = K / BK, per = (nk_all + splits - 1) / splits;
  const int kt0 = min(split * per, nk_all - 1);
  const int nk = max(1, min(nk_all, kt0 + per) - kt0);  // (splits <= nk_all: no empty slice)
  f32x4_t acc[S::MI][S::NJ];
#pragma unroll
  for (int i = 0; i < S::MI; ++i)
#pragma unroll
    for (int j = 0; j < S::NJ; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) acc[i][j][r] = 0.f;
  bf16x8_t fa[2][S::KS][S::MI], fb[2][S::KS][S::NJ];

  // (requests past the last tile re-read it, so that every step has the same count in flight)
  auto request = [&](int t, bf16_t *dst) __attribute__((always_inline)) {
    const int so = (kt0 + min(t, nk - 1)) * (BK * 2);
#pragma unroll
    for (int i = 0; i < S::IC; ++i)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(
          i < S::IA ? ra : rb,
          (__attribute__((address_space(3))) void *)(dst + (i * 4 + wave) * S::RPI * BK), 16,
          voff[i], so, 0, 0);
  };
  auto fragments = [&](int f, const bf16_t *src) __attribute__((always_inline)) {
#pragma unroll
    for (int ks = 0; ks < S::KS; ++ks) {
      const int c = ((ks * 4 + lg) ^ (lr % S::CPR)) * 8;
      const bf16_t *a = src + (wm * S::WM + lr) * BK + c;
      const bf16_t *b = src + (BM + wn * S::WN + lr) * BK + c;
#pragma unroll
      for (int i = 0; i < S::MI; ++i)
        fa[f][ks][i] = *reinterpret_cast<const bf16x8_t *>(a + i * 16 * BK);
#pragma unroll
      for (int j = 0; j < S::NJ; ++j)
        fb[f][ks][j] = *reinterpret_cast<const bf16x8_t *>(b + j * 16 * BK);
    }
  };
  auto step = [&](int t, int f, bf16_t *cur, const bf16_t *nxt) __attribute__((always_inline)) {
    AKVS_WAIT_LGKM();                 // the fragments of tile t are in registers
    AKVS_WAIT_VM((NST - 2) * S::IC);  // this wave's part of tile t + 1 landed
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    request(t + NST, cur);
    fragments(1 - f, nxt);
#pragma unroll
    for (int ks = 0; ks < S::KS; ++ks)
#pragma unroll
      for (int i = 0; i < S::MI; ++i)
#pragma unroll
        for (int j = 0; j < S::NJ; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[f][ks][j], fa[f][ks][i],
                                                              acc[i][j], 0, 0, 0);
    __builtin_amdgcn_sched_barrier(0);
  };
#pragma unroll
  for (int i = 0; i < NST; ++i) request(i, st[i]);
  AKVS_WAIT_VM((NST - 1) * S::IC);
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_sched_barrier(0);
  fragments(0, st[0]);
  for (int t = 0; t < nk; t += NST) {
#pragma unroll
    for (int i = 0; i < NST; ++i)
      if (i == 0 || t + i < nk) step(t + i, i & 1, st[i], st[(i + 1) % NST]);
  }
  AKVS_WAIT_VM(0);  // nothing lands in LDS after this block's end

  // acc[i][j][r]: row m0 + wm WM + 16 i + lr, tile column wn WN + 16 j + 4 lg + r
  if (MODE == EPI_RESID && splits > 1) {
#pragma unroll
    for (int i = 0; i < S::MI; ++i) {
      const int gm = m0 + wm * S::WM + i * 16 + lr;
      float *dst = part + ((size_t)split * M + gm) * N;
#pragma unroll
      for (int j = 0; j < S::NJ; ++j) {
        const int gn = n0 + wn * S::WN + j * 16 + lg * 4;
        if (gm < M_eff && gn < N)
          *reinterpret_cast<float4 *>(dst + gn) =
              make_float4(acc[i][j][0], acc[i][j][1], acc[i][j][2], acc[i][j][3]);
      }
    }
  } else if (MODE == EPI_RESID) {
    // every residual of the wave is requested before the first sum is stored
    float4 h[S::MI][S::NJ];
#pragma unroll
    for (int i = 0; i < S::MI; ++i) {
      const int gm = min(m0 + wm * S::WM + i * 16 + lr, M_eff - 1);
      const float *src = reinterpret_cast<const float *>(e.out) + (size_t)gm * e.ldo;
#pragma unroll
      for (int j = 0; j < S::NJ; ++j)
        h[i][j] = *reinterpret_cast<const float4 *>(
            src + min(n0 + wn * S::WN + j * 16 + lg * 4, N - 4));
    }
#pragma unroll
    for (int i = 0; i < S::MI; ++i) {
      const int gm = m0 + wm * S::WM + i * 16 + lr;
      float *dst = reinterpret_cast<float *>(e.out) + (size_t)gm * e.ldo;
#pragma unroll
      for (int j = 0; j < S::NJ; ++j) {
        const int gn = n0 + wn * S::WN + j * 16 + lg * 4;
        if (gm < M_eff && gn < N)
          *reinterpret_cast<float4 *>(dst + gn) =
              make_float4(h[i][j].x + acc[i][j][0], h[i][j].y + acc[i][j][1],
                          h[i][j].z + acc[i][j][2], h[i][j].w + acc[i][j][3]);
      }
    }
  } else if (MODE == EPI_SWIGLU) {
#pragma unroll
    for (int i = 0; i < S::MI; ++i) {
      const int gm = m0 + wm * S::WM + i * 16 + lr;
      bf16_t *dst = reinterpret_cast<bf16_t *>(e.out) + (size_t)gm * e.ldo;
#pragma unroll
      for (int j = 0; j < S::NJ / 2; ++j) {
        const int gn = n0 + wn * (S::WN / 2) + j * 16 + lg * 4;
        float v[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) v[r] = silu(acc[i][j][r]) * acc[i][j + S::NJ / 2][r];
        if (gm < M_eff && gn < N) store4(dst + gn, v[0], v[1], v[2], v[3]);
      }
    }
  } else {  // EPI_QKV: pair P is dims d, d + hd / 2 of head P / (hd / 2)
    const float2 *rope = reinterpret_cast<const float2 *>(e.rope);
#pragma unroll
    for (int i = 0; i < S::MI; ++i) {
      const int gm = m0 + wm * S::WM + i * 16 + lr;
      if (gm >= M_eff) continue;
      const int p = e.pos ? e.pos[gm] : e.pos0 + gm;
      const float2 *row = rope + (size_t)min(max(p - e.rope_base, 0), e.rope_rows - 1) * half;
#pragma unroll
      for (int j = 0; j < S::NJ / 2; ++j) {
        const int P = nt * (BN / 2) + wn * (S::WN / 2) + j * 16 + lg * 4;
        if (P >= N / 2) continue;
        const int d = P & (half - 1);
        const int col = e.n_off + (P >> half_shift) * e.hd + d;
        float lo[4], hi[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          lo[r] = acc[i][j][r];
          hi[r] = acc[i][j + S::NJ / 2][r];
        }
        if (col < e.hq_w + e.kv_w) {
          const float4 c0 = *reinterpret_cast<const float4 *>(row + d);
          const float4 c1 = *reinterpret_cast<const float4 *>(row + d + 2);
          const float cs[4] = {c0.x, c0.z, c1.x, c1.z}, sn[4] = {c0.y, c0.w, c1.y, c1.w};
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const float a = lo[r], b = hi[r];
            lo[r] = a * cs[r] - b * sn[r];
            hi[r] = b * cs[r] + a * sn[r];
          }
        }
        bf16_t *dst;
        const int drow = e.kv_by_pos ? p : gm;
        if (col < e.hq_w)
          dst = reinterpret_cast<bf16_t *>(e.q_out) + (size_t)gm * e.hq_w + col;
        else if (col < e.hq_w + e.kv_w)
          dst = reinterpret_cast<bf16_t *>(e.k_out) + (size_t)drow * e.kv_w + (col - e.hq_w);
        else
          dst = reinterpret_cast<bf16_t *>(e.v_out) + (size_t)drow * e.kv_w +
                (col - e.hq_w - e.kv_w);
        store4(dst, lo[0], lo[1], lo[2], lo[3]);
        store4(dst + half, hi[0], hi[1], hi[2], hi[3]);
      }
    }
  }
}

template <int BM, int BN, int BK, int NST, int MODE>
__global__ __launch_bounds__(256) void k_gemm_few(const bf16_t *__restrict__ A, int lda,
                                                  const bf16_t *__restrict__ B, int ldb, int M,
                                                  int N, int K, int b_rows,
                                                  const int32_t *m_dev, Epi e, int splits,
                                                  float *__restrict__ part) {
  // one LDS object per stage: the compiler then sees that a step's fragment reads and the
  // requests into another stage touch different memory, and does not wait for them
  constexpr int SZ = Few<BM, BN, BK>::STAGE;
#define AKVS_FEW_STAGE(i) \
  __shared__ __attribute__((aligned(16))) bf16_t st##i[NST > i ? SZ : 8];
  AKVS_FEW_STAGE(0) AKVS_FEW_STAGE(1) AKVS_FEW_STAGE(2)
  AKVS_FEW_STAGE(3) AKVS_FEW_STAGE(4) AKVS_FEW_STAGE(5)
#undef AKVS_FEW_STAGE
  bf16_t *const st[6] = {st0, st1, st2, st3, st4, st5};
  const int M_eff = m_dev ? min(M, *m_dev) : M;
  few_body<BM, BN, BK, NST, MODE>(st, A, lda, B, ldb, M, M_eff, N, K, b_rows, e, splits, part);
}

// h[r][c] += part[0][r][c] + part[1][r][c] + ..., in slice order: the second pass of a K split.
__global__ __launch_bounds__(256) void k_few_sum(const float *__restrict__ part, int splits, int M,
                                                 int N, const int32_t *m_dev,
                                                 float *__restrict__ h, int ldo) {
  const int M_eff = m_dev ? min(M, *m_dev) : M;
  const long long i = ((long long)blockIdx.x * 256 + threadIdx.x) * 4;
  if (i >= (long long)M_eff * N) return;
  const int r = (int)(i / N), c = (int)(i - (long long)r * N);
  float *dst = h + (size_t)r * ldo + c;
  const float4 old = *reinterpret_cast<const float4 *>(dst);
  float4 v[kFewMaxSplits];
#pragma unroll
  for (int s = 0; s < kFewMaxSplits; ++s)
    if (s < splits) v[s] = *reinterpret_cast<const float4 *>(part + (size_t)s * M * N + i);
  float4 a = v[0];
#pragma unroll
  for (int s = 1; s < kFewMaxSplits; ++s)
    if (s < splits) {
      a.x += v[s].x; a.y += v[s].y; a.z += v[s].z; a.w += v[s].w;
    }
  *reinterpret_cast<float4 *>(dst) =
      make_float4(old.x + a.x, old.y + a.y, old.z + a.z, old.w + a.w);
}

// The same sum by whole rows, followed by the RMSNorm of the row that the next projection
// reads: out = RMSNorm(h) * gain, with the element order and arithmetic of k_rmsnorm. One block
// per row; saves the norm's own launch and its read of h (203 rows of width 3072: 5.3 + 5.1
// us as two launches, 5.9 here).
constexpr int kSumNormChunks = 4;  // 2048 columns each
__global__ __launch_bounds__(256) void k_few_sum_norm(const float *__restrict__ part, int splits,
                                                      int M, int N, const int32_t *m_dev,
                                                      float *__restrict__ h, int ldo,
                                                      const bf16_t *__restrict__ gain, float eps,
                                                      bf16_t *__restrict__ out) {
  __shared__ float red[4];
  const int r = blockIdx.x;
  if (r >= (m_dev ? min(M, *m_dev) : M)) return;
  float *row = h + (size_t)r * ldo;
  float v[kSumNormChunks][8], g[kSumNormChunks][8];
  float ss = 0.f;
#pragma unroll
  for (int c = 0; c < kSumNormChunks; ++c) {
    const int e = threadIdx.x * 8 + c * 2048;
    if (e >= N) continue;
    load8(gain + e, g[c]);
    load8(row + e, v[c]);
    const float *p = part + (size_t)r * N + e;
    float q[kFewMaxSplits][8];
#pragma unroll
    for (int s = 0; s < kFewMaxSplits; ++s)
      if (s < splits) load8(p + (size_t)s * M * N, q[s]);
#pragma unroll
    for (int s = 1; s < kFewMaxSplits; ++s)
      if (s < splits) {
#pragma unroll
        for (int i = 0; i < 8; ++i) q[0][i] += q[s][i];
      }
#pragma unroll
    for (int i = 0; i < 8; ++i) v[c][i] += q[0][i];
    store8(row + e, v[c]);
  }
#pragma unroll
  for (int c = 0; c < kSumNormChunks; ++c) {
    if (threadIdx.x * 8 + c * 2048 < N) {
#pragma unroll
      for (int i = 0; i < 8; ++i) ss = fmaf(v[c][i], v[c][i], ss);
    }
  }
  ss = wave_sum(ss);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = ss;
  __syncthreads();
  const float tot = (red[0] + red[1]) + (red[2] + red[3]);
  const float inv = 1.0f / sqrtf(tot / (float)N + eps);
#pragma unroll
  for (int c = 0; c < kSumNormChunks; ++c) {
    const int e = threadIdx.x * 8 + c * 2048;
    if (e >= N) continue;
#pragma unroll
    for (int i = 0; i < 8; ++i) v[c][i] = v[c][i] * inv * g[c][i];
    store8(out + (size_t)r * N + e, v[c]);
  }
}

}  // namespace

template <int BM, int BN, int BK, int NST>
static void launch_few_tile(const void *A, int lda, const void *B, int ldb, int M, int N, int K,
                            const int32_t *m_dev, const Epi &e, int splits, float *part,
                            hipStream_t s) {
  const bool swiglu = e.mode == EPI_SWIGLU;
  const int bn_out = swiglu ? BN / 2 : BN;
  const dim3 g((unsigned)(((M + BM - 1) / BM) * ((N + bn_out - 1) / bn_out) * splits)), b(256);
  const bf16_t *a = reinterpret_cast<const bf16_t *>(A), *w = reinterpret_cast<const bf16_t *>(B);
#define AKVS_FEW(MODE_)                                                                      \
  hipLaunchKernelGGL((k_gemm_few<BM, BN, BK, NST, MODE_>), g, b, 0, s, a, lda, w, ldb, M, N, K, \
                     swiglu ? 2 * N : N, m_dev, e, splits, part)
  if (swiglu) AKVS_FEW(EPI_SWIGLU);
  else if (e.mode == EPI_QKV) AKVS_FEW(EPI_QKV);
  else AKVS_FEW(EPI_RESID);
#undef AKVS_FEW
}

hipError_t launch_few(int tile, int splits, const void *A, int lda, const void *B, int ldb, int M,
                      int N, int K, const int32_t *m_dev, const Epi &e, float *part,
                      hipStream_t s) {
#define AKVS_FEW_TILE(T, NST)                                                              \
  case T:                                                                                  \
    launch_few_tile<kFewTiles[T].bm, kFewTiles[T].bn, kFewTiles[T].bk, NST>(               \
        A, lda, B, ldb, M, N, K, m_dev, e, splits, part, s);                               \
    break
  static_assert(kFewCount == 5, "a case per tile");
  switch (tile) {
    AKVS_FEW_TILE(0, 6);
    AKVS_FEW_TILE(1, 4);
    AKVS_FEW_TILE(2, 4);
    AKVS_FEW_TILE(3, 4);
    AKVS_FEW_TILE(4, 4);
    default: return hipErrorInvalidValue;
  }
#undef AKVS_FEW_TILE
  return hipGetLastError();
}

hipError_t launch_few_sum(int splits, int M, int N, const int32_t *m_dev, const Epi &e,
                          const float *part, hipStream_t s, const NormAfter *norm, bool *normed) {
  if (norm && N <= kSumNormChunks * 2048 && N % 8 == 0) {
    hipLaunchKernelGGL(k_few_sum_norm, dim3(M), dim3(256), 0, s, part, splits, M, N, m_dev,
                       reinterpret_cast<float *>(e.out), e.ldo,
                       reinterpret_cast<const bf16_t *>(norm->gain), norm->eps,
                       reinterpret_cast<bf16_t *>(norm->out));
    *normed = true;
    return hipGetLastError();
  }
  const long long n4 = (long long)M * N / 4;
  hipLaunchKernelGGL(k_few_sum, dim3((unsigned)((n4 + 255) / 256)), dim3(256), 0, s, part, splits,
                     M, N, m_dev, reinterpret_cast<float *>(e.out), e.ldo);
  return hipGetLastError();
}

}  // namespace akvs
