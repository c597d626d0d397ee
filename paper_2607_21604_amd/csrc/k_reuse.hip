// Reuse-specific kernels: check-layer divergence, probe selection, per-unit offsets,
// the fused re-rotation + dequantisation + weighted correction, and the cache quantiser.
#include <algorithm>

#include "kernels.h"

namespace akvs {

// Rotate 8 lo/hi pairs (dims e0+i and e0+i+hd/2) by the angles of table row `p`.
__device__ __forceinline__ void rotate8(const float2 *rope_row, int e0, float (&lo)[8],
                                        float (&hi)[8]) {
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const float2 cs = rope_row[e0 + i];
    const float a = lo[i], b = hi[i];
    lo[i] = a * cs.x - b * cs.y;
    hi[i] = b * cs.x + a * cs.y;
  }
}

// The inverse map: rotation by minus the row's angle.
__device__ __forceinline__ void unrotate8(const float2 *rope_row, int e0, float (&lo)[8],
                                          float (&hi)[8]) {
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const float2 cs = rope_row[e0 + i];
    const float a = lo[i], b = hi[i];
    lo[i] = a * cs.x + b * cs.y;
    hi[i] = b * cs.x - a * cs.y;
  }
}

template <typename T>
__host__ __device__ __forceinline__ const T *as(const void *p) {
  return reinterpret_cast<const T *>(p);
}

// ---------------------------------------------------------------------------------------
// Divergence: one wave per token. Work unit = (head, 8 lo/hi pairs) = 16 elements.
template <typename TF>
__global__ void k_divergence(const TF *k_fresh, const TF *v_fresh, CacheLayer cache, int n_tokens,
                             int hkv, int hd, const int32_t *tok_delta, const float2 *rope,
                             int rope_rows, float *d_k, float *d_v) {
  const int lane = threadIdx.x & 63;
  const int t = blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
  if (t >= n_tokens) return;
  const int half = hd >> 1;
  const int units_per_head = half >> 3;
  const int units = hkv * units_per_head;
  int delta = tok_delta ? tok_delta[t] : 0;
  const bool bad = delta < 0 || delta >= rope_rows;
  if (bad) delta = 0;
  const float2 *rrow = rope + (size_t)delta * half;
  float sk = 0.f, sv = 0.f;
  for (int u = lane; u < units; u += 64) {
    const int h = u / units_per_head;
    const int e0 = (u - h * units_per_head) * 8;
    const size_t row = (size_t)t * hkv + h;
    float flo[8], fhi[8], clo[8], chi[8];
    // K
    load8(k_fresh + row * hd + e0, flo);
    load8(k_fresh + row * hd + e0 + half, fhi);
    cache_load8(cache.k, cache.k_meta, cache.dtype, row, hd, e0, clo);
    cache_load8(cache.k, cache.k_meta, cache.dtype, row, hd, e0 + half, chi);
    if (tok_delta) rotate8(rrow, e0, clo, chi);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const float a = flo[i] - clo[i], b = fhi[i] - chi[i];
      sk = fmaf(a, a, sk);
      sk = fmaf(b, b, sk);
    }
    // V
    load8(v_fresh + row * hd + e0, flo);
    load8(v_fresh + row * hd + e0 + half, fhi);
    cache_load8(cache.v, cache.v_meta, cache.dtype, row, hd, e0, clo);
    cache_load8(cache.v, cache.v_meta, cache.dtype, row, hd, e0 + half, chi);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const float a = flo[i] - clo[i], b = fhi[i] - chi[i];
      sv = fmaf(a, a, sv);
      sv = fmaf(b, b, sv);
    }
  }
  sk = wave_sum(sk);
  sv = wave_sum(sv);
  if (lane == 0) {
    d_k[t] = bad ? __builtin_nanf("") : sqrtf(sk);
    d_v[t] = bad ? __builtin_nanf("") : sqrtf(sv);
  }
}

hipError_t launch_divergence(const void *k_fresh, const void *v_fresh, int fresh_dtype,
                             CacheLayer cache, int n_tokens, int hkv, int hd,
                             const int32_t *tok_delta, const float *rope, int rope_rows,
                             float *d_k, float *d_v, hipStream_t s) {
  if (n_tokens == 0) return hipSuccess;
  dim3 g((n_tokens + 3) / 4), b(256);
  const float2 *r = reinterpret_cast<const float2 *>(rope);
  if (fresh_dtype == AKVS_BF16)
    hipLaunchKernelGGL(k_divergence<bf16_t>, g, b, 0, s, as<bf16_t>(k_fresh), as<bf16_t>(v_fresh),
                       cache, n_tokens, hkv, hd, tok_delta, r, rope_rows, d_k, d_v);
  else
    hipLaunchKernelGGL(k_divergence<float>, g, b, 0, s, as<float>(k_fresh), as<float>(v_fresh),
                       cache, n_tokens, hkv, hd, tok_delta, r, rope_rows, d_k, d_v);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------------
// Selection, pass 1: one block per unit. rank(j) = #{t : d_t > d_j or (d_t == d_j, t < j)};
// j is a probe iff rank(j) < b. Then the probe lists (ascending) are compacted by wave 0.
// A unit of n tokens makes n^2 comparisons on one block, so what counts is the length of each
// thread's chain of them: four lanes share a token, each taking four of every sixteen t (one
// 16-byte LDS read per side), and their counts are added inside the quad. 80 units of 200
// tokens: 17.4 us with one thread per token, 8.5 us here. The block has the threads that the
// longest unit needs, at most 1024: 2000 units of 8 tokens took 24 us in blocks of 1024, 15 us
// in blocks of one wave (16.5 in blocks of 256 with a thread per token).
constexpr int SEL_TILE = 1024, SEL_THREADS = 1024, SEL_LANES = 4;

__device__ __forceinline__ int quad_sum(int x) {
  x += __builtin_amdgcn_update_dpp(0, x, 0xB1, 0xf, 0xf, false);  // lane ^ 1
  return x + __builtin_amdgcn_update_dpp(0, x, 0x4E, 0xf, 0xf, false);  // lane ^ 2
}
__device__ __forceinline__ int quad_or(int x) {
  x |= __builtin_amdgcn_update_dpp(0, x, 0xB1, 0xf, 0xf, false);
  return x | __builtin_amdgcn_update_dpp(0, x, 0x4E, 0xf, 0xf, false);
}

__global__ __launch_bounds__(SEL_THREADS) void k_select_rank(
    const float *d_k, const float *d_v, const int4 *meta, int n_chunks, uint32_t flags,
    int32_t *probe_k, int32_t *probe_v, float *w_k, float *w_v, uint8_t *tok_flags,
    int32_t *chunk_rows) {
  __shared__ __attribute__((aligned(16))) float sk[SEL_TILE], sv[SEL_TILE];
  const int c = blockIdx.x;
  const int4 mc = meta[c];             // keys: (start, len, budget, csr offset)
  const int4 mcv = meta[n_chunks + c];  // values: same start and length, own budget
  const int s0 = mc.x, n = mc.y, b = mc.z, off = mc.w, bv_ = mcv.z, offv = mcv.w;
  const int bany = max(b, bv_);
  const bool given = (flags & AKVS_F_GIVEN_PROBES) != 0;
  const bool unit_w = (flags & AKVS_F_UNIT_WEIGHTS) != 0;
  const int part = threadIdx.x & (SEL_LANES - 1);
  for (int jb = 0; jb < n; jb += (int)blockDim.x / SEL_LANES) {
    const int j = jb + (int)threadIdx.x / SEL_LANES;
    const bool valid = j < n;
    float dk = (valid && bany > 0) ? d_k[s0 + j] : 0.f;
    float dv = (valid && bany > 0) ? d_v[s0 + j] : 0.f;
    // a NaN divergence ranks below every number (keeps exactly b probes per side)
    if (dk != dk) dk = -INFINITY;
    if (dv != dv) dv = -INFINITY;
    int rk = 0, rv = 0;
    if (!given && bany > 0) {
      for (int tb = 0; tb < n; tb += SEL_TILE) {
        const int tn = min(SEL_TILE, n - tb), tn16 = (tn + 15) & ~15;
        __syncthreads();
        for (int t = threadIdx.x; t < tn16; t += blockDim.x) {
          // (fill past the unit's end: below or equal to any value, at a later position)
          const float a = t < tn ? d_k[s0 + tb + t] : -INFINITY;
          const float bv = t < tn ? d_v[s0 + tb + t] : -INFINITY;
          sk[t] = (a != a) ? -INFINITY : a;
          sv[t] = (bv != bv) ? -INFINITY : bv;
        }
        __syncthreads();
        const int jr = j - tb;  // position of token j relative to this tile
        for (int t = part * 4; t < tn16; t += 16) {
          const float4 a = *reinterpret_cast<const float4 *>(sk + t);
          const float4 v = *reinterpret_cast<const float4 *>(sv + t);
          rk += (a.x > dk) || (a.x == dk && t < jr);
          rv += (v.x > dv) || (v.x == dv && t < jr);
          rk += (a.y > dk) || (a.y == dk && t + 1 < jr);
          rv += (v.y > dv) || (v.y == dv && t + 1 < jr);
          rk += (a.z > dk) || (a.z == dk && t + 2 < jr);
          rv += (v.z > dv) || (v.z == dv && t + 2 < jr);
          rk += (a.w > dk) || (a.w == dk && t + 3 < jr);
          rv += (v.w > dv) || (v.w == dv && t + 3 < jr);
        }
      }
    }
    rk = quad_sum(rk);
    rv = quad_sum(rv);
    int f = (rk < b ? 1 : 0) | (rv < bv_ ? 2 : 0);
    if (given) {
      f = 0;
      for (int k = part; k < b; k += SEL_LANES) f |= (probe_k[off + k] == s0 + j) ? 1 : 0;
      for (int k = part; k < bv_; k += SEL_LANES) f |= (probe_v[offv + k] == s0 + j) ? 2 : 0;
      f = quad_or(f);
    }
    if (!valid || part) continue;
    tok_flags[s0 + j] = (uint8_t)f;
    // w only multiplies the unit's offset, which is 0 when that side's b == 0
    w_k[s0 + j] = b == 0 ? 0.f : (unit_w ? 1.f : fmaxf(fminf(dk, 1.f), 0.f));
    w_v[s0 + j] = bv_ == 0 ? 0.f : (unit_w ? 1.f : fmaxf(fminf(dv, 1.f), 0.f));
  }
  __syncthreads();
  if (threadIdx.x >= 64) return;
  // wave 0: ascending compaction of the probe lists and the union count
  const int lane = threadIdx.x;
  int ck = 0, cv = 0, cu = 0;
  for (int jb = 0; jb < n; jb += 64) {
    const int j = jb + lane;
    const uint8_t f = j < n ? tok_flags[s0 + j] : 0;
    const uint64_t mk = __ballot((f & 1) != 0);
    const uint64_t mv = __ballot((f & 2) != 0);
    const uint64_t mu = __ballot(f != 0);
    const uint64_t below = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    if (!given) {
      if ((f & 1) && ck + __popcll(mk & below) < b) probe_k[off + ck + __popcll(mk & below)] = s0 + j;
      if ((f & 2) && cv + __popcll(mv & below) < bv_) probe_v[offv + cv + __popcll(mv & below)] = s0 + j;
    }
    ck += __popcll(mk);
    cv += __popcll(mv);
    cu += __popcll(mu);
  }
  if (lane == 0) chunk_rows[c] = cu;
}

// Selection, pass 2: block i < m writes unit i's recomputed rows at its offset in R; block m
// writes the query rows and |R|.
__global__ void k_select_rows(const int4 *meta, int n_chunks, int t_ctx, int q,
                              const uint8_t *tok_flags, const int32_t *chunk_rows, int32_t *rows,
                              int32_t *n_rows, int32_t *fresh_row) {
  const int c = blockIdx.x;
  const int lane = threadIdx.x;  // one wave
  int base = 0;
  for (int i = lane; i < c; i += 64) base += chunk_rows[i];
  for (int o = 32; o > 0; o >>= 1) base += __shfl_xor(base, o, 64);
  if (c == n_chunks) {
    for (int t = lane; t < q; t += 64) {
      rows[base + t] = t_ctx + t;
      fresh_row[t_ctx + t] = base + t;
    }
    if (lane == 0) *n_rows = base + q;
    return;
  }
  const int4 mc = meta[c];
  int cnt = 0;
  for (int jb = 0; jb < mc.y; jb += 64) {
    const int j = jb + lane;
    const uint8_t f = j < mc.y ? tok_flags[mc.x + j] : 0;
    const uint64_t m = __ballot(f != 0);
    const uint64_t below = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    if (j < mc.y) {
      if (f) {
        const int r = base + cnt + __popcll(m & below);
        rows[r] = mc.x + j;
        fresh_row[mc.x + j] = r;
      } else {
        fresh_row[mc.x + j] = -1;
      }
    }
    cnt += __popcll(m);
  }
}

hipError_t launch_select(const float *d_k, const float *d_v, const int32_t *meta, int n_chunks,
                         int len_max, int t_ctx, int q, uint32_t flags, int32_t *probe_k, int32_t *probe_v,
                         float *w_k, float *w_v, uint8_t *tok_flags, int32_t *chunk_rows,
                         int32_t *rows, int32_t *n_rows, int32_t *fresh_row, hipStream_t s) {
  const int4 *m4 = reinterpret_cast<const int4 *>(meta);
  const int threads = std::min(SEL_THREADS, (std::min(len_max, SEL_THREADS) * SEL_LANES + 63) & ~63);
  hipLaunchKernelGGL(k_select_rank, dim3(n_chunks), dim3(threads), 0, s, d_k, d_v, m4, n_chunks,
                     flags, probe_k, probe_v, w_k, w_v, tok_flags, chunk_rows);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_select_rows, dim3(n_chunks + 1), dim3(64), 0, s, m4, n_chunks, t_ctx, q,
                     tok_flags, chunk_rows, rows, n_rows, fresh_row);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------------
// Per-unit offsets. grid = (m units, Hkv heads, 2 sides); block = 256 threads in groups of
// hd/16 lanes. Lane l of a group owns the rotate-half pairs (8l + i, 8l + i + hd/2), i < 8,
// of the block's head, so a group reads one probe's head slice as two contiguous runs.
// Group g sums the probes k = g, g + G, ... of the unit in ascending k (two per step, both
// loads in flight); the G group partials are then added in a fixed order through LDS
// (each half of the block sums G/2 partials in group order, then the two halves), and
// the sum is divided by b_i: a deterministic fp32 order. Splitting by head gives
// m * Hkv * 2 blocks, enough to fill the chip with one short dependent chain each.
constexpr int OFF_THREADS = 256;

template <typename TF>
__global__ __launch_bounds__(OFF_THREADS) void k_chunk_offset(
    const TF *__restrict__ k_fresh, const TF *__restrict__ v_fresh,
    const int32_t *__restrict__ fresh_row, CacheLayer cache, const int4 *__restrict__ meta,
    const int32_t *__restrict__ probe_k, const int32_t *__restrict__ probe_v, uint32_t flags,
    int hkv, int hd, const float2 *__restrict__ rope, int rope_rows, float *mu_k, float *mu_v,
    const int32_t *fresh_base) {
  __shared__ float s_part[OFF_THREADS * 16];  // G partial head slices (G * hd floats)
  __shared__ float s_half[2 * 128];
  const int c = blockIdx.x, h = blockIdx.y, side = blockIdx.z;
  const int n_chunks = gridDim.x;
  const int lps = hd >> 4, G = OFF_THREADS / lps;
  const int g = threadIdx.x / lps, l = threadIdx.x - g * lps;
  const int half = hd >> 1, e0 = 8 * l;
  const size_t rstride = (size_t)hkv * hd, hoff = (size_t)h * hd;
  const int4 mc = meta[side * n_chunks + c];  // this side's table
  const int b = mc.z;
  float *mu = (side == 0 ? mu_k : mu_v) + (size_t)c * rstride + hoff;
  if (b == 0 || (flags & AKVS_F_NO_CORRECTION)) {
    if (threadIdx.x < hd) mu[threadIdx.x] = 0.f;
    return;
  }
  const bool pre_rope = side == 0 && (flags & AKVS_F_PRE_ROPE_OFFSETS);
  const int fresh_off = fresh_base ? *fresh_base : 0;
  const TF *fresh = side == 0 ? k_fresh : v_fresh;
  const void *cb = side == 0 ? cache.k : cache.v;
  const _Float16 *cm = side == 0 ? cache.k_meta : cache.v_meta;
  const int32_t *probes = (side == 0 ? probe_k : probe_v) + mc.w;
  const int delta = (mc.x >= 0 && mc.x < rope_rows) ? mc.x : 0;
  const float2 *rrow = rope + (size_t)delta * half;
  float alo[8], ahi[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) alo[i] = ahi[i] = 0.f;
  for (int k0 = g; k0 < b; k0 += 2 * G) {
    float flo[2][8], fhi[2][8], clo[2][8], chi[2][8];
    int jj[2];
    bool ok[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int k = k0 + u * G;
      int j = k < b ? probes[k] : -1;
      ok[u] = j >= mc.x && j < mc.x + mc.y;  // a token of this unit
      int r = ok[u] ? fresh_row[j] : -1;
      ok[u] = r >= 0;
      if (!ok[u]) {  // contributes nothing: read a valid row, drop it below
        j = mc.x;
        r = 0;
      } else {
        r += fresh_off;
      }
      jj[u] = j;
      const TF *fr = fresh + (size_t)r * rstride + hoff;
      load8(fr + e0, flo[u]);
      load8(fr + e0 + half, fhi[u]);
      const size_t crow = (size_t)j * hkv + h;
      cache_load8(cb, cm, cache.dtype, crow, hd, e0, clo[u]);
      cache_load8(cb, cm, cache.dtype, crow, hd, e0 + half, chi[u]);
    }
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      if (!ok[u]) continue;
      if (side == 0) rotate8(rrow, e0, clo[u], chi[u]);
      float dlo[8], dhi[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        dlo[i] = flo[u][i] - clo[u][i];
        dhi[i] = fhi[u][i] - chi[u][i];
      }
      if (pre_rope) unrotate8(rope + (size_t)min(jj[u], rope_rows - 1) * half, e0, dlo, dhi);
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        alo[i] += dlo[i];
        ahi[i] += dhi[i];
      }
    }
  }
  float *dst = s_part + g * hd;
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    dst[e0 + i] = alo[i];
    dst[e0 + half + i] = ahi[i];
  }
  __syncthreads();
  // thread = (element e, half p): partials p*G/2 .. (p+1)*G/2 - 1 in group order
  const int e = threadIdx.x % hd, p = threadIdx.x / hd;
  const int gh = G >> 1;
  if (p < 2) {
    float t = 0.f;
    for (int w = p * gh; w < (p + 1) * gh; ++w) t += s_part[w * hd + e];
    s_half[p * hd + e] = t;
  }
  __syncthreads();
  if (threadIdx.x < hd) mu[threadIdx.x] = (s_half[threadIdx.x] + s_half[hd + threadIdx.x]) / (float)b;
}

hipError_t launch_chunk_offset(const void *k_fresh, const void *v_fresh, int fresh_dtype,
                               const int32_t *fresh_row, CacheLayer cache, const int32_t *meta,
                               int n_chunks, const int32_t *probe_k, const int32_t *probe_v,
                               uint32_t flags, int hkv, int hd, const float *rope, int rope_rows,
                               float *mu_k, float *mu_v, hipStream_t s,
                               const int32_t *fresh_base) {
  if (hd != 64 && hd != 128) return hipErrorInvalidValue;
  if (n_chunks < 1) return hipSuccess;
  dim3 g(n_chunks, hkv, 2), b(OFF_THREADS);
  const int4 *m4 = reinterpret_cast<const int4 *>(meta);
  const float2 *r = reinterpret_cast<const float2 *>(rope);
  if (fresh_dtype == AKVS_BF16)
    hipLaunchKernelGGL(k_chunk_offset<bf16_t>, g, b, 0, s, as<bf16_t>(k_fresh),
                       as<bf16_t>(v_fresh), fresh_row, cache, m4, probe_k, probe_v, flags, hkv,
                       hd, r, rope_rows, mu_k, mu_v, fresh_base);
  else
    hipLaunchKernelGGL(k_chunk_offset<float>, g, b, 0, s, as<float>(k_fresh),
                       as<float>(v_fresh), fresh_row, cache, m4, probe_k, probe_v, flags, hkv,
                       hd, r, rope_rows, mu_k, mu_v, fresh_base);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------------
// Fused re-rotation + dequantisation + weighted correction (+ fresh rows), K and V.
// Position t < t_ctx: unit token; else query row.
// Unit holding context position t: the last i with meta[i].start <= t.
__device__ __forceinline__ int find_chunk(const int4 *meta, int n_chunks, int t) {
  int lo = 0, hi = n_chunks - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (meta[mid].x <= t) lo = mid; else hi = mid - 1;
  }
  return lo;
}

// find_chunk for a position that is the same in every lane of the wave, in place of a chain of
// log2(n) dependent loads: 128 starts per look, many units first narrowed by looks at 64 evenly
// spaced ones (40 units at 7B width from a 4-bit cache: 9.7 -> 8.9 us; 2000 units of 8 tokens,
// 4 heads of 128: 23.8 -> 21.3 us, but 33.6 where all starts were read through).
__device__ __forceinline__ int find_chunk_wave(const int4 *meta, int n_chunks, int t) {
  const int lane = threadIdx.x & 63;
  int lo = 0, span = n_chunks;  // the unit is one of lo .. lo + span - 1; starts ascend
  while (span > 128) {
    const int step = (span + 63) >> 6, at = lane * step;
    const uint64_t before = __ballot(at < span && meta[lo + min(at, span - 1)].x <= t);
    const int k = max(__popcll(before) - 1, 0) * step;
    lo += k;
    span = min(step, span - k);
  }
  const int x = meta[lo + min(lane, span - 1)].x, y = meta[lo + min(lane + 64, span - 1)].x;
  const int below = __popcll(__ballot(x <= t && lane < span)) +
                    __popcll(__ballot(y <= t && lane + 64 < span));
  return lo + max(below - 1, 0);
}

// Per position: source flags, unit and rotation offset (query rows: fresh, no unit).
struct CorrTok {
  int chunk, delta, fr;
  bool fresh_k, fresh_v;
};

__device__ __forceinline__ CorrTok corr_token(int t, int t_ctx, const uint8_t *tok_flags,
                                              const int32_t *fresh_row, const int32_t *tok_chunk,
                                              const int32_t *tok_delta, const int4 *meta,
                                              int n_chunks, int rope_rows, uint32_t flags,
                                              int fresh_off) {
  CorrTok c{0, 0, -1, true, true};
  const uint8_t f = (t < t_ctx) ? (tok_flags ? tok_flags[t] : 0) : 3;
  if (t < t_ctx) {
    if (tok_chunk) {
      c.chunk = tok_chunk[t];
      c.delta = tok_delta[t];
    } else if (meta) {
      c.chunk = find_chunk(meta, n_chunks, t);
      c.delta = meta[c.chunk].x;
    } else {
      c.delta = tok_delta[t];
    }
    if (c.delta < 0 || c.delta >= rope_rows) c.delta = 0;
    if (c.chunk < 0 || c.chunk >= n_chunks) c.chunk = 0;
  }
  const bool any = f != 0 && (flags & AKVS_F_FRESH_IF_RECOMPUTED);
  c.fresh_k = (f & 1) || any;
  c.fresh_v = (f & 2) || any;
  c.fr = (c.fresh_k || c.fresh_v) ? fresh_row[t] : -1;
  if (c.fr >= 0) c.fr += fresh_off;
  return c;
}

// The rest of one side once its cache values (of a unit token) are in lo / hi: fresh rows
// replace them, reused rows get the re-rotation and the weighted offset.
template <typename TS>
__device__ __forceinline__ void corr_finish(bool fresh, int fr, const TS *__restrict__ fresh_buf,
                                            int hkv, int h, int hd, int e0, const float2 *rrow,
                                            const float *mu, float w, float (&lo)[8],
                                            float (&hi)[8], const float2 *mu_rot = nullptr) {
  const int half = hd >> 1;
  if (fresh) {
    if (fr >= 0) {
      const TS *src = fresh_buf + ((size_t)fr * hkv + h) * hd;
      load8(src + e0, lo);
      load8(src + e0 + half, hi);
    } else {
#pragma unroll
      for (int i = 0; i < 8; ++i) lo[i] = hi[i] = 0.f;
    }
    return;
  }
  if (rrow) rotate8(rrow, e0, lo, hi);
  if (mu) {
    float ml[8], mh[8];
    load8(mu + e0, ml);
    load8(mu + e0 + half, mh);
    if (mu_rot) rotate8(mu_rot, e0, ml, mh);  // a pre-RoPE offset at the token's position
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      lo[i] = fmaf(w, ml[i], lo[i]);
      hi[i] = fmaf(w, mh[i], hi[i]);
    }
  }
}

// Thread = (CORR_T consecutive positions, head h, 8 lo/hi pairs): with Hkv*hd/16 = 64 a
// wave covers whole K and V rows. (Two positions per thread measured slower than one:
// fewer waves in flight outweigh the longer per-lane load queue.)
constexpr int CORR_T = 1;
template <typename TS>
__global__ __launch_bounds__(256) void k_correction(CacheLayer cache, const float *mu_k,
                                                    const float *mu_v, const float *w_k,
                                                    const float *w_v, const uint8_t *tok_flags,
                                                    const TS *__restrict__ k_fresh,
                                                    const TS *__restrict__ v_fresh,
                                                    const int32_t *fresh_row,
                                                    const int32_t *tok_chunk,
                                                    const int32_t *tok_delta, const int4 *meta,
                                                    int n_chunks, int t_ctx, int t_all, int hkv,
                                                    int hd, uint32_t flags, const float2 *rope,
                                                    int rope_rows, TS *__restrict__ k_corr,
                                                    TS *__restrict__ v_corr,
                                                    const int32_t *fresh_base) {
  const int half = hd >> 1;
  const int units = hkv * (half >> 3);
  const int fresh_off = fresh_base ? *fresh_base : 0;
  const long long gid = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  const long long grp = gid / units;
  const int u = (int)(gid - grp * units);
  const int t0 = (int)(grp * CORR_T);
  if (t0 >= t_all) return;
  const int h = u / (half >> 3);
  const int e0 = (u - h * (half >> 3)) * 8;
  float klo[CORR_T][8], khi[CORR_T][8], vlo[CORR_T][8], vhi[CORR_T][8];
#pragma unroll
  for (int i = 0; i < CORR_T; ++i) {
    const int t = min(t0 + i, t_all - 1);  // a repeated last position is computed twice
    const size_t orow = (size_t)t * hkv + h;
    // the cache rows of a unit token are requested before its flags are known, so they
    // arrive with the bookkeeping (wasted for the recomputed tokens, whose rows are fresh)
    if (t < t_ctx) {
      cache_load8(cache.k, cache.k_meta, cache.dtype, orow, hd, e0, klo[i]);
      cache_load8(cache.k, cache.k_meta, cache.dtype, orow, hd, e0 + half, khi[i]);
      cache_load8(cache.v, cache.v_meta, cache.dtype, orow, hd, e0, vlo[i]);
      cache_load8(cache.v, cache.v_meta, cache.dtype, orow, hd, e0 + half, vhi[i]);
    }
    const CorrTok c = corr_token(t, t_ctx, tok_flags, fresh_row, tok_chunk, tok_delta, meta,
                                 n_chunks, rope_rows, flags, fresh_off);
    const size_t mo = (size_t)c.chunk * hkv * hd + (size_t)h * hd;
    const float2 *mu_rot = (flags & AKVS_F_PRE_ROPE_OFFSETS)
                               ? rope + (size_t)min(t, rope_rows - 1) * half
                               : nullptr;
    // the weights cover the unit tokens only ([t_ctx]); query rows are always fresh
    const bool unit_tok = t < t_ctx;
    corr_finish(c.fresh_k, c.fr, k_fresh, hkv, h, hd, e0, rope + (size_t)c.delta * half,
                mu_k ? mu_k + mo : nullptr, (mu_k && unit_tok) ? w_k[t] : 0.f, klo[i], khi[i],
                mu_rot);
    corr_finish(c.fresh_v, c.fr, v_fresh, hkv, h, hd, e0, nullptr, mu_v ? mu_v + mo : nullptr,
                (mu_v && unit_tok) ? w_v[t] : 0.f, vlo[i], vhi[i]);
  }
#pragma unroll
  for (int i = 0; i < CORR_T; ++i) {
    const int t = t0 + i;
    if (t >= t_all) break;
    const size_t orow = (size_t)t * hkv + h;
    TS *ko = k_corr + orow * hd;
    TS *vo = v_corr + orow * hd;
    store8(ko + e0, klo[i]);
    store8(ko + e0 + half, khi[i]);
    store8(vo + e0, vlo[i]);
    store8(vo + e0 + half, vhi[i]);
  }
}

// The correction for bf16 and quantised unit caches. A thread serves one side (K or V)
// of a position's 16-element pair group, in few enough registers that eight waves fit on
// each SIMD, and reads only the rows it uses: the token's bookkeeping first, then either
// its cache row (reused) or its fresh row (recomputed), so the cache rows of recomputed
// tokens are never fetched. Same arithmetic as k_correction (bitwise the same results).
// k_correction holds both sides' float rows across the bookkeeping loads in 85 registers
// (five waves per SIMD) and moved 3.6 of the 5.2 TB/s that a plain kernel of the same access
// pattern reaches at the 32B-class size (131 MB per layer).
__device__ __forceinline__ void unpack_bf8(u32x4_t w, float (&o)[8]) {
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    o[2 * i] = __uint_as_float(w[i] << 16);
    o[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
  }
}
// SIMPLE: the reuse call's own case (bf16 unit cache, per-token unit and shift tables, every
// table present and valid, a fresh row for every recomputed position, neither
// AKVS_F_PRE_ROPE_OFFSETS nor AKVS_F_FRESH_IF_RECOMPUTED, no fresh-row base), with those
// checks taken out at compile time.
template <typename TS, bool SIMPLE>
__global__ __launch_bounds__(256) void k_correction_bf(CacheLayer cache, const float *mu_k,
                                                       const float *mu_v, const float *w_k,
                                                       const float *w_v, const uint8_t *tok_flags,
                                                       const TS *__restrict__ k_fresh,
                                                       const TS *__restrict__ v_fresh,
                                                       const int32_t *fresh_row,
                                                       const int32_t *tok_chunk,
                                                       const int32_t *tok_delta, const int4 *meta,
                                                       int n_chunks, int t_ctx, int t_all,
                                                       int hkv, int hd, uint32_t flags,
                                                       const float2 *rope, int rope_rows,
                                                       TS *__restrict__ k_corr,
                                                       TS *__restrict__ v_corr,
                                                       const int32_t *fresh_base) {
  const int half = hd >> 1;
  const int side_units = hkv * (half >> 3);  // threads per side and position
  const int fresh_off = (!SIMPLE && fresh_base) ? *fresh_base : 0;
  const long long gid = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  const long long grp = gid / (2 * side_units);
  int u = (int)(gid - grp * 2 * side_units);
  const int t = (int)grp;
  if (t >= t_all) return;
  const bool vside = u >= side_units;
  if (vside) u -= side_units;
  const int h = u / (half >> 3);
  const int e0 = (u - h * (half >> 3)) * 8;
  const size_t orow = (size_t)t * hkv + h;
  const bool unit_tok = t < t_ctx;
  // bookkeeping first, all of it at once (the row index of a recomputed position is read
  // whether or not the position is one), then only the rows this side uses: the cache row
  // of a reused token or the fresh row of a recomputed one
  const uint8_t f = unit_tok ? ((SIMPLE || tok_flags) ? tok_flags[t] : 0) : 3;
  int fr = (SIMPLE || fresh_row) ? fresh_row[t] : -1;
  int chunk = 0, delta = 0;
  if (unit_tok) {
    if (SIMPLE || tok_chunk) {
      chunk = tok_chunk[t];
      delta = tok_delta[t];
    } else if (meta) {
      // whole waves per position (all of the wave's lanes are here then): search together
      chunk = (2 * side_units) % 64 == 0 ? find_chunk_wave(meta, n_chunks, t)
                                         : find_chunk(meta, n_chunks, t);
      delta = meta[chunk].x;
    } else {
      delta = tok_delta[t];
    }
    if (delta < 0 || delta >= rope_rows) delta = 0;
    if (!SIMPLE && (chunk < 0 || chunk >= n_chunks)) chunk = 0;
  }
  const bool any = !SIMPLE && f != 0 && (flags & AKVS_F_FRESH_IF_RECOMPUTED);
  const bool fresh = (vside ? (f & 2) : (f & 1)) || any;
  if (!SIMPLE && fr >= 0) fr += fresh_off;
  float lo[8], hi[8];
  if (fresh) {
    if (SIMPLE || fr >= 0) {  // (the reuse call gives every recomputed position its row)
      const TS *src = (vside ? v_fresh : k_fresh) + ((size_t)max(fr, 0) * hkv + h) * hd;
      load8(src + e0, lo);
      load8(src + e0 + half, hi);
    } else {
#pragma unroll
      for (int i = 0; i < 8; ++i) lo[i] = hi[i] = 0.f;
    }
  } else {
    if (SIMPLE || cache.dtype == AKVS_BF16) {
      const bf16_t *cb = reinterpret_cast<const bf16_t *>(vside ? cache.v : cache.k) + orow * hd;
      unpack_bf8(__builtin_nontemporal_load(reinterpret_cast<const u32x4_t *>(cb + e0)), lo);
      unpack_bf8(__builtin_nontemporal_load(reinterpret_cast<const u32x4_t *>(cb + e0 + half)),
                 hi);
    } else {  // quantised unit caches: codes and their group's scale / zero
      const void *cb = vside ? cache.v : cache.k;
      const _Float16 *cm = vside ? cache.v_meta : cache.k_meta;
      cache_load8(cb, cm, cache.dtype, orow, hd, e0, lo);
      cache_load8(cb, cm, cache.dtype, orow, hd, e0 + half, hi);
    }
    const float *mu = vside ? mu_v : mu_k;
    const size_t mo = (size_t)chunk * hkv * hd + (size_t)h * hd;
    const float w = (SIMPLE || mu) ? (vside ? w_v[t] : w_k[t]) : 0.f;
    if (!vside) {
      const float2 *mu_rot = (!SIMPLE && (flags & AKVS_F_PRE_ROPE_OFFSETS))
                                 ? rope + (size_t)min(t, rope_rows - 1) * half
                                 : nullptr;
      corr_finish(false, -1, k_fresh, hkv, h, hd, e0, rope + (size_t)delta * half,
                  (SIMPLE || mu) ? mu + mo : nullptr, w, lo, hi, mu_rot);
    } else {
      corr_finish(false, -1, v_fresh, hkv, h, hd, e0, nullptr, (SIMPLE || mu) ? mu + mo : nullptr,
                  w, lo, hi);
    }
  }
  // streaming stores: the corrected rows are written once here (0.58 -> 0.64 of the HBM
  // peak at the 32B-class size, against ordinary stores)
  TS *o = (vside ? v_corr : k_corr) + orow * hd;
  if constexpr (sizeof(TS) == 2) {
    u32x4_t a, b;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      a[i] = pack_bf2(lo[2 * i], lo[2 * i + 1]);
      b[i] = pack_bf2(hi[2 * i], hi[2 * i + 1]);
    }
    __builtin_nontemporal_store(a, reinterpret_cast<u32x4_t *>(o + e0));
    __builtin_nontemporal_store(b, reinterpret_cast<u32x4_t *>(o + e0 + half));
  } else {
    store8(o + e0, lo);
    store8(o + e0 + half, hi);
  }
}

hipError_t launch_correction(CacheLayer cache, const float *mu_k, const float *mu_v,
                             const float *w_k, const float *w_v, const uint8_t *tok_flags,
                             const void *k_fresh, const void *v_fresh, const int32_t *fresh_row,
                             const int32_t *tok_chunk, const int32_t *tok_delta,
                             const int32_t *meta, int n_chunks, int t_ctx,
                             int t_all, int hkv, int hd, uint32_t flags, const float *rope,
                             int rope_rows, void *k_corr, void *v_corr, int out_dtype,
                             hipStream_t s,
                             const int32_t *fresh_base) {
  const int4 *m4 = reinterpret_cast<const int4 *>(meta);
  const long long threads = ((long long)t_all + CORR_T - 1) / CORR_T * hkv * (hd / 16);
  if (threads == 0) return hipSuccess;
  dim3 g((unsigned)((threads + 255) / 256)), b(256);
  const float2 *r = reinterpret_cast<const float2 *>(rope);
  if (cache.dtype != AKVS_F32 && CORR_T == 1) {
    const long long thr2 = (long long)t_all * 2 * hkv * (hd / 16);
    g = dim3((unsigned)((thr2 + 255) / 256));
    const bool simple = cache.dtype == AKVS_BF16 && tok_flags && fresh_row && tok_chunk &&
                        tok_delta && mu_k && mu_v && w_k && w_v && !fresh_base &&
                        !(flags & (AKVS_F_PRE_ROPE_OFFSETS | AKVS_F_FRESH_IF_RECOMPUTED));
    if (out_dtype == AKVS_BF16 && simple)
      hipLaunchKernelGGL((k_correction_bf<bf16_t, true>), g, b, 0, s, cache, mu_k, mu_v, w_k, w_v,
                         tok_flags, as<bf16_t>(k_fresh), as<bf16_t>(v_fresh), fresh_row,
                         tok_chunk, tok_delta, m4, n_chunks, t_ctx, t_all, hkv, hd, flags, r,
                         rope_rows, reinterpret_cast<bf16_t *>(k_corr),
                         reinterpret_cast<bf16_t *>(v_corr), fresh_base);
    else if (out_dtype == AKVS_BF16)
      hipLaunchKernelGGL((k_correction_bf<bf16_t, false>), g, b, 0, s, cache, mu_k, mu_v, w_k, w_v,
                         tok_flags, as<bf16_t>(k_fresh), as<bf16_t>(v_fresh), fresh_row,
                         tok_chunk, tok_delta, m4, n_chunks, t_ctx, t_all, hkv, hd, flags, r,
                         rope_rows, reinterpret_cast<bf16_t *>(k_corr),
                         reinterpret_cast<bf16_t *>(v_corr), fresh_base);
    else
      hipLaunchKernelGGL((k_correction_bf<float, false>), g, b, 0, s, cache, mu_k, mu_v, w_k, w_v,
                         tok_flags, as<float>(k_fresh), as<float>(v_fresh), fresh_row, tok_chunk,
                         tok_delta, m4, n_chunks, t_ctx, t_all, hkv, hd, flags, r, rope_rows,
                         reinterpret_cast<float *>(k_corr), reinterpret_cast<float *>(v_corr),
                         fresh_base);
    return hipGetLastError();
  }
  if (out_dtype == AKVS_BF16)
    hipLaunchKernelGGL(k_correction<bf16_t>, g, b, 0, s, cache, mu_k, mu_v, w_k, w_v, tok_flags,
                       as<bf16_t>(k_fresh), as<bf16_t>(v_fresh), fresh_row, tok_chunk, tok_delta,
                       m4, n_chunks, t_ctx, t_all, hkv, hd, flags, r, rope_rows,
                       reinterpret_cast<bf16_t *>(k_corr), reinterpret_cast<bf16_t *>(v_corr),
                       fresh_base);
  else
    hipLaunchKernelGGL(k_correction<float>, g, b, 0, s, cache, mu_k, mu_v, w_k, w_v, tok_flags,
                       as<float>(k_fresh), as<float>(v_fresh), fresh_row, tok_chunk, tok_delta,
                       m4, n_chunks, t_ctx, t_all, hkv, hd, flags, r, rope_rows,
                       reinterpret_cast<float *>(k_corr), reinterpret_cast<float *>(v_corr),
                       fresh_base);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------------
// Quantiser. Memory-bound by its bytes (read x once, write codes and metadata), so a lane
// takes 8 consecutive elements (16-byte loads of bf16) and a group of 64 sits on 8 lanes of
// one DPP row: its minimum and maximum are three DPP steps. A thread has QZ_U octets in
// flight.
// The codes are defined by IEEE quotients (x - zero) / scale, about ten VALU instructions
// each, which alone would take longer than the memory. The quotient is formed as a product
// with the group's reciprocal (off by at most 2 ulp); only where that lies so near a rounding
// boundary of the code that the two could round apart is the division made. The codes are
// the same, bit for bit.
// 28 x 8000 tokens of 4 heads of 128 (115 M bf16 elements) to 4 bits: 455 us with one element
// per lane, divisions and wave-wide reductions (k_quantize_any below), 60 us here
// (4.9 TB/s, what a large copy reaches).
constexpr int QZ_U = 4;

template <int CTRL>
__device__ __forceinline__ float dpp_f32(float x) {
  return __int_as_float(
      __builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xf, 0xf, false));
}
__device__ __forceinline__ float oct_max(float x) {  // over aligned groups of 8 lanes
  x = fmaxf(x, dpp_f32<0xB1>(x));    // lane ^ 1
  x = fmaxf(x, dpp_f32<0x4E>(x));    // lane ^ 2
  return fmaxf(x, dpp_f32<0x141>(x));  // the two quads of the 8 lanes
}
__device__ __forceinline__ float oct_min(float x) {
  x = fminf(x, dpp_f32<0xB1>(x));
  x = fminf(x, dpp_f32<0x4E>(x));
  return fminf(x, dpp_f32<0x141>(x));
}

// Quotient rounded to an integer code 0..levels (rne), from v = x - zero.
__device__ __forceinline__ uint32_t int_code(float tq, float levels) {
  return (uint32_t)(int)fminf(fmaxf(rintf(tq), 0.f), levels);
}

template <typename TX, int BITS>
__global__ __launch_bounds__(256) void k_quantize(const TX *__restrict__ x, long long octets,
                                                  uint8_t *__restrict__ codes,
                                                  uint32_t *__restrict__ meta) {
  const long long o0 = (long long)blockIdx.x * (256 * QZ_U) + threadIdx.x;
  float v[QZ_U][8];
#pragma unroll
  for (int u = 0; u < QZ_U; ++u)  // octets past the end re-read the last one
    load8(x + min(o0 + u * 256, octets - 1) * 8, v[u]);
#pragma unroll
  for (int u = 0; u < QZ_U; ++u) {
    const long long o = o0 + u * 256;
    if (o >= octets) break;  // whole groups: octets is a multiple of 8
    float lo = v[u][0], hi = v[u][0];
    if (BITS == 8) {
      hi = fabsf(hi);
#pragma unroll
      for (int i = 1; i < 8; ++i) hi = fmaxf(hi, fabsf(v[u][i]));
      hi = oct_max(hi);
    } else {
#pragma unroll
      for (int i = 1; i < 8; ++i) {
        lo = fminf(lo, v[u][i]);
        hi = fmaxf(hi, v[u][i]);
      }
      lo = oct_min(lo);
      hi = oct_max(hi);
    }
    constexpr float levels = BITS == 8 ? 448.f : (float)((1 << BITS) - 1);
    const _Float16 z16 = BITS == 8 ? (_Float16)0.f : (_Float16)lo;
    const _Float16 s16 = (_Float16)__fdiv_rn(BITS == 8 ? hi : hi - lo, levels);
    const float scale = (float)s16, zero = (float)z16;
    const float rs = __fdiv_rn(1.0f, scale);
    uint32_t w[BITS == 8 ? 2 : 1] = {};
    if (scale != 0.f) {
      float t[8];
      bool near = false;
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        if (BITS == 8) {
          t[i] = v[u][i] * rs;
          // half-way points of E4M3: 4 significant bits, steps of 2^-9 below 2^-6
          const float a = fabsf(t[i]);
          near |= a < 0.015625f
                      ? fabsf(__builtin_amdgcn_fractf(a * 512.f) - 0.5f) < 1e-4f
                      : ((__float_as_uint(a) + 16u - 0x80000u) & 0xfffffu) <= 32u;
        } else {
          t[i] = (v[u][i] - zero) * rs;
          near |= fabsf(__builtin_amdgcn_fractf(t[i]) - 0.5f) < 2e-5f;
        }
      }
      if (near) {
#pragma unroll
        for (int i = 0; i < 8; ++i)
          t[i] = __fdiv_rn(BITS == 8 ? v[u][i] : v[u][i] - zero, scale);
      }
      if (BITS == 8) {
#pragma unroll
        for (int i = 0; i < 8; ++i) t[i] = fminf(fmaxf(t[i], -448.f), 448.f);
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          int p = __builtin_amdgcn_cvt_pk_fp8_f32(t[4 * h], t[4 * h + 1], 0, false);
          w[h] = (uint32_t)__builtin_amdgcn_cvt_pk_fp8_f32(t[4 * h + 2], t[4 * h + 3], p, true);
        }
      } else {
#pragma unroll
        for (int i = 0; i < 8; ++i) w[0] |= int_code(t[i], levels) << (BITS * i);
      }
    }
    uint8_t *c = codes + o * BITS;
    if constexpr (BITS == 8)
      *reinterpret_cast<uint2 *>(c) = make_uint2(w[0], w[1]);
    else if constexpr (BITS == 4)
      *reinterpret_cast<uint32_t *>(c) = w[0];
    else
      *reinterpret_cast<uint16_t *>(c) = (uint16_t)w[0];
    if ((threadIdx.x & 7) == 0)
      meta[o >> 3] = (uint32_t)__builtin_bit_cast(uint16_t, s16) |
                     ((uint32_t)__builtin_bit_cast(uint16_t, z16) << 16);
  }
}

// The same with one wave per (row, group of 64); lane = element: for operands that are not aligned
// for k_quantize's loads and stores, and for few groups, which k_quantize leaves on few
// threads (64 elements each, in turn).
template <typename TX>
__global__ void k_quantize_any(const TX *x, int n_rows, int hd, int bits, uint8_t *codes,
                               _Float16 *meta) {
  const int lane = threadIdx.x & 63;
  const int groups = hd / 64;
  const long long gid = (long long)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
  if (gid >= (long long)n_rows * groups) return;
  const long long row = gid / groups;
  const int grp = (int)(gid - row * groups);
  const float v = load1(x + row * hd + grp * 64 + lane);
  if (bits == 8) {  // E4M3: symmetric, one fp16 scale per group
    const float amax = wave_max(fabsf(v));
    const _Float16 s16 = (_Float16)__fdiv_rn(amax, 448.f);
    const float scale = (float)s16;
    int code = 0;
    if (scale != 0.f) {
      const float t = fminf(fmaxf(__fdiv_rn(v, scale), -448.f), 448.f);
      code = __builtin_amdgcn_cvt_pk_fp8_f32(t, 0.f, 0, false) & 0xff;
    }
    codes[row * hd + grp * 64 + lane] = (uint8_t)code;
    if (lane == 0) {
      meta[2 * gid] = s16;
      meta[2 * gid + 1] = (_Float16)0.f;
    }
    return;
  }
  const float mn = wave_min(v), mx = wave_max(v);
  const float levels = (float)((1 << bits) - 1);
  const _Float16 z16 = (_Float16)mn;
  const _Float16 s16 = (_Float16)__fdiv_rn(mx - mn, levels);
  const float zero = (float)z16, scale = (float)s16;
  int code = 0;
  if (scale != 0.f) {
    const float tq = rintf(__fdiv_rn(v - zero, scale));
    code = (int)fminf(fmaxf(tq, 0.f), levels);
  }
  const int per = 8 / bits;
  int packed = code << (bits * (lane % per));
  for (int o = 1; o < per; o <<= 1) packed |= __shfl_xor(packed, o, 64);
  if (lane % per == 0) codes[row * (hd * bits / 8) + grp * (64 * bits / 8) + lane / per] = (uint8_t)packed;
  if (lane == 0) {
    meta[2 * gid] = s16;
    meta[2 * gid + 1] = z16;
  }
}

template <typename TX>
static void quantize_wide(const void *x, long long octets, int bits, uint8_t *codes,
                          _Float16 *meta, hipStream_t s) {
  const dim3 g((unsigned)((octets + 256 * QZ_U - 1) / (256 * QZ_U))), b(256);
  uint32_t *m = reinterpret_cast<uint32_t *>(meta);
  if (bits == 8)
    hipLaunchKernelGGL((k_quantize<TX, 8>), g, b, 0, s, as<TX>(x), octets, codes, m);
  else if (bits == 4)
    hipLaunchKernelGGL((k_quantize<TX, 4>), g, b, 0, s, as<TX>(x), octets, codes, m);
  else
    hipLaunchKernelGGL((k_quantize<TX, 2>), g, b, 0, s, as<TX>(x), octets, codes, m);
}

hipError_t launch_quantize(const void *x, int x_dtype, int n_rows, int hd, int bits,
                           uint8_t *codes, _Float16 *meta, hipStream_t s) {
  const long long waves = (long long)n_rows * (hd / 64);
  if (waves == 0) return hipSuccess;
  // rows and groups are dense: octet o holds elements 8o..8o+7 and codes byte o * bits on.
  // Groups from which k_quantize is the faster one (bf16, k_quantize and k_quantize_any: 4 bits,
  // 2000 groups 4.3 and 3.9 us, 8000 4.5 and 5.0; 8 bits, whose codes take three times the
  // arithmetic, 8000 6.0 and 4.4, 32000 6.2 and 8.6).
  const bool many = waves > (bits == 8 ? 16384 : 4096);
  const bool wide = many && (reinterpret_cast<uintptr_t>(x) & 15u) == 0 &&
                    (reinterpret_cast<uintptr_t>(codes) & 7u) == 0 &&
                    (reinterpret_cast<uintptr_t>(meta) & 3u) == 0;
  if (wide) {
    if (x_dtype == AKVS_BF16) quantize_wide<bf16_t>(x, waves * 8, bits, codes, meta, s);
    else quantize_wide<float>(x, waves * 8, bits, codes, meta, s);
    return hipGetLastError();
  }
  dim3 g((unsigned)((waves + 3) / 4)), b(256);
  if (x_dtype == AKVS_BF16)
    hipLaunchKernelGGL(k_quantize_any<bf16_t>, g, b, 0, s, as<bf16_t>(x), n_rows, hd, bits, codes,
                       meta);
  else
    hipLaunchKernelGGL(k_quantize_any<float>, g, b, 0, s, as<float>(x), n_rows, hd, bits, codes,
                       meta);
  return hipGetLastError();
}

}  // namespace akvs
