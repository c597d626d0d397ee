// Attention of (sparse, position-sorted) query rows over a causal key range.
//
// bf16 path: one block = a group of the query heads that read one KV head, over a tile of
// rows; each wave owns 32 rows of one query head. Keys stream through LDS in tiles of 64
// (K and V row-major), shared by every wave of the block. Scores are computed
// transposed, S^T = K Q^T, with MFMA 32x32x16 bf16: each lane then holds 16 scores of ONE
// query row (the other 16 of that row's 32 keys sit in lane ^ 32), and the probabilities
// already sit in the operand layout of the second product O^T = V^T P^T (the pairing of
// the 16 contraction slots with keys is a fixed permutation applied to both operands).
// The running maximum is only raised when a score exceeds it by more than 2^8, which
// keeps the rescaling of O off the common path while p = 2^(s - m) stays <= 256.
// Row tiles are launched longest-first (rows are sorted by position, so later tiles
// see more keys).
#include "kernels.h"

namespace akvs {

// V tile: 64 keys x hd, row-major as in memory, rows padded by 32 elements (64 bytes, a
// 16-bank shift per row). The P.V operand wants, per lane, 8 keys of ONE head dim; gfx950's
// transposing LDS read (ds_read_b64_tr_b16) delivers that from row-major rows: within
// each 16-lane group, lane j receives element j % 4 of the 8-byte chunk addressed by lane
// 4k + j / 4, for k = 0..3. So source lane s of a group points at key row +s/4, head dims
// 4*(s%4)..+3 of the group's 16 dims, and each lane gets 4 consecutive keys of its dim per
// read. Against the transposed V^T staging it replaced (VALU byte shuffles and 8-byte LDS
// stores in the loading waves), same bits: 1-4 % faster on the 32B, 7B and 3B shapes
// (standalone timing, not in the repository). A 32-lane read phase touches 4 rows x 64
// bytes, at 16-bank offsets: no conflicts.

// Block shape: 32-row waves. With about 250 VGPRs a compute unit holds eight waves, so blocks
// of 8 waves (one per unit) or 4 (two per unit) use every SIMD evenly; the first four waves
// stage the K / V tiles.
//  - 256 rows (8 waves sharing each K / V tile) when that still makes 512 blocks (32B probe
//    layer, 5527 rows over 16128 keys: 1094 us against 1383 us for blocks that grouped the
//    five query heads of a KV head over 32 rows, whose 5 waves leave SIMDs unevenly loaded);
//  - else 128 rows (4 waves) per block; when those make fewer than 512 blocks the key range
//    is split as well (see attn_splits). (32B probe layer at r = 1/10, 3050 rows: 664 us
//    against 751 us for the five-head 32-row blocks; the 3B full prefill measured the same
//    with three-head 64-row blocks.)
static inline int attn_waves(int rows, int hq) {
  return (long long)((rows + 255) / 256) * hq >= 512 ? 8 : 4;
}

// Short contexts run whole: a piece of the key range costs about 1.6 us per 64 keys, a split
// about 8 us more for its fixed part and the merge. Square calls (a full prefill) of 203, 384
// and 768 keys took 14, 19 and 25 us split (plan not counted), 11, 15 and 22 us whole; 64
// rows over 512 keys 12 us split, 18 us whole, hence the two bounds.
static inline bool attn_whole(int rows, int n_keys) {
  return n_keys <= 384 || (n_keys <= 768 && 2LL * rows >= n_keys);
}

// Planned split (launch_attention_plan, then launch_attention with the plan): for calls
// over few position-sorted rows, whose tiles leave block slots idle or end at very
// different times, the key range of each tile is cut into nearly equal pieces sized so
// that every block slot of the chip gets about the same work, and the pieces go out
// longest first. Block shape and item budget from the row bound (host):
//  - 4-wave 128-row blocks (two per CU) in one round, where the 128-row tiles fill at most
//    3/4 of the round's items (slots / heads) and are at least 3;
//  - else 8-wave 256-row blocks (one per CU): one round where their tiles fill at most
//    half of it, two rounds where they fill less than two;
//  - else no plan (the tiles alone fill the chip; launch_attention's own split applies).
// Measured on the 3B-class probe layers (1441 / 865 / 300 / 166 rows over 4516 keys):
// 75 / 53 / 38 / 35 us against 92 / 60 / 47 / 37 us; 7B-class (2802 / 1513 rows over
// 8128 keys) 199 / 129 against 215 / 155 us; the query rows of the last layer (64 over
// 4516 keys, 128 over 16128) 27 / 69 against 28 / 79 us. With one round for the 3B
// layers at 1992 rows over 4516 keys the 128-row blocks took 101 us against 89 us for two
// rounds of 256-row blocks, which is what sets the 3/4 bound (standalone harness, not in
// the repository).
// Few rows are also packed: the G query heads of a KV head over the same rows form one list
// of G x rows (row, head) pairs, row by row, so that a tile's 32-row waves are full and a K / V
// tile is read once for more of them. Taken where it leaves at least a tenth less padding,
// and the tiles are many or long (else it only leaves fewer blocks: 64 rows over 1000 keys
// 21 us packed, 18 us not). Up to 16 pieces per tile where few rows see many keys. Whole calls
// with their plan, without both -> with: 3B heads over 16000 keys 9 / 64 / 159 / 400 rows
// 51 / 65 / 70 / 87 -> 37 / 49 / 54 / 78 us, 32B heads 62 / 81 / 87 / 145 -> 38 / 52 / 61 / 101;
// 400 rows over 2500 and 5000 keys, 3B 36 and 48 -> 33 and 41; 159 rows over 1000 keys 23 -> 21.
// (16 pieces at 250 rows of the 32B heads, or under 2500 keys, cost 2 to 5 % more than 8.)
// Between 4096 and 6144 keys both are a matter of how full the chip is (timed at 4200 to 7000 keys,
// five head counts, 1 to 192 rows): 17 to 128 rows are packed there only where the heads one by
// one would make more than two rounds of blocks (64 rows over 5000 keys, 40 query heads: 35.7
// -> 35.0 us packed, but 24 heads 29.9 -> 32.1), and more than 128 rows take 16 pieces only
// where 8 leave compute units idle (159 rows over 4500 keys: 24 heads 32.3 us with 8, 34.9 with
// 16; 14 heads of 64 26.9 and 25.6).
struct AttnEqShape {
  int rb, budget, max_pc;
  bool use;
  int pack;  // query heads listed together: 1, or G
};
constexpr int kAttnMaxPieces = 8, kAttnFewPieces = 16;  // the merge's all-at-once path
constexpr int kAttnLongKeys = 4096, kAttnVeryLongKeys = 6144;
static inline int attn_max_pieces(int rows, int n_keys) {
  return rows <= 192 && n_keys > kAttnLongKeys ? kAttnFewPieces : kAttnMaxPieces;
}

// rb and budget for `rows` rows (or pairs) of `lists` row lists; false where the tiles fill
// the chip or the plan's 64 tiles do not cover them.
static inline bool attn_eq_blocks(long long rows, int lists, int cus, int *rb, int *budget) {
  const int p128 = 2 * cus / lists, p256 = cus / lists;
  const long long nt128 = (rows + 127) / 128, nt256 = (rows + 255) / 256;
  if (nt128 >= 3 && 4 * nt128 <= 3 * p128) {
    *rb = 128;
    *budget = p128;
  } else if (p256 >= 1 && 2 * nt256 <= p256) {
    *rb = 256;
    *budget = p256;
  } else if (p256 >= 1 && nt256 < 2 * p256) {
    *rb = 256;
    *budget = 2 * p256;
  } else {
    return false;
  }
  return (rows + *rb - 1) / *rb <= 64;
}

static inline AttnEqShape attn_eq_shape(int rows, int hq, int hkv, int n_keys, int hd, int dtype,
                                        long long part_rows, int cus) {
  AttnEqShape e{0, 0, 0, false, 1};
  if (dtype != AKVS_BF16 || rows <= 0 || hq <= 0 || (hd != 64 && hd != 128)) return e;
  if (attn_whole(rows, n_keys)) return e;
  if (!attn_eq_blocks(rows, hq, cus, &e.rb, &e.budget)) return e;
  const int G = hq / hkv;
  int rb, budget;
  const bool packs = rows > 128 || n_keys > kAttnVeryLongKeys ||
                     (n_keys > kAttnLongKeys && (rows <= 16 || kAttnFewPieces * hq > 2 * cus));
  if (G > 1 && packs &&
      attn_eq_blocks((long long)rows * G, hkv, cus, &rb, &budget)) {
    const long long single = (long long)((rows + e.rb - 1) / e.rb) * e.rb * hq;
    const long long packed = ((long long)rows * G + rb - 1) / rb * rb * hkv;
    if (10 * packed <= 9 * single) {
      e.rb = rb;
      e.budget = budget;
      e.pack = G;
    }
  }
  int most = attn_max_pieces(rows, n_keys);
  if (rows > 128 && n_keys <= kAttnVeryLongKeys) {
    const long long tiles = ((long long)rows * e.pack + e.rb - 1) / e.rb * (hq / e.pack);
    if (tiles * kAttnMaxPieces >= cus) most = kAttnMaxPieces;
  }
  e.max_pc = (int)std::min<long long>(most, part_rows / rows);
  e.use = e.max_pc >= 2;
  return e;
}

// The plan (one wave): tile t of rb rows sees kt_t = ceil(keys_t / 64) key tiles, keys_t
// its last row's position + 1. It is cut into c_t = ceil(kt_t / L) ranges of nearly equal
// length, L >= 2 the smallest with sum_t c_t <= max(tiles, budget) and c_t <= max_pc. (A piece of
// one key tile costs more than it saves: 159 rows of 40 / 8 heads over 512 keys 21.5 us unpacked,
// 22.9 packed in pieces of one tile, 19.4 of two; 250 rows of 32 / 8 heads 0.84x with two.) Items
// (tile, range) are numbered by the tile's range length, longest first (equal lengths:
// later tile first), a tile's ranges together. plan[0] = {tiles, items, max_t c_t},
// plan[1 + t] = {c_t, first item of tile t, kt_t} (c_t = 0 past the last tile).
struct PlanArgs {
  AttnPlanReq r;
  int rb, budget, max_pc, pack;
};
__global__ __launch_bounds__(64) void k_attn_plan(PlanArgs p0, PlanArgs p1, int n_keys) {
  const PlanArgs a = blockIdx.x ? p1 : p0;
  const int rb = a.rb, budget = a.budget, max_pc = a.max_pc, pack = a.pack, pos0 = a.r.pos0;
  const int32_t *pos = a.r.pos;
  int4 *plan = reinterpret_cast<int4 *>(a.r.plan);
  const int lane = threadIdx.x;
  int R = a.r.rows;
  if (a.r.rows_dev) R = min(R, *a.r.rows_dev);
  R *= pack;  // (row, head) pairs
  if (a.r.row_base && pos) pos += *a.r.row_base;
  const int nt = (R + rb - 1) / rb;
  int kt = 0;
  if (lane < nt) {
    const int e = (min((lane + 1) * rb, R) - 1) / pack;
    kt = (min(n_keys, (pos ? pos[e] : pos0 + e) + 1) + 63) >> 6;
  }
  int ktmax = kt;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) ktmax = max(ktmax, __shfl_xor(ktmax, o, 64));
  const int B = max(nt, budget);
  int lo = max(2, (ktmax + max_pc - 1) / max_pc), hi = max(lo, ktmax);
  while (lo < hi) {  // the same bounds in every lane
    const int L = (lo + hi) >> 1;
    int c = lane < nt ? (kt + L - 1) / L : 0;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) c += __shfl_xor(c, o, 64);
    if (c <= B) hi = L;
    else lo = L + 1;
  }
  const int c = lane < nt ? (kt + lo - 1) / lo : 0;
  const int p = lane < nt ? (kt + c - 1) / c : 0;  // the tile's longest range
  int off = 0, total = 0, cmax = 0;
  for (int u = 0; u < nt; ++u) {  // u is the same in every lane: lane reads, no LDS trips
    const int pu = __builtin_amdgcn_readlane(p, u), cu = __builtin_amdgcn_readlane(c, u);
    if (pu > p || (pu == p && u > lane)) off += cu;
    total += cu;
    cmax = max(cmax, cu);
  }
  plan[1 + lane] = make_int4(c, off, kt, 0);
  if (lane == 0) plan[0] = make_int4(nt, total, cmax, 0);
}

// Partial outputs of the key splits take 16 bits per value: bf16 (8 significant bits), but in a plan
// of packed heads or more than 8 pieces, which rounds more of a row's terms, fp16 (11) where the
// largest value of the row's partial lies in [2^-8, 65504], so that none overflows and the small
// ones lose less than in bf16; the last bit of such a partial's sum says which. Against 64 bits,
// 159 rows of the 7B heads over 8000 keys: 2.63e-3 in 8 pieces one by one, 2.76e-3 packed in 16
// with bf16 partials, 2.35e-3 this way; no call of 210 shapes slower.
typedef _Float16 half2_t __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t pack_part(float a, float b, bool half) {
  const half2_t h = {(_Float16)a, (_Float16)b};
  return half ? __builtin_bit_cast(uint32_t, h) : pack_bf2(a, b);
}
__device__ __forceinline__ void part_values(uint4 w, bool halves, float sum, float (&x)[8]) {
  const bool half = halves && (__float_as_uint(sum) & 1u);
  const uint32_t v[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const half2_t h = __builtin_bit_cast(half2_t, v[i]);
    x[2 * i] = half ? (float)h[0] : __uint_as_float(v[i] << 16);
    x[2 * i + 1] = half ? (float)h[1] : __uint_as_float(v[i] & 0xffff0000u);
  }
}

// A block serves 32 * nrb rows of one query head (pack 1), or as many (row, head) pairs of the
// G = pack query heads of KV head kvh: pair v is row v / G, head kvh * G + v % G. Wave w owns
// 32 of them. Waves 0-3
// stage each 64-key K / V tile in LDS for all of them (double buffered, the next tile in
// flight during the current one: hd 128 straight from global memory into LDS, hd 64 through
// registers). Block b serves KV head b % Hkv, so the blocks streaming one head's keys run on
// the same XCD and share its L2.
template <int HD, bool PREF>
__global__ __launch_bounds__(512) void k_attn_bf16(const bf16_t *__restrict__ Q,
                                                   const int32_t *pos, int pos0, int rows,
                                                   const int32_t *rows_dev,
                                                   const bf16_t *__restrict__ Kc,
                                                   const bf16_t *__restrict__ Vc, int n_keys,
                                                   int hq, int hkv, int pack, bool halves,
                                                   int nrb, int n_tiles, int n_splits,
                                                   int split_keys,
                                                   float scale_log2,
                                                   bf16_t *__restrict__ out,
                                                   bf16_t *__restrict__ part_o,
                                                   float *__restrict__ part_ml,
                                                   const int32_t *row_base,
                                                   const int4 *__restrict__ plan) {
  constexpr int KS = HD / 16;          // contraction steps of S
  constexpr int DB = HD / 32;          // 32-wide head-dim blocks of O
  constexpr int KST = HD + 8;          // K tile row stride (bf16)
  constexpr int VRS = HD + 32;         // V tile row stride (bf16)
  constexpr int CPK = HD / 8;          // 16-byte chunks per key row
  constexpr int LT = 256;              // loading threads (waves 0-3)
  constexpr int KCH = 64 * CPK / LT;   // K (and V) chunks per loading thread
  // DIR: the tiles go from global memory straight into LDS (hd 128; PREF: hd 64, 4 waves)
  constexpr bool DIR = !PREF && HD == 128;
  constexpr int KBUF = DIR ? 64 * HD : 64 * KST, VBUF = DIR ? 64 * HD : 64 * VRS;
  // the two buffers of a tile pair; with DIR separate LDS objects (see the loop below)
  __shared__ __attribute__((aligned(16))) bf16_t Ks[(DIR ? 1 : 2) * KBUF];
  __shared__ __attribute__((aligned(16))) bf16_t Vt[(DIR ? 1 : 2) * VBUF];
  __shared__ __attribute__((aligned(16))) bf16_t Ks1[DIR ? KBUF : 1];
  __shared__ __attribute__((aligned(16))) bf16_t Vt1[DIR ? VBUF : 1];
  __shared__ int s_max[8];
  if (row_base) {  // this call's rows start at row *row_base of q, pos and out
    const int rb0 = *row_base;
    Q += (size_t)rb0 * hq * HD;
    out += (size_t)rb0 * hq * HD;
    if (pos) pos += rb0;
  }
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int nw = blockDim.x >> 6;
  const bool loader = wave < 4;
  const int G = hq / hkv;
  const int kvh = blockIdx.x % hkv;
  int rest = (int)(blockIdx.x / hkv);
  const int lists = pack > 1 ? 1 : G;  // row lists of a KV head
  const int hg = rest % lists;
  rest /= lists;
  int R = rows;
  if (rows_dev) R = min(R, *rows_dev);
  R *= pack;
  const int rb_rows = 32 * nrb;
  int split, tile, n_part = n_splits, kv_begin = -1;
  if (plan) {  // item `rest` of the call's plan (see k_attn_plan)
    const int4 e = plan[1 + lane];  // (c = 0 past the last tile)
    const unsigned long long mine = __ballot(e.x > 0 && e.y <= rest && rest < e.y + e.x);
    if (mine == 0) return;  // past the last item (the whole block)
    const int t = __ffsll((long long)mine) - 1;
    const int c = __shfl(e.x, t, 64), first = __shfl(e.y, t, 64), kt = __shfl(e.z, t, 64);
    tile = t;
    split = rest - first;
    n_part = c;
    if (c > n_splits) return;  // not a plan for this launch's partial slots
    kv_begin = (split * kt / c) * 64;
    split_keys = ((split + 1) * kt / c) * 64 - kv_begin;
  } else {
    split = rest % n_splits;
    tile = n_tiles - 1 - rest / n_splits;
  }
  const int row0 = tile * rb_rows;
  if (tile < 0 || row0 >= R) return;
  const int hi = lane >> 5;  // which half of a row's 32 keys (and 32 dims) this lane holds
  const int v = row0 + wave * 32 + (lane & 31);
  const bool rvalid = v < R;
  const int r = pack > 1 ? v / pack : v;
  const int head = kvh * G + (pack > 1 ? v - r * pack : hg);
  const int rp = rvalid ? (pos ? pos[r] : pos0 + r) : -1;
  const int rpos = rvalid ? rp : 0;
  int wmax = rp, wmin = rvalid ? rp : 0x7fffffff;
#pragma unroll
  for (int o = 1; o < 32; o <<= 1) {
    wmax = max(wmax, __shfl_xor(wmax, o, 64));
    wmin = min(wmin, __shfl_xor(wmin, o, 64));
  }
  if (lane == 0) s_max[wave] = wmax;
  __syncthreads();
  int bmax = -1;
  for (int w = 0; w < nw; ++w) bmax = max(bmax, s_max[w]);
  // this block's keys: [kv_begin, kv_end) of split `split`
  if (kv_begin < 0) kv_begin = split * split_keys;
  const int kv_end = min(min(n_keys, bmax + 1), kv_begin + split_keys);
  const int nkt = kv_end > kv_begin ? (kv_end - kv_begin + 63) / 64 : 0;
  const size_t prow = ((size_t)split * rows + r) * hq + head;  // partial slot of this lane's row
  if (nkt == 0) {
    if (n_splits > 1 && rvalid && hi == 0) {
      part_ml[2 * prow] = -INFINITY;
      part_ml[2 * prow + 1] = 0.f;
    }
    return;
  }

  // Q^T operand of S: lane holds dims ks*16 + hi*8 .. +7 of its row
  bf16x8_t qf[KS];
  {
    const bf16_t *qrow = Q + ((size_t)(rvalid ? r : row0 / pack) * hq + head) * HD + hi * 8;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) qf[ks] = *reinterpret_cast<const bf16x8_t *>(qrow + ks * 16);
    // vmcnt(0): the query fragments are complete before the key loop, so the loop's waits
    // on the K / V prefetch never cover them
    __builtin_amdgcn_s_waitcnt(0x0f70);
  }
  f32x16_t o[DB];
#pragma unroll
  for (int db = 0; db < DB; ++db)
#pragma unroll
    for (int i = 0; i < 16; ++i) o[db][i] = 0.f;
  float m_run = -INFINITY, l_run = 0.f;  // l_run: this lane's half of the row sum

  // One K / V tile in the loading waves' registers. Keys past kv_end are clamped to the
  // last key: finite data that the score mask gives probability 0.
  u32x4_t kreg[DIR ? 1 : KCH], vreg[DIR ? 1 : KCH];
  const int klast = kv_end - 1;
  // DIR staging: global_load_lds, 16 bytes per lane, the 64 lanes of a loading wave filling
  // 1 KB = 4 unpadded rows of 256 bytes (lane p: row +p/16, 16-byte chunk position p%16).
  // Which global chunk a lane fetches sets the layout: chunk c of row r sits at position
  // c ^ (r & 15) for K and c ^ 4 (r & 3) for V, so that the 32 K rows of a fragment read
  // and the 4 V rows of a transposing read fall on distinct banks. No registers, no LDS
  // stores in the loading waves: 4.7 % faster on the 32B probe layer (986 -> 940 us), same
  // bits. The transposing V reads are inline assembly: through the builtin, the compiler
  // cannot tell them from the DMA's LDS writes and waits for the next tile's DMA before the
  // first of them, which cost the 4-wave blocks 20-27 % against register staging with
  // read-ahead; without that wait the 4-wave blocks are 3-8 % faster than the register
  // staging on the 3B probe layers (1/100 to 3/10 of the context), the 8-wave blocks about
  // 1 % (standalone harness, not in the repository).
  auto dma_to = [&](int key0_, bf16_t *kbuf, bf16_t *vbuf) {
    const int w = tid >> 6;  // loading wave 0..3
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int row = (i * 4 + w) * 4 + (lane >> 4);
      const int pc = lane & 15;
      const size_t gro = ((size_t)min(key0_ + row, klast) * hkv + kvh) * HD;
      __builtin_amdgcn_global_load_lds((const void *)(Kc + gro + (pc ^ (row & 15)) * 8),
                                       (__attribute__((address_space(3))) void *)(
                                           kbuf + (i * 4 + w) * 4 * HD),
                                       16, 0, 0);
      __builtin_amdgcn_global_load_lds((const void *)(Vc + gro + (pc ^ (4 * (row & 3))) * 8),
                                       (__attribute__((address_space(3))) void *)(
                                           vbuf + (i * 4 + w) * 4 * HD),
                                       16, 0, 0);
    }
  };
#define AKVS_KV_LOAD(KEY0)                                                                  \
  {                                                                                         \
    _Pragma("unroll") for (int i = 0; i < KCH; ++i) {                                       \
      const int c = tid + LT * i, kr = c / CPK, e0 = (c - kr * CPK) * 8;                    \
      const size_t o_ = ((size_t)min((KEY0) + kr, klast) * hkv + kvh) * HD + e0;            \
      kreg[i] = *reinterpret_cast<const u32x4_t *>(Kc + o_);                                \
      vreg[i] = *reinterpret_cast<const u32x4_t *>(Vc + o_);                                \
    }                                                                                       \
  }
#define AKVS_KV_STORE(KB, VB)                                                               \
  {                                                                                         \
    bf16_t *ks_ = (KB);                                                                     \
    bf16_t *vt_ = (VB);                                                                     \
    _Pragma("unroll") for (int i = 0; i < KCH; ++i) {                                       \
      const int c = tid + LT * i, kr = c / CPK, e0 = (c - kr * CPK) * 8;                    \
      *reinterpret_cast<u32x4_t *>(ks_ + kr * KST + e0) = kreg[i];                          \
      *reinterpret_cast<u32x4_t *>(vt_ + kr * VRS + e0) = vreg[i];                          \
    }                                                                                       \
  }

  if (DIR) {
    if (loader) dma_to(kv_begin, Ks, Vt);
    __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0)
  } else if (loader) {
    AKVS_KV_LOAD(kv_begin);
    AKVS_KV_STORE(Ks, Vt);
  }
  __syncthreads();
  // one 64-key tile from ks_ / vt_, the next one staged into nks_ / nvt_
  auto step = [&](int kt, const bf16_t *ks_in, const bf16_t *vt_in, bf16_t *nks_,
                  bf16_t *nvt_) __attribute__((always_inline)) {
    const bf16_t *ks_ = DIR ? ks_in : Ks + (kt & 1) * KBUF;
    const bf16_t *vt_ = DIR ? vt_in : Vt + (kt & 1) * VBUF;
    const int key0 = kv_begin + kt * 64;
    const bool more = kt + 1 < nkt;
    if (loader && more) {
      if (DIR) dma_to(key0 + 64, nks_, nvt_);
      else AKVS_KV_LOAD(key0 + 64);
    }
    // PREF (register-staged hd 64 blocks): the K fragments of a 32-key block are read ahead
    // (the tile's first block here, its second under the first block's softmax) and each
    // block's V^T fragments are requested before its score MFMAs, so no MFMA waits on its own
    // LDS read. It needs about 50 more registers.
    bf16x8_t kf[KS];
    if (PREF && key0 <= wmax) {
      const bf16_t *krow = ks_ + (lane & 31) * KST + hi * 8;
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) kf[ks] = *reinterpret_cast<const bf16x8_t *>(krow + ks * 16);
      static_assert(!DIR || !PREF, "the read-ahead reads the padded K layout");
    }
#pragma unroll
    for (int st = 0; st < 2; ++st) {
      const int sk0 = key0 + st * 32;
      if (sk0 <= wmax) {  // skip keys past every row of this wave
        // V^T operand of k-step t, head-dim block db: lane holds dim db*32 + lane%32 at the
        // keys of its 8 slots (slots 0-3: 16t + 4*hi + 0..3 of this 32-key block, 4-7: the
        // same + 8), two transposing reads of 4 keys each
        bf16x8_t vf[2][DB];
        auto read_v = [&](int t, int db) {
          typedef short v4s __attribute__((ext_vector_type(4)));
          // DIR: the 16-byte chunk db*4 + 2*((lane>>4)&1) + (lane&3)/2 of a row whose low two
          // bits are (lane>>2)&3 sits at db ^ ((lane>>2)&3) in place of db
          const bf16_t *vb =
              DIR ? vt_ + (st * 32 + 16 * t + 4 * hi + ((lane & 15) >> 2)) * HD +
                        (4 * (db ^ ((lane >> 2) & 3)) + 2 * ((lane >> 4) & 1) + ((lane & 3) >> 1)) * 8 +
                        (lane & 1) * 4
                  : vt_ + (st * 32 + 16 * t + 4 * hi + ((lane & 15) >> 2)) * VRS + db * 32 +
                        16 * ((lane >> 4) & 1) + 4 * (lane & 3);
          uint32_t vw[4];
          if constexpr (DIR) {
            // as assembly: the builtin carries no alias information, so the compiler would
            // wait for the next tile's DMA (vmcnt(0)) before it; the fragments are complete
            // at the explicit lgkmcnt(0) before the P.V MFMAs (below)
            typedef unsigned int u2_t __attribute__((ext_vector_type(2)));
            u2_t x0, x1;
            const uint32_t a0 =
                (uint32_t)(size_t)(__attribute__((address_space(3))) const bf16_t *)(vb);
            asm volatile("ds_read_b64_tr_b16 %0, %1" : "=v"(x0) : "v"(a0));
            asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(x1) : "v"(a0), "i"(8 * HD * 2));
            vw[0] = x0.x; vw[1] = x0.y; vw[2] = x1.x; vw[3] = x1.y;
          } else {
            const v4s r0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                (__attribute__((address_space(3))) v4s *)(vb));
            const v4s r1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                (__attribute__((address_space(3))) v4s *)(vb + 8 * VRS));
            uint2 x0, x1;
            __builtin_memcpy(&x0, &r0, 8);
            __builtin_memcpy(&x1, &r1, 8);
            vw[0] = x0.x; vw[1] = x0.y; vw[2] = x1.x; vw[3] = x1.y;
          }
          __builtin_memcpy(&vf[t][db], vw, 16);
        };
        if (PREF) {  // every V^T fragment of the block requested up front
#pragma unroll
          for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int db = 0; db < DB; ++db) read_v(t, db);
        }
        // S^T block: 32 keys x 32 rows; s[i] is key sk0 + (i/4)*8 + hi*4 + i%4 of row r
        f32x16_t sc;
#pragma unroll
        for (int i = 0; i < 16; ++i) sc[i] = 0.f;
        // K fragment of step ks: 16-byte chunk 2ks + hi of row st*32 + lane%32 (DIR: at its
        // swizzled position; st*32 is a multiple of 16, so the row's low bits are lane%16)
        const bf16_t *krow =
            ks_ + (st * 32 + (lane & 31)) * (DIR ? HD : KST) + (DIR ? 0 : hi * 8);
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
          const bf16x8_t a =
              PREF ? kf[ks]
                   : *reinterpret_cast<const bf16x8_t *>(
                         krow + (DIR ? ((2 * ks + hi) ^ (lane & 15)) * 8 : ks * 16));
          sc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, qf[ks], sc, 0, 0, 0);
        }
        if constexpr (DIR) {
          // V^T fragments behind the K fragments: LDS answers in order, so requested before the
          // scores they held up every score MFMA, and the softmax hides them as well (same bits;
          // 5534 rows of the 32B heads over 16128 keys 880 -> 864 us, 1413 of 3B over 4516 75 ->
          // 72.5, 2806 of 7B over 8128 202 -> 198)
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int db = 0; db < DB; ++db) read_v(t, db);
        }
        if (PREF && st == 0 && sk0 + 32 <= wmax) {
          const bf16_t *knext = ks_ + (32 + (lane & 31)) * KST + hi * 8;
#pragma unroll
          for (int ks = 0; ks < KS; ++ks)
            kf[ks] = *reinterpret_cast<const bf16x8_t *>(knext + ks * 16);
        }
        if (sk0 + 31 > wmin || sk0 + 31 >= kv_end) {  // causal / range mask needed
          // score i is key sk0 + hi*4 + (i/4)*8 + i%4: masked past min(row position, last key)
          const int lim = min(rpos, kv_end - 1) - (sk0 + hi * 4);
#pragma unroll
          for (int i = 0; i < 16; ++i)
            if ((i >> 2) * 8 + (i & 3) > lim) sc[i] = -INFINITY;
        }
        float mx = sc[0];
#pragma unroll
        for (int i = 1; i < 16; ++i) mx = fmaxf(mx, sc[i]);
        // raise the running maximum only when some score exceeds it by more than 2^8
        if (__ballot(mx * scale_log2 > m_run + 8.f)) {
          const float mp = fmaxf(mx, __shfl_xor(mx, 32, 64)) * scale_log2;
          const float m_new = fmaxf(m_run, mp);
          const float alpha = m_new == -INFINITY ? 1.f : __builtin_amdgcn_exp2f(m_run - m_new);
#pragma unroll
          for (int db = 0; db < DB; ++db) o[db] *= alpha;
          l_run *= alpha;
          m_run = m_new;
        }
        // rows with no key yet keep m = -inf: offset by 0 then (every p is 0)
        const float m_off = m_run == -INFINITY ? 0.f : m_run;
        float pv[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          pv[i] = __builtin_amdgcn_exp2f(fmaf(sc[i], scale_log2, -m_off));  // v_exp_f32: arguments <= 8
          l_run += pv[i];
        }
        if constexpr (DIR) {  // the assembly reads above: results complete here
          static_assert(DB == 4, "hd 128");
          asm volatile("s_waitcnt lgkmcnt(0)"
                       : "+v"(vf[0][0]), "+v"(vf[0][1]), "+v"(vf[0][2]), "+v"(vf[0][3]),
                         "+v"(vf[1][0]), "+v"(vf[1][1]), "+v"(vf[1][2]), "+v"(vf[1][3]));
        }
        // P^T operand of k-step t: slots hi*8 + j hold keys 16t + (j/4)*8 + hi*4 + j%4
#pragma unroll
        for (int t = 0; t < 2; ++t) {
          uint32_t pw[4];
#pragma unroll
          for (int j = 0; j < 4; ++j) pw[j] = pack_bf2(pv[8 * t + 2 * j], pv[8 * t + 2 * j + 1]);
          bf16x8_t pb;
          __builtin_memcpy(&pb, pw, 16);
#pragma unroll
          for (int db = 0; db < DB; ++db) {
            if (!PREF && !DIR) read_v(t, db);
            o[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[t][db], pb, o[db], 0, 0, 0);
          }
        }
      }
    }
    if (DIR) __builtin_amdgcn_s_waitcnt(0x0f70);  // this wave's DMA of the next tile landed
    else if (loader && more) AKVS_KV_STORE(Ks + ((kt + 1) & 1) * KBUF, Vt + ((kt + 1) & 1) * VBUF);
    __syncthreads();
  };
  if constexpr (DIR) {
    // unrolled by two over separate LDS objects, so that the compiler can see that a
    // step's reads and the next tile's DMA touch different memory and does not wait for
    // the DMA before the reads
    for (int kt = 0; kt < nkt; kt += 2) {
      step(kt, Ks, Vt, Ks1, Vt1);
      if (kt + 1 < nkt) step(kt + 1, Ks1, Vt1, Ks, Vt);
    }
  } else {
    // (the same step written out in the loop: as a lambda it cost the read-ahead variant
    // two spilled registers)
    for (int kt = 0; kt < nkt; ++kt) {
    const bf16_t *ks_ = Ks + (kt & 1) * KBUF;
    const bf16_t *vt_ = Vt + (kt & 1) * VBUF;
    const int key0 = kv_begin + kt * 64;
    const bool more = kt + 1 < nkt;
    if (loader && more) {
      AKVS_KV_LOAD(key0 + 64);
    }
    // PREF (register-staged hd 64 blocks): the K fragments of a 32-key block are read ahead
    // (the tile's first block here, its second under the first block's softmax) and each
    // block's V^T fragments are requested before its score MFMAs, so no MFMA waits on its own
    // LDS read. It needs about 50 more registers.
    bf16x8_t kf[KS];
    if (PREF && key0 <= wmax) {
      const bf16_t *krow = ks_ + (lane & 31) * KST + hi * 8;
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) kf[ks] = *reinterpret_cast<const bf16x8_t *>(krow + ks * 16);
      static_assert(!DIR || !PREF, "the read-ahead reads the padded K layout");
    }
#pragma unroll
    for (int st = 0; st < 2; ++st) {
      const int sk0 = key0 + st * 32;
      if (sk0 <= wmax) {  // skip keys past every row of this wave
        // V^T operand of k-step t, head-dim block db: lane holds dim db*32 + lane%32 at the
        // keys of its 8 slots (slots 0-3: 16t + 4*hi + 0..3 of this 32-key block, 4-7: the
        // same + 8), two transposing reads of 4 keys each
        bf16x8_t vf[2][DB];
        auto read_v = [&](int t, int db) {
          typedef short v4s __attribute__((ext_vector_type(4)));
          // DIR: the 16-byte chunk db*4 + 2*((lane>>4)&1) + (lane&3)/2 of a row whose low two
          // bits are (lane>>2)&3 sits at db ^ ((lane>>2)&3) in place of db
          const bf16_t *vb =
              DIR ? vt_ + (st * 32 + 16 * t + 4 * hi + ((lane & 15) >> 2)) * HD +
                        (4 * (db ^ ((lane >> 2) & 3)) + 2 * ((lane >> 4) & 1) + ((lane & 3) >> 1)) * 8 +
                        (lane & 1) * 4
                  : vt_ + (st * 32 + 16 * t + 4 * hi + ((lane & 15) >> 2)) * VRS + db * 32 +
                        16 * ((lane >> 4) & 1) + 4 * (lane & 3);
          const v4s r0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
              (__attribute__((address_space(3))) v4s *)(vb));
          const v4s r1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
              (__attribute__((address_space(3))) v4s *)(vb + 8 * (DIR ? HD : VRS)));
          uint2 x0, x1;
          __builtin_memcpy(&x0, &r0, 8);
          __builtin_memcpy(&x1, &r1, 8);
          uint32_t vw[4] = {x0.x, x0.y, x1.x, x1.y};
          __builtin_memcpy(&vf[t][db], vw, 16);
        };
        if (PREF) {
#pragma unroll
          for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int db = 0; db < DB; ++db) read_v(t, db);
        }
        // S^T block: 32 keys x 32 rows; s[i] is key sk0 + (i/4)*8 + hi*4 + i%4 of row r
        f32x16_t sc;
#pragma unroll
        for (int i = 0; i < 16; ++i) sc[i] = 0.f;
        // K fragment of step ks: 16-byte chunk 2ks + hi of row st*32 + lane%32 (DIR: at its
        // swizzled position; st*32 is a multiple of 16, so the row's low bits are lane%16)
        const bf16_t *krow =
            ks_ + (st * 32 + (lane & 31)) * (DIR ? HD : KST) + (DIR ? 0 : hi * 8);
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
          const bf16x8_t a =
              PREF ? kf[ks]
                   : *reinterpret_cast<const bf16x8_t *>(
                         krow + (DIR ? ((2 * ks + hi) ^ (lane & 15)) * 8 : ks * 16));
          sc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, qf[ks], sc, 0, 0, 0);
        }
        if (PREF && st == 0 && sk0 + 32 <= wmax) {
          const bf16_t *knext = ks_ + (32 + (lane & 31)) * KST + hi * 8;
#pragma unroll
          for (int ks = 0; ks < KS; ++ks)
            kf[ks] = *reinterpret_cast<const bf16x8_t *>(knext + ks * 16);
        }
        if (sk0 + 31 > wmin || sk0 + 31 >= kv_end) {  // causal / range mask needed
          // score i is key sk0 + hi*4 + (i/4)*8 + i%4: masked past min(row position, last key)
          const int lim = min(rpos, kv_end - 1) - (sk0 + hi * 4);
#pragma unroll
          for (int i = 0; i < 16; ++i)
            if ((i >> 2) * 8 + (i & 3) > lim) sc[i] = -INFINITY;
        }
        float mx = sc[0];
#pragma unroll
        for (int i = 1; i < 16; ++i) mx = fmaxf(mx, sc[i]);
        // raise the running maximum only when some score exceeds it by more than 2^8
        if (__ballot(mx * scale_log2 > m_run + 8.f)) {
          const float mp = fmaxf(mx, __shfl_xor(mx, 32, 64)) * scale_log2;
          const float m_new = fmaxf(m_run, mp);
          const float alpha = m_new == -INFINITY ? 1.f : __builtin_amdgcn_exp2f(m_run - m_new);
#pragma unroll
          for (int db = 0; db < DB; ++db) o[db] *= alpha;
          l_run *= alpha;
          m_run = m_new;
        }
        // rows with no key yet keep m = -inf: offset by 0 then (every p is 0)
        const float m_off = m_run == -INFINITY ? 0.f : m_run;
        float pv[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          pv[i] = __builtin_amdgcn_exp2f(fmaf(sc[i], scale_log2, -m_off));  // v_exp_f32: arguments <= 8
          l_run += pv[i];
        }
        // P^T operand of k-step t: slots hi*8 + j hold keys 16t + (j/4)*8 + hi*4 + j%4
#pragma unroll
        for (int t = 0; t < 2; ++t) {
          uint32_t pw[4];
#pragma unroll
          for (int j = 0; j < 4; ++j) pw[j] = pack_bf2(pv[8 * t + 2 * j], pv[8 * t + 2 * j + 1]);
          bf16x8_t pb;
          __builtin_memcpy(&pb, pw, 16);
#pragma unroll
          for (int db = 0; db < DB; ++db) {
            if (!PREF) read_v(t, db);
            o[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[t][db], pb, o[db], 0, 0, 0);
          }
        }
      }
    }
    if (loader && more) AKVS_KV_STORE(Ks + ((kt + 1) & 1) * KBUF, Vt + ((kt + 1) & 1) * VBUF);
    __syncthreads();
    }
  }
#undef AKVS_KV_LOAD
#undef AKVS_KV_STORE
  const float l_row = l_run + __shfl_xor(l_run, 32, 64);
  if (!rvalid) return;
  // o[db][i] is dim db*32 + (i/4)*8 + hi*4 + i%4 of row r
  if (n_splits > 1 && n_part == 1) {  // a whole tile: final output here; the merge skips
    if (hi == 0) {                     // the row (end mark in the first slot)
      part_ml[2 * prow] = -INFINITY;
      part_ml[2 * prow + 1] = -1.f;
    }
  } else if (n_splits > 1) {  // this split's output over its own keys + (max, sum)
    const float pinv = l_row > 0.f ? 1.0f / l_row : 0.f;  // no visible key: m = -inf, skipped
    float big = 0.f;
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        o[db][i] *= pinv;
        big = fmaxf(big, fabsf(o[db][i]));
      }
    big = fmaxf(big, __shfl_xor(big, 32, 64));
    const bool half = halves && big >= 0x1p-8f && big <= 65504.f;
    bf16_t *po = part_o + prow * HD + hi * 4;
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4) {
        *reinterpret_cast<uint2 *>(po + db * 32 + q4 * 8) =
            make_uint2(pack_part(o[db][4 * q4], o[db][4 * q4 + 1], half),
                       pack_part(o[db][4 * q4 + 2], o[db][4 * q4 + 3], half));
      }
    if (hi == 0) {
      part_ml[2 * prow] = m_run;
      part_ml[2 * prow + 1] =
          halves && l_row > 0.f ? __uint_as_float((__float_as_uint(l_row) & ~1u) | half) : l_row;
      if (split == n_part - 1 && n_part < n_splits) {  // end mark: no later split of this tile
        const size_t pend = ((size_t)n_part * rows + r) * hq + head;
        part_ml[2 * pend] = -INFINITY;
        part_ml[2 * pend + 1] = -1.f;
      }
    }
    return;
  }
  const float inv = 1.0f / l_row;
  bf16_t *orow = out + ((size_t)r * hq + head) * HD + hi * 4;
#pragma unroll
  for (int db = 0; db < DB; ++db)
#pragma unroll
    for (int q4 = 0; q4 < 4; ++q4)
      store4(orow + db * 32 + q4 * 8, o[db][4 * q4] * inv, o[db][4 * q4 + 1] * inv,
             o[db][4 * q4 + 2] * inv, o[db][4 * q4 + 3] * inv);
}

// Merge of the key splits of one (row, head): split s holds its output over its own keys,
// o_s (16 bits, normalised by its own sum l_s), and (m_s, l_s); the result is
// sum_s w_s o_s / sum_s w_s with w_s = 2^(m_s - max m) l_s, added in split order. A split
// whose keys all lie past the row (causal mask) holds m = -inf and l = 0 and is skipped, never
// multiplied in (its part_o slot holds whatever the workspace held); one of NaN scores holds
// m = -inf and l = NaN and makes NaN of the row. With a device-planned
// split a tile may use fewer splits than the launch's count: l = -1 after its last one
// ends the list (the slots past it are stale); l = -1 in the first slot marks a row whose
// tile ran as one piece and whose output the attention block wrote itself.
// Thread = 8 consecutive head dims of one (row, head) (16-byte loads and stores). Up to MAXS
// splits, all (m, l) pairs and partial outputs are requested at once; with more, the
// maxima first, then the splits in order.
template <int MAXS>
__global__ __launch_bounds__(256) void k_attn_combine(const bf16_t *__restrict__ part_o,
                                                      const float *__restrict__ part_ml,
                                                      int n_splits, int rows,
                                                      const int32_t *rows_dev, int hq, int hd,
                                                      bf16_t *__restrict__ out,
                                                      const int32_t *row_base,
                                                      const int4 *plan, bool halves) {
  const int per = hd >> 3;  // threads per (row, head)
  const long long gid = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  const long long item = gid / per;
  const int e0 = (int)(gid - item * per) * 8;
  int R = rows;
  if (rows_dev) R = min(R, *rows_dev);
  if (item >= (long long)R * hq) return;
  if (row_base) out += (size_t)*row_base * hq * hd;
  if (plan) n_splits = min(n_splits, plan[0].z);  // no tile of the plan has more pieces
  const size_t stride = (size_t)rows * hq;  // items per split
  float mx = -INFINITY, l = 0.f, a[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) a[i] = 0.f;
  if (n_splits <= MAXS) {  // every partial of this item requested at once
    float2 ml[MAXS];
    uint4 o[MAXS];
#pragma unroll
    for (int u = 0; u < MAXS; ++u) {
      if (u < n_splits) {
        const size_t pi = u * stride + item;
        ml[u] = *reinterpret_cast<const float2 *>(part_ml + 2 * pi);
        o[u] = *reinterpret_cast<const uint4 *>(part_o + pi * hd + e0);
      }
    }
    int n = n_splits;  // up to the first end mark
#pragma unroll
    for (int u = MAXS - 1; u >= 0; --u)
      if (u < n_splits && ml[u].y < 0.f) n = u;
#pragma unroll
    for (int u = 0; u < MAXS; ++u)
      if (u < n) mx = fmaxf(mx, ml[u].x);
    if (n == 0) return;  // the attention wrote this row's output itself
    const float moff = mx == -INFINITY ? 0.f : mx;
#pragma unroll
    for (int u = 0; u < MAXS; ++u) {
      if (u >= n || ml[u].y == 0.f) continue;
      const float w = exp2f(ml[u].x - moff) * ml[u].y;
      l += w;
      float x[8];
      part_values(o[u], halves, ml[u].y, x);
#pragma unroll
      for (int i = 0; i < 8; ++i) a[i] += w * x[i];
    }
  } else {
    int n = n_splits;  // up to the first end mark
    for (int sp = 0; sp < n; ++sp) {
      const float2 ml = *reinterpret_cast<const float2 *>(part_ml + 2 * (sp * stride + item));
      if (ml.y < 0.f) n = sp;
      else mx = fmaxf(mx, ml.x);
    }
    if (n == 0) return;
    const float moff = mx == -INFINITY ? 0.f : mx;
    for (int sp = 0; sp < n; ++sp) {
      const size_t pi = sp * stride + item;
      const float2 ml = *reinterpret_cast<const float2 *>(part_ml + 2 * pi);
      if (ml.y == 0.f) continue;  // no visible key: its part_o was never written
      float o[8];
      part_values(*reinterpret_cast<const uint4 *>(part_o + pi * hd + e0), halves, ml.y, o);
      const float w = exp2f(ml.x - moff) * ml.y;
      l += w;
#pragma unroll
      for (int i = 0; i < 8; ++i) a[i] += w * o[i];
    }
  }
  const float inv = 1.0f / l;
#pragma unroll
  for (int i = 0; i < 8; ++i) a[i] *= inv;
  store8(out + item * hd + e0, a);
}

// fp32 path (small models), on v_mfma_f32_16x16x4_f32. Block = 16 rows of one query head, 8
// waves that take the 16-key tiles in turn (wave w the tiles w, w + 8, ...), each with its own
// running maximum, sum and output, merged through LDS in wave order at the end: short calls
// are bound by dependent memory round trips, so a tile needs one (K and V together, requested
// a tile ahead) and no barrier. Scores are formed transposed, S^T = K Q^T: lane l holds the scores of row l % 16
// at keys 4 (l / 16) + 0..3 of the tile, which is the operand layout of O^T = V^T P^T as it is.
// 288 rows over 288 keys, 4 heads of 64: 30 us with one wave per (row, head) reading key rows
// a lane each, 17 us here without the tile ahead, 9 us with it.
template <int HD>
__global__ __launch_bounds__(512) void k_attn_f32(const float *__restrict__ Q, const int32_t *pos,
                                                  int pos0, int rows, const int32_t *rows_dev,
                                                  const float *__restrict__ Kc,
                                                  const float *__restrict__ Vc, int n_keys, int hq,
                                                  int hkv, float scale_log2,
                                                  float *__restrict__ out,
                                                  const int32_t *row_base) {
  constexpr int C = HD / 16, NW = 8;
  __shared__ float s_o[NW][HD][17];
  __shared__ float s_m[NW][16], s_l[NW][16];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int lr = lane & 15, lg = lane >> 4;
  const int row0 = blockIdx.x * 16, head = blockIdx.y;
  if (row_base) {
    const int rb0 = *row_base;
    Q += (size_t)rb0 * hq * HD;
    out += (size_t)rb0 * hq * HD;
    if (pos) pos += rb0;
  }
  int R = rows;
  if (rows_dev) R = min(R, *rows_dev);
  if (row0 >= R) return;
  const int kvh = head / (hq / hkv);
  const int r = row0 + lr;
  const bool rvalid = r < R;
  const int rp = rvalid ? (pos ? pos[r] : pos0 + r) : -1;
  const int lim = min(n_keys - 1, rp);  // the row's last key
  int last = lim;                       // the block's last key
#pragma unroll
  for (int o = 1; o < 16; o <<= 1) last = max(last, __shfl_xor(last, o, 64));
  f32x4_t qf[C];
  {
    const float *q = Q + ((size_t)(rvalid ? r : row0) * hq + head) * HD + lg * 4;
#pragma unroll
    for (int c = 0; c < C; ++c) qf[c] = *reinterpret_cast<const f32x4_t *>(q + 16 * c);
  }
  const f32x4_t zero = {0.f, 0.f, 0.f, 0.f};
  f32x4_t o[C];
#pragma unroll
  for (int c = 0; c < C; ++c) o[c] = zero;
  float m = -INFINITY, l = 0.f;  // of row lr (l: this lane's quarter of the keys)
  struct Tile {
    f32x4_t k[C];
    float v[C][4];
  };
  // keys past the block's last one re-read it (masked below)
  auto fetch = [&](Tile &t, int key0) __attribute__((always_inline)) {
    const float *k = Kc + ((size_t)min(key0 + lr, last) * hkv + kvh) * HD + lg * 4;
#pragma unroll
    for (int c = 0; c < C; ++c) t.k[c] = *reinterpret_cast<const f32x4_t *>(k + 16 * c);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float *v = Vc + ((size_t)min(key0 + lg * 4 + e, last) * hkv + kvh) * HD + lr;
#pragma unroll
      for (int c = 0; c < C; ++c) t.v[c][e] = v[16 * c];
    }
  };
  auto attend = [&](const Tile &t, int key0) __attribute__((always_inline)) {
    f32x4_t s0 = zero, s1 = zero;  // two chains of dependent MFMAs
#pragma unroll
    for (int c = 0; c < C; ++c)
#pragma unroll
      for (int e = 0; e < 4; e += 2) {
        s0 = __builtin_amdgcn_mfma_f32_16x16x4f32(t.k[c][e], qf[c][e], s0, 0, 0, 0);
        s1 = __builtin_amdgcn_mfma_f32_16x16x4f32(t.k[c][e + 1], qf[c][e + 1], s1, 0, 0, 0);
      }
    f32x4_t s = s0 + s1;
#pragma unroll
    for (int e = 0; e < 4; ++e)
      s[e] = key0 + lg * 4 + e <= lim ? s[e] * scale_log2 : -INFINITY;
    float mx = fmaxf(fmaxf(s[0], s[1]), fmaxf(s[2], s[3]));
    mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
    mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
    const float m_new = fmaxf(m, mx);
    const float off = m_new == -INFINITY ? 0.f : m_new;  // no key yet: every p is 0
    const float alpha = __builtin_amdgcn_exp2f(m - off);
    f32x4_t p;
#pragma unroll
    for (int e = 0; e < 4; ++e) p[e] = __builtin_amdgcn_exp2f(s[e] - off);
    l = l * alpha + ((p[0] + p[1]) + (p[2] + p[3]));
    m = m_new;
#pragma unroll
    for (int c = 0; c < C; ++c) o[c] *= alpha;
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int c = 0; c < C; ++c)
        o[c] = __builtin_amdgcn_mfma_f32_16x16x4f32(t.v[c][e], p[e], o[c], 0, 0, 0);
  };
  constexpr int STEP = NW * 16;
  Tile t0, t1;
  int key0 = wave * 16;
  if (key0 <= last) fetch(t0, key0);
  while (key0 <= last) {  // the next tile's loads are in flight while this one is used
    if (key0 + STEP <= last) fetch(t1, key0 + STEP);
    attend(t0, key0);
    key0 += STEP;
    if (key0 > last) break;
    if (key0 + STEP <= last) fetch(t0, key0 + STEP);
    attend(t1, key0);
    key0 += STEP;
  }
  l += __shfl_xor(l, 16, 64);
  l += __shfl_xor(l, 32, 64);
  // o[c][e] is dim 16 c + 4 lg + e of row lr
#pragma unroll
  for (int c = 0; c < C; ++c)
#pragma unroll
    for (int e = 0; e < 4; ++e) s_o[wave][16 * c + 4 * lg + e][lr] = o[c][e];
  if (lg == 0) {
    s_m[wave][lr] = m;
    s_l[wave][lr] = l;
  }
  __syncthreads();
  for (int i = wave; i < 16 && row0 + i < R; i += NW) {  // a wave per row, a lane per dim (or two)
    float mw[NW], lw[NW], mm = -INFINITY;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      mw[w] = s_m[w][i];
      lw[w] = s_l[w][i];
    }
#pragma unroll
    for (int w = 0; w < NW; ++w) mm = fmaxf(mm, mw[w]);
    float so[HD / 64] = {}, sl = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      // a wave without a key of the row has l = 0 (m = -inf is also what NaN scores leave, with
      // a sum of NaN); selected, not branched around, so that all LDS reads go out together
      const float a = __builtin_amdgcn_exp2f(mw[w] - mm);
      const bool none = lw[w] == 0.f;
#pragma unroll
      for (int c = 0; c < HD / 64; ++c) {
        const float x = fmaf(a, s_o[w][64 * c + lane][i], so[c]);
        so[c] = none ? so[c] : x;
      }
      sl = none ? sl : fmaf(a, lw[w], sl);
    }
    bool nan = false;
#pragma unroll
    for (int c = 0; c < HD / 64; ++c) nan |= so[c] != so[c];
    if (__ballot(nan && sl == sl) != 0) {
      // NaN over a sum that is none: an infinite or NaN value. It may be that of a key which
      // another row of the block sees and this one does not (its p of 0 makes NaN of it too), or
      // of the block's last key, which masked keys re-read: if there is one, the row is formed
      // again over its own keys, a lane per key for the scores.
      const int end = __shfl(lim, i, 64), far = __shfl(last, 0, 64);
      float odd = 0.f;  // NaN once a hidden value is infinite or NaN
      for (int k = max(min(end + 1, far), 0); k <= far; ++k) {
        const float *v = Vc + ((size_t)k * hkv + kvh) * HD + lane;
#pragma unroll
        for (int c = 0; c < HD / 64; ++c) odd = fmaf(v[64 * c], 0.f, odd);
      }
      const bool again = __ballot(odd != 0.f) != 0;
      const float *q = Q + ((size_t)(row0 + i) * hq + head) * HD;
      float rm = -INFINITY;
      if (again) {
        sl = 0.f;
#pragma unroll
        for (int c = 0; c < HD / 64; ++c) so[c] = 0.f;
      }
      for (int k0 = 0; again && k0 <= end; k0 += 64) {
        const float *k = Kc + ((size_t)min(k0 + lane, end) * hkv + kvh) * HD;
        f32x4_t s4 = zero;
        for (int d = 0; d < HD; d += 4)
          s4 += *reinterpret_cast<const f32x4_t *>(q + d) *
                *reinterpret_cast<const f32x4_t *>(k + d);
        const float sum = (s4[0] + s4[1]) + (s4[2] + s4[3]);
        const float s = k0 + lane <= end ? sum * scale_log2 : -INFINITY;
        const float m_new = fmaxf(rm, wave_max(s)), off = m_new == -INFINITY ? 0.f : m_new;
        const float p = __builtin_amdgcn_exp2f(s - off);
        const float alpha = __builtin_amdgcn_exp2f(rm - off);
        rm = m_new;
        sl = sl * alpha + wave_sum(p);
#pragma unroll
        for (int c = 0; c < HD / 64; ++c) so[c] *= alpha;
        for (int e = 0; e < 64 && k0 + e <= end; ++e) {
          const float pe = __shfl(p, e, 64);
          const float *v = Vc + ((size_t)(k0 + e) * hkv + kvh) * HD + lane;
#pragma unroll
          for (int c = 0; c < HD / 64; ++c) so[c] = fmaf(pe, v[64 * c], so[c]);
        }
      }
    }
#pragma unroll
    for (int c = 0; c < HD / 64; ++c)
      out[((size_t)(row0 + i) * hq + head) * HD + 64 * c + lane] = so[c] / sl;
  }
}

int attn_splits(int rows, int hq, int hkv, int n_keys) {
  if (hq < hkv || rows <= 0 || attn_whole(rows, n_keys)) return 1;
  const int rb = 32 * attn_waves(rows, hq);
  const long long base = (long long)((rows + rb - 1) / rb) * hq;
  if (base >= 512) return 1;                        // two blocks per compute unit already
  long long sp = (768 + base - 1) / base;           // else aim at ~768 blocks (measured)
  const long long cap = (n_keys + 255) / 256;        // at least 256 keys per split
  if (sp > cap) sp = cap;
  if (sp > 64) sp = 64;
  return sp < 1 ? 1 : (int)sp;
}

int attn_split_keys(int n_keys, int n_splits) {
  const int per = (n_keys + n_splits - 1) / n_splits;
  return (per + 63) / 64 * 64;
}

int attn_part_splits(int rows, int hq, int hkv, int hd, int n_keys, bool lean) {
  const int sp = attn_splits(rows, hq, hkv, n_keys);
  const int most = lean ? kAttnMaxPieces : attn_max_pieces(rows, n_keys);
  const AttnEqShape e = attn_eq_shape(rows, hq, hkv, n_keys, hd, AKVS_BF16,
                                      (long long)most * rows, gemm_cu_count());
  return e.use ? std::max(sp, most) : sp;
}

hipError_t launch_attention_plan(const AttnPlanReq *req, int n, int n_keys, int hq, int hkv,
                                 int hd, int dtype, long long part_rows, hipStream_t s) {
  PlanArgs p[2] = {};
  int used = 0;
  for (int i = 0; i < n; ++i) {
    const AttnEqShape e =
        attn_eq_shape(req[i].rows, hq, hkv, n_keys, hd, dtype, part_rows, gemm_cu_count());
    // (launch_attention will not read a plan that is not used either)
    if (e.use && req[i].plan) p[used++] = {req[i], e.rb, e.budget, e.max_pc, e.pack};
  }
  if (used == 0) return hipSuccess;
  hipLaunchKernelGGL(k_attn_plan, dim3(used), dim3(64), 0, s, p[0], p[1], n_keys);
  return hipGetLastError();
}

hipError_t launch_attention(const void *q, const int32_t *pos, int pos0, int rows,
                            const int32_t *rows_dev, const void *k, const void *v, int n_keys,
                            int hq, int hkv, int hd, int dtype, void *out, float *part_o,
                            float *part_ml, long long part_rows, hipStream_t s,
                            const int32_t *row_base, const int32_t *plan) {
  if (rows == 0) return hipSuccess;
  if (dtype == AKVS_BF16) {
    const float scale_log2 = 1.4426950408889634f / sqrtf((float)hd);
    const bf16_t *Q = reinterpret_cast<const bf16_t *>(q);
    const bf16_t *K = reinterpret_cast<const bf16_t *>(k);
    const bf16_t *V = reinterpret_cast<const bf16_t *>(v);
    bf16_t *O = reinterpret_cast<bf16_t *>(out);
    if (hq < hkv) return hipErrorInvalidValue;
    const AttnEqShape e =
        attn_eq_shape(rows, hq, hkv, n_keys, hd, dtype, part_rows, gemm_cu_count());
    const bool planned = plan && part_o && part_ml && e.use;  // as launch_attention_plan did
    int nrb, n_splits, split_keys = 0, n_tiles = 1, pack = 1, blocks;
    if (planned) {
      nrb = e.rb / 32;
      pack = e.pack;
      n_splits = e.max_pc;
      const long long n = ((long long)rows * pack + e.rb - 1) / e.rb;
      blocks = (int)std::max<long long>(n, e.budget) * (pack > 1 ? hkv : hq);
    } else {
      nrb = attn_waves(rows, hq);
      n_splits = part_o && part_ml ? attn_splits(rows, hq, hkv, n_keys) : 1;
      if ((long long)n_splits * rows > part_rows)
        n_splits = (int)std::max(1LL, part_rows / rows);
      split_keys = attn_split_keys(n_keys, n_splits);
      n_tiles = (rows + 32 * nrb - 1) / (32 * nrb);
      blocks = n_tiles * hq * n_splits;
    }
    const bool halves = planned && (pack > 1 || n_splits > kAttnMaxPieces);  // (see pack_part)
    const dim3 g(blocks), b(64 * nrb);
    const int4 *P = planned ? reinterpret_cast<const int4 *>(plan) : nullptr;
#define AKVS_ATTN(HD_, PREF_)                                                                    \
  hipLaunchKernelGGL((k_attn_bf16<HD_, PREF_>), g, b, 0, s, Q, pos, pos0, rows, rows_dev, K, V,    \
                     n_keys, hq, hkv, pack, halves, nrb, n_tiles, n_splits, split_keys,            \
                     scale_log2, O, reinterpret_cast<bf16_t *>(part_o), part_ml, row_base, P)
    if (hd == 128) {
      AKVS_ATTN(128, false);  // the direct-to-LDS staging, 4- and 8-wave blocks alike
    } else {
      if (nrb == 4) AKVS_ATTN(64, true); else AKVS_ATTN(64, false);  // (see PREF in the kernel)
    }
#undef AKVS_ATTN
    if (n_splits > 1) {
      hipError_t er = hipGetLastError();
      if (er != hipSuccess) return er;
      const dim3 gc((unsigned)(((long long)rows * hq * (hd / 8) + 255) / 256)), bc(256);
      const bf16_t *po = reinterpret_cast<const bf16_t *>(part_o);
      if (n_splits <= 8)
        hipLaunchKernelGGL((k_attn_combine<8>), gc, bc, 0, s, po, part_ml, n_splits, rows, rows_dev,
                           hq, hd, O, row_base, P, halves);
      else
        hipLaunchKernelGGL((k_attn_combine<16>), gc, bc, 0, s, po, part_ml, n_splits, rows,
                           rows_dev, hq, hd, O, row_base, P, halves);
    }
  } else {
    const float scale = 1.4426950408889634f / sqrtf((float)hd);
    dim3 g((rows + 15) / 16, hq), b(512);
    const float *Q = reinterpret_cast<const float *>(q);
    const float *K = reinterpret_cast<const float *>(k);
    const float *V = reinterpret_cast<const float *>(v);
    float *O = reinterpret_cast<float *>(out);
    if (hd == 128)
      hipLaunchKernelGGL(k_attn_f32<128>, g, b, 0, s, Q, pos, pos0, rows, rows_dev, K, V, n_keys,
                         hq, hkv, scale, O, row_base);
    else
      hipLaunchKernelGGL(k_attn_f32<64>, g, b, 0, s, Q, pos, pos0, rows, rows_dev, K, V, n_keys,
                         hq, hkv, scale, O, row_base);
  }
  return hipGetLastError();
}

}  // namespace akvs
