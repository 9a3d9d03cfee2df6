// Scoring pass kernels, gfx950 (Sec. 3.3 Eq. 6-7; Algorithm 1 scoring loop).
// Visual keys are located through the image table (copied into LDS), so no
// index map is built beforehand.
//
// Once every span row's log-sum-exp b_r (log2 domain) is known, the visual
// column sums of Eq. 6 are  sum_r 2^(c * <q_r, k_t> - b_r)  with
// c = scale * log2(e).  A workgroup owns 256 visual keys of one KV head and
// streams all (span token, grouped head) rows of that head past them:
// S = Q K^T with v_mfma_f32_32x32x16_bf16 puts one key column in each lane
// (16 rows per lane), so the column sums accumulate in-lane.  The same
// workgroup reads its keys' V rows once for the value-norm proxy (the norm of
// the concatenated cached heads), so the cache is read once per layer.
// Per-KV-head partials are reduced in a fixed order by the finalize kernel,
// which also applies the 1/(n_q H_q) mean and accumulates the layer into
// s = sum_l a v and A = sum_l a (Eq. 7).
#include <type_traits>

#include "common.h"

namespace conduit {
namespace {

constexpr float kInf = __builtin_inff();


// Finalize of one visual token: fixed-order sum over KV heads, the mean (or
// RMS) over rows and heads, the value norm, s = a v and the layer
// accumulation of Eq. 7.
// COHERENT: the partials were written by other workgroups of the running
// kernel with device-coherent stores, and are read the same way.
template <bool COHERENT = false>
__device__ __forceinline__ void finalize_token(const FinalizeParams &p, int t) {
  auto ld = [](const float *q) {
    return COHERENT ? __hip_atomic_load(q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : *q;
  };
  float cs = 0.f, sq = 0.f;
  for (int h = 0; h < p.n_kv_heads; ++h) {
    cs += ld(p.colsum_part + (int64_t)h * p.n_vis + t);
    if (!p.vnorm_in) sq += ld(p.vsq_part + (int64_t)h * p.n_vis + t);
  }
  const float a = p.rms ? sqrtf(cs / p.n_rows_f) : cs / p.n_rows_f;
  const float v = p.vnorm_in ? p.vnorm_in[t] : sqrtf(sq);
  const float s = a * v;
  if (p.accumulate) {
    p.s_acc[t] += s;
    p.a_acc[t] += a;
  } else {
    p.s_acc[t] = s;
    p.a_acc[t] = a;
  }
  if (p.a_out) p.a_out[t] = a;
  if (p.vnorm_out) p.vnorm_out[t] = v;
}


// The workgroups of the n_kv_heads KV heads of one key block each count
// their arrival once their partials are stored (device-coherent stores,
// waited for before the count); the last to arrive finalizes the block's
// keys, reading every head's partials in head order with device-coherent
// loads, as the finalize kernel does.  The counters are cleared by the kernel
// that runs before this one.  (A device-scope release/acquire fence pair per
// workgroup would write back and invalidate the XCD's L2 each time, which
// costs more than the separate finalize launch.)
// With several layers in the launch (nb > 0) the last of the nb * n_kv_heads
// workgroups of a key block finalizes every layer in layer order: the same
// fp32 additions, in the same order, as one finalize per layer.
__device__ __forceinline__ void finalize_layers_token(const FinalizeParams &p, const LayerTable &lt, int nb, int t) {
  const int64_t stride = (int64_t)p.n_kv_heads * p.n_vis;
  float s_acc = 0.f, a_acc = 0.f;
  for (int l = 0; l < nb; ++l) {
    float cs = 0.f, sq = 0.f;
    const float *vn = layer_entry(lt.vnorm, l);
    for (int h = 0; h < p.n_kv_heads; ++h) {
      const int64_t i = l * stride + (int64_t)h * p.n_vis + t;
      cs += __hip_atomic_load(const_cast<float *>(p.colsum_part + i), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (!vn) sq += __hip_atomic_load(const_cast<float *>(p.vsq_part + i), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    const float a = p.rms ? sqrtf(cs / p.n_rows_f) : cs / p.n_rows_f;
    const float v = vn ? vn[t] : sqrtf(sq);
    const float sv = a * v;
    if (l == 0 && !p.accumulate) {
      s_acc = sv;
      a_acc = a;
    } else {
      if (l == 0) {
        s_acc = p.s_acc[t];
        a_acc = p.a_acc[t];
      }
      s_acc += sv;
      a_acc += a;
    }
  }
  p.s_acc[t] = s_acc;
  p.a_acc[t] = a_acc;
}

__device__ __forceinline__ void finalize_when_last(const ColsumParams &p, const LayerTable &lt, int tid,
                                                   int n_threads) {
  __shared__ int s_last;
  __builtin_amdgcn_s_waitcnt(0);  // this wave's partial stores are complete
  __syncthreads();
  const int arrivals = p.n_kv_heads * (lt.n > 0 ? lt.n : 1);
  if (tid == 0)
    s_last = __hip_atomic_fetch_add(p.done + blockIdx.x, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) ==
             arrivals - 1;
  __syncthreads();
  if (!s_last) return;
  for (int i = tid; i < kColsumKeysPerBlock; i += n_threads) {
    const int t = blockIdx.x * kColsumKeysPerBlock + i;
    if (t >= p.n_vis) continue;
    if (lt.n > 0) finalize_layers_token(p.fin, lt, lt.n, t);
    else finalize_token<true>(p.fin, t);
  }
}

// One 1 KB direct-to-LDS transfer through a buffer resource (lane l's 16 bytes
// at byte voff land at LDS byte lds_addr + Imm + 16 l), written as assembly so
// that the compiler does not make every later LDS read wait for it, awaited by
// hand before the barrier that publishes it.
template <int Imm>
__device__ __forceinline__ void lds_dma16(__amdgpu_buffer_rsrc_t r, uint32_t lds_addr, uint32_t voff) {
  asm volatile("s_add_u32 m0, %0, %3\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds"
               :
               : "s"(lds_addr), "v"(voff), "s"(r), "i"(Imm)
               : "memory", "m0", "scc");
}

// The streamed rows' tiles: kQTile (span token, head) rows, D + 8 elements
// apart (the lanes of an operand read cover distinct banks), a whole number of
// 1 KB transfers.
constexpr int kQTile = 64;
constexpr int kQStages = 4;
constexpr int kBTiles = 8;
constexpr int kMergeRows = 2;    // rows per thread that are merged at once
constexpr int kMergeLoads = 6;   // splits asked for together
template <int D, bool MERGE>
struct ColsumSmem {
  alignas(16) u16 q[kQStages][kQTile][D + 8];
  // MERGE: every row's, else a ring
  alignas(16) float nb[MERGE ? kColsumMaxLsePairs / kQTile : kBTiles][kQTile];  // -b of the tiles' rows (doubled for RMS; past the last row: -inf)
  uint32_t off[kBTiles][kQTile];          // byte offsets of the tiles' rows
  int64_t row[kColsumKeysPerBlock];       // cache row of each key of the workgroup
  ImageLds img;
};

// RMS: accumulate alpha^2 = 2^(2 (c z - b)) (Eq. 4's surrogate) instead of
// alpha: the scale and b are doubled (exact).
// lt.n > 0: several layers, layer blockIdx.z (the column sums and norms of
// layer l sit l strides further on).
//
// A workgroup covers 256 keys; every wave holds the K rows of 32 NC of them and
// takes every row.  The loop runs over 32-row sub-tiles i with one product per
// slot: S(i+1) = Q K^T from the operand ring while 2^(c S(i) - b) is summed on
// the VALU and the ring receives the operands of i + 2; the last pair of tiles
// stands behind the loop, without transfers, and its last sub-tile without
// products.  The loop is bound by instruction issue (a product with 2
// exponentials, 2 FMAs and 2 additions takes 42 cycles at two waves per SIMD,
// each LDS read about 13 more, the product alone 32).
// NC = 2: 4 waves, each Q operand read from LDS feeds two products, and two
// workgroups per CU, so that one's start and end (K rows, norms, the finalize
// handoff: about 8 us against 25 of the loop at 1,792 rows) run beside the
// other's loop.  65,536 keys x 1,792 rows x 4 layers take 66 cycles per product
// over the whole kernel.
// NC = 1 (launches whose workgroups do not fill the chip twice): 8 waves, for
// start and end count there, and with 32 keys a wave asks for half the K rows
// and has half the products before its first sum.  A form with 64 keys and one
// row half of every tile per wave fetched each K row twice: whole scoring
// passes with given row statistics, that form and this one, 27.0 and 25.1 us
// (16,384 keys x 896 rows), 14.5 and 13.2 (1,892 x 119); d = 64, 38,087 x 161
// rows without, 37.9 and 31.6 (two workgroups per CU where the registers of d =
// 64 allow it).
// MERGE (NC = 1 only): the rows' b are merged from the statistics' split
// partials by every workgroup, asked for at its start and reduced after the K
// rows have been asked for, in place of the statistics kernel's merge, whose
// chain of waits at its end costs about 4 us (16k scoring 49.6 us with this
// merge and 54.0 with that one and 4 waves).  Rows and splits that there are
// not are left out (3,244 keys x 161 rows, 7 splits: 14.3 us with all 24 splits
// of two rows per thread reduced, 12.8 now).
template <int D, int NC, bool MERGE>
__global__ __launch_bounds__(512 / NC, NC == 1 && D == 64 && !MERGE ? 4 : 2) void colsum_bf16_kernel(
    ColsumParams p, LayerTable lt, int rms) {
  constexpr int KS = D / 16;
  constexpr int W = 8 / NC, kThreads = 64 * W;
  // The parameter block is read in one go: the empty statement makes every
  // scalar due here, otherwise each is loaded where it is first used, a chain
  // of about a dozen round trips before the first product.  The image table's
  // entries are on their way meanwhile.
  const int tid = threadIdx.x;
  const int img_off = p.tbl.off[min(tid, kMaxImages - 1)], img_pos = p.tbl.pos[min(tid, kMaxImages - 1)];
  asm volatile("" ::"s"(p.k), "s"(p.v), "s"(p.q), "s"(p.row_b), "s"(p.vnorm_in), "s"(p.colsum_part), "s"(p.vsq_part),
               "s"(p.k_stride), "s"(p.v_stride), "s"(p.pages.table), "s"(p.pages.shift), "s"(p.pages.n_pages),
               "s"(p.n_kv_heads), "s"(p.group), "s"(p.n_q_heads), "s"(p.n_q), "s"(p.n_vis), "s"(p.scale_log2),
               "s"(p.clear_u32), "s"(p.clear_n), "s"(p.done), "s"(p.tbl.n_images), "s"(lt.n));
  if constexpr (MERGE)
    asm volatile("" ::"s"(p.lse_part_m), "s"(p.lse_part_l), "s"(p.lse_ns), "s"(p.lse_layer_stride), "s"(p.lse_out));
  // This layer's pointers, in locals: p itself stays unwritten (a written
  // kernel parameter holding the image table would be copied to scratch).
  const bool ml = lt.n > 0;
  const int layer = ml ? (int)blockIdx.z : 0;
  const int64_t part_off = (int64_t)layer * p.n_kv_heads * p.n_vis;
  const void *k_l = ml ? layer_entry(lt.k, layer) : p.k;
  const void *v_l = ml ? layer_entry(lt.v, layer) : p.v;
  const void *q_l = ml ? layer_entry(lt.q, layer) : p.q;
  const float *row_b = ml ? layer_entry(lt.rowb, layer) : p.row_b;
  const float *vnorm_in = ml ? layer_entry(lt.vnorm, layer) : p.vnorm_in;
  float *colsum_part = p.colsum_part + part_off;
  float *vsq_part = p.vsq_part + part_off;
  __shared__ ColsumSmem<D, MERGE> sm;
  float *const nb = &sm.nb[0][0];

  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int col = lane & 31, half = lane >> 5;
  const int key0 = wave * 32 * NC;
  const int blk_key0 = blockIdx.x * kColsumKeysPerBlock;
  const int kvh = blockIdx.y;
  const int G = p.group;
  const int n_pair = p.n_q * G;
  const int n_tiles = (n_pair + kQTile - 1) / kQTile;
  const float b_scale = rms ? -2.f : -1.f;
  const float c = rms ? 2.f * p.scale_log2 : p.scale_log2;
  const u16 *Kg = static_cast<const u16 *>(k_l);
  const u16 *Vg = static_cast<const u16 *>(v_l);
  const u16 *Qg = static_cast<const u16 *>(q_l);
  // the statistics' merge marks, all read by now: unset for the next launch
  if (p.clear_u32)
    for (int i = ((blockIdx.z * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x) * kThreads + tid;
         i < p.clear_n; i += gridDim.x * gridDim.y * gridDim.z * kThreads)
      p.clear_u32[i] = 0;

  // Direct-to-LDS staging of Q tiles, two at a time: wave w takes transfers
  // w, w + W, ... below the last whole multiple of W of each tile, and one
  // left-over transfer (waves past the last repeat it: the same bytes to the
  // same place).  Row r of the KV head is span token r / G, head r mod G of
  // the group; each lane keeps the byte offset and the head of its row per
  // transfer and advances them by two tiles at a time.  Rows past n_pair lie
  // past the resource's bound and read as zeros (their 2^-inf adds nothing);
  // lanes that land in a row's padding start past it.
  constexpr int kPitchB = 2 * (D + 8);
  constexpr int kXfer = kQTile * kPitchB / 1024;
  static_assert(kXfer * 1024 == kQTile * kPitchB, "whole 1 KB transfers");
  constexpr int kFull = kXfer / W, kLeft = kXfer % W, kGroup = 2 * kFull + 1;
  static_assert(kLeft >= 1 && 2 * kLeft <= W, "one left-over transfer per wave");
  const int left = min(wave, 2 * kLeft - 1), left_x = kFull * W + left % kLeft;
  const bool left_b = left >= kLeft;  // of the second tile
  const uint32_t head_step = (uint32_t)D * 2u, tok_step = (uint32_t)p.n_q_heads * D * 2u;
  // Rows of two tiles at a time: their byte offsets from the KV head's first
  // row and their -b, one row per thread below 2 kQTile, kept as (token, head)
  // and advanced from pair to pair instead of being divided out; threads past
  // those rows do the same without storing.  Offsets go through a ring over
  // kBTiles tiles; transfer n of this lane reads its row's at off_at[n], and
  // adds its place in the row, chunk[n] (padding lanes: past the resource).
  const uint32_t r0 = tid & (2 * kQTile - 1);
  uint32_t row_tok = r0 / (uint32_t)G, row_head = r0 - row_tok * G;
  const uint32_t tok_adv = 2 * kQTile / (uint32_t)G, head_adv = 2 * kQTile % (uint32_t)G;
  const auto b_rsrc = buffer_rsrc(row_b, p.n_q * p.n_q_heads * 4);
  auto next_rows = [&]() __attribute__((always_inline)) {
    row_tok += tok_adv;
    row_head += head_adv;
    const bool wrap = row_head >= (uint32_t)G;
    row_tok += wrap;
    row_head -= wrap ? G : 0;
  };
  auto load_b = [&]() __attribute__((always_inline)) {
    return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(
                                         b_rsrc, (row_tok * p.n_q_heads + kvh * G + row_head) * 4u, 0, 0));
  };
  auto row_off = [&]() __attribute__((always_inline)) { return row_tok * tok_step + (kvh * G + row_head) * head_step; };
  auto neg_b = [&](float b, int r) __attribute__((always_inline)) { return r < n_pair ? b_scale * b : -kInf; };
  uint32_t off_at[kGroup], chunk[kGroup];
#pragma unroll
  for (int n = 0; n < kGroup; ++n) {
    const int x = n < 2 * kFull ? wave + W * (n / 2) : left_x;
    const int b = x * 1024 + 16 * lane, ch = (b % kPitchB) / 16;
    off_at[n] = b / kPitchB;
    chunk[n] = ch < D / 8 ? 16u * ch : 0x80000000u;
    asm volatile("" : "+v"(off_at[n]), "+v"(chunk[n]));
  }
  const auto q_rsrc = buffer_rsrc(Qg, p.n_q * p.n_q_heads * D * 2);
  const uint32_t q_lds = (uint32_t)(uintptr_t)&sm.q[0][0][0] + wave * 1024;
  constexpr uint32_t kStageB = kQTile * kPitchB;
  // Transfer n of a tile pair whose row offsets are at off_a and off_b, into
  // the stages at LDS addresses s_a, s_b (this wave's first transfer).
  auto dma_q = [&](auto n_tag, const uint32_t *off_a, const uint32_t *off_b, uint32_t s_a, uint32_t s_b)
      __attribute__((always_inline)) {
    constexpr int n = decltype(n_tag)::value;
    if constexpr (n < 2 * kFull) {
      lds_dma16<n / 2 * W * 1024>(q_rsrc, n & 1 ? s_b : s_a, (n & 1 ? off_b : off_a)[off_at[n]] + chunk[n]);
    } else {
      lds_dma16<0>(q_rsrc, (left_b ? s_b : s_a) + (left_x - wave) * 1024, (left_b ? off_b : off_a)[off_at[n]] + chunk[n]);
    }
  };
  auto each = [&](auto f) __attribute__((always_inline)) {  // f(n) for every transfer of the pair
    auto one = [&](auto n) __attribute__((always_inline)) {
      if constexpr (decltype(n)::value < kGroup) f(n);
    };
    one(std::integral_constant<int, 0>{});
    one(std::integral_constant<int, 1>{});
    one(std::integral_constant<int, 2>{});
    one(std::integral_constant<int, 3>{});
    one(std::integral_constant<int, 4>{});
    one(std::integral_constant<int, 5>{});
    one(std::integral_constant<int, 6>{});
    one(std::integral_constant<int, 7>{});
    one(std::integral_constant<int, 8>{});
    static_assert(kGroup <= 9, "every transfer");
  };
  // Offsets of tiles 0..5 and -b of tiles 0..3.  (Threads of the upper half
  // hold the same rows as the lower half's: they take the odd pairs.)
  // The loads of b (MERGE: of the first rows' split partials) stay in flight
  // until the K rows have been asked for.
  float b_first = 0.f;
  // MERGE: b = M + log2(sum_s l_s 2^(m_s - M)) over the splits of a row, in
  // split order, kMergeRows rows r0 + tid + i kThreads per thread (as far as
  // there are any), kMergeLoads splits in one go (as far as there are any);
  // the first key block also writes lse_out.  Slot (pb n_kv_heads + kvh) ns + s
  // holds split s of the rows of block pb.
  float mv[kMergeRows][MERGE ? kLseRegSplits : 1], lv[kMergeRows][MERGE ? kLseRegSplits : 1];
  auto ask_rows = [&](int r0) __attribute__((always_inline)) {
    constexpr int ppb = attn_pairs_per_block(false);
    const float *pm = p.lse_part_m + layer * p.lse_layer_stride, *pl = p.lse_part_l + layer * p.lse_layer_stride;
#pragma unroll
    for (int i = 0; i < kMergeRows; ++i) {
      if (i > 0 && r0 + i * kThreads >= n_pair) break;
      const uint32_t r = (uint32_t)min(r0 + tid + i * kThreads, n_pair - 1), pb = r / ppb;
      const int64_t at = ((int64_t)pb * p.n_kv_heads + kvh) * p.lse_ns * ppb + (r - pb * ppb);
#pragma unroll
      for (int s0 = 0; s0 < kLseRegSplits; s0 += kMergeLoads) {
        if (s0 < p.lse_ns) {
#pragma unroll
          for (int u = 0; u < kMergeLoads; ++u) {
            const int64_t e = at + (int64_t)min(s0 + u, p.lse_ns - 1) * ppb;
            mv[i][s0 + u] = pm[e];
            lv[i][s0 + u] = pl[e];
          }
        }
      }
    }
  };
  auto merge_rows = [&](int r0) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < kMergeRows; ++i) {
      if (i > 0 && r0 + i * kThreads >= n_pair) break;
      const int r = r0 + tid + i * kThreads;
      float M = mv[i][0], L = 0.f;
#pragma unroll
      for (int s0 = 0; s0 < kLseRegSplits; s0 += kMergeLoads)
        if (s0 < p.lse_ns) {
#pragma unroll
          for (int u = 0; u < kMergeLoads; ++u) M = fmaxf(M, mv[i][s0 + u]);  // (clamped loads repeat the last split)
        }
#pragma unroll
      for (int s0 = 0; s0 < kLseRegSplits; s0 += kMergeLoads)
        if (s0 < p.lse_ns) {
#pragma unroll
          for (int u = 0; u < kMergeLoads; ++u)
            L += s0 + u < p.lse_ns ? fast_exp2(mv[i][s0 + u] - M) * lv[i][s0 + u] : 0.f;
        }
      const float b = M + __log2f(L);
      if (r < n_tiles * kQTile) nb[r] = neg_b(b, r);
      if (p.lse_out && !ml && blockIdx.x == 0 && r < n_pair)
        p.lse_out[(int64_t)(r / G) * p.n_q_heads + kvh * G + r % G] = b * kLn2;
    }
  };
  if constexpr (MERGE) ask_rows(0);
  {
    if (wave == 2 || wave == 3) next_rows();
    if (wave < 4) {
      sm.off[0][tid] = row_off();
      if constexpr (!MERGE) b_first = load_b();
    }
    if (wave < 2) {  // to the rows of tiles 4 and 5
      next_rows();
      next_rows();
      sm.off[4][tid] = row_off();
    }
  }
  // The image table, before the transfers: a wait for it behind them would
  // wait for them too.
  static_assert(kThreads >= kMaxImages, "one image per thread");
  if (tid < p.tbl.n_images) {
    sm.img.off[tid] = img_off;
    sm.img.pos[tid] = img_pos;
  }
  if (tid == 0) {
    sm.img.off[p.tbl.n_images] = p.n_vis;
    sm.img.n_images = p.tbl.n_images;
  }
  __syncthreads();
  // tiles 0, 1 and 2 (the first iteration takes 3)
  each([&](auto n) __attribute__((always_inline)) { dma_q(n, sm.off[0], sm.off[1], q_lds, q_lds + kStageB); });
  // (a span of one or two tiles uses nothing of what it reads from them:
  // 16,384 keys of 8 heads of 128, 68 rows each: 39.2 us a pass with these
  // transfers, 38.7 without)
  if (n_tiles > 2)
    each([&](auto n) __attribute__((always_inline)) {
      if (decltype(n)::value < 2 * kFull ? decltype(n)::value % 2 == 0 : !left_b)
        dma_q(n, sm.off[2], sm.off[3], q_lds + 2 * kStageB, q_lds + 3 * kStageB);
    });

  // This lane's key columns, held as the B operands for every row tile.
  bf16x8 kreg[NC][KS];
  {
    // the keys' cache rows (page lookup included), also kept for the V rows;
    // the searches of the image table step together
    int tk[NC], lo[NC], hi[NC];
#pragma unroll
    for (int cb = 0; cb < NC; ++cb) {
      tk[cb] = min(blk_key0 + key0 + cb * 32 + col, p.n_vis - 1);
      lo[cb] = 0;
      hi[cb] = sm.img.n_images - 1;
    }
    while (lo[0] < hi[0] || lo[NC - 1] < hi[NC - 1]) {
#pragma unroll
      for (int cb = 0; cb < NC; ++cb) {
        const int mid = (lo[cb] + hi[cb] + 1) >> 1;
        const bool up = sm.img.off[mid] <= tk[cb];
        lo[cb] = up ? mid : lo[cb];  // lo = hi stays: its offset is at most tk
        hi[cb] = up ? hi[cb] : mid - 1;
      }
    }
    int64_t row[NC];
#pragma unroll
    for (int cb = 0; cb < NC; ++cb)
      row[cb] = kv_row(p.pages, sm.img.pos[lo[cb]] + (tk[cb] - sm.img.off[lo[cb]]));
#pragma unroll
    for (int cb = 0; cb < NC; ++cb) {
      if (half == 0) sm.row[key0 + cb * 32 + col] = row[cb];
      const u16 *krow = Kg + row[cb] * p.k_stride + kvh * D + 8 * half;
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) kreg[cb][ks] = as_bf16x8(ld16(krow + ks * 16));
    }
  }
  if constexpr (MERGE) {
    merge_rows(0);
    for (int r0 = kMergeRows * kThreads; r0 < n_pair; r0 += kMergeRows * kThreads) {
      ask_rows(r0);
      merge_rows(r0);
    }
  } else {
    if (wave < 4) nb[tid] = neg_b(b_first, tid);
  }
  __builtin_amdgcn_s_waitcnt(0);  // this wave's Q transfers (invisible to the compiler)
  __syncthreads();

  // S of sub-tile 0, the operands of sub-tile 1.
  bf16x8 ring[KS];
  f32x16 sa[NC], sb[NC];
  {
    const u16 *qrow = &sm.q[0][col][8 * half];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) ring[ks] = as_bf16x8(ld16(qrow + ks * 16));
#pragma unroll
    for (int cb = 0; cb < NC; ++cb) {
      sa[cb] = f32x16{};
#pragma unroll
      for (int ks = 0; ks < KS; ++ks)
        sa[cb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ring[ks], kreg[cb][ks], sa[cb], 0, 0, 0);
    }
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) ring[ks] = as_bf16x8(ld16(qrow + 32 * (D + 8) + ks * 16));
  }
  __syncthreads();  // every wave has read these tiles: the first iteration refills their stages

  float colsum[NC] = {};
  constexpr int kVPer = 16 / (NC * KS);  // accumulator registers (of every column) per slot
  // -b of the rows of sub-tile `sub` of a tile that this lane holds: register
  // v of lane (col, half) is row 8*(v/4) + 4*half + v%4 of its sub-tile
  auto b_of = [&](int tile, int sub) __attribute__((always_inline)) {
    return nb + (MERGE ? tile : tile & (kBTiles - 1)) * kQTile + 32 * sub + 4 * half;
  };
  f32x4 nb4 = *reinterpret_cast<const f32x4 *>(b_of(0, 0));  // rows 0..3 of the current sub-tile
  // One sub-step: cur = S(i), with b at bp; nxt receives S(i+1) from the ring
  // (Ops >= 1), the ring rows qsub * 32.. of stage qst (Ops = 2); bn: b of
  // sub-tile i + 1.
  auto step = [&](auto ops_tag, f32x16 (&cur)[NC], f32x16 (&nxt)[NC], int qst, int qsub, const float *bp,
                  const float *bn, auto hook) __attribute__((always_inline)) {
    constexpr int Ops = decltype(ops_tag)::value;
    const u16 *qrow = &sm.q[qst][32 * qsub + col][8 * half];
    f32x4 nbn = nb4;
    float last[NC] = {}, psum[NC] = {};
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int j = 0; j < NC * KS; ++j) {
      const int op = j / NC, cb = j % NC;
      if constexpr (Ops >= 1)
        nxt[cb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ring[op], kreg[cb][op], op == 0 ? f32x16{} : nxt[cb], 0, 0, 0);
      if constexpr (Ops == 2) {
        if (cb == NC - 1 && (op & 1)) {
          ring[op] = as_bf16x8(ld16(qrow + op * 16));
          ring[op - 1] = as_bf16x8(ld16(qrow + (op - 1) * 16));
        }
      }
#pragma unroll
      for (int v = j * kVPer; v < (j + 1) * kVPer; ++v) {
        if (v % 4 == 0) {  // the next four rows' b, four registers ahead
          nb4 = nbn;
          nbn = *reinterpret_cast<const f32x4 *>(v < 12 ? bp + 8 * (v / 4 + 1) : bn);
        }
#pragma unroll
        for (int u = 0; u < NC; ++u) {
          const float pe = fast_exp2(fmaf(cur[u][v], c, nb4[v % 4]));
          asm volatile("" ::"v"(pe));
          psum[u] += last[u];
          asm volatile("" ::"v"(psum[u]));
          last[u] = pe;
        }
      }
      hook(j);
      if constexpr (Ops >= 1) __builtin_amdgcn_sched_barrier(0);
    }
    nb4 = nbn;
#pragma unroll
    for (int u = 0; u < NC; ++u) {
      colsum[u] += psum[u] + last[u];
      asm volatile("" ::"v"(colsum[u]));
    }
  };
  constexpr std::integral_constant<int, 0> kSumOnly{};
  constexpr std::integral_constant<int, 1> kNoRead{};
  constexpr std::integral_constant<int, 2> kAll{};
  auto no_hook = [](int) __attribute__((always_inline)) {};
  // V rows of the workgroup's keys for the value norms (not read when the
  // norms are given), kVBatch 16-byte pieces per thread at a time; the first
  // batch arrives during the last but one iteration.
  const bool read_v = vnorm_in == nullptr;
  constexpr bool kVEarly = NC == 1;
  constexpr int VPT = kColsumKeysPerBlock * D / 8 / kThreads, kVBatch = VPT < 8 ? VPT : 8;
  u32x4 vv[kVBatch] = {};
  auto load_v = [&](int i0) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < kVBatch; ++i) {
      const int vi = tid + kThreads * (i0 + i);
      vv[i] = ld16(Vg + sm.row[vi / (D / 8)] * p.v_stride + kvh * D + (vi % (D / 8)) * 8);
    }
  };
  // Two tiles (t, t+1) per barrier while two more follow: reads tiles t+1,
  // t+2 while t+3, t+4 arrive.
  const int t_last = (n_tiles - 1) & ~1;  // the last pair (its second tile may not exist)
  constexpr int kMod = kBTiles - 1;
  int t = 0, st = 0;
  for (; t < t_last; t += 2, st ^= 2) {
    const int s1 = st + 1, s2 = st ^ 2, s3 = (st ^ 2) + 1;  // stages of t+1, t+2, t+3
    constexpr int kStep = NC * KS, kSpread = 4 * kStep / kGroup;
    static_assert(kSpread >= 1, "every transfer has a slot");
    const uint32_t *off_a = sm.off[(t + 4) & kMod], *off_b = sm.off[(t + 3) & kMod];
    const uint32_t s_a = q_lds + st * kStageB, s_b = q_lds + s3 * kStageB;
    auto slot = [&](int g) __attribute__((always_inline)) {
      each([&](auto n) __attribute__((always_inline)) {
        if (g == decltype(n)::value * kSpread) dma_q(n, off_a, off_b, s_a, s_b);
      });
    };
    if (kVEarly && read_v && t == t_last - 2) load_v(0);
    // -b of the rows of tiles t+4, t+5 and the offsets of t+6, t+7
    float bv = 0.f;
    if (wave < 2) {
      if constexpr (!MERGE) bv = load_b();
      next_rows();
      sm.off[(t + 6) & kMod][tid] = row_off();
    }
    step(kAll, sa, sb, s1, 0, b_of(t, 0), b_of(t, 1), [&](int j) __attribute__((always_inline)) { slot(j); });
    step(kAll, sb, sa, s1, 1, b_of(t, 1), b_of(t + 1, 0), [&](int j) __attribute__((always_inline)) { slot(kStep + j); });
    step(kAll, sa, sb, s2, 0, b_of(t + 1, 0), b_of(t + 1, 1),
         [&](int j) __attribute__((always_inline)) { slot(2 * kStep + j); });
    step(kAll, sb, sa, s2, 1, b_of(t + 1, 1), b_of(t + 2, 0),
         [&](int j) __attribute__((always_inline)) { slot(3 * kStep + j); });
    if (!MERGE && wave < 2) sm.nb[(t + 4) & kMod][tid] = neg_b(bv, (t + 4) * kQTile + tid);
    __builtin_amdgcn_s_waitcnt(0);  // this wave's transfers have landed
    __syncthreads();
  }
  // The last one or two tiles: everything they need is there.
  if (read_v && (!kVEarly || t_last == 0)) load_v(0);
  const bool pair = t + 1 < n_tiles;
  if (pair) {
    step(kAll, sa, sb, st + 1, 0, b_of(t, 0), b_of(t, 1), no_hook);
    step(kAll, sb, sa, st + 1, 1, b_of(t, 1), b_of(t + 1, 0), no_hook);
  }
  const float *b0 = b_of(pair ? t + 1 : t, 0), *b1 = b_of(pair ? t + 1 : t, 1);
  step(kNoRead, sa, sb, 0, 0, b0, b1, no_hook);
  step(kSumOnly, sb, sa, 0, 0, b1, b1, no_hook);

  // The lanes' halves of a key's rows.
#pragma unroll
  for (int cb = 0; cb < NC; ++cb) {
    colsum[cb] += __shfl_xor(colsum[cb], 32, 64);
    const int tk = blk_key0 + key0 + cb * 32 + col;
    if (half == 0 && tk < p.n_vis) store_coherent(colsum_part + (int64_t)kvh * p.n_vis + tk, colsum[cb]);
  }

  // Value-norm proxy: this head's share of ||V_t||^2.  Item vi covers
  // dims (vi % (D/8))*8 .. +7 of key vi / (D/8); the D/8 items of a key sit
  // in consecutive lanes and are summed with lane shuffles.
  static_assert((D / 8) <= 64 && 64 % (D / 8) == 0 && VPT % kVBatch == 0, "key items within a wave, whole batches");
  for (int i0 = 0; read_v && i0 < VPT; i0 += kVBatch) {
    if (i0 > 0) load_v(i0);
#pragma unroll
    for (int i = 0; i < kVBatch; ++i) {
      float sq = 0.f;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float lo = __builtin_bit_cast(float, vv[i][e] << 16);
        const float hi = __builtin_bit_cast(float, vv[i][e] & 0xffff0000u);
        sq = fmaf(lo, lo, sq);
        sq = fmaf(hi, hi, sq);
      }
#pragma unroll
      for (int o = 1; o < D / 8; o <<= 1) sq += __shfl_xor(sq, o, 64);
      const int vi = tid + kThreads * (i0 + i), tv = blk_key0 + vi / (D / 8);
      if (vi % (D / 8) == 0 && tv < p.n_vis) store_coherent(vsq_part + (int64_t)kvh * p.n_vis + tv, sq);
    }
  }
  if (p.done) finalize_when_last(p, lt, tid, kThreads);
}

// fp32 path: one wave per 64 visual keys of one KV head.  Lane j holds the
// K row of key j in registers; the (span token, grouped head) query rows and
// their log-sum-exps pass through LDS in chunks of 64 (loaded coalesced, read
// as broadcasts), and the lane sums 2^(c z - b) (or its square) over them.
// The lane's V row gives its share of ||V_t||^2.
template <int D>
__global__ __launch_bounds__(64) void colsum_f32_kernel(ColsumParams p, bool rms) {
  __shared__ alignas(16) float qs[64][D];
  __shared__ float bs[64];
  const int lane = threadIdx.x;
  const int t = blockIdx.x * 64 + lane;
  const int kvh = blockIdx.y;
  const bool tvalid = t < p.n_vis;
  const float *Kg = static_cast<const float *>(p.k);
  const float *Vg = static_cast<const float *>(p.v);
  const float *Qg = static_cast<const float *>(p.q);
  const int64_t pos = kv_row(p.pages, vis_position(p.tbl, tvalid ? t : p.n_vis - 1));  // cache row
  float kr[D];
#pragma unroll
  for (int e = 0; e < D; e += 4) {
    const f32x4 x = *reinterpret_cast<const f32x4 *>(Kg + pos * p.k_stride + kvh * D + e);
    kr[e] = x[0];
    kr[e + 1] = x[1];
    kr[e + 2] = x[2];
    kr[e + 3] = x[3];
  }
  // The V row's share of ||V_t||^2, loaded with the K row (in flight during
  // the first query chunk).
  float sq = 0.f;
  if (!p.vnorm_in) {
    const float *vr = Vg + pos * p.v_stride + kvh * D;
#pragma unroll
    for (int e = 0; e < D; e += 4) {
      const f32x4 x = *reinterpret_cast<const f32x4 *>(vr + e);
#pragma unroll
      for (int u = 0; u < 4; ++u) sq = fmaf(x[u], x[u], sq);
    }
  }
  const int G = p.group, n_pair = p.n_q * G;
  float colsum = 0.f;
  for (int c0 = 0; c0 < n_pair; c0 += 64) {
    const int rows = min(64, n_pair - c0);
    for (int cidx = lane; cidx < rows * (D / 4); cidx += 64) {
      const int rr = cidx / (D / 4), c4 = cidx % (D / 4), pr = c0 + rr;
      const int64_t qrow = (int64_t)(pr / G) * p.n_q_heads + kvh * G + pr % G;
      *reinterpret_cast<f32x4 *>(&qs[rr][4 * c4]) = *reinterpret_cast<const f32x4 *>(Qg + qrow * D + 4 * c4);
    }
    if (lane < rows) {
      const int pr = c0 + lane;
      const int64_t gq = (int64_t)(pr / G) * p.n_q_heads + kvh * G + pr % G;
      if (p.f32_ml) {
        // the statistics' key splits, merged as their merge launch would:
        // b = M + log2(sum_s l_s 2^(m_s - M)), splits in order
        const int64_t n_gp = (int64_t)p.n_q * p.n_q_heads;
        float M = -kInf;
        for (int sp = 0; sp < p.lse_ns; ++sp) M = fmaxf(M, p.f32_ml[sp * n_gp + gq].x);
        float L = 0.f;
        for (int sp = 0; sp < p.lse_ns; ++sp) {
          const float2 ml = p.f32_ml[sp * n_gp + gq];
          const float w = ml.y > 0.f ? fast_exp2(ml.x - M) : 0.f;
          L = fmaf(w, ml.y, L);
        }
        const float b = M + __log2f(L);
        if (blockIdx.x == 0 && p.lse_out) p.lse_out[gq] = b * kLn2;
        bs[lane] = b;
      } else {
        bs[lane] = p.row_b[gq];
      }
    }
    __syncthreads();
    for (int rr = 0; rr < rows; ++rr) {
      float d4[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int e = 0; e < D; e += 4) {
        const f32x4 qq = *reinterpret_cast<const f32x4 *>(&qs[rr][e]);
#pragma unroll
        for (int u = 0; u < 4; ++u) d4[u] = fmaf(qq[u], kr[e + u], d4[u]);
      }
      const float dot = (d4[0] + d4[1]) + (d4[2] + d4[3]);
      const float z = fmaf(dot, p.scale_log2, -bs[rr]);
      colsum += fast_exp2(rms ? 2.f * z : z);
    }
    __syncthreads();
  }
  if (!tvalid) return;
  p.colsum_part[(int64_t)kvh * p.n_vis + t] = colsum;
  if (!p.vnorm_in) p.vsq_part[(int64_t)kvh * p.n_vis + t] = sq;
}

__global__ void finalize_kernel(FinalizeParams p) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t < p.n_vis) finalize_token<false>(p, t);
}

// Value-norm table (Eq. 7's proxy, tabulated when the cache is built): one
// wave per visual token sums the squares of its row_elems cached values
// (all KV heads concatenated), 16 bytes per lane and step.
template <bool BF16>
__global__ __launch_bounds__(256) void value_norms_kernel(const void *v, int64_t v_stride, KvPages pages,
                                                          int row_elems, ImageTable tbl, float *out) {
  const int t = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (t >= tbl.n_vis) return;
  constexpr int EPC = BF16 ? 8 : 4;  // elements per 16-byte chunk
  const char *row = static_cast<const char *>(v) + kv_row(pages, vis_position(tbl, t)) * v_stride * (BF16 ? 2 : 4);
  float sq = 0.f;
  for (int c = lane; c < row_elems / EPC; c += 64) {
    const u32x4 w = ld16(row + 16 * c);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      if (BF16) {
        const float lo = __builtin_bit_cast(float, w[e] << 16);
        const float hi = __builtin_bit_cast(float, w[e] & 0xffff0000u);
        sq = fmaf(lo, lo, sq);
        sq = fmaf(hi, hi, sq);
      } else {
        // The element goes through a scalar first: hipcc compiled a bit_cast
        // of the vector-element lvalue itself into a read of element 0.
        const uint32_t u = w[e];
        const float x = __builtin_bit_cast(float, u);
        sq = fmaf(x, x, sq);
      }
    }
  }
  sq = wave_sum(sq);
  if (lane == 0) out[t] = sqrtf(sq);
}

}  // namespace

hipError_t launch_value_norms(const void *v, int64_t v_stride, const KvPages &pages, int32_t row_elems,
                              bool bf16, const ImageTable &tbl, float *out, hipStream_t s) {
  ProfScope ps("value_norms", s);
  const int blocks = (tbl.n_vis + 3) / 4;
  if (bf16) value_norms_kernel<true><<<blocks, 256, 0, s>>>(v, v_stride, pages, row_elems, tbl, out);
  else value_norms_kernel<false><<<blocks, 256, 0, s>>>(v, v_stride, pages, row_elems, tbl, out);
  return hipGetLastError();
}

hipError_t launch_colsum(const ColsumParams &p, int head_dim, bool bf16, bool rms, hipStream_t s,
                         const LayerTable *lt) {
  const LayerTable lt0 = lt ? *lt : LayerTable{};
  if (bf16) {
    const dim3 grid((p.n_vis + kColsumKeysPerBlock - 1) / kColsumKeysPerBlock, p.n_kv_heads, lt0.n > 0 ? lt0.n : 1);
    // Two 4-wave workgroups per CU when the launch has that many, else 8-wave
    // ones: scoring with given row statistics, 8 and 4 waves, 128 rows x 28
    // heads at d = 128: 24.7 and 25.2 us with 256 workgroups, 55.1 and 48.8
    // with 564; d = 64, 16 heads: 16.2 and 16.9 with 256, 19.9 and 20.3 with
    // 440, 25.1 and 24.6 with 564.  (Between 257 and 511 workgroups d = 128
    // runs two rounds of 8-wave ones, 39.9 us with 440 against 35.3.)
    const bool two = colsum_blocks(p.n_vis, p.n_kv_heads, lt0.n > 0 ? lt0.n : 1) >= kColsumFourWaveBlocks;
    if (p.lse_part_m && (two || p.lse_ns > kLseRegSplits || (int64_t)p.n_q * p.group > kColsumMaxLsePairs))
      return hipErrorInvalidValue;
    ProfScope ps("colsum", s);
    auto launch = [&](auto d) {
      constexpr int D = decltype(d)::value;
      if (two) colsum_bf16_kernel<D, 2, false><<<grid, 256, 0, s>>>(p, lt0, rms);
      else if (p.lse_part_m) colsum_bf16_kernel<D, 1, true><<<grid, 512, 0, s>>>(p, lt0, rms);
      else colsum_bf16_kernel<D, 1, false><<<grid, 512, 0, s>>>(p, lt0, rms);
    };
    if (head_dim == 128) launch(std::integral_constant<int, 128>{});
    else launch(std::integral_constant<int, 64>{});
  } else {
    dim3 grid((p.n_vis + 63) / 64, p.n_kv_heads);
    ProfScope ps("colsum_f32", s);
    if (head_dim == 128) colsum_f32_kernel<128><<<grid, 64, 0, s>>>(p, rms);
    else colsum_f32_kernel<64><<<grid, 64, 0, s>>>(p, rms);
  }
  return hipGetLastError();
}

hipError_t launch_finalize(const FinalizeParams &p, hipStream_t s) {
  ProfScope ps("finalize", s);
  finalize_kernel<<<(p.n_vis + 255) / 256, 256, 0, s>>>(p);
  return hipGetLastError();
}

}  // namespace conduit
