// Residual value-write error of a refresh set, gfx950 (Eq. 3 of the local
// residual-staleness model; App. D.1 isotropic Monte Carlo displacements and
// App. D.3 projected error).
//
// For displacement sample m, span row i and query head h the residual is
//   y = sum over visual t not in T of alpha_{i,h,t} xi^(m)_t[kv(h)],
// with alpha the cached-key attention of the scoring pass (normalised by the
// row's log-sum-exp, which the caller supplies), and the kernel reports
// ||y||^2.  xi is either kappa ||V_t|| / sqrt(H_kv D) * z_t (z given) or the
// cached value itself (stale values zeroed, App. D.3).
//
// The bf16 path is one MFMA pass per (key split, 256-pair block, KV head,
// sample): S^T = K Q^T for 64 visual keys, alpha = 2^(c s - b) straight from
// the known log-sum-exp (no running maximum), times the key's displacement
// scale (0 for refreshed keys and past the last visual token), and
// y^T += Xi^T (sigma alpha)^T with the displacement tile read through
// transposing LDS reads.  Partial y per split go to the workspace;
// residual_sum_kernel adds them in split order and squares.
#include "common.h"

namespace conduit {
namespace {

constexpr int KT = kAttnKeyTile;
constexpr int kWaves = 8, kThreads = kWaves * 64;  // 32 pairs per wave

// K rows are D + 8 elements apart, displacement rows D + 16 and interleaved
// within 16-key blocks (transposing operand reads free of bank conflicts);
// both pitches make a tile a whole number of 1 KB direct-to-LDS transfers.
// Three K and four displacement stages.
template <int D>
struct ResidualSmem {
  static constexpr int kPitch = D + 8, xPitch = D + 16;
  alignas(16) u16 k[3][KT][kPitch];
  alignas(16) u16 x[4][KT][xPitch];
};
// Per-key metadata of the split, and the image table (which lies in the tile
// stages until the first transfers).
struct ResidualKeys {
  alignas(16) float scale[(kResidualMaxTiles + 1) * KT];  // displacement scale: sigma_t, 1, or 0 (refreshed, past the end)
  uint32_t row[kResidualMaxTiles * KT];                   // cache row
};

// One 1 KB direct-to-LDS transfer: lane l's 16 bytes at src land at LDS byte
// lds_addr + 16 l.  Written as assembly so that the compiler does not make
// every later LDS read wait for it; awaited by hand before the barrier that
// publishes the tile.
__device__ __forceinline__ void lds_dma16(const void *src, uint32_t lds_addr) {
  asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dwordx4 %1, off" : : "s"(lds_addr), "v"(src) : "memory", "m0");
}

// s_waitcnt vmcnt(N), the other counters left open.
template <int N>
__device__ __forceinline__ void vm_wait() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (15 << 8));
}

// The tile loop is the refresh attention's pipeline: sub-step i (32 keys)
// holds one matrix product per slot, S^T(i+1) = K Q^T and y^T += Xi^T(i-1)
// P^T(i-1), beside the 16 probabilities P(i) = sigma 2^(c S(i) - b) on the
// VALU; operands pass through one register ring, read eight products ahead,
// and the tiles arrive by direct-to-LDS transfers spread over the slots, one
// tile per barrier (the per-key metadata leave no room for two).  The displacement scale multiplies the probability in 32
// bits, so the displacement tile is staged as it lies in memory and the
// product is rounded to bf16 once.  (With tiles staged through registers, one
// product's operands read at a time and the VALU work behind the products,
// the matrix cores were busy 33% of the time: 230 us a pass at 16,384 visual
// tokens, 128 x 28 rows and 5 samples.)
template <int D>
__global__ __launch_bounds__(kThreads, 1) void residual_bf16_kernel(ResidualParams p) {
  constexpr int KS = D / 16;                     // MFMA k-steps over the head dim
  constexpr int DT = D / 32;                     // 32-row tiles of y^T
  using Sm = ResidualSmem<D>;
  __shared__ Sm sm;
  __shared__ ResidualKeys keys;
  static_assert(sizeof(ImageLds) <= sizeof(sm.k), "image table fits the stages");
  ImageLds &img = *reinterpret_cast<ImageLds *>(&sm.k[0][0][0]);

  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int col = lane & 31, half = lane >> 5;
  const int split = blockIdx.x, pb = blockIdx.y;
  const int kvh = blockIdx.z % p.n_kv_heads, m = blockIdx.z / p.n_kv_heads;
  const int G = p.group;
  const int n_pairs = p.n_q * G;
  const float c = p.scale_log2;
  const bool iso = p.vnorm != nullptr;
  const int v_lane = v_operand_lane_offset_il<Sm::xPitch>(lane);

  image_table_to_lds(p.tbl, img, tid, kThreads);

  // The pair column owned by this lane; its query and log-sum-exp.
  const int pair = pb * kResidualPairs + wave * 32 + col;
  const bool valid = pair < n_pairs;
  const int r = valid ? pair / G : 0;
  const int gpair = r * p.n_q_heads + kvh * G + (valid ? pair % G : 0);
  bf16x8 qreg[KS];
  {
    const u16 *qrow = static_cast<const u16 *>(p.q) + (int64_t)gpair * D + 8 * half;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) qreg[ks] = as_bf16x8(valid ? ld16(qrow + ks * 16) : u32x4{0, 0, 0, 0});
  }
  const float neg_b = valid ? -p.row_b[gpair] : 0.f;

  const int tv_beg = split * p.tiles_per_split * KT;
  const int n_keys = min(tv_beg + p.tiles_per_split * KT, p.n_vis) - tv_beg;
  const int n_t = (n_keys + KT - 1) / KT;
  __syncthreads();  // image table in LDS
  // Per-key metadata of the split, resolved once (keys past its end get
  // scale 0).
  for (int j = tid; j < (n_t + 1) * KT; j += kThreads) {
    const int tv = tv_beg + min(j, n_keys - 1);
    if (j < n_t * KT) keys.row[j] = (uint32_t)kv_row(p.pages, vis_position(img, tv));
    keys.scale[j] = j >= n_keys || p.refreshed[tv] ? 0.f : (iso ? p.vnorm[tv] * p.sigma_scale : 1.f);
  }
  __syncthreads();

  // Direct-to-LDS staging, a K tile and a displacement tile at a time: wave w
  // takes transfers w, w + 8, ... below the last whole multiple of 8 of each
  // and one of the left-over ones (waves past the last repeat it: the same
  // bytes to the same place).  Transfer n of this lane fills key at[n] of its
  // tile (keys past the split repeat its last), from byte pos[n] of that key's
  // row (lanes that land in a row's padding repeat its last chunk).
  constexpr int kXferK = KT * Sm::kPitch * 2 / 1024, kXferX = KT * Sm::xPitch * 2 / 1024;
  static_assert(kXferK * 1024 == KT * Sm::kPitch * 2 && kXferX * 1024 == KT * Sm::xPitch * 2, "whole transfers");
  constexpr int kFull = kXferK / kWaves, xFull = kXferX / kWaves;
  constexpr int kLeft = kXferK % kWaves, xLeft = kXferX % kWaves;
  static_assert(kLeft >= 1 && xLeft >= 1 && kLeft + xLeft <= kWaves, "one left-over transfer per wave");
  constexpr int kGroup = xFull + kFull + 1;  // per wave; n: displacement, K, left-over
  const int left = min(wave, kLeft + xLeft - 1);
  const bool left_k = left < kLeft;
  const int left_x = left_k ? kFull * kWaves + left : xFull * kWaves + left - kLeft;
  const uint32_t k_row_b = 2u * (uint32_t)p.k_stride;
  const uint32_t x_row_b = iso ? 2u * (uint32_t)(p.n_kv_heads * D) : 2u * (uint32_t)p.disp_stride;
  const char *const k_base = static_cast<const char *>(p.k) + kvh * D * 2;
  const char *const x_base = static_cast<const char *>(p.disp) + kvh * D * 2 +
                             (iso ? ((int64_t)m * p.n_vis + tv_beg) * x_row_b : (int64_t)0);
  auto is_k = [&](int n) __attribute__((always_inline)) { return n < xFull ? false : n < kGroup - 1 ? true : left_k; };
  auto xfer = [&](int n) __attribute__((always_inline)) {
    return n < xFull ? wave + kWaves * n : n < kGroup - 1 ? wave + kWaves * (n - xFull) : left_x;
  };
  int at[kGroup], pos[kGroup];
#pragma unroll
  for (int n = 0; n < kGroup; ++n) {
    const int pitch_b = 2 * (is_k(n) ? Sm::kPitch : Sm::xPitch);
    const int b = xfer(n) * 1024 + 16 * lane, lrow = b / pitch_b;
    at[n] = is_k(n) ? lrow : (lrow & ~15) | v_interleaved_key(lrow & 15);
    pos[n] = 16 * min((b % pitch_b) / 16, D / 8 - 1);
    asm volatile("" : "+v"(at[n]), "+v"(pos[n]));
  }
  // Row (of the K cache, or of the displacement) of transfer n's key: K tile
  // tk, displacement tile tx.
  auto row_of = [&](int n, int tk, int tx) __attribute__((always_inline)) {
    const int j = min((is_k(n) ? tk : tx) * KT + at[n], n_keys - 1);
    return !is_k(n) && iso ? (uint32_t)j : keys.row[j];
  };
  // Transfer n into K stage sk or displacement stage sx.
  auto dma = [&](int n, uint32_t row, int sk, int sx) __attribute__((always_inline)) {
    const uint32_t st = is_k(n) ? (uint32_t)(uintptr_t)&sm.k[sk][0][0] : (uint32_t)(uintptr_t)&sm.x[sx][0][0];
    const char *src = (is_k(n) ? k_base : x_base) + (uint64_t)row * (is_k(n) ? k_row_b : x_row_b) + pos[n];
    lds_dma16(src, __builtin_amdgcn_readfirstlane(st + xfer(n) * 1024));
  };

  f32x16 y[DT];
#pragma unroll
  for (int dt = 0; dt < DT; ++dt) y[dt] = f32x16{};

  if (n_t > 0) {
    // The first sub-step's y^T products have no probabilities yet (zeros):
    // their displacement operands (stage 3, X(-1)) are zeros too, for a
    // displacement may be infinite.
    for (int i = tid; i < 32 * Sm::xPitch / 8; i += kThreads) st16(&sm.x[3][32][0] + 8 * i, u32x4{0, 0, 0, 0});
    // K(0), X(0); K(1), X(1); K(2)
    uint32_t rows[kGroup];
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
      for (int n = 0; n < kGroup; ++n)
        if (i < 2 || is_k(n)) dma(n, row_of(n, i, i), i, i);
#pragma unroll
    for (int n = 0; n < kGroup; ++n) rows[n] = row_of(n, 3, 2);
    vm_wait<0>();
    __syncthreads();

    bf16x8 ring[KS], pk[2];
    f32x16 sa, sb;
    {
      const u16 *krow = &sm.k[0][col][8 * half];
#pragma unroll
      for (int j = 0; j < KS; ++j) ring[j] = as_bf16x8(ld16(krow + j * 16));
      sa = f32x16{};
#pragma unroll
      for (int j = 0; j < KS; ++j) sa = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ring[j], qreg[j], sa, 0, 0, 0);
#pragma unroll
      for (int j = 0; j < KS; ++j) ring[j] = as_bf16x8(ld16(krow + 32 * Sm::kPitch + j * 16));
    }
    pk[0] = pk[1] = as_bf16x8(u32x4{0, 0, 0, 0});
    __syncthreads();  // every wave has read K(0): the first iteration refills its stage

    constexpr int kSlots = KS + 2 * DT, kEps = 16 / kSlots;
    static_assert(KS == 2 * DT, "one operand ring serves both product chains");
    f32x4 sc = *reinterpret_cast<const f32x4 *>(&keys.scale[4 * half]);  // scales of the sub-step's first four keys
    // Sub-step i (keys from j0 of the split): cur = S^T(i); nxt receives
    // S^T(i+1); K operands of i + 2 from stage kst, rows ksub * 32..;
    // displacement operands of i - 1 from stage xst, rows xsub * 32...
    auto step = [&](f32x16 &cur, f32x16 &nxt, int kst, int ksub, int xst, int xsub, int j0, auto hook)
        __attribute__((always_inline)) {
      const u16 *krow = &sm.k[kst][ksub * 32 + col][8 * half];
      const u16 *xrow = &sm.x[xst][xsub * 32][0] + v_lane;
      const float *sp = &keys.scale[j0 + 4 * half];
      u32x4 pn[2];
      float pe[16];
      f32x4 scn = sc;
      auto pack = [&](int e) __attribute__((always_inline)) {
        bf16x2 w;
        w[0] = static_cast<__bf16>(pe[e]);
        w[1] = static_cast<__bf16>(pe[e + 1]);
        const uint32_t u = __builtin_bit_cast(uint32_t, w);
        asm volatile("" ::"v"(u));
        pn[e / 8][(e % 8) / 2] = u;
      };
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int j = 0; j < kSlots; ++j) {
        if (j < KS) {
          nxt = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ring[j], qreg[j], j == 0 ? f32x16{} : nxt, 0, 0, 0);
          if (j & 1) {
            ring[j] = v_operand_il<Sm::xPitch>(xrow + (j / DT) * 16 * Sm::xPitch + (j % DT) * 32);
            ring[j - 1] = v_operand_il<Sm::xPitch>(xrow + ((j - 1) / DT) * 16 * Sm::xPitch + ((j - 1) % DT) * 32);
          }
        } else {
          const int jj = j - KS;
          y[jj % DT] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ring[jj], pk[jj / DT], y[jj % DT], 0, 0, 0);
          if (jj & 1) {
            ring[jj] = as_bf16x8(ld16(krow + jj * 16));
            ring[jj - 1] = as_bf16x8(ld16(krow + (jj - 1) * 16));
          }
        }
#pragma unroll
        for (int e = j * kEps; e < (j + 1) * kEps; ++e) {
          // register e holds key 8 * (e / 4) + 4 * half + e % 4 of the sub-tile
          if (e % 4 == 0) {
            sc = scn;
            scn = *reinterpret_cast<const f32x4 *>(sp + (e < 12 ? 8 * (e / 4 + 1) : 32));
          }
          pe[e] = fast_exp2(fmaf(cur[e], c, neg_b)) * sc[e % 4];  // b is the row's whole log-sum-exp: alpha <= 1
          asm volatile("" ::"v"(pe[e]));
          if (e >= 3 && (e & 1)) pack(e - 3);
        }
        hook(j);
        if (j == kSlots - 1) pack(14);
        __builtin_amdgcn_sched_barrier(0);
      }
      sc = scn;
      pk[0] = as_bf16x8(pn[0]);
      pk[1] = as_bf16x8(pn[1]);
    };
    // Iteration t reads K(t+1), X(t-1) and X(t) while K(t+2), X(t+1) (issued
    // one iteration ago) and K(t+3), X(t+2) arrive; at its end each wave waits
    // for all but the transfers it has just issued.
    int ks = 0;  // K stage of tile t
    for (int t = 0; t < n_t; ++t) {
      const int k1 = ks + 1 == 3 ? 0 : ks + 1;
      constexpr int kSpread = 2 * kSlots / (kGroup + 1);
      static_assert(kSpread >= 1 && kSpread * kGroup <= 2 * kSlots, "every transfer has a slot");
      auto issue = [&](int g) __attribute__((always_inline)) {
        if (g % kSpread == kSpread - 1 && g / kSpread < kGroup) {
          const int n = g / kSpread;
          dma(n, rows[n], ks, (t + 2) & 3);
          rows[n] = row_of(n, t + 4, t + 3);  // the next iteration's
        }
      };
      step(sa, sb, k1, 0, (t - 1) & 3, 1, t * KT, [&](int j) __attribute__((always_inline)) { issue(j); });
      step(sb, sa, k1, 1, t & 3, 0, t * KT + 32, [&](int j) __attribute__((always_inline)) { issue(kSlots + j); });
      vm_wait<kGroup>();
      __syncthreads();
      ks = k1;
    }
    vm_wait<0>();  // no transfer is in flight when the workgroup's LDS is released
    const int xlast = (n_t - 1) & 3;
    const u16 *xrow = &sm.x[xlast][32][0] + v_lane;
#pragma unroll
    for (int jj = 0; jj < 2 * DT; ++jj)
      y[jj % DT] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
          v_operand_il<Sm::xPitch>(xrow + (jj / DT) * 16 * Sm::xPitch + (jj % DT) * 32), pk[jj / DT], y[jj % DT], 0, 0, 0);
  }

  // Partial residual of this split: lane (pair, half) holds dims
  // dt*32 + 8*g4 + 4*half + 0..3 of its pair.
  if (valid) {
    float *dst = p.part + ((((int64_t)m * p.n_splits + split) * p.n_kv_heads + kvh) * p.pairs_pad + pair) * D;
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
      for (int g4 = 0; g4 < 4; ++g4) {
        f32x4 v4;
#pragma unroll
        for (int i = 0; i < 4; ++i) v4[i] = y[dt][4 * g4 + i];
        *reinterpret_cast<f32x4 *>(dst + dt * 32 + 8 * g4 + 4 * half) = v4;
      }
  }
}

// One wave per (sample, KV head, pair): the split partials added in split
// order, then the squared norm.
template <int D>
__global__ __launch_bounds__(256) void residual_sum_kernel(ResidualParams p) {
  constexpr int PER = D / 64;
  const int n_pairs = p.n_q * p.group;
  const int64_t wid = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (wid >= (int64_t)p.n_samples * p.n_kv_heads * n_pairs) return;
  const int pair = (int)(wid % n_pairs);
  const int kvh = (int)((wid / n_pairs) % p.n_kv_heads);
  const int m = (int)(wid / ((int64_t)n_pairs * p.n_kv_heads));
  float yv[PER];
#pragma unroll
  for (int i = 0; i < PER; ++i) yv[i] = 0.f;
  for (int s = 0; s < p.n_splits; ++s) {
    const float *src = p.part + ((((int64_t)m * p.n_splits + s) * p.n_kv_heads + kvh) * p.pairs_pad + pair) * D;
#pragma unroll
    for (int i = 0; i < PER; ++i) yv[i] += src[lane + 64 * i];
  }
  float sq = 0.f;
#pragma unroll
  for (int i = 0; i < PER; ++i) sq = fmaf(yv[i], yv[i], sq);
  sq = wave_sum(sq);
  if (lane == 0) {
    const int r = pair / p.group, h = kvh * p.group + pair % p.group;
    p.err_out[((int64_t)m * p.n_q + r) * p.n_q_heads + h] = sq;
  }
}

// fp32 path: one wave per (sample, span row, query head) over all visual
// keys, 64 keys per step, the residual accumulated per lane over D/64 dims.
template <int D>
__global__ __launch_bounds__(64) void residual_f32_kernel(ResidualParams p) {
  constexpr int PER = D / 64;
  __shared__ float qs[D];
  const int64_t gid = blockIdx.x;  // (m * n_q + r) * n_q_heads + h
  const int lane = threadIdx.x;
  const int h = (int)(gid % p.n_q_heads);
  const int r = (int)((gid / p.n_q_heads) % p.n_q);
  const int m = (int)(gid / ((int64_t)p.n_q_heads * p.n_q));
  const int kvh = h / p.group;
  const float *Kg = static_cast<const float *>(p.k);
  const float *Xg = static_cast<const float *>(p.disp);
  const bool iso = p.vnorm != nullptr;
  const float *q = static_cast<const float *>(p.q) + ((int64_t)r * p.n_q_heads + h) * D;
  for (int e = lane; e < D; e += 64) qs[e] = q[e];
  __syncthreads();
  const float b = p.row_b[(int64_t)r * p.n_q_heads + h];
  float yv[PER];
#pragma unroll
  for (int i = 0; i < PER; ++i) yv[i] = 0.f;
  for (int base = 0; base < p.n_vis; base += 64) {
    const int t = base + lane;
    float a = 0.f;
    if (t < p.n_vis && p.refreshed[t] == 0) {
      const float *kr = Kg + kv_row(p.pages, vis_position(p.tbl, t)) * p.k_stride + kvh * D;
      float dot = 0.f;
#pragma unroll 8
      for (int e = 0; e < D; ++e) dot = fmaf(qs[e], kr[e], dot);
      a = fast_exp2(fmaf(dot, p.scale_log2, -b)) * (iso ? p.vnorm[t] * p.sigma_scale : 1.f);
    }
    const int nk = min(64, p.n_vis - base);
    for (int j = 0; j < nk; ++j) {
      const float aj = __shfl(a, j, 64);
      if (aj == 0.f) continue;  // uniform: every lane reads the same aj
      const int tj = base + j;
      const float *xr = iso ? Xg + (((int64_t)m * p.n_vis + tj) * p.n_kv_heads + kvh) * D
                            : Xg + kv_row(p.pages, vis_position(p.tbl, tj)) * p.disp_stride + kvh * D;
#pragma unroll
      for (int i = 0; i < PER; ++i) yv[i] = fmaf(aj, xr[lane + 64 * i], yv[i]);
    }
  }
  float sq = 0.f;
#pragma unroll
  for (int i = 0; i < PER; ++i) sq = fmaf(yv[i], yv[i], sq);
  sq = wave_sum(sq);
  if (lane == 0) p.err_out[gid] = sq;
}

}  // namespace

hipError_t launch_residual(const ResidualParams &p, int head_dim, bool bf16, hipStream_t s) {
  if (bf16) {
    const int n_pb = p.pairs_pad / kResidualPairs;
    dim3 grid(p.n_splits, n_pb, p.n_kv_heads * p.n_samples);
    const int64_t waves = (int64_t)p.n_samples * p.n_kv_heads * p.n_q * p.group;
    {
      ProfScope ps("residual", s);
      if (head_dim == 128) residual_bf16_kernel<128><<<grid, kThreads, 0, s>>>(p);
      else residual_bf16_kernel<64><<<grid, kThreads, 0, s>>>(p);
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    ProfScope ps("residual_sum", s);
    const unsigned blocks = (unsigned)((waves + 3) / 4);
    if (head_dim == 128) residual_sum_kernel<128><<<blocks, 256, 0, s>>>(p);
    else residual_sum_kernel<64><<<blocks, 256, 0, s>>>(p);
  } else {
    ProfScope ps("residual_f32", s);
    const unsigned blocks = (unsigned)((int64_t)p.n_samples * p.n_q * p.n_q_heads);
    if (head_dim == 128) residual_f32_kernel<128><<<blocks, 64, 0, s>>>(p);
    else residual_f32_kernel<64><<<blocks, 64, 0, s>>>(p);
  }
  return hipGetLastError();
}

}  // namespace conduit
