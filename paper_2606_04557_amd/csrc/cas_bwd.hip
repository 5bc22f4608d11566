// Backward of multi-cartridge prefix attention on gfx950: the statistics
// pass for both dtypes, the fp32 dK/dV and dQ passes (v_mfma_f32_32x32x2f32,
// no down-conversion; bf16 runs the kernels of cas_bf16.hip) and the dQ
// split reduction for both dtypes.
//
// Three passes, all recomputing P from the stored row LSE:
//   bwd_pre:  D = rowsum(dO * O) and LSE*log2(e) per packed row (fp32).
//   dkdv:     key-stationary. A workgroup owns 32 keys of one distinct
//             cartridge (or of one row's self keys) and one kv head; its waves
//             share out every query row of the GQA group in every batch row
//             that references the cartridge, with Q/dO blocks staged through
//             LDS:
//               S = Q K^T, dP = dO V^T        (K, V held in registers)
//               P = exp2(S c - LSE2), dS = P (dP - D)
//               dV^T += dO^T P, dK^T += Q^T dS  (P, dS straight from the C
//                                                registers; Q/dO from LDS)
//             The sums stay in registers, so each key's gradient is written
//             once, to the owning segment's buffer, with no atomics; a
//             cartridge referenced by several rows accumulates all of them.
//   dq:       query-stationary, like the forward: per key tile
//               S^T = K Q^T, dP^T = V dO^T, dS^T = P^T (dP^T - D),
//               dQ^T += K^T dS^T
//             with optional key-axis splits whose fp32 partials are summed.
#include "cas_device.h"

namespace cas {

// 16 lanes per packed row; grid.y is the batch row.
template <typename T, int D>
__global__ __launch_bounds__(kThreads) void bwd_pre_kernel(PreParams p) {
  constexpr int LPR = 16;            // lanes per packed row
  constexpr int CPL = D / LPR;       // channels per lane
  const int64_t gid = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  const int b = blockIdx.y;
  const DevRow row = p.rows[b];
  const int nrows = row.len * p.g;
  const int64_t rb = gid / LPR;      // kvh * nrows + r
  const int li = (int)(gid % LPR);
  const bool live = rb < (int64_t)p.Hkv * nrows;
  const int Hq = p.Hkv * p.g;
  float acc = 0.0f;
  int h = 0, t = 0;
  if (live) {
    const int kvh = (int)(rb / nrows), r = (int)(rb % nrows);
    t = r / p.g;
    h = kvh * p.g + (r - t * p.g);
    const int64_t off = (((int64_t)row.tok0 + t) * Hq + h) * D + li * CPL;
    const T *op = (const T *)p.o + off;
    const T *dp = (const T *)p.d_o + off;
#pragma unroll
    for (int i = 0; i < CPL; ++i) acc += to_f32(op[i]) * to_f32(dp[i]);
  }
#pragma unroll
  for (int m = LPR / 2; m >= 1; m >>= 1) acc += __shfl_xor(acc, m, LPR);
  if (live && li == 0) {
    const int64_t R = (int64_t)row.tok0 * Hq + rb;
    p.nd[R] = -acc;
    p.lse2[R] = p.lse[(int64_t)row.lse0 + (int64_t)h * p.lse_hs + t] * kLog2e;
  }
}

// 32 keys per workgroup. The four waves share the keys and take every fourth
// 32-row block of the queries each, staged through a wave's own LDS (no
// workgroup barrier until their sums meet at the end), with the next block's
// rows in flight while a block is worked on. Bound by the matrix products of
// one wave per SIMD: a wave's chain over the queries is a quarter of what it
// was with 32 keys per wave and 128 per workgroup, and four times the
// workgroups cover the compute units (2 x 128 keys, 64 queries, d = 64: 33.7 ->
// 17.5 us; 3 x 400 keys, 400 queries, d = 128, 8 KV heads: 269 -> 187 us).
template <int D>
__global__ __launch_bounds__(kThreads) void dkdv_kernel(DkdvParams p) {
  using T = float;
  using M = Mma<T>;
  using Frag = typename M::Frag;
  constexpr int NSTEP = D / M::kStep;
  constexpr int RB = 32;                      // query rows of a block
  constexpr int DT = D / 32;
  constexpr int RS = lds_row_stride<T, D>();
  constexpr int CPR = D / 4;                  // 16-byte chunks per row
  constexpr int NC = RB * CPR / 64;           // chunks of a block per lane
  constexpr int WAVE = 2 * RB * RS;           // floats of a wave's Q and dO blocks
  static_assert(2 * DT * 16 * 64 <= WAVE, "a wave's sums fit where its blocks were");

  __shared__ __attribute__((aligned(16))) T blocks[kWaves * WAVE];
  __shared__ float stats[kWaves][2][RB];

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int G = lane >> 5, n = lane & 31;
  T *const q_row = blocks + wave * WAVE;
  T *const do_row = q_row + RB * RS;
  float *const lse2_l = stats[wave][0], *const nd_l = stats[wave][1];
  const DevWg wg = p.order[blockIdx.x];
  const int kvh = wg.kvh, key0 = wg.tile * kDkdvKeyTileFp32;
  const int g = p.g, Hkv = p.Hkv, Hq = Hkv * g;
  const float c = p.scale_log2;

  const T *kbase;
  const T *vbase;
  T *dkp;
  T *dvp;
  int64_t st;
  int klen, use_b = 0, use_e = 1;
  const bool self = wg.owner < 0;
  const int self_b = -1 - wg.owner;
  if (!self) {
    const DevCart cd = p.carts[wg.owner];
    klen = cd.len;
    kbase = (const T *)cd.k + kvh * cd.stride_head;
    vbase = (const T *)cd.v + kvh * cd.stride_head;
    dkp = cd.dk ? (T *)cd.dk + kvh * cd.stride_head : nullptr;
    dvp = cd.dv ? (T *)cd.dv + kvh * cd.stride_head : nullptr;
    st = cd.stride_tok;
    use_b = cd.use_begin;
    use_e = cd.use_end;
  } else {
    const DevRow sr = p.rows[self_b];
    klen = sr.len;
    const int64_t base = ((int64_t)sr.tok0 * Hkv + kvh) * D;
    kbase = (const T *)p.k_self + base;
    vbase = (const T *)p.v_self + base;
    dkp = p.dk_self ? (T *)p.dk_self + base : nullptr;
    dvp = p.dv_self ? (T *)p.dv_self + base : nullptr;
    st = (int64_t)Hkv * D;
  }
  const int my_key = key0 + n;
  const bool key_ok = my_key < klen;

  // The wave's blocks: every fourth of the uses' 32-row blocks, in order (self
  // keys: from the first block that sees the tile's first key).
  const int blk0 = self ? (key0 * g) / RB : 0;
  int u = use_b, blk = blk0 + wave, nrows = 0, tok0 = 0;
  auto open_use = [&]() {
    const DevRow rw = p.rows[self ? self_b : p.uses[u]];
    nrows = rw.len * g;
    tok0 = rw.tok0;
  };
  // Moves to the use that holds block blk, counted from the current use.
  auto settle = [&]() {
    while (u < use_e) {
      open_use();
      const int nb = (nrows + RB - 1) / RB;
      if (blk < nb) return true;
      blk -= nb;
      ++u;
    }
    return false;
  };
  u32x4 qr[NC], dor[NC];
  float stat_n[2] = {INFINITY, 0.0f};
  auto fetch = [&]() {
    const int r0 = blk * RB, nv = min(RB, nrows - r0);
    const int64_t head0 = ((int64_t)tok0 * Hq + kvh * g) * D;
#pragma unroll
    for (int i = 0; i < NC; ++i) {
      const int ch = lane + 64 * i, r = ch / CPR, cc = ch % CPR;
      const int rr = r0 + r, t = rr / g;
      const int64_t off = head0 + ((int64_t)t * Hq + (rr - t * g)) * D + cc * 4;
      const u32x4 z = {0u, 0u, 0u, 0u};
      qr[i] = r < nv ? *reinterpret_cast<const u32x4 *>((const T *)p.q + off) : z;
      dor[i] = r < nv ? *reinterpret_cast<const u32x4 *>((const T *)p.d_o + off) : z;
    }
    const int64_t pk = (int64_t)tok0 * Hq + (int64_t)kvh * nrows + r0 + n;
    stat_n[0] = n < nv ? p.lse2[pk] : INFINITY;
    stat_n[1] = n < nv ? p.nd[pk] : 0.0f;
  };
  bool more = settle();
  if (more) fetch();

  Frag kf[NSTEP], vf[NSTEP];
#pragma unroll
  for (int s = 0; s < NSTEP; ++s) {
    kf[s] = key_ok ? global_frag<T>(kbase + my_key * st, s, G) : M::zero();
    vf[s] = key_ok ? global_frag<T>(vbase + my_key * st, s, G) : M::zero();
  }
  f32x16 dk[DT], dv[DT];
#pragma unroll
  for (int dt = 0; dt < DT; ++dt) {
    dk[dt] = zero16();
    dv[dt] = zero16();
  }

  while (more) {
    const int r0 = blk * RB, nv = min(RB, nrows - r0);
#pragma unroll
    for (int i = 0; i < NC; ++i) {
      const int ch = lane + 64 * i, r = ch / CPR, cc = ch % CPR;
      *reinterpret_cast<u32x4 *>(q_row + r * RS + cc * 4) = qr[i];
      *reinterpret_cast<u32x4 *>(do_row + r * RS + cc * 4) = dor[i];
    }
    if (G == 0) {
      lse2_l[n] = stat_n[0];
      nd_l[n] = stat_n[1];
    }
    // The wave's own LDS writes, then reads of them by its other lanes.
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    blk += kWaves;
    more = settle();
    if (more) fetch();
    // (Self keys: the first block sees the tile's first key.)
    const bool need_mask = self && key0 + kDkdvKeyTileFp32 - 1 > r0 / g;

    f32x16 sa = zero16(), dpa = zero16();
#pragma unroll
    for (int s = 0; s < NSTEP; ++s) {
      sa = M::run(row_frag<T, D>(q_row, n, s, G), kf[s], sa);
      dpa = M::run(row_frag<T, D>(do_row, n, s, G), vf[s], dpa);
    }
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      const int ql = crow(j, G);
      float pv = exp2f(fmaf(sa[j], c, -lse2_l[ql]));
      if (need_mask) pv = (my_key <= (r0 + ql) / g) ? pv : 0.0f;
      pv = key_ok ? pv : 0.0f;
      const float ds = pv * (dpa[j] + nd_l[ql]);
      sa[j] = pv;
      dpa[j] = ds;
    }
#pragma unroll
    for (int s = 0; s < 16; ++s)
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) {
        dv[dt] = M::run(trans_frag_f32<D>(do_row, 0, s, G, dt * 32 + n), sa[s], dv[dt]);
        dk[dt] = M::run(trans_frag_f32<D>(q_row, 0, s, G, dt * 32 + n), dpa[s], dk[dt]);
      }
    // Reads of this block before the next block's writes.
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  }

  // The waves' sums meet in LDS, [sum][register][lane] per wave (each wave
  // writes where its own blocks were); wave w adds up and stores sums w, w + 4,
  // ... of the DT dK and DT dV ones.
  T *const mine = q_row;
#pragma unroll
  for (int dt = 0; dt < DT; ++dt)
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      mine[(dt * 16 + j) * 64 + lane] = dk[dt][j];
      mine[((DT + dt) * 16 + j) * 64 + lane] = dv[dt][j];
    }
  __syncthreads();
  const float sc = p.scale;
  for (int x = wave; x < 2 * DT; x += kWaves) {
    float sum[16];
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      sum[j] = 0.0f;
#pragma unroll
      for (int v = 0; v < kWaves; ++v) sum[j] += blocks[v * WAVE + (x * 16 + j) * 64 + lane];
    }
    const bool is_dk = x < DT;
    T *const dst = is_dk ? dkp : dvp;
    const float m = is_dk ? sc : 1.0f;
    const int dt = is_dk ? x : x - DT;
    if (dst && key_ok) {
#pragma unroll
      for (int jj = 0; jj < 4; ++jj)
        store4(dst + my_key * st + dt * 32 + jj * 8 + G * 4, sum[jj * 4 + 0] * m, sum[jj * 4 + 1] * m, sum[jj * 4 + 2] * m,
               sum[jj * 4 + 3] * m);
    }
  }
}

// As in the forward, the next tile's rows are loaded while a tile is worked on,
// and with 64 channels two workgroups share a compute unit.
template <int D>
__global__ __launch_bounds__(kThreads, D == 64 ? 2 : 1) void dq_kernel(DqParams p) {
  using T = float;
  using M = Mma<T>;
  using Frag = typename M::Frag;
  constexpr int NSTEP = D / M::kStep;
  constexpr int QS = kDqRowsPerWave / 32;
  constexpr int KT = kKeyTile;
  constexpr int NSUB = KT / 32;
  constexpr int DT = D / 32;
  constexpr int RS = lds_row_stride<T, D>();

  __shared__ __attribute__((aligned(16))) T k_row[KT * RS];
  __shared__ __attribute__((aligned(16))) T v_row[KT * RS];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int G = lane >> 5, n = lane & 31;
  int bid = blockIdx.x;
  const int qblk = bid % p.nqblk;
  bid /= p.nqblk;
  const int kvh = bid % p.Hkv;
  bid /= p.Hkv;
  const int split = bid % p.splits;
  const int b = bid / p.splits;

  const int g = p.g, Hkv = p.Hkv, Hq = Hkv * g;
  const DevRow row = p.rows[b];
  const int tok0 = row.tok0, len = row.len, nrows = len * g;
  const int wg_row0 = qblk * kDqRowsPerWg;
  if (wg_row0 >= nrows) return;   // grid sized for the longest row
  const int wg_row1 = min(nrows, wg_row0 + kDqRowsPerWg);
  const int row0 = wg_row0 + wave * kDqRowsPerWave;
  const bool wave_active = row0 < nrows;
  const int wave_t_lo = row0 / g;
  const int wave_t_hi = (min(row0 + kDqRowsPerWave, nrows) - 1) / g;
  const int wg_t_hi = (wg_row1 - 1) / g;
  const float c = p.scale_log2;

  Frag qf[QS][NSTEP], df[QS][NSTEP];
  float lse2r[QS], ndr[QS];
  const int64_t pk = (int64_t)tok0 * Hq + (int64_t)kvh * nrows;
#pragma unroll
  for (int qs = 0; qs < QS; ++qs) {
    const int r = row0 + 32 * qs + n;
    if (r < nrows) {
      const int t = r / g, hh = r - t * g;
      const int64_t off = (((int64_t)tok0 + t) * Hq + kvh * g + hh) * D;
#pragma unroll
      for (int s = 0; s < NSTEP; ++s) {
        qf[qs][s] = global_frag<T>((const T *)p.q + off, s, G);
        df[qs][s] = global_frag<T>((const T *)p.d_o + off, s, G);
      }
      lse2r[qs] = p.lse2[pk + r];
      ndr[qs] = p.nd[pk + r];
    } else {
#pragma unroll
      for (int s = 0; s < NSTEP; ++s) {
        qf[qs][s] = M::zero();
        df[qs][s] = M::zero();
      }
      lse2r[qs] = INFINITY;
      ndr[qs] = 0.0f;
    }
  }
  f32x16 acc[DT][QS];
#pragma unroll
  for (int dt = 0; dt < DT; ++dt)
#pragma unroll
    for (int qs = 0; qs < QS; ++qs) acc[dt][qs] = zero16();

  const int ptiles = row.prefix_tiles;
  const int ntiles = ptiles + wg_t_hi / KT + 1;
  const int tb = (int)((int64_t)ntiles * split / p.splits);
  const int te = (int)((int64_t)ntiles * (split + 1) / p.splits);
  int seg = row.seg_begin;

  // Where the rows of a tile are; asked for in increasing order.
  struct Tile {
    const T *kp;
    const T *vp;
    int64_t st;
    int nvalid, self0;
  };
  auto locate = [&](int tile) {
    Tile x;
    if (tile < ptiles) {
      for (;;) {
        const DevSeg sd = p.segs[seg];
        if (tile < sd.tile_begin + (sd.len + KT - 1) / KT) break;
        ++seg;
      }
      const DevSeg sd = p.segs[seg];
      const int key0 = (tile - sd.tile_begin) * KT;
      x.kp = (const T *)sd.k + kvh * sd.stride_head + (int64_t)key0 * sd.stride_tok;
      x.vp = (const T *)sd.v + kvh * sd.stride_head + (int64_t)key0 * sd.stride_tok;
      x.st = sd.stride_tok;
      x.nvalid = min(KT, sd.len - key0);
      x.self0 = -1;
    } else {
      x.self0 = (tile - ptiles) * KT;
      x.kp = (const T *)p.k_self + (((int64_t)tok0 + x.self0) * Hkv + kvh) * D;
      x.vp = (const T *)p.v_self + (((int64_t)tok0 + x.self0) * Hkv + kvh) * D;
      x.st = (int64_t)Hkv * D;
      x.nvalid = min(KT, len - x.self0);
    }
    return x;
  };
  RowTile<T, D, KT> kr, vr;
  auto fetch = [&](const Tile &x) {
    kr.fetch([&](int r) { return x.kp + r * x.st; }, x.nvalid, tid);
    vr.fetch([&](int r) { return x.vp + r * x.st; }, x.nvalid, tid);
  };
  Tile next{};
  if (tb < te) {
    next = locate(tb);
    fetch(next);
  }
  for (int tile = tb; tile < te; ++tile) {
    const int nvalid = next.nvalid, self0 = next.self0;
    __syncthreads();
    kr.put(k_row, tid);
    vr.put(v_row, tid);
    __syncthreads();
    if (tile + 1 < te) {
      next = locate(tile + 1);
      fetch(next);
    }

    if (!wave_active) continue;
    if (self0 >= 0 && self0 > wave_t_hi) continue;
    const bool need_mask = (nvalid < KT) || (self0 >= 0 && self0 + KT - 1 > wave_t_lo);

#pragma unroll
    for (int sub = 0; sub < NSUB; ++sub) {
      f32x16 sa[QS], dpa[QS];
#pragma unroll
      for (int qs = 0; qs < QS; ++qs) {
        sa[qs] = zero16();
        dpa[qs] = zero16();
      }
#pragma unroll
      for (int s = 0; s < NSTEP; ++s) {
        const Frag kfr = row_frag<T, D>(k_row, 32 * sub + n, s, G);
        const Frag vfr = row_frag<T, D>(v_row, 32 * sub + n, s, G);
#pragma unroll
        for (int qs = 0; qs < QS; ++qs) {
          sa[qs] = M::run(kfr, qf[qs][s], sa[qs]);
          dpa[qs] = M::run(vfr, df[qs][s], dpa[qs]);
        }
      }
#pragma unroll
      for (int qs = 0; qs < QS; ++qs) {
        const int t = (row0 + 32 * qs + n) / g;
#pragma unroll
        for (int j = 0; j < 16; ++j) {
          float pv = exp2f(fmaf(sa[qs][j], c, -lse2r[qs]));
          if (need_mask) {
            const int key = 32 * sub + crow(j, G);
            const bool ok = key < nvalid && (self0 < 0 || self0 + key <= t);
            pv = ok ? pv : 0.0f;
          }
          sa[qs][j] = pv * (dpa[qs][j] + ndr[qs]);
        }
      }
#pragma unroll
      for (int s = 0; s < 16; ++s)
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) {
          const float a = trans_frag_f32<D>(k_row, sub, s, G, dt * 32 + n);
#pragma unroll
          for (int qs = 0; qs < QS; ++qs) acc[dt][qs] = M::run(a, sa[qs][s], acc[dt][qs]);
        }
    }
  }

#pragma unroll
  for (int qs = 0; qs < QS; ++qs) {
    const int r = row0 + 32 * qs + n;
    if (r >= nrows) continue;
    const int t = r / g, h = kvh * g + (r - t * g);
    if (p.splits == 1) {
      const float sc = p.scale;
      T *op = (T *)p.dq + (((int64_t)tok0 + t) * Hq + h) * D;
#pragma unroll
      for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int jj = 0; jj < 4; ++jj)
          store4(op + dt * 32 + jj * 8 + G * 4, acc[dt][qs][jj * 4 + 0] * sc,
                 acc[dt][qs][jj * 4 + 1] * sc, acc[dt][qs][jj * 4 + 2] * sc,
                 acc[dt][qs][jj * 4 + 3] * sc);
    } else {
      const int64_t prow = split * p.plane + pk + r;
      float *op = p.part_dq + prow * D;
#pragma unroll
      for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int jj = 0; jj < 4; ++jj)
          store4(op + dt * 32 + jj * 8 + G * 4, acc[dt][qs][jj * 4 + 0], acc[dt][qs][jj * 4 + 1],
                 acc[dt][qs][jj * 4 + 2], acc[dt][qs][jj * 4 + 3]);
    }
  }
}

// One thread per 4 channels of a packed row; grid.y is the batch row. The
// partials of eight splits are in flight at once (summed in split order): 16
// splits of 512 rows 9.0 -> 6.4 us with the launch and its timing events.
template <typename T, int D>
__global__ __launch_bounds__(kThreads) void dq_reduce_kernel(DqReduceParams p) {
  constexpr int CPR = D / 4;
  const int64_t idx = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  const int b = blockIdx.y;
  const DevRow row = p.rows[b];
  const int nrows = row.len * p.g;
  const int64_t rb = idx / CPR;          // kvh * nrows + r
  const int c4 = (int)(idx % CPR);
  if (rb >= (int64_t)p.Hkv * nrows) return;
  const int64_t plane = p.plane;
  const int64_t R = (int64_t)row.tok0 * p.Hkv * p.g + rb;
  const float *src = p.part_dq + R * D + c4 * 4;
  f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
  constexpr int U = 8;
  for (int s0 = 0; s0 < p.splits; s0 += U) {
    f32x4 v[U];
#pragma unroll
    for (int u = 0; u < U; ++u)
      v[u] = *reinterpret_cast<const f32x4 *>(src + (int64_t)min(s0 + u, p.splits - 1) * plane * D);
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (s0 + u < p.splits) acc += v[u];
  }
  const int kvh = (int)(rb / nrows), r = (int)(rb % nrows);
  const int t = r / p.g, h = kvh * p.g + (r - t * p.g);
  const int Hq = p.Hkv * p.g;
  T *op = (T *)p.dq + (((int64_t)row.tok0 + t) * Hq + h) * D + c4 * 4;
  store4(op, acc[0] * p.scale, acc[1] * p.scale, acc[2] * p.scale, acc[3] * p.scale);
}

template <typename T, int D>
static hipError_t launch_pre_t(const PreParams &p, hipStream_t s) {
  const int64_t n = (int64_t)p.Hkv * p.nrows_max * 16;
  hipLaunchKernelGGL((bwd_pre_kernel<T, D>), dim3((unsigned)((n + kThreads - 1) / kThreads), (unsigned)p.B),
                     dim3(kThreads), 0, s, p);
  return hipGetLastError();
}

hipError_t launch_bwd_pre(const PreParams &p, DType dt, int D, hipStream_t s) {
  if (dt == kBF16) return D == 64 ? launch_pre_t<__bf16, 64>(p, s) : launch_pre_t<__bf16, 128>(p, s);
  return D == 64 ? launch_pre_t<float, 64>(p, s) : launch_pre_t<float, 128>(p, s);
}

template <int D>
static hipError_t launch_dkdv_t(const DkdvParams &p, int n_wg, hipStream_t s) {
  hipLaunchKernelGGL((dkdv_kernel<D>), dim3((unsigned)n_wg), dim3(kThreads), 0, s, p);
  return hipGetLastError();
}

hipError_t launch_dkdv(const DkdvParams &p, DType dt, int D, int n_wg, hipStream_t s) {
  if (dt == kBF16) return launch_dkdv_bf16(p, D, n_wg, s);
  return D == 64 ? launch_dkdv_t<64>(p, n_wg, s) : launch_dkdv_t<128>(p, n_wg, s);
}

template <int D>
static hipError_t launch_dq_t(const DqParams &p, hipStream_t s) {
  const int64_t grid = (int64_t)p.nqblk * p.Hkv * p.splits * p.B;
  hipLaunchKernelGGL((dq_kernel<D>), dim3((unsigned)grid), dim3(kThreads), 0, s, p);
  return hipGetLastError();
}

hipError_t launch_dq(const DqParams &p, DType dt, int D, hipStream_t s) {
  if (dt == kBF16) return launch_dq_bf16(p, D, s);
  return D == 64 ? launch_dq_t<64>(p, s) : launch_dq_t<128>(p, s);
}

template <typename T, int D>
static hipError_t launch_dq_reduce_t(const DqReduceParams &p, hipStream_t s) {
  const int64_t n = (int64_t)p.Hkv * p.nrows_max * (D / 4);
  hipLaunchKernelGGL((dq_reduce_kernel<T, D>), dim3((unsigned)((n + kThreads - 1) / kThreads), (unsigned)p.B),
                     dim3(kThreads), 0, s, p);
  return hipGetLastError();
}

hipError_t launch_dq_reduce(const DqReduceParams &p, DType dt, int D, hipStream_t s) {
  if (dt == kBF16) return D == 64 ? launch_dq_reduce_t<__bf16, 64>(p, s) : launch_dq_reduce_t<__bf16, 128>(p, s);
  return D == 64 ? launch_dq_reduce_t<float, 64>(p, s) : launch_dq_reduce_t<float, 128>(p, s);
}

}  // namespace cas
