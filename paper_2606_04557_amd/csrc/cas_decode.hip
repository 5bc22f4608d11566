// Short-query / decode attention over a paged KV pool (forward only): the
// retrieved cartridges' pages, then the request's own pages, with the last
// n queries of the key sequence as the new tokens (paper: Section
// "Inference", paragraph "Cartridge RAG", and the appendix on cartridge
// sizes for the 16-token pages of the serving engine's KV cache).
//
// A decode step has very few query rows per (request, KV head) (n * g, e.g.
// 4) against thousands of keys, so the work is streaming K and V out of HBM.
// One workgroup takes a block of up to 16 (NB = 1) or 32 (NB = 2) packed rows
// of one KV head and a range of 32-key tiles of a segment of keys: a request's
// own, or a page run that several requests share, whose rows then take one
// pass over it together (the host cuts the segments so that the compute units
// are full; a request's partials are merged by their LSE). Its four waves work independently on
// every fourth tile of the range, so no wave ever waits on another until the
// end, where the four partial softmax states are combined through LDS. The
// products use v_mfma_f32_16x16x32_bf16, whose 16 columns fit the few rows of
// a decode step; with NB = 2 each K and V fragment feeds two of them, so 17 to
// 32 rows stream the request's keys once instead of twice. K and V go from
// memory straight into registers, one tile ahead of their use: K already in
// the MFMA operand layout (each lane loads 16 bytes of one key row per step)
// into the other of two register sets, V in whole rows into the registers
// that its write into the wave's LDS tile (read transposed for the PV
// product) has just freed: one V set instead of two is what leaves room for a
// second row block without spills. Loads go through buffer resources whose
// scalar base is the tile's page, so lane offsets are loop constants. Page
// addresses come from the page table (scalar loads, a tile ahead of the loads
// that use them). Per tile and wave: S^T = K Q^T, an online-softmax update,
// and O^T += V^T P^T with P^T straight from the score registers.
//
// Bound by HBM. Per call, before and after the second row block and the
// single V set: 16 requests x 8 new tokens x 4 heads per group over ~4,250
// keys 101.6 -> 72.2 us; 64 requests x 1 new token over 4,161 keys 177.9 ->
// 175.2 us (1.09 GB of K and V, 0.73 GB of it distinct). With the runs shared
// between those 64 requests (each 4 of 256 cartridges) streamed once: 146.8 us;
// 50 requests over 3 of 16 cartridges 82 -> 28 us of kernel.
#include "cas_device.h"

namespace cas {

namespace {

constexpr int kDecWaves = 4;

typedef __attribute__((address_space(3))) char lds_char_t;

__device__ __forceinline__ f32x4 mfma16(bf16x8 a, bf16x8 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// NB: 16-row blocks of one workgroup (1 or 2).
template <int D, int NB>
__global__ __launch_bounds__(kDecWaves * 64) __attribute__((amdgpu_waves_per_eu(2, 2)))
void decode_bf16_kernel(DecodeParams p) {
  static_assert(kDecRows == 16, "one 16-column MFMA block of rows");
  constexpr int NQ = D / 32;                  // 32-channel steps of the score product
  constexpr int NDB = D / 16;                 // 16-channel blocks of the PV product
  constexpr int TB = kDecTile * D * 2;        // bytes of one 32-key V tile
  constexpr int CPR = D / 8;                  // 16-byte chunks per key row
  constexpr int RPI = 64 / CPR;               // key rows per V load instruction
  constexpr int NI = kDecTile / RPI;          // V load instructions per tile
  constexpr int OS = NDB * 4 * 64;            // floats of one wave's O^T of a row block in the closing combine
  static_assert(OS * 4 == TB, "a wave's O^T of one row block fills its V tile");
  // Each wave's V tile (the closing combine reuses it for the wave's O^T, one
  // row block after the other); m and l of every wave and row block.
  __shared__ __attribute__((aligned(1024))) char vs[kDecWaves * TB];
  __shared__ __attribute__((aligned(16))) float ml[kDecWaves * NB * 128];

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int j = lane & 15, bq = lane >> 4;    // MFMA column (row of the block) and k-group
  const DevDecodeWork w = load_const(p.work, (int)blockIdx.x);
  const int g = p.g, Hkv = p.Hkv, Hq = Hkv * g, P = p.page_size;
  const int kvh = __builtin_amdgcn_readfirstlane(w.kvh);
  const int kv_len = __builtin_amdgcn_readfirstlane(w.nkeys);   // keys of the segment
  // Row block rb of lane (j, bq): row row0 + 16 rb + j. Rows past the
  // workgroup's see every key (their Q is zero and nothing of theirs is stored).
  bool row_ok[NB];
  int my_R[NB], my_lim[NB], my_part[NB];                  // row of q, o and the partial planes; last key; partial
#pragma unroll
  for (int rb = 0; rb < NB; ++rb) {
    row_ok[rb] = 16 * rb + j < w.nrows;
    DevDecodeRow r{0, kv_len - 1, -1};
    if (row_ok[rb]) r = p.rows[w.row0 + 16 * rb + j];
    my_R[rb] = r.base + kvh * g;
    my_lim[rb] = r.lim;
    my_part[rb] = r.part < 0 ? -1 : r.part + w.piece;
  }
  const float c = p.scale_log2;
  char *const vt = vs + wave * TB;

  // Q as the B operand: step st of lane (j, bq) is channels 32 st + 8 bq ..
  // + 7 of row j.
  bf16x8 qf[NB][NQ];
#pragma unroll
  for (int rb = 0; rb < NB; ++rb) {
    const __bf16 *qp = (const __bf16 *)p.q + (int64_t)my_R[rb] * D + 8 * bq;
#pragma unroll
    for (int st = 0; st < NQ; ++st)
      qf[rb][st] = row_ok[rb] ? *reinterpret_cast<const bf16x8 *>(qp + 32 * st) : Mma<__bf16>::zero();
  }

  // The pages of a tile's keys 0..15 (a) and 16..31 (b): one page when pages
  // hold 32 or more tokens, since tiles start at multiples of 32.
  struct TilePages {
    int a, b;
  };
  auto tile_pages = [&](int tile) __attribute__((always_inline)) {
    TilePages tp{0, 0};
    const int k0 = tile * kDecTile;
    if (k0 < kv_len) {
      tp.a = load_const(p.page_ids, w.page0 + k0 / P);
      tp.b = k0 + 16 < kv_len ? load_const(p.page_ids, w.page0 + (k0 + 16) / P) : tp.a;
    }
    return tp;
  };
  // K and V of a tile come in two halves of 16 keys, each inside one page:
  // buffer resources over the half's valid rows of this KV head (scalar base
  // address; rows at or past kv_len read as zero), so the lane offsets are
  // the same for every tile.
  const int row_bytes = Hkv * D * 2;
  struct HalfRsrc {
    BufRsrc h[2];
  };
  auto half_rsrc = [&](const void *pool, int tile, const TilePages &tp) __attribute__((always_inline)) {
    HalfRsrc r;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int k0 = tile * kDecTile + 16 * h;
      const int valid = min(16, kv_len - k0);
      const int64_t off = (((int64_t)(h ? tp.b : tp.a) * P + (k0 & (P - 1))) * Hkv + kvh) * D;
      r.h[h] = make_rsrc((const __bf16 *)pool + off, valid > 0 ? (valid - 1) * row_bytes + D * 2 : 0);
    }
    return r;
  };
  auto load16 = [&](BufRsrc rs, int off) __attribute__((always_inline)) {
    return __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(rs, off, 0, 0));
  };
  // K of a tile as the A operand: fragment kb * NQ + st of lane (j, bq) is
  // channels 32 st + 8 bq .. + 7 of key 16 kb + j.
  const int koff = j * row_bytes + 16 * bq;
  auto load_k = [&](int tile, const TilePages &tp, bf16x8 (&kr)[2 * NQ]) __attribute__((always_inline)) {
    const HalfRsrc r = half_rsrc(p.k_pages, tile, tp);
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
      for (int st = 0; st < NQ; ++st) kr[kb * NQ + st] = load16(r.h[kb], koff + 64 * st);
  };
  // V of a tile in whole rows: load i of a lane is chunk lane % CPR of key
  // row RPI * i + lane / CPR.
  const int voff = (lane / CPR) * row_bytes + (lane % CPR) * 16;
  auto load_v = [&](int tile, const TilePages &tp, bf16x8 (&vr)[NI]) __attribute__((always_inline)) {
    const HalfRsrc r = half_rsrc(p.v_pages, tile, tp);
#pragma unroll
    for (int i = 0; i < NI; ++i) vr[i] = load16(r.h[2 * i / NI], voff + (i % (NI / 2)) * RPI * row_bytes);
  };
  // V rows into the wave's LDS tile (16-byte chunks XOR-swizzled by row). Row
  // RPI i + lane / CPR of load i differs from row lane / CPR by a constant in
  // the address and one in the swizzle. (The asm keeps the compiler from
  // holding every address in a register of its own.)
  const int wbase = (lane / CPR) * (D * 2) + (((lane % CPR) ^ swz<D>(lane / CPR)) << 4);
  auto write_v = [&](const bf16x8 (&vr)[NI]) __attribute__((always_inline)) {
    int w0 = wbase;
    asm volatile("" : "+v"(w0));
#pragma unroll
    for (int i = 0; i < NI; ++i)
      *reinterpret_cast<bf16x8 *>(vt + (w0 ^ (swz<D>(RPI * i) << 4)) + RPI * i * (D * 2)) = vr[i];
  };
  // V^T as the A operand of the PV product for channel block db: lane (j, bq)
  // holds channel 16 db + j of keys 4 bq .. 4 bq + 3 and 16 + 4 bq .. + 3, the
  // keys its P^T registers hold. Each transposed read of a 16-lane group
  // covers 4 key rows x 16 channels; lane j addresses row j / 4, channels
  // 4 (j % 4) .. + 3 of it and receives channel j of all four rows. Channel
  // block db moves the chunk index by an XOR with 2 db, and rows 16 apart
  // share their swizzle.
  const int vrow = 4 * bq + (j >> 2);
  const int tbase = vrow * (D * 2) + ((((j & 3) >> 1) ^ swz<D>(vrow)) << 4) + (j & 1) * 8;
  auto vt_frag = [&](int t0, int db) __attribute__((always_inline)) {
    const lds_char_t *base = (const lds_char_t *)vt + (t0 ^ (db << 5));
    const i16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4_t *)base);
    const i16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4_t *)(base + 16 * D * 2));
    typedef short i16x8 __attribute__((ext_vector_type(8)));
    return __builtin_bit_cast(bf16x8, (i16x8)__builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
  };

  float m_run[NB], l_run[NB];
  f32x4 oacc[NB][NDB];
#pragma unroll
  for (int rb = 0; rb < NB; ++rb) {
    m_run[rb] = -INFINITY;
    l_run[rb] = 0.0f;
#pragma unroll
    for (int db = 0; db < NDB; ++db) oacc[rb][db] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  }

  auto compute = [&](int tile, const bf16x8 (&kr)[2 * NQ]) __attribute__((always_inline)) {
    const int key0 = tile * kDecTile;
    bf16x8 pf[NB];
#pragma unroll
    for (int rb = 0; rb < NB; ++rb) {
      // S^T: register e of score block kb of lane (j, bq) is key 16 kb + 4 bq + e, row j.
      f32x4 s[2];
#pragma unroll
      for (int kb = 0; kb < 2; ++kb) {
        s[kb] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int st = 0; st < NQ; ++st) s[kb] = mfma16(kr[kb * NQ + st], qf[rb][st], s[kb]);
      }
      if (key0 + kDecTile - 1 > w.full) {
        const int lim = my_lim[rb] - key0 - 4 * bq;
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
          for (int e = 0; e < 4; ++e) s[kb][e] = 16 * kb + e <= lim ? s[kb][e] : -INFINITY;
      }
      float mx = -INFINITY;
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int e = 0; e < 4; ++e) mx = fmaxf(mx, s[kb][e]);
      mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
      mx = fmaxf(mx, __shfl_xor(mx, 32, 64)) * c;
      const float m_new = fmaxf(m_run[rb], mx);
      const float mu = m_new == -INFINITY ? 0.0f : m_new;
      const float alpha = fast_exp2(m_run[rb] - mu);
      float ls = 0.0f;
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float pv = fast_exp2(fmaf(s[kb][e], c, -mu));
          ls += pv;
          pf[rb][4 * kb + e] = (__bf16)pv;
        }
      l_run[rb] = l_run[rb] * alpha + ls;
      m_run[rb] = m_new;
#pragma unroll
      for (int db = 0; db < NDB; ++db) oacc[rb][db] *= alpha;
    }
    int t0 = tbase;
    asm volatile("" : "+v"(t0));
#pragma unroll
    for (int db = 0; db < NDB; ++db) {
      const bf16x8 vf = vt_frag(t0, db);
#pragma unroll
      for (int rb = 0; rb < NB; ++rb) oacc[rb][db] = mfma16(vf, pf[rb], oacc[rb][db]);
    }
  };

  // Tiles tile0 + wave, + 4, ...: the K loads of the wave's next tile go out
  // before this tile's V is written to LDS, its V loads right after (into the
  // registers that the write has just read), and both are in flight while
  // this tile's products run; the page ids come one tile earlier still.
  bf16x8 kra[2 * NQ], krb[2 * NQ], vr[NI];
  int t = w.tile0 + wave;
  TilePages next{};
  if (t < w.tile1) {
    const TilePages tp = tile_pages(t);
    load_k(t, tp, kra);
    load_v(t, tp, vr);
    next = tile_pages(t + kDecWaves);
  }
  auto step = [&](int tile, bf16x8 (&kc)[2 * NQ], bf16x8 (&kn)[2 * NQ]) __attribute__((always_inline)) {
    const int tn = tile + kDecWaves;
    const bool more = tn < w.tile1;
    const TilePages pn = next;
    if (more) load_k(tn, pn, kn);
    write_v(vr);
    if (more) {
      load_v(tn, pn, vr);
      next = tile_pages(tn + kDecWaves);
    }
    compute(tile, kc);
  };
  for (; t < w.tile1; t += 2 * kDecWaves) {
    step(t, kra, krb);
    if (t + kDecWaves >= w.tile1) break;
    step(t + kDecWaves, krb, kra);
  }

  // Combine the four waves' partial softmax states, one row block after the
  // other. Per wave: O^T [db][e][lane] in its V tile, m and the row sum of l
  // per lane in ml.
#pragma unroll
  for (int rb = 0; rb < NB; ++rb) {
    const float l_row = l_run[rb] + __shfl_xor(l_run[rb], 16, 64);
    const float l_all = l_row + __shfl_xor(l_row, 32, 64);
    __syncthreads();   // every wave is done with its V tile (or the block before)
    float *const mine = reinterpret_cast<float *>(vt);
    float *const mlb = ml + rb * kDecWaves * 128;
#pragma unroll
    for (int db = 0; db < NDB; ++db)
#pragma unroll
      for (int e = 0; e < 4; ++e) mine[(db * 4 + e) * 64 + lane] = oacc[rb][db][e];
    mlb[wave * 128 + lane] = m_run[rb];
    mlb[wave * 128 + 64 + lane] = l_all;
    __syncthreads();
    if (row_ok[rb]) {
      float M = -INFINITY;
  #pragma unroll
      for (int v = 0; v < kDecWaves; ++v) M = fmaxf(M, mlb[v * 128 + lane]);
      float wv[kDecWaves];
      float L = 0.0f;
  #pragma unroll
      for (int v = 0; v < kDecWaves; ++v) {
        const float mv = mlb[v * 128 + lane];
        wv[v] = (M == -INFINITY || mv == -INFINITY) ? 0.0f : fast_exp2(mv - M);
        L += wv[v] * mlb[v * 128 + 64 + lane];
      }
      const int64_t R = my_R[rb];
      const float inv = L > 0.0f ? 1.0f / L : 0.0f;
      // Wave v stores channel blocks v, v + 4, ...: lane (j, bq) channels
      // 16 db + 4 bq .. + 3 of row j.
      for (int db = wave; db < NDB; db += kDecWaves) {
        f32x4 o = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  #pragma unroll
        for (int v = 0; v < kDecWaves; ++v) {
          const float *ov = reinterpret_cast<const float *>(vs + v * TB);
  #pragma unroll
          for (int e = 0; e < 4; ++e) o[e] += wv[v] * ov[(db * 4 + e) * 64 + lane];
        }
        const int ch = 16 * db + 4 * bq;
        if (my_part[rb] < 0)
          store4((__bf16 *)p.o + R * D + ch, o[0] * inv, o[1] * inv, o[2] * inv, o[3] * inv);
        else
          store4(p.part_o + (my_part[rb] * p.plane + R) * D + ch, o[0] * inv, o[1] * inv, o[2] * inv, o[3] * inv);
      }
      if (wave == 0 && bq == 0) {
        // A NaN sum stays NaN (and in the merge, so that it gives what one pass would).
        const float lse = L == 0.0f ? -INFINITY : (M + log2f(L)) * kLn2;
        if (my_part[rb] < 0) {
          const int t = my_R[rb] / Hq, h = my_R[rb] - t * Hq;
          if (p.lse != nullptr) p.lse[(int64_t)h * p.Tq + t] = lse;
        } else {
          p.part_lse[my_part[rb] * p.plane + R] = lse;
        }
      }
    }
  }
}

// LSE-weighted combination of a request's partials. A (query token, head) row
// is D/4 lanes of 4 channels each, GR of these lane groups taking every GR-th
// partial; their sums meet in LDS. Bound by latency: one group
// walking 17 splits in a row took 9.5 us of a single request's decode step
// (32 rows, 4 workgroups); eight groups per row, one workgroup each, take
// 3.9 us (the whole call 25.6 -> 23.4 us, most of it host work by then).
template <int D, int GR>
__global__ __launch_bounds__(256) void decode_merge_kernel(DecodeParams p) {
  constexpr int CPR = D / 4;
  constexpr int RPW = 256 / (CPR * GR);   // rows per workgroup
  __shared__ f32x4 acc_l[256];
  __shared__ float w_l[256];
  const int tid = threadIdx.x;
  const int c4 = tid % CPR, gr = (tid / CPR) % GR;
  const int64_t R = (int64_t)blockIdx.x * RPW + tid / (CPR * GR);
  const int Hq = p.Hkv * p.g;
  const bool live = R < p.plane;
  const int t = live ? (int)(R / Hq) : 0;
  const int ns = live ? p.tok_parts[t] : 0;
  float mx = -INFINITY;
  for (int s = c4; s < ns; s += CPR) mx = fmaxf(mx, p.part_lse[s * p.plane + R]);
#pragma unroll
  for (int m = CPR / 2; m >= 1; m >>= 1) mx = fmaxf(mx, __shfl_xor(mx, m, CPR));
  float w_sum = 0.0f;
  f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll 4
  for (int s = gr; s < ns; s += GR) {
    const float ls = p.part_lse[s * p.plane + R];
    const float wgt = ls == -INFINITY ? 0.0f : expf(ls - mx);
    w_sum += wgt;
    acc += wgt * *reinterpret_cast<const f32x4 *>(p.part_o + (s * p.plane + R) * D + c4 * 4);
  }
  if constexpr (GR > 1) {
    acc_l[tid] = acc;
    w_l[tid] = w_sum;
    __syncthreads();
    if (gr == 0) {
#pragma unroll
      for (int k = 1; k < GR; ++k) {
        acc += acc_l[tid + k * CPR];
        w_sum += w_l[tid + k * CPR];
      }
    }
  }
  if (gr != 0 || ns <= 1) return;   // (a request with one partial wrote its output itself)
  // (As for one partial: a row without weight is zero with LSE -inf, NaN stays in O and LSE.)
  const float inv = w_sum > 0.0f ? 1.0f / w_sum : 0.0f;
  store4((__bf16 *)p.o + R * D + c4 * 4, acc[0] * inv, acc[1] * inv, acc[2] * inv, acc[3] * inv);
  if (c4 == 0 && p.lse != nullptr) p.lse[(R - (int64_t)t * Hq) * p.Tq + t] = w_sum == 0.0f ? -INFINITY : mx + logf(w_sum);
}

}  // namespace

hipError_t launch_decode_bf16(const DecodeParams &p, int D, int n_work, int row_blocks, hipStream_t s) {
  const dim3 grid((unsigned)n_work), wg(kDecWaves * 64);
  if (D == 64) {
    if (row_blocks == 1) hipLaunchKernelGGL((decode_bf16_kernel<64, 1>), grid, wg, 0, s, p);
    else hipLaunchKernelGGL((decode_bf16_kernel<64, 2>), grid, wg, 0, s, p);
  } else {
    if (row_blocks == 1) hipLaunchKernelGGL((decode_bf16_kernel<128, 1>), grid, wg, 0, s, p);
    else hipLaunchKernelGGL((decode_bf16_kernel<128, 2>), grid, wg, 0, s, p);
  }
  return hipGetLastError();
}

// Groups per row: four and eight only where each takes at least two of the
// partials of the call's longest row (max_parts). With fewer the extra
// workgroups cost more than the shorter walk saves: 4,096 rows of 5 splits take
// 6.7 us with eight groups, 4.8 us with two, 4.9 us with one walking them all.
template <int D>
static void launch_decode_merge_t(const DecodeParams &p, int max_parts, hipStream_t s) {
  auto grid = [&](int gr) { const int64_t rpw = 256 / (D / 4 * gr); return dim3((unsigned)((p.plane + rpw - 1) / rpw)); };
  if (max_parts >= 16) hipLaunchKernelGGL((decode_merge_kernel<D, 8>), grid(8), dim3(256), 0, s, p);
  else if (max_parts >= 8) hipLaunchKernelGGL((decode_merge_kernel<D, 4>), grid(4), dim3(256), 0, s, p);
  else hipLaunchKernelGGL((decode_merge_kernel<D, 2>), grid(2), dim3(256), 0, s, p);
}

hipError_t launch_decode_merge_bf16(const DecodeParams &p, int D, int max_parts, hipStream_t s) {
  if (D == 64) launch_decode_merge_t<64>(p, max_parts, s);
  else launch_decode_merge_t<128>(p, max_parts, s);
  return hipGetLastError();
}

}  // namespace cas
