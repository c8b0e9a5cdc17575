// fp32 attention on the bf16 matrix cores: the body of attn_kernel for fp32
// inputs. Work items, masks, evidence and outputs are attn_kernel's; what
// differs is the contraction.
//
// The fp32 MFMA runs at 1/16 of the bf16 rate, and both products of a tile on
// it bound the fp32 kernel (83 TFLOP/s of the 153 a large fp32 product
// reaches; 537 us a layer of 75 frames x 64 tokens, 28/4 heads, d = 128; now
// 305 us, and the output's relative error against fp64 5.0e-7, now 3.3e-7).
// Here every fp32 operand is the exact sum of three bf16 values, x = h + m + l with
// h = RNE(x), m = RNE(x - h), l = x - h - m (8 + 8 + 8 significant bits), and
// a product is the six partial products down to 2^-17 of it, each exact in
// the fp32 accumulator: h h, h m, m h, m m, h l, l h. What is left out, m l,
// l m and l l, is at most 2^-24 of the product, half an ulp (m is up to 2^-8 of
// x, l up to 2^-17), where an fp32 product enters its accumulator exactly; in
// return there are fewer roundings of the accumulator than on the fp32 MFMA (a
// bf16 step sums 16 products).
//
// The sum of three is exact only while the last bit of x is in bf16's range:
// for |x| >= 2^-100 with room to spare. Probabilities go in times 2^40, so that
// all that exp2 returns are (sums and accumulators are scaled back at the end).
// A nonzero V below 2^-100, or a Q or K of 2^60 and more (against which an
// inexact factor below 2^-100 could count), is marked with a NaN where it is
// split; an infinity's split is NaN by itself. A wave that ends with a
// non-finite row sum or accumulator computes its rows again with fp32 MFMA
// straight from global memory.
//
// A key tile is taken 32 keys at a time. Its K and V rows come as fp32 by
// direct global -> LDS loads, each thread then reads back the chunks it
// loaded itself, splits them and writes the three bf16 planes of K (K-tile
// swizzle) and V (transposed-read swizzle); the next half's loads are issued
// right after, so they run beside the MFMAs. Planes and raw rows are 80 KB at
// d = 128: two work-groups share a CU, and one splits (VALU, LDS writes)
// while the other multiplies. (The top-p form's tile list takes it to 84 KB
// there: one work-group a CU, without that overlap. 75 frames, retention and
// all: 1,278 us, 1,823 with fp32 MFMA, whose 128 KB held one as well.)
#pragma once
#include <type_traits>

#include "attn_tiles.h"
#include "kernels.h"

namespace evisel {
namespace {

template <int D>
struct F32Split {
  static constexpr int kKeys = 32;                 // keys of a half tile
  static constexpr int RC = D / 8;                 // 16-byte bf16 chunks a row
  static constexpr int PB = kKeys * RC * 16;       // bytes of a plane
  static constexpr int RAW = kKeys * D * 4;        // raw bytes of K or V
  static constexpr int NU = kKeys * RC / kThreads; // chunks per thread
  static constexpr int kSmem = 6 * PB + 2 * RAW;
  static constexpr float kPScale = 0x1p40f;        // on the probabilities
  static constexpr float kLeast = 0x1p-100f;       // V, unless 0
  static constexpr float kMost = 0x1p60f;          // Q and K

  // x = p[0] + p[1] + p[2], each rounded to nearest even
  __device__ static void split(const f32x8 x, bf16x8 (&p)[3]) {
    p[0] = __builtin_convertvector(x, bf16x8);
    const f32x8 r = x - __builtin_convertvector(p[0], f32x8);
    p[1] = __builtin_convertvector(r, bf16x8);
    p[2] = __builtin_convertvector(r - __builtin_convertvector(p[1], f32x8),
                                   bf16x8);
  }
  // whether 8 values of Q or K, or of V, are past what the split is used for
  __device__ static bool past_qk(const f32x4 a, const f32x4 b) {
    float x = 0.f;
#pragma unroll
    for (int e = 0; e < 4; ++e)
      x = fmaxf(x, fmaxf(__builtin_fabsf(a[e]), __builtin_fabsf(b[e])));
    return x >= kMost;
  }
  __device__ static bool past_v(const f32x4 a, const f32x4 b) {
    // twice the bits less 2: without the sign, and +-0 on top
    uint32_t x = 0xFFFFFFFFu;
#pragma unroll
    for (int e = 0; e < 4; ++e)
      x = min(x, min((__float_as_uint(a[e]) << 1) - 2u,
                     (__float_as_uint(b[e]) << 1) - 2u));
    return x < (__builtin_bit_cast(uint32_t, kLeast) << 1) - 2u;
  }
  // NaN in the highest part: the rows' results are not finite
  __device__ static void poison(bf16x8 (&p)[3], bool past) {
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    u32x4 h = __builtin_bit_cast(u32x4, p[0]);
    h[0] |= past ? 0x7FC07FC0u : 0u;
    p[0] = __builtin_bit_cast(bf16x8, h);
  }
  // 8 values of Q or K
  __device__ static void split_qk(const f32x4 a, const f32x4 b,
                                  bf16x8 (&p)[3]) {
    split(__builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7), p);
    poison(p, past_qk(a, b));
  }
  // The lane's operand of step kk from the planes of 32 K rows.
  __device__ static void k_read(const EV_LDS char* kpl, int l32, int g, int kk,
                                bf16x8 (&f)[3]) {
    const EV_LDS char* a =
        kpl + (l32 * RC + ((2 * kk + g) ^ swz<kSwzK, RC>(l32))) * 16;
#pragma unroll
    for (int q = 0; q < 3; ++q) f[q] = *(const EV_LDS bf16x8*)(a + q * PB);
  }
  // One step's six partial products; the logits are hi + lo.
  __device__ static void qk_step(const bf16x8 (&f)[3], const bf16x8 q0,
                                 const bf16x8 q1, const bf16x8 q2, f32x16& lo,
                                 f32x16& hi) {
    mm(f[2], q0, lo);
    mm(f[1], q1, lo);
    mm(f[0], q2, lo);
    mm(f[1], q0, lo);
    mm(f[0], q1, lo);
    mm(f[0], q0, hi);
  }
  __device__ static void mm(bf16x8 x, bf16x8 y, f32x16& c) {
    c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x, y, c, 0, 0, 0);
  }
  // The same logits with fp32 MFMA, from the lane's K and Q rows in memory.
  __device__ static void qk_f32(const float* kr, const float* qr, int g,
                                f32x16& s) {
    s = f32x16{};
    for (int u = 0; u < D / 8; ++u) {
      const f32x4 a = *(const f32x4*)(kr + g * (D / 2) + 4 * u);
      const f32x4 b = *(const f32x4*)(qr + g * (D / 2) + 4 * u);
#pragma unroll
      for (int e = 0; e < 4; ++e)
        s = __builtin_amdgcn_mfma_f32_32x32x2f32(a[e], b[e], s, 0, 0, 0);
    }
  }
};

template <int D, bool TOPP>
__device__ __forceinline__ void attn_f32_item(const DevPlan& pl,
                                              const Workspace& ws,
                                              const AttnCall& ac, char* smem,
                                              short* clist, int* n_kept) {
  using X = F32Split<D>;
  constexpr int RC = X::RC, PB = X::PB, NMT = D / 32, KK = D / 16;
  EV_LDS char* const kpl = (EV_LDS char*)smem;     // K planes h, m, l
  EV_LDS char* const vpl = kpl + 3 * PB;           // V planes
  EV_LDS char* const raw = kpl + 6 * PB;           // [wave][K, V][loads]

  const WorkItem it = pl.items[blockIdx.x];
  if (it.qblock < 0) return;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, g = lane >> 5;
  const int hsub = wave >> 1;
  const bool uni = it.qblock2 >= 0;
  const int nhalf = uni ? 2 : it.nheads;
  const bool active = hsub < nhalf;
  const int hd1 = uni ? it.head : it.head + 1;
  const int h = active && hsub ? hd1 : it.head;
  const int kvh = it.head / (pl.hq / pl.hkv);
  const int qbid = uni && hsub ? it.qblock2 : it.qblock;
  const BlockDesc qb = pl.blocks[qbid];
  const bool is_text = it.slot >= 0;
  const int qrow = 32 * (wave & 1) + l32;
  const bool qvalid = active && qrow < qb.len;
  const int qpos = qb.start + qrow;
  int n = it.kb_end - it.kb_begin;
  const int b0 = it.kb_begin;
  const float c2 = ac.scale_log2;
  const float* const kg = (const float*)ac.k + (size_t)kvh * D;
  const float* const vg = (const float*)ac.v + (size_t)kvh * D;
  const uint32_t rowbytes = (uint32_t)pl.hkv * D * 4;
  const float* const qg =
      (const float*)ac.q + ((size_t)(qvalid ? qpos : qb.start) * pl.hq + h) * D;

  // The lane's query row as three planes of the QK B operand.
  bf16x8 qf[3][KK];
#pragma unroll
  for (int kk = 0; kk < KK; ++kk) {
    const f32x4 a = *(const f32x4*)(qg + 16 * kk + 8 * g);
    const f32x4 b = *(const f32x4*)(qg + 16 * kk + 8 * g + 4);
    bf16x8 p[3];
    X::split_qk(a, b, p);
#pragma unroll
    for (int u = 0; u < 3; ++u) qf[u][kk] = p[u];
  }

  // Chunk u of this thread: row crow + u * CSTEP, 8 values from 8 * ccol. Its
  // two 16-byte halves are two loads, at 16 * lane of the wave's slots.
  constexpr int CSTEP = kThreads / RC;
  const int crow = tid / RC, ccol = tid % RC;
  EV_LDS char* const kraw = raw + wave * (X::NU * 2 * 1024);
  EV_LDS char* const vraw = kraw + X::RAW;
  auto issue = [&](int start, int len) {   // len in 1 .. 32
    const char* kb = (const char*)kg + (size_t)start * rowbytes;
    const char* vb = (const char*)vg + (size_t)start * rowbytes;
#pragma unroll
    for (int u = 0; u < X::NU; ++u) {
      const uint32_t off =
          (uint32_t)min(crow + u * CSTEP, len - 1) * rowbytes + ccol * 32;
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        lds_dma16((uint32_t)(uintptr_t)kraw + (2 * u + e) * 1024, kb,
                  off + 16 * e);
        lds_dma16((uint32_t)(uintptr_t)vraw + (2 * u + e) * 1024, vb,
                  off + 16 * e);
      }
    }
  };
  // raw rows -> planes (this thread's own chunks)
  auto split_tile = [&]() {
#pragma unroll
    for (int u = 0; u < X::NU; ++u) {
      const int row = crow + u * CSTEP;
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        const EV_LDS char* src = (t ? vraw : kraw) + 2 * u * 1024 + lane * 16;
        const f32x4 a = *(const EV_LDS f32x4*)src;
        const f32x4 b = *(const EV_LDS f32x4*)(src + 1024);
        bf16x8 p[3];
        X::split(__builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7), p);
        X::poison(p, t ? X::past_v(a, b) : X::past_qk(a, b));
        const int ch =
            ccol ^ (t ? swz<kSwzV, RC>(row) : swz<kSwzK, RC>(row));
        EV_LDS char* const dst = (t ? vpl : kpl) + (row * RC + ch) * 16;
#pragma unroll
        for (int q = 0; q < 3; ++q) *(EV_LDS bf16x8*)(dst + q * PB) = p[q];
      }
    }
  };

  // ---- tile descriptors, 64 at a time (as attn_kernel)
  int dsc_start = 0, dsc_len = 1, dsc_region = 0, dsc_aux = 0, dsc_loc = -1,
      dsc_pos = 0;
  auto load_batch = [&](int batch) {
    const int t = batch * 64 + lane;
    if (t < n) {
      const int pos = TOPP ? (int)clist[t] : t;
      const BlockDesc bd =
          uni ? pl.ptile_desc[b0 + pos] : pl.col_desc[b0 + pos];
      dsc_start = bd.start;
      dsc_len = bd.len;
      dsc_region = bd.region;
      dsc_aux = bd.aux;
      if (uni) {
        const PairedTile pt = pl.ptile[b0 + pos];
        dsc_pos = hsub ? pt.pos[1] : pt.pos[0];
        if (TOPP) {
          const int loc = pl.blk_local[pt.block];
          dsc_loc = pt.block == qbid ? -1 : loc;
          if (dsc_pos >= 0 && dsc_loc >= 0 &&
              !((ws.ubits[((size_t)it.head * pl.nb + qbid) * pl.W +
                          (loc >> 5)] >> (loc & 31)) & 1u))
            dsc_pos = -1;
        }
      } else {
        dsc_pos = b0 + pos;
        if (TOPP) {
          const int bid = pl.col[b0 + pos];
          dsc_loc = bid == it.qblock ? -1 : pl.blk_local[bid];
        }
      }
    }
  };
  struct Tile {
    int start, len, region, aux, loc, pos;
  };
  auto desc = [&](int t) {
    const int l = t & 63;
    Tile d;
    d.start = __builtin_amdgcn_readlane(dsc_start, l);
    d.len = __builtin_amdgcn_readlane(dsc_len, l);
    d.region = __builtin_amdgcn_readlane(dsc_region, l);
    d.aux = __builtin_amdgcn_readlane(dsc_aux, l);
    d.loc = TOPP ? __builtin_amdgcn_readlane(dsc_loc, l) : -1;
    d.pos = __builtin_amdgcn_readlane(dsc_pos, l);
    return d;
  };
  // top-p: the CSR positions of the candidate tiles some row of the item kept
  if constexpr (TOPP) {
    if (wave == 0) {
      const uint32_t* ub =
          ws.ubits + ((size_t)it.head * pl.nb + it.qblock) * pl.W;
      const size_t hstride = (size_t)pl.nb * pl.W;
      int base = 0;
      for (int c0 = 0; c0 < n; c0 += 64) {
        const int t = c0 + lane;
        bool keep = false;
        if (t < n && uni) {
          const PairedTile pt = pl.ptile[b0 + t];
          const int loc = pl.blk_local[pt.block];
          for (int k = 0; k < 2; ++k) {
            const int own = k ? it.qblock2 : it.qblock;
            if (pt.pos[k] < 0) continue;
            if (loc < 0 || pt.block == own) {
              keep = true;
            } else {
              const unsigned wd =
                  ws.ubits[((size_t)it.head * pl.nb + own) * pl.W +
                           (loc >> 5)];
              keep = keep || ((wd >> (loc & 31)) & 1u);
            }
          }
        } else if (t < n) {
          const int bid = pl.col[b0 + t];
          const int loc = pl.blk_local[bid];
          if (loc < 0 || bid == it.qblock) {
            keep = true;
          } else {
            unsigned wd = 0u;
            for (int i = 0; i < it.nheads; ++i)
              wd |= ub[i * hstride + (loc >> 5)];
            keep = (wd >> (loc & 31)) & 1u;
          }
        }
        const unsigned long long m = __ballot(keep);
        const int pos = __builtin_amdgcn_mbcnt_hi(
            (unsigned)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)m, 0u));
        if (keep) clist[base + pos] = (short)t;
        base += __popcll(m);
      }
      if (lane == 0) *n_kept = base;
    }
    __syncthreads();
    n = __builtin_amdgcn_readfirstlane(*n_kept);
  }

  // ---- per-row state
  float m_ref = neg_inf(), l_part = 0.f, nv_part = 0.f, fr_part = 0.f;
  f32x16 o[NMT];
#pragma unroll
  for (int i = 0; i < NMT; ++i) o[i] = f32x16{};
  SeqDesc sq{};
  if (is_text) sq = pl.seqs[it.seq];
  const int trow = qb.aux + qrow - sq.textrow0;
  float* const seg_row = ws.seg + (size_t)h * pl.segtot + sq.segbase +
                         (size_t)trow * sq.n_frames - sq.frame0;
  const bool vis_ff = ac.segv != nullptr && !is_text && qb.region == kVis;
  const int fpt = kTile / pl.Nv;
  float* const segv_row =
      vis_ff ? ac.segv + (size_t)h * pl.nnz * fpt * kTile + qrow : nullptr;
  const uint32_t* rrow =
      TOPP ? ws.rbits + ((size_t)h * pl.nb + qbid) * pl.W * 64 + qrow
           : nullptr;
  auto row_bits = [&](int loc) -> unsigned {
    return loc < 0 ? ~0u : rrow[(size_t)(loc >> 5) * 64];
  };

  // keys of half c after the row (causal) or past the tile's end -> -inf
  auto mask_half = [&](f32x16& s, int c, const Tile& t) {
    if (t.len < kTile || t.start + t.len - 1 > qb.start) {
      const int x = min(qpos - t.start, t.len - 1) - 4 * g - 32 * c;
#pragma unroll
      for (int r = 0; r < 16; ++r)
        if (8 * (r >> 2) + (r & 3) > x) s[r] = neg_inf();
    }
  };
  // exact reference: row max of the half; accumulators rescaled if it rises
  auto half_ref = [&](f32x16& s, bool kept) {
    if (TOPP && __any(!kept)) {
#pragma unroll
      for (int r = 0; r < 16; ++r) s[r] = kept ? s[r] : neg_inf();
    }
    float mx = neg_inf();
#pragma unroll
    for (int r = 0; r < 16; ++r) mx = fmaxf(mx, s[r]);
    mx = pair_max(mx);
    const float m_new = fmaxf(m_ref, mx * c2);
    const bool need = m_new > m_ref + kRescaleSlack;
    const bool resc = need && m_ref != neg_inf();
    if (__any(resc)) {
      const float alpha = resc ? exp2_(m_ref - m_new) : 1.f;
      l_part *= alpha;
      nv_part *= alpha;
      fr_part *= alpha;
#pragma unroll
      for (int i = 0; i < NMT; ++i) o[i] *= alpha;
    }
    m_ref = need ? m_new : m_ref;
  };
  // probabilities, and with them row sums and accumulators, times 2^40 (SPLIT)
  // or as they are (the fp32 MFMA pass)
  auto probs = [&](f32x16& s, float mu, auto split) -> float {
    float ts = 0.f;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      s[r] = exp2_(fmaf(s[r], c2, -mu)) * (split.value ? X::kPScale : 1.f);
      ts += s[r];
    }
    return ts;
  };
  // per-frame log2 partial masses of half c (query rows; visual rows with
  // frame cues), or the query rows' non-visual mass
  auto evidence = [&](const f32x16& s, float ts, int c, const Tile& t,
                      auto split) {
    constexpr float kUnit = split.value ? 1.f / X::kPScale : 1.f;
    if (!is_text && !vis_ff) return;
    const float mu = m_ref == neg_inf() ? 0.f : m_ref;
    if (t.region == kVis) {
      float* const dst = is_text ? seg_row + t.aux
                                 : segv_row + (size_t)t.pos * fpt * kTile;
      const int dstride = is_text ? 1 : kTile;
      if (pl.Nv == kTile) {
        fr_part = c ? fr_part + ts : ts;
        if (c) {
          const float f = pair_sum(fr_part);
          if (g == 0 && qvalid) *dst = mu + log2_(f * kUnit);
        }
      } else {
        float g4[4];
#pragma unroll
        for (int q = 0; q < 4; ++q)
          g4[q] = pair_sum(s[4 * q] + s[4 * q + 1] + s[4 * q + 2] +
                           s[4 * q + 3]);
        const int lg = __builtin_ctz((unsigned)pl.Nv) - 3;   // log2(N_v / 8)
        const int nseg = 32 / pl.Nv;
        for (int si = 0; si < nseg; ++si) {
          float f = 0.f;
#pragma unroll
          for (int q = 0; q < 4; ++q) f += (q >> lg) == si ? g4[q] : 0.f;
          if (g == 0 && qvalid && 32 * c + si * pl.Nv < t.len)
            dst[(c * nseg + si) * dstride] = mu + log2_(f * kUnit);
        }
      }
    } else if (is_text) {
      nv_part += ts;
    }
  };

  // ---- products of a half tile from the planes
  typename Bf16Path<D>::PvOff pvo;
  Bf16Path<D>::pv_offsets(pvo, lane);
  // (the operands of a step are read during the step before; the barriers
  // keep the scheduler from reading further ahead than the registers allow)
  auto qk_half = [&](f32x16& s) {
    f32x16 lo = {}, hi = {};
    bf16x8 kf[2][3];
    X::k_read(kpl, l32, g, 0, kf[0]);
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) {
      if (kk + 1 < KK) X::k_read(kpl, l32, g, kk + 1, kf[(kk + 1) & 1]);
      X::qk_step(kf[kk & 1], qf[0][kk], qf[1][kk], qf[2][kk], lo, hi);
      __builtin_amdgcn_sched_barrier(0);
    }
    s = hi + lo;
  };
  auto v_read = [&](bf16x8 (&f)[3], int ks, int mt) {
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      const EV_LDS char* a0 = vpl + q * PB + pvo.v[mt] + 16 * ks * RC * 16;
      const i16x4 lohi[2] = {
          __builtin_amdgcn_ds_read_tr16_b64_v4i16((EV_LDS i16x4*)a0),
          __builtin_amdgcn_ds_read_tr16_b64_v4i16(
              (EV_LDS i16x4*)(a0 + 8 * RC * 16))};
      f[q] = __builtin_bit_cast(bf16x8, lohi);
    }
  };
  auto pv_half = [&](const f32x16& p) {
    bf16x8 pb[2][3];
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      f32x8 x;
#pragma unroll
      for (int e = 0; e < 8; ++e) x[e] = p[8 * ks + e];
      X::split(x, pb[ks]);
    }
    bf16x8 vf[2][3];
    v_read(vf[0], 0, 0);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < 2 * NMT; ++i) {
      const int ks = i / NMT, mt = i % NMT;
      if (i + 1 < 2 * NMT) v_read(vf[(i + 1) & 1], (i + 1) / NMT, (i + 1) % NMT);
      const bf16x8(&f)[3] = vf[i & 1];
      X::mm(f[2], pb[ks][0], o[mt]);
      X::mm(f[1], pb[ks][1], o[mt]);
      X::mm(f[0], pb[ks][2], o[mt]);
      X::mm(f[1], pb[ks][0], o[mt]);
      X::mm(f[0], pb[ks][1], o[mt]);
      X::mm(f[0], pb[ks][0], o[mt]);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  auto compute = [&](const Tile& t, int c, unsigned bits) {
    f32x16 s;
    qk_half(s);
    mask_half(s, c, t);
    const bool kept = !TOPP || t.loc < 0 || ((bits >> (t.loc & 31)) & 1u);
    // once every row of the wave has a reference, the row max is needed only
    // if a probability against it exceeds 2^kFastSlack (or is not finite)
    bool exact = __any(m_ref == neg_inf());
    float ts = 0.f;
    if (!exact) {
      ts = probs(s, kept ? m_ref : __builtin_inff(), std::true_type{});
      exact = __any(!(ts <= kFastBound * X::kPScale));
      if (exact) {
        qk_half(s);
        mask_half(s, c, t);
      }
    }
    if (exact) {
      half_ref(s, kept);
      ts = probs(s, m_ref == neg_inf() ? 0.f : m_ref, std::true_type{});
    }
    l_part += ts;
    evidence(s, ts, c, t, std::true_type{});
    pv_half(s);
  };

  // ---- the item's half tiles: half j + 1 streams in while j is computed
  load_batch(0);
  Tile cur = desc(0);
  unsigned bits = ~0u;
  if (n > 0) {
    issue(cur.start, min(cur.len, 32));
    if (TOPP) bits = row_bits(cur.loc);
  }
  for (int t = 0, c = 0; t < n;) {
    const bool more = c == 0 && cur.len > 32;      // this tile's second half
    const int t2 = more ? t : t + 1;
    Tile nxt = cur;
    unsigned nbits = bits;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();                               // the planes are free
    split_tile();
    if (t2 < n) {
      if (!more) {
        if ((t2 & 63) == 0) load_batch(t2 >> 6);
        nxt = desc(t2);
        if (TOPP) nbits = row_bits(nxt.loc);
      }
      const int k0 = more ? 32 : 0;
      issue(nxt.start + k0, min(nxt.len - k0, 32));
    }
    __syncthreads();                               // the planes are written
    // (a half that lies after every row of the wave is all masked)
    if (active && cur.pos >= 0 &&
        cur.start + 32 * c <= qb.start + 32 * (wave & 1) + 31)
      compute(cur, c, bits);
    c = more ? 1 : 0;
    t = t2;
    cur = nxt;
    bits = nbits;
  }
  if (!active) return;

  // ---- rows with a non-finite result: again in fp32 throughout
  float unit = 1.f / X::kPScale;
  float chk = l_part - l_part;
#pragma unroll
  for (int i = 0; i < NMT; ++i)
#pragma unroll
    for (int r = 0; r < 16; ++r) chk += o[i][r] - o[i][r];
  if (__any(qvalid && chk != 0.f)) {
    unit = 1.f;
    m_ref = neg_inf();
    l_part = nv_part = fr_part = 0.f;
#pragma unroll
    for (int i = 0; i < NMT; ++i) o[i] = f32x16{};
    for (int t = 0; t < n; ++t) {
      if ((t & 63) == 0) load_batch(t >> 6);
      const Tile d = desc(t);
      if (d.pos < 0) continue;
      const unsigned wd = TOPP ? row_bits(d.loc) : ~0u;
      const bool kept = !TOPP || d.loc < 0 || ((wd >> (d.loc & 31)) & 1u);
      for (int c = 0; c < 2 && 32 * c < d.len; ++c) {
        f32x16 s;
        X::qk_f32(kg + (size_t)(d.start + min(32 * c + l32, d.len - 1)) *
                           pl.hkv * D,
                  qg, g, s);
        mask_half(s, c, d);
        half_ref(s, kept);
        const float ts =
            probs(s, m_ref == neg_inf() ? 0.f : m_ref, std::false_type{});
        l_part += ts;
        evidence(s, ts, c, d, std::false_type{});
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int key = min(32 * c + 8 * (r >> 2) + 4 * g + (r & 3),
                              d.len - 1);
          const float* const vr = vg + (size_t)(d.start + key) * pl.hkv * D;
#pragma unroll
          for (int mt = 0; mt < NMT; ++mt)
            o[mt] = __builtin_amdgcn_mfma_f32_32x32x2f32(
                vr[32 * mt + l32], s[r], o[mt], 0, 0, 0);
        }
      }
    }
  }

  // ---- outputs, straight from the lanes' rows
  const float l_tot = pair_sum(l_part) * unit, nv_tot = pair_sum(nv_part) * unit;
  if (!qvalid) return;
  if (!is_text) {
    const float inv = unit / l_tot;
#pragma unroll
    for (int mt = 0; mt < NMT; ++mt)
#pragma unroll
      for (int r4 = 0; r4 < 4; ++r4) {
        const f32x4 v = {o[mt][4 * r4] * inv, o[mt][4 * r4 + 1] * inv,
                         o[mt][4 * r4 + 2] * inv, o[mt][4 * r4 + 3] * inv};
        *(f32x4*)((float*)ac.o + ((size_t)qpos * pl.hq + h) * D + 32 * mt +
                  8 * r4 + 4 * g) = v;
      }
    if (g == 0 && ac.lse)
      ac.lse[(size_t)h * pl.S + qpos] = (m_ref + log2_(l_tot)) * kLn2;
    if (g == 0 && ac.lse2v)
      ac.lse2v[(size_t)h * pl.S + qpos] = m_ref + log2_(l_tot);
  } else {
    const int slot =
        uni ? (hsub ? it.slot2 : it.slot) : it.slot + hsub * it.nch;
    float* const po = ws.pO + ((size_t)slot * kTile + qrow) * D;
#pragma unroll
    for (int mt = 0; mt < NMT; ++mt)
#pragma unroll
      for (int r4 = 0; r4 < 4; ++r4) {
        const f32x4 v = {o[mt][4 * r4] * unit, o[mt][4 * r4 + 1] * unit,
                         o[mt][4 * r4 + 2] * unit,
                         o[mt][4 * r4 + 3] * unit};
        *(f32x4*)(po + 32 * mt + 8 * r4 + 4 * g) = v;
      }
    if (g == 0) {
      const size_t ix = (size_t)slot * kTile + qrow;
      ws.pM[ix] = m_ref;
      ws.pL[ix] = l_tot;
      ws.pNV[ix] = nv_tot > 0.f ? m_ref + log2_(nv_tot) : neg_inf();
    }
  }
}

// The fp32 form of the intra-frame cue's products (intra_kernel, attn.hip):
// acc[c] += the probabilities of the wave's heads at keys 32 c .. 32 c + 31 of
// block qb. The logits are the attention pass's, by the same split and in the
// same order, so that their rounding cancels against the saved LSE's: 21
// frames x 64 tokens, d = 128, LSE up to 70: the maps are 1.7e-6 off fp64
// (2-norm), 5.8e-6 with fp32 MFMA here, 3.2e-6 with fp32 MFMA in both passes.
// smem: the planes of both 32-key halves. (75 frames x 64 tokens, 28/4 heads,
// d = 128: the layer with cues takes 353 us, 378 with fp32 MFMA here.)
template <int D>
__device__ __forceinline__ void intra_f32_part(const DevPlan& pl,
                                               const Workspace& ws,
                                               const AttnCall& ac,
                                               const BlockDesc& qb, int kvh,
                                               int tid, int wave, char* smem,
                                               f32x16 (&acc)[2]) {
  using X = F32Split<D>;
  constexpr int RC = X::RC, PB = X::PB, KK = D / 16, CSTEP = kThreads / RC;
  EV_LDS char* const kpl = (EV_LDS char*)smem;
  const int lane = tid & 63, l32 = lane & 31, g = lane >> 5;
  const int qrow = 32 * (wave & 1) + l32;
  const bool qvalid = qrow < qb.len;
  const int qpos = qb.start + (qvalid ? qrow : 0);
  const int group = pl.hq / pl.hkv;
  const float* const kg = (const float*)ac.k + (size_t)kvh * D;
  const int crow = tid / RC, ccol = tid % RC;
#pragma unroll
  for (int u = 0; u < 2 * X::NU; ++u) {
    const int row = crow + u * CSTEP, r32 = row & 31;
    const float* const src =
        kg + (size_t)(qb.start + min(row, qb.len - 1)) * pl.hkv * D + 8 * ccol;
    bf16x8 p[3];
    X::split_qk(*(const f32x4*)src, *(const f32x4*)(src + 4), p);
    EV_LDS char* const dst = kpl + (row >> 5) * 3 * PB +
                             (r32 * RC + (ccol ^ swz<kSwzK, RC>(r32))) * 16;
#pragma unroll
    for (int q = 0; q < 3; ++q) *(EV_LDS bf16x8*)(dst + q * PB) = p[q];
  }
  unsigned vis = 0u;   // bit 16 c + r: the row sees key r of half c, in its frame
#pragma unroll
  for (int i = 0; i < 32; ++i) {
    const int kl = 32 * (i >> 4) + 8 * ((i & 15) >> 2) + 4 * g + (i & 3);
    if (qvalid && kl <= qrow && kl / pl.Nv == qrow / pl.Nv) vis |= 1u << i;
  }
  // waves 0-1 take the group's even heads, waves 2-3 the odd ones; a step's
  // query values are read for the next head once they are used
  f32x4 raw[KK][2];
  auto q_row = [&](int hi) {
    return (const float*)ac.q +
           ((size_t)qpos * pl.hq + kvh * group + hi) * D;
  };
  auto fetch = [&](int hi, int kk) {
    const float* const src = q_row(hi) + 16 * kk + 8 * g;
    raw[kk][0] = *(const f32x4*)src;
    raw[kk][1] = *(const f32x4*)(src + 4);
  };
  int hi = wave >> 1;
  if (hi < group)
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) fetch(hi, kk);
  __syncthreads();
  for (; hi < group; hi += 2) {
    const float l2 = ws.lse2v[(size_t)(kvh * group + hi) * pl.S + qpos];
    const bool more = hi + 2 < group;
    f32x16 lo[2] = {f32x16{}, f32x16{}}, s[2] = {f32x16{}, f32x16{}};
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) {
      bf16x8 q[3];
      X::split_qk(raw[kk][0], raw[kk][1], q);
      if (more) fetch(hi + 2, kk);
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        bf16x8 f[3];
        X::k_read(kpl + c * 3 * PB, l32, g, kk, f);
        X::qk_step(f, q[0], q[1], q[2], lo[c], s[c]);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    bool bad = false;
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      s[c] = s[c] + lo[c];
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const float x = vis >> (16 * c + r) & 1u ? s[c][r] : 0.f;
        bad = bad || x - x != 0.f;
      }
    }
    if (__any(bad))   // as the attention pass: again with fp32 MFMA
#pragma unroll
      for (int c = 0; c < 2; ++c)
        X::qk_f32(kg + (size_t)(qb.start + min(32 * c + l32, qb.len - 1)) *
                           pl.hkv * D,
                  q_row(hi), g, s[c]);
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int r = 0; r < 16; ++r)
        acc[c][r] += vis >> (16 * c + r) & 1u
                         ? exp2_(fmaf(s[c][r], ac.scale_log2, -l2)) : 0.f;
  }
}

}  // namespace
}  // namespace evisel
