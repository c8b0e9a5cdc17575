// Query-row merge, evidence reduction and frame aggregation (gfx950).
//
// combine_evidence_kernel: one launch, three independent parts (ranges of
//   the block index), so that no part waits for another:
//   combine    one work-group per (query-token tile, head): merges the
//              tile's chunk partials into O and the LSE, sixteen threads per
//              row (each a contiguous D/16 slice);
//   evidence   one work-group per (64 frames, head): E[h, f] = sum over the
//              query rows r of f's video of exp2(seg[h, r, f] - lse2[h, r]),
//              i.e. each row's softmax mass on frame f (the query-frame cue
//              of Evidence Decomposition, kept as a raw sum over the query
//              rows). 16 row groups sum strided rows and are added in a fixed
//              order in LDS, one store per output: no atomics, bitwise
//              reproducible. Adjacent threads read adjacent frames of the
//              same row, so every load is coalesced;
//   text mass  one work-group per (head, video), only when requested: the
//              video's query-row mass on non-visual keys (system prefix and
//              query tokens); one wavefront per tile, rows and then tiles
//              added in a fixed order.
//   Every part that needs a row's log2 LSE rebuilds it from the chunk
//   partials the same way: the largest chunk reference, then the rescaled
//   chunk row sums added in chunk order. The evidence part computes the
//   LSE of the rows its frames read once into LDS (when they fit).
// frame_mean_kernel: one launch, two independent parts (ranges of the block
//   index):
//   means      E_qf[l, t] = sum_h E[l, h, t] / (Hq * n_text) and the mean
//              over layers (heads averaged per layer, layer kept); 32 frames
//              x 32 layer groups per work-group, layers added in a fixed
//              order;
//   E_ff       when requested, see e_ff_part.
// topk_kernel: per video, rank r(t) = #{t' : e(t') > e(t) or (e(t') == e(t)
//   and t' < t)}; frames with r(t) < k land at topk[offset + r(t)]. Ranks of a
//   strict total order are a permutation, so every slot gets one writer.
#include <type_traits>

#include "kernels.h"

namespace evisel {
namespace {

typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kTile = 64;
constexpr float kLn2 = 0.69314718055994530942f;

__device__ __forceinline__ float neg_inf() { return -__builtin_inff(); }
__device__ __forceinline__ float exp2_(float x) {
  return __builtin_amdgcn_exp2f(x);
}
__device__ __forceinline__ float log2_(float x) {
  return __builtin_amdgcn_logf(x);
}

// Chunks are taken kChunkGroup at a time, their loads in flight together (past
// the last chunk: its own again, not counted); one at a time each waited for
// its own round trip, about 1.4 us a chunk over the two passes below (references,
// then sums; up to four chunks need one round trip for both). One code path
// for all counts: groups of 8, 4, 2 and 1 take less time from 8 chunks on,
// but the longer code 0.7 us more on three.
constexpr int kChunkGroup = 4;

// References and row sums of row r in chunk slots slot0 + c .. (nch in all).
struct ChunkRefs {
  float m[kChunkGroup], l[kChunkGroup];
  __device__ __forceinline__ void load(const Workspace& ws, int slot0, int nch,
                                       int c, int r) {
#pragma unroll
    for (int u = 0; u < kChunkGroup; ++u) {
      const size_t ix = (size_t)(slot0 + min(c + u, nch - 1)) * kTile + r;
      m[u] = ws.pM[ix];
      l[u] = ws.pL[ix];
    }
  }
  __device__ __forceinline__ float most() const {
    float M = neg_inf();
#pragma unroll
    for (int u = 0; u < kChunkGroup; ++u) M = fmaxf(M, m[u]);
    return M;
  }
  // weight of chunk u in a row of reference M
  __device__ __forceinline__ float weight(int u, float M) const {
    return m[u] == neg_inf() ? 0.f : exp2_(m[u] - M);
  }
};

// Largest reference of row r over all chunks, those of the first group in g.
__device__ __forceinline__ float row_ref(const Workspace& ws, int slot0,
                                         int nch, int r, const ChunkRefs& g) {
  float M = g.most();
  for (int c = kChunkGroup; c < nch; c += kChunkGroup) {
    float m[kChunkGroup];
#pragma unroll
    for (int u = 0; u < kChunkGroup; ++u)
      m[u] = ws.pM[(size_t)(slot0 + min(c + u, nch - 1)) * kTile + r];
#pragma unroll
    for (int u = 0; u < kChunkGroup; ++u) M = fmaxf(M, m[u]);
  }
  return M;
}

// log2 LSE of row r of a query-token tile from its chunk partials (chunk
// slots slot0 .. slot0 + nch - 1; at least one).
__device__ __forceinline__ float row_lse2(const Workspace& ws, int slot0,
                                          int nch, int r) {
  ChunkRefs g;
  g.load(ws, slot0, nch, 0, r);
  const float M = row_ref(ws, slot0, nch, r, g);
  float L = 0.f;
  for (int c = 0;;) {
#pragma unroll
    for (int u = 0; u < kChunkGroup; ++u)
      if (c + u < nch) L += g.weight(u, M) * g.l[u];
    if ((c += kChunkGroup) >= nch) break;
    g.load(ws, slot0, nch, c, r);
  }
  return M + log2_(L);
}

// Sum over the 64 lanes of a wavefront, in a fixed butterfly order (the
// same result on every lane, reproducible run to run).
__device__ __forceinline__ float wave_sum(float x) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) x += __shfl_xor(x, o, 64);
  return x;
}

// Row `rr` (0-based) of video sq's query tokens, head h.
__device__ __forceinline__ float text_row_lse2(const DevPlan& pl,
                                               const Workspace& ws,
                                               const SeqDesc& sq, int h,
                                               int rr) {
  const TextTile tt = pl.tiles[sq.tile0 + (rr >> 6)];
  return row_lse2(ws, tt.slot0 + h * tt.n_chunks, tt.n_chunks, rr & 63);
}

constexpr int kCeThreads = 1024;
constexpr int kEvFrames = 64, kEvRows = kCeThreads / kEvFrames;   // 16
constexpr int kLseCache = 4096;   // query rows whose LSE the evidence part
                                  // keeps in LDS

template <int D, bool F32>
__global__ __launch_bounds__(kCeThreads) void combine_evidence_kernel(
    const DevPlan pl, const Workspace ws, const AttnCall ac,
    float* __restrict__ ev, float* __restrict__ tm) {
  __shared__ float red[kEvRows][kEvFrames];
  __shared__ float l2c[kLseCache];
  const int tid = threadIdx.x;
  const int n_comb = pl.n_tiles * pl.hq;
  const int n_fb = (pl.T + kEvFrames - 1) / kEvFrames;
  int bid = blockIdx.x;

  if (bid < n_comb) {
    // ---- combine: tile bid % n_tiles, head bid / n_tiles
    constexpr int DP = D / 16;
    const TextTile tt = pl.tiles[bid % pl.n_tiles];
    const int h = bid / pl.n_tiles;
    const BlockDesc qb = pl.blocks[tt.qblock];
    const int r = tid >> 4, part = tid & 15;
    if (r >= qb.len) return;
    const int slot0 = tt.slot0 + h * tt.n_chunks;
    ChunkRefs g;
    f32x4 t[kChunkGroup][DP / 4];
    auto load = [&](int c) {
      g.load(ws, slot0, tt.n_chunks, c, r);
#pragma unroll
      for (int u = 0; u < kChunkGroup; ++u) {
        const int slot = slot0 + min(c + u, tt.n_chunks - 1);
        const float* po = ws.pO + ((size_t)slot * kTile + r) * D + part * DP;
#pragma unroll
        for (int i = 0; i < DP / 4; ++i) t[u][i] = *(const f32x4*)(po + 4 * i);
      }
    };
    load(0);
    const float M = row_ref(ws, slot0, tt.n_chunks, r, g);
    float L = 0.f;
    float acc[DP];
#pragma unroll
    for (int i = 0; i < DP; ++i) acc[i] = 0.f;
    for (int c = 0;;) {
#pragma unroll
      for (int u = 0; u < kChunkGroup; ++u) {
        if (c + u >= tt.n_chunks) break;
        const float w = g.weight(u, M);
        L += w * g.l[u];
#pragma unroll
        for (int i = 0; i < DP; ++i) acc[i] += w * t[u][i / 4][i % 4];
      }
      if ((c += kChunkGroup) >= tt.n_chunks) break;
      load(c);
    }
    const float inv = 1.f / L;
    const int qpos = qb.start + r;
#pragma unroll
    for (int i = 0; i < DP; i += 4) {
      const f32x4 v = {acc[i] * inv, acc[i + 1] * inv, acc[i + 2] * inv,
                       acc[i + 3] * inv};
      const size_t off = ((size_t)qpos * pl.hq + h) * D + part * DP + i;
      if (F32)
        *(f32x4*)((float*)ac.o + off) = v;
      else
        *(bf16x4*)((__bf16*)ac.o + off) = __builtin_convertvector(v, bf16x4);
    }
    if (part == 0 && ac.lse)
      ac.lse[(size_t)h * pl.S + qpos] = (M + log2_(L)) * kLn2;
    return;
  }
  bid -= n_comb;

  if (bid < n_fb * pl.hq) {
    // ---- evidence: frames [f0, f0 + 64) of head h
    const int h = bid / n_fb, f0 = (bid % n_fb) * kEvFrames;
    const int fl = tid % kEvFrames, rg = tid / kEvFrames;
    const int f = f0 + fl, fv = min(f, pl.T - 1);
    const int n0 = pl.frame_seq[f0];
    const int n1 = pl.frame_seq[min(f0 + kEvFrames, pl.T) - 1];
    const SeqDesc sq = pl.seqs[pl.frame_seq[fv]];
    const float* src = ws.seg + (size_t)h * pl.segtot + sq.segbase +
                       (fv - sq.frame0);
    // the first rows' partial masses are in flight while the LSEs are built
    constexpr int kPre = 8;
    float pre[kPre];
#pragma unroll
    for (int i = 0; i < kPre; ++i) {
      const int r = rg + i * kEvRows;
      pre[i] = r < sq.n_text ? src[(size_t)r * sq.n_frames] : 0.f;
    }
    // the query rows of the videos these frames belong to are consecutive
    const SeqDesc s0 = pl.seqs[n0], s1 = pl.seqs[n1];
    const int r0 = s0.textrow0, nrows = s1.textrow0 + s1.n_text - r0;
    const bool cached = nrows <= kLseCache;
    if (cached) {
      for (int n = n0; n <= n1; ++n) {
        const SeqDesc sn = pl.seqs[n];
        for (int rr = tid; rr < sn.n_text; rr += kCeThreads)
          l2c[sn.textrow0 - r0 + rr] = text_row_lse2(pl, ws, sn, h, rr);
      }
      __syncthreads();
    }
    float acc = 0.f;
    if (f < pl.T) {
      const float* l2 = l2c + (sq.textrow0 - r0);
      auto lse = [&](int r) {
        return cached ? l2[r] : text_row_lse2(pl, ws, sq, h, r);
      };
#pragma unroll
      for (int i = 0; i < kPre; ++i) {
        const int r = rg + i * kEvRows;
        if (r < sq.n_text) acc += exp2_(pre[i] - lse(r));
      }
#pragma unroll 4
      for (int r = rg + kPre * kEvRows; r < sq.n_text; r += kEvRows)
        acc += exp2_(src[(size_t)r * sq.n_frames] - lse(r));
    }
    red[rg][fl] = acc;
    __syncthreads();
    if (rg == 0 && f < pl.T) {
      float t = 0.f;
#pragma unroll
      for (int i = 0; i < kEvRows; ++i) t += red[i][fl];
      ev[(size_t)h * pl.T + f] = t;
    }
    return;
  }
  bid -= n_fb * pl.hq;

  // ---- text mass of (head, video): wave w takes the video's tiles w,
  // w + 16, ...; lane = row of the tile
  const int h = bid / pl.n_seq, n = bid % pl.n_seq;
  const SeqDesc sq = pl.seqs[n];
  const int lane = tid & 63, wave = tid >> 6;
  float wsum = 0.f;
  for (int i = wave; i < sq.n_tiles; i += kCeThreads / 64) {
    const TextTile tt = pl.tiles[sq.tile0 + i];
    float nv = 0.f;
    if (lane < pl.blocks[tt.qblock].len) {
      const int slot0 = tt.slot0 + h * tt.n_chunks;
      const float l2 = row_lse2(ws, slot0, tt.n_chunks, lane);
      for (int c = 0; c < tt.n_chunks; c += kChunkGroup) {
        float x[kChunkGroup];
#pragma unroll
        for (int u = 0; u < kChunkGroup; ++u)
          x[u] = ws.pNV[(size_t)(slot0 + min(c + u, tt.n_chunks - 1)) * kTile +
                        lane];
#pragma unroll
        for (int u = 0; u < kChunkGroup; ++u)
          if (c + u < tt.n_chunks) nv += exp2_(x[u] - l2);
      }
    }
    wsum += wave_sum(nv);
  }
  float* part = &red[0][0];
  if (lane == 0) part[wave] = wsum;
  __syncthreads();
  if (wave == 0) {
    const float t = wave_sum(lane < kCeThreads / 64 ? part[lane] : 0.f);
    if (lane == 0) tm[(size_t)h * pl.n_seq + n] = t;
  }
}

constexpr int kFmFrames = 32, kFmLayers = 32;
constexpr int kFmThreads = kFmFrames * kFmLayers;
template <int N>
using Int = std::integral_constant<int, N>;

// E_ff[l, t]: the mean over t's earlier frames of A_ff[t, b] and the mean
// over its later frames of A_ff[a, t], averaged over the sides that exist
// (pairs outside the sparse pattern are 0). One wavefront per frame and
// kEffLayers layers: the frame's pair indexes are read once and the layers'
// values are in flight together, so the chain of dependent reads (offsets,
// indexes, values) is paid once per kEffLayers layers. Lanes take strided
// pairs, then a butterfly adds the lanes (fixed order, every lane ends with
// the same bits).
constexpr int kEffLayers = 4, kEffRuns = 8;

__device__ __forceinline__ void e_ff_part(const DevPlan& pl,
                                          const float* __restrict__ pr,
                                          int n_layers, int wv,
                                          float* __restrict__ e_ff) {
  const int lane = threadIdx.x & 63;
  const int n_lg = (n_layers + kEffLayers - 1) / kEffLayers;
  const int t = wv / n_lg, l0 = (wv % n_lg) * kEffLayers;
  if (t >= pl.T) return;
  const int o0 = pl.ff_out_ptr[t], o1 = pl.ff_out_ptr[t + 1];
  const int i0 = pl.ff_in_ptr[t], i1 = pl.ff_in_ptr[t + 1];
  const SeqDesc sq = pl.seqs[pl.frame_seq[t]];
  float o[kEffLayers], in[kEffLayers];
#pragma unroll
  for (int u = 0; u < kEffLayers; ++u) o[u] = in[u] = 0.f;
  // eight runs of 64 pairs at a time: a sink frame is the key frame of every
  // later frame, and its list would be a chain of as many round trips
  auto side = [&](const int* idx, int a, int b, float (&acc)[kEffLayers]) {
    for (int i = a + lane; i < b; i += 64 * kEffRuns) {
      int ix[kEffRuns];
      float x[kEffRuns][kEffLayers];
#pragma unroll
      for (int r = 0; r < kEffRuns; ++r)
        ix[r] = i + 64 * r < b ? idx[i + 64 * r] : -1;
#pragma unroll
      for (int r = 0; r < kEffRuns; ++r)
#pragma unroll
        for (int u = 0; u < kEffLayers; ++u)
          x[r][u] = ix[r] >= 0 && l0 + u < n_layers
                        ? pr[(size_t)(l0 + u) * pl.n_pairs + ix[r]]
                        : 0.f;
#pragma unroll
      for (int r = 0; r < kEffRuns; ++r)
#pragma unroll
        for (int u = 0; u < kEffLayers; ++u) acc[u] += x[r][u];
    }
  };
  side(pl.ff_out_idx, o0, o1, o);
  side(pl.ff_in_idx, i0, i1, in);
  const int tl = t - sq.frame0, F = sq.n_frames;
#pragma unroll
  for (int u = 0; u < kEffLayers; ++u) {
    if (l0 + u >= n_layers) break;
    const float so = wave_sum(o[u]), si = wave_sum(in[u]);
    float acc = 0.f;
    int ns = 0;
    if (tl > 0) {
      acc += so / (float)tl;
      ++ns;
    }
    if (tl < F - 1) {
      acc += si / (float)(F - 1 - tl);
      ++ns;
    }
    if (lane == 0)
      e_ff[(size_t)(l0 + u) * pl.T + t] = ns ? acc / (float)ns : 0.f;
  }
}

// Means of frames t0 .. t0 + 31 (t < t_end stored): the caller's 1,024
// threads are 32 frames x 32 layer groups, layers added in a fixed order. The
// first 32 threads return the frames' pooled means.
__device__ __forceinline__ float mean_part(const DevPlan& pl,
                                           const float* __restrict__ ev,
                                           int n_layers, int t0, int t_end,
                                           float (&red)[kFmLayers][kFmFrames],
                                           float* __restrict__ e_layer,
                                           float* __restrict__ e_qf) {
  const int tl = threadIdx.x % kFmFrames, lg = threadIdx.x / kFmFrames;
  const int t = t0 + tl;
  float part = 0.f;
  if (t < t_end) {
    const SeqDesc sq = pl.seqs[pl.frame_seq[t]];
    const float denom = (float)pl.hq * (float)sq.n_text;
    for (int l = lg; l < n_layers; l += kFmLayers) {
      const float* src = ev + (size_t)l * pl.hq * pl.T + t;
      float s = 0.f;
      // The heads by sixteen, then the rest by 8, 4, 2 and 1, a group's loads
      // in flight: one loop unrolled by 14 left up to 13 round trips behind it.
      // The means alone, 28 layers x 20,000 frames, with 12 heads: 5.5 us
      // (10.1 with that loop, 5.9 unrolled by four); 28 heads: 12.0 (11.8, 12.9).
      auto heads = [&](auto n) {
        float x[n.value];
#pragma unroll
        for (int u = 0; u < n.value; ++u) x[u] = src[(size_t)u * pl.T];
        src += (size_t)n.value * pl.T;
#pragma unroll
        for (int u = 0; u < n.value; ++u) s += x[u];
      };
      for (int h = pl.hq; h >= 16; h -= 16) heads(Int<16>{});
      if (pl.hq & 8) heads(Int<8>{});
      if (pl.hq & 4) heads(Int<4>{});
      if (pl.hq & 2) heads(Int<2>{});
      if (pl.hq & 1) heads(Int<1>{});
      const float v = s / denom;
      if (e_layer) e_layer[(size_t)l * pl.T + t] = v;
      part += v;
    }
  }
  red[lg][tl] = part;
  __syncthreads();
  float pooled = 0.f;
  if (lg == 0 && t < t_end) {
#pragma unroll
    for (int i = 0; i < kFmLayers; ++i) pooled += red[i][tl];
    pooled /= (float)n_layers;
    e_qf[t] = pooled;
  }
  return pooled;
}

__device__ __forceinline__ float rank_key(float x) {
  return x != x ? -__builtin_inff() : x;   // NaN ranks like -inf
}

// Output offset of video n's top-k: the earlier videos' counts (one wave).
__device__ __forceinline__ int topk_offset(const DevPlan& pl,
                                           const int* __restrict__ kps, int n,
                                           int lane) {
  int off = 0;
  for (int i = lane; i < n; i += 64)
    off += min(max(kps[i], 0), pl.seqs[i].n_frames);
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) off += __shfl_xor(off, o);
  return off;
}

// SMALL (no video has more than kTopkFrames frames): one work-group per video
// takes its means in two steps of 32 frames and ranks them itself, so that a
// short probe needs one launch here and not two (32 fp32 frames to their
// top-k: 44.6 us with two, 43.2 with one).
constexpr int kTopkFrames = 64;

template <bool SMALL>
__global__ __launch_bounds__(kFmThreads) void frame_mean_kernel(
    const DevPlan pl, const float* __restrict__ ev, int n_layers,
    float* __restrict__ e_layer, float* __restrict__ e_qf,
    const int* __restrict__ kps, int* __restrict__ topk,
    const float* __restrict__ pairs, float* __restrict__ e_ff) {
  __shared__ float red[kFmLayers][kFmFrames];
  const int n_mean = SMALL ? pl.n_seq : (pl.T + kFmFrames - 1) / kFmFrames;
  if ((int)blockIdx.x >= n_mean) {
    e_ff_part(pl, pairs, n_layers,
              ((int)blockIdx.x - n_mean) * (kFmThreads / 64) +
                  (int)(threadIdx.x >> 6),
              e_ff);
    return;
  }
  if constexpr (!SMALL) {
    mean_part(pl, ev, n_layers, blockIdx.x * kFmFrames, pl.T, red, e_layer,
              e_qf);
  } else {
    __shared__ float score[kTopkFrames];
    const int n = blockIdx.x, lane = threadIdx.x & 63;
    const SeqDesc sq = pl.seqs[n];
    const int F = sq.n_frames;
    for (int f0 = 0; f0 < F; f0 += kFmFrames) {
      if (f0) __syncthreads();   // red is free
      const float e = mean_part(pl, ev, n_layers, sq.frame0 + f0,
                                sq.frame0 + F, red, e_layer, e_qf);
      if (threadIdx.x < kFmFrames)
        score[f0 + threadIdx.x] = rank_key(e);
    }
    __syncthreads();
    if (threadIdx.x >= 64) return;
    const int k = min(max(kps[n], 0), F);
    const int off = topk_offset(pl, kps, n, lane);
    const float v = score[min(lane, F - 1)];
    int rank = 0;
    for (int u = 0; u < F; ++u)
      rank += score[u] > v || (score[u] == v && u < lane);
    if (lane < F && rank < k) topk[off + rank] = lane;
  }
}

// One work-group per video and 64 of its frames (lane = frame): the video's
// scores pass through LDS kTopkChunk at a time, every wavefront counts those
// of its share that rank before the lane's frame (ties before it in frame
// order: >= among the frames before the work-group's own 64, > after them),
// and the wavefronts' counts are added. A frame costs two instructions per
// score and wavefront; one work-group per video (each frame against all
// scores, one LDS read each) took 60 us on 1,024 frames.
constexpr int kTopkThreads = 512;
constexpr int kTopkWaves = kTopkThreads / 64;
constexpr int kTopkChunk = 4096;

__global__ __launch_bounds__(kTopkThreads) void topk_kernel(
    const DevPlan pl, const float* __restrict__ e_qf,
    const int* __restrict__ kps, int* __restrict__ topk) {
  __shared__ __attribute__((aligned(16))) float vals[kTopkChunk];
  __shared__ int part[kTopkWaves][64];
  const int n = blockIdx.x;
  const SeqDesc sq = pl.seqs[n];
  const int F = sq.n_frames, f0 = blockIdx.y * kTopkFrames;
  if (f0 >= F) return;
  const int k = min(max(kps[n], 0), F);
  if (k == 0) return;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const float* src = e_qf + sq.frame0;
  const int t = f0 + lane;
  const float v = rank_key(src[min(t, F - 1)]);
  int rank = 0;
  for (int c0 = 0; c0 < F; c0 += kTopkChunk) {
    const int m = min(kTopkChunk, F - c0);
    if (c0) __syncthreads();
    // past the end: NaN, which no comparison counts
    const int m4 = (m + 3) & ~3;
    for (int i = tid; i < m4; i += kTopkThreads)
      vals[i] = i < m ? rank_key(src[c0 + i]) : __builtin_nanf("");
    __syncthreads();
    // this wave's share, in fours: before the 64 frames, among them, after
    const int per = ((m4 >> 2) + kTopkWaves - 1) / kTopkWaves;
    const int a = min(wave * per, m4 >> 2) * 4;
    const int b = min((wave + 1) * per, m4 >> 2) * 4;
    const int lo = min(max(f0 - c0, a), b);           // multiples of 4
    const int hi = min(max(f0 + kTopkFrames - c0, a), b);
    typedef float f4 __attribute__((ext_vector_type(4)));
    for (int i = a; i < lo; i += 4) {
      const f4 w = *(const f4*)(vals + i);
#pragma unroll
      for (int e = 0; e < 4; ++e) rank += w[e] >= v;
    }
    for (int i = lo; i < hi; i += 4) {
      const f4 w = *(const f4*)(vals + i);
#pragma unroll
      for (int e = 0; e < 4; ++e)
        rank += w[e] > v || (w[e] == v && c0 + i + e < t);
    }
    for (int i = hi; i < b; i += 4) {
      const f4 w = *(const f4*)(vals + i);
#pragma unroll
      for (int e = 0; e < 4; ++e) rank += w[e] > v;
    }
  }
  part[wave][lane] = rank;
  __syncthreads();
  if (wave) return;
  rank = 0;
#pragma unroll
  for (int w = 0; w < kTopkWaves; ++w) rank += part[w][lane];
  const int off = topk_offset(pl, kps, n, lane);
  if (t < F && rank < k) topk[off + rank] = t;
}

// Cross-frame cue of one layer: one wavefront per frame pair (a, b). Lane r
// < N_v owns row r of frame a; it adds, over the heads in order, the row's
// normalised mass on frame b, exp2(partial - LSE), from the partial the
// attention pass left for that key tile. A top-p tile that no row of head
// h's work item kept was never computed and adds nothing. The lanes are
// then summed by a butterfly (every lane ends with the same bits) and the
// pair gets the mean over heads and frame a's rows.
constexpr int kPairWaves = 4;

constexpr int kPairHeads = 8;

__device__ __forceinline__ void frame_pair(const DevPlan& pl,
                                           const Workspace& ws, int pi,
                                           float* __restrict__ out) {
  const int lane = threadIdx.x & 63;
  if (pi >= pl.n_pairs) return;
  const FramePair fp = pl.pairs[pi];
  const int fpt = 64 / pl.Nv;
  const BlockDesc qb = pl.blocks[fp.qblock];
  const int kb = pl.col[fp.pos];
  const int loc = pl.blk_local[kb];
  const bool always = !pl.topp || kb == fp.qblock || loc < 0;
  const int group = pl.hq / pl.hkv;
  const bool rv = lane < pl.Nv;
  const int row = fp.roff + (rv ? lane : 0);
  // heads in groups of kPairHeads: the group's loads go out together, the
  // sum still runs in head order
  float acc = 0.f;
  for (int hb = 0; hb < pl.hq; hb += kPairHeads) {
    float sv[kPairHeads], l2[kPairHeads];
    bool dn[kPairHeads];
#pragma unroll
    for (int u = 0; u < kPairHeads; ++u) {
      const int h = hb + u;
      bool done = always;
      if (!always && h < pl.hq) {
        const int g0 = (h / group) * group;
        const int h0 = g0 + ((h - g0) / kHeadsPerItem) * kHeadsPerItem;
        const int nh = min(kHeadsPerItem, g0 + group - h0);
        unsigned wd = 0u;
        for (int i = 0; i < nh; ++i)
          wd |= ws.ubits[((size_t)(h0 + i) * pl.nb + fp.qblock) * pl.W +
                         (loc >> 5)];
        done = (wd >> (loc & 31)) & 1u;
      }
      dn[u] = done && rv && h < pl.hq;
      sv[u] = dn[u] ? ws.segv[(((size_t)h * pl.nnz + fp.pos) * fpt +
                                fp.koff) * 64 + row]
                    : 0.f;
      l2[u] = dn[u] ? ws.lse2v[(size_t)h * pl.S + qb.start + row] : 0.f;
    }
#pragma unroll
    for (int u = 0; u < kPairHeads; ++u)
      if (dn[u]) acc += exp2_(sv[u] - l2[u]);
  }
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) acc += __shfl_xor(acc, o);
  if (lane == 0) out[pi] = acc / ((float)pl.hq * (float)pl.Nv);
}

// The frame cues' last step, one launch (256 frames x 64 tokens, 28/4 heads: the
// layer takes 259 us, 261 with two launches): work-groups [0, n_pair_blocks) take
// the cross-frame pairs, the others the intra-frame maps, whose partial sums
// per kv head (intra_kernel) are added in kv head order and divided by Hq.
constexpr int kReduceVec = 4;   // map entries per thread (N_v^2 is a multiple)

__global__ __launch_bounds__(64 * kPairWaves) void cue_finish_kernel(
    const DevPlan pl, const Workspace ws, int n_pair_blocks,
    float* __restrict__ pairs_out, float* __restrict__ intra_out) {
  if ((int)blockIdx.x < n_pair_blocks) {
    frame_pair(pl, ws, blockIdx.x * kPairWaves + (int)(threadIdx.x >> 6),
               pairs_out);
    return;
  }
  const size_t n = (size_t)pl.T * pl.Nv * pl.Nv;
  const size_t e = ((size_t)(blockIdx.x - n_pair_blocks) * (64 * kPairWaves) +
                    threadIdx.x) * kReduceVec;
  if (e >= n) return;
  const float inv = 1.f / (float)pl.hq;
  f32x4 t = {};
  for (int kvh = 0; kvh < pl.hkv; ++kvh)
    t += *(const f32x4*)(ws.intra_part + kvh * n + e);
  t *= inv;
  float* const dst = intra_out + e;
  if (((uintptr_t)dst & 15) == 0) {
    *(f32x4*)dst = t;
  } else {   // the caller's map is 4-byte aligned only
#pragma unroll
    for (int i = 0; i < kReduceVec; ++i) dst[i] = t[i];
  }
}

}  // namespace

hipError_t launch_cue_finish(const DevPlan& p, const Workspace& w,
                             float* pairs_out, float* intra_out,
                             hipStream_t s) {
  const int pb =
      pairs_out ? (p.n_pairs + kPairWaves - 1) / kPairWaves : 0;
  const size_t n = intra_out ? (size_t)p.T * p.Nv * p.Nv : 0;
  constexpr size_t kPer = 64 * kPairWaves * kReduceVec;
  const size_t blocks = pb + (n + kPer - 1) / kPer;
  if (blocks == 0) return hipSuccess;
  if (blocks > 0x7FFFFFFF) return hipErrorInvalidValue;
  cue_finish_kernel<<<dim3((unsigned)blocks), dim3(64 * kPairWaves), 0, s>>>(
      p, w, pb, pairs_out, intra_out);
  return hipGetLastError();
}

hipError_t launch_combine_evidence(const DevPlan& p, const Workspace& w,
                                   const AttnCall& c, float* ev, float* tm,
                                   hipStream_t s) {
  const int n_fb = (p.T + kEvFrames - 1) / kEvFrames;
  const int blocks =
      p.n_tiles * p.hq + n_fb * p.hq + (tm ? p.hq * p.n_seq : 0);
  dim3 grid(blocks), block(kCeThreads);
  if (c.fp32) {
    if (c.d == 64)
      combine_evidence_kernel<64, true><<<grid, block, 0, s>>>(p, w, c, ev, tm);
    else
      combine_evidence_kernel<128, true><<<grid, block, 0, s>>>(p, w, c, ev,
                                                                tm);
  } else {
    if (c.d == 64)
      combine_evidence_kernel<64, false><<<grid, block, 0, s>>>(p, w, c, ev,
                                                                tm);
    else
      combine_evidence_kernel<128, false><<<grid, block, 0, s>>>(p, w, c, ev,
                                                                 tm);
  }
  return hipGetLastError();
}

hipError_t launch_frame_evidence(const DevPlan& p, const float* evidence,
                                 int32_t n_layers, float* e_qf_layer,
                                 float* e_qf, const int32_t* k_per_seq,
                                 int32_t* topk, const float* pairs,
                                 float* e_ff, hipStream_t s) {
  const bool small = k_per_seq && p.max_frames <= kTopkFrames;
  int64_t blocks = small ? p.n_seq : (p.T + kFmFrames - 1) / kFmFrames;
  if (e_ff) {
    constexpr int kWaves = kFmThreads / 64;
    const int64_t waves =
        (int64_t)p.T * ((n_layers + kEffLayers - 1) / kEffLayers);
    blocks += (waves + kWaves - 1) / kWaves;
  }
  if (blocks > 0x7FFFFFFF) return hipErrorInvalidValue;
  const dim3 grid((unsigned)blocks), block(kFmThreads);
  if (small)
    frame_mean_kernel<true><<<grid, block, 0, s>>>(
        p, evidence, n_layers, e_qf_layer, e_qf, k_per_seq, topk, pairs, e_ff);
  else
    frame_mean_kernel<false><<<grid, block, 0, s>>>(
        p, evidence, n_layers, e_qf_layer, e_qf, k_per_seq, topk, pairs, e_ff);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess || !k_per_seq || small) return e;
  // (at most 65,536 frames per video: 1,024 in y)
  topk_kernel<<<dim3(p.n_seq, (p.max_frames + kTopkFrames - 1) / kTopkFrames),
                dim3(kTopkThreads), 0, s>>>(p, e_qf, k_per_seq, topk);
  return hipGetLastError();
}

}  // namespace evisel
