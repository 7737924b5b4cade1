// Blockwise vocabulary projection loss (the MoP paper's data-tensor-parallel
// projection, Sec. 3.4 eq. voc-fwd-loss, on one device: P = 1, blocks of the
// vocabulary instead of ranks).  Y = X W_voc is never written anywhere:
//  * forward, per block of `vblock` columns: one bf16 matrix-core product
//    whose epilogue reduces each row's logits to a (max, sum exp(y - max))
//    pair per 64 columns and picks up the target's logit; a one-wave-per-row
//    kernel merges the block's pairs, in column order, into the row's running
//    pair (blocks in order, so the result is a function of the inputs and
//    vblock alone, bit for bit).  The forward walks as many of the caller's
//    blocks at once as its partial pairs fit the workspace for (fwd_span
//    below);
//  * backward, per block: the product is recomputed and its epilogue turns
//    each logit into the logit gradient G = dl ([v == t] - exp(y - lse)),
//    rounded to bf16 (the only per-block buffer, N x vblock bf16); then
//    dX += G W_block^T (fp32, the block's columns cut into K ranges that
//    accumulate into separate fp32 slabs so the product fills the chip) and
//    dW[:, block] = X^T G (bf16, each column written once).
// All products run on the library's grouped GEMM kernel (dense modes).  When
// V is not a multiple of 8 the rows of W and dW are not 16-byte aligned: each
// block of W is first copied into a padded buffer (the product's direct loads
// to LDS want aligned pieces), dW is stored in place.  The same copy takes the
// place of rows so long that a tile's rows lie further apart than a buffer
// descriptor reaches (beyond 34 million columns in the forward, 4 million in
// the backward), and blocks longer than that are cut (reach, below).
#include "common.h"

#include <algorithm>

namespace moe {
namespace {

// Merge of two (max, sum of exp(y - max)) pairs; an empty pair is (-inf, 0).
// The fused add is written out, so that every caller rounds alike.
__device__ __forceinline__ void lse_merge(float& m, float& s, float m2, float s2) {
  const float mm = fmaxf(m, m2);
  if (mm == -__builtin_huge_valf()) return;  // both empty
  s = __builtin_fmaf(s2, __expf(m2 - mm), s * __expf(m - mm));
  m = mm;
}

// W waves per row n: the partial pairs part[n][0..ng) of the caller's blocks
// of per groups each (the last may have fewer).  A block's pairs are merged in
// order (lane l takes groups l, l + 64, ... ascending, then a fixed xor tree
// over the lanes); the blocks' pairs then go into the row's running pair
// (m, s) in order, so the result does not depend on how many blocks a launch
// takes.  A block of fewer than 64 groups takes `sub` lanes of a wave (a power
// of two, per <= sub): the other lanes would hold empty pairs, which merge
// without a trace.  The last launch turns the row's pair into its results:
// lse_n = m_n + log s_n, loss_n = y_{n, t_n} - lse_n.  Bound by latency (loads,
// then up to twelve dependent shuffles and exponentials a block): where one
// wave would come round its 64 / sub blocks often, four waves share a row, 128 /
// sub blocks each at a time (N = 1000, H = 520, V = 32003 in blocks of 4096,
// loss and gradients: 497 us against 500 with one wave a row, and 499 with the
// results in a launch of their own; forward of N = 2048, H = 64, V = 8192 in
// blocks of 512: 20 us, with sub = 64 27, with sub = 8 but four waves 22).
template <int W>
__global__ __launch_bounds__(256) void voc_merge_kernel(const float2* __restrict__ part, int ng,
                                                        int per, int sub, int64_t N,
                                                        float* __restrict__ m,
                                                        float* __restrict__ s, int first, int last,
                                                        const float* __restrict__ yt,
                                                        float* __restrict__ loss,
                                                        float* __restrict__ lse) {
  constexpr int U = W == 1 ? 1 : 2;
  __shared__ float2 blk[W == 1 ? 1 : 64 * U * W];  // a block's pair each
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, wv = wave % W;
  const int64_t n = static_cast<int64_t>(blockIdx.x) * (4 / W) + wave / W;
  if (n >= N) return;  // W = 4: the whole workgroup
  const int nsub = 64 / sub, li = lane & (sub - 1), sl = lane / sub;
  const int nb = U * W * nsub;  // blocks at a time
  const float2* row = part + n * ng;
  float rm = 0.0f, rs = 0.0f;
  if (!first) {
    rm = m[n];
    rs = s[n];
  }
  for (int g0 = 0; g0 < ng; g0 += nb * per) {
    float tm[U], ts[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      tm[u] = -__builtin_huge_valf();
      ts[u] = 0.0f;
      const int b = g0 + ((u * W + wv) * nsub + sl) * per, e = b + per < ng ? b + per : ng;
      for (int c = b + li; c < e; c += sub) {
        const float2 p = row[c];
        lse_merge(tm[u], ts[u], p.x, p.y);
      }
    }
    for (int o = 1; o < sub; o <<= 1) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const float m2 = __shfl_xor(tm[u], o, 64), s2 = __shfl_xor(ts[u], o, 64);
        // both lanes of a pair compute the same merge in the same operand order
        float a = lane & o ? m2 : tm[u], b = lane & o ? s2 : ts[u];
        lse_merge(a, b, lane & o ? tm[u] : m2, lane & o ? ts[u] : s2);
        tm[u] = a;
        ts[u] = b;
      }
    }
    if constexpr (W == 1) {
      for (int q = 0; q < nsub && g0 + q * per < ng; ++q) {
        const float pm = __shfl(tm[0], q * sub, 64), ps = __shfl(ts[0], q * sub, 64);
        if (first && g0 == 0 && q == 0) {
          rm = pm;
          rs = ps;
        } else {
          lse_merge(rm, rs, pm, ps);
        }
      }
    } else {
      if (li == 0) {
#pragma unroll
        for (int u = 0; u < U; ++u) blk[(u * W + wv) * nsub + sl] = make_float2(tm[u], ts[u]);
      }
      __syncthreads();
      for (int q = 0; q < nb && g0 + q * per < ng; ++q) {
        const float2 p = blk[q];
        if (first && g0 == 0 && q == 0) {
          rm = p.x;
          rs = p.y;
        } else {
          lse_merge(rm, rs, p.x, p.y);
        }
      }
      __syncthreads();
    }
  }
  if (lane == 0 && wv == 0) {
    if (last) {
      const float l = rm + logf(rs);
      lse[n] = l;
      loss[n] = yt[n] - l;
    } else {
      m[n] = rm;
      s[n] = rs;
    }
  }
}

// dx[i] = bf16(sum over slabs b ascending of dxa[b][i]), 8 values per thread
__global__ __launch_bounds__(256) void voc_dx_sum_kernel(const float* __restrict__ dxa, int slabs,
                                                         int64_t n, uint16_t* __restrict__ dx) {
  const int64_t i = (static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x) * 8;
  if (i >= n) return;  // n = N H is a multiple of 8
  float v[8];
  {
    const float4 a = *reinterpret_cast<const float4*>(dxa + i);
    const float4 b = *reinterpret_cast<const float4*>(dxa + i + 4);
    v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w; v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
  }
  for (int sl = 1; sl < slabs; ++sl) {
    const float* p = dxa + static_cast<int64_t>(sl) * n + i;
    const float4 a = *reinterpret_cast<const float4*>(p);
    const float4 b = *reinterpret_cast<const float4*>(p + 4);
    v[0] += a.x; v[1] += a.y; v[2] += a.z; v[3] += a.w; v[4] += b.x; v[5] += b.y; v[6] += b.z;
    v[7] += b.w;
  }
  *reinterpret_cast<uint4*>(dx + i) = make_uint4(pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]),
                                                 pack_bf16x2(v[4], v[5]), pack_bf16x2(v[6], v[7]));
}

// wst[h][c] = c < vb ? w[h][v0 + c] : 0 for c < vbp (padded copy of a block),
// eight columns a thread
__global__ __launch_bounds__(256) void voc_stage_kernel(const uint16_t* __restrict__ w, int64_t V,
                                                        int64_t v0, int vb, int vbp, int H,
                                                        uint16_t* __restrict__ wst) {
  const int64_t i = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
  const int per = vbp / 8;
  if (i >= static_cast<int64_t>(H) * per) return;
  const int64_t h = i / per;
  const int c = static_cast<int>(i - h * per) * 8;
  const uint16_t* src = w + h * V + v0 + c;
  uint32_t p[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const uint32_t lo = c + 2 * q < vb ? src[2 * q] : 0u;
    const uint32_t hi = c + 2 * q + 1 < vb ? src[2 * q + 1] : 0u;
    p[q] = lo | (hi << 16);
  }
  *reinterpret_cast<uint4*>(wst + i * 8) = make_uint4(p[0], p[1], p[2], p[3]);
}

hipError_t stage(const uint16_t* w, int64_t V, int64_t v0, int vb, int vbp, int H, uint16_t* wst,
                 hipStream_t s) {
  const int64_t n = static_cast<int64_t>(H) * (vbp / 8);
  voc_stage_kernel<<<static_cast<unsigned>(ceil_div(n, 256)), 256, 0, s>>>(w, V, v0, vb, vbp, H, wst);
  return hipGetLastError();
}

__global__ __launch_bounds__(256) void voc_zero_bf16_kernel(uint16_t* __restrict__ p, int64_t n) {
  const int64_t i = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
  if (i < n) p[i] = 0;
}

// The products address a tile's rows of an operand by 32-bit offsets from the
// first, within the 2^31 - 16 bytes of a buffer descriptor: true if `rows`
// rows of `pitch` elements, the last read up to element `tail`, fit.  Rows per
// operand: 32 (one half step) where the contraction index runs over rows (W in
// the logits, G in dW), 256 (a tile) where it runs along them (G and W in dX).
constexpr int64_t REACH = 0x7ffffff0;
bool reach(int64_t rows, int64_t pitch, int64_t tail) {
  return 2 * ((rows - 1) * pitch + tail) <= REACH;
}
// the longest pitch (a multiple of 64) whose `rows` rows fit
int64_t max_pitch(int64_t rows) { return REACH / (2 * rows) / 64 * 64; }

// W read through a padded copy of a block?
bool staged_fwd(int H, int64_t V) {
  return (V % 8) != 0 || !reach(std::min(H, 32), V, 128);
}
bool staged_bwd(int H, int64_t V, int64_t vb) {
  return staged_fwd(H, V) || !reach(std::min(H, 256), V, std::min(vb, V));
}
// The caller's block, cut where the copy (forward) or G and the copy
// (backward) would have rows out of reach.
int64_t fwd_block(int H, int64_t V, int64_t vblock) {
  const int64_t most = max_pitch(std::min(H, 32));
  return staged_fwd(H, V) && std::min(vblock, V) > most ? most : vblock;
}
// The block that the forward walks: the caller's, less what is beyond a whole
// number of groups of 64 columns.  A block that ended inside a group could not
// be part of a longer product (its columns would fall into other groups, and
// the pairs be other sums), and had to be a launch of its own: N = 500, H =
// 520, V = 32000 in blocks of 1000 took 458 us in 32 launches, 35 in one.
int64_t fwd_step(int H, int64_t V, int64_t vblock) {
  const int64_t b = fwd_block(H, V, vblock);
  return b < V && b > 64 ? b / 64 * 64 : b;
}
int64_t bwd_block(int64_t N, int H, int64_t V, int64_t vblock) {
  const int64_t rows = std::max<int64_t>(N, staged_bwd(H, V, vblock) ? H : 1);
  const int64_t most = max_pitch(std::min<int64_t>(rows, 256));
  return std::min(vblock, V) > most ? most : vblock;
}

// K ranges of the dX product: enough (row tile x column tile x range) work
// items for about two per compute unit of a 256-CU device, each range at
// least 512 columns (a multiple of 64)
int64_t dx_kspan(int64_t N, int H, int64_t vblock) {
  const int64_t tiles = std::max<int64_t>(1, ceil_div(N, 256) * ceil_div(H, 256));
  int64_t S = std::min<int64_t>(8, std::max<int64_t>(1, ceil_div(512, tiles)));
  S = std::max<int64_t>(1, std::min<int64_t>(S, vblock / 512));
  return align_up(static_cast<size_t>(ceil_div(vblock, S)), 64);
}

}  // namespace

namespace {
size_t fwd_bytes(int64_t N, int H, int64_t V, int64_t span);
// Columns the forward takes at once: the largest multiple of vblock whose
// partial pairs (and staged copy of W) fit the workspace that
// moe_vocab_loss_workspace_bytes() asks for, which the backward's buffers
// set.  One product of many tiles instead of one per block: fewer launches
// and partly filled last rounds (N = 1000, H = 520, V = 32003 in blocks of
// 4096: 8 products and merges become 2; N = 4096, H = 2048, V = 200000: 13
// become 1).  Blocks of fewer than 64 columns stay alone.  A copy of W stays
// within reach and one launch (2^31 threads of eight columns).
int64_t fwd_span(int64_t N, int H, int64_t V, int64_t vblock) {
  const size_t room = std::max(vocab_fwd_ws_bytes(N, H, V, vblock), vocab_bwd_ws_bytes(N, H, V, vblock));
  vblock = fwd_step(H, V, vblock);
  if (vblock % 64 != 0) return vblock;
  int64_t most = std::min<int64_t>(ceil_div(V, vblock), ((int64_t{1} << 40) - 1) / (N * vblock));
  if (staged_fwd(H, V))
    most = std::min(most, std::min(max_pitch(std::min(H, 32)), (int64_t{1} << 34) / H) / vblock);
  int64_t lo = 1, hi = std::max<int64_t>(1, most);  // the largest m in [lo, hi] that fits
  while (lo < hi) {
    const int64_t mid = (lo + hi + 1) / 2;
    if (fwd_bytes(N, H, V, mid * vblock) <= room) lo = mid; else hi = mid - 1;
  }
  return lo * vblock;
}
}  // namespace

size_t vocab_fwd_ws_bytes(int64_t N, int H, int64_t V, int64_t vblock) {
  return fwd_bytes(N, H, V, fwd_block(H, V, vblock));
}

namespace {
size_t fwd_bytes(int64_t N, int H, int64_t V, int64_t span) {
  const int64_t vb = std::min(span, V);
  size_t b = align_up(sizeof(float) * 2 * static_cast<size_t>(N) * ceil_div(vb, 64), 256);  // pairs
  b += 3 * align_up(sizeof(float) * static_cast<size_t>(N), 256);  // running max, sum; target logit
  if (staged_fwd(H, V))
    b += align_up(sizeof(uint16_t) * static_cast<size_t>(H) * align_up(vb, 8), 256);
  return b + 256;
}
}  // namespace

size_t vocab_bwd_ws_bytes(int64_t N, int H, int64_t V, int64_t vblock) {
  vblock = bwd_block(N, H, V, vblock);
  const int64_t vb = std::min(vblock, V);
  const int64_t vbp = align_up(vb, 8);
  const int64_t slabs = ceil_div(vb, dx_kspan(N, H, vblock));
  size_t b = align_up(sizeof(uint16_t) * static_cast<size_t>(N) * vbp, 256);            // G
  b += align_up(sizeof(float) * static_cast<size_t>(slabs) * N * H, 256);                // dX slabs
  if (staged_bwd(H, V, vblock))
    b += align_up(sizeof(uint16_t) * static_cast<size_t>(H) * vbp, 256);  // W
  return b + 256;
}

hipError_t launch_vocab_fwd(const uint16_t* x, const uint16_t* w, const int32_t* target,
                            int64_t N, int H, int64_t V, int64_t vblock, float* loss, float* lse,
                            void* ws, size_t ws_bytes, hipStream_t s) {
  if (N == 0) return hipSuccess;
  // a caller with room for the forward alone gets its blocks one by one
  const int64_t span = ws_bytes >= vocab_bwd_ws_bytes(N, H, V, vblock) ? fwd_span(N, H, V, vblock)
                                                                         : fwd_step(H, V, vblock);
  const int64_t vbmax = std::min(span, V);
  // groups of 64 columns per block
  const int per = static_cast<int>(ceil_div(std::min(fwd_step(H, V, vblock), V), 64));
  int sub = 1;
  while (sub < 64 && sub < per) sub *= 2;
  char* p = static_cast<char*>(ws);
  float* part = reinterpret_cast<float*>(p);
  p += align_up(sizeof(float) * 2 * static_cast<size_t>(N) * ceil_div(vbmax, 64), 256);
  float* m = reinterpret_cast<float*>(p);
  p += align_up(sizeof(float) * static_cast<size_t>(N), 256);
  float* sm = reinterpret_cast<float*>(p);
  p += align_up(sizeof(float) * static_cast<size_t>(N), 256);
  float* yt = reinterpret_cast<float*>(p);
  p += align_up(sizeof(float) * static_cast<size_t>(N), 256);
  uint16_t* wst = staged_fwd(H, V) ? reinterpret_cast<uint16_t*>(p) : nullptr;
  const int n = static_cast<int>(N);
  for (int64_t b0 = 0; b0 < V; b0 += span) {
    const int vb = static_cast<int>(std::min<int64_t>(span, V - b0));
    const uint16_t* wb = w;
    int64_t ldw = V, bc0 = b0;
    if (wst != nullptr) {
      const int vbp = static_cast<int>(align_up(vb, 8));
      if (hipError_t e = stage(w, V, b0, vb, vbp, H, wst, s); e != hipSuccess) return e;
      wb = wst;
      ldw = vbp;
      bc0 = 0;
    }
    if (hipError_t e = launch_vocab_logits_mfma(x, wb, ldw, bc0, b0, n, H, vb, target, part, yt, s);
        e != hipSuccess)
      return e;
    prof_begin(K_VOC_LSE, s);
    const int ng = static_cast<int>(ceil_div(vb, 64));
    const float2* pairs = reinterpret_cast<const float2*>(part);
    const int first = b0 == 0, last = b0 + span >= V;
    const int64_t rounds = ceil_div(ceil_div(ng, per), 64 / sub);  // of one wave a row
    if (rounds <= (sub < 64 ? 4 : 1) || N > (int64_t{1} << 23))  // or rows enough
      voc_merge_kernel<1><<<static_cast<unsigned>(ceil_div(N, 4)), 256, 0, s>>>(
          pairs, ng, per, sub, N, m, sm, first, last, yt, loss, lse);
    else
      voc_merge_kernel<4><<<static_cast<unsigned>(N), 256, 0, s>>>(pairs, ng, per, sub, N, m, sm,
                                                                   first, last, yt, loss, lse);
    prof_end(K_VOC_LSE, s);
    if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t launch_vocab_bwd(const uint16_t* x, const uint16_t* w, const int32_t* target,
                            const float* lse, const float* dloss, int64_t N, int H, int64_t V,
                            int64_t vblock, uint16_t* dx, uint16_t* dw, void* ws, hipStream_t s) {
  if (N == 0) {  // no tokens: the weight gradient is exact zeros (dx is empty)
    const int64_t nw = static_cast<int64_t>(H) * V;
    voc_zero_bf16_kernel<<<static_cast<unsigned>(ceil_div(nw, 256)), 256, 0, s>>>(dw, nw);
    return hipGetLastError();
  }
  vblock = bwd_block(N, H, V, vblock);
  const int64_t vbmax = std::min(vblock, V);
  const int64_t vbpmax = align_up(vbmax, 8);
  // a range longer than the block is the block (vblock itself may exceed an int)
  const int kspan = static_cast<int>(
      std::min<int64_t>(dx_kspan(N, H, vblock), static_cast<int64_t>(align_up(vbmax, 64))));
  const int slabs = static_cast<int>(ceil_div(vbmax, kspan));  // the first block fills them all
  char* p = static_cast<char*>(ws);
  uint16_t* G = reinterpret_cast<uint16_t*>(p);
  p += align_up(sizeof(uint16_t) * static_cast<size_t>(N) * vbpmax, 256);
  float* dxa = reinterpret_cast<float*>(p);
  p += align_up(sizeof(float) * static_cast<size_t>(slabs) * N * H, 256);
  uint16_t* wst = staged_bwd(H, V, vblock) ? reinterpret_cast<uint16_t*>(p) : nullptr;
  const int n = static_cast<int>(N);
  for (int64_t b0 = 0; b0 < V; b0 += vblock) {
    const int vb = static_cast<int>(std::min<int64_t>(vblock, V - b0));
    const int64_t gp = align_up(vb, 8);
    const uint16_t* wb = w;
    int64_t ldw = V, bc0 = b0;
    if (wst != nullptr) {
      if (hipError_t e = stage(w, V, b0, vb, static_cast<int>(gp), H, wst, s); e != hipSuccess)
        return e;
      wb = wst;
      ldw = gp;
      bc0 = 0;
    }
    if (hipError_t e = launch_vocab_grad_mfma(x, wb, ldw, bc0, b0, n, H, vb, target, lse, dloss, G,
                                              gp, s);
        e != hipSuccess)
      return e;
    if (hipError_t e = launch_vocab_dx_mfma(G, gp, wb, ldw, bc0, n, H, vb, kspan, b0 == 0, dxa, s);
        e != hipSuccess)
      return e;
    if (hipError_t e = launch_vocab_dw_mfma(x, G, gp, n, H, vb, dw, V, b0, s); e != hipSuccess)
      return e;
  }
  const int64_t nx = N * H;
  voc_dx_sum_kernel<<<static_cast<unsigned>(ceil_div(nx / 8, 256)), 256, 0, s>>>(dxa, slabs, nx, dx);
  return hipGetLastError();
}

}  // namespace moe
