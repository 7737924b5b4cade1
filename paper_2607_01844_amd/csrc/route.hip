// Router of the MoE layer on gfx950: logits and top-k softmax gates.
//
// Logits follow one fixed fp32 order (a fused-multiply-add chain over the
// hidden index ascending from +0.0f, then one add of the bias) so that the
// expert choice is reproducible bit for bit.  The fp32 matrix instruction
// keeps that order: v_mfma_f32_16x16x4_f32 adds its four products to the
// accumulator one after another in ascending k, each as a fused multiply-add
// rounded to nearest even, denormals, infinities and zeros included (checked
// bit for bit against fmaf chains, and by the routing tests against the
// oracle's).  So the hidden index runs through the matrix cores, at twice the
// vector ALUs' fp32 rate without packed instructions; it is never split
// between accumulators.
#include "common.h"

namespace moe {
namespace {

typedef int i32x4r __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) char lds_byte;

#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
// 16 bytes per lane, global -> LDS (lane i writes LDS [lds + 16 i, +16));
// completion is tracked by hand with vmcnt.
__device__ __forceinline__ void w_load_lds16(const i32x4r& rsrc, uint32_t voff, uint32_t lds) {
  asm volatile("s_mov_b32 m0, %0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds"
               :
               : "s"(lds), "v"(voff), "s"(rsrc)
               : "memory", "m0");
}
// 4 bytes per lane (lane i writes LDS [lds + 4 i, +4))
__device__ __forceinline__ void w_load_lds4(const i32x4r& rsrc, uint32_t voff, uint32_t lds) {
  asm volatile("s_mov_b32 m0, %0\n\tbuffer_load_dword %1, %2, 0 offen lds"
               :
               : "s"(lds), "v"(voff), "s"(rsrc)
               : "memory", "m0");
}
#pragma clang diagnostic pop
template <int N>
__device__ __forceinline__ void wait_vm() {
  asm volatile("s_waitcnt vmcnt(%0)" : : "n"(N) : "memory");
}

// Bound by the fp32 matrix cores where the tiles fill the chip (T = 65536, d =
// 4096, E = 128: 624 us = 110 TFLOP/s of 157; the vector-ALU chains it replaces
// took 1365 us; T = 16384, d = 7168, E = 384: 1538 -> 811 us, and 900 on
// average among a layer's other kernels), by one wave's chain of d / 4
// dependent instructions where they do not (T = 1000, d = 4096, E = 128: 95 ->
// 33 us; T = 16, d = 2048, E = 64: 36 -> 18 us).
// Block = GT x GE waves, each WT x WE tiles of 16 tokens x 16 experts (one
// v_mfma_f32_16x16x4_f32 accumulator each: A = x, lane l row l % 16 and
// k = l / 16; B = W_r, lane l column l % 16 and k = l / 16).  Chunks of KC
// hidden indices move to LDS with direct-to-LDS loads, DEPTH chunks deep: the
// block's token rows [TB][KC] bf16 and the weights [KC][EB] fp32 (columns
// past E and rows past d as zeros; neither reaches a stored logit).  Both
// images carry an XOR swizzle on the loading side that spreads a fragment
// read over all 64 banks: x rows of KC / 8 16-byte chunks, chunk c of row r
// at c ^ (r / (16 / CPR)) % CPR; weight rows in groups of 16 columns, group
// g of row k at g ^ k % 4 (fewer than four groups: EB = 32 at g ^ (k / 2) % 2,
// EB = 16 in place).  VEC = 4 loads weights 16 bytes at a time (E a multiple
// of 4, so that no piece crosses a row's end), VEC = 1 four.
template <int WT, int WE, int GT, int GE, int KC, int DEPTH, int VEC>
__global__ __launch_bounds__(64 * GT * GE) void route_logits_kernel(
    const uint16_t* __restrict__ x, const float* __restrict__ w, const float* __restrict__ bias,
    int64_t T, int d, int E, float* __restrict__ logits) {
  constexpr int NW = GT * GE;
  constexpr int TB = 16 * WT * GT, EB = 16 * WE * GE;
  constexpr int XCH = TB * KC * 2, WCH = KC * EB * 4, CHUNK = XCH + WCH;  // bytes per chunk
  constexpr int LX = XCH / 1024 / NW, LW = WCH / (256 * VEC) / NW;        // loads per wave
  // chunks in the ring: DEPTH, fewer where the loads in flight would exceed
  // the vector-memory counter
  constexpr int NBUF = DEPTH < 2 + 63 / (LX + LW) ? DEPTH : 2 + 63 / (LX + LW);
  constexpr int CPR = KC / 8;                    // 16-byte chunks per x row
  constexpr int RP = CPR >= 16 ? 1 : 16 / CPR;   // x rows per 256 bytes
  static_assert(XCH % (1024 * NW) == 0 && WCH % (256 * VEC * NW) == 0 && NBUF * CHUNK <= 160 * 1024,
                "chunk shape");
  __shared__ __align__(1024) char ws[NBUF * CHUNK];
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l16 = lane & 15, q = lane >> 4;
  const int64_t t0 = static_cast<int64_t>(blockIdx.x) * TB;
  const int e0 = blockIdx.y * EB;
  const int tw = (wv / GE) * 16 * WT, ew = (wv % GE) * 16 * WE;  // the wave's tokens, experts

  auto rsrc = [](const void* p, int64_t bytes) {
    const uint64_t addr = reinterpret_cast<uint64_t>(p);
    i32x4r r;
    r[0] = __builtin_amdgcn_readfirstlane(static_cast<int>(addr & 0xffffffffu));
    r[1] = __builtin_amdgcn_readfirstlane(static_cast<int>((addr >> 32) & 0xffffu));
    r[2] = static_cast<int>(bytes > 0x7ffffff0 ? 0x7ffffff0 : (bytes < 0 ? 0 : bytes));
    r[3] = 0x00020000;
    return r;
  };
  const i32x4r rw = rsrc(w, static_cast<int64_t>(d) * E * 4);
  const i32x4r rx = rsrc(x + t0 * d, (T - t0) * d * 2);
  constexpr uint32_t OOB = 0x80000000u;  // past every range: reads as zero
  auto wswz = [](int k) { return EB >= 64 ? (k & 3) : EB == 32 ? ((k >> 1) & 1) : 0; };
  const uint32_t lds0 = static_cast<uint32_t>(reinterpret_cast<uintptr_t>((const lds_byte*)(ws)));
  // lane offsets of the next chunk's loads.  x columns past d (the next
  // row's values) and zero rows past T land where no batch or store reaches;
  // weight rows past d lie past the buffer's range.
  uint32_t xoff[LX], woff[LW];
#pragma unroll
  for (int i = 0; i < LX; ++i) {
    const int p = (wv * LX + i) * 64 + lane;  // 16-byte piece of the image
    const int r = p / CPR, ch = (p % CPR) ^ ((r / RP) % CPR);
    xoff[i] = static_cast<uint32_t>((r * d + ch * 8) * 2);
  }
#pragma unroll
  for (int i = 0; i < LW; ++i) {
    const int p = ((wv * LW + i) * 64 + lane) * VEC;  // first float of the piece
    const int k = p / EB, pos = p % EB;
    const int e = e0 + (((pos >> 4) ^ wswz(k)) << 4) + (pos & 15);
    woff[i] = e < E ? (static_cast<uint32_t>(k) * E + e) * 4u : OOB;
  }
  uint32_t slot = 0;  // ring position of the next chunk to load
  auto issue_chunk = [&]() __attribute__((always_inline)) {
    const uint32_t dst = lds0 + slot;
#pragma unroll
    for (int i = 0; i < LX; ++i) {
      w_load_lds16(rx, xoff[i], dst + (wv * LX + i) * 1024);
      xoff[i] += KC * 2;
    }
#pragma unroll
    for (int i = 0; i < LW; ++i) {
      const uint32_t to = dst + XCH + (wv * LW + i) * 256 * VEC;
      if constexpr (VEC == 4) w_load_lds16(rw, woff[i], to);
      else w_load_lds4(rw, woff[i], to);
      woff[i] += static_cast<uint32_t>(KC * 4) * E;
    }
    slot = slot == (NBUF - 1) * CHUNK ? 0 : slot + CHUNK;
  };

  f32x4 acc[WT][WE];
#pragma unroll
  for (int a = 0; a < WT; ++a)
#pragma unroll
    for (int b = 0; b < WE; ++b) acc[a][b] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  // the bf16 value q of four (in two words) as fp32 bits: one byte permute
  const uint32_t sel = 0x01000c0cu + 0x02020000u * q;
  // eight hidden indices (a batch) of one chunk: their fragments, and two
  // matrix instructions per tile, k ascending.  Fragments are read AHEAD
  // batches early, since the compiler keeps them close to their use (T = 8192,
  // d = 4096, E = 128: 100 -> 94 us; T = 1000: 46 -> 43).
  constexpr int AHEAD = WT * WE == 1 ? 3 : 1;
  struct Frags {
    uint4 x[WT];
    float w[2][WE];
  };
  Frags fr[AHEAD + 1];
  auto read = [&](Frags& f, const char* cb, int bl) __attribute__((always_inline)) {
#pragma unroll
    for (int a = 0; a < WT; ++a) {
      const int r = tw + 16 * a + l16;
      f.x[a] = *reinterpret_cast<const uint4*>(cb + r * (KC * 2) + ((bl ^ ((r / RP) % CPR)) << 4));
    }
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int k = 8 * bl + 4 * h + q;
      const float* row = reinterpret_cast<const float*>(cb + XCH) + k * EB + l16;
#pragma unroll
      for (int b = 0; b < WE; ++b) f.w[h][b] = row[((ew >> 4) + b ^ wswz(k)) << 4];
    }
  };
  auto mma = [&](const Frags& f) __attribute__((always_inline)) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
#pragma unroll
      for (int a = 0; a < WT; ++a) {
        const float av = __uint_as_float(h ? __builtin_amdgcn_perm(f.x[a].w, f.x[a].z, sel)
                                           : __builtin_amdgcn_perm(f.x[a].y, f.x[a].x, sel));
#pragma unroll
        for (int b = 0; b < WE; ++b)
          acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x4f32(av, f.w[h][b], acc[a][b], 0, 0, 0);
      }
    }
  };
  const int nch = (d + KC - 1) / KC;
#pragma unroll
  for (int c = 0; c < NBUF - 1; ++c) issue_chunk();
  uint32_t rd = 0;  // ring position of the chunk being computed
  for (int c = 0; c < nch; ++c) {
    wait_vm<(LX + LW) * (NBUF - 2)>();  // this wave's part of chunk c has landed
    __syncthreads();                    // everyone's part; chunk c - 1 is consumed
    issue_chunk();                      // chunk c + NBUF - 1, into chunk c - 1's buffer
    const char* cb = ws + rd;
    rd = rd == (NBUF - 1) * CHUNK ? 0 : rd + CHUNK;
    const int nbl = min(KC, d - c * KC) / 8;  // batches in this chunk (d is a multiple of 8)
    if (nbl == KC / 8) {
      constexpr int NB = KC / 8;
      static_for<AHEAD>([&](auto B) { read(fr[B], cb, B); });
      static_for<NB>([&](auto B) {
        constexpr int bl = B;
        if constexpr (bl + AHEAD < NB) read(fr[(bl + AHEAD) % (AHEAD + 1)], cb, bl + AHEAD);
        __builtin_amdgcn_sched_barrier(0);  // the reads stay ahead of the products
        mma(fr[bl % (AHEAD + 1)]);
      });
    } else {
      for (int bl = 0; bl < nbl; ++bl) {
        read(fr[0], cb, bl);
        mma(fr[0]);
      }
    }
  }
  wait_vm<0>();  // the trailing chunks' loads are done before the block ends
  // accumulator word r of lane l: token 4 q + r, expert l16 of the tile
#pragma unroll
  for (int b = 0; b < WE; ++b) {
    const int e = e0 + ew + 16 * b + l16;
    if (e >= E) continue;
    const float be = bias ? bias[e] : 0.0f;
#pragma unroll
    for (int a = 0; a < WT; ++a) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int64_t t = t0 + tw + 16 * a + 4 * q + r;
        if (t < T) logits[t * E + e] = bias ? acc[a][b][r] + be : acc[a][b][r];
      }
    }
  }
}

// Largest of 64 lanes' unsigned values, in every lane: row shifts and
// broadcasts in the vector ALUs (no LDS permutes).
__device__ __forceinline__ uint32_t wave_max_u32(uint32_t v) {
#define ROUTE_DPP_MAX(ctrl, rows) \
  v = max(v, static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(v), ctrl, rows, 0xf, false)))
  ROUTE_DPP_MAX(0x111, 0xf);  // row_shr:1
  ROUTE_DPP_MAX(0x112, 0xf);  // row_shr:2
  ROUTE_DPP_MAX(0x114, 0xf);  // row_shr:4
  ROUTE_DPP_MAX(0x118, 0xf);  // row_shr:8: lane 15 of each row of 16 has the row's
  ROUTE_DPP_MAX(0x142, 0xa);  // row_bcast:15 into rows 1 and 3
  ROUTE_DPP_MAX(0x143, 0xc);  // row_bcast:31 into rows 2 and 3: lane 63 has the wave's
#undef ROUTE_DPP_MAX
  return static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(v), 63));
}

// One wave per token: k rounds of a wave-wide arg-max over the not yet
// chosen experts, ordered by (logit descending, index ascending).  Lane i
// keeps slot i.  Gates: softmax over all E (renorm = 0) or over the chosen k.
// A NaN logit ranks as -inf, so every round picks a valid expert (the
// lowest free index when all free logits are -inf or NaN); gates of such a
// token are unspecified.
//   A logit's key is its bits in an order-preserving unsigned form (-0 as
// +0); a taken or missing expert has key 0, below -inf's.  A round is the
// wave's largest key and, of the lanes that hold it, the first, slot by slot
// (expert = lane + 64 slot).  Reducing (value, index) pairs with LDS permutes
// instead took 82 us at T = 65536, E = 128, k = 8.
template <int NV>
__global__ __launch_bounds__(256) void route_topk_kernel(const float* __restrict__ logits,
                                                         int64_t T, int E, int k, int renorm,
                                                         int32_t* __restrict__ idx,
                                                         float* __restrict__ gate) {
  const int lane = threadIdx.x & 63;
  const int64_t t = static_cast<int64_t>(blockIdx.x) * 4 + (threadIdx.x >> 6);
  if (t >= T) return;
  const float* l = logits + t * E;
  float v[NV];
  uint32_t key[NV];
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    const int e = lane + 64 * i;
    v[i] = -__builtin_huge_valf();
    key[i] = 0u;
    if (e < E) {
      const float le = l[e];
      v[i] = le != le ? -__builtin_huge_valf() : le;
      const uint32_t u = v[i] == 0.0f ? 0u : __float_as_uint(v[i]);
      key[i] = u ^ (static_cast<uint32_t>(static_cast<int32_t>(u) >> 31) | 0x80000000u);
    }
  }
  float my_v = 0.0f, m = 0.0f;
  int my_e = 0;
  for (int s = 0; s < k; ++s) {
    uint32_t best = key[0];
#pragma unroll
    for (int i = 1; i < NV; ++i) best = max(best, key[i]);
    best = wave_max_u32(best);
    int be = 0;
    bool found = false;
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      const uint64_t has = __ballot(key[i] == best);
      if (!found && has != 0ull) {
        found = true;
        const int first = __builtin_ctzll(has);
        be = 64 * i + first;
        if (lane == first) key[i] = 0u;
      }
    }
    const float bv = __uint_as_float(best ^ (best >> 31 ? 0x80000000u : 0xffffffffu));
    if (s == 0) m = bv;
    if (lane == s) {
      my_v = bv;
      my_e = be;
    }
  }
  float part = 0.0f;
  if (renorm == 0) {
#pragma unroll
    for (int i = 0; i < NV; ++i)
      if (lane + 64 * i < E) part += expf(v[i] - m);
  } else if (lane < k) {
    part = expf(my_v - m);
  }
  const float den = wave_sum(part);
  if (lane < k) {
    idx[t * k + lane] = my_e;
    gate[t * k + lane] = expf(my_v - m) / den;
  }
}

template <int WT, int WE, int GT, int GE, int KC, int DEPTH>
hipError_t run_logits(const uint16_t* x, const float* w, const float* bias, int64_t T, int d,
                      int E, float* logits, hipStream_t s) {
  const dim3 grid(static_cast<unsigned>(ceil_div(T, 16 * WT * GT)),
                  static_cast<unsigned>(ceil_div(E, 16 * WE * GE)));
  prof_begin(K_ROUTE_LOGITS, s);
  if ((E & 3) == 0)
    route_logits_kernel<WT, WE, GT, GE, KC, DEPTH, 4><<<grid, 64 * GT * GE, 0, s>>>(x, w, bias, T, d,
                                                                                  E, logits);
  else
    route_logits_kernel<WT, WE, GT, GE, KC, DEPTH, 1><<<grid, 64 * GT * GE, 0, s>>>(x, w, bias, T, d,
                                                                                  E, logits);
  prof_end(K_ROUTE_LOGITS, s);
  return hipGetLastError();
}

// Tile by size: the largest block tile that still gives every CU two blocks
// and whose last column of blocks is not mostly padding.  Larger tiles read
// less through the L2 per product (128 x 128: 3 bytes per matrix-core cycle
// and CU, 32 x 32: 24), smaller ones fill the chip (logits and top-k
// together: at T = 8192, d = 4096, E = 128 blocks of 32 x 64 take 94 us,
// 64 x 64 103, 128 x 128 326; at T = 65536 128 x 128 takes 639 us, 32 x 64
// 708).  Below that 32 x 32 blocks of four waves as soon as more than half of
// the CUs get one (T = 4096, d = 2048, E = 64: 28 us against 45), then blocks
// of one wave and one 16 x 16 tile, which spread the weights that a few
// tokens read over the most CUs (T = 16: 23 us against 25).
hipError_t pick_logits(const uint16_t* x, const float* w, const float* bias, int64_t T, int d,
                       int E, float* logits, hipStream_t s) {
  const int64_t cus = device_cus();
  auto blocks = [&](int tb, int eb) -> int64_t {
    const int64_t et = ceil_div(E, eb);
    if (et * eb * 4 > 5 * static_cast<int64_t>(align_up(E, 16))) return 0;
    return ceil_div(T, tb) * et;
  };
  if (blocks(128, 128) >= 2 * cus)
    return run_logits<4, 4, 2, 2, 32, 3>(x, w, bias, T, d, E, logits, s);
  if (blocks(64, 128) >= 2 * cus)
    return run_logits<2, 4, 2, 2, 32, 4>(x, w, bias, T, d, E, logits, s);
  if (blocks(64, 64) >= 2 * cus)
    return run_logits<2, 2, 2, 2, 64, 3>(x, w, bias, T, d, E, logits, s);
  if (blocks(32, 64) >= 2 * cus)
    return run_logits<1, 2, 2, 2, 64, 4>(x, w, bias, T, d, E, logits, s);
  if (blocks(32, 32) * 2 > cus)
    return run_logits<1, 1, 2, 2, 64, 4>(x, w, bias, T, d, E, logits, s);
  return run_logits<1, 1, 1, 1, 128, 4>(x, w, bias, T, d, E, logits, s);
}

}  // namespace

hipError_t launch_route(const uint16_t* x, const float* w, const float* bias, int64_t T, int d,
                        int E, int k, int renorm, int32_t* idx, float* gate, float* logits,
                        hipStream_t s) {
  if (T == 0) return hipSuccess;
  if (hipError_t err = pick_logits(x, w, bias, T, d, E, logits, s); err != hipSuccess) return err;

  const unsigned grid = static_cast<unsigned>(ceil_div(T, 4));
  prof_begin(K_ROUTE_TOPK, s);
  if (E <= 64)
    route_topk_kernel<1><<<grid, 256, 0, s>>>(logits, T, E, k, renorm, idx, gate);
  else if (E <= 128)
    route_topk_kernel<2><<<grid, 256, 0, s>>>(logits, T, E, k, renorm, idx, gate);
  else if (E <= 256)
    route_topk_kernel<4><<<grid, 256, 0, s>>>(logits, T, E, k, renorm, idx, gate);
  else if (E <= 512)
    route_topk_kernel<8><<<grid, 256, 0, s>>>(logits, T, E, k, renorm, idx, gate);
  else
    route_topk_kernel<16><<<grid, 256, 0, s>>>(logits, T, E, k, renorm, idx, gate);
  prof_end(K_ROUTE_TOPK, s);
  return hipGetLastError();
}

}  // namespace moe
