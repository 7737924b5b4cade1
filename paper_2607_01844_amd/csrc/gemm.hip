// Grouped SwiGLU expert GEMMs and the dense products: the schedule kernel,
// the choice of the tile, and the launches.  The kernel is in gemm_kernel.h;
// this file holds its 256-row tile.
#include "gemm_kernel.h"

#include <algorithm>
#include <cmath>

namespace moe {
using namespace gemm;
namespace {

// Per-expert prefixes over experts in index order: tiles of up to `rows` rows
// (mt_start), K steps, or other tiles, of up to `krows` rows (wk_start) and
// experts with rows (nz_start).  One workgroup, E_loc <= 1024.
__global__ __launch_bounds__(1024) void gemm_sched_kernel(const int32_t* __restrict__ offsets,
                                                          int E_loc, int rows, int krows,
                                                          int32_t* __restrict__ mt_start,
                                                          int32_t* __restrict__ wk_start,
                                                          int32_t* __restrict__ nz_start) {
  __shared__ int wsum[3][16];
  const int e = threadIdx.x;
  const int n = (e < E_loc) ? offsets[e + 1] - offsets[e] : 0;
  const int v[3] = {(n + rows - 1) / rows, (n + krows - 1) / krows, n > 0 ? 1 : 0};
  int32_t* const out[3] = {mt_start, wk_start, nz_start};
  const int lane = e & 63, w = e >> 6;
  int incl[3] = {v[0], v[1], v[2]};
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      const int u = __shfl_up(incl[c], o, 64);
      if (lane >= o) incl[c] += u;
    }
  }
  if (lane == 63)
#pragma unroll
    for (int c = 0; c < 3; ++c) wsum[c][w] = incl[c];
  __syncthreads();
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    int base = 0;
    for (int q = 0; q < w; ++q) base += wsum[c][q];
    if (e < E_loc) out[c][e] = base + incl[c] - v[c];
    if (e == E_loc - 1) out[c][E_loc] = base + incl[c];
  }
}

struct GemmWs {
  int32_t* mt_start;
  int32_t* wk_start;
  int32_t* nz_start;
  uint16_t* act;
  uint16_t* dhg;
  uint16_t* dhu;
};

GemmWs carve(void* ws, int64_t cap, int E_loc, int f, bool bwd) {
  char* p = static_cast<char*>(ws);
  GemmWs w{};
  w.mt_start = reinterpret_cast<int32_t*>(p);
  p += align_up(sizeof(int32_t) * (E_loc + 1), 256);
  w.wk_start = reinterpret_cast<int32_t*>(p);
  p += align_up(sizeof(int32_t) * (E_loc + 1), 256);
  w.nz_start = reinterpret_cast<int32_t*>(p);
  p += align_up(sizeof(int32_t) * (E_loc + 1), 256);
  const size_t act_bytes = align_up(sizeof(uint16_t) * static_cast<size_t>(cap) * f, 256);
  w.act = reinterpret_cast<uint16_t*>(p);
  p += act_bytes;
  if (bwd) {
    w.dhg = reinterpret_cast<uint16_t*>(p);
    p += act_bytes;
    w.dhu = reinterpret_cast<uint16_t*>(p);
  }
  return w;
}

// Persistent grid: the workgroups the chip holds at once (a multiple of the 8
// XCDs).
int64_t pgrid(int wgs) {
  const int64_t g = (device_cus() / NXCD) * NXCD * wgs;
  return g > 0 ? g : NXCD;
}

template <int MODE>
hipError_t run_gemm(const GemmArgs& a, bool small, int kid, hipStream_t s) {
  prof_begin(kid, s);
  if (small)
    launch_small(MODE, static_cast<unsigned>(pgrid(Geom<TILE_S>::WGS)), a, s);
  else
    grouped_gemm_kernel<MODE, TILE><<<static_cast<unsigned>(pgrid(Geom<TILE>::WGS)),
                                      Geom<TILE>::NTHR, 0, s>>>(a);
  prof_end(kid, s);
  return hipGetLastError();
}

// The 128-row tile where 256-row tiles would use less than two thirds of the
// CUs over their rounds (a full chip runs the large tile about 1.5 times as
// fast, since it reads its operands half as often).  Both sides measured (whole
// passes, 256- against 128-row tiles): 12 experts of 275 rows, d = 520, f =
// 328 (75 tiles) 251 -> 191 us a training step; the vocabulary loss in blocks
// of 64 tiles 987 -> 610 us; and beyond the line the vocabulary loss in
// products of 512 tiles 12.2 -> 13.6 ms, mid's training step (1408 tiles) 1830
// -> 2164 us, its weight gradients alone 1830 -> 1964.  The row-grouped
// products count capacity, not rows: a bound that costs no wait, and above the
// real tile count where experts or rows are absent.
bool use_small(int64_t tiles) {
  const int64_t cus = device_cus();
  return 3 * tiles < 2 * cus * ceil_div(tiles, cus);
}
// The down product and the data gradients take it too at 16 rows per expert or
// fewer on average, where a product is its weights' stream and two workgroups a
// CU keep more of it in flight (64 experts of 8 rows, d = 2048, f = 1408: down
// 78 -> 70 us, data gradients 261 -> 201; beyond the line 128 experts of 62
// rows, d = 4096: 1043 -> 1194 us a forward).
bool few_rows(int64_t rows, int64_t experts) { return rows <= 16 * experts; }
// The weight gradients of few rows write far more than they read, in pieces
// half as long on the 128-row tile (the same 64 experts 306 us against 357, 128
// of 8 rows, d = 4096, f = 1536 1107 against 1420): a tile a quarter as large
// costs three eighths, which pays where 256-row tiles leave CUs idle (48
// experts, 96 rows in all, d = 264, f = 328, the backward 52 -> 44 us).  Of 341
// layers of few rows the down product is more than 4 % off its better tile in
// 16; by the two-thirds rule alone in 54.
bool small_weights(int64_t t256, int64_t t128) {
  const int64_t cus = device_cus();
  return use_small(t256) || 3 * ceil_div(t128, cus) < 8 * ceil_div(t256, cus);
}
// Upper bound of the row tiles of E_loc experts with up to cap rows in all.
int64_t row_tiles(int64_t cap, int E_loc) { return std::min<int64_t>(cap, E_loc) + cap / TILE; }

// That bound says nothing of a CU that gets two 128-row tiles and its neighbour
// one, or of tiles that do not exist: 16 experts of 139 rows, d = 2048, f =
// 1536 have 192 gate/up tiles, counted as 288 (73 us on them, 86 on 768 small
// ones); 12 of 75, d = 5120 141 against 167; 8 of 83, d = f = 4096 163 against
// 183.  And the gate/up product's weights lie along f: of few rows per expert,
// its 128-row tile reads them in pieces half as long, which pays where it fills
// idle CUs (256- against 128-row tiles: 8 experts of 12 rows, d = 7168, f = 72
// 86 us against 54, 24 of one row, d = 2560, f = 768 55 against 39) and costs
// where both fill the chip (128 of 8, d = 4096, f = 1536 585 against 690, 32 of
// 8, d = 7168, f = 2048 364 against 435).  So these products weigh what their
// busiest CU does, `rows` rows spread evenly over the experts that get
// any at random.  A tile costs a fixed part and, per K step, its operands' rows
// and columns: 1000 + steps (h + 256) for a 256-row tile of h rows; 500 a pair
// + 0.95 steps (h + 128) for a 128-row tile (a fit to 760 random layers, both
// tiles measured).
bool large_cheaper(int64_t rows, int64_t experts, int64_t n256, int64_t n128, int64_t K) {
  const int64_t cus = device_cus(), ks = ceil_div(K, BK);
  const double e = static_cast<double>(experts), m = static_cast<double>(rows);
  rows = std::max<int64_t>(1, rows);
  const int64_t any = static_cast<int64_t>(std::ceil(-e * std::expm1(-m / e)));
  const int64_t p = std::max<int64_t>(1, std::min(any, std::min(rows, experts)));
  const int64_t n = ceil_div(rows, p), m256 = ceil_div(n, TILE), m128 = ceil_div(n, TILE_S);
  auto height = [&](int64_t mt) { return 32 * std::max<int64_t>(2, ceil_div(n, 32 * mt)); };
  const int64_t t256 = p * m256 * n256, t128 = p * m128 * n128;
  return 20 * ceil_div(t256, cus) * (1000 + ks * (height(m256) + 256)) <
         20 * ceil_div(t128, 2 * cus) * 500 + 19 * ceil_div(t128, cus) * ks * (height(m128) + 128);
}
// The host knows the capacity alone, so the 256-row tile has to be the cheaper
// one at less as well: at a quarter and an eighth of the rows (one rank's share)
// or, of few rows, on half of the experts (a rank that holds those of its own).
// A product of fewer tiles than the capacity's would lose more on it (3 experts
// of 1051 rows of 4206, d = 760, f = 336, a forward 65 -> 89 us) than one of all
// of them gains.
bool keep_large(int64_t cap, int E_loc, int64_t n256, int64_t n128, int64_t K) {
  if (!large_cheaper(cap, E_loc, n256, n128, K)) return false;
  if (few_rows(cap, E_loc)) return large_cheaper(cap, ceil_div(E_loc, 2), n256, n128, K);
  return large_cheaper(cap / 4, E_loc, n256, n128, K) &&
         large_cheaper(cap / 8, E_loc, n256, n128, K);
}

hipError_t sched(const int32_t* offsets, int E_loc, int rows, int krows, const GemmWs& w,
                 hipStream_t s) {
  prof_begin(K_GEMM_SCHED, s);
  gemm_sched_kernel<<<1, 1024, 0, s>>>(offsets, E_loc, rows, krows, w.mt_start, w.wk_start,
                                       w.nz_start);
  prof_end(K_GEMM_SCHED, s);
  return hipGetLastError();
}

}  // namespace

size_t gemm_ws_bytes(int64_t cap, int E_loc, int d, int f, unsigned flags) {
  (void)d;
  const bool bwd = flags != 0;
  const size_t act_bytes = align_up(sizeof(uint16_t) * static_cast<size_t>(cap) * f, 256);
  return 3 * align_up(sizeof(int32_t) * (E_loc + 1), 256) + act_bytes * (bwd ? 3 : 1) + 256;
}

hipError_t launch_ffn_fwd(const uint16_t* x_perm, const int32_t* offsets, int E_loc, int64_t cap,
                          int d, int f, const uint16_t* wg, const uint16_t* wu,
                          const uint16_t* wd, uint16_t* hg, uint16_t* hu, uint16_t* y,
                          void* ws, hipStream_t s) {
  GemmWs w = carve(ws, cap, E_loc, f, false);
  const int64_t rt = row_tiles(cap, E_loc);
  const bool idle = use_small(rt * std::max(ceil_div(f, TILE / 2), ceil_div(d, TILE)));
  const bool few = few_rows(cap, E_loc);
  // gate/up, down
  const bool small = (idle || few) &&
                     !keep_large(cap, E_loc, ceil_div(f, TILE / 2), ceil_div(f, TILE_S / 2), d);
  const bool small_d =
      few || (idle && !keep_large(cap, E_loc, ceil_div(d, TILE), ceil_div(d, TILE_S), f));
  int32_t* mt_down = w.mt_start;
  if (small && small_d && E_loc <= REG_EXPERTS) {
    w.mt_start = mt_down = nullptr;  // the kernels form the tables
  } else {
    // no product of the forward counts K steps: their table holds the down
    // product's row tiles where these are other ones
    const bool both = small != small_d;
    if (both) mt_down = w.wk_start;
    if (hipError_t e = sched(offsets, E_loc, small ? TILE_S : TILE,
                             !both ? BK : small_d ? TILE_S : TILE, w, s);
        e != hipSuccess)
      return e;
  }
  GemmArgs a{};
  a.x_perm = x_perm; a.wg = wg; a.wu = wu; a.wd = wd;
  a.offsets = offsets; a.mt_start = w.mt_start; a.wk_start = w.wk_start; a.nz_start = w.nz_start;
  a.hg = hg; a.hu = hu; a.act = w.act; a.act_in = w.act; a.y = y;
  a.E_loc = E_loc; a.d = d; a.f = f;
  a.NT = static_cast<int>(ceil_div(f, (small ? TILE_S : TILE) / 2));
  if (hipError_t e = run_gemm<FWD_GATE_UP>(a, small, K_GEMM_FWD_GATE_UP, s); e != hipSuccess)
    return e;
  a.mt_start = mt_down;
  a.NT = static_cast<int>(ceil_div(d, small_d ? TILE_S : TILE));
  return run_gemm<FWD_DOWN>(a, small_d, K_GEMM_FWD_DOWN, s);
}

hipError_t launch_ffn_bwd(const uint16_t* dy, const uint16_t* x_perm, const uint16_t* hg,
                          const uint16_t* hu, const int32_t* offsets, int E_loc, int64_t cap,
                          int d, int f, const uint16_t* wg, const uint16_t* wu,
                          const uint16_t* wd, uint16_t* dx, uint16_t* dwg, uint16_t* dwu,
                          uint16_t* dwd, unsigned flags, void* ws, hipStream_t s) {
  GemmWs w = carve(ws, cap, E_loc, f, true);
  const int64_t rt = row_tiles(cap, E_loc);
  // the data gradients share one table of row tiles, and so a tile
  const bool small =
      few_rows(cap, E_loc) ||
      (use_small(rt * std::max(ceil_div(f, TILE), ceil_div(d, TILE))) &&
       !(keep_large(cap, E_loc, ceil_div(f, TILE), ceil_div(f, TILE_S), d) &&
         keep_large(cap, E_loc, ceil_div(d, TILE), ceil_div(d, TILE_S), 2 * int64_t{f})));
  const int S = small ? TILE_S : TILE;
  const int64_t experts = std::min<int64_t>(cap, E_loc);
  const bool wgrad = (flags & MOE_BWD_WGRAD) != 0;
  const bool small_g = small_weights(experts * ceil_div(d, TILE) * ceil_div(f, TILE / 2),
                                     experts * ceil_div(d, TILE_S) * ceil_div(f, TILE_S / 2));
  const bool small_d = small_weights(experts * ceil_div(f, TILE) * ceil_div(d, TILE),
                                     experts * ceil_div(f, TILE_S) * ceil_div(d, TILE_S));
  if (small && (!wgrad || (small_g && small_d)) && E_loc <= REG_EXPERTS)
    w.mt_start = nullptr;  // the kernels form the tables
  else if (hipError_t e = sched(offsets, E_loc, S, BK, w, s); e != hipSuccess)
    return e;
  GemmArgs a{};
  a.x_perm = x_perm; a.wg = wg; a.wu = wu; a.wd = wd;
  a.hg_in = hg; a.hu_in = hu; a.dy = dy;
  a.offsets = offsets; a.mt_start = w.mt_start; a.wk_start = w.wk_start; a.nz_start = w.nz_start;
  a.dhg = w.dhg; a.dhu = w.dhu; a.act = w.act;
  a.dhg_in = w.dhg; a.dhu_in = w.dhu; a.act_in = w.act;
  a.dx = dx; a.dwg = dwg; a.dwu = dwu; a.dwd = dwd;
  a.E_loc = E_loc; a.d = d; a.f = f;
  a.NT = static_cast<int>(ceil_div(f, S));
  if (hipError_t e = run_gemm<DGRAD_DOWN>(a, small, K_GEMM_DGRAD_DOWN, s); e != hipSuccess)
    return e;
  if (flags & MOE_BWD_DGRAD) {
    a.NT = static_cast<int>(ceil_div(d, S));
    if (hipError_t e = run_gemm<DGRAD_GATE_UP>(a, small, K_GEMM_DGRAD_GATE_UP, s);
        e != hipSuccess)
      return e;
  }
  if (wgrad) {
    const int Sg = small_g ? TILE_S : TILE;
    a.MT = static_cast<int>(ceil_div(d, Sg));
    a.NT = static_cast<int>(ceil_div(f, Sg / 2));
    if (hipError_t e = run_gemm<WGRAD_GATE_UP>(a, small_g, K_GEMM_WGRAD_GATE_UP, s);
        e != hipSuccess)
      return e;
    const int Sd = small_d ? TILE_S : TILE;
    a.MT = static_cast<int>(ceil_div(f, Sd));
    a.NT = static_cast<int>(ceil_div(d, Sd));
    if (hipError_t e = run_gemm<WGRAD_DOWN>(a, small_d, K_GEMM_WGRAD_DOWN, s); e != hipSuccess)
      return e;
  }
  return hipSuccess;
}

// ------------------------------------------------------ dense products
namespace {
template <int MODE>
hipError_t run_dense(GemmArgs& a, int kid, hipStream_t s) {
  auto tiles = [&](int S) {
    a.MT = static_cast<int>(ceil_div(a.dM, S));
    a.NT = static_cast<int>(ceil_div(a.dN, Traits<MODE>::DUAL ? S / 2 : S));
    return static_cast<int64_t>(a.batches) * a.MT * a.NT;
  };
  const int64_t n = tiles(TILE);
  if (n <= 0) return hipSuccess;
  const bool small = use_small(n);
  if (small) tiles(TILE_S);
  return run_gemm<MODE>(a, small, kid, s);
}
}  // namespace

hipError_t launch_router_dw_mfma(const uint16_t* x, const uint16_t* dl3, int64_t T, int d, int E,
                                 int64_t ld3, int64_t chunk, float* part, hipStream_t s) {
  GemmArgs a{};
  a.da = x; a.db = dl3; a.dc = part;
  a.a_ld = d; a.b_ld = ld3; a.c_ld = E; a.c_bstride = static_cast<int64_t>(d) * E;
  a.dM = d; a.dN = E; a.dK = static_cast<int>(T); a.dE = E;
  a.kspan = static_cast<int>(chunk); a.batches = static_cast<int>(ceil_div(T, chunk));
  return run_dense<RT_DW>(a, K_ROUTE_DW, s);
}

hipError_t launch_router_dx_mfma(const uint16_t* dl3, const uint16_t* w3, int64_t T, int d, int E,
                                 int64_t ld3, int accumulate, uint16_t* dx, hipStream_t s) {
  GemmArgs a{};
  a.da = dl3; a.db = w3; a.dc = dx;
  a.a_ld = ld3; a.b_ld = d; a.c_ld = d;
  a.dM = static_cast<int>(T); a.dN = d; a.dK = 3 * E; a.kspan = 3 * E; a.batches = 1;
  a.flag = accumulate;
  return run_dense<RT_DX>(a, K_ROUTE_DX, s);
}

hipError_t launch_vocab_logits_mfma(const uint16_t* x, const uint16_t* w, int64_t ldw, int64_t bc0,
                                    int64_t v0, int N, int H, int vb, const int32_t* target,
                                    float* part, float* yt, hipStream_t s) {
  GemmArgs a{};
  a.da = x; a.db = w; a.dc = part; a.target = target; a.yt = yt;
  a.a_ld = H; a.b_ld = ldw; a.bc0 = bc0; a.v0 = v0;
  a.dM = N; a.dN = vb; a.dK = H; a.kspan = H; a.batches = 1;
  return run_dense<VOC_FWD>(a, K_VOC_LOGITS, s);
}

hipError_t launch_vocab_grad_mfma(const uint16_t* x, const uint16_t* w, int64_t ldw, int64_t bc0,
                                  int64_t v0, int N, int H, int vb, const int32_t* target,
                                  const float* lse, const float* dloss, uint16_t* G, int64_t gp,
                                  hipStream_t s) {
  GemmArgs a{};
  a.da = x; a.db = w; a.dc = G; a.target = target; a.lse = lse; a.dloss = dloss;
  a.a_ld = H; a.b_ld = ldw; a.c_ld = gp; a.bc0 = bc0; a.v0 = v0;
  a.dM = N; a.dN = vb; a.dK = H; a.kspan = H; a.batches = 1;
  return run_dense<VOC_GRAD>(a, K_VOC_GRAD, s);
}

hipError_t launch_vocab_dx_mfma(const uint16_t* G, int64_t gp, const uint16_t* w, int64_t ldw,
                                int64_t bc0, int N, int H, int vb, int kspan, int first,
                                float* dxa, hipStream_t s) {
  GemmArgs a{};
  a.da = G; a.db = w; a.dc = dxa;
  a.a_ld = gp; a.b_ld = ldw; a.c_ld = H; a.c_bstride = static_cast<int64_t>(N) * H; a.bc0 = bc0;
  a.dM = N; a.dN = H; a.dK = vb; a.kspan = kspan;
  a.batches = static_cast<int>(ceil_div(vb, kspan));
  a.flag = first;
  return run_dense<VOC_DX>(a, K_VOC_DX, s);
}

hipError_t launch_vocab_dw_mfma(const uint16_t* x, const uint16_t* G, int64_t gp, int N, int H,
                                int vb, uint16_t* dw, int64_t ldd, int64_t cc0, hipStream_t s) {
  GemmArgs a{};
  a.da = x; a.db = G; a.dc = dw;
  a.a_ld = H; a.b_ld = gp; a.c_ld = ldd; a.cc0 = cc0;
  a.dM = H; a.dN = vb; a.dK = N; a.kspan = N; a.batches = 1;
  return run_dense<VOC_DW>(a, K_VOC_DW, s);
}

}  // namespace moe
