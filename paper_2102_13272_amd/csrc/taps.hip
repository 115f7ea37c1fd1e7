// The channel contraction of the mixed nest and of F(2,3) chains where level-1
// digit 3 is dead (r below the nest's taps): no real tap then has level-1 digit
// 2, so the 9 live points of a group come from 2 x 2 taps per (input, output) channel pair,
//
//   G w: q = 0: w0,  q = 1: (w0 + w1) / 2,  q = 2: (w0 - w1) / 2   on each axis.
//
// U keeps those 4 values instead of the 9 points, [live group][2 k1r + k1c][M]
// [Np], and this kernel forms the points in registers: 10 additions per 9 MFMA
// operands, the halves left to the final fold.  V holds the live points, [live
// group][3 q1r + q1c][M][Tp] (Np, Tp: N, T rounded up to 4).  Z is the other
// contractions' [P/16][N][T][4], after the level-1 A^T.
//
// What bounds it: the operands' stream.  Every U and V value is used once per
// block of a group, so the bytes are U + V + Z, and U is the larger operand.
// On the 31x31 layer (5184 groups, 128 x 128 channels, 64 tiles) U falls from
// 3.06 to 1.36 GB, of 5.27 GB in all.
//
// Work-group: a BM x BN block of (n, t) of one group, all 9 points at once
// (9 accumulator sets of WTM x WTN per wavefront), so V is read once per BM
// output channels and a group's points need no second pass over U.  A chunk is
// 8 channels of U's 4 planes and V's 9; four LDS stages filled by direct
// global->LDS loads, two to three chunks in flight, running on across the
// work-group's items (persistent, items dealt as in contract_deep_persist).
// The barrier that opens a chunk lies inside the one before it, between its two
// 4-channel products, so that the new chunk's first fragments are read while
// the matrix units still have work (31x31 layer, 1.04-1.12 -> 1.00-1.05 ms;
// 13x13 128 -> 128, 400 tiles, 0.497 -> 0.451).  Rows are stored rotated by 16
// values per channel (mod 4), so that the 4 channels of a fragment lie in
// different banks.
//
// Measured, contraction alone: 31x31 128 -> 128 (64 tiles) 1.17 -> 1.00-1.05 ms,
// 97.8 GFLOP at 93-98 TFLOP/s (62 % of the fp32 matrix peak) and 3.57 GB; 17x17
// 64 -> 64 (32 tiles, from the general quad kernel) 0.316 -> 0.146 ms; 13x13
// 64 -> 64 (200 tiles) 98 -> 84 us.  The matrix units wait on LDS and barriers for
// about a fifth of the time, and on memory for the rest of what is left.
//
// Operand lane maps of v_mfma_f32_16x16x4f32 (wave64):
//   A (16x4):  lane l holds A[l%16][l/16]
//   B (4x16):  lane l holds B[l/16][l%16]
//   D (16x16): lane l, register v holds D[4*(l/16)+v][l%16]
#include "taps.h"

#include <map>
#include <mutex>
#include <utility>

#include "nwg_internal.h"

namespace nwg {
namespace {

typedef float floatx4 __attribute__((ext_vector_type(4)));

constexpr int kCh = 8;                       // channels of a chunk

// Place of column c in row k (channel) of a staged plane of COLS columns.
template <int COLS>
__device__ __forceinline__ int place(int k, int c) {
  // 64 and more columns: the 4 channels of a fragment 16 banks apart; 32: rows
  // alternate between the bank halves, the second pair 16 further
  return COLS >= 64 ? (c + 16 * (k & 3)) & (COLS - 1) : (c + 16 * ((k >> 1) & 1)) & (COLS - 1);
}

// PLANES x 8 channels x COLS columns of one chunk -> LDS.  A wavefront's load j
// copies 64 quads; its lanes' offsets from the chunk's first value are kept.
template <int PLANES, int COLS, int NW>
struct ChunkLoader {
  static constexpr int LOADS = PLANES * kCh * COLS / 4 / 64;   // of the work-group
  static constexpr int EVERY = LOADS / NW, EXTRA = LOADS % NW; // per wave; waves with one more
  unsigned off[EVERY + (EXTRA ? 1 : 0)];
  // columns from c0 of rows of ld values (quads past the row re-read its last)
  __device__ __forceinline__ void init(int wave, int lane, int M, int ld, int c0) {
#pragma unroll
    for (int j = 0; j < EVERY + (EXTRA ? 1 : 0); ++j) {
      const int f = (wave + j * NW) * 64 + lane;       // quad of the chunk's buffer
      const int row = f / (COLS / 4), at = f - row * (COLS / 4);
      const int plane = row / kCh, k = row - plane * kCh;
      // the column quad whose place this is
      const int q = (COLS >= 64 ? at - 4 * (k & 3) : at - 4 * ((k >> 1) & 1)) & (COLS / 4 - 1);
      int c = c0 + 4 * q;
      if (c > ld - 4) c = ld - 4;
      off[j] = plane < PLANES ? (unsigned)((plane * M + k) * ld + c) : 0u;
    }
  }
  __device__ __forceinline__ void load(const float* __restrict__ base, float* dst, int wave) const {
#pragma unroll
    for (int j = 0; j < EVERY; ++j)
      __builtin_amdgcn_global_load_lds(
          (const void*)(base + off[j]),
          (__attribute__((address_space(3))) void*)(dst + (wave + j * NW) * 256), 16, 0, 0);
    if constexpr (EXTRA > 0) {
      if (wave < EXTRA)
        __builtin_amdgcn_global_load_lds(
            (const void*)(base + off[EVERY]),
            (__attribute__((address_space(3))) void*)(dst + (wave + EVERY * NW) * 256), 16, 0, 0);
    }
  }
};

// Group of the live list's (ir-th row prefix, ic-th column prefix): live_group
// in 32 bits.
__device__ __forceinline__ int group_at(const GroupMap& m, int ir, int ic) {
  unsigned pr = (unsigned)select_bit(m.mask0, m.mask1, ir), pc = (unsigned)select_bit(m.mask0, m.mask1, ic);
  int g = 0;
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    if (d < m.nd) {
      const unsigned l = (unsigned)m.rad[d];
      g += (int)(pr % l) * m.wr[d] + (int)(pc % l) * m.wc[d];
      pr /= l;
      pc /= l;
    }
  }
  return g;
}

template <int BM, int BN, int WM, int WN>
__global__ __launch_bounds__(64 * WM * WN) __attribute__((amdgpu_waves_per_eu(2))) void contract_taps(
    const float* __restrict__ U, const float* __restrict__ V, float4* __restrict__ Z, int M, int N,
    int T, int Np, int Tp, int ntb, int nnb, int G, int wpx, GroupMap gm) {
  constexpr int NW = WM * WN;
  constexpr int WTM = BM / WM, WTN = BN / WN, FM = WTM / 16, FN = WTN / 16;
  using LA = ChunkLoader<4, BM, NW>;
  using LB = ChunkLoader<9, BN, NW>;
  static_assert(LA::EXTRA == 0 && LA::LOADS * 64 == 4 * kCh * BM / 4 && LB::LOADS * 64 == 9 * kCh * BN / 4,
                "chunks of whole loads");
  constexpr int LPC = LA::EVERY + LB::EVERY;           // loads per chunk, one more in some waves
  __shared__ float A0[4 * kCh * BM], A1[4 * kCh * BM], A2[4 * kCh * BM], A3[4 * kCh * BM];
  __shared__ float B0[9 * kCh * BN], B1[9 * kCh * BN], B2[9 * kCh * BN], B3[9 * kCh * BN];

  // this work-group's items: first + i * wpx, i < mine
  // (fewer than 2^31 items in all)
  const unsigned items = (unsigned)ntb * (unsigned)nnb * (unsigned)G;
  const unsigned xcd = blockIdx.x % 8, jx = blockIdx.x / 8;
  const unsigned q = items / 8, rem = items % 8;
  const unsigned xstart = xcd < rem ? xcd * (q + 1) : rem * (q + 1) + (xcd - rem) * q;
  const unsigned xcount = q + (xcd < rem ? 1 : 0);
  const int mine = xcount > jx ? (int)((xcount - 1 - jx) / (unsigned)wpx + 1) : 0;
  if (mine == 0) return;                               // uniform over the work-group
  const unsigned first = xstart + jx;

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave / WN, wn = wave % WN;
  const int lr = lane & 15, lk = lane >> 4;
  const bool more = wave < LB::EXTRA;
  const int nk = M / kCh;

  floatx4 acc[9][FM][FN];
#pragma unroll
  for (int p = 0; p < 9; ++p)
#pragma unroll
    for (int c = 0; c < FM; ++c)
#pragma unroll
      for (int d = 0; d < FN; ++d) acc[p][c][d] = floatx4{0.f, 0.f, 0.f, 0.f};
  // this lane's places in the rows of its fragments (row k = 4 kk + lk)
  int pa[FM], pb[FN];
#pragma unroll
  for (int c = 0; c < FM; ++c) pa[c] = lk * BM + place<BM>(lk, wm * WTM + 16 * c + lr);
#pragma unroll
  for (int d = 0; d < FN; ++d) pb[d] = lk * BN + place<BN>(lk, wn * WTN + 16 * d + lr);

  // request cursor: item ri, chunk rc
  LA la;
  LB lb;
  const float* Ug = U;
  const float* Vg = V;
  int ri = 0, rc = 0;
  auto set_req_item = [&](int i) {
    unsigned b = first + (unsigned)(i * wpx);
    const int tb = (int)(b % (unsigned)ntb);
    b /= (unsigned)ntb;
    const int nb = (int)(b % (unsigned)nnb);
    const unsigned li = b / (unsigned)nnb;             // place in the live list
    Ug = U + (size_t)li * 4 * M * Np;
    Vg = V + (size_t)li * 9 * M * Tp;
    la.init(wave, lane, M, Np, nb * BM);
    lb.init(wave, lane, M, Tp, tb * BN);
  };
  // past the last item the last chunk is requested again, into a buffer that
  // is never read, so every step issues the same loads
  auto request_next = [&](float* An, float* Bn) {
    la.load(Ug + (size_t)rc * kCh * Np, An, wave);
    lb.load(Vg + (size_t)rc * kCh * Tp, Bn, wave);
    if (rc + 1 < nk) {
      ++rc;
    } else if (ri + 1 < mine) {
      ++ri;
      rc = 0;
      set_req_item(ri);
    }
  };
  // item it done: the level-1 fold, with the halves of G, and Z
  auto finish = [&](int it) {
    unsigned b = first + (unsigned)(it * wpx);
    const int tb = (int)(b % (unsigned)ntb);
    b /= (unsigned)ntb;
    const int nb = (int)(b % (unsigned)nnb);
    b /= (unsigned)nnb;
    const int ir = (int)(b / (unsigned)gm.np);
    const int g = group_at(gm, ir, (int)b - ir * gm.np);
    float4* __restrict__ Zg = Z + (size_t)g * N * T;
#pragma unroll
    for (int c = 0; c < FM; ++c)
#pragma unroll
      for (int d = 0; d < FN; ++d) {
        floatx4 z0[3], z1[3];                          // per q1r, i1c = 0 and 1
#pragma unroll
        for (int qr = 0; qr < 3; ++qr) {
          const floatx4 e = acc[3 * qr][c][d], f = acc[3 * qr + 1][c][d], h = acc[3 * qr + 2][c][d];
          z0[qr] = e + 0.5f * (f + h);
          z1[qr] = 0.5f * (f - h);
          acc[3 * qr][c][d] = acc[3 * qr + 1][c][d] = acc[3 * qr + 2][c][d] =
              floatx4{0.f, 0.f, 0.f, 0.f};
        }
        const floatx4 o0 = z0[0] + 0.5f * (z0[1] + z0[2]), o1 = z1[0] + 0.5f * (z1[1] + z1[2]);
        const floatx4 o2 = 0.5f * (z0[1] - z0[2]), o3 = 0.5f * (z1[1] - z1[2]);
        const int col = tb * BN + wn * WTN + 16 * d + lr;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int row = nb * BM + wm * WTM + 16 * c + 4 * lk + v;
          if (row < N && col < T)
            Zg[(size_t)row * T + col] = make_float4(o0[v], o1[v], o2[v], o3[v]);
        }
      }
  };
  // the fragments of 4 channels (kk = 0, 1) of a chunk, and their products
  struct Frag {
    float a[4][FM], b[9][FN];
  };
  auto read = [&](Frag& f, const float* Ac, const float* Bc, int kk) {
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
      for (int c = 0; c < FM; ++c) f.a[t][c] = Ac[(t * kCh + 4 * kk) * BM + pa[c]];
#pragma unroll
    for (int p = 0; p < 9; ++p)
#pragma unroll
      for (int d = 0; d < FN; ++d) f.b[p][d] = Bc[(p * kCh + 4 * kk) * BN + pb[d]];
  };
  auto multiply = [&](const Frag& f) {
#pragma unroll
    for (int c = 0; c < FM; ++c) {
      // the 9 points from the taps, without G's halves
      const float x[3] = {f.a[0][c], f.a[0][c] + f.a[1][c], f.a[0][c] - f.a[1][c]};
      const float y[3] = {f.a[2][c], f.a[2][c] + f.a[3][c], f.a[2][c] - f.a[3][c]};
#pragma unroll
      for (int qc = 0; qc < 3; ++qc) {
        const float u[3] = {x[qc], x[qc] + y[qc], x[qc] - y[qc]};
#pragma unroll
        for (int qr = 0; qr < 3; ++qr)
#pragma unroll
          for (int d = 0; d < FN; ++d)
            acc[3 * qr + qc][c][d] = __builtin_amdgcn_mfma_f32_16x16x4f32(
                u[qr], f.b[3 * qr + qc][d], acc[3 * qr + qc][c][d], 0, 0, 0);
      }
    }
  };
  int it = 0, kc = 0;                                  // item and chunk being multiplied
  Frag f0, f1;
  // Chunk c in (Ac, Bc), its first fragments in f0; chunk c + 1 in (A1, B1).
  // The barrier that opens chunk c + 1 lies between the chunk's two products,
  // so its fragments are read while the second product runs.  The chunk's new
  // request (c + 3) overwrites chunk c - 1, whose reads ended before it.
  auto step = [&](const float* Ac, const float* Bc, const float* A1, const float* B1, float* An,
                  float* Bn) {
    if (it >= mine) return;                            // uniform: past the last chunk
    read(f1, Ac, Bc, 1);
    multiply(f0);
    if (more)
      wait_vmcnt<LPC + 1>();
    else
      wait_vmcnt<LPC>();
    __builtin_amdgcn_s_barrier();
    request_next(An, Bn);
    read(f0, A1, B1, 0);
    multiply(f1);
    if (++kc == nk) {
      finish(it);
      ++it;
      kc = 0;
    }
  };

  set_req_item(0);
  request_next(A0, B0);
  request_next(A1, B1);
  request_next(A2, B2);
  if (more)
    wait_vmcnt<2 * (LPC + 1)>();
  else
    wait_vmcnt<2 * LPC>();
  __builtin_amdgcn_s_barrier();
  read(f0, A0, B0, 0);
  while (it < mine) {
    step(A0, B0, A1, B1, A3, B3);
    step(A1, B1, A2, B2, A0, B0);
    step(A2, B2, A3, B3, A1, B1);
    step(A3, B3, A0, B0, A2, B2);
  }
  wait_vmcnt<0>();                                     // the repeated tail loads land before exit
}

template <int BM, int BN, int WM, int WN>
hipError_t launch(const nwg_plan_info& g, const float* U, const float* V, float* Z, hipStream_t s) {
  const int T = (int)g.T, Np = (g.N + 3) & ~3, Tp = (T + 3) & ~3;
  const int ntb = (T + BN - 1) / BN, nnb = (g.N + BM - 1) / BM;
  const GroupMap gm = taps_groups(g);
  if ((double)ntb * nnb * gm.np * gm.np >= 2147483648.0) return hipErrorInvalidValue;
  int dev = 0, cus = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
  if (e != hipSuccess) return e;
  const auto k = &contract_taps<BM, BN, WM, WN>;
  const int occ = taps_occupancy(dev, reinterpret_cast<const void*>(k), 64 * WM * WN);
  if (occ <= 0 || cus < 8) return hipErrorInvalidValue;
  const int wpx = cus / 8 * occ;                       // work-groups per XCD
  k<<<8 * wpx, 64 * WM * WN, 0, s>>>(U, V, reinterpret_cast<float4*>(Z), g.M, g.N, T, Np, Tp, ntb,
                                     nnb, gm.np * gm.np, wpx, gm);
  return hipGetLastError();
}

}  // namespace

int taps_occupancy(int dev, const void* kernel, int threads) {
  static std::mutex mu;
  static std::map<std::pair<int, const void*>, int> cache;
  std::lock_guard<std::mutex> lock(mu);
  const auto key = std::make_pair(dev, kernel);
  const auto it = cache.find(key);
  if (it != cache.end()) return it->second;
  int b = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&b, kernel, threads, 0) != hipSuccess) {
    (void)hipGetLastError();
    b = 0;
  }
  cache[key] = b;
  return b;
}

hipError_t launch_contract_taps(const nwg_plan_info& g, const float* U, const float* V, float* Z,
                                hipStream_t s) {
  if (!taps_applies(g) || (((uintptr_t)U | (uintptr_t)V | (uintptr_t)Z) & 15))
    return hipErrorInvalidValue;
  // the block with the least padded area, weighed by what a block's products take
  // (31x31 128 -> 128, 64 tiles: 1.05 ms on 128 x 64, 1.19 on 64 x 32, 1.26 on
  // 32 x 32; 17x17 64 -> 64, 32 tiles: 0.36, 0.146, 0.153; 31x31 32 -> 32, 64
  // tiles: 0.27, 0.18, 0.15)
  auto area = [&](int bm, int bn) {
    return (double)((g.N + bm - 1) / bm * bm) * (double)((g.T + bn - 1) / bn * bn);
  };
  const double a = area(128, 64), b = 1.14 * area(64, 32), c = 1.2 * area(32, 32);
  if (a <= b && a <= c) return launch<128, 64, 4, 2>(g, U, V, Z, s);
  if (b <= c) return launch<64, 32, 2, 2>(g, U, V, Z, s);
  return launch<32, 32, 2, 2>(g, U, V, Z, s);
}

}  // namespace nwg
