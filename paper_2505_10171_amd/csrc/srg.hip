// srg.hip -- BF16 matrix-core training and inference of the run-outcome
// surrogate (see include/srg.h) for gfx950.
//
// The network is small (212,275 parameters): a layer's product over a batch is a
// few microseconds, so what counts is launches and the latency of the chain.
// Inference is one kernel, its activations in LDS (k_mlp).  A training batch is two:
// everything that is independent per row (k_train_rows: forward, loss, backward
// through the layers), then everything that sums over rows (k_train_weights:
// weight and bias gradients, with the Adam update of what a workgroup owns).
// Weights are kept in BF16 in the order the matrix instructions read them.
#include <hip/hip_runtime.h>
#include <stdarg.h>
#include <stdio.h>
#include <string.h>

#include <algorithm>
#include <new>
#include <random>
#include <type_traits>
#include <vector>

#include "../../include/lbm.h"
#include "../../include/srg.h"

namespace srg {

typedef __bf16 bf16;
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int NL = 5;                                  // layers
constexpr int KIN[NL] = {32, 256, 256, 256, 256};      // padded fan-in
constexpr int NOUT[NL] = {256, 256, 256, 256, 64};     // padded fan-out
constexpr int KREAL[NL] = {SRG_IN, 256, 256, 256, 256};
constexpr int NREAL[NL] = {256, 256, 256, 256, SRG_OUT};
constexpr int NCLS = 3, NTRAJ = 48;
// offsets of layer l: weights and biases in the padded parameter vector, weights
// in the fragment copies
__host__ __device__ constexpr int w_at(int l) {
  return l == 0 ? 0 : 32 * 256 + 256 + (l - 1) * (256 * 256 + 256);
}
__host__ __device__ constexpr int b_at(int l) { return w_at(l) + (l == 0 ? 32 : 256) * (l == 4 ? 64 : 256); }
__host__ __device__ constexpr int t_at(int l) { return l == 0 ? 0 : 32 * 256 + (l - 1) * 256 * 256; }
constexpr int ALIGN = 256;

// ---------------------------------------------------------- weight layouts
// The matrix instructions read their weight operand straight from memory, so
// each weight matrix W (K x N, FP32) is kept as BF16 in the order of the
// fragments: 64 lanes x 8 values (1 KB) per fragment, one coalesced 16-byte load
// per lane, and no LDS between (a wave's columns are its own).
//   wf: forward, 32x32x16: fragment (n / 32, k / 16), lane n % 32 + 32 (k / 8 % 2)
//   wg: forward, 16x16x32: fragment (n / 16, k / 32), lane n % 16 + 16 (k / 8 % 4)
//   wb: backward, 16x16x32: fragment (k / 16, n / 32), lane k % 16 + 16 (n / 8 % 4)
__device__ __forceinline__ int wf_index(int K, int k, int n) {
  return ((n >> 5) * (K >> 4) + (k >> 4)) * 512 + ((((k >> 3) & 1) << 5) + (n & 31)) * 8 + (k & 7);
}
__device__ __forceinline__ int wg_index(int K, int k, int n) {
  return ((n >> 4) * (K >> 5) + (k >> 5)) * 512 + ((((k >> 3) & 3) << 4) + (n & 15)) * 8 + (k & 7);
}
__device__ __forceinline__ int wb_index(int N, int k, int n) {
  return ((k >> 4) * (N >> 5) + (n >> 5)) * 512 + ((((n >> 3) & 3) << 4) + (k & 15)) * 8 + (n & 7);
}
struct Weights {
  const bf16 *wf[NL], *wg[NL], *wb[NL];
  const float* b[NL];
};
__device__ __forceinline__ bf16x8 frag(const bf16* w, int f, int lane) {
  return *(const bf16x8*)(w + ((size_t)f * 64 + lane) * 8);
}

// Activation tiles in LDS: rows of 256 BF16, the 16-byte chunk c of row r at
// position c ^ (r % 32), so that the rows of an A fragment read distinct banks.
__device__ __forceinline__ bf16* mlp_row(bf16* act, int row, int chunk) {
  return act + row * 256 + ((chunk ^ (row & 31)) << 3);
}
// row within a 32x32 result of a lane's value r (its column is lane % 32)
__device__ __forceinline__ int row32(int r, int half) { return (r >> 2) * 8 + half * 4 + (r & 3); }

// ---------------------------------------------------------------- inference
// Whole forward pass of 32 RB rows per workgroup.  The activations stay in LDS
// through the five layers; a wave takes 32 RT rows by 32 CT columns of a layer
// with v_mfma_f32_32x32x16_bf16 and reads its weight fragments from L2, AHEAD K
// steps ahead, the first of a layer before the barrier that ends the one before.
// What bounds it: with few rows the latency of five layers (1 to 8,192 rows 9 to
// 12 us with 32 rows per workgroup, 26 with 128 and the weights staged through
// LDS behind barriers, as it was); with many the two streams of fragments, A from
// LDS and the weights from L2, which a wave of 64 rows loads at the CU's 64 bytes
// per clock while it multiplies, one of 128 rows at half that (65,536 rows: 39 us
// with 64 rows, 35 with 128 and two workgroups per CU, 52 before).  A wave of
// 128 rows by 64 columns reads less of both, but one workgroup per CU waits at its
// barriers (51), and two spill (49).
constexpr int MLP_ROWS_32 = 8192;   // up to here 32 rows per workgroup, one per CU
constexpr int MLP_ROWS_64 = 32768;  // up to here 64 (32,768 rows 22 us either way,
                                    // 16,384 15 against 20), beyond 128
constexpr size_t mlp_lds(int RB) { return (size_t)RB * 32 * 256 * 2; }

template <int RB, int RT, int CT, int AHEAD>
__global__ __launch_bounds__(64 * (RB / RT) * (8 / CT))
    __attribute__((amdgpu_waves_per_eu(4, 8))) void k_mlp(const float* __restrict__ X, int n,
                                                          Weights a, float* __restrict__ y) {
  extern __shared__ __attribute__((aligned(16))) bf16 act[];
  constexpr int CW = 8 / CT, NW = (RB / RT) * CW, T = 64 * NW, ROWS = 32 * RB;
  const int t = threadIdx.x, lane = t & 63, w = t >> 6, fr = lane & 31, fk = lane >> 5;
  const int rw = w / CW, cw = w % CW;
  const int m0 = blockIdx.x * ROWS;
  // inputs padded to 32 features: four chunks a row, the features in the first
  for (int q = t; q < ROWS * 4; q += T) {
    const int row = q >> 2, ch = q & 3;
    bf16x8 v;
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = (bf16)0.f;
    if (ch == 0 && m0 + row < n) {
      const float* x = X + (long long)(m0 + row) * SRG_IN;
#pragma unroll
      for (int e = 0; e < SRG_IN; ++e) v[e] = (bf16)x[e];
    }
    *(bf16x8*)mlp_row(act, row, ch) = v;
  }
  bf16x8 b[AHEAD][CT];
  // fragments of the wave's columns: K steps ks of layer l (KS of them)
  auto fetch = [&](const bf16* W, int KS, int ks, bf16x8* v) {
#pragma unroll
    for (int j = 0; j < CT; ++j) v[j] = frag(W, (cw * CT + j) * KS + ks, lane);
  };
  f32x16 acc[RT][CT];
  auto clear = [&]() {
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
      for (int j = 0; j < CT; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
  };
  auto product = [&](int ks, const bf16x8* v) {
#pragma unroll
    for (int i = 0; i < RT; ++i) {
      const bf16x8 av = *(const bf16x8*)mlp_row(act, 32 * (rw * RT + i) + fr, 2 * ks + fk);
#pragma unroll
      for (int j = 0; j < CT; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av, v[j], acc[i][j], 0, 0, 0);
    }
  };
  auto relu_out = [&](const float* bias) {
#pragma unroll
    for (int j = 0; j < CT; ++j) {
      const int col = 32 * (cw * CT + j) + fr;
      const float bn = bias[col];
#pragma unroll
      for (int i = 0; i < RT; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r)
          mlp_row(act, 32 * (rw * RT + i) + row32(r, fk), col >> 3)[col & 7] =
              (bf16)fmaxf(acc[i][j][r] + bn, 0.f);
    }
  };
  // first layer: K = 32, two steps
  fetch(a.wf[0], 2, 0, b[0]);
  fetch(a.wf[0], 2, 1, b[1]);
  clear();
  __syncthreads();
  product(0, b[0]);
  product(1, b[1]);
  // its own A reads are done: the next layer's first fragments
#pragma unroll
  for (int u = 0; u < AHEAD; ++u) fetch(a.wf[1], 16, u, b[u]);
  __syncthreads();
  relu_out(a.b[0]);
  for (int l = 1; l < NL - 1; ++l) {
    clear();
    __syncthreads();
    const bf16* W = a.wf[l];
    // not unrolled past the fragments in flight: the compiler would hoist the
    // loads of the whole layer and spill
#pragma unroll 1
    for (int k4 = 0; k4 < 16; k4 += AHEAD) {
#pragma unroll
      for (int u = 0; u < AHEAD; ++u) {
        product(k4 + u, b[u]);
        if (k4 + AHEAD < 16) fetch(W, 16, k4 + AHEAD + u, b[u]);
      }
    }
    if (l + 1 < NL - 1) {
#pragma unroll
      for (int u = 0; u < AHEAD; ++u) fetch(a.wf[l + 1], 16, u, b[u]);
    }
    __syncthreads();
    relu_out(a.b[l]);
  }
  __syncthreads();
  // output layer: RB x 2 tiles of 32 rows by 32 of the 64 padded columns
  constexpr int OC = NW >= 2 * RB ? 1 : 2;           // column tiles per wave
  constexpr int OR = NW >= 2 * RB ? 1 : RB / NW;     // row tiles per wave
  const int r0 = OC == 1 ? w >> 1 : w * OR, c0 = OC == 1 ? w & 1 : 0;
  if (r0 < RB) {
    f32x16 o[OR][OC];
#pragma unroll
    for (int i = 0; i < OR; ++i)
#pragma unroll
      for (int j = 0; j < OC; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[i][j][r] = 0.f;
#pragma unroll 4
    for (int ks = 0; ks < 16; ++ks) {
      bf16x8 v[OC];
#pragma unroll
      for (int j = 0; j < OC; ++j) v[j] = frag(a.wf[4], (c0 + j) * 16 + ks, lane);
#pragma unroll
      for (int i = 0; i < OR; ++i) {
        const bf16x8 av = *(const bf16x8*)mlp_row(act, 32 * (r0 + i) + fr, 2 * ks + fk);
#pragma unroll
        for (int j = 0; j < OC; ++j)
          o[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av, v[j], o[i][j], 0, 0, 0);
      }
    }
#pragma unroll
    for (int j = 0; j < OC; ++j) {
      const int col = 32 * (c0 + j) + fr;
      if (col >= SRG_OUT) continue;
      const float bn = a.b[4][col];
#pragma unroll
      for (int i = 0; i < OR; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int row = m0 + 32 * (r0 + i) + row32(r, fk);
          if (row < n) y[(long long)row * SRG_OUT + col] = o[i][j][r] + bn;
        }
    }
  }
}

// ---------------------------------------------------- training: the row pass
// Forward pass, loss, output gradient and the gradients dz of every layer's
// pre-activation for 32 rows per workgroup (eight waves, a wave 32 columns of a
// layer): everything in a batch that is independent per row, in one launch.
// Written for the weight pass: the padded BF16 inputs, the activations of the
// hidden layers, and dz of all five layers.  A batch of 256 rows is eight
// workgroups and waits on the latency of its nine products, each of whose weight
// fragments are requested one product ahead; layer by layer it was ten launches.
// A whole batch with its weight pass: 256 rows 34 us (160 before, 24 launches),
// 64 rows 28, 1,024 rows 64, 4,096 rows 144.
// BIG: the hidden layers' forward products with v_mfma_f32_32x32x16_bf16 (batches
// of a multiple of 128 rows, as always), else 16x16x32 like all others; the two
// round their sums differently, so the choice stays with the batch size.
struct RowArgs {
  const bf16* X;       // packed inputs (rows of 32), row perm[off + r] or r
  const int* perm;
  int off;
  const int* lab;      // per input row
  const float* traj;
  float w_traj, inv_B;
  Weights w;
  bf16* xb;            // outputs: inputs by batch row (32 wide)
  bf16* act[NL];       // act[l]: input of layer l >= 1 (256 wide)
  bf16* dz[NL];        // 256 wide, the last 64
  float* loss;         // sum (atomic)
};
constexpr size_t ROW_LDS = (size_t)5 * 32 * 256 * 2 + (size_t)32 * 64 * 4;

template <bool BIG>
__global__ __launch_bounds__(512) void k_train_rows(RowArgs g) {
  extern __shared__ __attribute__((aligned(16))) bf16 rows_lds[];
  bf16* const a_[4] = {rows_lds, rows_lds + 8192, rows_lds + 16384, rows_lds + 24576};
  bf16* const d_ = rows_lds + 32768;  // the current dz; before that the inputs
  float* const Y = (float*)(rows_lds + 40960);
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const int fr = lane & 31, fk = lane >> 5;        // 32x32x16 lanes
  const int gr = lane & 15, gk = lane >> 4;        // 16x16x32 lanes
  const int m0 = blockIdx.x * 32;
  bf16x8 b[16];
  // weight fragments of one product: the wave's 32 columns, all K steps
  auto fetch32 = [&](const bf16* W, int KS) {
#pragma unroll
    for (int ks = 0; ks < 16; ++ks)
      if (ks < KS) b[ks] = frag(W, w * KS + ks, lane);
  };
  auto fetch16 = [&](const bf16* W, int KS) {  // two column tiles, KS <= 8
#pragma unroll
    for (int ks = 0; ks < 8; ++ks)
#pragma unroll
      for (int j = 0; j < 2; ++j)
        if (ks < KS) b[2 * ks + j] = frag(W, (2 * w + j) * KS + ks, lane);
  };
  auto fetch_fwd = [&](int l) {
    if (BIG)
      fetch32(g.w.wf[l], KIN[l] / 16);
    else
      fetch16(g.w.wg[l], KIN[l] / 32);
  };
  fetch_fwd(0);
  // inputs: 32 rows of four chunks
  if (t < 128) {
    const int row = t >> 2, ch = t & 3;
    const long long src = g.perm ? g.perm[g.off + m0 + row] : m0 + row;
    const bf16x8 v = *(const bf16x8*)(g.X + src * 32 + ch * 8);
    *(bf16x8*)mlp_row(d_, row, ch) = v;
    if (g.xb != g.X || g.perm) *(bf16x8*)(g.xb + (long long)(m0 + row) * 32 + ch * 8) = v;
  }
  __syncthreads();
  // 16x16x32 products of the wave's 32 columns from tile A (two row tiles)
  f32x4 c4[2][2];
  auto product16 = [&](bf16* A, int KS) {
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j) c4[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) {
      if (ks >= KS) break;
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const bf16x8 av = *(const bf16x8*)mlp_row(A, 16 * i + gr, 4 * ks + gk);
#pragma unroll
        for (int j = 0; j < 2; ++j)
          c4[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, b[2 * ks + j], c4[i][j], 0, 0, 0);
      }
    }
  };
  // a tile's rows to memory, 16 bytes per thread and turn
  auto store_tile = [&](bf16* A, bf16* dst) {
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int q = t + 512 * u, row = q >> 5, ch = q & 31;
      *(bf16x8*)(dst + (long long)(m0 + row) * 256 + ch * 8) = *(const bf16x8*)mlp_row(A, row, ch);
    }
  };
  // ---- forward
  auto layer = [&](int l, bf16* A, bf16* O, auto KSTEPS) {
    constexpr int K = decltype(KSTEPS)::value;
    const float* bias = g.w.b[l];
    if (BIG) {
      f32x16 acc;
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[r] = 0.f;
#pragma unroll
      for (int ks = 0; ks < K / 16; ++ks) {
        const bf16x8 av = *(const bf16x8*)mlp_row(A, fr, 2 * ks + fk);
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av, b[ks], acc, 0, 0, 0);
      }
      if (l + 1 < NL - 1) fetch_fwd(l + 1);
      const int col = 32 * w + fr;
      const float bn = bias[col];
#pragma unroll
      for (int r = 0; r < 16; ++r)
        mlp_row(O, row32(r, fk), col >> 3)[col & 7] = (bf16)fmaxf(acc[r] + bn, 0.f);
    } else {
      product16(A, K / 32);
      if (l + 1 < NL - 1) fetch_fwd(l + 1);
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const int col = 32 * w + 16 * j + gr;
        const float bn = bias[col];
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int r = 0; r < 4; ++r)
            mlp_row(O, 16 * i + gk * 4 + r, col >> 3)[col & 7] =
                (bf16)fmaxf(c4[i][j][r] + bn, 0.f);
      }
    }
    __syncthreads();
    store_tile(O, g.act[l + 1]);
  };
  layer(0, d_, a_[0], std::integral_constant<int, 32>());
  layer(1, a_[0], a_[1], std::integral_constant<int, 256>());
  layer(2, a_[1], a_[2], std::integral_constant<int, 256>());
  layer(3, a_[2], a_[3], std::integral_constant<int, 256>());
  // output layer: 2 x 4 tiles of 16x16, a wave each
  {
    const int i = w >> 2, j = w & 3;
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) b[ks] = frag(g.w.wg[4], j * 8 + ks, lane);
    f32x4 o = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) {
      const bf16x8 av = *(const bf16x8*)mlp_row(a_[3], 16 * i + gr, 4 * ks + gk);
      o = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, b[ks], o, 0, 0, 0);
    }
    fetch16(g.w.wb[4], 2);
    const int col = 16 * j + gr;
    const float bn = g.w.b[4][col];
#pragma unroll
    for (int r = 0; r < 4; ++r) Y[(16 * i + gk * 4 + r) * 64 + col] = o[r] + bn;
  }
  __syncthreads();
  // ---- loss and dL/dy: 16 threads per row, three trajectory values each
  {
    const int r = t >> 4, u = t & 15;
    const long long row = g.perm ? g.perm[g.off + m0 + r] : m0 + r;
    const float* y = Y + r * 64;
    const float* tr = g.traj + row * NTRAJ;
    const float sc = 2.f * g.w_traj * g.inv_B / (float)NTRAJ;
    auto put = [&](int col, float v) {
      const bf16 x = (bf16)v;
      mlp_row(d_, r, col >> 3)[col & 7] = x;
      g.dz[4][(long long)(m0 + r) * 64 + col] = x;
    };
    float se2 = 0.f;
#pragma unroll
    for (int e = 0; e < 3; ++e) {
      const int j = u + 16 * e;
      const float df = y[NCLS + j] - tr[j];
      se2 += df * df;
      put(NCLS + j, sc * df);
    }
    if (u < 64 - SRG_OUT) put(SRG_OUT + u, 0.f);
    for (int o = 8; o > 0; o >>= 1) se2 += __shfl_xor(se2, o, 16);
    float l = 0.f;
    if (u == 0) {
      const float mx = fmaxf(y[0], fmaxf(y[1], y[2]));
      float e[NCLS], se = 0.f;
#pragma unroll
      for (int c = 0; c < NCLS; ++c) {
        e[c] = __expf(y[c] - mx);
        se += e[c];
      }
      const int lb = g.lab[row];
#pragma unroll
      for (int c = 0; c < NCLS; ++c) put(c, (e[c] / se - (c == lb ? 1.f : 0.f)) * g.inv_B);
      l = (-(y[lb] - mx - __logf(se)) + g.w_traj * se2 / (float)NTRAJ) * g.inv_B;
    }
    for (int o = 32; o > 0; o >>= 1) l += __shfl_xor(l, o, 64);
    if (lane == 0) atomicAdd(g.loss, l);
  }
  __syncthreads();
  // ---- backward: dz of layer l - 1 = (dz_l W_l^T) relu'(act[l])
#pragma unroll
  for (int l = NL - 1; l > 0; --l) {
    product16(d_, NOUT[l] / 32);
    if (l > 1) fetch16(g.w.wb[l - 1], 8);
    __syncthreads();  // every wave has read dz_l
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int col = 32 * w + 16 * j + gr;
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int row = 16 * i + gk * 4 + r;
          const float av = (float)mlp_row(a_[l - 1], row, col >> 3)[col & 7];
          mlp_row(d_, row, col >> 3)[col & 7] = (bf16)(av > 0.f ? c4[i][j][r] : 0.f);
        }
    }
    __syncthreads();
    store_tile(d_, g.dz[l - 1]);
  }
}

// ------------------------------------------------- training: the weight pass
// Gradients of all weights (dW_l = a_l^T dz_l over the batch) and biases (column
// sums of dz_l) in one launch, a workgroup per 64x64 tile or 64 bias columns,
// and with APPLY the Adam update of what the workgroup owns: the gradient never
// leaves its registers, and the BF16 copies of the new weights are written in
// their fragment orders.  The batch is the contraction, in steps of 32 rows
// through LDS (both operands transposed while staging), the next four steps' rows in
// flight.  56 + 17 workgroups on 256 CUs: bound by the latency of the B / 32
// steps; ten gradient launches, Adam and five transposes before.
struct WeightArgs {
  const bf16* x;        // batch inputs (32 wide)
  const bf16* act[NL];
  const bf16* dz[NL];
  int B;
  float *p, *m, *v, *g;
  bf16 *wf, *wg, *wb;   // layer l at t_off[l]
  float lr, bc1, bc2;
};
// of five pointers the l-th (selects: an indexed argument array would be copied
// to scratch)
template <class T>
__device__ __forceinline__ T* pick(T* const* a, int l) {
  T* r = a[4];
#pragma unroll
  for (int k = 3; k >= 0; --k) r = l == k ? a[k] : r;
  return r;
}
// tile b of the weight gradients: layer and tile origin; b counts layer 0's four
// tiles, 16 for each hidden layer and the last layer's four
constexpr int W_TILES = 4 + 3 * 16 + 4, B_TILES = 4 * 4 + 1;
constexpr int COLSUM_WAVES = 16;
constexpr int W_AHEAD = 4;  // K steps of rows in flight

// a parameter with its moments, read well before its update: read in turn behind
// the stores of the one before, each would wait for those (16 round trips of a lane)
struct AdamState {
  float p, m, v;
};
__device__ __forceinline__ AdamState adam_load(const WeightArgs& g, int i) {
  return AdamState{g.p[i], g.m[i], g.v[i]};
}
__device__ __forceinline__ float adam(const WeightArgs& g, int i, const AdamState& a, float gi) {
  const float mi = 0.9f * a.m + 0.1f * gi;
  const float vi = 0.999f * a.v + 0.001f * gi * gi;
  g.m[i] = mi;
  g.v[i] = vi;
  const float pi = a.p - g.lr * (mi / g.bc1) / (sqrtf(vi / g.bc2) + 1e-8f);
  g.p[i] = pi;
  return pi;
}

template <bool APPLY>
__global__ __launch_bounds__(256) void k_train_weights(WeightArgs g) {
  constexpr int LD = 40;  // LDS row: 32 batch rows + 8 padding (80 bytes)
  __shared__ __attribute__((aligned(16))) bf16 As[64 * LD], Bs[64 * LD];
  __shared__ float part[COLSUM_WAVES][64];
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  if (blockIdx.x >= W_TILES) {
    // column sums of 64 columns: 16 interleaved groups of 8 rows, added in order
    const int bt = blockIdx.x - W_TILES, l = bt >> 2, n = (bt & 3) * 64 + lane;
    const int ld = l == 4 ? 64 : 256, i = b_at(l) + n;
    AdamState st = {};
    if (APPLY && w == 0) st = adam_load(g, i);
    const bf16* D = pick(g.dz, l);
    // a wave its four groups together, 32 rows in flight: group after group the
    // sums were the longest chain of the launch (a batch of 256 rows 38 -> 34 us,
    // 1,024 rows 92 -> 64, 4,096 rows 290 -> 144)
    float sum[4] = {0.f, 0.f, 0.f, 0.f};
    for (int c0 = 0; c0 < g.B; c0 += 8 * COLSUM_WAVES) {
      float v[4][8];
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          const int m = c0 + 8 * (w + 4 * q) + u;
          v[q][u] = (float)D[(long long)min(m, g.B - 1) * ld + n];
          if (m >= g.B) v[q][u] = 0.f;
        }
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int u = 0; u < 8; ++u) sum[q] += v[q][u];
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) part[w + 4 * q][lane] = sum[q];
    __syncthreads();
    if (w == 0) {
      float s = 0.f;
#pragma unroll
      for (int q = 0; q < COLSUM_WAVES; ++q) s += part[q][lane];
      if (APPLY)
        adam(g, i, st, s);
      else
        g.g[i] = s;
    }
    return;
  }
  const int bt = blockIdx.x;
  const int l = bt < 4 ? 0 : bt < 52 ? 1 + ((bt - 4) >> 4) : 4;
  const int tile = bt < 4 ? bt : bt < 52 ? (bt - 4) & 15 : bt - 52;
  const int m0 = l == 0 ? 0 : l == 4 ? tile * 64 : (tile >> 2) * 64;
  const int n0 = l == 4 ? 0 : (tile & 3) * 64;
  const int M = l == 0 ? 32 : 256, N = l == 4 ? 64 : 256;
  const bf16* A = l == 0 ? g.x : pick(g.act, l);
  const bf16* D = pick(g.dz, l);
  const int wm = (w >> 1) * 32, wn = (w & 1) * 32;
  // staging: thread t moves eight columns of batch row t / 8 of both operands
  const int sk = t >> 3, sc = (t & 7) * 8;
  const bool ma = m0 + sc < M;
  const bf16x8 zero8 = {};
  auto load_a = [&](int k0) {
    return ma ? *(const bf16x8*)(A + (long long)(k0 + sk) * M + m0 + sc) : zero8;
  };
  auto load_d = [&](int k0) { return *(const bf16x8*)(D + (long long)(k0 + sk) * N + n0 + sc); };
  f32x4 acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  bf16x8 va[W_AHEAD], vd[W_AHEAD];
#pragma unroll
  for (int u = 0; u < W_AHEAD; ++u)
    if (32 * u < g.B) {
      va[u] = load_a(32 * u);
      vd[u] = load_d(32 * u);
    }
  const int fr = lane & 15, fk = (lane >> 4) * 8;
  // lane holds rows (lane / 16) * 4 + r (r = 0..3) of column lane % 16 per block
  auto row = [&](int i, int r) { return m0 + wm + i * 16 + (lane >> 4) * 4 + r; };
  auto col = [&](int j) { return n0 + wn + j * 16 + (lane & 15); };
  AdamState st[2][2][4];
  if (APPLY) {
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          st[i][j][r] = adam_load(g, w_at(l) + min(row(i, r), M - 1) * N + col(j));
  }
  auto step = [&](int k0, bf16x8& na, bf16x8& nd) {
    __syncthreads();
#pragma unroll
    for (int j = 0; j < 8; ++j) As[(sc + j) * LD + sk] = na[j];
#pragma unroll
    for (int j = 0; j < 8; ++j) Bs[(sc + j) * LD + sk] = nd[j];
    __syncthreads();
    if (k0 + 32 * W_AHEAD < g.B) {
      na = load_a(k0 + 32 * W_AHEAD);
      nd = load_d(k0 + 32 * W_AHEAD);
    }
    bf16x8 a[2], b[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) a[i] = *(const bf16x8*)(As + (wm + i * 16 + fr) * LD + fk);
#pragma unroll
    for (int j = 0; j < 2; ++j) b[j] = *(const bf16x8*)(Bs + (wn + j * 16 + fr) * LD + fk);
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[i], b[j], acc[i][j], 0, 0, 0);
  };
  for (int k0 = 0; k0 < g.B; k0 += 32 * W_AHEAD)
#pragma unroll
    for (int u = 0; u < W_AHEAD; ++u)
      if (k0 + 32 * u < g.B) step(k0 + 32 * u, va[u], vd[u]);
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int n = col(j);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int k = row(i, r);
        if (k >= M) continue;
        const int e = w_at(l) + k * N + n;
        if (APPLY) {
          const bf16 x = (bf16)adam(g, e, st[i][j][r], acc[i][j][r]);
          g.wf[t_at(l) + wf_index(M, k, n)] = x;
          g.wg[t_at(l) + wg_index(M, k, n)] = x;
          g.wb[t_at(l) + wb_index(N, k, n)] = x;
        } else {
          g.g[e] = acc[i][j][r];
        }
      }
    }
}

// the fragment copies of one weight matrix W (K x N)
__global__ void k_pack(const float* __restrict__ W, int K, int N, bf16* __restrict__ wf,
                       bf16* __restrict__ wg, bf16* __restrict__ wb) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= K * N) return;
  const int k = t / N, n = t - k * N;
  const bf16 x = (bf16)W[t];
  wf[wf_index(K, k, n)] = x;
  wg[wg_index(K, k, n)] = x;
  wb[wb_index(N, k, n)] = x;
}

}  // namespace srg

using namespace srg;

namespace {
size_t aup(size_t v) { return (v + ALIGN - 1) / ALIGN * ALIGN; }

struct Layout {
  size_t w_off[NL], b_off[NL], n_par;  // offsets (elements) in the padded vector
  size_t t_off[NL], n_wt;              // weight copies in fragment order
  size_t off_p, off_g, off_m, off_v, off_wf, off_wg, off_wb, off_xall, off_lab, off_traj, off_perm,
      off_xb, off_act[NL], off_dz[NL], off_acc, off_xin, off_yout, total;
};

Layout make_layout(int max_batch, int max_train) {
  Layout L{};
  size_t e = 0;
  for (int l = 0; l < NL; ++l) {
    L.w_off[l] = w_at(l);
    L.b_off[l] = b_at(l);
    L.t_off[l] = t_at(l);
  }
  L.n_par = e = b_at(NL - 1) + NOUT[NL - 1];
  const size_t t = L.n_wt = t_at(NL - 1) + (size_t)KIN[NL - 1] * NOUT[NL - 1];
  size_t o = 0;
  auto take = [&](size_t bytes) {
    size_t r = o;
    o = aup(o + std::max<size_t>(bytes, 1));
    return r;
  };
  L.off_p = take(4 * e);
  L.off_g = take(4 * e);
  L.off_m = take(4 * e);
  L.off_v = take(4 * e);
  L.off_wf = take(2 * t);
  L.off_wg = take(2 * t);
  L.off_wb = take(2 * t);
  L.off_xall = take(2 * 32 * (size_t)max_train);
  L.off_lab = take(4 * (size_t)max_train);
  L.off_traj = take(4 * NTRAJ * (size_t)max_train);
  L.off_perm = take(4 * (size_t)max_train);
  L.off_xb = take(2 * 32 * (size_t)max_batch);
  for (int l = 1; l < NL; ++l) L.off_act[l] = take(2 * 256 * (size_t)max_batch);
  for (int l = 0; l < NL; ++l) L.off_dz[l] = take(2 * (size_t)NOUT[l] * max_batch);
  L.off_acc = take(64);
  L.off_xin = take(4 * SRG_IN * (size_t)max_batch);
  L.off_yout = take(4 * SRG_OUT * (size_t)max_batch);
  L.total = o;
  return L;
}

uint16_t host_bf16(float f) {  // round to nearest even
  uint32_t u;
  memcpy(&u, &f, 4);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}
}  // namespace

constexpr int PIN_ROWS = 1024;

struct srg_ctx {
  hipStream_t stream;
  char* ws;
  Layout L;
  int max_batch, max_train, n_train = 0;
  int step = 0;  // Adam step count
  int err = 0;
  char msg[256];
  // pinned host rows that the kernel reads and writes itself, for small batches
  // in host arrays (PIN_ROWS inputs, then as many outputs); null where none was given
  float* pin = nullptr;
  float* pin_dev = nullptr;
  float* p() { return (float*)(ws + L.off_p); }
  float* g() { return (float*)(ws + L.off_g); }
  bf16* wf() { return (bf16*)(ws + L.off_wf); }
  bf16* wg() { return (bf16*)(ws + L.off_wg); }
  bf16* wb() { return (bf16*)(ws + L.off_wb); }
  bf16* xb() { return (bf16*)(ws + L.off_xb); }
  bf16* act(int l) { return (bf16*)(ws + L.off_act[l]); }
  bf16* dz(int l) { return (bf16*)(ws + L.off_dz[l]); }
  Weights weights() {
    Weights a;
    for (int l = 0; l < NL; ++l) {
      a.wf[l] = wf() + L.t_off[l];
      a.wg[l] = wg() + L.t_off[l];
      a.wb[l] = wb() + L.t_off[l];
      a.b[l] = p() + L.b_off[l];
    }
    return a;
  }
};

static int srg_err(srg_ctx* c, int code, const char* fmt, ...) {
  if (c && c->err == 0) {
    c->err = code;
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(c->msg, sizeof c->msg, fmt, ap);
    va_end(ap);
  }
  return code;
}

#define SCHK(ctx, call)                                                              \
  do {                                                                               \
    hipError_t e_ = (call);                                                          \
    if (e_ != hipSuccess)                                                            \
      return srg_err((ctx), LBM_EHIP, "%s failed: %s", #call, hipGetErrorString(e_)); \
  } while (0)

// more than 64 KB of dynamic LDS needs the attribute, once per kernel and device
static hipError_t allow_lds(const void* kernel, size_t bytes, unsigned long long* done) {
  int dev = 0;
  if (hipError_t e = hipGetDevice(&dev)) return e;
  if (dev < 64 && (__atomic_load_n(done, __ATOMIC_RELAXED) >> dev) & 1ull) return hipSuccess;
  hipError_t e =
      hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
  if (e == hipSuccess && dev < 64) __atomic_fetch_or(done, 1ull << dev, __ATOMIC_RELAXED);
  return e;
}

template <int RB, int RT, int CT, int AHEAD>
static hipError_t launch_mlp(srg_ctx* c, const float* X, int n, float* y) {
  static_assert(mlp_lds(RB) <= 64 * 1024, "no attribute needed");
  hipLaunchKernelGGL((k_mlp<RB, RT, CT, AHEAD>), dim3((n + 32 * RB - 1) / (32 * RB)),
                     dim3(64 * (RB / RT) * (8 / CT)), mlp_lds(RB), c->stream, X, n, c->weights(), y);
  return hipGetLastError();
}

// the pinned rows of a context; neither call disturbs a capture that this
// thread may have open on another stream
static void free_pin(float* pin) {
  if (!pin) return;
  hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
  (void)hipThreadExchangeStreamCaptureMode(&mode);
  (void)hipHostFree(pin);
  (void)hipThreadExchangeStreamCaptureMode(&mode);
}

static void alloc_pin(srg_ctx* c) {
  hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
  (void)hipThreadExchangeStreamCaptureMode(&mode);
  void *pin = nullptr, *dev = nullptr;
  bool ok = hipHostMalloc(&pin, sizeof(float) * PIN_ROWS * (SRG_IN + SRG_OUT),
                          hipHostMallocDefault) == hipSuccess;
  if (ok && hipHostGetDevicePointer(&dev, pin, 0) != hipSuccess) {
    (void)hipHostFree(pin);
    ok = false;
  }
  (void)hipThreadExchangeStreamCaptureMode(&mode);
  if (ok) {
    c->pin = (float*)pin;
    c->pin_dev = (float*)dev;
  } else {
    (void)hipGetLastError();  // small host batches are copied then
  }
}

// inference over n rows of FP32 inputs X (n x 6) to y (n x 51), both visible to
// the device: the whole pass in one kernel, the activations in LDS
static int infer(srg_ctx* c, const float* X, int n, float* y) {
  if (n <= MLP_ROWS_32)
    SCHK(c, (launch_mlp<1, 1, 1, 4>(c, X, n, y)));
  else if (n <= MLP_ROWS_64)
    SCHK(c, (launch_mlp<2, 2, 1, 4>(c, X, n, y)));
  else
    SCHK(c, (launch_mlp<4, 4, 1, 2>(c, X, n, y)));
  return LBM_OK;
}

// one batch up to the gradients of the pre-activations: B rows of X (packed
// inputs), row perm[off + r] of it (perm null: row r) as batch row r
static int row_pass(srg_ctx* c, const bf16* X, const int* perm, int off, int B, const int* lab,
                    const float* traj, float w_traj, float* loss) {
  RowArgs g{};
  g.X = X;
  g.perm = perm;
  g.off = off;
  g.lab = lab;
  g.traj = traj;
  g.w_traj = w_traj;
  g.inv_B = 1.0f / (float)B;
  g.w = c->weights();
  g.xb = c->xb();
  for (int l = 0; l < NL; ++l) {
    g.act[l] = l ? c->act(l) : nullptr;
    g.dz[l] = c->dz(l);
  }
  g.loss = loss;
  static unsigned long long done[2] = {0, 0};
  if (B % 128 == 0) {
    SCHK(c, allow_lds((const void*)k_train_rows<true>, ROW_LDS, &done[0]));
    hipLaunchKernelGGL(k_train_rows<true>, dim3(B / 32), dim3(512), ROW_LDS, c->stream, g);
  } else {
    SCHK(c, allow_lds((const void*)k_train_rows<false>, ROW_LDS, &done[1]));
    hipLaunchKernelGGL(k_train_rows<false>, dim3(B / 32), dim3(512), ROW_LDS, c->stream, g);
  }
  SCHK(c, hipGetLastError());
  return LBM_OK;
}

// the gradients of the parameters into the gradient vector, or (apply) Adam
static int weight_pass(srg_ctx* c, int B, bool apply, float lr) {
  WeightArgs g{};
  g.x = c->xb();
  for (int l = 0; l < NL; ++l) {
    g.act[l] = l ? c->act(l) : nullptr;
    g.dz[l] = c->dz(l);
  }
  g.B = B;
  g.p = c->p();
  g.m = (float*)(c->ws + c->L.off_m);
  g.v = (float*)(c->ws + c->L.off_v);
  g.g = c->g();
  g.wf = c->wf();
  g.wg = c->wg();
  g.wb = c->wb();
  g.lr = lr;
  if (apply) {
    ++c->step;
    g.bc1 = 1.f - powf(0.9f, (float)c->step);
    g.bc2 = 1.f - powf(0.999f, (float)c->step);
    hipLaunchKernelGGL(k_train_weights<true>, dim3(W_TILES + B_TILES), dim3(256), 0, c->stream, g);
  } else {
    hipLaunchKernelGGL(k_train_weights<false>, dim3(W_TILES + B_TILES), dim3(256), 0, c->stream, g);
  }
  SCHK(c, hipGetLastError());
  return LBM_OK;
}

// the fragment copies of all weights
static int pack_weights(srg_ctx* c) {
  for (int l = 0; l < NL; ++l) {
    const int n = KIN[l] * NOUT[l];
    const size_t o = c->L.t_off[l];
    hipLaunchKernelGGL(k_pack, dim3((n + 255) / 256), dim3(256), 0, c->stream,
                       c->p() + c->L.w_off[l], KIN[l], NOUT[l], c->wf() + o, c->wg() + o,
                       c->wb() + o);
  }
  SCHK(c, hipGetLastError());
  return LBM_OK;
}

extern "C" {

size_t srg_workspace_bytes(int32_t max_batch, int32_t max_train) {
  if (max_batch < 64 || max_batch % 64 != 0 || max_train < 0) return 0;
  return make_layout(max_batch, max_train).total;
}

int srg_create(void* dev_workspace, size_t ws_bytes, int32_t max_batch, int32_t max_train,
               void* hip_stream, srg_ctx** out) {
  if (!out) return LBM_EINVAL;
  *out = nullptr;
  const size_t need = srg_workspace_bytes(max_batch, max_train);
  if (need == 0 || !dev_workspace) return LBM_EINVAL;
  if (ws_bytes < need) return LBM_ENOMEM;
  if (((uintptr_t)dev_workspace) % ALIGN != 0) return LBM_EINVAL;
  srg_ctx* c = new (std::nothrow) srg_ctx();
  if (!c) return LBM_ENOMEM;
  c->stream = (hipStream_t)hip_stream;
  c->ws = (char*)dev_workspace;
  c->L = make_layout(max_batch, max_train);
  c->max_batch = max_batch;
  c->max_train = max_train;
  c->msg[0] = 0;
  *out = c;
  // zero parameters, gradients, moments (padding stays zero forever)
  SCHK(c, hipMemsetAsync(c->ws, 0, c->L.off_xall, c->stream));
  alloc_pin(c);
  SCHK(c, hipStreamSynchronize(c->stream));
  return LBM_OK;
}

int srg_set_params(srg_ctx* c, const float* params) {
  if (!c || !params) return LBM_EINVAL;
  if (c->err) return LBM_ESTATE;
  std::vector<float> pad(c->L.n_par, 0.f);
  size_t k = 0;
  for (int l = 0; l < NL; ++l) {
    for (int i = 0; i < KREAL[l]; ++i)
      for (int j = 0; j < NREAL[l]; ++j) pad[c->L.w_off[l] + (size_t)i * NOUT[l] + j] = params[k++];
    for (int j = 0; j < NREAL[l]; ++j) pad[c->L.b_off[l] + j] = params[k++];
  }
  const size_t nb = 4 * c->L.n_par;
  SCHK(c, hipMemcpyAsync(c->p(), pad.data(), nb, hipMemcpyHostToDevice, c->stream));
  SCHK(c, hipMemsetAsync(c->ws + c->L.off_m, 0, nb, c->stream));
  SCHK(c, hipMemsetAsync(c->ws + c->L.off_v, 0, nb, c->stream));
  if (int rc = pack_weights(c)) return rc;
  c->step = 0;
  SCHK(c, hipStreamSynchronize(c->stream));
  return LBM_OK;
}

static void unpad(const srg_ctx* c, const std::vector<float>& pad, float* out) {
  size_t k = 0;
  for (int l = 0; l < NL; ++l) {
    for (int i = 0; i < KREAL[l]; ++i)
      for (int j = 0; j < NREAL[l]; ++j) out[k++] = pad[c->L.w_off[l] + (size_t)i * NOUT[l] + j];
    for (int j = 0; j < NREAL[l]; ++j) out[k++] = pad[c->L.b_off[l] + j];
  }
}

int srg_get_params(srg_ctx* c, float* params) {
  if (!c || !params) return LBM_EINVAL;
  if (c->err) return LBM_ESTATE;
  std::vector<float> pad(c->L.n_par);
  SCHK(c, hipMemcpyAsync(pad.data(), c->p(), 4 * c->L.n_par, hipMemcpyDeviceToHost, c->stream));
  SCHK(c, hipStreamSynchronize(c->stream));
  unpad(c, pad, params);
  return LBM_OK;
}

static int upload_set(srg_ctx* c, const float* X, const int32_t* label, const float* traj, int n,
                      size_t off_x, size_t off_lab, size_t off_traj) {
  std::vector<uint16_t> xb((size_t)n * 32, 0);
  for (int r = 0; r < n; ++r)
    for (int j = 0; j < SRG_IN; ++j) xb[(size_t)r * 32 + j] = host_bf16(X[(size_t)r * SRG_IN + j]);
  SCHK(c, hipMemcpyAsync(c->ws + off_x, xb.data(), 2 * xb.size(), hipMemcpyHostToDevice, c->stream));
  if (label)
    SCHK(c, hipMemcpyAsync(c->ws + off_lab, label, 4 * (size_t)n, hipMemcpyHostToDevice, c->stream));
  if (traj)
    SCHK(c, hipMemcpyAsync(c->ws + off_traj, traj, 4 * (size_t)NTRAJ * n, hipMemcpyHostToDevice,
                           c->stream));
  SCHK(c, hipStreamSynchronize(c->stream));
  return LBM_OK;
}

int srg_set_train(srg_ctx* c, const float* X, const int32_t* label, const float* traj, int32_t n) {
  if (!c || !X || !label || !traj || n < 1) return LBM_EINVAL;
  if (c->err) return LBM_ESTATE;
  if (n > c->max_train) return srg_err(c, LBM_ERANGE, "training set larger than max_train");
  for (int i = 0; i < n; ++i)
    if (label[i] < 0 || label[i] >= NCLS) return srg_err(c, LBM_EINVAL, "label out of range");
  int rc = upload_set(c, X, label, traj, n, c->L.off_xall, c->L.off_lab, c->L.off_traj);
  if (rc) return rc;
  c->n_train = n;
  return LBM_OK;
}

int srg_train(srg_ctx* c, int32_t epochs, int32_t batch, float lr, float w_traj, uint64_t seed,
              float* epoch_loss) {
  if (!c) return LBM_EINVAL;
  if (c->err) return LBM_ESTATE;
  if (epochs < 0 || batch < 64 || batch % 64 != 0 || batch > c->max_batch || batch > c->n_train)
    return srg_err(c, LBM_EINVAL, "batch must be a multiple of 64, <= max_batch and the set size");
  const int n = c->n_train, nb = n / batch;
  std::mt19937_64 rng(seed);
  std::vector<int> perm(n);
  float* acc = (float*)(c->ws + c->L.off_acc);
  int* dperm = (int*)(c->ws + c->L.off_perm);
  for (int e = 0; e < epochs; ++e) {
    for (int i = 0; i < n; ++i) perm[i] = i;
    std::shuffle(perm.begin(), perm.end(), rng);
    SCHK(c, hipMemcpyAsync(dperm, perm.data(), 4 * (size_t)n, hipMemcpyHostToDevice, c->stream));
    SCHK(c, hipMemsetAsync(acc, 0, 4, c->stream));
    for (int b = 0; b < nb; ++b) {
      int rc = row_pass(c, (const bf16*)(c->ws + c->L.off_xall), dperm, b * batch, batch,
                        (const int*)(c->ws + c->L.off_lab), (const float*)(c->ws + c->L.off_traj),
                        w_traj, acc);
      if (rc) return rc;
      rc = weight_pass(c, batch, true, lr);
      if (rc) return rc;
    }
    float s = 0.f;
    SCHK(c, hipMemcpyAsync(&s, acc, 4, hipMemcpyDeviceToHost, c->stream));
    SCHK(c, hipStreamSynchronize(c->stream));
    if (epoch_loss) epoch_loss[e] = nb > 0 ? s / nb : 0.f;
  }
  return LBM_OK;
}

int srg_gradients(srg_ctx* c, const float* X, const int32_t* label, const float* traj, int32_t n,
                  float w_traj, float* grads, float* loss) {
  if (!c || !X || !label || !traj || !grads) return LBM_EINVAL;
  if (c->err) return LBM_ESTATE;
  if (n < 64 || n % 64 != 0 || n > c->max_batch)
    return srg_err(c, LBM_EINVAL, "n must be a multiple of 64 and <= max_batch");
  for (int i = 0; i < n; ++i)
    if (label[i] < 0 || label[i] >= NCLS) return srg_err(c, LBM_EINVAL, "label out of range");
  // the batch goes through the training-set buffers' batch slots: inputs in
  // Xb, labels and trajectories in the (batch-sized) prefix of dedicated rows
  std::vector<uint16_t> xb((size_t)n * 32, 0);
  for (int r = 0; r < n; ++r)
    for (int j = 0; j < SRG_IN; ++j) xb[(size_t)r * 32 + j] = host_bf16(X[(size_t)r * SRG_IN + j]);
  bf16* Xb = (bf16*)(c->ws + c->L.off_xb);
  SCHK(c, hipMemcpyAsync(Xb, xb.data(), 2 * xb.size(), hipMemcpyHostToDevice, c->stream));
  // labels and trajectories staged in the FP32 output buffer region of the
  // inference path (sized max_batch x 51 floats >= n x 49)
  int* dlab = (int*)(c->ws + c->L.off_yout);
  float* dtr = (float*)(c->ws + c->L.off_yout) + n;
  SCHK(c, hipMemcpyAsync(dlab, label, 4 * (size_t)n, hipMemcpyHostToDevice, c->stream));
  SCHK(c, hipMemcpyAsync(dtr, traj, 4 * (size_t)NTRAJ * n, hipMemcpyHostToDevice, c->stream));
  float* acc = (float*)(c->ws + c->L.off_acc);
  SCHK(c, hipMemsetAsync(acc, 0, 4, c->stream));
  int rc = row_pass(c, Xb, nullptr, 0, n, dlab, dtr, w_traj, acc);
  if (rc) return rc;
  rc = weight_pass(c, n, false, 0.f);
  if (rc) return rc;
  std::vector<float> pad(c->L.n_par);
  SCHK(c, hipMemcpyAsync(pad.data(), c->g(), 4 * c->L.n_par, hipMemcpyDeviceToHost, c->stream));
  float s = 0.f;
  SCHK(c, hipMemcpyAsync(&s, acc, 4, hipMemcpyDeviceToHost, c->stream));
  SCHK(c, hipStreamSynchronize(c->stream));
  unpad(c, pad, grads);
  if (loss) *loss = s;
  return LBM_OK;
}

int srg_predict(srg_ctx* c, const float* X, int32_t n, float* y, int32_t src_is_device,
                int32_t dst_is_device) {
  if (!c || !X || !y || n < 1) return LBM_EINVAL;
  if (c->err) return LBM_ESTATE;
  if (c->pin && !src_is_device && !dst_is_device && n <= PIN_ROWS) {
    // a copy each way costs more than the rows: the kernel takes them from pinned
    // memory and leaves the outputs there (256 rows 53 us with the copies, 27 so)
    const size_t in = (size_t)SRG_IN * PIN_ROWS;
    memcpy(c->pin, X, sizeof(float) * SRG_IN * (size_t)n);
    if (int rc = infer(c, c->pin_dev, n, c->pin_dev + in)) return rc;
    SCHK(c, hipStreamSynchronize(c->stream));
    memcpy(y, c->pin + in, sizeof(float) * SRG_OUT * (size_t)n);
    return LBM_OK;
  }
  float* xin = (float*)(c->ws + c->L.off_xin);
  float* yout = (float*)(c->ws + c->L.off_yout);
  for (int r0 = 0; r0 < n; r0 += c->max_batch) {
    const int m = std::min(c->max_batch, n - r0);
    const float* src = X + (size_t)r0 * SRG_IN;
    if (!src_is_device) {
      SCHK(c, hipMemcpyAsync(xin, src, 4 * (size_t)SRG_IN * m, hipMemcpyHostToDevice, c->stream));
      src = xin;
    }
    float* dst = dst_is_device ? y + (size_t)r0 * SRG_OUT : yout;
    int rc = infer(c, src, m, dst);
    if (rc) return rc;
    if (!dst_is_device) {
      SCHK(c, hipMemcpyAsync(y + (size_t)r0 * SRG_OUT, yout, 4 * (size_t)SRG_OUT * m,
                             hipMemcpyDeviceToHost, c->stream));
      SCHK(c, hipStreamSynchronize(c->stream));
    }
  }
  if (!src_is_device) SCHK(c, hipStreamSynchronize(c->stream));
  return LBM_OK;
}

int srg_sync(srg_ctx* c) {
  if (!c) return LBM_EINVAL;
  if (c->err) return LBM_ESTATE;
  SCHK(c, hipStreamSynchronize(c->stream));
  return LBM_OK;
}

void srg_destroy(srg_ctx* c) {
  if (!c) return;
  (void)hipStreamSynchronize(c->stream);
  free_pin(c->pin);
  delete c;
}

const char* srg_last_error(const srg_ctx* c) {
  if (!c || c->err == 0) return nullptr;
  return c->msg;
}

}  // extern "C"
