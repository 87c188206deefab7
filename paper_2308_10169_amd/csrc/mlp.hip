// Learned initializer (device code): occupancy raster of each instance's
// map, a BF16 MLP (FP32 accumulation on gfx950 MFMA) that proposes one
// initial path per group, its MSE backward pass and Adam with FP32 master
// weights.  GEMMs run on v_mfma_f32_16x16x32_bf16.
#include "common.h"
#include "mlp.h"

namespace sepso {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// FP32 -> BF16, round to nearest even (finite inputs).
__device__ __forceinline__ uint16_t to_bf16(float f) {
  const uint32_t u = __float_as_uint(f);
  const uint32_t r = u + 0x7FFFu + ((u >> 16) & 1u);
  return (uint16_t)(r >> 16);
}
__device__ __forceinline__ float from_bf16(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

// ---------------------------------------------------------------------------
// Input features of instance i (row i of X): 64 x 64 occupancy (cell centre
// inside any obstacle polygon, even-odd rule) followed by start and target
// normalised by the map size; zero padding up to kLinInPad.  An edge is read
// once for a thread's sixteen cells (once per cell it was a chain of scalar
// loads): 256 instances of 4 rectangles 39 -> 14 us.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void raster_kernel(Pools pl, uint16_t* X, int ldx,
                                                     int32_t* eligible) {
  const int inst = blockIdx.x;
  const InstDesc& d = pl.desc[inst];
  const float2* verts = pl.verts + d.eo;
  const int32_t* pp = pl.poly_ptr + d.plo;
  uint16_t* row = X + (int64_t)inst * ldx;
  // a thread's cells are one column's, every fourth row: bit i of a word is
  // row r0 + 4 i
  constexpr int kCells = kRaster * kRaster / 256;
  const int c = threadIdx.x % kRaster, r0 = threadIdx.x / kRaster;
  const float px = (c + 0.5f) * d.width / kRaster;
  uint32_t inside = 0;
  for (int q = 0; q < d.n_polys; ++q) {
    const int v0 = pp[q], m = pp[q + 1] - v0;
    uint32_t odd = 0;
    for (int j = 0; j < m; ++j) {
      const float2 a = verts[v0 + j], b = verts[v0 + (j + 1 == m ? 0 : j + 1)];
#pragma unroll
      for (int i = 0; i < kCells; ++i) {
        const float py = (r0 + 4 * i + 0.5f) * d.height / kRaster;
        if ((a.y > py) != (b.y > py)) {  // the same for a whole wave
          const float xc = a.x + (py - a.y) * (b.x - a.x) / (b.y - a.y);
          if (px < xc) odd ^= 1u << i;
        }
      }
    }
    inside |= odd;
  }
#pragma unroll
  for (int i = 0; i < kCells; ++i) row[(r0 + 4 * i) * kRaster + c] = inside >> i & 1 ? 0x3F80 : 0;  // 1.0 or 0.0
  if (threadIdx.x < kLinInPad - kRaster * kRaster) {
    const int j = threadIdx.x;
    const float4 e = pl.ends[inst];
    float v = 0.f;
    if (j == 0) v = e.x / d.width;
    if (j == 1) v = e.y / d.height;
    if (j == 2) v = e.z / d.width;
    if (j == 3) v = e.w / d.height;
    row[kRaster * kRaster + j] = to_bf16(v);
  }
  if (threadIdx.x == 0) eligible[inst] = (d.G == kLinGroups && d.W == kLinW) ? 1 : 0;
}

// The epilogue of NI x NJ groups of four consecutive FP32 results: group
// (i, j) is C(row + 16 i, col + 16 j .. + 3).  What it reads is loaded for all
// groups before the first is finished; groups outside M x N read C(0, 0)'s and
// are not stored.
template <int NI, int NJ>
__device__ __forceinline__ void apply_epi(const Epi& ep, int M, int N, int row, int col, f32x4 (&v)[NI][NJ]) {
  auto in = [&](int i, int j) { return row + 16 * i < M && col + 16 * j < N; };
  auto at = [&](int i, int j) { return (int64_t)(row + 16 * i) * ep.ldo + col + 16 * j; };
  auto pack = [](const f32x4& x) {
    return make_uint2(to_bf16(x[0]) | (uint32_t)to_bf16(x[1]) << 16, to_bf16(x[2]) | (uint32_t)to_bf16(x[3]) << 16);
  };
#define EACH                     \
  _Pragma("unroll") for (int i = 0; i < NI; ++i) _Pragma("unroll") for (int j = 0; j < NJ; ++j)
  if (ep.mode == EPI_MASK) {
    typedef uint16_t u16x4 __attribute__((ext_vector_type(4)));
    u16x4 m[NI][NJ];
    EACH m[i][j] = *reinterpret_cast<const u16x4*>(ep.mask + (in(i, j) ? at(i, j) : 0));
    EACH if (in(i, j)) {
      f32x4 x = v[i][j];
#pragma unroll
      for (int r = 0; r < 4; ++r) x[r] = from_bf16(m[i][j][r]) > 0.f ? x[r] : 0.f;
      *reinterpret_cast<f32x4*>(ep.out_f32 + at(i, j)) = x;
      *reinterpret_cast<uint2*>(ep.out_bf16 + at(i, j)) = pack(x);
    }
    return;
  }
  f32x4 bias[NJ];
#pragma unroll
  for (int j = 0; j < NJ; ++j) bias[j] = *reinterpret_cast<const f32x4*>(ep.bias + (in(0, j) ? col + 16 * j : 0));
  if (ep.mode == EPI_BIAS_RELU_BF16) {
    EACH if (in(i, j)) {
      f32x4 x = v[i][j] + bias[j];
#pragma unroll
      for (int r = 0; r < 4; ++r) x[r] = x[r] > 0.f ? x[r] : 0.f;
      *reinterpret_cast<uint2*>(ep.out_bf16 + at(i, j)) = pack(x);
    }
  } else if (ep.mode == EPI_BIAS_F32) {
    EACH if (in(i, j)) *reinterpret_cast<f32x4*>(ep.out_f32 + at(i, j)) = v[i][j] + bias[j];
  } else {  // EPI_BIAS_LOSS: also dy = 2 (y - target) / (rows * columns) in BF16
    f32x4 tg[NI][NJ];
    EACH tg[i][j] = *reinterpret_cast<const f32x4*>(ep.target + (in(i, j) ? at(i, j) : 0));
    EACH if (in(i, j)) {
      const f32x4 y = v[i][j] + bias[j];
      *reinterpret_cast<f32x4*>(ep.out_f32 + at(i, j)) = y;
      *reinterpret_cast<uint2*>(ep.out_bf16 + at(i, j)) = pack(ep.scale * (y - tg[i][j]));
    }
  }
#undef EACH
}

// Blocks of a launch go to the eight XCDs in turn.  The place of block L in an
// order that gives every XCD one contiguous stretch of it, so that the tiles
// that read the same operand rows, neighbours in that order, share an L2.
__device__ __forceinline__ int xcd_order(int L, int n) {
  const int x = L & 7;
  return x * (n >> 3) + min(x, n & 7) + (L >> 3);
}

// ---------------------------------------------------------------------------
// C[M x N] = A[M x K] * B[N x K]^T, BF16 in (k contiguous in both), FP32
// accumulate; K % 32 == 0, N % 32 == 0.  The sum over k is taken in slices of
// kper MFMA steps of 32, each from zero, and the slices are added in order:
// the accumulators of a finished slice go to the running total in registers,
// so that no slice goes through memory and the epilogue follows in the same
// launch.  The products are taken as B A^T, which leaves a lane with four
// consecutive columns of one row.
//
// gemm_small_kernel: few rows and a short K.  What bounds it is one block's
// chain of latencies, so a block takes a 32 x 32 tile and its eight waves a
// slice each, operands straight from memory to registers (two steps' loads in
// flight, no barrier), the slices meeting in LDS once at the end.  256 rows x
// 512 x 512: 4.4 us a launch (64 x 64 tiles through LDS, a slice per block and
// a second launch adding them up: 11.5; gemm_nt_kernel's 64 x 64: 5.6).
// ---------------------------------------------------------------------------
constexpr int kSmallWaves = 8;
constexpr int kSmallPitch = 36;  // floats per row of a partial tile in LDS

__global__ __launch_bounds__(64 * kSmallWaves) void gemm_small_kernel(const uint16_t* __restrict__ A, int lda,
                                                                      const uint16_t* __restrict__ B, int ldb,
                                                                      int M, int N, int steps, int kper, int S,
                                                                      Epi ep) {
  __shared__ __attribute__((aligned(16))) float s_part[kSmallWaves * 32 * kSmallPitch];
  const int t = threadIdx.x, lane = t & 63, w = __builtin_amdgcn_readfirstlane(t >> 6);
  const int r16 = lane & 15, kq = (lane >> 4) * 8;
  const int idx = xcd_order(blockIdx.x, gridDim.x), tn = N / 32;
  const int m0 = idx / tn * 32, n0 = (idx - idx / tn * tn) * 32;
  const uint16_t *pa[2], *pb[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {  // rows past M read row M - 1 and are not stored
    pa[i] = A + (int64_t)min(m0 + i * 16 + r16, M - 1) * lda + kq;
    pb[i] = B + (int64_t)(n0 + i * 16 + r16) * ldb + kq;
  }
  f32x4 acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  constexpr int U = 2;
  const int beg = w * kper, end = min(steps, beg + kper);  // S <= kSmallWaves; waves past it find nothing
  for (int k = beg; k < end; k += U) {
    bf16x8 a[U][2], b[U][2];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int kk = 32 * min(k + u, end - 1);
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        a[u][i] = *reinterpret_cast<const bf16x8*>(pa[i] + kk);
        b[u][i] = *reinterpret_cast<const bf16x8*>(pb[i] + kk);
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (k + u < end) {
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int j = 0; j < 2; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[u][j], a[u][i], acc[i][j], 0, 0, 0);
      }
  }
  // D layout: lane holds row (lane % 16), columns 4*(lane/16) .. +3
  if (w < S) {
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j)
        *reinterpret_cast<f32x4*>(&s_part[(w * 32 + i * 16 + r16) * kSmallPitch + j * 16 + (lane >> 4) * 4]) = acc[i][j];
  }
  __syncthreads();
  if (t < 256) {
    const float* p = s_part + (t >> 3) * kSmallPitch + (t & 7) * 4;
    f32x4 v[1][1] = {{*reinterpret_cast<const f32x4*>(p)}};
    for (int z = 1; z < S; ++z) v[0][0] += *reinterpret_cast<const f32x4*>(p + z * 32 * kSmallPitch);
    apply_epi<1, 1>(ep, M, N, m0 + (t >> 3), n0 + (t & 7) * 4, v);
  }
}

// The same product on BM x BN tiles through LDS, one wave per WM x WN: k-steps
// of 64 in three LDS buffers, one barrier per step; each half step's operand
// reads are issued ahead of the other half's MFMAs, and the next step but one
// goes to LDS in between, from registers that its loads had two steps to
// reach.  A row's eight 16-byte chunks are permuted by the row's low three
// bits, so that stores and operand reads spread over all banks without
// padding (no conflicts counted).
// What bounds it is LDS: at 128 x 128 a step's operand reads (96 KB at 256 B a
// cycle) and stores (32 KB, half that rate or less) take longer than its
// MFMAs; loads from memory are hidden (37.4 us against 36 with every row the
// same one).  8192 x 512 x 4128: 73.8 + 7.4 us (two slices added up by a second
// launch) -> 43 us in a training step, 37 by itself (930 TFLOP/s); 8192 x 512
// x 512: 17 -> 12 us.
template <int BM, int BN, int WM, int WN, int D = 2>
__global__ __launch_bounds__(64 * (BM / WM) * (BN / WN)) void gemm_nt_kernel(
    const uint16_t* __restrict__ A, int lda, const uint16_t* __restrict__ B, int ldb, int M, int N, int steps,
    int kper, Epi ep) {
  static_assert(D >= 2 && 6 % D == 0, "the loop takes six steps");
  constexpr int T = 64 * (BM / WM) * (BN / WN), NI = WM / 16, NJ = WN / 16;
  constexpr int CA = (BM * 8 + T - 1) / T, CB = BN * 8 / T;  // 16-byte chunks per thread and step
  __shared__ __attribute__((aligned(16))) uint16_t s_t[3][(BM + BN) * 64];
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const int tn = (N + BN - 1) / BN, idx = xcd_order(blockIdx.x, gridDim.x);
  const int m0 = idx / tn * BM, n0 = (idx - idx / tn * tn) * BN;
  const int wm = w / (BN / WN) * WM, wn = w % (BN / WN) * WN;
  const int r16 = lane & 15, kg = lane >> 4;
  const int tr = t >> 3, tc = t & 7;  // row (of T / 8 at a time) and chunk this thread carries
  struct Stage {
    u32x4 a[CA], b[CB];
  } r[D];
  auto fetch = [&](Stage& f, int k) {  // k: MFMA step; the second half of a last odd step is not used
    // (past the end: the last stage again, not used)
    const bool whole = k + 1 < steps;
    const int kk = 32 * (whole ? k : steps - 1) + (whole ? tc : tc & 3) * 8;
#pragma unroll
    for (int c = 0; c < CA; ++c)
      f.a[c] = *reinterpret_cast<const u32x4*>(A + (int64_t)min(m0 + tr + c * (T / 8), M - 1) * lda + kk);
#pragma unroll
    for (int c = 0; c < CB; ++c)
      f.b[c] = *reinterpret_cast<const u32x4*>(B + (int64_t)min(n0 + tr + c * (T / 8), N - 1) * ldb + kk);
  };
  auto stash_a = [&](const Stage& f, uint16_t* s) {
#pragma unroll
    for (int c = 0; c < CA; ++c) {
      const int row = tr + c * (T / 8);
      if (BM * 8 % T == 0 || row < BM)  // whole waves
        *reinterpret_cast<u32x4*>(s + row * 64 + ((tc ^ (row & 7)) << 3)) = f.a[c];
    }
  };
  auto stash_b = [&](const Stage& f, uint16_t* s) {
#pragma unroll
    for (int c = 0; c < CB; ++c) {
      const int row = tr + c * (T / 8);
      *reinterpret_cast<u32x4*>(s + (BM + row) * 64 + ((tc ^ (row & 7)) << 3)) = f.b[c];
    }
  };
  f32x4 acc[NI][NJ], tot[NI][NJ];
#pragma unroll
  for (int i = 0; i < NI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int i = 0; i < NI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j) tot[i][j] = f32x4{-0.f, -0.f, -0.f, -0.f};  // + x is x, whatever x
  int left = kper;  // steps left of the current slice
  auto end_slice = [&]() {
    left = kper;
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        tot[i][j] += acc[i][j];
        acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
      }
  };
#pragma unroll
  for (int c = 0; c < 2; ++c) fetch(r[c], 2 * c);
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    stash_a(r[c], s_t[c]);
    stash_b(r[c], s_t[c]);
  }
#pragma unroll
  for (int c = 0; c < D; ++c) fetch(r[c], 4 + 2 * c);
  __syncthreads();
  auto frag = [&](const uint16_t* s, int row, int h) {
    return *reinterpret_cast<const bf16x8*>(s + row * 64 + (((4 * h + kg) ^ (row & 7)) << 3));
  };
  bf16x8 a[2][NI], b[2][NJ];
  auto read = [&](const uint16_t* s, int h) {
#pragma unroll
    for (int i = 0; i < NI; ++i) a[h][i] = frag(s, wm + i * 16 + r16, h);
#pragma unroll
    for (int j = 0; j < NJ; ++j) b[h][j] = frag(s, BM + wn + j * 16 + r16, h);
  };
  auto product = [&](int h) {
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
      for (int j = 0; j < NJ; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[h][j], a[h][i], acc[i][j], 0, 0, 0);
    if (--left == 0) end_slice();
  };
  read(s_t[0], 0);
  // The 64 k from step k on, in buffer s0, their first half's operands read; s1
  // holds the next 64, f those after it, which go to s2.  At the barrier every
  // wave has read what it needs of s0 and, a step ago, stored its part of s1.
  auto step = [&](int k, const uint16_t* s0, const uint16_t* s1, uint16_t* s2, Stage& f) {
    read(s0, 1);
    stash_a(f, s2);
    if (k < steps) product(0);
    __syncthreads();
    read(s1, 0);
    stash_b(f, s2);
    if (k + 1 < steps) product(1);
    fetch(f, k + 4 + 2 * D);
  };
  for (int k0 = 0; k0 < steps; k0 += 12) {
#pragma unroll
    for (int c = 0; c < 6; ++c)
      step(k0 + 2 * c, s_t[c % 3], s_t[(c + 1) % 3], s_t[(c + 2) % 3], r[c % D]);
  }
  if (left < kper) end_slice();
  apply_epi<NI, NJ>(ep, M, N, m0 + wm + r16, n0 + wn + kg * 4, tot);
}

// One Adam step of one parameter (the fused multiply-adds written out).
__device__ __forceinline__ float adam_one(const AdamStep& a, float p, float& m, float& v, float g) {
  m = fmaf(1.f - a.b1, g, a.b1 * m);
  v = fmaf(g, (1.f - a.b2) * g, a.b2 * v);
  return p - a.lr * (m / a.c1) / (sqrtf(v / a.c2) + a.eps);
}

// ---------------------------------------------------------------------------
// Weight gradients of all four layers, dW = dZ^T In (sum over the batch's
// rows k), with the Adam step in the epilogue where a.adam.on; the same launch
// also takes the bias gradients' partial column sums and the loss's row sums,
// which read what these products' operands came from.
//
// Both operands have k as their slow index; they go to LDS as they lie and the
// transposing LDS reads hand each lane its eight consecutive k.  A row's
// 32-byte units are permuted by bits of k such that the sixteen rows one such
// read touches spread over all banks.  Steps, buffers and the slices of the
// sum over k are those of gemm_nt_kernel.
//
// Large batches are bound by the steps as there (0.54 us per 64 k, one block
// of eight waves on 176 of the CUs), small ones by the optimizer state's 73 MB
// (10 of the 20 us at 256 rows).  8192 rows: 209 us (four products of which
// three with a second launch for their slices, eight launches of column sums,
// two of the loss, and Adam's) -> 99-109 in a training step, 95 by itself; 256
// rows: 100 -> 21 us.
// ---------------------------------------------------------------------------
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));

// Halves offset of 16-byte chunk c of row k in a tile of P columns.
template <int P>
__device__ __forceinline__ int dw_at(int k, int c) {
  const int perm = P == 64 ? ((k >> 1) & 1) | ((k >> 2) & 2) : (k & 3) | ((k >> 1) & 4);
  return k * P + ((c ^ 2 * perm) << 3);
}

// Eight consecutive k (from row k0 + 8 kg) of column 16 unit + lane % 16.
template <int P>
__device__ __forceinline__ bf16x8 dw_frag(const uint16_t* s, int k0, int unit, int lane) {
  const int row = k0 + (lane >> 4) * 8 + ((lane & 15) >> 2);
  auto read = [&](int k) {
    const uint16_t* q = s + dw_at<P>(k, 2 * unit) + (lane & 3) * 4;
    return __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)q);
  };
  const s16x4 lo = read(row), hi = read(row + 4);
  return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
}

template <int BM, int BN, int WM, int WN>
__device__ __forceinline__ void dw_tile(const DwSet& d, int tile, int K, const AdamStep& ad, uint16_t* s_t) {
  constexpr int T = 64 * (BM / WM) * (BN / WN), NI = WM / 16, NJ = WN / 16;
  constexpr int LA = BM / 8, LB = BN / 8;                // 16-byte chunks per row of k
  constexpr int CA = 64 * LA / T, CB = 64 * LB / T;      // and per thread and step
  constexpr int kBuf = 64 * (BM + BN);                   // halves: 64 rows of A, then of B
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const int tm = (d.M + BM - 1) / BM, n0 = tile / tm * BN, m0 = (tile - tile / tm * tm) * BM;
  const int wm = w / (BN / WN) * WM, wn = w % (BN / WN) * WN;
  const int r16 = lane & 15, kg = lane >> 4, steps = K / 32;
  struct Stage {
    u32x4 a[CA], b[CB];
  } r[2];
  const int ac = t % LA, ar = t / LA, bc = t % LB, br = t / LB;
  const uint16_t* pa = d.A + (m0 + ac * 8 < d.M ? m0 + ac * 8 : 0);  // columns past M (N): any, not stored
  const uint16_t* pb = d.B + (n0 + bc * 8 < d.N ? n0 + bc * 8 : 0);
  auto fetch = [&](Stage& f, int k) {  // rows past K: the last, not used
#pragma unroll
    for (int c = 0; c < CA; ++c)
      f.a[c] = *reinterpret_cast<const u32x4*>(pa + (int64_t)min(32 * k + ar + T / LA * c, K - 1) * d.M);
#pragma unroll
    for (int c = 0; c < CB; ++c)
      f.b[c] = *reinterpret_cast<const u32x4*>(pb + (int64_t)min(32 * k + br + T / LB * c, K - 1) * d.ldb);
  };
  auto stash_a = [&](const Stage& f, uint16_t* s) {
#pragma unroll
    for (int c = 0; c < CA; ++c) *reinterpret_cast<u32x4*>(s + dw_at<BM>(ar + T / LA * c, ac)) = f.a[c];
  };
  auto stash_b = [&](const Stage& f, uint16_t* s) {
#pragma unroll
    for (int c = 0; c < CB; ++c) *reinterpret_cast<u32x4*>(s + 64 * BM + dw_at<BN>(br + T / LB * c, bc)) = f.b[c];
  };
  f32x4 acc[NI][NJ], tot[NI][NJ];
#pragma unroll
  for (int i = 0; i < NI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int i = 0; i < NI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j) tot[i][j] = f32x4{-0.f, -0.f, -0.f, -0.f};
  int left = d.kper;
  auto end_slice = [&]() {
    left = d.kper;
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        tot[i][j] += acc[i][j];
        acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
      }
  };
#pragma unroll
  for (int c = 0; c < 2; ++c) fetch(r[c], 2 * c);
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    stash_a(r[c], s_t + (c) * kBuf);
    stash_b(r[c], s_t + (c) * kBuf);
    fetch(r[c], 4 + 2 * c);
  }
  __syncthreads();
  bf16x8 a[2][NI], b[2][NJ];
  auto read = [&](const uint16_t* s, int h) {
#pragma unroll
    for (int i = 0; i < NI; ++i) a[h][i] = dw_frag<BM>(s, 32 * h, wm / 16 + i, lane);
#pragma unroll
    for (int j = 0; j < NJ; ++j) b[h][j] = dw_frag<BN>(s + 64 * BM, 32 * h, wn / 16 + j, lane);
  };
  auto product = [&](int h) {
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
      for (int j = 0; j < NJ; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[h][j], a[h][i], acc[i][j], 0, 0, 0);
    if (--left == 0) end_slice();
  };
  read(s_t, 0);
  // as in gemm_nt_kernel
  auto step = [&](int k, const uint16_t* s0, const uint16_t* s1, uint16_t* s2, Stage& f) {
    read(s0, 1);
    stash_a(f, s2);
    if (k < steps) product(0);
    __syncthreads();
    read(s1, 0);
    stash_b(f, s2);
    if (k + 1 < steps) product(1);
    fetch(f, k + 8);
  };
  for (int k0 = 0; k0 < steps; k0 += 12) {
#pragma unroll
    for (int c = 0; c < 6; ++c)
      step(k0 + 2 * c, s_t + (c % 3) * kBuf, s_t + ((c + 1) % 3) * kBuf, s_t + ((c + 2) % 3) * kBuf, r[c & 1]);
  }
  if (left < d.kper) end_slice();
  // 16-row stripe i: parameters and moments, the next stripe's loads in flight
  struct Rows {
    f32x4 p[NJ], m[NJ], v[NJ];
  } q0, q1;
  const int mr = m0 + wm + r16, nc = n0 + wn + kg * 4;
  auto in = [&](int i, int j) { return mr + 16 * i < d.M && nc + 16 * j < d.N; };
  auto at = [&](int i, int j) { return (int64_t)(mr + 16 * i) * d.N + nc + 16 * j; };
  auto load = [&](Rows& q, int i) {
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      const int64_t o = in(i, j) ? at(i, j) : 0;
      q.p[j] = *reinterpret_cast<const f32x4*>(d.p + o);
      q.m[j] = *reinterpret_cast<const f32x4*>(d.m + o);
      q.v[j] = *reinterpret_cast<const f32x4*>(d.v + o);
    }
  };
  if (ad.on) load(q0, 0);
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    Rows& q = i & 1 ? q1 : q0;
    if (ad.on && i + 1 < NI) load(i & 1 ? q0 : q1, i + 1);
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      if (!in(i, j)) continue;
      const f32x4 g = tot[i][j];
      const int64_t o = at(i, j);
      if (!ad.on) {
        *reinterpret_cast<f32x4*>(d.g + o) = g;
        continue;
      }
      uint32_t h[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        float m1 = q.m[j][r], v1 = q.v[j][r];
        q.p[j][r] = adam_one(ad, q.p[j][r], m1, v1, g[r]);
        q.m[j][r] = m1;
        q.v[j][r] = v1;
        h[r] = to_bf16(q.p[j][r]);
      }
      *reinterpret_cast<f32x4*>(d.p + o) = q.p[j];
      *reinterpret_cast<f32x4*>(d.m + o) = q.m[j];
      *reinterpret_cast<f32x4*>(d.v + o) = q.v[j];
      *reinterpret_cast<uint2*>(d.p16 + (int64_t)(mr + 16 * i) * d.ldb + nc + 16 * j) = make_uint2(h[0] | h[1] << 16, h[2] | h[3] << 16);
      if (d.pT) {
#pragma unroll
        for (int r = 0; r < 4; ++r) d.pT[(int64_t)(nc + 16 * j + r) * d.M + mr + 16 * i] = (uint16_t)h[r];
      }
    }
  }
}

template <int BM, int BN, int WM, int WN>
__global__ __launch_bounds__(64 * (BM / WM) * (BN / WN)) void dw_kernel(DwArgs a) {
  __shared__ __attribute__((aligned(16))) uint16_t s_t[3 * 64 * (BM + BN)];
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  if ((int)blockIdx.x < a.tiles) {
    const int idx = xcd_order(blockIdx.x, a.tiles);
    int l = 0;
    while (l + 1 < 4 && idx >= a.w[l + 1].first) ++l;
    dw_tile<BM, BN, WM, WN>(a.w[l], idx - a.w[l].first, a.K, a.adam, s_t);
    return;
  }
  if (t >= 256) return;  // the rest is work for four waves
  int u = (int)blockIdx.x - a.tiles;
  const int B = a.K;
  if (u >= a.col_blocks) {
    // squared errors of 32 rows, a wave per row: lanes sum columns lane,
    // lane + 64, ... in order, then a butterfly over the wave
    const int r0 = (u - a.col_blocks) * 32;
    for (int r = r0 + w; r < min(r0 + 32, B); r += 4) {
      float e[5], acc = 0.f;
#pragma unroll
      for (int j = 0; j < 5; ++j) {
        const int64_t o = (int64_t)r * kLinOut + lane + 64 * j;
        e[j] = a.y[o] - a.target[o];
      }
#pragma unroll
      for (int j = 0; j < 5; ++j) acc = fmaf(e[j], e[j], acc);
#pragma unroll
      for (int m = 32; m > 0; m >>= 1) acc += __shfl_xor(acc, m);
      if (lane == 0) a.row_sq[r] = acc;
    }
    return;
  }
  // Partial column sums (bias gradients) of one layer's dZ, in a fixed order:
  // 64 columns of a chunk of cr rows, wave w summing rows w, w + 4, ... (eight
  // loads in flight per lane), the four sums added in wave order.
  int l = 0;
  while (l + 1 < 4 && u >= a.c[l + 1].first) ++l;
  const ColSet& c = a.c[l];
  u -= c.first;
  const int nb = (c.n + 63) / 64, y = u / nb, j = (u - y * nb) * 64 + lane;
  const int r0 = y * c.cr, r1 = min(B, r0 + c.cr);
  float s = 0.f;
  if (j < c.n) {
    if (c.dz) {
#pragma unroll 8
      for (int r = r0 + w; r < r1; r += 4) s += c.dz[(int64_t)r * c.n + j];
    } else {  // the last layer's dZ is 2 (y - target) / (rows * columns)
#pragma clang fp contract(off)
#pragma unroll 8
      for (int r = r0 + w; r < r1; r += 4)
        s += a.scale * (a.y[(int64_t)r * c.n + j] - a.target[(int64_t)r * c.n + j]);
    }
  }
  float* ps = reinterpret_cast<float*>(s_t);
  ps[64 * w + lane] = s;
  __syncthreads();
  if (w == 0 && j < c.n) c.part[(int64_t)y * c.n + j] = ((ps[lane] + ps[64 + lane]) + ps[128 + lane]) + ps[192 + lane];
}

// Bias gradients from the chunks' sums, with the Adam step where a.adam.on,
// and (last block) the loss.  32 columns per 256 threads, eight threads per
// column: thread `sub` adds chunks sub, sub + 8, ... in order, then the eight
// sums are added pairwise in a fixed tree.  The loss: thread t sums rows t,
// t + 1024, ... eight loads at a time, a butterfly per wave, then the sixteen
// wave sums in wave order.
__global__ __launch_bounds__(1024) void bias_kernel(DwArgs a, float loss_scale, float* loss) {
  __shared__ float ps[4][8][32];
  const int t = threadIdx.x;
  if (blockIdx.x + 1 == gridDim.x) {
    float* s = &ps[0][0][0];
    const int lane = t & 63, B = a.K;
    float acc = 0.f;
    for (int r0 = t; r0 < B; r0 += 8 * 1024) {
      float v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = r0 + u * 1024 < B ? a.row_sq[r0 + u * 1024] : 0.f;
#pragma unroll
      for (int u = 0; u < 8; ++u) acc += v[u];
    }
#pragma unroll
    for (int m = 32; m > 0; m >>= 1) acc += __shfl_xor(acc, m);
    if (lane == 0) s[t >> 6] = acc;
    __syncthreads();
    if (t == 0) {
      float tot = 0.f;
      for (int w = 0; w < 16; ++w) tot += s[w];
      loss[0] = tot * loss_scale;
    }
    return;
  }
  const int part = t >> 8, c = t & 31, sub = (t >> 5) & 7;
  int u = 4 * blockIdx.x + part, l = 0;  // 32 columns each, layer after layer
  while (l < 4 && u >= (a.c[l].n + 31) / 32) u -= (a.c[l++].n + 31) / 32;
  const ColSet& cs = a.c[l < 4 ? l : 3];
  const int j = l < 4 ? u * 32 + c : cs.n, R = (a.K + cs.cr - 1) / cs.cr;
  float s = 0.f;
  if (j < cs.n) {
#pragma unroll 4
    for (int y = sub; y < R; y += 8) s += cs.part[(int64_t)y * cs.n + j];
  }
  ps[part][sub][c] = s;
  __syncthreads();
  if (sub == 0 && j < cs.n) {
    const auto& q = ps[part];
    const float g = ((q[0][c] + q[1][c]) + (q[2][c] + q[3][c])) + ((q[4][c] + q[5][c]) + (q[6][c] + q[7][c]));
    if (a.adam.on) {
      float m = cs.m[j], v = cs.v[j];
      cs.p[j] = adam_one(a.adam, cs.p[j], m, v, g);
      cs.m[j] = m;
      cs.v[j] = v;
    } else {
      cs.g[j] = g;
    }
  }
}

// Training targets of instance i: its final group bests, normalised by the
// map size (row i of T, Eq.(10) layout per group).
__global__ __launch_bounds__(256) void targets_kernel(Pools pl, float* T, int ldt) {
  const int inst = blockIdx.x;
  const InstDesc& d = pl.desc[inst];
  const int D = 2 * d.W;
  for (int j = threadIdx.x; j < d.G * D && j < ldt; j += blockDim.x) {
    const int dd = j % D;
    T[(int64_t)inst * ldt + j] = pl.gbest_pos[d.gpo + j] / (dd < d.W ? d.width : d.height);
  }
}

// BF16 copies of a weight matrix (M x N), as it lies and (pT) transposed.
__global__ __launch_bounds__(256) void cvt_bf16_kernel(const float* p, uint16_t* p16, int ld, uint16_t* pT, int M, int N) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= (int64_t)M * N) return;
  const int m = (int)(i / N), n = (int)(i - (int64_t)m * N);
  const uint16_t h = to_bf16(p[i]);
  p16[(int64_t)m * ld + n] = h;
  if (pT) pT[(int64_t)n * M + m] = h;
}

// Accept the network's proposals: eligible instances with a finite output
// get per-group initial paths (clamped to the map); others fall back.
__global__ __launch_bounds__(256) void proposal_kernel(Pools pl, const float* Y, int ldy,
                                                       const int32_t* eligible) {
  const int inst = blockIdx.x;
  const InstDesc& d = pl.desc[inst];
  __shared__ int s_ok;
  if (threadIdx.x == 0) s_ok = eligible[inst];
  __syncthreads();
  const int D = 2 * d.W;
  if (s_ok) {
    for (int j = threadIdx.x; j < kLinOut; j += blockDim.x)
      if (!isfinite(Y[(int64_t)inst * ldy + j])) atomicAnd(&s_ok, 0);
  }
  __syncthreads();
  if (s_ok) {
    for (int j = threadIdx.x; j < d.G * D; j += blockDim.x) {
      const int dd = j % D;
      const float hi = dd < d.W ? d.width : d.height;
      float u = Y[(int64_t)inst * ldy + j];
      u = u < 0.f ? 0.f : (u > 1.f ? 1.f : u);
      pl.proposal[d.gpo + j] = u * hi;
    }
  }
  if (threadIdx.x == 0) pl.ctl[inst].use_learned = s_ok;
}

// ---------------------------------------------------------------------------
void launch_raster(const Pools& pl, int n_inst, uint16_t* X, int ldx, int32_t* eligible,
                   hipStream_t s) {
  hipLaunchKernelGGL(raster_kernel, dim3(n_inst), dim3(256), 0, s, pl, X, ldx, eligible);
}

// MFMA steps of 32 per slice of a sum over K: the sum's order, which every
// kernel above keeps whatever its tiles, so that a training run gives the same
// weights on all of them.  (The slices are those of a grid of 128 x 128 or
// 64 x 64 tiles whose blocks share out K until there are two per CU.)
static int slice_steps(bool weights, int M, int N, int K) {
  const int tiles128 = ((N + 127) / 128) * ((M + 127) / 128);
  const int T = tiles128 >= 64 || (weights && K >= 2048) ? 128 : 64;
  const int smax = T == 128 && tiles128 < 64 ? 16 : 8;
  const int tiles = ((N + T - 1) / T) * ((M + T - 1) / T), steps = K / 32;
  const int64_t floats = 4 * kLinHidden * kLinInPad;
  int S = 1;
  const bool whole = T == 128 && tiles >= 256 && K <= 1024;
  while (!whole && S < smax && tiles * S < 512 && S * 2 <= steps && (int64_t)S * 2 * M * N <= floats) S *= 2;
  return steps > 0 ? (steps + S - 1) / S : 1;
}

void launch_gemm(const uint16_t* A, int lda, const uint16_t* B, int ldb, int M, int N, int K, const Epi& ep,
                 hipStream_t s) {
  const int steps = K / 32, kper = slice_steps(false, M, N, K), S = (steps + kper - 1) / kper;
  // The largest tiles that still leave most CUs one (M x 512, K = 4128, us:
  // M = 6144 35.4 by 128 x 128 and 42.6 by 64 x 128; 4096 35.1 and 26.2; 3072
  // 25.5 by 64 x 128, 64 x 64 29; 2048 25.0 and 21.4), and the kernel without
  // LDS staging for slices of two steps (K = 512, M = 512 4.4 and 5.7 by 64 x
  // 64; M = 1024 6.1 and 5.8).
  auto tiles = [&](int bm, int bn) { return ((M + bm - 1) / bm) * ((N + bn - 1) / bn); };
#define NT(BM, BN, WM, WN, D)                                                                                       \
  hipLaunchKernelGGL((gemm_nt_kernel<BM, BN, WM, WN, D>), dim3(tiles(BM, BN)), dim3(64 * (BM / WM) * (BN / WN)), 0, \
                     s, A, lda, B, ldb, M, N, steps, kper, ep)
  if (tiles(128, 128) >= 160)
    NT(128, 128, 64, 32, 2);
  else if (tiles(64, 128) >= 160)
    NT(64, 128, 32, 32, 2);
  else if (kper <= 2 && S <= kSmallWaves && tiles(32, 32) <= 256)
    hipLaunchKernelGGL(gemm_small_kernel, dim3(tiles(32, 32)), dim3(64 * kSmallWaves), 0, s, A, lda, B, ldb, M, N,
                       steps, kper, S, ep);
  else if (K < 2048)
    NT(64, 64, 16, 32, 2);
  else  // few blocks and a long K: the inputs' rows come from HBM, six steps ahead
    NT(64, 64, 16, 32, 6);
#undef NT
}

int col_chunk(int B, int n) { return (int64_t)((n + 63) / 64) * ((B + 255) / 256) >= 128 ? 256 : 32; }

void launch_weight_grads(DwArgs a, float loss_scale, float* loss, hipStream_t s) {
  // 128 x 128 tiles: 4096 rows 46 us against 48 by 64 x 64 (without Adam), 8192
  // 79 against 91; 2048 rows 33 against 29
  const int T = a.K >= 4096 ? 128 : 64;
  int tiles = 0, cols = 0, fin = 0;
  for (int l = 0; l < 4; ++l) {
    DwSet& w = a.w[l];
    w.kper = slice_steps(true, w.M, w.N, a.K);
    w.first = tiles;
    tiles += ((w.M + T - 1) / T) * ((w.N + T - 1) / T);
    ColSet& c = a.c[l];
    c.cr = col_chunk(a.K, c.n);
    c.first = cols;
    cols += ((c.n + 63) / 64) * ((a.K + c.cr - 1) / c.cr);
    fin += (c.n + 31) / 32;
  }
  a.tiles = tiles;
  a.col_blocks = cols;
  const dim3 grid(tiles + cols + (a.K + 31) / 32);
  if (T == 128)
    hipLaunchKernelGGL((dw_kernel<128, 128, 64, 32>), grid, dim3(512), 0, s, a);
  else
    hipLaunchKernelGGL((dw_kernel<64, 64, 16, 32>), grid, dim3(512), 0, s, a);
  hipLaunchKernelGGL(bias_kernel, dim3((fin + 3) / 4 + 1), dim3(1024), 0, s, a, loss_scale, loss);
}

void launch_targets(const Pools& pl, int n_inst, float* T, int ldt, hipStream_t s) {
  hipLaunchKernelGGL(targets_kernel, dim3(n_inst), dim3(256), 0, s, pl, T, ldt);
}

void launch_cvt_bf16(const float* p, uint16_t* p16, int ld, uint16_t* pT, int M, int N, hipStream_t s) {
  const int64_t count = (int64_t)M * N;
  hipLaunchKernelGGL(cvt_bf16_kernel, dim3((unsigned)((count + 255) / 256)), dim3(256), 0, s, p, p16, ld, pT, M, N);
}

void launch_proposal(const Pools& pl, int n_inst, const float* Y, int ldy, const int32_t* eligible,
                     hipStream_t s) {
  hipLaunchKernelGGL(proposal_kernel, dim3(n_inst), dim3(256), 0, s, pl, Y, ldy, eligible);
}

}  // namespace sepso
