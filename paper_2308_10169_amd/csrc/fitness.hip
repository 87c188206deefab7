// Path fitness of given paths on a polygonal map (Eq.(11)-(13)): polyline
// length L over [start, waypoints, target], Q = proper crossings of the W+1
// segments with every polygon edge, F = L + alpha * Q^beta.  Stateless: the
// caller passes device inputs and outputs; one launch, fit_kernel, and no
// device memory besides.
//
// Orientation arithmetic: a segment p -> q is kept as (dx, dy) and the line
// constant nc = dy*p.x - dx*p.y, so orient(p, q, v) = dx*v.y - dy*v.x + nc
// is two FMAs; an edge a -> b likewise as (ex, ey) and ce = ex*a.y - ey*a.x.
// A test counts when both pairs of orientations have strictly opposite
// signs; touching and collinear contacts never count.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cfloat>
#include <cmath>

#include "../../include/sepso.h"
#include "internal.h"

namespace sepso {
namespace {

constexpr int kFitVerts = 2560;  // vertices staged in LDS per pass (20 KiB)
constexpr int kFitPolys = 736;   // polygons per pass (boxes and words of 818 pieces 16 KiB)
constexpr int kFitLong = 32;     // a polygon of more edges is cut into chains
constexpr int kFitChain = 31;    // edges of a chain (32 vertices)
constexpr float kFitBig = 0x1p62f;
constexpr int kFitMaxThreads = 512;

// LDS of one block: staged vertices, boxes and words of the pieces (a piece is a
// polygon, or a chain of a long one), two counts of pieces past the polygons',
// the block's path points with the crossings and the length of the segment that
// starts at each, and a queue per wave.  At most 64 KiB (K * threads <= 1024,
// so ppr * (W + 2) <= 1536).
struct FitLds {
  int verts, polys, pieces;                          // capacities
  int box, word, extra, pts, cross, len, queue, bytes;  // byte offsets (vertices at 0)
};

__host__ __device__ inline FitLds fit_lds(int n_polys, int n_vert, int threads, int n_pts) {
  FitLds l{};
  l.verts = n_vert < kFitVerts ? (n_vert + 1) & ~1 : kFitVerts;  // 16-byte aligned boxes after them
  l.polys = n_polys < kFitPolys ? n_polys : kFitPolys;
  // m vertices make ceil(m / kFitChain) - 1 < m / kFitChain pieces more than one
  l.pieces = l.polys + l.verts / kFitChain;
  l.box = 8 * l.verts;
  l.word = l.box + 16 * l.pieces;
  l.extra = l.word + 4 * l.pieces;
  l.pts = (l.extra + 8 + 7) & ~7;
  l.cross = l.pts + 8 * n_pts;
  l.len = l.cross + 4 * n_pts;
  l.queue = l.len + 4 * n_pts;
  l.bytes = l.queue + 8 * threads;  // 128 words per wave
  return l;
}

__device__ __forceinline__ bool opposite(float a, float b) {
  return (a < 0.f && b > 0.f) || (a > 0.f && b < 0.f);
}

// w = 2 w + !(|o| > r), two instructions (a NaN on either side gives 1).
__device__ __forceinline__ void push_near(uint32_t& w, float o, float r) {
  asm("v_cmp_ngt_f32_e64 vcc, |%1|, %2\n\tv_addc_co_u32_e32 %0, vcc, %0, %0, vcc"
      : "+v"(w)
      : "v"(o), "v"(r)
      : "vcc");
}

// One block: `rounds` times `ppr` whole paths, K segments per thread.
//
// What bounds it is VALU issue: a segment's test against one edge is about 18
// instructions, and most pairs have no contact.  So each segment first tests
// its line against every polygon's bounding box -- two FMAs for the box
// centre's orientation o, two for r = |dx| h + |dy| w, one comparison -- and
// only polygons whose box the line may meet are tested edge by edge.  The box
// sizes and r carry a margin above the rounding of o and of the vertices' own
// orientations (about 4 u (|dx| Y + |dy| X) each with u = 2^-24, X and Y the
// largest coordinates; the margin is 16 u of it), so |o| > r means that the
// edge-by-edge test would find every vertex strictly on one side and count
// nothing: the counts are those of testing every pair, bit for bit.  (Segments
// and boxes whose numbers pass kFitBig, where the products of both may leave the
// range of a float, are near everything.)  Skipping
// by the segment's own extent as well would need a tolerance that near-
// parallel contacts break, so it is left out.
//
// The lines of 64 lanes meet different polygons (one in thirty of a dense
// map), so the (segment, polygon) pairs to test go through a queue in LDS and
// any lane takes any pair, 64 at a time; with a queue per lane half the lanes
// sat idle (607 us on the large case below).  Vertices, boxes and words are
// staged in LDS, by polygon ranges that fit when the map is larger.  A polygon
// of more than kFitLong edges goes in chains of kFitChain, each with a box of
// its own like a polygon; one that exceeds a pass by itself, a pass at a time.
// (Walked edge by edge by each wave, such polygons took up to 2.3 times what
// testing every pair takes: a block's few waves wait on every edge in turn.)
//
// 32768 uniform paths of 64 waypoints on 600 polygons (2400 edges): 1803 -> 390
// us a call; 1360 paths of 20 on 30 rectangles: 28.2 -> 8.5 us; 128 paths of 8
// on 4 rectangles: 13.5 -> 8.2 us, of which the host's call and the launch are
// most; 8192 paths of 20 on 24 polygons of 100 edges: 257 -> 77 us; 32768 of 8
// on one of 20000: 2042 -> 105 us (before: every pair tested, three launches).
template <int K>
__global__ __launch_bounds__(kFitMaxThreads) void fit_kernel(
    int n_polys, const int32_t* __restrict__ pptr, const float* __restrict__ verts, int n_vert,
    const float* __restrict__ ends, const float* __restrict__ paths, int n_paths, int W, int ppr,
    int rounds, float alpha, int beta, float* f, float* L, int32_t* Q) {
  extern __shared__ __attribute__((aligned(16))) char s_fit[];
  const int t = threadIdx.x, B = blockDim.x, lane = t & 63;
  const int S = W + 1, N = W + 2;  // segments and points per path
  const FitLds lds = fit_lds(n_polys, n_vert, B, ppr * N);
  float* s_vf = reinterpret_cast<float*>(s_fit);
  const float2* s_v = reinterpret_cast<const float2*>(s_fit);
  float4* s_box = reinterpret_cast<float4*>(s_fit + lds.box);
  // a piece's first vertex (12 bits), edges less one (5), and the vertex its last
  // edge ends in (12: a closed polygon's first); kNoPiece: nothing to test
  uint32_t* s_word = reinterpret_cast<uint32_t*>(s_fit + lds.word);
  int* s_extra = reinterpret_cast<int*>(s_fit + lds.extra);  // of this pass and the next, in turn
  constexpr uint32_t kNoPiece = 0x80000000u;
  auto word = [](int first, int edges, int last) { return (uint32_t)(first | (edges - 1) << 12 | last << 17); };
  float2* s_pt = reinterpret_cast<float2*>(s_fit + lds.pts);
  int* s_cross = reinterpret_cast<int*>(s_fit + lds.cross);
  float* s_len = reinterpret_cast<float*>(s_fit + lds.len);
  uint32_t* s_queue = reinterpret_cast<uint32_t*>(s_fit + lds.queue) + 2 * (t - lane);
  const bool one_pass = n_vert <= lds.verts && n_polys <= lds.polys;
  auto offset = [&](int q) { return min(max(pptr[q], 0), n_vert); };  // inside whatever it holds
  int pieces = 0, turn = 0;  // staged pieces; passes staged so far

  for (int rd = 0; rd < rounds; ++rd) {
    const int path0 = (blockIdx.x * rounds + rd) * ppr;
    if (path0 >= n_paths) break;  // the whole block
    float px[K], py[K], qx[K], qy[K], dx[K], dy[K], nc[K], tol[K];
    int pt[K];  // the segment's first point among the block's
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const int i = t + k * B, pl = i / S, s = i - pl * S;
      px[k] = py[k] = qx[k] = qy[k] = 0.f;
      pt[k] = i + pl;
      const bool active = pl < ppr && path0 + pl < n_paths;
      if (active) {
        const float* x = paths + (int64_t)(path0 + pl) * 2 * W;
        // points s and s + 1 of [start, w_1..w_W, target]
        const float* p = s == 0 ? ends : x + s - 1;
        px[k] = p[0];
        py[k] = p[s == 0 ? 1 : W];
        const float* q = s == W ? ends + 2 : x + s;
        qx[k] = q[0];
        qy[k] = q[s == W ? 1 : W];
      }
      dx[k] = qx[k] - px[k];
      dy[k] = qy[k] - py[k];
      nc[k] = fmaf(dy[k], px[k], -(dx[k] * py[k]));
      // the margin's share of the segment's own coordinates (and a floor far
      // above the rounding of subnormal values); idle lanes are near nothing
      tol[k] = active ? fmaf(0x1p-20f, fabsf(dx[k] * py[k]) + fabsf(dy[k] * px[k]), 1e-37f) : -1.f;
      if (active && fmaxf(fabsf(dx[k]), fabsf(dy[k])) > kFitBig) tol[k] = INFINITY;
      if (active) {
        s_pt[pt[k]] = make_float2(px[k], py[k]);
        if (s == W) s_pt[pt[k] + 1] = make_float2(qx[k], qy[k]);
        s_cross[pt[k]] = 0;
        s_len[pt[k]] = __builtin_amdgcn_sqrtf(fmaf(dx[k], dx[k], dy[k] * dy[k]));  // v_sqrt_f32, within 1 ulp
      }
    }
    if (rd == 0 && t < 2) s_extra[t] = 0;
    __syncthreads();

    // the queue's pairs from `first` on, one per lane of the first n
    auto work_off = [&](int first, int n) {
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      if (lane < n) {
        const uint32_t e = s_queue[first + lane];
        const int i = e & 2047u, q = e >> 11;
        const uint32_t w = s_word[q];
        // a zero-length segment is near every box, also those that hold nothing to test
        if (w == kNoPiece) return;
        const int v0 = w & 4095u, m = (w >> 12 & 31u) + 1, last = w >> 17;
        const float2 a = s_pt[i], b = s_pt[i + 1];
        const float ddx = b.x - a.x, ddy = b.y - a.y, c = fmaf(ddy, a.x, -(ddx * a.y));
        // strict sides of vertex j, bit m - 1 - j
        uint32_t neg = 0, pos = 0;
        auto side = [&](const float2& v) {
          const float o = fmaf(ddx, v.y, fmaf(-ddy, v.x, c));
          neg = 2 * neg + (o < 0.f ? 1u : 0u);
          pos = 2 * pos + (o > 0.f ? 1u : 0u);
        };
        for (int j = 0; j < m; ++j) side(s_v[v0 + j]);
        // the vertex that edge j starts in and, in the word's next place, the
        // one it ends in: j + 1, or `last` (a closed polygon's vertex 0)
        const uint32_t n0 = neg, p0 = pos;
        if (last == v0) {
          neg = (neg << 1) | (neg >> (m - 1));
          pos = (pos << 1) | (pos >> (m - 1));
        } else {
          side(s_v[last]);
        }
        uint32_t st = ((n0 & pos) | (p0 & neg)) & (0xffffffffu >> (32 - m));
        int n_cross = 0;
        while (st) {
          const int bit = 31 - __clz(st), j = m - 1 - bit;
          st ^= 1u << bit;
          const float2 g = s_v[v0 + j], h = s_v[bit == 0 ? last : v0 + j + 1];
          const float ex = h.x - g.x, ey = h.y - g.y, ce = fmaf(ex, g.y, -(ey * g.x));
          const float o3 = fmaf(ex, a.y, fmaf(-ey, a.x, -ce));
          const float o4 = fmaf(ex, b.y, fmaf(-ey, b.x, -ce));
          n_cross += opposite(o3, o4) ? 1 : 0;
        }
        if (n_cross) atomicAdd(&s_cross[i], n_cross);
      }
    };

    int done = 0;  // edges of polygon q0 behind us, when it exceeds a pass by itself
    for (int q0 = 0; q0 < n_polys;) {
      // this pass: polygons q0 .. q1 - 1, their vertices from v0 on, or the chain
      // of `chain` edges of q0 from its vertex `done` on
      int q1 = n_polys, chain = 0;
      const int v0 = one_pass ? 0 : offset(q0);
      if (!one_pass) {  // the longest range that fits
        int lo = q0, hi = min(q0 + lds.polys, n_polys);
        while (lo < hi) {
          const int mid = (lo + hi + 1) >> 1;
          if (offset(mid) - v0 <= lds.verts)
            lo = mid;
          else
            hi = mid - 1;
        }
        q1 = lo;
        if (q1 == q0) chain = min(offset(q0 + 1) - v0 - done, lds.verts - 1);
      }
      if (!one_pass || rd == 0) {
        if (!one_pass) __syncthreads();  // the last pass has been read
        int* extra = s_extra + (turn & 1);
        const float* g = verts + 2 * (int64_t)(v0 + done);
        if (chain == 0) {
          const int np = q1 - q0, nv = one_pass ? n_vert : max(offset(q1) - v0, 0);
          for (int i = t; i < 2 * nv; i += B) s_vf[i] = g[i];
          for (int i = t; i < np; i += B) {
            const int a = min(max(pptr[q0 + i] - v0, 0), nv), m = min(max(pptr[q0 + i + 1] - v0, 0), nv) - a;
            s_word[i] = m < 1 ? kNoPiece : m <= kFitLong ? word(a, m, a) : word(a, kFitChain, a + kFitChain);
            if (m > kFitLong) {  // the other chains, after the polygons
              const int more = (m - 1) / kFitChain;
              int at = np + atomicAdd(extra, more);
              for (int j = 1; j <= more; ++j, ++at) {
                const int s = j * kFitChain, e = min(m, s + kFitChain);
                if (at < lds.pieces) s_word[at] = word(a + s, e - s, e == m ? a : a + e);
              }
            }
          }
        } else {
          // a chain's vertices, its last edge's end (the polygon's first vertex
          // after its last) among them
          const bool closes = v0 + done + chain == offset(q0 + 1);
          for (int i = t; i < 2 * chain; i += B) s_vf[i] = g[i];
          if (t < 2) s_vf[2 * chain + t] = closes ? verts[2 * (int64_t)v0 + t] : g[2 * chain + t];
          for (int i = t; i * kFitChain < chain; i += B) {
            const int s = i * kFitChain, e = min(chain, s + kFitChain);
            s_word[i] = word(s, e - s, e);
          }
        }
        __syncthreads();
        // (more than there is room for only if the offsets are malformed)
        pieces = chain ? (chain + kFitChain - 1) / kFitChain : min(q1 - q0 + *extra, lds.pieces);
        if (t == 0) s_extra[(turn + 1) & 1] = 0;
        ++turn;
        for (int i = t; i < pieces; i += B) {
          const uint32_t w = s_word[i];
          float4 b = make_float4(0.f, 0.f, -FLT_MAX, -FLT_MAX);  // nothing to test here
          if (w != kNoPiece) {
            const int a = w & 4095u, m = (w >> 12 & 31u) + 1, last = w >> 17;
            float x0 = s_v[last].x, x1 = x0, y0 = s_v[last].y, y1 = y0;
            for (int j = last == a ? 1 : 0; j < m; ++j) {
              const float2 v = s_v[a + j];
              x0 = fminf(x0, v.x);
              x1 = fmaxf(x1, v.x);
              y0 = fminf(y0, v.y);
              y1 = fmaxf(y1, v.y);
            }
            // centre and half sides, the latter with the margin
            b.x = 0.5f * x0 + 0.5f * x1;
            b.y = 0.5f * y0 + 0.5f * y1;
            b.z = fmaf(fmaxf(x1 - b.x, b.x - x0), 1.f + 0x1p-19f, 0x1p-20f * fmaxf(fabsf(x0), fabsf(x1)));
            b.w = fmaf(fmaxf(y1 - b.y, b.y - y0), 1.f + 0x1p-19f, 0x1p-20f * fmaxf(fabsf(y0), fabsf(y1)));
            if (fmaxf(fmaxf(fabsf(x0), fabsf(x1)), fmaxf(fabsf(y0), fabsf(y1))) > kFitBig) b.z = b.w = INFINITY;
          }
          s_box[i] = b;
        }
        __syncthreads();
      }
      int queued = 0;  // the wave's
      for (int i0 = 0; i0 < pieces; i0 += 32) {
        const int n = min(32, pieces - i0);
        uint32_t near[K];
#pragma unroll
        for (int k = 0; k < K; ++k) near[k] = 0;
        auto test = [&](int i) {
          const float4 b = s_box[i0 + i];
#pragma unroll
          for (int k = 0; k < K; ++k) {
            const float o = fmaf(dx[k], b.y, fmaf(-dy[k], b.x, nc[k]));
            const float r = fmaf(fabsf(dx[k]), b.w, fmaf(fabsf(dy[k]), b.z, tol[k]));
            push_near(near[k], o, r);
          }
        };
        int i = 0;
        for (; i + 8 <= n; i += 8) {
#pragma unroll
          for (int u = 0; u < 8; ++u) test(i + u);
        }
        for (; i < n; ++i) test(i);
        // polygon i0 + n - 1 - bit of every set bit joins the wave's queue
#pragma unroll
        for (int k = 0; k < K; ++k) {
          uint32_t w = tol[k] > 0.f ? near[k] : 0u;
          for (;;) {
            const uint64_t has = __builtin_amdgcn_ballot_w64(w != 0u);
            if (has == 0ull) break;
            if (w != 0u) {
              const int bit = 31 - __clz(w);
              w ^= 1u << bit;
              const int at = __builtin_amdgcn_mbcnt_hi((uint32_t)(has >> 32),
                                                       __builtin_amdgcn_mbcnt_lo((uint32_t)has, 0u));
              const int q = i0 + n - 1 - bit;
              s_queue[queued + at] = (uint32_t)q << 11 | (uint32_t)pt[k];
            }
            queued += __popcll(has);
            if (queued >= 64) {
              queued -= 64;
              work_off(queued, 64);
            }
          }
        }
      }
      work_off(0, queued);
      done += chain;
      if (chain == 0 || v0 + done == offset(q0 + 1)) {
        q0 = max(q1, q0 + 1);
        done = 0;
      }
    }

    __syncthreads();
    const int p = path0 + t;
    if (t < ppr && p < n_paths) {
      int q = 0;
      float l = 0.f;
      for (int s = 0; s < S; ++s) {  // segment order: deterministic
        q += s_cross[t * N + s];
        l += s_len[t * N + s];
      }
      const float qf = (float)q;
      float pw = 1.f;
      for (int b = 0; b < beta; ++b) pw *= qf;
      f[p] = fmaf(alpha, pw, l);
      L[p] = l;
      Q[p] = q;
    }
    if (rd + 1 < rounds) __syncthreads();  // the sums are read before the points change
  }
}

size_t a256(size_t x) { return (x + 255) & ~size_t(255); }

// Bytes a caller's workspace must hold: records of 32 bytes per vertex and
// two words per segment.  The kernel keeps all of it on chip; the size and
// its checks stand for callers that carve their memory by them.
size_t fit_workspace(int64_t n_vert, int64_t n_paths, int W) {
  const size_t n_seg = (size_t)(n_paths * (W + 1));
  return a256(32 * (size_t)n_vert) + 2 * a256(4 * n_seg);
}

sepso_status fit_check(int32_t n_polys, int32_t n_vert, int32_t n_paths, int32_t W, float alpha,
                       int32_t beta) {
  if (n_polys < 0 || n_vert < 0) return fail(SEPSO_E_ARG, "fitness: n_polys and n_vert must be >= 0");
  if (n_vert > 0 && n_polys < 1) return fail(SEPSO_E_ARG, "fitness: vertices without polygons");
  if (n_paths < 0) return fail(SEPSO_E_ARG, "fitness: n_paths must be >= 0");
  if (W < 1 || W > kMaxW) return fail(SEPSO_E_ARG, "fitness: waypoints must be in [1, %d]", kMaxW);
  if ((int64_t)n_paths * (W + 1) > 0x7fffffffLL)
    return fail(SEPSO_E_ARG, "fitness: n_paths * (waypoints + 1) exceeds 2^31 - 1");
  if (beta < 1) return fail(SEPSO_E_ARG, "fitness: beta must be >= 1");
  if (!std::isfinite(alpha)) return fail(SEPSO_E_ARG, "fitness: alpha must be finite");
  return SEPSO_OK;
}

template <int K>
void fit_launch(int threads, int n_polys, const int32_t* pptr, const float* verts, int n_vert,
                const float* ends, const float* paths, int n_paths, int W, int rounds, float alpha,
                int beta, float* f, float* L, int32_t* Q, hipStream_t s) {
  const int ppr = K * threads / (W + 1);
  const int64_t per_block = (int64_t)ppr * rounds;
  const unsigned blocks = (unsigned)((n_paths + per_block - 1) / per_block);
  hipLaunchKernelGGL(fit_kernel<K>, dim3(blocks), dim3(threads), fit_lds(n_polys, n_vert, threads, ppr * (W + 2)).bytes,
                     s, n_polys, pptr, verts, n_vert, ends, paths, n_paths, W, ppr, rounds, alpha, beta, f,
                     L, Q);
}

// Threads per block, segments per thread and whole paths per block and round.
// Many segments: 512 threads of two segments each (a box is read from LDS once
// for both), a few rounds per block so that staging the map is paid once for
// several thousand segments.  Few: the smallest block that holds whole paths
// without leaving more than a quarter of its threads idle, one segment per
// thread, so that the call spreads over as many CUs as it can.
sepso_status fit_run(int32_t n_polys, int32_t n_vert, const int32_t* d_pptr, const float* d_verts,
                     const float* d_ends, const float* d_paths, int32_t n_paths, int32_t W,
                     float alpha, int32_t beta, float* d_f, float* d_L, int32_t* d_Q, hipStream_t s) {
  const int S = W + 1;
  if (n_vert == 0) n_polys = 0;  // polygons without vertices have no edges
  if ((int64_t)n_paths * S >= (1 << 18)) {
    const int ppr = 2 * kFitMaxThreads / S;
    const int rounds = std::max(1, (n_paths + ppr * 1024 - 1) / (ppr * 1024));
    fit_launch<2>(kFitMaxThreads, n_polys, d_pptr, d_verts, n_vert, d_ends, d_paths, n_paths, W, rounds,
                  alpha, beta, d_f, d_L, d_Q, s);
  } else {
    int threads = 64;
    while (threads < 256 && 4 * (threads / S * S) < 3 * threads) threads *= 2;
    fit_launch<1>(threads, n_polys, d_pptr, d_verts, n_vert, d_ends, d_paths, n_paths, W, 1, alpha, beta,
                  d_f, d_L, d_Q, s);
  }
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(SEPSO_E_HIP, "fitness launch: %s", hipGetErrorString(e));
  return SEPSO_OK;
}

sepso_status fit_pointers(int32_t n_vert, const int32_t* d_pptr, const float* d_verts,
                          const float* d_ends, const float* d_paths, int32_t n_paths, float* d_f,
                          float* d_L, int32_t* d_Q) {
  if (n_vert > 0 && (!d_pptr || !d_verts))
    return fail(SEPSO_E_ARG, "fitness: poly_ptr and verts must be device pointers");
  if (n_paths > 0 && (!d_ends || !d_paths || !d_f || !d_L || !d_Q))
    return fail(SEPSO_E_ARG, "fitness: ends, paths and the outputs must be device pointers");
  return SEPSO_OK;
}

}  // namespace
}  // namespace sepso

using namespace sepso;

extern "C" {

sepso_status sepso_fitness_workspace_bytes(int32_t n_vert, int32_t n_paths, int32_t waypoints,
                                           size_t* bytes) {
  if (!bytes) return fail(SEPSO_E_ARG, "fitness: bytes is NULL");
  if (n_vert < 0 || n_paths < 0) return fail(SEPSO_E_ARG, "fitness: sizes must be >= 0");
  if (waypoints < 1 || waypoints > kMaxW)
    return fail(SEPSO_E_ARG, "fitness: waypoints must be in [1, %d]", kMaxW);
  *bytes = fit_workspace(n_vert, n_paths, waypoints);
  return SEPSO_OK;
}

sepso_status sepso_fitness(int32_t n_polys, int32_t n_vert, const int32_t* d_poly_ptr,
                           const float* d_verts, const float* d_ends, const float* d_paths,
                           int32_t n_paths, int32_t waypoints, float alpha, int32_t beta,
                           float* d_f, float* d_L, int32_t* d_Q, void* d_ws, size_t ws_bytes,
                           void* stream) {
  sepso_status st = fit_check(n_polys, n_vert, n_paths, waypoints, alpha, beta);
  if (st == SEPSO_OK)
    st = fit_pointers(n_vert, d_poly_ptr, d_verts, d_ends, d_paths, n_paths, d_f, d_L, d_Q);
  if (st != SEPSO_OK) return st;
  if (n_paths == 0) return SEPSO_OK;
  const size_t need = fit_workspace(n_vert, n_paths, waypoints);
  if (!d_ws || (reinterpret_cast<uintptr_t>(d_ws) & 255))
    return fail(SEPSO_E_ARG, "fitness: workspace must be a 256-byte aligned device pointer");
  if (ws_bytes < need)
    return fail(SEPSO_E_NOMEM, "fitness: workspace of %zu bytes, %zu needed", ws_bytes, need);
  return fit_run(n_polys, n_vert, d_poly_ptr, d_verts, d_ends, d_paths, n_paths, waypoints, alpha,
                 beta, d_f, d_L, d_Q, static_cast<hipStream_t>(stream));
}

}  // extern "C"

// The workspace-free variant: the same launch, for requests up to the size it
// has always taken.
namespace {
constexpr size_t kFitScratchBytes = size_t(8) << 20;
}

extern "C" {

sepso_status sepso_fitness_noalloc(int32_t n_polys, int32_t n_vert, const int32_t* d_poly_ptr,
                                   const float* d_verts, const float* d_ends, const float* d_paths,
                                   int32_t n_paths, int32_t waypoints, float alpha, int32_t beta,
                                   float* d_f, float* d_L, int32_t* d_Q, void* stream) {
  sepso_status st = fit_check(n_polys, n_vert, n_paths, waypoints, alpha, beta);
  if (st == SEPSO_OK)
    st = fit_pointers(n_vert, d_poly_ptr, d_verts, d_ends, d_paths, n_paths, d_f, d_L, d_Q);
  if (st != SEPSO_OK) return st;
  if (n_paths == 0) return SEPSO_OK;
  const size_t need = fit_workspace(n_vert, n_paths, waypoints);
  if (need > kFitScratchBytes)
    return fail(SEPSO_E_ARG,
                "fitness_noalloc: %d paths of %d waypoints on %d vertices need %zu bytes of "
                "scratch; the allocation-free variant holds %zu (use sepso_fitness with a workspace)",
                n_paths, waypoints, n_vert, need, kFitScratchBytes);
  return fit_run(n_polys, n_vert, d_poly_ptr, d_verts, d_ends, d_paths, n_paths, waypoints, alpha,
                 beta, d_f, d_L, d_Q, static_cast<hipStream_t>(stream));
}

}  // extern "C"
