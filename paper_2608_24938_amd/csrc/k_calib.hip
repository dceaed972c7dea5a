// Projector calibration: per-pair sufficient statistics and the closed-form
// scalar projector and loss (Sec. 4.2, Eq. calibration_outputs,
// Eq. scalar_projector, Eq. projection_loss; Appendix A protocol; Appendix B,
// Eq. A1-A2).  The expert outputs u = E_e(x) come from the expert GEMMs run
// with weight 1 on every evaluated (token, expert) pair.
//
// gram:     G_i[a][b] = <u_{i,a}, u_{i,b}> in float64 for the evaluated experts of token i
// pairs:    per ordered pair (s, t), with w = ||u_s||: A += w G[s][t], V += w G[t][t],
//           C += w G[s][s], n += 1, over one m-tile of source s's rows (the rows are
//           in token order)
// finalize: the tiles of s in order; S = A / (V + lambda) (clipped),
//           L = max(0, C - 2 S A + S^2 V) / (C + eps);
//           h_e = mean ||u_e|| over the tokens that evaluated e.
#include "common.hpp"
#include "kernels.hpp"

namespace exfold {

// One thread per (token, expert): its position among the token's evaluated
// experts (-1: none), and the route lists of the expert GEMMs.
__global__ __launch_bounds__(256) void calib_routes_kernel(const int32_t *__restrict__ topk_ids, int m,
                                                           int N, int K, int mode,
                                                           int32_t *__restrict__ route_ids,
                                                           float *__restrict__ route_w,
                                                           int16_t *__restrict__ pos) {
  const long long idx = (long long)blockIdx.x * 256 + threadIdx.x;
  if (idx >= (long long)m * N) return;
  const int i = (int)(idx / N), e = (int)(idx % N);
  if (mode == EXFOLD_CAL_COMMON) {
    route_ids[idx] = e;
    route_w[idx] = 1.0f;
    pos[idx] = (int16_t)e;
    return;
  }
  const int32_t *row = topk_ids + (long long)i * K;
  int p = -1;
  for (int k = 0; k < K; ++k)
    if (clamp_id(row[k], N) == e) p = k;
  pos[idx] = (int16_t)p;
  if (e < K) {
    route_ids[(long long)i * K + e] = clamp_id(row[e], N);
    route_w[(long long)i * K + e] = 1.0f;
  }
}

hipError_t launch_calib_routes(const int32_t *topk_ids, int m, int N, int K, int mode,
                               int32_t *route_ids, float *route_w, int16_t *pos, hipStream_t s) {
  if (m <= 0) return hipSuccess;
  const long long n = (long long)m * N;
  calib_routes_kernel<<<(unsigned)((n + 255) / 256), 256, 0, s>>>(topk_ids, m, N, K, mode, route_ids, route_w,
                                                                  pos);
  return hipGetLastError();
}

// Gram matrices on the float64 MFMA (16x16x4; a product of two float32 values is
// exact in float64, the sums are rounded, in one fixed order).
// A tile's 16 rows are the rows of 16 / P tokens side by side (P: kr rounded up
// to a power of two; kr > 16: one token, 16 x 16 tiles ta <= tb).  Lane l holds
// eight consecutive columns of row l % 16 at 8 (l / 16), and MFMA step q takes
// element q of every lane: any assignment of columns to steps is a valid
// reduction order, so rows load in whole 128-byte pieces and, on a diagonal
// tile, one register serves as both operands.  The four waves split d and their
// partial tiles are added in wave order.  Each row is read once (bound by the
// read of the expert rows: 268 MB for 4096 tokens x 8 x 2048); one wave per
// pair of rows read every row kr + 1 times: 264 -> 68 us at that size (4.0 TB/s).
typedef double f64x4 __attribute__((ext_vector_type(4)));

template <bool DIAG>
__global__ __launch_bounds__(256) void calib_gram_kernel(const float *__restrict__ Y,
                                                         const int32_t *__restrict__ slot_row, int m, int kr,
                                                         int P, int d, double *__restrict__ gram) {
  __shared__ double red[4][256];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int ta = 0, tb = 0;
  if (!DIAG) {  // blockIdx.y -> (ta, tb), ta <= tb, row-major over the upper triangle of tiles
    const int nt = (kr + 15) / 16;
    int rem = blockIdx.y;
    while (rem >= nt - ta) {
      rem -= nt - ta;
      ++ta;
    }
    tb = ta + rem;
  }
  // row r of the tile: token i0 + r / P, evaluated expert r % P (kr <= 16), or 16 t + r
  const int i0 = blockIdx.x * (DIAG ? 16 / P : 1);
  auto row_of = [&](int t, bool &live) -> const float * {
    const int r = lane & 15;
    const int i = DIAG ? i0 + r / P : i0;
    const int a = DIAG ? r % P : t * 16 + r;
    live = i < m && a < kr;
    return Y + (long long)slot_row[live ? (long long)i * kr + a : 0] * d + (lane >> 4) * 8;
  };
  bool la, lb = false;
  const float *ya = row_of(ta, la);
  const float *yb = DIAG ? ya : row_of(tb, lb);
  const int span = d / 4;  // d % 128 == 0: whole steps of 32 columns
  f64x4 acc = {0.0, 0.0, 0.0, 0.0};
  constexpr int U = 2;     // steps whose loads are issued together
  for (int c0 = wave * span; c0 < (wave + 1) * span; c0 += 32 * U) {
    float4 va[U][2], vb[U][2];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int c = c0 + 32 * u;
      const bool in = c < (wave + 1) * span;
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        va[u][q] = make_float4(0.f, 0.f, 0.f, 0.f);
        if (in && la) va[u][q] = *reinterpret_cast<const float4 *>(ya + c + 4 * q);
        if (!DIAG) {
          vb[u][q] = make_float4(0.f, 0.f, 0.f, 0.f);
          if (in && lb) vb[u][q] = *reinterpret_cast<const float4 *>(yb + c + 4 * q);
        }
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const float fa[4] = {va[u][q].x, va[u][q].y, va[u][q].z, va[u][q].w};
        const float fb[4] = {DIAG ? fa[0] : vb[u][q].x, DIAG ? fa[1] : vb[u][q].y, DIAG ? fa[2] : vb[u][q].z,
                             DIAG ? fa[3] : vb[u][q].w};
#pragma unroll
        for (int e = 0; e < 4; ++e)
          acc = __builtin_amdgcn_mfma_f64_16x16x4f64((double)fa[e], (double)fb[e], acc, 0, 0, 0);
      }
  }
  // register r of lane l: row l / 16 + 4 r, column l % 16
#pragma unroll
  for (int r = 0; r < 4; ++r) red[wave][((lane >> 4) + 4 * r) * 16 + (lane & 15)] = acc[r];
  __syncthreads();
  const int r = threadIdx.x >> 4, c = threadIdx.x & 15;
  const double v = ((red[0][threadIdx.x] + red[1][threadIdx.x]) + red[2][threadIdx.x]) + red[3][threadIdx.x];
  if (DIAG) {
    const int i = i0 + r / P, a = r % P, b = c % P;
    if (r / P == c / P && i < m && a < kr && b < kr) gram[((long long)i * kr + a) * kr + b] = v;
  } else {
    const int a = ta * 16 + r, b = tb * 16 + c;
    if (a < kr && b < kr) {
      gram[((long long)i0 * kr + a) * kr + b] = v;
      if (ta != tb) gram[((long long)i0 * kr + b) * kr + a] = v;
    }
  }
}

hipError_t launch_calib_gram(const float *Y, const int32_t *slot_row, int m, int kr, int d,
                             double *gram, hipStream_t s) {
  if (m <= 0) return hipSuccess;
  if (kr <= 16) {
    int P = 1;
    while (P < kr) P *= 2;
    const int per = 16 / P;
    calib_gram_kernel<true><<<(m + per - 1) / per, 256, 0, s>>>(Y, slot_row, m, kr, P, d, gram);
  } else {
    const int nt = (kr + 15) / 16;
    calib_gram_kernel<false><<<dim3(m, nt * (nt + 1) / 2), 256, 0, s>>>(Y, slot_row, m, kr, 16, d, gram);
  }
  return hipGetLastError();
}

// Sums of one m-tile (at most bm rows, token order) of source s: block b is
// tile b of the permutation's tile list.  Thread (g, t) owns target t and the
// g-th run of the tile's rows; the runs are added in order through LDS.  The
// self pair (s, s) carries sum w and the row count (the norms).  Bound by the
// gathers of two products a pair; the rows' own entries are loaded once a tile.  One thread a pair, and one an
// expert for the norms, walking every token was a chain of m dependent loads:
// 4096 tokens, top-8 of 128 experts took 1434 + 1361 us, now 16 + 5 us (30 with
// the rows' own entries loaded by every thread).
constexpr int kPairThreads = 1024, kPairBatch = 8;
constexpr int kPairRows = 128;  // tallest tile of the GEMM planner (wide tiles are listed in 128-row units)

__global__ __launch_bounds__(kPairThreads) void calib_pairs_kernel(
    const double *__restrict__ gram, const int16_t *__restrict__ pos, const int32_t *__restrict__ offsets,
    const int32_t *__restrict__ tile_start, const int32_t *__restrict__ row_token,
    const int32_t *__restrict__ row_slot, int bm, int N, int NP, int kr, double *__restrict__ part) {
  __shared__ double red[3][kPairThreads];
  __shared__ int redn[kPairThreads];
  __shared__ int tok[kPairRows], self[kPairRows];          // the rows' tokens and positions of s
  __shared__ double norm[kPairRows], square[kPairRows];    // ||u_s|| and its square
  const int b = blockIdx.x;
  if (b >= tile_start[N]) return;
  __shared__ int src;  // the source whose tiles hold b (one round trip: every thread tests one)
  if (threadIdx.x < N && tile_start[threadIdx.x] <= b && b < tile_start[threadIdx.x + 1]) src = threadIdx.x;
  __syncthreads();
  const int s = src;
  const int r0 = offsets[s] + (b - tile_start[s]) * bm, r1 = min(r0 + bm, offsets[s + 1]);
  const int rows = r1 - r0;  // at most bm <= kPairRows (launch_calib_finalize)
  if ((int)threadIdx.x < rows) {
    const int i = row_token[r0 + threadIdx.x], a = row_slot[r0 + threadIdx.x] - i * kr;
    const double uu = gram[((long long)i * kr + a) * kr + a];
    tok[threadIdx.x] = i;
    self[threadIdx.x] = a;
    square[threadIdx.x] = uu;
    norm[threadIdx.x] = sqrt(uu);
  }
  __syncthreads();
  const int G = kPairThreads / NP, g = threadIdx.x / NP, t = threadIdx.x % NP;
  const int per = (rows + G - 1) / G;
  const int q0 = g * per, q1 = min(q0 + per, rows);
  double A = 0.0, V = 0.0, C = 0.0;
  int n = 0;
  if (t < N)
    for (int q = q0; q < q1; q += kPairBatch) {
      // loads of a batch of rows issued together: positions, then the products
      int pb[kPairBatch];
      double uv[kPairBatch], vv[kPairBatch];
#pragma unroll
      for (int u = 0; u < kPairBatch; ++u) pb[u] = q + u < q1 ? pos[(long long)tok[q + u] * N + t] : -1;
#pragma unroll
      for (int u = 0; u < kPairBatch; ++u)
        if (pb[u] >= 0) {
          const double *Gi = gram + (long long)tok[q + u] * kr * kr;
          uv[u] = Gi[self[q + u] * kr + pb[u]];
          vv[u] = Gi[pb[u] * kr + pb[u]];
        }
#pragma unroll
      for (int u = 0; u < kPairBatch; ++u)
        if (pb[u] >= 0) {
          const double w = norm[q + u];
          if (t == s) {
            A += w;
          } else {
            A += w * uv[u];
            V += w * vv[u];
            C += w * square[q + u];
          }
          ++n;
        }
    }
  red[0][threadIdx.x] = A;
  red[1][threadIdx.x] = V;
  red[2][threadIdx.x] = C;
  redn[threadIdx.x] = n;
  __syncthreads();
  if (threadIdx.x >= N) return;
  for (int k = 1; k < G; ++k) {
    A += red[0][k * NP + threadIdx.x];
    V += red[1][k * NP + threadIdx.x];
    C += red[2][k * NP + threadIdx.x];
    n += redn[k * NP + threadIdx.x];
  }
  double *out = part + (long long)b * 4 * N + threadIdx.x;
  out[0] = A;
  out[N] = V;
  out[2 * N] = C;
  out[3 * N] = (double)n;
}

// Threads of the first N N / 256 blocks: one pair each (the tiles of its source
// in order).  Last block: the norms.
__global__ __launch_bounds__(256) void calib_finalize_kernel(const double *__restrict__ part,
                                                             const int32_t *__restrict__ tile_start, int m,
                                                             int N, double lambda, double clip,
                                                             float *__restrict__ S, float *__restrict__ L,
                                                             float *__restrict__ h,
                                                             double *__restrict__ stats) {
  if (blockIdx.x == gridDim.x - 1) {
    __shared__ double hv[kMaxExperts];
    __shared__ int seen[kMaxExperts];
    __shared__ double fill;
    const int e = threadIdx.x;
    if (e < N) {
      double sum = 0.0, cnt = 0.0;
      if (m > 0)
        for (int b = tile_start[e]; b < tile_start[e + 1]; ++b) {
          sum += part[(long long)b * 4 * N + e];
          cnt += part[(long long)b * 4 * N + 3 * N + e];
        }
      hv[e] = cnt > 0.0 ? sum / cnt : 0.0;
      seen[e] = cnt > 0.0;
    }
    __syncthreads();
    if (e < kWave) {  // mean of the observed norms, in a fixed association
      double sum = 0.0, cnt = 0.0;
      for (int x = e; x < N; x += kWave)
        if (seen[x]) {
          sum += hv[x];
          cnt += 1.0;
        }
      sum = wave_sum_f64(sum);
      cnt = wave_sum_f64(cnt);
      if (e == 0) fill = cnt > 0.0 ? sum / cnt : 0.0;
    }
    __syncthreads();
    if (e < N) h[e] = (float)(seen[e] ? hv[e] : fill);
    return;
  }
  const int idx = blockIdx.x * 256 + threadIdx.x;
  if (idx >= N * N) return;
  const int s = idx / N, t = idx % N;
  double A = 0.0, V = 0.0, C = 0.0, n = 0.0;
  if (s != t && m > 0)
    for (int b = tile_start[s]; b < tile_start[s + 1]; ++b) {
      const double *p = part + (long long)b * 4 * N + t;
      A += p[0];
      V += p[N];
      C += p[2 * N];
      n += p[3 * N];
    }
  double sc, lo;
  if (s == t) {
    sc = 1.0;
    lo = 0.0;
  } else if (n == 0.0) {
    sc = 0.0;
    lo = 1e30;
  } else {
    const double den = V + lambda;
    sc = (den != 0.0) ? A / den : 0.0;
    if (clip > 0.0) sc = fmin(fmax(sc, -clip), clip);
    const double resid = C - 2.0 * sc * A + sc * sc * V;
    lo = fmax(0.0, resid) / (C + 1e-12);
  }
  S[idx] = (float)sc;
  L[idx] = (float)lo;
  if (stats) {
    stats[4LL * idx + 0] = A;
    stats[4LL * idx + 1] = V;
    stats[4LL * idx + 2] = C;
    stats[4LL * idx + 3] = n;
  }
}

size_t calib_partial_doubles(int rows, int N, int bm) { return (size_t)(rows / bm + N) * 4 * N; }

hipError_t launch_calib_finalize(const double *gram, const int16_t *pos, const PermBuffers &pb, int bm, int m,
                                 int N, int kr, double lambda, double clip, double *part, float *S, float *L,
                                 float *h, double *pair_stats, hipStream_t s) {
  if (m > 0) {
    // calib_pairs_kernel holds a tile's rows in LDS
    if (bm < 1 || bm > kPairRows) return hipErrorInvalidValue;
    int NP = 64;
    while (NP < N) NP *= 2;
    calib_pairs_kernel<<<m * kr / bm + N, kPairThreads, 0, s>>>(gram, pos, pb.offsets, pb.tile_start0,
                                                                pb.row_token, pb.row_slot, bm, N, NP, kr, part);
  }
  calib_finalize_kernel<<<(N * N + 255) / 256 + 1, 256, 0, s>>>(part, pb.tile_start0, m, N, lambda, clip, S, L,
                                                                h, pair_stats);
  return hipGetLastError();
}

}  // namespace exfold
