// Householder QR of the FP32 factorization, one half block (QR_HB columns) at
// a time, from Gram matrices (included by la.hip).
//
// A panel of QR_NB columns splits into its top block A1 (QR_NB rows) and its
// tail A2 (all rows below).  Every inner product the reflectors need is a
// combination of A1's entries and of the tail's Gram matrix A2^H A2, so the
// panel is factored from these 32 x 32 blocks alone: the factorization leaves
// R, V1 (the reflectors' top rows), T, and an upper triangular X with
// V2 = A2 X for the tails.  With the Gram taken against the half's remaining
// columns too, W = T^H V^H A of their update comes from the same blocks, and
// [V2 | A2 W'] = A2 [X | X W] is one product.  Per panel that is one pass over
// the half's rows (qr_half_rows_kernel: the last panel's product, then the
// next panel's Gram of the rows just updated) and one small factorization
// (qr_half_factor_kernel), against 32 exchanges of column sums between
// workgroups and three products before.
//
// Accuracy: the Gram, the factorization of the blocks, X and the products
// with A2 are FP64, only A, V, R and T are rounded to FP32.  The squared norm
// left in column j, g = x^H G x with x = X e_j before scaling, carries the
// rounding of G's entries, about 1e-16 (sum_i |x_i| ||a_i||)^2.  Where that
// exceeds 3e-8 g (half of FP32's rounding; QRH_LOSS) the panel is split: the
// reflectors before column j are applied to the tails, and the rest goes on
// from a new Gram: by a row pass and another factorization launch where the
// caller expects such panels (the face-split generators of the first
// recompression stage, whose panels lose three to seven digits) and for the
// tallest ones, else by the factorization's workgroup itself.
//
// Bound: the blocks' factorization by its chain of 32 dependent columns
// (sqrt, reciprocal and two LDS round trips each), the row pass by the FP64
// matrix cores (10 to 20 kflop a row and panel); both are far from the memory
// rate.
#pragma once

namespace nd {
namespace {

constexpr int QRH_ROWS = 64;             // rows per step of the row pass
constexpr double QRH_LOSS = 4e-9;        // g >= QRH_LOSS (sum_i |x_i| ||a_i||)^2
constexpr int QRH_LD = QRH_ROWS + 2;     // LDS stride of a column (bank spread)
// columns of a panel's block row: the panel's at 0, the half's remaining ones
// from QR_NB on (a wide problem's last panel may have fewer than QR_NB columns
// and more than QR_HB - QR_NB remaining)
constexpr int QRH_W = QR_HB + QR_NB;
constexpr size_t QRH_XY = (size_t)QR_NB * QRH_W * sizeof(double2);
constexpr size_t QRH_A1 = (size_t)QR_NB * QRH_W * sizeof(float2);
constexpr int QRH_MAXC = 32;             // most row chunks (partial Grams) of a problem
// Tall panels, from QRH_TALL steps on in lists of few problems: more chunks, of
// four steps or more, with their partials in the pool's stream scratch (the
// workspace holds 13 at 128 columns).  A step of the row pass takes a workgroup
// 19 us, the sum of a chunk's partials 1 us, so a panel of 100 000 x 128 spent
// 2.3 ms on 13 of the device's 256 CUs.
constexpr int QRH_TALL = 64;
constexpr int QRH_MAXC_TALL = 128;
struct QrhPart {
  double2* tall;   // nullptr: the partials lie in the problems' scratch
  size_t stride;   // elements of a problem's partials there
  int maxc;        // most chunks of a problem
};

// A problem's scratch: the block W, W2, S of geqrf's workspace, which only the
// steps between halves use.  xy: [X | Y] (QR_NB x QRH_W, leading dimension
// QR_NB); a1: the panel's top rows (QR_NB x QRH_W); part: partial Grams,
// QR_NB x ncw each.
// A split panel's state between its passes: the top block, the reflectors' tau
// and the first column left (jb: the panel is done).
struct QrhState {
  double2 a[QR_NB * QR_NB], tau[QR_NB];
  int js;
};
constexpr size_t QRH_ST = (sizeof(QrhState) + 255) / 256 * 256;
struct QrhScratch {
  double2* xy;
  QrhState* st[2];   // by parity of the pass that wrote it
  float2* a1;
  double2* part;
  int ncw, cap;
};
__device__ inline QrhScratch qrh_scratch(const QRDesc<float>& d, int prob, int H0,
                                         const QrhPart& pp) {
  const size_t el = (size_t)2 * QR_OB * max(d.n, 1) + (size_t)QR_OB * QR_OB;
  char* base = (char*)(d.Tw - el);
  QrhScratch s;
  s.ncw = (min(d.n - H0, QR_HB) + 15) / 16 * 16;
  s.ncw = max(s.ncw, QR_NB);
  s.xy = (double2*)base;
  s.a1 = (float2*)(base + QRH_XY);
  s.st[0] = (QrhState*)(base + QRH_XY + QRH_A1);
  s.st[1] = (QrhState*)(base + QRH_XY + QRH_A1 + QRH_ST);
  s.part = (double2*)(base + QRH_XY + QRH_A1 + 2 * QRH_ST);
  s.cap = (int)((el * sizeof(float2) - QRH_XY - QRH_A1 - 2 * QRH_ST) /
                (sizeof(double2) * QR_NB * s.ncw));
  if (pp.tall) {
    s.part = pp.tall + prob * pp.stride;
    s.cap = (int)(pp.stride / (QR_NB * s.ncw));
  }
  return s;
}
// row chunks of `rows` rows: their number and the steps of each
__host__ __device__ inline int qrh_chunks(int rows, int maxc, int cap, int& per) {
  const int sub = (rows + QRH_ROWS - 1) / QRH_ROWS;
  int mc = maxc < cap ? maxc : cap;
  if (mc > QRH_MAXC) mc = sub / 4 > QRH_MAXC ? (sub / 4 < mc ? sub / 4 : mc) : QRH_MAXC;
  per = (sub + mc - 1) / mc;
  per = per > 1 ? per : 1;
  return (sub + per - 1) / per;
}

__device__ __forceinline__ void mfma_c(double2 a, double2 b, dbl4& re, dbl4& im) {
  re = mfma16(a.x, b.x, re);
  im = mfma16(a.x, b.y, im);
  re = mfma16(-a.y, b.y, re);
  im = mfma16(a.y, b.x, im);
}
__device__ __forceinline__ double2 widen(float2 v) { return make_double2((double)v.x, (double)v.y); }
__device__ __forceinline__ float2 narrow(double x, double y) {
  return make_float2((float)x, (float)y);
}

// A 32 x 32 block in the registers of four waves, as mm32 leaves it: rows
// 16 (wave / 2) + lane / 16 + 4 v of column 16 (wave % 2) + lane % 16
struct Tile {
  dbl4 re, im;
};
__device__ __forceinline__ int tile_row(int v) {
  return 16 * (threadIdx.x >> 7) + ((threadIdx.x & 63) >> 4) + 4 * v;
}
__device__ __forceinline__ int tile_col() {
  return 16 * ((threadIdx.x >> 6) & 1) + (threadIdx.x & 15);
}
// One step's rows of the Gram of the first QR_NB columns of An (their rows from
// jb on, counted from the panel's first) against all 16 ctile: wave w takes the
// rows' half w % 2 against column tiles w / 2, w / 2 + 2, ..., so that all four
// have work from two tiles on (with a wave per column tile two had none at the
// end of a half: 1000 of 300 x 64 with the columns' update 299 -> 267 us).
__device__ __forceinline__ void qrh_gram_step(const float2 (&An)[QR_HB][QRH_LD], int ctile, int r0,
                                              int jb, dbl4 (&gr)[4], dbl4 (&gi)[4]) {
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lo = lane & 15, hi = lane >> 4, a = wave & 1;
  if (a >= ctile) return;
  auto rows = [&](int s) {
    const int r = 4 * s + hi;
    double2 v = make_double2(0.0, 0.0);
    if (r0 + r >= jb) v = widen(An[16 * a + lo][r]);
    v.y = -v.y;
    return v;
  };
  // two tiles at a time (four chains of matrix instructions), then one
#pragma unroll
  for (int t = 0; t < 4; t += 2) {
    const int tile = (wave >> 1) + 2 * t;
    if (tile + 2 < ctile) {
#pragma unroll 4
      for (int s = 0; s < QRH_ROWS / 4; ++s) {
        const double2 v = rows(s);
        mfma_c(v, widen(An[16 * tile + lo][4 * s + hi]), gr[t], gi[t]);
        mfma_c(v, widen(An[16 * tile + 32 + lo][4 * s + hi]), gr[t + 1], gi[t + 1]);
      }
    } else if (tile < ctile) {
#pragma unroll 4
      for (int s = 0; s < QRH_ROWS / 4; ++s)
        mfma_c(rows(s), widen(An[16 * tile + lo][4 * s + hi]), gr[t], gi[t]);
    }
  }
}
__device__ __forceinline__ void qrh_gram_store(double2* part, int ctile, const dbl4 (&gr)[4],
                                               const dbl4 (&gi)[4]) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, a = wave & 1;
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    const int tile = (wave >> 1) + 2 * t;
    if (tile >= ctile) continue;
#pragma unroll
    for (int v = 0; v < 4; ++v)
      stc(part + 16 * a + (lane >> 4) + 4 * v + (size_t)QR_NB * (16 * tile + (lane & 15)),
          make_double2(gr[t][v], gi[t][v]));
  }
}

// The rows from the end of the panel before j1 (PREV) on: with that panel's
// [X | Y], V2 = A2 X replaces the panel's tail and A2 Y leaves the half's
// remaining columns; then, where a panel starts at j1, the Gram of its tail
// against these columns, one partial per workgroup, and a copy of its top
// rows.  Without PREV: the first panel's Gram alone (j1 = H0).
template <bool PREV, class AS>
__global__ __launch_bounds__(256, 2) void qr_half_rows_kernel(
    const QRDesc<float>* __restrict__ descs, AS active, int H0, int j1, QrhPart pp) {
  __shared__ float2 An[QR_HB][QRH_LD];
  const QRDesc<float> d = descs[active[blockIdx.y]];
  const int kmin = min(d.m, d.n), hend = min(d.n, H0 + QR_HB);
  const int j0 = j1 - QR_NB;
  const int jb = PREV ? min(QR_NB, kmin - j0) : 0;    // columns of the last panel
  const int rb = PREV ? j0 + jb : H0;                  // first row, first remaining column
  const int nc = max(hend - rb, 0);
  const bool next = (!PREV || jb == QR_NB) && j1 < min(kmin, H0 + QR_HB);
  const int jbn = next ? min(QR_NB, kmin - j1) : 0;
  const int rows = d.m - rb;
  const QrhScratch sc = qrh_scratch(d, active[blockIdx.y], H0, pp);
  int per;
  const int nck = qrh_chunks(rows, pp.maxc, sc.cap, per);
  if ((int)blockIdx.x >= max(nck, 1)) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int lo = lane & 15, hi = lane >> 4;
  const int ntile = PREV ? 2 + (nc + 15) / 16 : 0;     // [panel | remaining columns]
  const int ctile = (nc + 15) / 16;
  // this wave's column tiles: wave, wave + 4
  double2 xy[2][8];
  if constexpr (PREV) {
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int s = 0; s < 8; ++s) {
        const int k = 4 * s + hi, c = 16 * (wave + 4 * t) + lo;
        xy[t][s] = wave + 4 * t < ntile && k < jb ? ldc(sc.xy + k + (size_t)QR_NB * c)
                                                  : make_double2(0.0, 0.0);
      }
  }
  dbl4 gr[4], gi[4];
#pragma unroll
  for (int t = 0; t < 4; ++t) gr[t] = gi[t] = dbl4{0, 0, 0, 0};
  float2* Ap = d.A + rb + (int64_t)j0 * d.lda;         // the panel's tail
  float2* Ac = d.A + rb + (int64_t)rb * d.lda;         // the remaining columns
  const int r1 = min(rows, ((int)blockIdx.x + 1) * per * QRH_ROWS);
  for (int r0 = blockIdx.x * per * QRH_ROWS; r0 < r1; r0 += QRH_ROWS) {
    if constexpr (PREV) {
      // 16 rows at a time (registers)
#pragma unroll 1
      for (int h = 0; h < QRH_ROWS; h += 16) {
        const int r = r0 + h + lo;
        float2 ap[8], old[2][4];
#pragma unroll
        for (int s = 0; s < 8; ++s) {
          const int k = 4 * s + hi;
          ap[s] = r < rows && k < jb ? ldc(Ap + r + (int64_t)k * d.lda) : make_float2(0.f, 0.f);
        }
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            const int c = 16 * (wave + 4 * t - 2) + hi + 4 * v;
            old[t][v] = r < rows && c >= 0 && c < nc ? ldc(Ac + r + (int64_t)c * d.lda)
                                                     : make_float2(0.f, 0.f);
          }
        __syncthreads();   // every wave has read these rows of the panel; An is free
#pragma unroll
        for (int t = 0; t < 2; ++t) {
          const int tile = wave + 4 * t;
          if (tile >= ntile) continue;
          // D(column, row): 16 consecutive rows a column in the lanes
          dbl4 re = {0, 0, 0, 0}, im = {0, 0, 0, 0};
#pragma unroll
          for (int s = 0; s < 8; ++s) mfma_c(xy[t][s], widen(ap[s]), re, im);
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            if (tile < 2) {
              const int c = 16 * tile + hi + 4 * v;
              if (r < rows && c < jb) stc(Ap + r + (int64_t)c * d.lda, narrow(re[v], im[v]));
            } else {
              const int c = 16 * (tile - 2) + hi + 4 * v;
              const float2 n =
                  narrow((double)old[t][v].x - re[v], (double)old[t][v].y - im[v]);
              if (r < rows && c < nc) stc(Ac + r + (int64_t)c * d.lda, n);
              An[c][h + lo] = n;   // zero past the rows and columns
            }
          }
        }
      }
    } else {
      __syncthreads();
      for (int e = tid; e < 16 * ctile * QRH_ROWS; e += 256) {
        const int r = e % QRH_ROWS, c = e / QRH_ROWS;
        An[c][r] = r0 + r < rows && c < nc ? ldc(Ac + r0 + r + (int64_t)c * d.lda)
                                           : make_float2(0.f, 0.f);
      }
    }
    if (!next) continue;   // uniform over the workgroup
    __syncthreads();
    if (r0 == 0)
      for (int e = tid; e < QR_NB * QRH_W; e += 256) {
        const int i = e % QR_NB, c = e / QR_NB;
        const int cc = c < QR_NB ? c : jbn + c - QR_NB;
        const bool ok = i < jbn && cc < nc && (c >= QR_NB || c < jbn);
        stc(sc.a1 + e, ok ? An[cc][i] : make_float2(0.f, 0.f));
      }
    qrh_gram_step(An, ctile, r0, jbn, gr, gi);
  }
  if (!next) return;
  qrh_gram_store(sc.part + (size_t)blockIdx.x * QR_NB * sc.ncw, ctile, gr, gi);
}

// The row pass of a split panel: A2 <- A2 X on its tail (X is the identity on
// the final columns), and the new Gram against the half's remaining columns.
template <class AS>
__global__ __launch_bounds__(256, 2) void qr_half_split_kernel(
    const QRDesc<float>* __restrict__ descs, AS active, int H0, int j0, QrhPart pp, int pass) {
  __shared__ float2 An[QR_HB][QRH_LD];
  const QRDesc<float> d = descs[active[blockIdx.y]];
  const int jb = min(QR_NB, min(d.m, d.n) - j0), rows = d.m - j0;
  const int nc = min(d.n, H0 + QR_HB) - j0, ctile = (nc + 15) / 16;
  const QrhScratch sc = qrh_scratch(d, active[blockIdx.y], H0, pp);
  int per;
  const int nck = qrh_chunks(rows, pp.maxc, sc.cap, per);
  if ((int)blockIdx.x >= nck || sc.st[pass & 1]->js == jb) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int lo = lane & 15, hi = lane >> 4;
  float2* Ap = d.A + j0 + (int64_t)j0 * d.lda;
  dbl4 gr[4], gi[4];
#pragma unroll
  for (int t = 0; t < 4; ++t) gr[t] = gi[t] = dbl4{0, 0, 0, 0};
  const int r1 = min(rows, ((int)blockIdx.x + 1) * per * QRH_ROWS);
  for (int r0 = blockIdx.x * per * QRH_ROWS; r0 < r1; r0 += QRH_ROWS) {
    __syncthreads();
    for (int e = tid; e < 16 * ctile * QRH_ROWS; e += 256) {
      const int r = e % QRH_ROWS, c = e / QRH_ROWS;
      if (c >= jb)
        An[c][r] = r0 + r < rows && c < nc ? ldc(Ap + r0 + r + (int64_t)c * d.lda)
                                           : make_float2(0.f, 0.f);
    }
    const int r = r0 + 16 * wave + lo;   // a wave its own 16 rows of the panel
    const bool tail = r >= jb && r < rows;
    float2 ap[8];
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      const int k = 4 * s + hi;
      ap[s] = tail && k < jb ? ldc(Ap + r + (int64_t)k * d.lda) : make_float2(0.f, 0.f);
    }
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      dbl4 re = {0, 0, 0, 0}, im = {0, 0, 0, 0};
#pragma unroll
      for (int s = 0; s < 8; ++s)
        mfma_c(ldc(sc.xy + 4 * s + hi + QR_NB * (16 * t + lo)), widen(ap[s]), re, im);
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int c = 16 * t + hi + 4 * v;
        const float2 n = narrow(re[v], im[v]);
        if (tail && c < jb) stc(Ap + r + (int64_t)c * d.lda, n);
        if (c < jb) An[c][16 * wave + lo] = n;
      }
    }
    __syncthreads();
    qrh_gram_step(An, ctile, r0, jb, gr, gi);
  }
  qrh_gram_store(sc.part + (size_t)blockIdx.x * QR_NB * sc.ncw, ctile, gr, gi);
}

// D = sum_k fa(i, k) fb(k, j), 32 x 32, by four waves (one 16 x 16 tile each):
// element (16 (wave / 2) + lane / 16 + 4 v, 16 (wave % 2) + lane % 16) in
// register v
template <class FA, class FB>
__device__ __forceinline__ void mm32(FA fa, FB fb, dbl4& re, dbl4& im) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int i = 16 * (wave >> 1) + (lane & 15), j = 16 * (wave & 1) + (lane & 15);
#pragma unroll
  for (int s = 0; s < 8; ++s) {
    const int k = 4 * s + (lane >> 4);
    mfma_c(fa(i, k), fb(k, j), re, im);
  }
}
template <class F>
__device__ __forceinline__ void mm32_out(const dbl4& re, const dbl4& im, F put) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int v = 0; v < 4; ++v)
    put(16 * (wave >> 1) + (lane >> 4) + 4 * v, 16 * (wave & 1) + (lane & 15),
        make_double2(re[v], im[v]));
}

typedef double2 (*Blk)[QR_NB + 1];
struct QrhLds {
  double2 G[QR_NB][QR_NB + 1];    // tail Gram, then T
  double2 X[QR_NB][QR_NB + 1];
  double2 P[QR_NB][QR_NB + 1];    // temporaries
  union {
    double2 Q[QR_NB][QR_NB + 1];
    struct {                      // while the columns are factored
      double2 row[2][4][QR_NB];   // pivot row of the Gram, of A1, pivot column of A1, of X
    };
  };
  float2 V[QR_NB][QR_NB + 1];     // V1, explicit unit lower
  double2 tau[QR_NB], scal[QR_NB];
  double norm[QR_NB], beta[QR_NB];
};

// 1 / sqrt(v) and 1 / v of positive normal v: the hardware's estimates and two
// Newton steps
__device__ __forceinline__ double rsqrt64(double v) {
  double y = __builtin_amdgcn_rsq(v);
#pragma unroll
  for (int i = 0; i < 2; ++i) y = fma(0.5 * y, fma(-v * y, y, 1.0), y);
  return y;
}
__device__ __forceinline__ double rcp64(double v) {
  double y = __builtin_amdgcn_rcp(v);
#pragma unroll
  for (int i = 0; i < 2; ++i) y = fma(y, fma(-v, y, 1.0), y);
  return y;
}

// t -= p q^T (conj(p) with CJ): one 4-step product for the real and one for the
// imaginary part; p's rows and q's columns come one a lane (lane % 16), the
// lanes of k = 0 hold the first term of each product, those of k = 1 the second;
// q is zero in the lanes of k = 2, 3
template <bool CJ>
__device__ __forceinline__ void rank1_sub(Tile& t, double2 p, double2 q) {
  const bool odd = (threadIdx.x & 16) != 0;
  const double px = -p.x, py = CJ ? -p.y : p.y;
  const double qa = odd ? q.y : q.x, qb = odd ? q.x : q.y;
  t.re = mfma16(odd ? py : px, qa, t.re);
  t.im = mfma16(odd ? -py : px, qb, t.im);
}

// Panel columns js .. of the blocks: g the Gram over the rows from the pivot
// on, a the top block (A1 / R / V1), x the tails' transform.  The pivot
// column's reflector is kept unscaled, (alpha - beta, x): its multiples f are
// all the other columns need, so a step is three rank-one updates on the
// matrix cores; tiles that no later step reads are left as they are.  A step is
// a chain: of its some 2500 clk the reads of LDS take 300, the split test 270, the
// scalars 260, the multiples and updates 780, publishing the next pivot 530 and
// the barrier 350.  So everything uniform is scalar, and a lane derives the
// multiples of one column of its tile (the wave of the off-diagonal tile of g
// two): 2800 clk a step before, 8 panels of 600 x 128 66 -> 62 us, 1000 of 300 x 64
// 345 -> 310.  With the updates one step late, beside the next step's scalars,
// the corrections of what that step reads cost more than the updates' latency.
// On return the columns js .. j - 1 of a (rows below the diagonal) and of x are scaled
// to v_0 = 1 and a's diagonal holds R.  Returns the first column whose Gram has
// lost too much (QRH_LOSS; jb when none has; column js itself is always taken).
__device__ inline int qrh_factor(QrhLds& S, Tile& g, Tile& a, Tile& x, int js, int jb) {
  const int tid = threadIdx.x, lane = tid & 63, lo = lane & 15, hi = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), ti = wave >> 1, tj = wave & 1;
  const int c1 = 16 * tj + lo, c2 = 16 * ti + lo;
  const double2 z = make_double2(0.0, 0.0);
  js = __builtin_amdgcn_readfirstlane(js);
  jb = __builtin_amdgcn_readfirstlane(jb);
  // row j of the Gram and of A1, column j of A1 and of X, as the tiles hold them
  auto publish = [&](int j) {
    double2(*p)[QR_NB] = S.row[j & 1];
    if (j >> 4 == ti) {
      const int w = (j >> 2) & 3;
      const double2 gv = w == 0   ? make_double2(g.re[0], g.im[0])
                         : w == 1 ? make_double2(g.re[1], g.im[1])
                         : w == 2 ? make_double2(g.re[2], g.im[2])
                                  : make_double2(g.re[3], g.im[3]);
      const double2 av = w == 0   ? make_double2(a.re[0], a.im[0])
                         : w == 1 ? make_double2(a.re[1], a.im[1])
                         : w == 2 ? make_double2(a.re[2], a.im[2])
                                  : make_double2(a.re[3], a.im[3]);
      if (hi == (j & 3)) {
        p[0][c1] = gv;
        p[1][c1] = av;
      }
    }
    if (j >> 4 == tj && lo == (j & 15)) {
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int i = 16 * ti + hi + 4 * v;
        p[2][i] = make_double2(a.re[v], a.im[v]);
        p[3][i] = make_double2(x.re[v], x.im[v]);
      }
    }
  };
#pragma unroll
  for (int v = 0; v < 4; ++v)
    if (tile_row(v) == c1) S.norm[c1] = sqrt(fmax(g.re[v], 0.0));
  publish(js);
  __syncthreads();
  const double n0 = S.norm[lo], n1 = S.norm[16 + lo];   // the columns' norms at js
  int j = js;
  for (; j < jb; ++j) {
    double2(*p)[QR_NB] = S.row[j & 1];
    const double gjj = p[0][j].x;
    const double2 al = p[1][j];
    const double2 rg1 = p[0][c1], ra1 = p[1][c1];
    double2 ca = p[2][c2];
    const double2 x0 = p[3][lo], x1 = p[3][16 + lo], cx = ti ? x1 : x0;
    // sum_i |x_i| ||a_i|| over the pivot column of X: lane 0's order of the sum, the
    // same in every wave (all take the same turn below)
    double wx = fma(fabs(x0.x) + fabs(x0.y), n0, (fabs(x1.x) + fabs(x1.y)) * n1);
    wx += dpp_get<0x121, 0xF>(wx);
    wx += dpp_get<0x122, 0xF>(wx);
    wx += dpp_get<0x124, 0xF>(wx);
    wx += dpp_get<0x128, 0xF>(wx);
    if (j > js && __builtin_amdgcn_readfirstlane((int)!(gjj >= QRH_LOSS * wx * wx))) break;
    // squared norm from the pivot on: gjj, and no less than |alpha|^2; beta =
    // -sign(Re alpha) nrm, tau = 1 - alpha / beta, scal = 1 / (alpha - beta)
    const double a2 = fma(al.x, al.x, al.y * al.y), nn = fmax(gjj, a2);
    const double rn = rsqrt64(nn), nrm = nn * rn, ax = fabs(al.x);
    const double id = rcp64(fma(2.0 * nrm, ax, nn + a2));   // 1 / |alpha - beta|^2
    const bool none = !(gjj > a2) && al.y == 0.0;           // nothing below the pivot: H = I
    const double beta = none ? al.x : al.x >= 0.0 ? -nrm : nrm;
    const double dx = al.x - beta;
    double2 tau = make_double2(fma(ax, rn, 1.0), al.x >= 0.0 ? al.y * rn : -al.y * rn);
    double2 scal = make_double2(dx * id, -al.y * id);
    if (__builtin_amdgcn_readfirstlane((int)none)) tau = scal = z;
    if (tid == 0) {
      S.tau[j] = tau;
      S.scal[j] = scal;
      S.beta[j] = beta;
    }
    // column c: u = v^H a_c over the reflector's rows, tu = conj(tau) u, its
    // row of R and its multiple f of the unscaled reflector
    auto tu_of = [&](double2 rg, double2 ra) {
      return cmulc(tau, cadd(ra, cmulc(scal, csub(rg, cmulc(al, ra)))));
    };
    if (j < 16 * tj + 15) {   // this wave's columns reach past the pivot
      const double2 tu1 = tu_of(rg1, ra1);
      // lanes 32 .. 63 hold k = 2, 3 of the updates: zero
      const bool on = c1 > j && lane < 32;
      const double2 f = on ? cmul(scal, tu1) : z;
      const double2 r1 = on ? csub(ra1, tu1) : z;
      rank1_sub<false>(x, cx, f);
      if (j < 16 * ti + 16) {
        ca = c2 > j ? ca : c2 == j ? make_double2(dx, al.y) : z;
        rank1_sub<false>(a, ca, f);
        if (ti <= tj) {
          double2 r2 = r1;
          if (ti < tj) {
            const double2 rg2 = p[0][c2], ra2 = p[1][c2];
            r2 = csub(ra2, tu_of(rg2, ra2));
          }
          if (!(c2 > j)) r2 = z;
          rank1_sub<true>(g, r2, r1);
        }
      }
    }
    if (j + 1 < jb) publish(j + 1);
    __syncthreads();
  }
  __syncthreads();
  if (c1 >= js && c1 < j) {
    const double2 scal = S.scal[c1];
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int i = tile_row(v);
      const double2 xs = cmul(make_double2(x.re[v], x.im[v]), scal);
      const double2 as = cmul(make_double2(a.re[v], a.im[v]), scal);
      x.re[v] = xs.x;
      x.im[v] = xs.y;
      if (i > c1) {
        a.re[v] = as.x;
        a.im[v] = as.y;
      } else if (i == c1) {
        a.re[v] = S.beta[c1];
        a.im[v] = 0.0;
      }
    }
  }
  __syncthreads();
  return j;
}

// The s x s blocks right of each even inverted s x s diagonal block of the unit
// upper triangle S.G: B <- -M1 (B M2); 16 s entries, one a thread.  The sums run
// over whole blocks (the triangles' zeros are stored), so that their reads of
// LDS go out together.
template <int s>
__device__ inline void qrh_inv_level(QrhLds& S) {
  const int tid = threadIdx.x, blk = tid / (s * s), e = tid % (s * s);
  const int i = e % s, c = e / s, r0 = 2 * s * blk, c0 = r0 + s;
  const bool on = tid < 16 * s;
  __syncthreads();
  if (on) {
    double2 t = make_double2(0.0, 0.0);
#pragma unroll
    for (int k = 0; k < s; ++k) t = cadd(t, cmul(S.G[r0 + i][c0 + k], S.G[c0 + k][c0 + c]));
    S.Q[r0 + i][c0 + c] = t;
  }
  __syncthreads();
  if (on) {
    double2 t = make_double2(0.0, 0.0);
#pragma unroll
    for (int k = 0; k < s; ++k) t = cadd(t, cmul(S.G[r0 + i][r0 + k], S.Q[r0 + k][c0 + c]));
    S.G[r0 + i][c0 + c] = make_double2(-t.x, -t.y);
  }
}

// S.G holds V^H V (32 x 32): replaced by T = (I + D striu(V^H V))^{-1} D, D =
// diag(tau), the unit upper triangle inverted by doubling its inverted blocks
__device__ inline void qrh_t_factor(QrhLds& S) {
  const int tid = threadIdx.x;
  for (int e = tid; e < QR_NB * QR_NB; e += 256) {
    const int i = e & 31, c = e >> 5;
    const double2 z = make_double2(0.0, 0.0);
    S.G[i][c] = i < c ? cmul(S.tau[i], S.G[i][c]) : i == c ? make_double2(1.0, 0.0) : z;
  }
  qrh_inv_level<1>(S);
  qrh_inv_level<2>(S);
  qrh_inv_level<4>(S);
  qrh_inv_level<8>(S);
  qrh_inv_level<16>(S);
  __syncthreads();
  for (int e = tid; e < QR_NB * QR_NB; e += 256) {
    const int i = e & 31, c = e >> 5;
    S.G[i][c] = cmul(S.G[i][c], S.tau[c]);
  }
  __syncthreads();
}

// C(i, c) = sum over rows of conj(V(r, i)) B(r, c) for 32 x 32 columns, read
// from memory by one workgroup
__device__ inline void qrh_gram_rows(const float2* V, int nv, const float2* B, int nbc, int64_t ld,
                                     int rows, dbl4& re, dbl4& im) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int i = 16 * (wave >> 1) + (lane & 15), j = 16 * (wave & 1) + (lane & 15);
  for (int r0 = 0; r0 < rows; r0 += 32) {
    float2 v[8], b[8];
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      const int r = r0 + 4 * s + (lane >> 4);
      v[s] = r < rows && i < nv ? ldc(V + r + i * ld) : make_float2(0.f, 0.f);
      b[s] = r < rows && j < nbc ? ldc(B + r + j * ld) : make_float2(0.f, 0.f);
    }
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      double2 w = widen(v[s]);
      w.y = -w.y;
      mfma_c(w, widen(b[s]), re, im);
    }
  }
}

// Panel [j0, j0 + 32) of each problem from the partial Grams and the copy of
// its top rows.  Workgroups x of a problem factor the same blocks and take the
// remaining columns' blocks of 32 x, x + (gridDim.x - 1), ...; the last one
// moves the rows above the panel inside its block of QR_OB columns from A to
// R (see geqrf_batched).  pass > 0 goes on with the panels that the pass before
// split (their state is in the scratch); with `more` another pass follows, else
// a split panel is finished here, by workgroup 0.
template <class AS>
__global__ __launch_bounds__(256, 2) void qr_half_factor_kernel(
    const QRDesc<float>* __restrict__ descs, AS active, int H0, int j0, QrhPart pp, int pass,
    bool more) {
  __shared__ QrhLds S;
  const QRDesc<float> d = descs[active[blockIdx.y]];
  const int kmin = min(d.m, d.n), hend = min(d.n, H0 + QR_HB);
  const int jb = min(QR_NB, kmin - j0);
  const int nt = max(hend - j0 - jb, 0), nq = (nt + QR_NB - 1) / QR_NB;
  const int tid = threadIdx.x, c = tid & 31, ig = tid >> 5;
  const int nw = gridDim.x - 1;
  if ((int)blockIdx.x == nw) {
    if (pass > 0) return;
    const int J0 = j0 - j0 % QR_OB, na = j0 - J0;
    for (int e = tid; e < jb * na; e += 256) {
      const int r = J0 + e % na, cc = j0 + e / na;
      float2* pa = d.A + r + (int64_t)cc * d.lda;
      stc(d.R + r + (int64_t)cc * d.ldr, ldc(pa));
      stc(pa, make_float2(0.f, 0.f));
    }
    return;
  }
  if (blockIdx.x > 0 && (int)blockIdx.x >= nq) return;
  const bool first = blockIdx.x == 0;
  const QrhScratch sc = qrh_scratch(d, active[blockIdx.y], H0, pp);
  const int rows = d.m - j0;
  QrhState* const out = sc.st[pass & 1];
  const QrhState* const in = sc.st[(pass & 1) ^ 1];
  int js = pass > 0 ? in->js : 0;
  if (pass > 0 && js == jb) {
    if (first && tid == 0) out->js = jb;
    return;
  }
  int per;
  const int nck = qrh_chunks(rows, pp.maxc, sc.cap, per);
  // sum of the partial Grams' columns c0 .. c0 + 31 (n of them) into B
  auto load_gram = [&](Blk B, int c0, int n) {
    double2 s[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) s[k] = make_double2(0.0, 0.0);
    const double2* p = sc.part + (size_t)QR_NB * c0 + tid;
    for (int z = 0; z < nck; z += 8) {   // 32 loads in flight
      double2 v[8][4];
#pragma unroll
      for (int y = 0; y < 8; ++y)
#pragma unroll
        for (int k = 0; k < 4; ++k)
          v[y][k] = z + y < nck && ig + 8 * k < n
                        ? ldc(p + (size_t)(z + y) * QR_NB * sc.ncw + 256 * k)
                        : make_double2(0.0, 0.0);
#pragma unroll
      for (int y = 0; y < 8; ++y)
#pragma unroll
        for (int k = 0; k < 4; ++k) s[k] = cadd(s[k], v[y][k]);
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) B[c][ig + 8 * k] = s[k];   // row c, column ig + 8 k
  };
  Tile g, a, x;
  load_gram((Blk)S.G, 0, jb);
#pragma unroll
  for (int k = 0; k < 4; ++k)
    S.P[c][ig + 8 * k] = pass > 0 ? ldc(in->a + tid + 256 * k) : widen(ldc(sc.a1 + tid + 256 * k));
  if (pass > 0 && tid < QR_NB) S.tau[tid] = in->tau[tid];
  __syncthreads();
  // register tiles to and from LDS
  auto put = [&](Blk B, const Tile& t) {
#pragma unroll
    for (int v = 0; v < 4; ++v) B[tile_row(v)][tile_col()] = make_double2(t.re[v], t.im[v]);
  };
  auto identity = [&](Tile& t) {
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      t.re[v] = tile_row(v) == tile_col() ? 1.0 : 0.0;
      t.im[v] = 0.0;
    }
  };
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const double2 p = S.P[tile_row(v)][tile_col()];
    a.re[v] = p.x;
    a.im[v] = p.y;
  }
  identity(x);
  // Gram over all rows from js on: the tail's and the top block's
  auto total_gram = [&](int js) {
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const double2 t = S.G[tile_row(v)][tile_col()];
      g.re[v] = t.x;
      g.im[v] = t.y;
    }
    mm32([&](int i, int k) { return k >= js ? cconj(S.P[k][i]) : make_double2(0.0, 0.0); },
         [&](int k, int j) { return S.P[k][j]; }, g.re, g.im);
  };
  total_gram(js);
  js = qrh_factor(S, g, a, x, js, jb);
  float2* A2 = d.A + j0 + jb + (int64_t)j0 * d.lda;    // tails
  float2* Ar = d.A + j0 + (int64_t)(j0 + jb) * d.lda;  // remaining columns
  const int rt = rows - jb;
  if (js < jb && more) {
    put((Blk)S.X, x);
    put((Blk)S.P, a);
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      stc(sc.xy + tid + 256 * k, S.X[c][ig + 8 * k]);
      stc(out->a + tid + 256 * k, S.P[c][ig + 8 * k]);
    }
    if (tid < QR_NB) out->tau[tid] = S.tau[tid];
    if (tid == 0) out->js = js;
    return;
  }
  if (first && tid == 0) out->js = jb;
  auto apply_x = [&]() {
    // A2 <- A2 X in place, a wave its own 16 rows, and the new tails' Gram
    const int lane = tid & 63, wave = tid >> 6, lo = lane & 15, hi = lane >> 4;
    for (int r0 = 16 * wave; r0 < rt; r0 += 64) {
      float2 ap[8];
      const int r = r0 + lo;
#pragma unroll
      for (int s = 0; s < 8; ++s) {
        const int k = 4 * s + hi;
        ap[s] = r < rt && k < jb ? ldc(A2 + r + (int64_t)k * d.lda) : make_float2(0.f, 0.f);
      }
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        dbl4 re = {0, 0, 0, 0}, im = {0, 0, 0, 0};
#pragma unroll
        for (int s = 0; s < 8; ++s) mfma_c(S.X[4 * s + hi][16 * t + lo], widen(ap[s]), re, im);
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int cc = 16 * t + hi + 4 * v;
          if (r < rt && cc < jb) stc(A2 + r + (int64_t)cc * d.lda, narrow(re[v], im[v]));
        }
      }
    }
    __syncthreads();
    Tile t = {{0, 0, 0, 0}, {0, 0, 0, 0}};
    qrh_gram_rows(A2, jb, A2, jb, d.lda, rt, t.re, t.im);
    put((Blk)S.G, t);
    __syncthreads();
  };
  // a panel that split: workgroup 0 finishes it and its updates alone (the tails
  // are transformed in place)
  const bool alone = js < jb;
  if (alone && !first) return;
  while (js < jb) {
    put((Blk)S.X, x);
    __syncthreads();
    apply_x();
    identity(x);
    put((Blk)S.P, a);
    __syncthreads();
    total_gram(js);
    js = qrh_factor(S, g, a, x, js, jb);
  }
  // V1, rounded as stored, and X of the last pass
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const int i = tile_row(v), j = tile_col();
    S.V[i][j] = i > j ? narrow(a.re[v], a.im[v]) : make_float2(i == j && i < jb ? 1.f : 0.f, 0.f);
  }
  if (tile_col() >= jb) x.re = x.im = dbl4{0, 0, 0, 0};
  put((Blk)S.X, x);
  if (tid < QR_NB && tid >= jb) S.tau[tid] = make_double2(0.0, 0.0);
  __syncthreads();
  auto vat = [&](int i, int k) { return widen(S.V[i][k]); };
  auto vadj = [&](int i, int k) { return cconj(widen(S.V[k][i])); };
  // V^H V = V1^H V1 + X^H G X
  Tile vv = {{0, 0, 0, 0}, {0, 0, 0, 0}};
  mm32([&](int i, int k) { return S.G[i][k]; }, [&](int k, int j) { return S.X[k][j]; }, vv.re,
       vv.im);
  put((Blk)S.P, vv);
  __syncthreads();
  vv.re = vv.im = dbl4{0, 0, 0, 0};
  mm32([&](int i, int k) { return cconj(S.X[k][i]); }, [&](int k, int j) { return S.P[k][j]; },
       vv.re, vv.im);
  mm32(vadj, vat, vv.re, vv.im);
  __syncthreads();
  put((Blk)S.G, vv);
  __syncthreads();
  qrh_t_factor(S);
  if (first) {
    const int blk = (j0 % QR_OB) / QR_NB;
    float2* Tw = d.Tw + (int64_t)blk * QR_NB * QR_NB;
    float2* Ap = d.A + j0 + (int64_t)j0 * d.lda;
    float2* Rp = d.R + j0 + (int64_t)j0 * d.ldr;
    // through P, so that consecutive threads store consecutive rows
    put((Blk)S.P, a);
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int i = c, cc = ig + 8 * k;
      const double2 t = S.G[i][cc], r = S.P[i][cc];
      stc(Tw + i + QR_NB * cc, i < jb && cc < jb ? narrow(t.x, t.y) : make_float2(0.f, 0.f));
      if (i < jb && cc < jb) {
        stc(Ap + i + (int64_t)cc * d.lda, S.V[i][cc]);
        stc(Rp + i + (int64_t)cc * d.ldr, i <= cc ? narrow(r.x, r.y) : make_float2(0.f, 0.f));
      }
      stc(sc.xy + i + QR_NB * cc, S.X[i][cc]);
    }
  }
  for (int q = blockIdx.x; q < nq; q += alone ? 1 : nw) {
    const int n = min(QR_NB, nt - QR_NB * q);
    __syncthreads();
    // W = T^H (V1^H A1 + X^H G); A1 -= V1 W; Y = X W
    if (!alone) {
      load_gram((Blk)S.Q, jb + QR_NB * q, n);
    } else {
      Tile t = {{0, 0, 0, 0}, {0, 0, 0, 0}};
      qrh_gram_rows(A2, jb, Ar + jb + (int64_t)QR_NB * q * d.lda, n, d.lda, rt, t.re, t.im);
      put((Blk)S.Q, t);
    }
#pragma unroll
    for (int k = 0; k < 4; ++k)
      S.P[c][ig + 8 * k] = widen(ldc(sc.a1 + tid + 256 * k + QR_NB * QR_NB * (q + 1)));
    __syncthreads();
    dbl4 re = {0, 0, 0, 0}, im = {0, 0, 0, 0};
    mm32(vadj, [&](int k, int j) { return S.P[k][j]; }, re, im);
    mm32([&](int i, int k) { return cconj(S.X[k][i]); }, [&](int k, int j) { return S.Q[k][j]; },
         re, im);
    __syncthreads();
    mm32_out(re, im, [&](int i, int j, double2 v) { S.Q[i][j] = v; });
    __syncthreads();
    re = im = dbl4{0, 0, 0, 0};
    mm32([&](int i, int k) { return cconj(S.G[k][i]); }, [&](int k, int j) { return S.Q[k][j]; },
         re, im);
    __syncthreads();
    mm32_out(re, im, [&](int i, int j, double2 v) { S.Q[i][j] = v; });
    __syncthreads();
    re = im = dbl4{0, 0, 0, 0};
    mm32(vat, [&](int k, int j) { return S.Q[k][j]; }, re, im);
    mm32_out(re, im, [&](int i, int j, double2 v) {
      const double2 o = S.P[i][j];
      if (i < jb && j < n)
        stc(Ar + i + (int64_t)(QR_NB * q + j) * d.lda, narrow(o.x - v.x, o.y - v.y));
    });
    re = im = dbl4{0, 0, 0, 0};
    mm32([&](int i, int k) { return S.X[i][k]; }, [&](int k, int j) { return S.Q[k][j]; }, re, im);
    mm32_out(re, im, [&](int i, int j, double2 v) {
      stc(sc.xy + i + QR_NB * (QR_NB * (q + 1) + j), v);
    });
  }
}

}  // namespace
}  // namespace nd

namespace nd {

// Panels of the half block at H0 of every problem in `act` (kmin > H0), with
// their updates of the half's remaining columns.
static void qr_half_panels(DescPool& pool, const QRDesc<float>* dd,
                           const std::vector<QRDesc<float>>& d, const std::vector<int>& act,
                           int H0, bool graded) {
  // about 2048 row chunks over the batch (two workgroups a CU, four rounds);
  // fewer, longer chunks leave CUs idle, more add partial Grams to sum
  int tallest = 0;
  for (int i : act) tallest = std::max(tallest, d[i].m - H0);
  const int nact = std::max<int>(1, (int)act.size());
  QrhPart pp{nullptr, 0, std::max(1, std::min(QRH_MAXC, 2048 / nact))};
  const size_t room = kGemmPartBytes / (sizeof(double2) * d.size());
  if (tallest > QRH_TALL * QRH_ROWS && room / (QR_NB * QR_HB) >= QRH_MAXC &&
      2048 / nact > QRH_MAXC) {
    pp.tall = (double2*)pool.stream_scratch(kGemmPartBytes);
    if (pp.tall) {
      pp.stride = room;
      pp.maxc = std::min(QRH_MAXC_TALL, 2048 / nact);
    }
  }
  auto rows_pass = [&](const std::vector<int>& a, int j1, bool prev) {
    int rows = 0;
    for (int i : a) rows = std::max(rows, d[i].m - (prev ? j1 - QR_NB : H0));
    const int gx = std::max(1, std::min(pp.maxc, (rows + QRH_ROWS - 1) / QRH_ROWS));
    with_descs(pool, a.data(), a.size(), [&](auto as) {
      using AS = decltype(as);
      // covers every problem's chunks: at most maxc, and no more than steps
      dim3 grid((unsigned)gx, (unsigned)a.size());
      if (prev)
        hipLaunchKernelGGL((qr_half_rows_kernel<true, AS>), grid, dim3(256), 0, pool.stream, dd,
                           as, H0, j1, pp);
      else
        hipLaunchKernelGGL((qr_half_rows_kernel<false, AS>), grid, dim3(256), 0, pool.stream, dd,
                           as, H0, j1, pp);
    });
  };
  rows_pass(act, H0, false);
  std::vector<int> cur;
  for (int j0 = H0; j0 < H0 + QR_HB; j0 += QR_NB) {
    cur.clear();
    int nq = 0, mr = 0;
    for (int i : act) {
      const int kmin = qr_kmin(d[i].m, d[i].n);
      if (kmin <= j0) continue;
      cur.push_back(i);
      const int nt = std::min(d[i].n, H0 + QR_HB) - j0 - std::min(QR_NB, kmin - j0);
      nq = std::max(nq, (nt + QR_NB - 1) / QR_NB);
      mr = std::max(mr, d[i].m - j0);
    }
    if (cur.empty()) break;
    ProfScope ps(pool.stream, KC_QRPANEL, 0.0, (int)cur.size(), mr, 0, 0, 0);
    // one workgroup per remaining block of 32 columns while that leaves CUs
    // idle (each repeats the panel's factorization), else one per problem
    const unsigned nw = (int)cur.size() * nq <= device_cus() ? std::max(nq, 1) : 1;
    // graded lists: two further passes for the panels that split, each a row
    // pass and a factorization (some 30 us where no panel needs them, 2% of a
    // factorization with leaves of 16 384 rows if theirs had one); the tallest
    // panels of other lists one (a split finished by one workgroup takes 0.2 ms
    // for 600 rows, 0.5 for 4000; 60 000 x 256 of rank 20 spent 16 of 24 ms so)
    const int passes = graded ? 3 : mr > 8 * QRH_TALL * QRH_ROWS ? 2 : 1;
    const int gx = std::max(1, std::min(pp.maxc, (mr + QRH_ROWS - 1) / QRH_ROWS));
    with_descs(pool, cur.data(), cur.size(), [&](auto as) {
      using AS = decltype(as);
      for (int p = 0; p < passes; ++p) {
        const bool more = p + 1 < passes;
        hipLaunchKernelGGL((qr_half_factor_kernel<AS>), dim3(nw + 1, (unsigned)cur.size()),
                           dim3(256), 0, pool.stream, dd, as, H0, j0, pp, p, more);
        if (more)
          hipLaunchKernelGGL((qr_half_split_kernel<AS>), dim3((unsigned)gx, (unsigned)cur.size()),
                             dim3(256), 0, pool.stream, dd, as, H0, j0, pp, p);
      }
    });
    rows_pass(cur, j0 + QR_NB, true);
  }
  ND_HIP(hipGetLastError());
}

}  // namespace nd
