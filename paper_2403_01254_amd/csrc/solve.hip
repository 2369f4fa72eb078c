// Normal-equation assembly, FP64 Cholesky solve and SE(3) pose update of one
// Gauss-Newton / IRLS step (Sec. V-A): with the weights frozen, the step
// solves (H_red + mu I) delta = -b_red over every frame except the fixed one
// and moves T_m <- T_m exp(delta_m^) (right perturbation, eps = [rho; phi]).
//
// Assembly is one thread per entry of the system, summing that entry's
// contributing edge blocks in edge order (host-built lists, deterministic).
// The solve is one workgroup per problem: systems up to 128 unknowns are
// eliminated in LDS, one frame's columns at a time, and so are the blocks of
// larger ones where few frames share an edge (solve_plan.h); the others run a
// blocked right-looking Cholesky with 32-wide panels, the panel kept in LDS for
// the trailing update.  Sets of small problems run the whole step, from the
// finalisation's partial sums to the moved poses, in one kernel (k_step).
#include "edge_sums.h"
#include "solve_plan.h"

namespace rkhsba {
namespace {

__device__ inline int sym_index(int r, int c) {
  if (r > c) { const int t = r; r = c; c = t; }
  return r * 6 - (r * (r - 1)) / 2 + (c - r);
}

// reduced index <-> frame when frame `fixed` is removed (fixed < 0: none)
__device__ inline int frame_of_reduced(int k, int fixed) { return (fixed >= 0 && k >= fixed) ? k + 1 : k; }

// Entry (row, col) of problem S's H, and entry `row` of its b: the contributing edges' values in edge order.
__device__ inline double h_entry(const SolveArgs& a, const ProbSys& S, int row, int col) {
  const int fa = frame_of_reduced(row / 6, S.fixed), fc = frame_of_reduced(col / 6, S.fixed);
  const int r = row % 6, s = col % 6;
  const int32_t* start = a.blk_start + S.blk0 + fa * S.K + fc;
  double v = 0.0;
  for (int k = start[0]; k < start[1]; ++k) {
    const int code = a.blk_list[k];
    const double* eo = a.edge_out + (int64_t)(code >> 2) * kEdgeVals;
    switch (code & 3) {
      case 0: v += eo[13 + sym_index(r, s)]; break;
      case 1: v += eo[34 + sym_index(r, s)]; break;
      case 2: v += eo[55 + 6 * r + s]; break;
      default: v += eo[55 + 6 * s + r]; break;
    }
  }
  return v;
}
__device__ inline double b_entry(const SolveArgs& a, const ProbSys& S, int row) {
  const int fa = frame_of_reduced(row / 6, S.fixed), r = row % 6;
  const int32_t* start = a.vec_start + S.vec0 + fa;
  double v = 0.0;
  for (int k = start[0]; k < start[1]; ++k) {
    const int code = a.vec_list[k];
    v += a.edge_out[(int64_t)(code >> 1) * kEdgeVals + ((code & 1) ? 7 : 1) + r];
  }
  return v;
}

// One thread per entry of a problem's system (grid.y = problem).
__global__ __launch_bounds__(256) void k_assemble(SolveArgs a) {
  const ProbSys S = a.sys[blockIdx.y];
  const int n = S.n;
  const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (idx < (int64_t)n * n) a.H[S.h_off + idx] = h_entry(a, S, (int)(idx / n), (int)(idx % n));
  else if (idx < (int64_t)n * n + n) a.b[S.v_off + idx - (int64_t)n * n] = b_entry(a, S, (int)(idx - (int64_t)n * n));
}

// F (times sigma^2) and the pair count of the current evaluation of a problem (one wavefront, fixed summation
// order).
__device__ inline void record_loss(const SolveArgs& a, const ProbSys& S) {
  const int lane = threadIdx.x & 63;
  double F = 0.0, np = 0.0;
  for (int e = S.e0 + lane; e < S.e0 + S.E; e += 64) {
    F += a.edge_out[(int64_t)e * kEdgeVals];
    np += a.edge_out[(int64_t)e * kEdgeVals + 91];
  }
  F = wave_sum(F);
  np = wave_sum(np);
  const int iter = a.state[S.state_off];
  if (lane == 0 && iter >= 0 && iter <= S.n_iter) {
    a.loss_hist[S.hist_off + iter] = S.sigma2 * F;
    a.pairs_hist[S.hist_off + iter] = np;
  }
}

__global__ __launch_bounds__(64) void k_loss_only(SolveArgs a) { record_loss(a, a.sys[blockIdx.x]); }

// T <- T exp(xi^): closed-form SE(3) exponential (Rodrigues for the rotation,
// V = I + B K + C K^2 for the translation), series for small angles.
__device__ __noinline__ void right_update(double* T, double r0, double r1, double r2, double p0, double p1, double p2) {
  const double rho[3] = {r0, r1, r2}, phi[3] = {p0, p1, p2};
  const double th2 = phi[0] * phi[0] + phi[1] * phi[1] + phi[2] * phi[2];
  const double th = sqrt(th2);
  double A, B, C;
  if (th < 1e-4) {
    A = 1.0 - th2 / 6.0 + th2 * th2 / 120.0;
    B = 0.5 - th2 / 24.0 + th2 * th2 / 720.0;
    C = 1.0 / 6.0 - th2 / 120.0 + th2 * th2 / 5040.0;
  } else {
    double s, c;
    sincos(th, &s, &c);
    A = s / th;
    B = (1.0 - c) / th2;
    C = (th - s) / (th2 * th);
  }
  const double K[3][3] = {{0.0, -phi[2], phi[1]}, {phi[2], 0.0, -phi[0]}, {-phi[1], phi[0], 0.0}};
  double K2[3][3];
  for (int r = 0; r < 3; ++r)
    for (int c = 0; c < 3; ++c) K2[r][c] = K[r][0] * K[0][c] + K[r][1] * K[1][c] + K[r][2] * K[2][c];
  double Re[3][3], V[3][3];
  for (int r = 0; r < 3; ++r)
    for (int c = 0; c < 3; ++c) {
      const double I = r == c ? 1.0 : 0.0;
      Re[r][c] = I + A * K[r][c] + B * K2[r][c];
      V[r][c] = I + B * K[r][c] + C * K2[r][c];
    }
  double te[3];
  for (int r = 0; r < 3; ++r) te[r] = V[r][0] * rho[0] + V[r][1] * rho[1] + V[r][2] * rho[2];
  double R[3][3], t[3];
  for (int r = 0; r < 3; ++r) {
    for (int c = 0; c < 3; ++c) R[r][c] = T[3 * r + c];
    t[r] = T[9 + r];
  }
  for (int r = 0; r < 3; ++r) {
    for (int c = 0; c < 3; ++c) T[3 * r + c] = R[r][0] * Re[0][c] + R[r][1] * Re[1][c] + R[r][2] * Re[2][c];
    T[9 + r] = R[r][0] * te[0] + R[r][1] * te[1] + R[r][2] * te[2] + t[r];
  }
}

__device__ __forceinline__ double block_sum(double v, double* sh) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  v = wave_sum(v);
  __syncthreads();
  if (lane == 0) sh[w] = v;
  __syncthreads();
  double t = 0.0;
  for (int k = 0; k < (int)(blockDim.x >> 6); ++k) t += sh[k];
  __syncthreads();
  return t;
}

// A double read from one lane of the wavefront (lane index uniform).
__device__ inline double lane_value(double v, int lane) {
  const int lo = __builtin_amdgcn_readlane(__double2loint(v), lane);
  const int hi = __builtin_amdgcn_readlane(__double2hiint(v), lane);
  return __hiloint2double(hi, lo);
}

// ---- systems that fit in LDS (n <= kLdsSystem unknowns, 6 per frame)
//
// (H + mu I) delta = -b as L D L^T delta = -b (L unit lower triangular, no square roots), eliminated right-looking
// in blocks of one frame's 6 columns, with -b as one more row: after the elimination row n holds y = D^-1 L^-1 (-b),
// and L^T delta = y is solved in one wavefront with two rows per lane.  A block step has two barriers; the threads
// of the rows below each factor the 6 x 6 diagonal block for themselves (it is short, and a barrier less).  One
// column per barrier and a separate forward solve took 0.7 us per unknown (n = 42: 32 us a solve; now the whole step
// around it takes 17).
//
// The rounding is that of the elimination column by column: mu joins the diagonal before any update, an update takes
// the later row divided by the pivot and the earlier one undivided, one fused multiply-add per column in their order,
// and the reciprocals are correctly rounded.  A view that leaves a direction nearly free (a reduced H with eigenvalues
// below mu) makes 1e-8 of pose out of another order's last bits, and other pair counts out of that.
constexpr int kSolveThreads = 1024;
constexpr int kLdsDoubles = kLdsSystem * (kLdsSystem + 1);  // shared buffer of both paths

struct SmallShared {
  double A[(kLdsSystem + 1) * (kLdsSystem + 1)];  // rows 0 .. n (n: -b), row stride n + 1; lower triangle used
  double t[6][kLdsSystem + 1];                    // the panel's rows before the division by the pivots
  int bad;                                        // a pivot was not positive
};

// 1 / d, correctly rounded: the hardware estimate, two Newton steps, and a last one from the exact residual, a
// division's own chain without the scaling of its operands' exponents.  The ends of the range, where a step could
// leave it, divide.
__device__ inline double reciprocal(double d) {
  if (!(d > 1e-290 && d < 1e290)) return 1.0 / d;
  double r = __builtin_amdgcn_rcp(d);
  r = fma(fma(-d, r, 1.0), r, r);
  r = fma(fma(-d, r, 1.0), r, r);
  return fma(fma(-d, r, 1.0), r, r);
}

// L D L^T of a diagonal block in d (lower triangle; d[r][c] * rd[c] is L below the diagonal, rd the reciprocal
// pivots), column by column, and a row x of the columns' rest in step with it.
__device__ __forceinline__ void eliminate_block(double (&d)[6][6], double (&x)[6], double (&rd)[6], bool& ok) {
#pragma unroll
  for (int j = 0; j < 6; ++j) {
    ok = ok && d[j][j] > 0.0;
    rd[j] = reciprocal(d[j][j]);
#pragma unroll
    for (int r = j + 1; r < 6; ++r) {
      const double l = d[r][j] * rd[j];
#pragma unroll
      for (int c = j + 1; c <= r; ++c) d[r][c] = fma(-l, d[c][j], d[r][c]);
    }
    const double l = x[j] * rd[j];
#pragma unroll
    for (int c = j + 1; c < 6; ++c) x[c] = fma(-l, d[c][j], x[c]);
  }
}

// S.A holds the lower triangle of H and -b; all threads of the block.  Solution in row n; false (in every thread) when
// a pivot is not positive.
__device__ __forceinline__ bool solve_small(int n, double mu, SmallShared& S) {
  const int t = threadIdx.x, tx = t & 31, ty = t >> 5, ld = n + 1;
  double* A = S.A;
  if (t == 0) S.bad = 0;
  __syncthreads();
  for (int p = 0; p < n; p += 6) {
    const int m0 = p + 6;
    // rows below the block, and its own first row's thread (for the pivot test of the last block)
    if (t <= n - m0) {
      const int i = m0 + t;
      double d[6][6], x[6], rd[6];
      bool ok = true;
#pragma unroll
      for (int r = 0; r < 6; ++r)
#pragma unroll
        for (int c = 0; c <= r; ++c) d[r][c] = A[(p + r) * ld + p + c] + (r == c && p == 0 ? mu : 0.0);
#pragma unroll
      for (int c = 0; c < 6; ++c) x[c] = A[i * ld + p + c];
      eliminate_block(d, x, rd, ok);
      if (!ok) S.bad = 1;
#pragma unroll
      for (int c = 0; c < 6; ++c) {
        S.t[c][i] = x[c];
        A[i * ld + p + c] = x[c] * rd[c];
      }
      if (t == n - m0) {  // (row n's thread) the block's own L, for the backward solve
#pragma unroll
        for (int r = 1; r < 6; ++r)
#pragma unroll
          for (int c = 0; c < r; ++c) S.t[c][p + r] = d[r][c] * rd[c];
      }
    }
    __syncthreads();
    if (S.bad) return false;  // every thread reads the same flag
    // trailing rows and columns, row n included; the block's L moves to its place
    for (int i = m0 + ty; i <= n; i += 32)
      for (int k = m0 + tx; k <= min(i, n - 1); k += 32) {
        double v = A[i * ld + k] + (i == k && p == 0 ? mu : 0.0);
#pragma unroll
        for (int c = 0; c < 6; ++c) v = fma(-A[i * ld + p + c], S.t[c][k], v);
        A[i * ld + k] = v;
      }
    if (t < 36) {
      const int r = t / 6, c = t % 6;
      if (c < r) A[(p + r) * ld + p + c] = S.t[c][p + r];
    }
    __syncthreads();
  }
  if (t < 64) {  // L^T x = y, columns from the last
    double u0 = t < n ? A[n * ld + t] : 0.0, u1 = t + 64 < n ? A[n * ld + t + 64] : 0.0;
#pragma unroll 6
    for (int j = n - 1; j > 0; --j) {
      const double l0 = t < j ? A[j * ld + t] : 0.0, l1 = t + 64 < j ? A[j * ld + t + 64] : 0.0;
      const double xj = lane_value(j < 64 ? u0 : u1, j & 63);
      u0 = fma(-l0, xj, u0);
      u1 = fma(-l1, xj, u1);
    }
    if (t < n) A[n * ld + t] = u0;
    if (t + 64 < n) A[n * ld + t + 64] = u1;
  }
  __syncthreads();
  return true;
}

// Right-looking elimination of an n x n symmetric block held in LDS (row
// stride ld, lower triangle used), without square roots: step j subtracts
// a_ij a_kj / d_j from every trailing entry (j < k <= i), d_j the pivot of
// step j.  Afterwards the block holds M (unit-free lower factor: A = M D^-1 M^T
// with D = diag(d)), and rd[j] = 1 / d_j.  One barrier per step; threads form a
// 32 x 32 grid over the trailing rows and columns.  Returns false (in every
// thread) when a pivot is not positive.
__device__ __forceinline__ bool eliminate_lds(double* A, int n, int ld, double* rd) {
  const int t = threadIdx.x, tx = t & 31, ty = t >> 5;
  for (int j = 0; j < n; ++j) {
    const double d = A[j * ld + j];
    if (!(d > 0.0)) return false;  // every thread read the same pivot
    const double inv = 1.0 / d;
    if (t == 0) rd[j] = inv;
    for (int i = j + 1 + ty; i < n; i += 32) {
      const double aij = A[i * ld + j] * inv;
      for (int k = j + 1 + tx; k <= i; k += 32) A[i * ld + k] -= aij * A[k * ld + j];
    }
    __syncthreads();
  }
  return true;
}

// ---- larger systems: blocked right-looking Cholesky in global memory
//
// Panels of NB columns: the diagonal block is eliminated in LDS and scaled to
// L11; the rows below solve L21 = A21 L11^-T and are kept in LDS for the
// trailing update A22 -= L21 L21^T.  While the panel has at most kPanelCols
// rows (every system up to ~500 unknowns), each row is solved in registers
// (one row per thread, the 32 steps unrolled) and the panel is stored column
// by column, so that the trailing update's 4 x 4 register tiles, whose rows
// and columns are 32 apart, read it without bank conflicts and write A22 with
// consecutive threads on consecutive columns.  Larger panels are solved and
// read in place in global memory, with contiguous tiles.  Then L y = -b and
// L^T delta = y, panel by panel.
constexpr int NB = 32;
constexpr int kPanelCols = (kLdsDoubles - NB * (NB + 1) - 2 * NB) / NB;  // rows of a column-major panel

// Zero rows of L21: many systems are block-sparse (each frame has a few neighbours in the pose graph), and
// the factor keeps the profile of the matrix.  For systems whose panels all fit in LDS, flags[p * W + w] (W =
// ceil(n / 32) words per panel) records, bit b, whether row 32 w + b of the factor has a nonzero entry in panel
// p's columns; the row solve, the trailing update and both triangular solves skip what a zero row would
// contribute (exact zeros: the factor and the solution are the same bit for bit).  flags == nullptr: every row
// counts as nonzero.
constexpr int kFlagRows = NB + kPanelCols;  // the largest system every panel of which is solved in LDS
constexpr int kFlagWords = ((kFlagRows + 31) / 32) * ((kFlagRows + 31) / 32);

__device__ __forceinline__ void solve_blocked(const ProbSys& S, const SolveArgs& a, double mu, double* buf, int32_t* status,
                              uint32_t* flags) {
  const int n = S.n, t = threadIdx.x, tx = t & 31, ty = t >> 5;
  const int W = (n + 31) / 32;
  if (n > kFlagRows) flags = nullptr;
  static_assert(NB == 32, "one flag word per panel row chunk");
  __shared__ int32_t live_chunks[(kFlagRows + 31) / 32];
  __shared__ int32_t n_live;
  __shared__ uint32_t chunk_mask;  // bit c: rows m0 + 32 c .. m0 + 32 c + 31 hold a nonzero row of L21
  double* H = a.H + S.h_off;
  double* Dg = buf;                       // NB x (NB + 1) diagonal block
  double* rd = buf + NB * (NB + 1);       // NB reciprocal pivots / diagonal
  double* yb = rd + NB;                   // NB solution entries of a panel
  double* P = yb + NB;                    // the panel L21, column-major (P[j * m + r])
  for (int i = t; i < n; i += kSolveThreads) H[(int64_t)i * n + i] += mu;
  __syncthreads();
  for (int kb = 0; kb < n; kb += NB) {
    const int nb = min(NB, n - kb), m0 = kb + nb, m = n - m0;
    for (int idx = t; idx < nb * nb; idx += kSolveThreads) {
      const int i = idx / nb, k = idx - i * nb;
      if (k <= i) Dg[i * (NB + 1) + k] = H[(int64_t)(kb + i) * n + kb + k];
    }
    __syncthreads();
    if (!eliminate_lds(Dg, nb, NB + 1, rd)) {
      if (t == 0) *status = -4;
      return;
    }
    // scale to L11: L_jj = sqrt(d_j), L_ij = M_ij / sqrt(d_j); rd <- 1 / L_jj
    for (int idx = t; idx < nb * nb; idx += kSolveThreads) {
      const int i = idx / nb, k = idx - i * nb;
      if (k <= i) {
        const double sk = sqrt(rd[k]);  // 1 / sqrt(d_k)
        const double v = (i == k) ? 1.0 / sk : Dg[i * (NB + 1) + k] * sk;
        Dg[i * (NB + 1) + k] = v;
        H[(int64_t)(kb + i) * n + kb + k] = v;
      }
    }
    __syncthreads();
    if (t < nb) rd[t] = 1.0 / Dg[t * (NB + 1) + t];
    __syncthreads();
    if (m <= kPanelCols) {
      // panel rows in registers, stored column-major: P[j * m + r] = L21[r][j]; a zero row of A21 stays zero
      const int pw = kb / 32;  // this panel's flag words start at pw * W
      for (int r0 = 0; r0 < m; r0 += kSolveThreads) {  // uniform trip count (the ballot below)
        const int r = r0 + t;
        bool nz = false;
        if (r < m) {
          double* row = H + (int64_t)(m0 + r) * n + kb;
          double x[NB];
#pragma unroll
          for (int j = 0; j < NB; ++j) x[j] = j < nb ? row[j] : 0.0;
#pragma unroll
          for (int j = 0; j < NB; ++j) nz = nz || x[j] != 0.0;
          if (nz) {
#pragma unroll
            for (int j = 0; j < NB; ++j) {
              if (j < nb) {
                const double* Lj = Dg + j * (NB + 1);
                double s0 = x[j], s1 = 0.0;
#pragma unroll
                for (int k = 0; k + 1 < j; k += 2) {
                  s0 -= Lj[k] * x[k];
                  s1 -= Lj[k + 1] * x[k + 1];
                }
                if (j & 1) s0 -= Lj[j - 1] * x[j - 1];
                x[j] = (s0 + s1) * rd[j];
              }
            }
          }
#pragma unroll
          for (int j = 0; j < NB; ++j)
            if (j < nb) {
              if (nz) row[j] = x[j];
              P[j * m + r] = x[j];
            }
        }
        if (flags) {  // rows m0 + r0 + 64 w' + lane: two whole words per wavefront (m0 and r0 are multiples of 32)
          const uint64_t bits = __ballot(nz);
          const int wd = (m0 + r0 + (t & ~63)) / 32;
          if ((t & 63) == 0 && wd < W) flags[pw * W + wd] = (uint32_t)bits;
          if ((t & 63) == 32 && wd + 1 < W) flags[pw * W + wd + 1] = (uint32_t)(bits >> 32);
        }
      }
      __syncthreads();
      // the 32-row chunks of A22 with a nonzero row of L21 in this panel
      if (t == 0) {  // (m == 0, the last panel, has no chunk; otherwise m0 is a multiple of 32)
        int c = 0;
        uint32_t mask = 0;
        for (int w = m0 / 32; m > 0 && w < W; ++w)
          if (!flags || flags[pw * W + w]) {
            live_chunks[c++] = w * 32 - m0;
            mask |= 1u << (w - m0 / 32);
          }
        n_live = c;
        chunk_mask = mask;
      }
      __syncthreads();
      const int nl = n_live, nc = (m + 31) / 32;
      if (2 * nl <= nc) {
        // few live chunks: one 32 x 32 tile per pair of them, one entry per thread, the NB products summed in
        // the same order as below
        for (int u = 0; u < nl; ++u)
          for (int v = 0; v <= u; ++v) {
            const int i = live_chunks[u] + ty, k = live_chunks[v] + tx;
            if (i < m && k <= i) {
              double acc = 0.0;
              for (int j = 0; j < nb; ++j) acc = fma(P[j * m + i], P[j * m + k], acc);
              H[(int64_t)(m0 + i) * n + m0 + k] -= acc;
            }
          }
        __syncthreads();
        continue;
      }
      // A22 -= L21 L21^T over 128 x 128 blocks on or below the diagonal (those with a nonzero row of L21 on
      // both sides); thread (tx, ty) takes rows a0 + ty + 32p and columns b0 + tx + 32q
      const uint32_t cm = chunk_mask;
      for (int a0 = 0; a0 < m; a0 += 128)
        for (int b0 = 0; b0 <= a0; b0 += 128) {
          if (!((cm >> (a0 / 32)) & 0xFu) || !((cm >> (b0 / 32)) & 0xFu)) continue;
          double acc[4][4];
#pragma unroll
          for (int p = 0; p < 4; ++p)
#pragma unroll
            for (int q = 0; q < 4; ++q) acc[p][q] = 0.0;
          for (int j = 0; j < nb; ++j) {
            const double* Pj = P + j * m;
            double li[4], lk[4];
#pragma unroll
            for (int p = 0; p < 4; ++p) {
              const int i = a0 + ty + 32 * p, k = b0 + tx + 32 * p;
              li[p] = i < m ? Pj[i] : 0.0;
              lk[p] = k < m ? Pj[k] : 0.0;
            }
#pragma unroll
            for (int p = 0; p < 4; ++p)
#pragma unroll
              for (int q = 0; q < 4; ++q) acc[p][q] = fma(li[p], lk[q], acc[p][q]);
          }
#pragma unroll
          for (int p = 0; p < 4; ++p)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              const int i = a0 + ty + 32 * p, k = b0 + tx + 32 * q;
              if (i < m && k <= i) H[(int64_t)(m0 + i) * n + m0 + k] -= acc[p][q];
            }
        }
      __syncthreads();
      continue;
    }
    // larger panels: rows solved and read in place in global memory
    for (int r = t; r < m; r += kSolveThreads) {
      double* x = H + (int64_t)(m0 + r) * n + kb;
      for (int j = 0; j < nb; ++j) {
        const double* Lj = Dg + j * (NB + 1);
        double s0 = x[j], s1 = 0.0;
        int k = 0;
        for (; k + 1 < j; k += 2) {
          s0 -= Lj[k] * x[k];
          s1 -= Lj[k + 1] * x[k + 1];
        }
        if (k < j) s0 -= Lj[k] * x[k];
        x[j] = (s0 + s1) * rd[j];
      }
    }
    __syncthreads();
    // trailing update of the lower triangle of A22
    const int tiles = (m + 3) / 4;
    for (int ti = ty; ti < tiles; ti += 32) {
      for (int tk = tx; tk <= ti; tk += 32) {
        double acc[4][4];
#pragma unroll
        for (int p = 0; p < 4; ++p)
#pragma unroll
          for (int q = 0; q < 4; ++q) acc[p][q] = 0.0;
        for (int j = 0; j < nb; ++j) {
          double li[4], lk[4];
#pragma unroll
          for (int p = 0; p < 4; ++p) {
            const int ri = 4 * ti + p, rk = 4 * tk + p;
            li[p] = ri < m ? H[(int64_t)(m0 + ri) * n + kb + j] : 0.0;
            lk[p] = rk < m ? H[(int64_t)(m0 + rk) * n + kb + j] : 0.0;
          }
#pragma unroll
          for (int p = 0; p < 4; ++p)
#pragma unroll
            for (int q = 0; q < 4; ++q) acc[p][q] = fma(li[p], lk[q], acc[p][q]);
        }
#pragma unroll
        for (int p = 0; p < 4; ++p)
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const int i = 4 * ti + p, k = 4 * tk + q;
            if (i < m && k <= i) H[(int64_t)(m0 + i) * n + m0 + k] -= acc[p][q];
          }
      }
    }
    __syncthreads();
  }

  double* y = a.delta + S.v_off;
  const double* b = a.b + S.v_off;
  for (int i = t; i < n; i += kSolveThreads) y[i] = -b[i];
  __syncthreads();
  // L y = -b: each diagonal block staged in LDS (with the reciprocals of its diagonal) and solved in
  // wavefront 0, then the rows below updated by all threads
  auto stage_diag = [&](int kb, int nb) __attribute__((always_inline)) {
    for (int idx = t; idx < nb * nb; idx += kSolveThreads) {
      const int i = idx / nb, k = idx - i * nb;
      if (k <= i) Dg[i * (NB + 1) + k] = H[(int64_t)(kb + i) * n + kb + k];
    }
    if (t < nb) rd[t] = 1.0 / H[(int64_t)(kb + t) * n + kb + t];
    __syncthreads();
  };
  for (int kb = 0; kb < n; kb += NB) {
    const int nb = min(NB, n - kb);
    stage_diag(kb, nb);
    if (t < 64) {
      double v = t < nb ? y[kb + t] : 0.0;
      for (int j = 0; j < nb; ++j) {
        const double yj = lane_value(v, j) * rd[j];
        if (t == j) v = yj;
        else if (t > j && t < nb) v -= Dg[t * (NB + 1) + j] * yj;
      }
      if (t < nb) {
        y[kb + t] = v;
        yb[t] = v;
      }
    }
    __syncthreads();
    for (int i = kb + nb + t; i < n; i += kSolveThreads) {
      if (flags && !((flags[(kb / 32) * W + i / 32] >> (i & 31)) & 1u)) continue;  // zero row of this panel
      const double* row = H + (int64_t)i * n + kb;
      double v = y[i];
      for (int j = 0; j < nb; ++j) v -= row[j] * yb[j];
      y[i] = v;
    }
    __syncthreads();
  }
  // L^T delta = y
  for (int kb = ((n - 1) / NB) * NB; kb >= 0; kb -= NB) {
    const int nb = min(NB, n - kb);
    stage_diag(kb, nb);
    if (t < 64) {
      double v = t < nb ? y[kb + t] : 0.0;
      for (int j = nb - 1; j >= 0; --j) {
        const double xj = lane_value(v, j) * rd[j];
        if (t == j) v = xj;
        else if (t < j) v -= Dg[j * (NB + 1) + t] * xj;
      }
      if (t < nb) {
        y[kb + t] = v;
        yb[t] = v;
      }
    }
    __syncthreads();
    for (int i = t; i < kb; i += kSolveThreads) {
      if (flags && !flags[(i / 32) * W + kb / 32]) continue;  // rows kb .. kb + nb - 1 are zero in i's panel
      double v = y[i];
      for (int j = 0; j < nb; ++j) v -= H[(int64_t)(kb + j) * n + i] * yb[j];
      y[i] = v;
    }
    __syncthreads();
  }
}

// ---- larger sparse systems: block elimination in LDS by the host's plan (solve_plan.h)
//
// As solve_small, one frame's 6 columns a step and -b as one more row, but only the blocks that the plan holds, and
// the system assembled from the edges' values straight into them.  A chain of latencies: 63 steps of 2 us and their
// way back for 64 LiDAR frames with 6 edges each, 0.20 ms, where the blocked dense elimination took 0.52 (12 panels
// of 32 columns through global memory) and the assembly of H before it 0.01.
//
// Its order is the plan's, so its last bits are not the dense elimination's.  Where the system leaves a direction
// nearly free, they would become poses and pair counts: a pivot that elimination leaves below kWellPosed of its
// diagonal entry sends the system to the dense elimination.  LiDAR maps of 23 to 64 frames have smallest pivots of 3e-3
// and more of their diagonal (poses then agree to 1e-11), open chains of 24 to 48 clouds up to 25 m from their frames'
// origins 6e-5 to 3e-4 (1e-10, mostly 1e-12), depth frames in front of one wall and clouds along a line 6e-6 and less.
// Handed over, 24 to 64 such frames take the dense elimination's time (219 us an iteration of 24 small clouds before
// and so, 94 by blocks): the small pivot comes early.
constexpr double kWellPosed = 1e-5;

struct SparseShared {
  double d[kSparseLds / sizeof(double)];
};

// Solution in y (global, n, in frame order).  0: moved; 1: no pair touches a free frame; -1: a pivot is too small,
// for the dense elimination to look at (the same in every thread).
__device__ __forceinline__ int solve_sparse(const SolveArgs& a, const ProbSys& S, SparseShared& sh, double* __restrict__ red,
                            int* __restrict__ bad, double* __restrict__ y) {
  const int t = threadIdx.x;
  const uint16_t* __restrict__ plan = a.plans + S.plan0;
  const int words = sparse_words(plan[0], plan[1], plan[2]);
  const int doubles = (int)sparse_doubles(plan[0], plan[1], plan[3]);
  double* L = sh.d;
  uint16_t* local = reinterpret_cast<uint16_t*>(sh.d + doubles);
  for (int i = t; i < words; i += kSolveThreads) local[i] = plan[i];
  if (t == 0) *bad = 0;
  __syncthreads();
  const int nf = local[0], n_off = local[1], n = 6 * nf;
  // offsets of the plan's pieces in `local`
  const int o_order = kSparseHeader, o_col = o_order + nf, o_upd = o_col + nf + 1, o_row = o_upd + nf + 1;
  const int o_cols = o_row + n_off, o_list = o_cols + n_off;
  double* rhs = L + 36 * (nf + n_off);
  double* diag = rhs + n;                       // the diagonal before the elimination
  double* T = diag + n;  // a column's rows before the division by the pivots; last: the right side
  double* dl = T + 6 * (6 * (int)local[3] + 1);  // the diagonal block's L
  double tr = 0.0;
  for (int e = t; e < 36 * (nf + n_off); e += kSolveThreads) {
    const int blk = e / 36, q = e - 36 * blk, r = q / 6, c = q - 6 * r;
    const int row = blk < nf ? blk : local[o_row + blk - nf], col = blk < nf ? blk : local[o_cols + blk - nf];
    const double v = h_entry(a, S, 6 * local[o_order + row] + r, 6 * local[o_order + col] + c);
    L[e] = v;
    if (blk < nf && r == c) tr += v;
  }
  for (int i = t; i < n; i += kSolveThreads) rhs[i] = -b_entry(a, S, 6 * local[o_order + i / 6] + i % 6);
  tr = block_sum(tr, red);
  if (!(tr > 0.0)) return 1;
  const double mu = S.damping_rel * tr / n;
  for (int i = t; i < n; i += kSolveThreads) {
    diag[i] = L[36 * (i / 6) + 7 * (i % 6)];
    L[36 * (i / 6) + 7 * (i % 6)] += mu;
  }
  __syncthreads();
  for (int p = 0; p < nf; ++p) {
    const int c0 = local[o_col + p], rows = local[o_col + p + 1] - c0;
    if (t <= 6 * rows) {
      double d[6][6], x[6], rd[6];
      bool ok = true;
      const int at = t < 6 * rows ? 36 * (nf + c0) + 6 * t : (int)(rhs - L) + 6 * p;  // row t, or the right side
#pragma unroll
      for (int r = 0; r < 6; ++r)
#pragma unroll
        for (int c = 0; c <= r; ++c) d[r][c] = L[36 * p + 6 * r + c];
#pragma unroll
      for (int c = 0; c < 6; ++c) x[c] = L[at + c];
      eliminate_block(d, x, rd, ok);
#pragma unroll
      for (int c = 0; c < 6; ++c) {
        T[6 * t + c] = x[c];
        L[at + c] = x[c] * rd[c];
      }
      if (t == 6 * rows) {
#pragma unroll
        for (int j = 0; j < 6; ++j) ok = ok && d[j][j] > kWellPosed * diag[6 * p + j];
        if (!ok) *bad = 1;
#pragma unroll
        for (int r = 1; r < 6; ++r)
#pragma unroll
          for (int c = 0; c < r; ++c) dl[r * (r - 1) / 2 + c] = d[r][c] * rd[c];
      }
    }
    __syncthreads();
    if (*bad) return -1;
    const int u0 = local[o_upd + p], n_entries = 36 * (local[o_upd + p + 1] - u0);
    for (int e = t; e < n_entries + 6 * rows; e += kSolveThreads) {
      if (e < n_entries) {
        const int u = e / 36, q = e - 36 * u, r = q / 6, c = q - 6 * r;
        const int bi = local[o_list + 3 * (u0 + u)] - c0, bk = local[o_list + 3 * (u0 + u) + 1];
        const int target = 36 * local[o_list + 3 * (u0 + u) + 2] + q;
        double v = L[target];
#pragma unroll
        for (int k = 0; k < 6; ++k) v = fma(-T[6 * (6 * bi + r) + k], L[36 * (nf + bk) + 6 * c + k], v);
        L[target] = v;
      } else {
        const int i = e - n_entries, r = i % 6;
        const int target = 6 * local[o_row + c0 + i / 6] + r;
        double v = rhs[target];
#pragma unroll
        for (int k = 0; k < 6; ++k) v = fma(-T[6 * 6 * rows + k], L[36 * (nf + c0) + 6 * i + k], v);
        rhs[target] = v;
      }
    }
    if (t < 36 && t % 6 < t / 6) L[36 * p + t] = dl[(t / 6) * (t / 6 - 1) / 2 + t % 6];
    __syncthreads();
  }
  if (t < 64) {  // L^T x = y, one frame a step: lanes 8 g + c sum column c over the blocks g, g + 8, ..
    const int g = t >> 3, c = t & 7;
    for (int p = nf - 1; p >= 0; --p) {
      const int c0 = local[o_col + p], rows = local[o_col + p + 1] - c0;
      double v = 0.0;
      if (c < 6)
        for (int i = g; i < rows; i += 8) {
          const int xr = 6 * local[o_row + c0 + i];
#pragma unroll
          for (int r = 0; r < 6; ++r) v = fma(L[36 * (nf + c0 + i) + 6 * r + c], rhs[xr + r], v);
        }
      v += __shfl_xor(v, 8, 64);
      v += __shfl_xor(v, 16, 64);
      v += __shfl_xor(v, 32, 64);
      double u = c < 6 ? rhs[6 * p + c] - v : 0.0;
#pragma unroll
      for (int j = 5; j > 0; --j) {
        const double xj = lane_value(u, j);
        if (c < j) u = fma(-L[36 * p + 6 * j + c], xj, u);
      }
      if (t < 6) {
        rhs[6 * p + t] = u;
        y[6 * local[o_order + p] + t] = u;
      }
      wave_sync();
    }
  }
  __syncthreads();
  return 0;
}

union SolveShared {
  SparseShared sparse;
  SmallShared small;
  struct {
    double buf[kLdsDoubles];
    uint32_t zflags[kFlagWords];
  } blocked;
};

// One workgroup per problem: damped solve and pose update.  A problem whose
// iteration count has reached n_iter (its last evaluation gave the final
// loss) is left unchanged.  Every branch below is block-uniform.
__global__ __launch_bounds__(kSolveThreads) void k_solve_update(SolveArgs a) {
  __shared__ SolveShared sh;
  __shared__ double red[kSolveThreads / 64];
  __shared__ int bad;
  const ProbSys S = a.sys[blockIdx.x];
  int32_t* st = a.state + S.state_off;
  const int iter = st[0];
  const bool run = iter < S.n_iter && st[1] == 0 && S.n > 0;
  __syncthreads();
  if (run) {
    const int n = S.n, t = threadIdx.x;
    bool moved = false, dense = S.plan0 < 0;
    if (!dense) {
      const int e = solve_sparse(a, S, sh.sparse, red, &bad, a.delta + S.v_off);
      moved = e == 0;
      dense = e < 0;
      if (dense) {  // (the lower triangle is what the elimination reads)
        for (int i = t >> 6; i < n; i += kSolveThreads / 64)
          for (int k = t & 63; k <= i; k += 64) a.H[S.h_off + (int64_t)i * n + k] = h_entry(a, S, i, k);
        for (int i = t; i < n; i += kSolveThreads) a.b[S.v_off + i] = b_entry(a, S, i);
        __threadfence_block();
        __syncthreads();
      }
    }
    if (dense) {
      const double* H = a.H + S.h_off;
      double tr = 0.0;
      for (int i = t; i < n; i += kSolveThreads) tr += H[(int64_t)i * n + i];
      tr = block_sum(tr, red);
      if (tr > 0.0) {  // otherwise no pair touches a free frame: nothing moves
        const double mu = S.damping_rel * tr / n;
        if (n <= kLdsSystem) {
          for (int idx = t; idx < n * n; idx += kSolveThreads) {
            const int i = idx / n, k = idx - i * n;
            if (k <= i) sh.small.A[i * (n + 1) + k] = H[idx];
          }
          for (int i = t; i < n; i += kSolveThreads) sh.small.A[n * (n + 1) + i] = -a.b[S.v_off + i];
          moved = solve_small(n, mu, sh.small);
          if (!moved && t == 0) st[1] = -4;
          if (moved && t < n) a.delta[S.v_off + t] = sh.small.A[n * (n + 1) + t];
        } else {
          solve_blocked(S, a, mu, sh.blocked.buf, st + 1, sh.blocked.zflags);
          __syncthreads();
          moved = st[1] == 0;
        }
      }
    }
    __syncthreads();
    if (moved) {
      const double* y = a.delta + S.v_off;
      for (int k = t; k < n / 6; k += kSolveThreads) {
        const double* xi = y + 6 * k;
        right_update(a.poses + 12 * (S.slot0 + frame_of_reduced(k, S.fixed)), xi[0], xi[1], xi[2], xi[3], xi[4], xi[5]);
      }
    }
  }
  __syncthreads();
  if (threadIdx.x == 0 && iter <= S.n_iter) st[0] = iter + 1;
}

// What follows an evaluation's finalisation, for sets of small problems (small_step): one workgroup per problem sums
// and expands its edges, one wavefront each (unless k_edge_reduce has), records the loss, and then writes H and b as well (STEP_SYSTEM), or
// (STEP_SOLVE) assembles the system in LDS, solves it, moves the poses and prepares the next evaluation's edge
// transforms.  The same operations in the same order as k_edge_reduce, k_assemble, k_loss_only,
// k_solve_update and k_edge_setup, which a large set needs more than one workgroup for: launches and the gaps
// between them are most of a small iteration (2 frames x 5,000 points: 57 us an iteration, now
// 28, of which this kernel 11.3; 8 frames and 28 edges of 2,000 points: 15).  One chain of reads after another,
// and its code, 15 KB, is fetched anew every iteration; with the loss, H and b read one after the other by the
// same wavefront the two took 12.4 and 17.
template <int MODE, int STEP, typename TT>
__global__ __launch_bounds__(kSolveThreads) void k_step(SolveArgs a, StepArgs u) {
  __shared__ SmallShared sh;
  __shared__ EdgeSums<TT> sums[kSolveThreads / 64];
  const ProbSys S = a.sys[blockIdx.x];
  const int t = threadIdx.x, w = t >> 6;
  if (blockIdx.x == 0 && t == 0 && u.n_items) *u.n_items = 0u;  // of the next evaluation's sweep
  if (u.partial)
    for (int e = S.e0 + w; e < S.e0 + S.E; e += kSolveThreads / 64)
      reduce_edge<TT>(u.partial, u.edges[e], u.xf[e], MODE, sums[w], u.edge_out + (int64_t)e * kEdgeVals);
  __threadfence_block();
  __syncthreads();
  // the loss, H and b by different wavefronts: each is a chain of dependent reads
  const int n = S.n, back = kSolveThreads - 1 - t;
  if (w == 8) record_loss(a, S);
  if constexpr (STEP == STEP_SYSTEM) {
    for (int idx = t; idx < n * n; idx += kSolveThreads) a.H[S.h_off + idx] = h_entry(a, S, idx / n, idx % n);
    if (back < n) a.b[S.v_off + back] = b_entry(a, S, back);
  }
  if constexpr (STEP == STEP_SOLVE) {
    int32_t* st = a.state + S.state_off;
    const int iter = st[0];
    const bool run = iter < S.n_iter && st[1] == 0 && n > 0;
    if (run) {
      double* A = sh.A;
      for (int e = t; e < n * (n + 1) / 2; e += kSolveThreads) {  // the lower triangle
        int i = (int)((sqrtf(8.0f * (float)e + 1.0f) - 1.0f) * 0.5f);
        i += (i + 1) * (i + 2) / 2 <= e ? 1 : 0;
        i -= i * (i + 1) / 2 > e ? 1 : 0;
        const int k = e - i * (i + 1) / 2;
        A[i * (n + 1) + k] = h_entry(a, S, i, k);
      }
      if (back < n) A[n * (n + 1) + back] = -b_entry(a, S, back);
      __syncthreads();
      // every wavefront for itself, in block_sum's order
      const int lane = t & 63;
      double tr = wave_sum(lane < n ? A[lane * (n + 2)] : 0.0);
      if (n > 64) tr += wave_sum(lane + 64 < n ? A[(lane + 64) * (n + 2)] : 0.0);
      if (tr > 0.0) {  // otherwise no pair touches a free frame: nothing moves
        if (solve_small(n, S.damping_rel * tr / n, sh)) {
          for (int k = t; k < n / 6; k += kSolveThreads) {
            const int at = n * (n + 1) + 6 * k;
            right_update(a.poses + 12 * (S.slot0 + frame_of_reduced(k, S.fixed)), A[at], A[at + 1], A[at + 2],
                         A[at + 3], A[at + 4], A[at + 5]);
          }
        } else if (t == 0) {
          st[1] = -4;
        }
      }
    }
    __threadfence_block();
    __syncthreads();
    if (t == 0 && iter <= S.n_iter) st[0] = iter + 1;
    for (int e = S.e0 + t; e < S.e0 + S.E; e += kSolveThreads) {
      EdgeXf o;
      rule_relative(a.poses + 12 * u.edges[e].m, a.poses + 12 * u.edges[e].n, o.R, o.t);
      u.xf[e] = o;
    }
  }
}

}  // namespace

hipError_t launch_assemble(const SolveArgs& a, hipStream_t st) {
  if (a.n_prob <= 0) return hipSuccess;
  const int64_t n = a.n_max;
  const int64_t work = n * n + n;
  if (work > 0) k_assemble<<<dim3((unsigned)((work + 255) / 256), (unsigned)a.n_prob), 256, 0, st>>>(a);
  k_loss_only<<<a.n_prob, 64, 0, st>>>(a);
  return hipGetLastError();
}

template <int MODE, typename TT>
static void run_step(const SolveArgs& a, const StepArgs& u, int step, hipStream_t st) {
  const unsigned nb = (unsigned)a.n_prob;
  if (step == STEP_LOSS) k_step<MODE, STEP_LOSS, TT><<<nb, kSolveThreads, 0, st>>>(a, u);
  else if constexpr (MODE == MODE_NORMAL) {
    if (step == STEP_SYSTEM) k_step<MODE, STEP_SYSTEM, TT><<<nb, kSolveThreads, 0, st>>>(a, u);
    else k_step<MODE, STEP_SOLVE, TT><<<nb, kSolveThreads, 0, st>>>(a, u);
  }
}

bool small_step(const ProbSys& S) { return S.n <= kLdsSystem && S.E <= kStepEdges; }

hipError_t launch_step(const SolveArgs& a, const StepArgs& u, int mode, int step, bool fp32_sums, hipStream_t st) {
  if (a.n_prob <= 0) return hipSuccess;
  if (step == STEP_NONE || (mode == MODE_LOSS && step > STEP_LOSS)) return hipErrorInvalidValue;
  if (mode == MODE_LOSS) {
    if (fp32_sums) run_step<MODE_LOSS, float>(a, u, step, st);
    else run_step<MODE_LOSS, double>(a, u, step, st);
  } else {
    if (fp32_sums) run_step<MODE_NORMAL, float>(a, u, step, st);
    else run_step<MODE_NORMAL, double>(a, u, step, st);
  }
  return hipGetLastError();
}

hipError_t launch_solve_update(const SolveArgs& a, hipStream_t st) {
  if (a.n_prob > 0) k_solve_update<<<a.n_prob, kSolveThreads, 0, st>>>(a);
  return hipGetLastError();
}

hipError_t launch_loss_only(const SolveArgs& a, hipStream_t st) {
  if (a.n_prob > 0) k_loss_only<<<a.n_prob, 64, 0, st>>>(a);
  return hipGetLastError();
}

}  // namespace rkhsba
