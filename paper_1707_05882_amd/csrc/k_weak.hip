// Eigen-decomposition of the weakly coupled orders by a block perturbation iteration.
//
// At Fourier order m the scattering couples directions with a strength that falls like the
// expansion coefficients of degree m and above, while the unscattered part of G = F~ E~ is the
// diagonal 1/mu_i^2 on the four Stokes components of node i. From some order on (5 to 10 for the
// usual phase functions, out of 2 N) G is a small perturbation of that diagonal, and the general
// eigensolver's 25 n^3 latency-bound operations per order are not needed. With d_i the mean of the
// diagonal of G's 4 x 4 block of node i, Delta = G - diag(d), and U normalised to the identity in its
// diagonal blocks, G U = U blockdiag(Lambda_j) is, block column by block column,
//     Lambda_j = d_j + P_jj,   U_ij = -(P_ij - U_ij P_jj) / (d_i - d_j)   (i != j),   P = Delta U,
// which is iterated from U = I. Each step multiplies the error by about the ratio of coupling to
// eigenvalue distance, so an order of strength 1e-3 takes four or five steps of 2 n^3 matrix-core
// operations. Blocks, not single columns: the four Stokes components of a node are degenerate
// without scattering, and their 4 x 4 block Lambda_j is diagonalised at the end (eig4.hpp).
//
// The decision is made from the iteration itself, per order: it is accepted when the change of every
// block column falls to rounding (extrapolated by its measured rate), and given up when it does
// not shrink, when the block of a node is close to defective, or when eigenvectors grow large;
// such an order goes to the general eigensolver, which skips the accepted ones. The products are
// formed entry by entry with G's own grading (row i scales with 1/mu_i^2), so the eigenpairs of the
// small eigenvalues come out to their own rounding and need no refinement step: against the oracle
// the response of an accepted order has at most the error of the refined general solver (1e-12 to
// 2e-11 at N = 32, 64).
//
// Above n = 128 only the faint orders are taken (kWeakFaint). There the general solver's own error in
// the orders of moderate coupling, whose clusters of four nearly equal eigenvalues it cannot separate,
// reaches 1e-7 of the rms of F_r (against 3e-10 here), so taking those orders as well would be more
// accurate and faster still, but would move results by that much; with the faint orders alone they
// stay within 1e-8 of it.
//
// Work split: block columns are independent, so a workgroup takes a panel of 64, 32 or 16 columns
// (n <= 128, 256, 512: the panel fills 64 KB of LDS) and keeps it there over all steps, with no
// exchange between workgroups. Per step the panel is the B operand of v_mfma_f64_16x16x4 and G
// streams from the L2 as the A operand: a lane loads four consecutive entries of a row, which serve
// as the k index 4 (lane / 16) + s of MFMA step s, so every load is a full 32-byte piece of a
// 128-byte row segment. The panels of one order run on one XCD and share its L2.
//
// Measured (with the stages that skip the accepted orders): 72 layers of 64 orders at N = 32 96.8 ->
// 43.2 ms; 64 layers of N = 16 to 64 252 -> 149 ms; N = 128 with 256 orders 868 -> 532 ms.
#include "eig4.hpp"
#include "vbrdf_internal.hpp"

namespace vbrdf {

typedef double double4_t __attribute__((ext_vector_type(4)));

constexpr int kWeakCells = 8192;     // doubles of a panel: 16 ceil(n / 16) rows x its columns
constexpr int kWeakNodes = 16;       // nodes of the widest panel
constexpr int kWeakMaxSteps = 48;    // an order foreseen to need more is given up
constexpr double kWeakMaxU = 50.0;   // largest entry of U accepted
// Largest entry of U after the first step (outside its diagonal blocks) of an order taken above
// n = kWeakAllMaxN; the difference from the general solver is a few per cent of the order's response
constexpr double kWeakFaint = 3e-10;
constexpr double kWeakUlp = 2.220446049250313e-16;

struct WeakLds {
  double U[kWeakCells];               // the panel of U, row-major
  double gap[kWeakCells / 16];        // 1 / (d_i - d_j) per node pair; scratch of the 4 x 4 solves later
  double P[kWeakNodes * 16];          // P_jj of the panel's nodes
  double Q[kWeakNodes * 16];
  double d[kMaxN];
  unsigned long long stat[2][kWeakNodes][2];  // largest change and largest entry per block column (bits)
  int stop[2];
};

// The iteration on one panel: kRt row tiles per wave, kCt column tiles of 16 per panel (kRt kCt = 4
// accumulators). Returns whether it converged; U and the blocks P_jj are left in LDS.
template <int kRt, int kCt>
__device__ __forceinline__ bool weak_panel(const Item& it, double* base, int panel, WeakLds& s) {
  constexpr int C = 16 * kCt, CN = C / 4;
  const int n = it.n, N = it.N, nt = (n + 15) >> 4;
  const int c0 = panel * C;
  const double* __restrict__ G = base + (int64_t)kBufG * n * n;
  double* ex = base + extras_off(n);
  int* flag = weak_flag(ex, n);
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int cn = min(CN, N - c0 / 4);  // nodes of this panel

  for (int i = tid; i < N; i += kWeakThreads) {
    const double* g = G + (int64_t)(4 * i) * (n + 1);
    s.d[i] = 0.25 * ((g[0] + g[n + 1]) + (g[2 * (n + 1)] + g[3 * (n + 1)]));
  }
  if (tid < 2 * kWeakNodes * 2) s.stat[tid / (2 * kWeakNodes)][(tid / 2) % kWeakNodes][tid & 1] = 0;
  __syncthreads();
  for (int t = tid; t < nt * 4 * CN; t += kWeakThreads) {
    const int i = t / CN, j = c0 / 4 + t % CN;
    s.gap[t] = (i < N && j < N && i != j) ? 1.0 / (s.d[i] - s.d[j]) : 0.0;
  }
  __syncthreads();
  // first step from U = I: U_ij = -G_ij / (d_i - d_j)
  double first = 0.0;
  for (int t = tid; t < nt * 16 * C; t += kWeakThreads) {
    const int r = t / C, c = t % C, col = c0 + c;
    double v = 0.0;
    if (r < n && col < n)
      v = (r >> 2) == (col >> 2) ? (r == col ? 1.0 : 0.0) : -G[(int64_t)r * n + col] * s.gap[(r >> 2) * CN + (c >> 2)];
    s.U[t] = v;
    if (r < n && col < n && (r >> 2) != (col >> 2)) first = v == v ? fmax(first, fabs(v)) : INFINITY;
  }
  if (n > kWeakAllMaxN) {
    for (int o = 1; o < 64; o <<= 1) first = fmax(first, __shfl_xor(first, o));
    if (lane == 0) s.P[wave] = first;
  }
  __syncthreads();
  if (n > kWeakAllMaxN) {
    for (int w = 0; w < kWeakThreads / 64; ++w) first = fmax(first, s.P[w]);
    if (!(first <= kWeakFaint)) return false;  // uniform
    __syncthreads();
  }

  double prev = 1.0;  // relative change of the step before (the first step: all of it)
  int slow = 0;
  bool ok = false;
  for (int step = 0; step < kWeakMaxSteps; ++step) {
    int ln = lane;
    asm volatile("" : "+v"(ln));  // addresses are formed anew in each step: kept, they would spill
    const int li = ln & 15, lk = ln >> 4;
    double4_t acc[kRt][kCt];
#pragma unroll
    for (int a = 0; a < kRt; ++a)
#pragma unroll
      for (int b = 0; b < kCt; ++b) acc[a][b] = (double4_t){0.0, 0.0, 0.0, 0.0};
    // rows beyond the matrix read its last row, entries beyond a row its start: the former are not
    // used, the latter meet zero rows of U (n is a multiple of 4, so a lane's four entries are inside
    // or outside together)
    const double* row[kRt];
#pragma unroll
    for (int a = 0; a < kRt; ++a) row[a] = G + (int64_t)min((wave + 8 * a) * 16 + li, n - 1) * n;
    if (wave < nt) {
#pragma unroll 1
      for (int kk = 0; kk < nt; ++kk) {  // the four waves of a SIMD cover one another's loads
        double4_t g[kRt];
        const int k = kk * 16 + 4 * lk;
#pragma unroll
        for (int a = 0; a < kRt; ++a) g[a] = *reinterpret_cast<const double4_t*>(row[a] + (k < n ? k : 0));
#pragma unroll
        for (int a = 0; a < kRt; ++a)
          if (wave + 8 * a == kk && (li >> 2) == lk) {  // Delta: the diagonal entry of this lane's row
            const double di = s.d[min(kk * 4 + lk, N - 1)];
#pragma unroll
            for (int q = 0; q < 4; ++q) g[a][q] -= (li & 3) == q ? di : 0.0;
          }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          double b[kCt];
#pragma unroll
          for (int c = 0; c < kCt; ++c) b[c] = s.U[(kk * 16 + 4 * lk + q) * C + c * 16 + li];
#pragma unroll
          for (int a = 0; a < kRt; ++a) {
            if (wave + 8 * a >= nt) continue;  // uniform
#pragma unroll
            for (int c = 0; c < kCt; ++c)
              acc[a][c] = __builtin_amdgcn_mfma_f64_16x16x4f64(g[a][q], b[c], acc[a][c], 0, 0, 0);
          }
        }
      }
      // accumulator register v of a tile: row 16 tile + lk + 4 v, that is Stokes component lk of
      // node 4 tile + v; column li of the column tile
#pragma unroll
      for (int a = 0; a < kRt; ++a)
#pragma unroll
        for (int c = 0; c < kCt; ++c) {
          const int cb = c * 4 + (li >> 2), j = c0 / 4 + cb;
#pragma unroll
          for (int v = 0; v < 4; ++v)
            if ((wave + 8 * a) * 4 + v == j && j < N) s.P[cb * 16 + lk * 4 + (li & 3)] = acc[a][c][v];
        }
    }
    __syncthreads();
    if (tid < 2 * kWeakNodes) s.stat[(step + 1) & 1][tid >> 1][tid & 1] = 0;
    if (tid == 0) s.stop[step & 1] = __hip_atomic_load(flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >= 0;
    double dmax[kCt], umax[kCt];
#pragma unroll
    for (int c = 0; c < kCt; ++c) dmax[c] = umax[c] = 0.0;
#pragma unroll
    for (int a = 0; a < kRt; ++a)
#pragma unroll
      for (int c = 0; c < kCt; ++c) {
        const int cb = c * 4 + (li >> 2), j = c0 / 4 + cb;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int i = (wave + 8 * a) * 4 + v;
          if (i < N && j < N && i != j) {
            const double* u = s.U + (4 * i + lk) * C + cb * 4;
            double p = acc[a][c][v];
#pragma unroll
            for (int q = 0; q < 4; ++q) p -= u[q] * s.P[cb * 16 + q * 4 + (li & 3)];
            p *= -s.gap[i * CN + cb];
            dmax[c] = fmax(dmax[c], fabs(p - u[li & 3]));
            // fmax drops a NaN operand: keep it visible
            umax[c] = p == p ? fmax(umax[c], fabs(p)) : INFINITY;
            acc[a][c][v] = p;
          }
          __builtin_amdgcn_sched_barrier(0);  // one entry's operands at a time (registers)
        }
      }
    __syncthreads();
#pragma unroll
    for (int a = 0; a < kRt; ++a)
#pragma unroll
      for (int c = 0; c < kCt; ++c) {
        const int cb = c * 4 + (li >> 2), j = c0 / 4 + cb;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int i = (wave + 8 * a) * 4 + v;
          if (i < N && j < N && i != j) s.U[(4 * i + lk) * C + c * 16 + li] = acc[a][c][v];
        }
      }
#pragma unroll
    for (int c = 0; c < kCt; ++c) {
      for (int o = 1; o < 64; o = o == 2 ? 16 : 2 * o) {  // the 4 columns of a block, the 4 row groups
        dmax[c] = fmax(dmax[c], __shfl_xor(dmax[c], o));
        umax[c] = fmax(umax[c], __shfl_xor(umax[c], o));
      }
      if ((ln & 51) == 0) {  // lanes 0, 4, 8, 12
        unsigned long long* st = s.stat[step & 1][c * 4 + (li >> 2)];
        atomicMax(st, (unsigned long long)__double_as_longlong(dmax[c]));
        atomicMax(st + 1, (unsigned long long)__double_as_longlong(umax[c]));
      }
    }
    __syncthreads();
    if (s.stop[step & 1]) break;  // another panel of this order has given up
    double r = 0.0, big = 0.0;
    for (int j = 0; j < cn; ++j) {
      const double dj = __longlong_as_double((long long)s.stat[step & 1][j][0]);
      const double uj = __longlong_as_double((long long)s.stat[step & 1][j][1]);
      big = fmax(big, uj);
      if (dj > 0.0) r = fmax(r, dj / uj);
    }
    if (!(big <= kWeakMaxU)) break;
    const double rate = r / prev;
    // what the steps left out would still change: r rate / (1 - rate)
    if (r <= 4.0 * kWeakUlp || (rate < 0.9 && r * rate <= kWeakUlp * (1.0 - rate))) {
      ok = true;
      break;
    }
    if (rate > 0.8) {
      if (r <= 32.0 * kWeakUlp) {  // the change has reached the rounding of the products
        ok = true;
        break;
      }
      if (++slow > 2) break;
    }
    // steps still needed at this rate, after the first few have settled it
    if (step >= 4 && rate < 1.0 && step + log(r * (1.0 / kWeakUlp)) / -log(rate) > kWeakMaxSteps) break;
    prev = r;
  }
  return ok;
}

// Grid: xcd_grid(n_items, panels) workgroups, panels = the largest number of panels of an item;
// k_legendre has set every item's flag.
__global__ __launch_bounds__(kWeakThreads, 4) void k_weak_eigen(const Item* items, int n_items, int panels, double* ws,
                                                                const int32_t* status) {
  int g, panel;
  xcd_split(blockIdx.x, panels, g, panel);
  // Consecutive items go to the XCDs in turn, so a layer of 8 k orders would put the same orders of
  // every layer, with their like step counts, on one XCD: every eight are rotated by a hash.
  const unsigned rot = ((unsigned)(g >> 3) * 0x9E3779B1u) >> 29;
  g = (g & ~7) | ((g + rot) & 7);
  if (g >= n_items) return;
  const Item it = items[g];
  const int n = it.n, tid = threadIdx.x, C = weak_cols(n), c0 = panel * C;
  if (status[it.layer] != 0 || c0 >= n) return;
  __shared__ WeakLds s;
  double* base = ws + it.ws;
  bool ok;
  if (n <= 128)
    ok = weak_panel<1, 4>(it, base, panel, s);
  else if (n <= 256)
    ok = weak_panel<2, 2>(it, base, panel, s);
  else
    ok = weak_panel<4, 1>(it, base, panel, s);
  double* ex = base + extras_off(n);
  if (!ok) {  // uniform
    if (tid == 0) __hip_atomic_store(weak_flag(ex, n), 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return;
  }
  // a thread per node diagonalises Lambda_j - d_j = P_jj
  if (tid < min(C / 4, it.N - c0 / 4)) {
    const int j = c0 / 4 + tid;
    // (the gaps are done with: scratch)
    if (!eig4(s.P + tid * 16, s.Q + tid * 16, s.gap + tid * 32, ex + 4 * j, ex + n + 4 * j, 8.0 * kWeakUlp * s.d[j]))
      __hip_atomic_store(weak_flag(ex, n), 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    for (int q = 0; q < 4; ++q) ex[4 * j + q] += s.d[j];
  }
  __syncthreads();
  double* __restrict__ Uo = base + (int64_t)kBufU * n * n;
  for (int t = tid; t < n * C; t += kWeakThreads) {
    const int r = t / C, c = t % C;
    if (c0 + c >= n) continue;
    const double* u = s.U + r * C + (c & ~3);
    const double* q = s.Q + (c >> 2) * 16 + (c & 3);
    Uo[(int64_t)r * n + c0 + c] = u[0] * q[0] + u[1] * q[4] + u[2] * q[8] + u[3] * q[12];
  }
}

}  // namespace vbrdf
