// LU factorisation with partial pivoting of systems of up to 192 rows, the matrix in registers.
//
// Held in LDS with a workgroup barrier per column, a factorisation took 196 us at n = 128, of which
// 75 us were the LDS traffic of the rank-1 updates and the rest the latency of 128 columns. Here
// wave w < kT keeps rows 16 w .. 16 w + 15 as accumulator tiles of v_mfma_f64_16x16x4, one for each 16
// columns, and one more wave factors panels of 16 columns: rows in its lanes (row = lane + 64 i),
// the 16 columns in registers, the pivot by a maximum over the wave, the pivot row by lane reads, no
// barrier and no LDS access within a panel. Per panel
//   A  the panel wave factors the panel, while the others give the columns right of it the update of
//      the panel before,
//   B  the other waves hand over the pivot rows of their tiles,
//   C  the panel wave solves L11 U12 = A12, a column per lane, the others write the panel to memory,
//   D  the next panel's columns take the update A22 -= L21 U12 and go to the panel wave.
// Row exchanges stay logical: a row keeps its place, with its multiplier zero once it has been
// the pivot row, so that its tiles then hold its row of Uu. The operations on an element and their order
// are those of the column by column form and of the blocked one (k_lu): all give the same bits. Bound by the
// panel wave's chain of n columns: 560 cycles each up to n = 64 (a row per lane), 820 up to 128, 980 up to
// 192, next to 370 for the solve of 64 columns of U12 and 80 to 250 for each of the other phases, by 16 columns.
// Measured, the form before -> now: n = 32 41 -> 14 us, n = 64 81 -> 24 us, n = 128 196 -> 85 us, n = 160
// (blocked) 220 -> 148 us; 9216 systems of n = 128 4.48 -> 1.96 ms. The sizes end at 192, where both kinds of waves
// are at their limit of 128 registers without private scratch, which callers that must not allocate rely on
// (k_lu_mid at n = 160: 170 us). There a lane of the panel wave solves for one column at a time,
// and tiles beyond the matrix are updated like the others (branches around them took registers).
#include "vbrdf_internal.hpp"

namespace vbrdf {

typedef double double4_t __attribute__((ext_vector_type(4)));

// The values of the one lane in e, read under it as the execution mask (8 cycles a word; a lane read by a
// register's index takes 12). For a wave whose 64 lanes are all active. The two scalar instructions at
// the end are the wait states between a lane read and a vector instruction that takes its result.
template <int kN>
__device__ __forceinline__ void lane_values(uint64_t e, const double (&v)[kN], double (&out)[kN]) {
  static_assert(kN == 1 || kN == 2 || kN == 4 || kN == 8, "");
  int lo[kN], hi[kN];
  if constexpr (kN == 1)
    asm volatile(
        "s_mov_b64 exec, %2\n"
        "v_readfirstlane_b32 %0, %3\n"
        "v_readfirstlane_b32 %1, %4\n"
        "s_mov_b64 exec, -1\n"
        "s_nop 0"
        : "=&s"(lo[0]), "=&s"(hi[0])
        : "s"(e), "v"(__double2loint(v[0])), "v"(__double2hiint(v[0])));
  if constexpr (kN == 2)
    asm volatile(
        "s_mov_b64 exec, %4\n"
        "v_readfirstlane_b32 %0, %5\n"
        "v_readfirstlane_b32 %1, %6\n"
        "v_readfirstlane_b32 %2, %7\n"
        "v_readfirstlane_b32 %3, %8\n"
        "s_mov_b64 exec, -1\n"
        "s_nop 0"
        : "=&s"(lo[0]), "=&s"(hi[0]), "=&s"(lo[1]), "=&s"(hi[1])
        : "s"(e), "v"(__double2loint(v[0])), "v"(__double2hiint(v[0])), "v"(__double2loint(v[1])), "v"(__double2hiint(v[1])));
  if constexpr (kN == 4)
    asm volatile(
        "s_mov_b64 exec, %8\n"
        "v_readfirstlane_b32 %0, %9\n"
        "v_readfirstlane_b32 %1, %10\n"
        "v_readfirstlane_b32 %2, %11\n"
        "v_readfirstlane_b32 %3, %12\n"
        "v_readfirstlane_b32 %4, %13\n"
        "v_readfirstlane_b32 %5, %14\n"
        "v_readfirstlane_b32 %6, %15\n"
        "v_readfirstlane_b32 %7, %16\n"
        "s_mov_b64 exec, -1\n"
        "s_nop 0"
        : "=&s"(lo[0]), "=&s"(hi[0]), "=&s"(lo[1]), "=&s"(hi[1]), "=&s"(lo[2]), "=&s"(hi[2]), "=&s"(lo[3]), "=&s"(hi[3])
        : "s"(e), "v"(__double2loint(v[0])), "v"(__double2hiint(v[0])), "v"(__double2loint(v[1])), "v"(__double2hiint(v[1])), "v"(__double2loint(v[2])), "v"(__double2hiint(v[2])), "v"(__double2loint(v[3])), "v"(__double2hiint(v[3])));
  if constexpr (kN == 8)
    asm volatile(
        "s_mov_b64 exec, %16\n"
        "v_readfirstlane_b32 %0, %17\n"
        "v_readfirstlane_b32 %1, %18\n"
        "v_readfirstlane_b32 %2, %19\n"
        "v_readfirstlane_b32 %3, %20\n"
        "v_readfirstlane_b32 %4, %21\n"
        "v_readfirstlane_b32 %5, %22\n"
        "v_readfirstlane_b32 %6, %23\n"
        "v_readfirstlane_b32 %7, %24\n"
        "v_readfirstlane_b32 %8, %25\n"
        "v_readfirstlane_b32 %9, %26\n"
        "v_readfirstlane_b32 %10, %27\n"
        "v_readfirstlane_b32 %11, %28\n"
        "v_readfirstlane_b32 %12, %29\n"
        "v_readfirstlane_b32 %13, %30\n"
        "v_readfirstlane_b32 %14, %31\n"
        "v_readfirstlane_b32 %15, %32\n"
        "s_mov_b64 exec, -1\n"
        "s_nop 0"
        : "=&s"(lo[0]), "=&s"(hi[0]), "=&s"(lo[1]), "=&s"(hi[1]), "=&s"(lo[2]), "=&s"(hi[2]), "=&s"(lo[3]), "=&s"(hi[3]), "=&s"(lo[4]), "=&s"(hi[4]), "=&s"(lo[5]), "=&s"(hi[5]), "=&s"(lo[6]), "=&s"(hi[6]), "=&s"(lo[7]), "=&s"(hi[7])
        : "s"(e), "v"(__double2loint(v[0])), "v"(__double2hiint(v[0])), "v"(__double2loint(v[1])), "v"(__double2hiint(v[1])), "v"(__double2loint(v[2])), "v"(__double2hiint(v[2])), "v"(__double2loint(v[3])), "v"(__double2hiint(v[3])), "v"(__double2loint(v[4])), "v"(__double2hiint(v[4])), "v"(__double2loint(v[5])), "v"(__double2hiint(v[5])), "v"(__double2loint(v[6])), "v"(__double2hiint(v[6])), "v"(__double2loint(v[7])), "v"(__double2hiint(v[7])));
#pragma unroll
  for (int i = 0; i < kN; ++i) out[i] = __hiloint2double(hi[i], lo[i]);
}

// Columns kC .. 15 of the row of the one lane in e.
template <int kC>
__device__ __forceinline__ void row_values(uint64_t e, const double (&a)[16], double (&u)[16]) {
  if constexpr (kC < 16) {
    constexpr int kN = 16 - kC >= 8 ? 8 : (16 - kC >= 4 ? 4 : (16 - kC >= 2 ? 2 : 1));
    double v[kN], o[kN];
#pragma unroll
    for (int i = 0; i < kN; ++i) v[i] = a[kC + i];
    lane_values<kN>(e, v, o);
#pragma unroll
    for (int i = 0; i < kN; ++i) u[kC + i] = o[i];
    row_values<kC + kN>(e, a, u);
  }
}

template <int kCtrl>
__device__ __forceinline__ uint32_t dpp_umax(uint32_t v) {
  return max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, kCtrl, 0xf, 0xf, true));
}

// Largest v over the 64 lanes, in all of them.
__device__ __forceinline__ uint32_t wave_umax(uint32_t v) {
  v = dpp_umax<0xB1>(v);   // neighbours, pairs, halves of a row of 16, rows
  v = dpp_umax<0x4E>(v);
  v = dpp_umax<0x141>(v);
  v = dpp_umax<0x140>(v);
  v = dpp_umax<0x142>(v);  // lane 15 of a row into the next row, then lane 31 into the upper half
  v = dpp_umax<0x143>(v);
  return __builtin_amdgcn_readlane((int)v, 63);
}

// Entry and position of the pivot row, and its columns right of q: the one row in e[kI], ..., e[kPer - 1].
template <int kPer, int q, int kI>
__device__ __forceinline__ void pivot_row(const uint64_t (&e)[kPer], const double (&a)[kPer][16],
                                          const int (&pos)[kPer], double& piv, int& pb, double (&u)[16]) {
  if constexpr (kI + 1 < kPer)
    if (e[kI] == 0) return pivot_row<kPer, q, kI + 1>(e, a, pos, piv, pb, u);
  const double v[2] = {a[kI][q], __hiloint2double(0, pos[kI])};
  double o[2];
  lane_values<2>(e[kI], v, o);
  piv = o[0];
  pb = __double2loint(o[1]);
  row_values<q + 1>(e[kI], a[kI], u);
}

// Factors panel columns k0 .. min(k0 + 16, n) - 1. a[i][c]: row lane + 64 i, column k0 + c. pos[i]: the
// row's position, below the column for a row that has been the pivot, -1 for lanes without a row. The
// columns go to P (multipliers where the row has not been the pivot). A column without a pivot (beyond n,
// or nothing but NaN) leaves rows and positions as they are; the caller counts the pivots and looks at
// their values (leaving the panel from within made the compiler copy what follows for each column).
template <int kPer, int q = 0>
__device__ __forceinline__ void lu_panel(double (&a)[kPer][16], int (&pos)[kPer], int k0, double* P, int ld) {
  if constexpr (q < 16) {
    const int k = k0 + q, lane = threadIdx.x & 63;
    // The pivot: the largest modulus (a NaN is passed over), ties to the smaller position. The moduli
    // are compared as integers, upper words (plus one, zero for rows that are out) first; those alone
    // nearly always decide.
    uint32_t key[kPer], best = 0;
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
      const uint32_t h = (uint32_t)__double2hiint(a[i][q]) & 0x7fffffffu;
      key[i] = pos[i] >= k && h <= 0x7ff00000u ? h + 1 : 0u;
      best = max(best, key[i]);
    }
    best = wave_umax(best);
    uint64_t e[kPer];
    int hits = 0, from = k;
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
      e[i] = __builtin_amdgcn_uicmp(key[i], best, 32);  // equal
      hits += __builtin_popcountll(e[i]);
    }
    if (__builtin_expect(hits != 1, 0)) {
      uint32_t low = 0, p = 0;
#pragma unroll
      for (int i = 0; i < kPer; ++i)
        if (key[i] == best) low = max(low, (uint32_t)__double2loint(a[i][q]));
      low = wave_umax(low);
#pragma unroll
      for (int i = 0; i < kPer; ++i) {
        key[i] = key[i] != 0 && key[i] == best && (uint32_t)__double2loint(a[i][q]) == low
                     ? 0x10000u - (uint32_t)pos[i]
                     : 0u;
        p = max(p, key[i]);
      }
      best = wave_umax(p);
#pragma unroll
      for (int i = 0; i < kPer; ++i) e[i] = __builtin_amdgcn_uicmp(key[i], best, 32);
      if (best == 0) {
        best = ~0u;
        from = -2;
      }
    }
    double u[16], piv = 0.0;
    int pb = 0;
    pivot_row<kPer, q, 0>(e, a, pos, piv, pb, u);
    const double inv = 1.0 / piv;
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
      pos[i] = pos[i] == from ? pb : pos[i];
      if (key[i] == best) pos[i] = k;
      const bool active = pos[i] > k;
      const double x = a[i][q] * inv, l = active ? x : 0.0;
      P[q * ld + lane + 64 * i] = active ? x : a[i][q];
#pragma unroll
      for (int c = q + 1; c < 16; ++c) a[i][c] = fma(-l, u[c], a[i][c]);
    }
    lu_panel<kPer, q + 1>(a, pos, k0, P, ld);
  }
}

// U12 = L11^-1 A12 in place for the columns lane + 64 i < cols of Ub; sL[s 16 + t] = L11(t, s). For a wave
// with registers to spare. The loads are a column ahead of their use and no more: their address waits for
// the entries before.
template <int kPer>
__device__ __forceinline__ void lu_solve(const double* sL, double* Ub, int ldu, int cols) {
  const int lane = threadIdx.x & 63;
  double x[kPer][16];
#pragma unroll
  for (int i = 0; i < kPer; ++i) {
    const int c = min(lane + 64 * i, cols - 1);
#pragma unroll
    for (int t = 0; t < 16; ++t) x[i][t] = Ub[t * ldu + c];
  }
  double l[16], ln[16];
#pragma unroll
  for (int t = 1; t < 16; ++t) l[t] = sL[t];
#pragma unroll
  for (int s = 0; s < 15; ++s) {
    int z = 0;
#pragma unroll
    for (int i = 0; i < kPer; ++i) asm volatile("" : "+v"(z), "+v"(x[i][s]));
#pragma unroll
    for (int t = s + 2; t < 16; ++t) ln[t] = sL[z + (s + 1) * 16 + t];
#pragma unroll
    for (int t = s + 1; t < 16; ++t)
#pragma unroll
      for (int i = 0; i < kPer; ++i) x[i][t] = fma(-l[t], x[i][s], x[i][t]);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int t = s + 2; t < 16; ++t) l[t] = ln[t];
  }
#pragma unroll
  for (int i = 0; i < kPer; ++i)
    if (lane + 64 * i < cols)
#pragma unroll
      for (int t = 0; t < 16; ++t) Ub[t * ldu + lane + 64 * i] = x[i][t];
}

// Buffer b.src[side] = P^T L Uu of the systems with n_above < n <= 16 kT (side = blockIdx.y: S' and T'
// of the boundary solve, or U^T of the eigenpair refinement). The factor is written transposed into
// b.dst[side], AT[j n + c] = A(c, j), so that column j of Uu (c <= j) and of L (c > j) are contiguous for
// the right division; pivots and 1 / Uu_kk go to the extras block. kT + 1 waves.
template <int kT>
__global__ __launch_bounds__(64 * (kT + 1)) void k_lu_reg(const Item* items, double* ws, int32_t* status, LuBufs b,
                                                          int n_above) {
  const Item it = items[blockIdx.x];
  if (it.n <= n_above || it.n > 16 * kT || layer_failed(status, it.layer) || weak_done(b.skip_weak, ws, it)) return;
  constexpr int kPer = (kT + 3) / 4;
  constexpr bool kTight = kPer == 3;         // both kinds of waves are at their limit of 128 registers
  constexpr int kSolve = kTight ? 1 : kPer;  // columns of U12 that a lane solves for at a time
  constexpr int kLd = 16 * kT + 4;    // columns of P and T: 16 lanes a column apart spread over the banks
  constexpr int kLdu = 16 * kT + 16;  // rows of Ub: two halves of 16 lanes a row apart, likewise
  __shared__ double P[16 * kLd], T[16 * kLd], Ub[16 * kLdu];
  __shared__ __attribute__((aligned(16))) double sL[16 * 16];
  __shared__ int tpos[16 * kT], perm[16 * kT], bad;
  const int n = it.n, which = blockIdx.y, lane = threadIdx.x & 63, lr = lane & 15, kq = lane >> 4;
  const int wv = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  double* base = ws + it.ws;
  double* ex = base + extras_off(n);
  if (b.only_flagged && !boundary_flags(ex, n)->fallback[which]) return;
  const double* __restrict__ A = buf_ptr(ws, it, b.src[which]);
  double* __restrict__ AT = buf_ptr(ws, it, b.dst[which]);
  const int R = (n + 15) >> 4;
  // The two kinds of waves run their own loops, which meet at the same barriers: one before the
  // first panel, and 1 to 4 for each panel (only 1 for the last, or for one that failed).
  if (wv == kT) {
    __builtin_amdgcn_s_setprio(3);
    double a[kPer][16];
    int pos[kPer];
#pragma unroll
    for (int i = 0; i < kPer; ++i) pos[i] = lane + 64 * i < n ? lane + 64 * i : -1;
    if (lane == 0) bad = 0;
    __syncthreads();
    for (int p = 0; p < R; ++p) {
      const int k0 = 16 * p;
#pragma unroll
      for (int i = 0; i < kPer; ++i) {
        const int row = min(lane + 64 * i, 16 * kT - 1);
#pragma unroll
        for (int c = 0; c < 16; ++c) a[i][c] = T[c * kLd + row];
      }
      lu_panel<kPer>(a, pos, k0, P, kLd);
      int pivots = 0;
#pragma unroll
      for (int i = 0; i < kPer; ++i) {
        const int row = lane + 64 * i, t = pos[i] - k0;
        tpos[row] = t;
        bool good = false;
        if (t >= 0 && t < 16 && pos[i] < n) {
          perm[pos[i]] = row;
          const double d = P[t * kLd + row];
          good = d != 0.0 && isfinite(d);
        }
        pivots += __popcll(__ballot(good));
      }
      if (pivots != min(16, n - k0) && lane == 0) {
        bad = 1;
        status[it.layer] = -5;
      }
      __syncthreads();  // 1
      if (bad) return;
      if (p + 1 == R) break;
      for (int t = lane; t < 256; t += 64)  // L11, for the solve
        sL[t] = P[(t >> 4) * kLd + perm[k0 + (t & 15)]];
      __syncthreads();  // 2
      for (int c0 = 0; c0 < 16 * (R - 1 - p); c0 += 64 * kSolve)
        lu_solve<kSolve>(sL, Ub + c0, kLdu, 16 * (R - 1 - p) - c0);
      __syncthreads();  // 3
      __syncthreads();  // 4
    }
  } else {
    double4_t X[kT];  // X[j]: columns of panel p + j, rows 16 wv + 4 v + kq (v: component)
    const bool rows = wv < R;
#pragma unroll
    for (int j = 0; j < kT; ++j)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int row = 16 * wv + 4 * v + kq, col = 16 * j + lr;
        X[j][v] = row < n && col < n ? A[(int64_t)row * n + col] : 0.0;
      }
#pragma unroll
    for (int v = 0; v < 4; ++v) T[lr * kLd + 16 * wv + 4 * v + kq] = X[0][v];
    __syncthreads();
    auto store = [&](int p) {  // panel p in the original order of rows, which the end permutes
      int ln = lane;
      asm volatile("" : "+v"(ln));
#pragma unroll 1
      for (int c = wv; c < min(16, n - 16 * p); c += kT)
#pragma unroll
        for (int i = 0; i < kPer; ++i)
          if (ln + 64 * i < n) AT[(int64_t)(16 * p + c) * n + ln + 64 * i] = P[c * kLd + ln + 64 * i];
    };
    // (the last panel after the loop: left from its middle, the loop would keep two copies of the tiles)
    for (int p = 0; p + 1 < R; ++p) {
      const int rem = R - 1 - p;
      int ln = lane;
      asm volatile("" : "+v"(ln));  // addresses are formed anew for each panel: kept, they would spill
      const int lr = ln & 15, kq = ln >> 4;
      __syncthreads();  // 1
      if (bad) return;
      if (rows)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int t = tpos[16 * wv + 4 * v + kq];
          if (t >= 0 && t < 16)
#pragma unroll
            for (int j = 1; j < kT; ++j)
              if (kTight || j <= rem) Ub[t * kLdu + 16 * (j - 1) + lr] = X[j][v];
        }
      __syncthreads();  // 2
      store(p);
      __syncthreads();  // 3
      double l[4];
      const int late = tpos[16 * wv + lr];
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const double x = P[(4 * t + kq) * kLd + 16 * wv + lr];
        l[t] = late > 4 * t + kq ? -x : 0.0;
      }
      auto update = [&](int j) {
#pragma unroll
        for (int t = 0; t < 4; ++t)
          X[j] = __builtin_amdgcn_mfma_f64_16x16x4f64(l[t], Ub[(4 * t + kq) * kLdu + 16 * (j - 1) + lr], X[j], 0, 0, 0);
      };
      if (rows) {
        update(1);
#pragma unroll
        for (int v = 0; v < 4; ++v) T[lr * kLd + 16 * wv + 4 * v + kq] = X[1][v];
      }
      __syncthreads();  // 4
      if (rows)
#pragma unroll
        for (int j = 2; j < kT; ++j)
          if (kTight || j <= rem) update(j);
      // The tiles are copied now, in another block of the compiled loop than the instructions that wrote them, where
      // the compiler has left out the wait states between the two.
      __builtin_amdgcn_sched_barrier(0);
      asm volatile("s_nop 15\n\ts_nop 3");
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int j = 1; j + 1 < kT; ++j) X[j] = X[j + 1];
    }
    __syncthreads();  // 1
    if (bad) return;
    store(R - 1);
  }
  __syncthreads();  // the factor in the original order of rows is in memory, the final order in perm
  double* id = ex + (4 + which) * (int64_t)n;
  int* pm = reinterpret_cast<int*>(ex + 2 * (int64_t)n) + which * n;
  for (int i = threadIdx.x; i < n; i += 64 * (kT + 1)) {
    pm[i] = perm[i];
    id[i] = 1.0 / AT[(int64_t)i * n + perm[i]];
  }
  __syncthreads();
  constexpr int kCols = 4;
  for (int j0 = kCols * wv; j0 < n; j0 += kCols * (kT + 1)) {  // n is a multiple of 4
    double x[kCols][kPer];
#pragma unroll
    for (int j = 0; j < kCols; ++j)
#pragma unroll
      for (int i = 0; i < kPer; ++i)
        if (lane + 64 * i < n) x[j][i] = AT[(int64_t)(j0 + j) * n + perm[lane + 64 * i]];
#pragma unroll
    for (int j = 0; j < kCols; ++j)
#pragma unroll
      for (int i = 0; i < kPer; ++i)
        if (lane + 64 * i < n) AT[(int64_t)(j0 + j) * n + lane + 64 * i] = x[j][i];
  }
}
// The systems of kLuRegMaxn < n <= kLuMidMaxn rows, in place: panels of 16 columns by wave 0 as above (four rows
// in each lane), the matrix in global memory. Then a wave per block of 16 columns to the right: U12 =
// L11^-1 A12 by forward substitution, in the B-operand layout of v_mfma_f64_16x16x4 (x[t] = row 4 t +
// lane / 16, column lane % 16), and A22 -= L21 U12 in 16 x 16 tiles, the next tile loading meanwhile.
// The order of operations on an element is k_lu's, whose panels (a barrier for each of four phases of a column,
// 5 k cycles) took most of its time: 1536 systems of n = 256 7.15 -> 3.47 ms. Above 256 rows a lane's share no longer fits its registers.
__global__ __launch_bounds__(kLuThreadsBig) void k_lu_mid(const Item* items, double* ws, int32_t* status, LuBufs b) {
  const Item it = items[blockIdx.x];
  if (it.n <= kLuRegMaxn || it.n > kLuMidMaxn || layer_failed(status, it.layer) || weak_done(b.skip_weak, ws, it)) return;
  constexpr int kPer = kLuMidMaxn / 64, kLd = kLuMidMaxn + 1, NT = kLuThreadsBig, nw = NT / 64;
  __shared__ double S[16 * kLd], P[16 * kLd], sL[16 * 17];
  __shared__ int perm[kLuMidMaxn], bad;
  const int n = it.n, which = blockIdx.y, tid = threadIdx.x, lane = tid & 63, lr = lane & 15, kq = lane >> 4;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  double* base = ws + it.ws;
  double* ex = base + extras_off(n);
  if (b.only_flagged && !boundary_flags(ex, n)->fallback[which]) return;
  double* __restrict__ A = buf_ptr(ws, it, b.src[which]);
  double* __restrict__ AT = buf_ptr(ws, it, b.dst[which]);
  double* id = ex + (4 + which) * (int64_t)n;
  int* pm = reinterpret_cast<int*>(ex + 2 * (int64_t)n) + which * n;
  for (int i = tid; i < n; i += NT) perm[i] = i;
  if (tid == 0) bad = 0;
  __syncthreads();
  for (int k0 = 0; k0 < n; k0 += 16) {
    const int m = n - k0, w = min(16, m);
    if (wv == 0) {
      double a[kPer][16];
      int pos[kPer], row[kPer];
#pragma unroll
      for (int i = 0; i < kPer; ++i) {
        const int r = lane + 64 * i;
        row[i] = perm[k0 + min(r, m - 1)];
        pos[i] = r < m ? k0 + r : -1;
        const double* __restrict__ ar = A + (int64_t)row[i] * n + k0;
#pragma unroll
        for (int c = 0; c < 16; ++c) a[i][c] = ar[min(c, w - 1)];
      }
#pragma unroll
      for (int i = 0; i < kPer; ++i)
#pragma unroll
        for (int c = 4; c < 16; ++c) a[i][c] = c < w ? a[i][c] : 0.0;  // w is a multiple of 4
      lu_panel<kPer>(a, pos, k0, S, kLd);
      int pivots = 0;
#pragma unroll
      for (int i = 0; i < kPer; ++i) {
        const int r = lane + 64 * i, t = pos[i] - k0;
        bool good = false;
        if (r < m) {
          perm[pos[i]] = row[i];
#pragma unroll
          for (int c = 0; c < 16; ++c) P[c * kLd + t] = S[c * kLd + r];
          if (t < w) {
            const double d = S[t * kLd + r];
            good = d != 0.0 && isfinite(d);
            id[pos[i]] = 1.0 / d;
          }
        }
        pivots += __popcll(__ballot(good));
      }
      if (pivots != w && lane == 0) {
        bad = 1;
        status[it.layer] = -5;
      }
    }
    __syncthreads();
    if (bad) return;
    for (int t = tid; t < m * 16; t += NT)
      if (t % 16 < w) A[(int64_t)perm[k0 + t / 16] * n + k0 + t % 16] = P[(t % 16) * kLd + t / 16];
    const int r0 = k0 + 16;
    if (r0 >= n) break;
    if (tid < 256) {  // strictly lower part of L11, zeros elsewhere
      const int s = tid / 16, r = tid % 16;
      sL[s * 17 + r] = r > s ? P[s * kLd + r] : 0.0;
    }
    __syncthreads();
    const int nrest = n - r0;
    for (int cb = wv; cb * 16 < nrest; cb += nw) {
      const int col = r0 + cb * 16 + lr, colc = min(col, n - 1);
      const bool live = col < n;
      double x[4];
#pragma unroll
      for (int t = 0; t < 4; ++t) x[t] = A[(int64_t)perm[k0 + 4 * t + kq] * n + colc];
      double nx[4];  // the next tile of A22
      auto load = [&](int rb) {
#pragma unroll
        for (int v = 0; v < 4; ++v) nx[v] = A[(int64_t)perm[min(r0 + rb * 16 + kq + 4 * v, n - 1)] * n + colc];
      };
      load(0);
#pragma unroll
      for (int s = 0; s < 15; ++s) {
        const double xs = __shfl(x[s >> 2], ((s & 3) << 4) | lr);
#pragma unroll
        for (int t = s >> 2; t < 4; ++t) x[t] -= sL[s * 17 + 4 * t + kq] * xs;
      }
      if (live)
#pragma unroll
        for (int t = 0; t < 4; ++t) A[(int64_t)perm[k0 + 4 * t + kq] * n + col] = x[t];
      for (int rb = 0; rb * 16 < nrest; ++rb) {
        double4_t acc = {nx[0], nx[1], nx[2], nx[3]};
        load(rb + 1);
        const int pi = min(16 + rb * 16 + lr, m - 1);  // rows past the end are not stored
#pragma unroll
        for (int t = 0; t < 4; ++t)
          acc = __builtin_amdgcn_mfma_f64_16x16x4f64(-P[(4 * t + kq) * kLd + pi], x[t], acc, 0, 0, 0);
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int pos = r0 + rb * 16 + kq + 4 * v;
          if (pos < n && live) A[(int64_t)perm[pos] * n + col] = acc[v];
        }
      }
    }
    __syncthreads();
  }
  // the factor transposed and in its final order, 16 columns at a time through LDS
  __syncthreads();
  for (int j0 = 0; j0 < n; j0 += 16) {
    const int w = min(16, n - j0);
    for (int t = tid; t < n * 16; t += NT) S[(t % 16) * kLd + t / 16] = A[(int64_t)perm[t / 16] * n + min(j0 + t % 16, n - 1)];
    __syncthreads();
    for (int j = wv; j < w; j += nw)
      for (int c = lane; c < n; c += 64) AT[(int64_t)(j0 + j) * n + c] = S[j * kLd + c];
    __syncthreads();
  }
  for (int i = tid; i < n; i += NT) pm[i] = perm[i];
}

template __global__ void k_lu_reg<4>(const Item*, double*, int32_t*, LuBufs, int);
template __global__ void k_lu_reg<8>(const Item*, double*, int32_t*, LuBufs, int);
template __global__ void k_lu_reg<12>(const Item*, double*, int32_t*, LuBufs, int);

}  // namespace vbrdf
