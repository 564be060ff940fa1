// Panel and triangular kernels of the blocked LU solve of (I - P0) X = P0, one
// workgroup per matrix, panels of 32 columns.
//
// A panel is a serial chain of 32 pivot searches and rank-1 updates, so it is
// latency that counts.  Each thread keeps one row of the panel in registers
// and rows stay where they are until the end (a thread tracks its row's
// position); a column costs one barrier: before it every wave leaves its best
// candidate row in LDS, after it all threads pick the winner and update.  The
// row interchanges then go into the triangular solve, where a thread owns a
// column of U12 or of the right-hand side and keeps its 32 entries in
// registers, so that the other columns are read and written once.
// Before, panel steps and triangular rows each went through global memory with
// a barrier per level of the search: for 404 matrices of order 250 (ms, all
// panels) 1.53 + 2.36 and 1.27 (back substitution) against 0.99 and 0.25; two
// panels per trailing update save 0.9 ms of its 2.8.
#include <hip/hip_runtime.h>

#include "gw_device.h"
#include "gw_kernels.h"

namespace {

constexpr int kNb = 32;
constexpr int kWaveOrder = 48;

// x - a b
__device__ __forceinline__ double2 cfnma(double2 a, double2 b, double2 x) {
  x.x = __builtin_fma(a.y, b.y, __builtin_fma(-a.x, b.x, x.x));
  x.y = __builtin_fma(-a.y, b.x, __builtin_fma(-a.x, b.y, x.y));
  return x;
}
__device__ __forceinline__ double2 cinv(double2 a) {
  const double den = a.x * a.x + a.y * a.y;
  return den > 0.0 ? double2{a.x / den, -a.y / den} : double2{0.0, 0.0};
}
__device__ __forceinline__ unsigned wave_max(unsigned x) {
  x = dpp_max<0xB1>(x);                      // lane ^ 1
  x = dpp_max<0x4E>(x);                      // lane ^ 2
  x = dpp_max<0x141>(x);                     // mirror within 8 lanes
  x = dpp_max<0x140>(x);                     // mirror within 16 lanes
  x = max(x, (unsigned)__builtin_amdgcn_ds_swizzle((int)x, 0x401F));   // lane ^ 16
  return max((unsigned)__builtin_amdgcn_readlane((int)x, 0), (unsigned)__builtin_amdgcn_readlane((int)x, 32));
}

}  // namespace

// Factors columns j0 .. j0+31 of A (rows j0 .. n-1, at most NT of them), then
// applies the interchanges and L11^{-1} to the columns right of the panel and
// to all columns of B.  second: the panel before (columns j0-32 ..) has not
// been applied to those columns yet, only to this panel; its part enters here,
// row by row of its U12, and its L rows take part in the interchanges, so that
// one update of 64 columns follows both panels.  The pivot is the largest remaining |re| + |im| of the
// column to 2^-10, the uppermost row among equals.
template <int NT, bool second>
__global__ void __launch_bounds__(NT) wlu_factor_k(double2* A, double2* B, const int* sel, int n, int j0, int* flag) {
  constexpr int NW = NT / 64;
  __shared__ double2 cand[2][NW][kNb];
  __shared__ unsigned keys[2][NW];
  __shared__ double2 L[kNb][kNb + 1], Lp[second ? kNb : 1][kNb + 1];
  __shared__ int src[kNb], dpos[kNb], dsrc[kNb], nd_s;
  const size_t nn = (size_t)n * n;
  double2* Am = A + blockIdx.x * nn;
  double2* Bm = B + (size_t)(sel ? sel[blockIdx.x] : blockIdx.x) * nn;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int m = n - j0, w = min(kNb, m);
  if (tid == 0) nd_s = 0;
  for (int e = tid; e < kNb * (kNb + 1); e += NT) L[0][e] = double2{0.0, 0.0};   // rows past a short panel
  double2 x[kNb];
  bool open = tid < m;
  int pos = tid;
  {
    const double2* p = Am + (size_t)(j0 + (open ? tid : 0)) * n + j0;
#pragma unroll
    for (int c = 0; c < kNb; ++c) x[c] = c < w ? p[c] : double2{0.0, 0.0};
  }
#pragma unroll
  for (int j = 0; j < kNb; ++j)
    if (j < w) {
      const int b = j & 1;
      const double v = fabs(x[j].x) + fabs(x[j].y);
      const unsigned hi = (unsigned)(__builtin_bit_cast(unsigned long long, v) >> 32);
      const unsigned key = open ? (hi & ~1023u) | (unsigned)(1023 - pos) : 0u;
      const unsigned top = wave_max(key);
      if (open && key == top) {
#pragma unroll
        for (int c = j; c < kNb; ++c) cand[b][wave][c] = x[c];
      }
      if (lane == 0) keys[b][wave] = top;
      __syncthreads();
      unsigned best = keys[b][0];
      int from = 0;
#pragma unroll
      for (int i = 1; i < NW; ++i) {
        const unsigned k = keys[b][i];
        if (k > best) {
          best = k;
          from = i;
        }
      }
      from = __builtin_amdgcn_readfirstlane(from);
      const int p = 1023 - (int)(best & 1023u);
      const double2* u = cand[b][from];
      const double2 piv = u[j];
      if (tid == 0 && !(fabs(piv.x) + fabs(piv.y) > 0.0)) atomicOr(flag, 1);
      const double2 pinv = cinv(piv);
      if (pos == p && open) {
        open = false;
        pos = j;
      } else if (pos == j) {
        pos = p;
      }
      if (open) {
        const double2 f = cmul(x[j], pinv);
        x[j] = f;
#pragma unroll
        for (int c = j + 1; c < kNb; ++c) x[c] = cfnma(f, u[c], x[c]);
      }
    }
  __syncthreads();
  if (tid < m) {
    double2* p = Am + (size_t)(j0 + pos) * n + j0;
#pragma unroll
    for (int c = 0; c < kNb; ++c)
      if (c < w) p[c] = x[c];
    if (pos < w) {
      src[pos] = tid;
#pragma unroll
      for (int c = 0; c < kNb; ++c) L[pos][c] = x[c];
    } else if (tid < w) {
      // a row pushed out of the panel's block
      const int i = atomicAdd(&nd_s, 1);
      dpos[i] = pos;
      dsrc[i] = tid;
    }
  }
  __syncthreads();
  const int nd = nd_s, right = n - j0 - w, left = second ? kNb : 0;
  if constexpr (second) {
    // L of the panel before in this panel's rows, in their final order
    for (int e = tid; e < kNb * kNb; e += NT) {
      const int i = e / kNb, t = e - i * kNb;
      Lp[i][t] = i < w ? Am[(size_t)(j0 + src[i]) * n + j0 - kNb + t] : double2{0.0, 0.0};
    }
    __syncthreads();
  }
  for (int e = tid; e < left + right + n; e += NT) {
    const int er = e - left;
    double2* M = (er < 0 ? Am + (j0 + er) : er < right ? Am + (j0 + w + er) : Bm + (er - right)) + (size_t)j0 * n;
#pragma unroll
    for (int i = 0; i < kNb; ++i) x[i] = i < w ? M[(size_t)src[i] * n] : double2{0.0, 0.0};
    for (int d = 0; d < nd; d += 8) {
      double2 z[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) z[i] = M[(size_t)dsrc[min(d + i, nd - 1)] * n];
#pragma unroll
      for (int i = 0; i < 8; ++i)
        if (d + i < nd) M[(size_t)dpos[d + i] * n] = z[i];
    }
    if (second && er >= 0) {
      const double2* u = M - (size_t)kNb * n;
      double2 y[4];
#pragma unroll
      for (int t = 0; t < 4; ++t) y[t] = u[(size_t)t * n];
#pragma unroll
      for (int t = 0; t < kNb; ++t) {
        const double2 yt = y[t % 4];
        if (t + 4 < kNb) y[t % 4] = u[(size_t)(t + 4) * n];
#pragma unroll
        for (int i = 0; i < kNb; ++i) {
          if constexpr (second) x[i] = cfnma(Lp[i][t], yt, x[i]);
          if (i % 8 == 7) __builtin_amdgcn_sched_barrier(0);   // eight entries of L in flight
        }
      }
    }
    const int ws = second && er < 0 ? 0 : w;   // the panel before is only interchanged
#pragma unroll
    for (int t = 0; t < kNb - 1; ++t)
      if (t + 1 < ws) {
#pragma unroll
        for (int i = t + 1; i < kNb; ++i) x[i] = cfnma(L[i][t], x[t], x[i]);
        __builtin_amdgcn_sched_barrier(0);   // L is read as it is used, not ahead into registers
      }
#pragma unroll
    for (int i = 0; i < kNb; ++i)
      if (i < w) M[(size_t)i * n] = x[i];
  }
}

// Rows j0 .. j0+31 of B <- U11^{-1} B: a thread per column, its 32 entries in
// registers, U11 and the inverses of its diagonal in LDS.
template <int NT>
__global__ void __launch_bounds__(NT) wlu_back_k(const double2* A, double2* B, const int* sel, int n, int j0) {
  __shared__ double2 U[kNb][kNb + 1];
  const size_t nn = (size_t)n * n;
  const double2* Am = A + blockIdx.x * nn + (size_t)j0 * n + j0;
  double2* Bm = B + (size_t)(sel ? sel[blockIdx.x] : blockIdx.x) * nn + (size_t)j0 * n;
  const int w = min(kNb, n - j0);
  for (int e = threadIdx.x; e < kNb * kNb; e += NT) {
    const int r = e / kNb, c = e % kNb;
    if (r < w && c < w && r <= c) {
      const double2 v = Am[(size_t)r * n + c];
      U[r][c] = r == c ? cinv(v) : v;
    }
  }
  __syncthreads();
  for (int c = threadIdx.x + NT * blockIdx.y; c < n; c += NT * gridDim.y) {
    double2 y[kNb];
#pragma unroll
    for (int i = 0; i < kNb; ++i) y[i] = i < w ? Bm[(size_t)i * n + c] : double2{0.0, 0.0};
#pragma unroll
    for (int t = kNb - 1; t >= 0; --t)
      if (t < w) {
        y[t] = cmul(y[t], U[t][t]);
#pragma unroll
        for (int i = 0; i < t; ++i) y[i] = cfnma(U[i][t], y[t], y[i]);
        __builtin_amdgcn_sched_barrier(0);   // U is read as it is used, not ahead into registers
      }
#pragma unroll
    for (int i = 0; i < kNb; ++i)
      if (i < w) Bm[(size_t)i * n + c] = y[i];
  }
}

hipError_t wlu_factor_launch(double2* A, double2* B, const int* sel, int n, int j0, bool second, long long nmat,
                             int* flag, hipStream_t st) {
  if (nmat <= 0) return hipSuccess;
  if (n - j0 > 512) return hipErrorInvalidValue;
  const unsigned g = (unsigned)nmat;
  // a small matrix within a wave: no barrier to wait at, and four times as many
  // matrices at once (2624 of order 16: 180 us a solve with 256 threads, 130 with
  // 64; from order 56 on 41 matrices take 5% longer)
  if (n <= kWaveOrder) {
    if (second) wlu_factor_k<64, true><<<g, 64, 0, st>>>(A, B, sel, n, j0, flag);
    else wlu_factor_k<64, false><<<g, 64, 0, st>>>(A, B, sel, n, j0, flag);
  } else if (n - j0 <= 256) {
    if (second) wlu_factor_k<256, true><<<g, 256, 0, st>>>(A, B, sel, n, j0, flag);
    else wlu_factor_k<256, false><<<g, 256, 0, st>>>(A, B, sel, n, j0, flag);
  } else {
    if (second) wlu_factor_k<512, true><<<g, 512, 0, st>>>(A, B, sel, n, j0, flag);
    else wlu_factor_k<512, false><<<g, 512, 0, st>>>(A, B, sel, n, j0, flag);
  }
  return hipGetLastError();
}

hipError_t wlu_back_launch(const double2* A, double2* B, const int* sel, int n, int j0, long long nmat, hipStream_t st) {
  if (nmat <= 0) return hipSuccess;
  if (n <= kWaveOrder) {
    wlu_back_k<64><<<(unsigned)nmat, 64, 0, st>>>(A, B, sel, n, j0);
  } else {
    const dim3 grid((unsigned)nmat, (unsigned)((n + 255) / 256));
    wlu_back_k<256><<<grid, 256, 0, st>>>(A, B, sel, n, j0);
  }
  return hipGetLastError();
}
