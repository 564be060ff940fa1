// Dyson equation for nao <= 32: one wave inverts one matrix
// M = (i w_n + mu) S - H0 - Sig_inf - Sig_iw in registers.
//
// The wave inverts M^T, so that consecutive lanes read consecutive elements.
// Lane l holds row l % R and the columns l / R + CG i (R = 8, 16 or 32 rows,
// CG = 64 / R column groups), so a step of the in-place Gauss-Jordan
// elimination is the broadcast of one column across the groups (a lane
// permutation), of the pivot row through a wave-private strip of LDS, and one
// complex multiply-add per held entry.  Rows stay where they are: the pivot of
// step j is the largest remaining entry of column j (to 2^-14), found with
// lane permutations, and the two permutations are undone when the inverse is
// written or traced.  No barrier and no workgroup-wide search: the workgroup
// version (dyson_k, larger nao) spends its time in those: 336 us for 6400
// matrices of nao 26 against 114 us, of which the LDS broadcasts take about half.
#include <hip/hip_runtime.h>

#include "gw_device.h"
#include "gw_kernels.h"

namespace {

__device__ __forceinline__ double readlane_d(double x, int l) {
  const unsigned long long u = __builtin_bit_cast(unsigned long long, x);
  const unsigned lo = __builtin_amdgcn_readlane((unsigned)u, l), hi = __builtin_amdgcn_readlane((unsigned)(u >> 32), l);
  return __builtin_bit_cast(double, (unsigned long long)hi << 32 | lo);
}
// largest x over each aligned group of R lanes
template <int R> __device__ __forceinline__ unsigned group_max(unsigned x) {
  x = dpp_max<0xB1>(x);                      // quad_perm: lane ^ 1
  x = dpp_max<0x4E>(x);                      // quad_perm: lane ^ 2
  x = dpp_max<0x141>(x);                     // mirror within 8 lanes
  if constexpr (R >= 16) x = dpp_max<0x140>(x);   // mirror within 16 lanes
  if constexpr (R >= 32) x = max(x, (unsigned)__builtin_amdgcn_ds_swizzle((int)x, 0x401F));   // lane ^ 16
  return x;
}

}  // namespace

template <int R, int NC>
__global__ void __launch_bounds__(256) dyson_reg_k(DysonArgs a, int nw, int total) {
  constexpr int CG = 64 / R;
  __shared__ double2 strip[4][CG * NC];
  __shared__ int perm_s[4][R];
  __shared__ double dens_s[4][R];
  const int lane = threadIdx.x & 63, r = lane % R, cg = lane / R;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int mat = blockIdx.x * 4 + wave;
  if (mat >= total) return;                  // whole waves; no barrier below
  const int k = mat % a.nk, iw = mat / a.nk % nw, im = mat / a.nk / nw;
  const int n = a.nao;
  const size_t nn = (size_t)n * n;
  const double w = a.wF[iw], mu = im == 0 ? a.mu : a.more[im - 1];
  double2* row = strip[wave];
  int* perm = perm_s[wave];
  double* dens = dens_s[wave];
  double2 m[NC];
#pragma unroll
  for (int i = 0; i < NC; ++i) {
    const int c = cg + CG * i;
    m[i] = double2{0.0, 0.0};
    if (r < n && c < n) {
      const size_t e = (size_t)k * nn + (size_t)(c * n + r);
      const double2 s = a.S[e], h = a.H0[e];
      m[i].x = mu * s.x - w * s.y - h.x;
      m[i].y = mu * s.y + w * s.x - h.y;
      if (a.Sinf) {
        const double2 q = a.Sinf[e];
        m[i].x -= q.x;
        m[i].y -= q.y;
      }
      if (a.Siw) {
        const double2 q = a.Siw[(size_t)iw * a.nk * nn + e];
        m[i].x -= q.x;
        m[i].y -= q.y;
      }
    }
  }
  bool open = r < n, bad = false, zero = false;   // open: the row has not been a pivot
  int mycol = 0;                             // the step whose pivot this row was
#pragma unroll
  for (int i = 0; i < NC; ++i)
    for (int g = 0; g < CG; ++g) {
      const int j = g + CG * i;
      if (j >= n) break;
      // column j in every group
      const int src = r + R * g;
      const double2 f{__shfl(m[i].x, src, 64), __shfl(m[i].y, src, 64)};
      const double v = fabs(f.x) + fabs(f.y);
      const unsigned hi = (unsigned)(__builtin_bit_cast(unsigned long long, v) >> 32);
      const unsigned key = open ? (hi & ~63u) | (unsigned)(63 - r) : 0u;
      const int p = 63 - (int)(__builtin_amdgcn_readfirstlane(group_max<R>(key)) & 63u);
      const double2 fp{readlane_d(f.x, p), readlane_d(f.y, p)};
      const double fa = fabs(fp.x) + fabs(fp.y);
      if (!(fa > 0.0)) bad = true;
      if (fa == 0.0) zero = true;
      const double den = fp.x * fp.x + fp.y * fp.y;
      const double inv = den > 0.0 ? 1.0 / den : 0.0;
      const double2 pinv{fp.x * inv, -fp.y * inv};
      const bool piv = r == p;
      if (piv) {
        open = false;
        mycol = j;
#pragma unroll
        for (int c = 0; c < NC; ++c) {
          row[cg + CG * c] = m[c];
          m[c] = double2{0.0, 0.0};
        }
      }
      if (lane == 0) {
        perm[j] = p;
        dens[j] = den;
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
      // pivot row: row pinv; other rows: m - f pinv row; column j: the factor
      const double2 t = cmul(f, pinv);
      const double2 q = piv ? pinv : double2{-t.x, -t.y};
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        const double2 u = row[cg + CG * c];
        m[c].x = __builtin_fma(-q.y, u.y, __builtin_fma(q.x, u.x, m[c].x));
        m[c].y = __builtin_fma(q.y, u.x, __builtin_fma(q.x, u.y, m[c].y));
      }
      if (cg == g) m[i] = q;
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
    }
  // a count's zero pivot makes the count infinite: those of a launch may have
  // been asked for in vain
  if (bad && lane == 0 && !a.part) atomicOr(a.flag, 1);
  // row r holds row mycol of the transposed inverse, its entry c the column perm[c]
  if (a.logdet) {
    double l = lane < n ? 0.5 * log(dens[lane]) : 0.0;
    for (int o = 32; o > 0; o >>= 1) l += __shfl_xor(l, o, 64);
    if (lane == 0) a.logdet[(size_t)iw * a.nk + k] = l;
  }
  const bool have = r < n;
  double tr = 0.0, ti = 0.0;
#pragma unroll
  for (int i = 0; i < NC; ++i) {
    const int c = cg + CG * i;
    if (!have || c >= n) continue;
    const int pc = perm[c];
    if (a.G) a.G[((size_t)iw * a.nk + k) * nn + (size_t)(pc * n + mycol)] = m[i];
    if (a.part) {                            // tr[G S]
      const double2 s = a.S[(size_t)k * nn + (size_t)(mycol * n + pc)];
      tr += m[i].x * s.x - m[i].y * s.y;
      ti += m[i].x * s.y + m[i].y * s.x;
    }
  }
  if (a.part) {
    for (int o = 32; o > 0; o >>= 1) {
      tr += __shfl_xor(tr, o, 64);
      ti += __shfl_xor(ti, o, 64);
    }
    if (lane == 0) {
      const double2 rr = a.rrow[iw];
      a.part[mat] = rr.x * tr - rr.y * ti + (zero ? (double)INFINITY : 0.0);
    }
  }
}

// nmu matrices sets: mu = a.mu, a.more[0], ...; part[(im * nw + n) * nk + k]
hipError_t dyson_reg_launch(const DysonArgs& a, int nw, int nmu, hipStream_t st) {
  const long long total = (long long)nmu * nw * a.nk;
  if (total > 0x7fffffffLL) return hipErrorInvalidConfiguration;
  const dim3 grid((unsigned)((total + 3) / 4));
  const int n = a.nao;
#define DYSON_CALL(R, NC) dyson_reg_k<R, NC><<<grid, 256, 0, st>>>(a, nw, (int)total)
  if (n <= 8) DYSON_CALL(8, 1);
  else if (n <= 12) DYSON_CALL(16, 3);
  else if (n <= 16) DYSON_CALL(16, 4);
  else if (n <= 20) DYSON_CALL(32, 10);
  else if (n <= 26) DYSON_CALL(32, 13);
  else DYSON_CALL(32, 16);
#undef DYSON_CALL
  return hipGetLastError();
}

// out[b] = scale * sum of x[b n .. b n + n) in a fixed order
__global__ void __launch_bounds__(1024) sum_rows_k(const double* x, int n, double scale, double* out) {
  __shared__ double s[1024];
  x += (size_t)blockIdx.x * n;
  double acc = 0.0;
  for (int i = threadIdx.x; i < n; i += 1024) acc += x[i];
  s[threadIdx.x] = acc;
  __syncthreads();
  for (int h = 512; h > 0; h >>= 1) {
    if ((int)threadIdx.x < h) s[threadIdx.x] += s[threadIdx.x + h];
    __syncthreads();
  }
  if (threadIdx.x == 0) out[blockIdx.x] = scale * s[0];
}

hipError_t sum_rows_launch(const double* x, int n, int rows, double scale, double* out, hipStream_t st) {
  sum_rows_k<<<rows, 1024, 0, st>>>(x, n, scale, out);
  return hipGetLastError();
}
