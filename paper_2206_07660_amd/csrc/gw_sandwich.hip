// Products of three small matrices per auxiliary function Q, in fp64 MFMA:
//
//  * sand_prod_k   Y(t, k, Q) = L(t, k) V(k, Q) R(t, k)          (stored)
//  * sand_sum_k    O(t, k) += alpha sum_Q op(A_Q) G(t, k) op(B_Q) (reduced)
//
// with nao x nao matrices.  They carry the producers of the polarization and
// the last contraction of the self-energy, of the exchange and of their
// adjoints.  Both chain two products without moving data: a 16 x 16 result of
// v_mfma_f64_16x16x4_f64 has row 4 r + lane / 16, column lane % 16 in register
// r, which is the B operand of K-step r of the next product.  The small
// matrices of (t, k) stay in LDS as operand fragments; the matrices of Q
// stream through registers, the next Q in flight during the second product.
// Complex products take three real ones (Gauss): P1 = sum ar br,
// P2 = sum ai bi, P3 = sum (ar + ai)(br + bi), re = P1 - P2, im = P3 - P1 - P2.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "gw_device.h"
#include "gw_kernels.h"

namespace {

constexpr unsigned kOut = 0x80000000u;   // buffer offset past the record count: reads zeros

// Waves of a workgroup: NB column blocks times QW streams of Q.
template <int NB> struct Waves { static constexpr int qw = NB == 1 ? 4 : NB == 4 ? 1 : 2, n = NB * qw; };

struct Frag {
  double r, i, s;   // re, im, re + im
};
template <bool CJ = false> __device__ __forceinline__ Frag frag(double2 v) {
  return Frag{v.x, v.y, CJ ? v.x - v.y : v.x + v.y};
}
// a fragment as stored in LDS, with or without its sum
__device__ __forceinline__ void put_frag(Frag& d, double2 v) { d = frag(v); }
__device__ __forceinline__ void put_frag(double2& d, double2 v) { d = v; }
__device__ __forceinline__ Acc3 acc3_zero() { return Acc3{d4{0, 0, 0, 0}, d4{0, 0, 0, 0}, d4{0, 0, 0, 0}}; }
__device__ __forceinline__ void mma3(const Frag& a, const Frag& b, Acc3& c) {
  c.p1 = __builtin_amdgcn_mfma_f64_16x16x4f64(a.r, b.r, c.p1, 0, 0, 0);
  c.p2 = __builtin_amdgcn_mfma_f64_16x16x4f64(a.i, b.i, c.p2, 0, 0, 0);
  c.p3 = __builtin_amdgcn_mfma_f64_16x16x4f64(a.s, b.s, c.p3, 0, 0, 0);
}
// CJ: one factor was conjugated, its imaginary part entering with its stored
// sign, so that p2 counts with the other sign
template <bool CJ = false> __device__ __forceinline__ Frag acc3_frag(const Acc3& c, int r) {
  const double re = CJ ? c.p1[r] + c.p2[r] : c.p1[r] - c.p2[r];
  const double s = __builtin_fma(CJ ? 2.0 : -2.0, c.p2[r], c.p3[r]);
  return Frag{re, s - re, s};
}

// x + a b
__device__ __forceinline__ double2 cfma(double2 a, double2 b, double2 x) {
  x.x = __builtin_fma(-a.y, b.y, __builtin_fma(a.x, b.x, x.x));
  x.y = __builtin_fma(a.y, b.x, __builtin_fma(a.x, b.y, x.y));
  return x;
}

// Fragments of a small matrix in LDS, zero past nao.  ROWS: lane l of
// fragment (b, s) holds M[16 b + l % 16][4 s + l / 16] (an A operand),
// otherwise M[4 s + l / 16][16 b + l % 16] (a B operand); herm: of M^H.
template <int NB, int KS, bool ROWS, class F>
__device__ __forceinline__ void lds_fragments(F* dst, const double2* M, int n, bool herm, int nthreads) {
  for (int e = threadIdx.x; e < NB * KS * 64; e += nthreads) {
    const int l = e & 63, f = e >> 6, b = f / KS, s = f - b * KS;
    const int x = 16 * b + (l & 15), y = 4 * s + (l >> 4);
    const int r = ROWS ? x : y, c = ROWS ? y : x;
    double2 v{0.0, 0.0};
    if (r < n && c < n) {
      v = M[herm ? c * n + r : r * n + c];
      if (herm) v.y = -v.y;
    }
    put_frag(dst[e], v);
  }
}

// (t, k, Q range) of this workgroup.  The dispatcher deals workgroup ids
// round-robin over the 8 XCDs; each XCD gets a contiguous range of logical
// ids with t fastest, so that the V matrices of a (k, Q range) stay in its L2
// while every t uses them.
struct SandPos {
  int t, k, q0, q1;
};
__device__ __forceinline__ SandPos sand_pos(int nt, int nk, int naux, int qlen) {
  const unsigned w = blockIdx.x, total = gridDim.x;
  const unsigned xcd = w % 8u, slot = w / 8u, per = total / 8u, rem = total % 8u;
  const unsigned id = xcd < rem ? xcd * (per + 1u) + slot : rem * (per + 1u) + (xcd - rem) * per + slot;
  const unsigned chunks = ((unsigned)naux + (unsigned)qlen - 1u) / (unsigned)qlen;
  SandPos p;
  p.t = (int)(id % (unsigned)nt);
  const unsigned r = id / (unsigned)nt;
  p.q0 = (int)(r % chunks) * qlen;
  p.k = (int)(r / chunks);
  p.q1 = min(p.q0 + qlen, naux);
  (void)nk;
  return p;
}

}  // namespace

// Y = L V R.  T = V R, then Y = L T; a wave owns 16 columns of Y.  Bound by
// the MFMAs (nao 26 pads to 32 x 32 x 28) or, at small nao, by the stores.
template <int KS>
__global__ void __launch_bounds__(64 * Waves<(KS + 3) / 4>::n) sand_prod_k(SandProd d) {
  constexpr int NB = (KS + 3) / 4, QW = Waves<NB>::qw, NT = 64 * Waves<NB>::n;
  constexpr bool kWhole = NB <= 2;   // all fragments of the next V_Q fit in registers
  // (without the sums: forming them cost no more than the longer LDS reads here)
  __shared__ double2 ldsL[NB * KS * 64], ldsR[NB * KS * 64];
  const int n = d.nao, n2 = n * n;
  const SandPos p = sand_pos(d.nt, d.nk, d.naux, d.qlen);
  const int kq = d.tab[p.k];
  lds_fragments<NB, KS, true>(ldsL, d.L + p.t * d.tsL + (long long)p.k * n2, n, d.hermL != 0, NT);
  lds_fragments<NB, KS, false>(ldsR, d.R + p.t * d.tsR + (long long)(d.tabR ? kq : p.k) * n2, n, false, NT);
  __syncthreads();
  const int lane = threadIdx.x & 63, r16 = lane & 15, kl = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int jb = wave % NB, qs = wave / NB;
  const double2* V = d.V + p.k * d.svk;
  double2* Y = d.Y + p.t * d.tsY + p.k * d.svk;
  unsigned vo[NB];
#pragma unroll
  for (int b = 0; b < NB; ++b) vo[b] = 16 * b + r16 < n ? (unsigned)(((16 * b + r16) * n + kl) * 16) : kOut;
  double2 f[kWhole ? NB : 1][kWhole ? KS : 1];
  auto ld = [&](__amdgpu_buffer_rsrc_t rs, int b, int s) {
    return buf_load<double2>(rs, 4 * s + kl < n ? vo[b] : kOut, (unsigned)(64 * s));
  };
  auto fetch = [&](int Q) {
    if constexpr (kWhole) {
      const __amdgpu_buffer_rsrc_t rs = buf_rsrc(V + (long long)Q * n2);
#pragma unroll
      for (int s = 0; s < KS; ++s)
#pragma unroll
        for (int b = 0; b < NB; ++b) f[b][s] = ld(rs, b, s);
    }
  };
  int Q = p.q0 + qs;
  if (Q < p.q1) fetch(Q);
  for (; Q < p.q1; Q += QW) {
    Acc3 T[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) T[b] = acc3_zero();
    if constexpr (kWhole) {
#pragma unroll
      for (int s = 0; s < KS; ++s) {
        const Frag br = frag(ldsR[(jb * KS + s) * 64 + lane]);
#pragma unroll
        for (int b = 0; b < NB; ++b) mma3(frag(f[b][s]), br, T[b]);
      }
      fetch(min(Q + QW, p.q1 - 1));   // the next Q, in flight during the second product
      __builtin_amdgcn_sched_barrier(0);
    } else {
      const __amdgpu_buffer_rsrc_t rs = buf_rsrc(V + (long long)Q * n2);
      double2 g[2][NB];
#pragma unroll
      for (int b = 0; b < NB; ++b) g[0][b] = ld(rs, b, 0);
#pragma unroll
      for (int s = 0; s < KS; ++s) {
        if (s + 1 < KS) {
#pragma unroll
          for (int b = 0; b < NB; ++b) g[(s + 1) & 1][b] = ld(rs, b, s + 1);
        }
        __builtin_amdgcn_sched_barrier(0);
        const Frag br = frag(ldsR[(jb * KS + s) * 64 + lane]);
#pragma unroll
        for (int b = 0; b < NB; ++b) mma3(frag(g[s & 1][b]), br, T[b]);
      }
    }
    double2* y = Y + (long long)Q * n2;
    const int col = 16 * jb + r16;
    Frag t[KS];
#pragma unroll
    for (int s = 0; s < KS; ++s) t[s] = acc3_frag(T[s / 4], s % 4);
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      Acc3 o = acc3_zero();
#pragma unroll
      for (int s = 0; s < KS; ++s) {
        mma3(frag(ldsL[(b * KS + s) * 64 + lane]), t[s], o);
        if constexpr (!kWhole) __builtin_amdgcn_sched_barrier(0);
      }
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int row = 16 * b + 4 * r + kl;
        if (row < n && col < n) {
          double2 v{o.p1[r] - o.p2[r], o.p3[r] - o.p1[r] - o.p2[r]};
          double2* z = y + row * n + col;
          if (d.accumulate) {
            v.x += z->x;
            v.y += z->y;
          }
          *z = v;
        }
      }
    }
  }
}

// Y = L V R of matrices of N <= 4 orbitals, a thread per row of a Y_Q on vector
// instructions: a 16 x 16 block of sand_prod_k would hold one such matrix and
// take 0.43 ns of the chip whatever its size.  Bound by the stores of Y (a row
// is contiguous, and the rows of a wave are); L and R of (t, k) are read from
// LDS by all lanes at once.  One q of the polarization at 4x4x4, naux 220, 100
// nodes, 1 / 2 / 3 / 4 orbitals: 626 / 786 / 1066 / 1298 us with sand_prod_k, 109
// / 282 / 608 / 952 with this one; from 5 orbitals on sand_prod_k is the faster.
template <int N>
__global__ void __launch_bounds__(256) sand_small_k(SandProd d, int chunks) {
  __shared__ double2 sL[N * N], sR[N * N];
  const int chunk = blockIdx.x % chunks, r = blockIdx.x / chunks;
  const int k = r % d.nk, t = r / d.nk, kq = d.tab[k];
  constexpr int n2 = N * N;
  if (threadIdx.x < n2) {
    const int i = threadIdx.x / N, j = threadIdx.x % N;
    double2 l = d.L[t * d.tsL + (long long)k * n2 + (d.hermL ? j * N + i : i * N + j)];
    if (d.hermL) l.y = -l.y;
    sL[threadIdx.x] = l;
    sR[threadIdx.x] = d.R[t * d.tsR + (long long)(d.tabR ? kq : k) * n2 + threadIdx.x];
  }
  __syncthreads();
  const int e = chunk * (int)blockDim.x + threadIdx.x;
  if (e >= d.naux * N) return;
  const int Q = e / N, c = e - Q * N;
  const double2* V = d.V + k * d.svk + (long long)Q * n2;
  double2 u[N];
#pragma unroll
  for (int a = 0; a < N; ++a) u[a] = double2{0.0, 0.0};
#pragma unroll
  for (int x = 0; x < N; ++x) {
    const double2 l = sL[c * N + x];
#pragma unroll
    for (int a = 0; a < N; ++a) u[a] = cfma(l, V[x * N + a], u[a]);
  }
  double2* y = d.Y + t * d.tsY + k * d.svk + (long long)Q * n2 + c * N;
#pragma unroll
  for (int b = 0; b < N; ++b) {
    double2 v = d.accumulate ? y[b] : double2{0.0, 0.0};
#pragma unroll
    for (int a = 0; a < N; ++a) v = cfma(u[a], sR[a * N + b], v);
    y[b] = v;
  }
}

// O += alpha sum_Q op(A_Q) G op(B_Q); BH false: A_Q^H G B_Q, true: A_Q G B_Q^H.
// T = G op(B_Q), then the sum over Q of op(A_Q) T stays in the accumulators; a
// wave owns 16 columns of O and one stream of Q, the streams add through LDS
// in a fixed order.  Neither product touches memory, where separate GEMMs
// wrote and read a (t, k, Q) array of nao^2 blocks for the first one.
template <int KS, bool BH, class T>
__global__ void __launch_bounds__(64 * Waves<(KS + 3) / 4>::n) sand_sum_k(SandSum d) {
  constexpr int NB = (KS + 3) / 4, QW = Waves<NB>::qw, NT = 64 * Waves<NB>::n;
  constexpr bool kWhole = NB <= 2;
  constexpr unsigned ES = sizeof(T);
  // fragments of G, then (in their place) the sums of the other Q streams
  constexpr int kFrag = NB * KS * 64 * (int)sizeof(Frag);
  constexpr int kRed = QW > 1 ? (QW - 1) * NB * NB * 4 * 64 * (int)sizeof(double2) : 0;
  __shared__ __attribute__((aligned(16))) char lds_raw[kFrag > kRed ? kFrag : kRed];
  Frag* const ldsG = (Frag*)lds_raw;
  double2* const lds = (double2*)lds_raw;
  const int n = d.nao, n2 = n * n;
  const SandPos p = sand_pos(d.nt, d.nk, d.naux, d.qlen);
  const int kq = d.tab[p.t * d.tstab + p.k];
  lds_fragments<NB, KS, true>(ldsG, d.G + p.t * d.tsG + (long long)(d.tabG ? kq : p.k) * n2, n, d.hermG != 0, NT);
  __syncthreads();
  const int lane = threadIdx.x & 63, r16 = lane & 15, kl = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int jb = wave % NB, qs = wave / NB;
  const T* A = (const T*)d.A + p.t * d.tsA + p.k * d.skA;
  const T* B = (const T*)d.B + p.t * d.tsB + p.k * d.skB;
  // lane offsets of the fragments: rows of the matrix across the lanes (BH)
  // or its columns
  unsigned voA[NB], voB;
#pragma unroll
  for (int b = 0; b < NB; ++b) {
    const int x = 16 * b + r16;
    voA[b] = x < n ? (unsigned)(BH ? x * n + kl : kl * n + x) * ES : kOut;
  }
  {
    const int x = 16 * jb + r16;
    voB = x < n ? (unsigned)(BH ? x * n + kl : kl * n + x) * ES : kOut;
  }
  const unsigned step = (BH ? 4u : 4u * (unsigned)n) * ES;
  auto ld = [&](__amdgpu_buffer_rsrc_t rs, unsigned v, int s) {
    return to_d2(buf_load<T>(rs, 4 * s + kl < n ? v : kOut, step * (unsigned)s));
  };
  // conjugations: B^H takes conj(B) in the first product, A^H conj(A) in the second
  auto fa = [&](double2 v) { return frag<!BH>(v); };
  auto fb = [&](double2 v) { return frag<BH>(v); };
  double2 a[kWhole ? NB : 1][kWhole ? KS : 1], b[kWhole ? KS : 1];
  auto fetchA = [&](int Q) {
    if constexpr (kWhole) {
      const __amdgpu_buffer_rsrc_t rs = buf_rsrc(A + Q * d.sqA);
#pragma unroll
      for (int s = 0; s < KS; ++s)
#pragma unroll
        for (int i = 0; i < NB; ++i) a[i][s] = ld(rs, voA[i], s);
    }
  };
  auto fetchB = [&](int Q) {
    if constexpr (kWhole) {
      const __amdgpu_buffer_rsrc_t rs = buf_rsrc(B + Q * d.sqB);
#pragma unroll
      for (int s = 0; s < KS; ++s) b[s] = ld(rs, voB, s);
    }
  };
  Acc3 o[NB];
#pragma unroll
  for (int i = 0; i < NB; ++i) o[i] = acc3_zero();
  int Q = p.q0 + qs;
  if (Q < p.q1) {
    fetchB(Q);
    fetchA(Q);
  }
  for (; Q < p.q1; Q += QW) {
    Acc3 X[NB];
#pragma unroll
    for (int i = 0; i < NB; ++i) X[i] = acc3_zero();
    const int Qn = min(Q + QW, p.q1 - 1);
    if constexpr (kWhole) {
#pragma unroll
      for (int s = 0; s < KS; ++s) {
        const Frag x = fb(b[s]);
#pragma unroll
        for (int i = 0; i < NB; ++i) mma3(ldsG[(i * KS + s) * 64 + lane], x, X[i]);
      }
      fetchB(Qn);
      __builtin_amdgcn_sched_barrier(0);
    } else {
      const __amdgpu_buffer_rsrc_t rs = buf_rsrc(B + Q * d.sqB);
      double2 g[2];
      g[0] = ld(rs, voB, 0);
#pragma unroll
      for (int s = 0; s < KS; ++s) {
        if (s + 1 < KS) g[(s + 1) & 1] = ld(rs, voB, s + 1);
        __builtin_amdgcn_sched_barrier(0);
        const Frag x = fb(g[s & 1]);
#pragma unroll
        for (int i = 0; i < NB; ++i) mma3(ldsG[(i * KS + s) * 64 + lane], x, X[i]);
      }
    }
    if constexpr (kWhole) {
#pragma unroll
      for (int s = 0; s < KS; ++s) {
        const Frag t = acc3_frag<BH>(X[s / 4], s % 4);
#pragma unroll
        for (int i = 0; i < NB; ++i) mma3(fa(a[i][s]), t, o[i]);
      }
      fetchA(Qn);
      __builtin_amdgcn_sched_barrier(0);
    } else {
      const __amdgpu_buffer_rsrc_t rs = buf_rsrc(A + Q * d.sqA);
      double2 g[2][NB];
#pragma unroll
      for (int i = 0; i < NB; ++i) g[0][i] = ld(rs, voA[i], 0);
#pragma unroll
      for (int s = 0; s < KS; ++s) {
        if (s + 1 < KS) {
#pragma unroll
          for (int i = 0; i < NB; ++i) g[(s + 1) & 1][i] = ld(rs, voA[i], s + 1);
        }
        __builtin_amdgcn_sched_barrier(0);
        const Frag t = acc3_frag<BH>(X[s / 4], s % 4);
#pragma unroll
        for (int i = 0; i < NB; ++i) mma3(fa(g[s & 1][i]), t, o[i]);
      }
    }
  }
  if constexpr (QW > 1) {
    __syncthreads();                  // every wave is past its last use of the fragments
    if (qs > 0) {
      double2* w = lds + ((qs - 1) * NB + jb) * NB * 4 * 64;
#pragma unroll
      for (int i = 0; i < NB; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const Frag v = acc3_frag<!BH>(o[i], r);
          w[(i * 4 + r) * 64 + lane] = double2{v.r, v.i};
        }
    }
    __syncthreads();
    if (qs > 0) return;
  }
  // with Q splits each split writes its sum to part, and sand_fold_k adds them
  double2* O = d.part ? d.part + (((long long)(p.q0 / d.qlen) * d.nt + p.t) * d.nk + p.k) * n2
                      : d.O + p.t * d.tsO + (long long)(d.tabO ? kq : p.k) * n2;
  const bool add = d.accumulate && !d.part;
  const int col = 16 * jb + r16;
#pragma unroll
  for (int i = 0; i < NB; ++i)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const Frag v = acc3_frag<!BH>(o[i], r);
      double re = v.r, im = v.i;
      if constexpr (QW > 1) {
#pragma unroll
        for (int w = 1; w < QW; ++w) {
          const double2 x = lds[(((w - 1) * NB + jb) * NB * 4 + i * 4 + r) * 64 + lane];
          re += x.x;
          im += x.y;
        }
      }
      const int row = 16 * i + 4 * r + kl;
      if (row >= n || col >= n) continue;
      double2* z = O + row * n + col;
      double2 c{0.0, 0.0};
      if (add) c = *z;
      *z = double2{c.x + d.alpha * re, c.y + d.alpha * im};
    }
}

// O[t][k'] (+)= the sum of its Q splits, in their order.  fold_t: one more sum,
// over t (O[k'] from every (split, t)).
__global__ void __launch_bounds__(256) sand_fold_k(SandSum d, int nsplit, int fold_t) {
  const int n2 = d.nao * d.nao;
  const long long per = (long long)d.nk * n2, one = (long long)d.nt * per;
  const long long e = blockIdx.x * 256LL + threadIdx.x;
  if (e >= (fold_t ? per : one)) return;
  const int terms = fold_t ? nsplit * d.nt : nsplit;
  const long long stride = fold_t ? per : one;
  double re = 0.0, im = 0.0;
#pragma unroll 8
  for (int s = 0; s < terms; ++s) {
    const double2 v = d.part[s * stride + e];
    re += v.x;
    im += v.y;
  }
  const int t = (int)(e / per);
  const int r = (int)(e - t * per), k = r / n2;
  double2* z = d.O + t * d.tsO + (long long)(d.tabO ? d.tab[t * d.tstab + k] : k) * n2 + (r - k * n2);
  if (d.accumulate) {
    re += z->x;
    im += z->y;
  }
  *z = double2{re, im};
}

// out[Q] = alpha sum_{k,e} op(V[k][Q][e]) X[k][e'], e' = e or its transpose;
// one workgroup per Q, which reads its blocks of V once.
template <class T>
__global__ void __launch_bounds__(256) vdot_k(const T* V, const double2* X, double2* out, int nk, int naux, int nao,
                                              double alpha, int conj, int transpose) {
  __shared__ double sr[256], si[256];
  const int n2 = nao * nao, tid = threadIdx.x;
  double re = 0.0, im = 0.0;
  for (int k = 0; k < nk; ++k) {
    const T* v = V + ((long long)k * naux + blockIdx.x) * n2;
    const double2* x = X + (long long)k * n2;
    for (int e = tid; e < n2; e += 256) {
      double2 a = to_d2(v[e]);
      if (conj) a.y = -a.y;
      const int r = e / nao;
      const double2 b = x[transpose ? (e - r * nao) * nao + r : e];
      re += a.x * b.x - a.y * b.y;
      im += a.x * b.y + a.y * b.x;
    }
  }
  sr[tid] = re;
  si[tid] = im;
  __syncthreads();
  for (int h = 128; h > 0; h >>= 1) {
    if (tid < h) {
      sr[tid] += sr[tid + h];
      si[tid] += si[tid + h];
    }
    __syncthreads();
  }
  if (tid == 0) out[blockIdx.x] = double2{alpha * sr[0], alpha * si[0]};
}

hipError_t vdot_launch(const void* V, int tv, const double2* X, double2* out, int nk, int naux, int nao, double alpha,
                       bool conj, bool transpose, hipStream_t st) {
  if (nk <= 0 || naux <= 0) return hipSuccess;
  if (tv)
    vdot_k<<<naux, 256, 0, st>>>((const float2*)V, X, out, nk, naux, nao, alpha, conj, transpose);
  else
    vdot_k<<<naux, 256, 0, st>>>((const double2*)V, X, out, nk, naux, nao, alpha, conj, transpose);
  return hipGetLastError();
}

// K-steps of 4 that hold nao, among the compiled counts: exact for nao 5 .. 8,
// 13 .. 16, 21 .. 32 and some larger ones.  Counts between are left out to keep
// the instantiations few (eight for each of five kernels): nao 9 .. 12 run 4
// steps for 3 and 17 .. 20 run 6 for 5, where the polarization of one q (2x2x2,
// nao 12 / 18, 24 nodes) still takes 49 / 142 us against 199 / 444 of the GEMMs
// before.
#define SAND_KS(nao, CALL)             \
  do {                                 \
    const int ks_ = ((nao) + 3) / 4;   \
    if (ks_ <= 2) { CALL(2); }         \
    else if (ks_ <= 4) { CALL(4); }    \
    else if (ks_ <= 6) { CALL(6); }    \
    else if (ks_ == 7) { CALL(7); }    \
    else if (ks_ == 8) { CALL(8); }    \
    else if (ks_ <= 10) { CALL(10); }  \
    else if (ks_ <= 12) { CALL(12); }  \
    else { CALL(15); }                 \
  } while (0)

hipError_t sand_prod_launch(const SandProd& d0, hipStream_t st) {
  if (d0.nt <= 0 || d0.nk <= 0 || d0.naux <= 0) return hipSuccess;
  if (d0.nao < 1 || d0.nao > 60) return hipErrorInvalidValue;
  SandProd d = d0;
  if (d.nao <= 4) {
    const int rows = d.naux * d.nao, nt = std::min(256, (rows + 63) / 64 * 64), chunks = (rows + nt - 1) / nt;
    const long long wgs = (long long)d.nt * d.nk * chunks;
    if (wgs > 0x7fffffffLL) return hipErrorInvalidConfiguration;
    const dim3 grid((unsigned)wgs);
    if (d.nao == 1) sand_small_k<1><<<grid, nt, 0, st>>>(d, chunks);
    else if (d.nao == 2) sand_small_k<2><<<grid, nt, 0, st>>>(d, chunks);
    else if (d.nao == 3) sand_small_k<3><<<grid, nt, 0, st>>>(d, chunks);
    else sand_small_k<4><<<grid, nt, 0, st>>>(d, chunks);
    return hipGetLastError();
  }
  // Q ranges: as long as 2048 workgroups remain (the LDS fill costs about two
  // Q), but not below 8
  const long long base = (long long)d.nt * d.nk;
  long long chunks = std::max(1LL, std::min<long long>((2048 + base - 1) / base, (d.naux + 7) / 8));
  d.qlen = (int)((d.naux + chunks - 1) / chunks);
  chunks = (d.naux + d.qlen - 1) / d.qlen;
  if (base * chunks > 0x7fffffffLL) return hipErrorInvalidConfiguration;
  const dim3 grid((unsigned)(base * chunks));
#define SAND_CALL(KS) sand_prod_k<KS><<<grid, 64 * Waves<(KS + 3) / 4>::n, 0, st>>>(d)
  SAND_KS(d.nao, SAND_CALL);
#undef SAND_CALL
  return hipGetLastError();
}

hipError_t sand_sum_launch(const SandSum& d0, hipStream_t st) {
  if (d0.nt <= 0 || d0.nk <= 0 || d0.naux <= 0) return hipSuccess;
  if (d0.nao < 1 || d0.nao > 60) return hipErrorInvalidValue;
  SandSum d = d0;
  // Q splits where (t, k) leaves the chip idle: up to 1024 workgroups, but at
  // least 8 Q for every wave
  const long long base = (long long)d.nt * d.nk;
  const int streams = d.nao <= 16 ? 4 : d.nao <= 48 ? 2 : 1;
  long long split = std::min<long long>((1024 + base - 1) / base, d.naux / (8 * streams));
  split = std::max(1LL, std::min<long long>(split, d.part_elems / (base * d.nao * d.nao)));
  d.qlen = (int)((d.naux + split - 1) / split);
  split = (d.naux + d.qlen - 1) / d.qlen;
  if (split == 1 && !d.fold_t) d.part = nullptr;
  if (d.fold_t && d.part_elems < base * d.nao * d.nao) return hipErrorInvalidValue;
  if (base * split > 0x7fffffffLL) return hipErrorInvalidConfiguration;
  const dim3 grid((unsigned)(base * split));
#define SAND_CALL(KS)                                                                       \
  do {                                                                                      \
    constexpr int nt_ = 64 * Waves<(KS + 3) / 4>::n;                                        \
    if (d.tv == 0) {                                                                        \
      if (d.bh) sand_sum_k<KS, true, double2><<<grid, nt_, 0, st>>>(d);                     \
      else sand_sum_k<KS, false, double2><<<grid, nt_, 0, st>>>(d);                         \
    } else {                                                                                \
      if (d.bh) sand_sum_k<KS, true, float2><<<grid, nt_, 0, st>>>(d);                      \
      else sand_sum_k<KS, false, float2><<<grid, nt_, 0, st>>>(d);                          \
    }                                                                                       \
  } while (0)
  SAND_KS(d.nao, SAND_CALL);
#undef SAND_CALL
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || !d.part) return e;
  const long long len = (long long)d.nk * d.nao * d.nao * (d.fold_t ? 1 : d.nt);
  sand_fold_k<<<(unsigned)((len + 255) / 256), 256, 0, st>>>(d, (int)split, d.fold_t);
  return hipGetLastError();
}
