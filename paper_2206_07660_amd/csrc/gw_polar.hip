// The long contraction of the polarization in fp64:
//   P(t)[Q][Q'] = alpha sum_{k,e} Y(t)[k][Q][e] conj(V[k][Q'][e])
// for a range of tau nodes t that share V, optionally only on and above the
// diagonal (Hermitian P).  pol_acc_k forms 16 x 16 blocks over a part of the K
// sum, pol_fin_k adds the parts and writes P, its mirror image and the
// transposed matrix of -q.
//
// The MFMAs bound it, so the split aims at executing few of them: three real
// products per complex one (Gauss), and the output cut into 16 x 16 blocks
// dealt to the waves up to 7 each (3 accumulator sets of 7 blocks are 168
// VGPRs: two waves per SIMD), so that a triangle wastes only the lower halves
// of its diagonal blocks (64 x 64 tiles of naux 150 execute 2.2 times the
// triangle, the blocks 1.24 times).  The rows of Y and V that a workgroup's
// blocks need go through two LDS stages of 4 k as operand fragments (lane
// order, no bank conflicts): each is read from L2 once per workgroup, and the
// loads of the next stage have a whole stage of MFMAs (7 x 3 x 64 cycles times
// two waves per SIMD) to arrive.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "gw_device.h"
#include "gw_kernels.h"

namespace {

constexpr int kMaxBlk = 7;      // blocks of a wave
constexpr int kPartBlk = 28;    // blocks of a workgroup (4 waves)
constexpr int kSuper = 16;      // largest side of a superblock

// A part: up to kPartBlk consecutive blocks (row by row) of one superblock pair.
struct Part {
  int r0, c0, rows, cols;   // superblock pair: first block row / column, sizes
  int b0, cnt;              // first block inside it, number of blocks
  int g0;                   // number of the first block in the whole matrix
  bool diag;                // triangular superblock
};

__host__ __device__ inline int pair_blocks(int rows, int cols, bool diag) {
  return diag ? rows * (rows + 1) / 2 : rows * cols;
}

// Walks the superblock pairs of nb x nb blocks cut into ns superblocks per side.
template <class F> __host__ __device__ inline void each_pair(int nb, int ns, bool tri, F f) {
  for (int I = 0; I < ns; ++I)
    for (int J = tri ? I : 0; J < ns; ++J) {
      const int r0 = I * nb / ns, r1 = (I + 1) * nb / ns, c0 = J * nb / ns, c1 = (J + 1) * nb / ns;
      if (f(r0, c0, r1 - r0, c1 - c0, tri && I == J)) return;
    }
}

__device__ inline Part find_part(int nb, int ns, bool tri, int part, int per) {
  Part p{};
  int left = part, g = 0;
  each_pair(nb, ns, tri, [&](int r0, int c0, int rows, int cols, bool diag) {
    const int n = pair_blocks(rows, cols, diag), np = (n + per - 1) / per;
    if (left < np) {
      const int len = (n + np - 1) / np;   // parts of equal length
      p = Part{r0, c0, rows, cols, left * len, min(len, n - left * len), g + left * len, diag};
      return true;
    }
    left -= np;
    g += n;
    return false;
  });
  return p;
}

// Row and column, inside the superblock pair, of its block b.
__host__ __device__ inline void block_rc(int cols, bool diag, int b, int& r, int& c) {
  if (diag) {
    r = 0;
    int len = cols;
    while (b >= len) {
      b -= len;
      ++r;
      --len;
    }
    c = r + b;
  } else {
    r = b / cols;
    c = b - r * cols;
  }
}

struct Acc3 {
  d4 p1, p2, p3;
};

}  // namespace

// W waves, each loading L fragments per stage; a workgroup's blocks touch at
// most W * L fragment rows (checked by the launcher).
template <int W, int L>
__global__ void __launch_bounds__(64 * W) pol_acc_k(PolAcc d) {
  __shared__ double2 lds[2][W * L * 64];
  const int lane = threadIdx.x & 63, r16 = lane & 15, kl = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // contiguous logical ids per XCD (ids are dealt round-robin over the 8):
  // the parts of one (K part, t) meet in an L2, then the next t of the K part
  const unsigned w = blockIdx.x, total = gridDim.x;
  const unsigned xcd = w % 8u, slot = w / 8u, per = total / 8u, rem = total % 8u;
  const unsigned id = xcd < rem ? xcd * (per + 1u) + slot : rem * (per + 1u) + (xcd - rem) * per + slot;
  const int part = (int)(id % (unsigned)d.nparts);
  const unsigned r = id / (unsigned)d.nparts;
  const int t = (int)(r % (unsigned)d.nt), sp = (int)(r / (unsigned)d.nt);
  const Part p = find_part(d.nb, d.ns, d.tri != 0, part, d.per);

  // fragment rows of the part: block rows ra.. and block columns ca..
  int ra, ca, rz, cz, rt, ct;
  block_rc(p.cols, p.diag, p.b0, ra, ca);
  block_rc(p.cols, p.diag, p.b0 + p.cnt - 1, rz, cz);
  const int na = rz - ra + 1;
  if (na > 1) {
    ca = p.diag ? min(ca, ra + 1) : 0;
    cz = p.cols - 1;
  }
  const int nf = na + cz - ca + 1;

  const int nsteps_all = (d.K + 3) / 4;
  const int s0 = sp * d.steps, s1 = min(s0 + d.steps, nsteps_all);
  // this lane's fragment elements: row pointers and the running K offset
  const double2* src[L];
  bool has[L];
#pragma unroll
  for (int l = 0; l < L; ++l) {
    const int f = wave + W * l;
    has[l] = f < nf;
    const bool y = f < na;
    const int row = 16 * (y ? p.r0 + ra + f : p.c0 + ca + (f - na)) + r16;
    src[l] = (y ? d.Y + t * d.tsY : d.V) + (long long)min(row, d.naux - 1) * d.n2;
  }
  int e = 0;
  long long koff = 0;
  int kk = 4 * s0 + kl;             // k of the next stage to load
  {
    const int k = kk / d.n2;
    e = kk - k * d.n2;
    koff = (long long)k * d.sv + e;
  }
  double2 f[L];
  bool ok = true;
  auto fetch = [&]() {
    // lanes past K read k = 0 of their row and store zeros
    ok = kk < d.K;
    const long long o = ok ? koff : 0;
#pragma unroll
    for (int l = 0; l < L; ++l)
      if (has[l]) f[l] = src[l][o];
    kk += 4;
    e += 4;
    koff += 4;
    if (e >= d.n2) {                // n2 >= 4: one carry
      e -= d.n2;
      koff += d.sv - d.n2;
    }
  };
  auto stash = [&](int stage) {
#pragma unroll
    for (int l = 0; l < L; ++l)
      if (has[l]) lds[stage][(wave + W * l) * 64 + lane] = ok ? f[l] : double2{0.0, 0.0};
  };

  // this wave's blocks
  const int m = (p.cnt + W - 1) / W;
  const int mine = min(m, p.cnt - wave * m);   // may be <= 0
  int fa[kMaxBlk], fb[kMaxBlk];
#pragma unroll
  for (int b = 0; b < kMaxBlk; ++b) {
    block_rc(p.cols, p.diag, p.b0 + min(wave * m + b, p.cnt - 1), rt, ct);
    fa[b] = (rt - ra) * 64 + lane;
    fb[b] = (na + ct - ca) * 64 + lane;
  }
  Acc3 o[kMaxBlk];
#pragma unroll
  for (int b = 0; b < kMaxBlk; ++b) o[b].p1 = o[b].p2 = o[b].p3 = d4{0, 0, 0, 0};

  if (s0 < s1) {
    fetch();
    stash(0);
    __syncthreads();
    for (int s = s0; s < s1; ++s) {
      const int st = (s - s0) & 1;
      if (s + 1 < s1) fetch();
      __builtin_amdgcn_sched_barrier(0);   // the loads first, then the MFMAs they hide behind
#pragma unroll
      for (int b = 0; b < kMaxBlk; ++b)
        if (b < mine) {
          const double2 x = lds[st][fa[b]], v = lds[st][fb[b]];
          o[b].p1 = __builtin_amdgcn_mfma_f64_16x16x4f64(x.x, v.x, o[b].p1, 0, 0, 0);
          o[b].p2 = __builtin_amdgcn_mfma_f64_16x16x4f64(x.y, -v.y, o[b].p2, 0, 0, 0);
          o[b].p3 = __builtin_amdgcn_mfma_f64_16x16x4f64(x.x + x.y, v.x - v.y, o[b].p3, 0, 0, 0);
        }
      if (s + 1 < s1) stash(st ^ 1);
      __syncthreads();
    }
  }
  double2* out = d.part + (((long long)sp * d.nt + t) * d.nblk + p.g0 + wave * m) * 256 + lane;
#pragma unroll
  for (int b = 0; b < kMaxBlk; ++b)
    if (b < mine) {
#pragma unroll
      for (int q = 0; q < 4; ++q)
        out[b * 256 + q * 64] = double2{o[b].p1[q] - o[b].p2[q], o[b].p3[q] - o[b].p1[q] - o[b].p2[q]};
    }
}

// One workgroup per block and node: adds the K parts in their order, scales,
// and writes the block of P (of an accumulated P: adds to it), with tri its
// conjugate mirror image, and with M the transposed matrix of the node.
// Bound by HBM; both orientations are written along rows through LDS.
__global__ void __launch_bounds__(256) pol_fin_k(PolAcc d) {
  __shared__ double2 s[16][17];
  const int tid = threadIdx.x, g = blockIdx.x, t = blockIdx.y;
  int bi = 0, bj = 0, left = g;
  each_pair(d.nb, d.ns, d.tri != 0, [&](int r0, int c0, int rows, int cols, bool diag) {
    const int n = pair_blocks(rows, cols, diag);
    if (left >= n) {
      left -= n;
      return false;
    }
    block_rc(cols, diag, left, bi, bj);
    bi += r0;
    bj += c0;
    return true;
  });
  const double2* x = d.part + ((long long)t * d.nblk + g) * 256 + tid;
  const long long stride = (long long)d.nt * d.nblk * 256;
  double re = 0.0, im = 0.0;
  for (int sp = 0; sp < d.nsplit; ++sp) {
    const double2 v = x[sp * stride];
    re += v.x;
    im += v.y;
  }
  const int n = d.naux;
  double2* P = d.P + (long long)t * n * n;
  double2* M = d.M ? d.M - (long long)t * n * n : nullptr;
  {
    const int r = 4 * (tid >> 6) + ((tid & 63) >> 4), c = tid & 15;
    const int R = 16 * bi + r, C = 16 * bj + c;
    double2 v{d.alpha * re, d.alpha * im};
    if (R < n && C < n && d.accumulate) {
      const double2 old = P[(long long)R * n + C];
      v.x += old.x;
      v.y += old.y;
    }
    s[r][c] = v;
  }
  __syncthreads();
  const int y = tid >> 4, c = tid & 15;
  const bool tri = d.tri != 0, diag = tri && bi == bj;
  {
    // (16 bi + y, 16 bj + c); below the diagonal of a diagonal block the
    // conjugate of the entry above
    const int R = 16 * bi + y, C = 16 * bj + c;
    if (R < n && C < n) {
      double2 v = s[y][c];
      if (diag && y > c) {
        v = s[c][y];
        v.y = -v.y;
      }
      P[(long long)R * n + C] = v;
      if (M && tri) {              // P^T = conj(P) of a Hermitian P
        v.y = -v.y;
        if (diag && y == c) v.y = -v.y;
        M[(long long)R * n + C] = v;
      }
    }
  }
  if (diag) return;
  const int R = 16 * bj + y, C = 16 * bi + c;
  if (R < n && C < n) {
    const double2 v = s[c][y];
    if (tri) P[(long long)R * n + C] = double2{v.x, -v.y};
    if (M) M[(long long)R * n + C] = v;
  }
}

static int pol_supers(int nb) { return (nb + kSuper - 1) / kSuper; }

long long pol_acc_blocks(int naux, bool tri) {
  const int nb = (naux + 15) / 16;
  return tri ? (long long)nb * (nb + 1) / 2 : (long long)nb * nb;
}

hipError_t pol_acc_launch(const PolAcc& d0, long long part_elems, hipStream_t st) {
  if (d0.nt <= 0 || d0.naux <= 0 || d0.K <= 0) return hipSuccess;
  PolAcc d = d0;
  if (d.n2 < 4 || d.nt > 65535) return hipErrorInvalidValue;
  d.nb = (d.naux + 15) / 16;
  d.ns = pol_supers(d.nb);
  d.nblk = (int)pol_acc_blocks(d.naux, d.tri != 0);
  if (part_elems < (long long)d.nt * d.nblk * 256) return hipErrorInvalidValue;
  // one wave up to 7 blocks, two up to 14, otherwise four per workgroup
  const int W = d.nblk <= kMaxBlk ? 1 : d.nblk <= 2 * kMaxBlk ? 2 : 4;
  d.per = W == 4 ? kPartBlk : kMaxBlk * W;
  d.nparts = 0;
  each_pair(d.nb, d.ns, d.tri != 0, [&](int, int, int rows, int cols, bool diag) {
    d.nparts += (pair_blocks(rows, cols, diag) + d.per - 1) / d.per;
    return false;
  });
  // K parts: two waves per SIMD run at once; the count that ends its rounds
  // of workgroups soonest (a part costs about 24 steps of start and end)
  const long long slots = 256 * (8 / W), wgs = (long long)d.nparts * d.nt;
  const int steps = (d.K + 3) / 4;
  const long long room = part_elems / ((long long)d.nt * d.nblk * 256);
  int best = 1;
  double cost = 0.0;
  for (int s = 1; s <= 64 && s <= room && s <= steps; ++s) {
    const double c = (double)((wgs * s + slots - 1) / slots) * ((steps + s - 1) / s + 24);
    if (s == 1 || c < cost) {
      best = s;
      cost = c;
    }
  }
  d.steps = (steps + best - 1) / best;
  d.nsplit = (steps + d.steps - 1) / d.steps;
  if (wgs * d.nsplit > 0x7fffffffLL) return hipErrorInvalidConfiguration;
  const dim3 grid((unsigned)(wgs * d.nsplit));
  if (W == 1) pol_acc_k<1, 6><<<grid, 64, 0, st>>>(d);
  else if (W == 2) pol_acc_k<2, 4><<<grid, 128, 0, st>>>(d);
  else pol_acc_k<4, 5><<<grid, 256, 0, st>>>(d);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  pol_fin_k<<<dim3((unsigned)d.nblk, (unsigned)d.nt), 256, 0, st>>>(d);
  return hipGetLastError();
}
