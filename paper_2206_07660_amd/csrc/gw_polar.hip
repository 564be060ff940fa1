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
// triangle, the blocks 1.24 times).  fp64 MFMAs and vector instructions share
// the SIMD's fp64 pipe here (measured: each v_xor_b32 between 16x16x4 MFMAs
// costs 5 cycles, each v_add_f64 10, of 64 per MFMA), so the loop keeps the
// latter out: the rows of Y and V that a workgroup's blocks need go through
// LDS as operand fragments with their sums re +- im formed once per workgroup,
// and addresses are per-stage increments or scalars.  Two LDS stages of 8 k:
// each row is read from L2 in whole lines once per workgroup, and loads have a
// whole stage of MFMAs (2 x 7 x 3 x 64 cycles times two waves per SIMD) to
// arrive; half of the waves change stages in each half of a stage, so that the
// two waves of a SIMD rarely leave its pipe together.  Measured for one q (ms,
// 64 x 64 tiles of zgemm_k with four products before): 18.0 vs 22.5 at 4x4x4,
// nao 26, naux 250, 100 nodes (0.70 of the MFMA peak executed); 0.69 vs 1.76 at
// 3x3x3, nao 16, naux 150, 60 nodes.  A short K sum that leaves most of
// the chip idle is cut into smaller parts (general / Hermitian G at 2x2x2, nao
// 4, naux 150, 20 nodes, us a call: 45 / 49 on the tiles, 71 / 48 on parts of
// 56 blocks, 40 / 29 on parts of 8).
#include <hip/hip_runtime.h>

#include <algorithm>

#include "gw_device.h"
#include "gw_kernels.h"

namespace {

constexpr int kMaxBlk = 7;      // blocks of a wave
constexpr int kPartBlk = 56;    // blocks of the largest workgroup (8 waves)
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

// One element of a fragment in LDS; the 24-byte lane stride visits every bank
// once per 32 lanes.
struct Elem {
  double r, i, s;
};

}  // namespace

// W waves of M blocks each, loading L fragment rows per stage; a workgroup's
// blocks touch at most W * L fragment rows.  A wave past the last block
// repeats it, so that the loop has no branches.  AL: n2 is a multiple of 4, so
// the four k of a fragment never straddle two k-points and the K offset is a
// scalar.
template <int W, int L, int M, bool AL>
__global__ void __launch_bounds__(64 * W) pol_acc_k(PolAcc d) {
  __shared__ Elem lds[4 * W * L * 64];
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

  const int s0 = sp * d.steps, s1 = min(s0 + d.steps, (d.K + 7) / 8);
  // fragment rows of this wave: matrix, byte offset of this lane's row, place
  // in a stage and sign of the sum (rows past the last repeat it: the same
  // values to the same place)
  const double2* src[L];
  unsigned vo[L];
  double sg[L];
  int at[L];
#pragma unroll
  for (int l = 0; l < L; ++l) {
    const int f = min(wave + W * l, nf - 1);
    const bool y = f < na;
    const int row = 16 * (y ? p.r0 + ra + f : p.c0 + ca + (f - na)) + r16;
    src[l] = y ? d.Y + t * d.tsY : d.V;
    sg[l] = y ? 1.0 : -1.0;               // B = conj(V)
    vo[l] = ((unsigned)min(row, d.naux - 1) * (unsigned)d.n2 + (unsigned)kl) * 16u;
    at[l] = (f * 64 + lane) * (int)sizeof(Elem);
  }
  // k = ku n2 + e0 starts the stage to load
  const int n2 = d.n2, nk = d.K / n2;
  int k0 = 8 * s0, ku = k0 / n2, e0 = k0 - ku * n2;
  double2 f[2][L];
  auto fetch = [&]() {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      // k past K reads its row's first elements (stash stores zeros)
      if constexpr (AL) {
        const long long kb = k0 + 4 * h < d.K ? ku * d.sv + e0 : 0;
#pragma unroll
        for (int l = 0; l < L; ++l) f[h][l] = *(const double2*)((const char*)(src[l] + kb) + vo[l]);
        e0 += 4;
        if (e0 >= n2) {
          e0 -= n2;
          ++ku;
        }
      } else {
        const long long kb = min(ku, nk - 1) * d.sv;
        unsigned e = (unsigned)(e0 + kl), c = 0;
        if (e >= (unsigned)n2) {
          e -= n2;
          c = (unsigned)d.sv;
        }
        if (k0 + 4 * h + kl >= d.K) e = c = 0;
        const unsigned eo = (e + c - (unsigned)kl) * 16u;
#pragma unroll
        for (int l = 0; l < L; ++l) f[h][l] = *(const double2*)((const char*)(src[l] + kb) + (unsigned long long)(vo[l] + eo));
        e0 += 4;
        if (e0 >= n2) {                    // n2 >= 4: one carry
          e0 -= n2;
          ++ku;
        }
      }
    }
    k0 += 8;
  };
  // into the stage at byte offset `stage`; kk: its first k
  char* const lb = (char*)lds;
  constexpr int kHalf = W * L * 64 * (int)sizeof(Elem), kStage = 2 * kHalf;
  auto stash = [&](int stage, int kk) {
    if (!AL && kk + 8 > d.K) {
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int l = 0; l < L; ++l)
          if (kk + 4 * h + kl >= d.K) f[h][l] = double2{0.0, 0.0};
    }
#pragma unroll
    for (int l = 0; l < L; ++l) {
      char* q = lb + stage + at[l];
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const double2 v = f[h][l];
        *(Elem*)(q + h * kHalf) = Elem{v.x, v.y, __builtin_fma(sg[l], v.y, v.x)};
      }
    }
  };

  // this wave's blocks
  const int m = (p.cnt + W - 1) / W;
  const int mine = min(m, p.cnt - wave * m);   // may be <= 0
  int fa[M], fb[M];                            // byte offsets of their fragments in the current stage
#pragma unroll
  for (int b = 0; b < M; ++b) {
    block_rc(p.cols, p.diag, p.b0 + min(wave * m + min(b, m - 1), p.cnt - 1), rt, ct);
    fa[b] = ((rt - ra) * 64 + lane) * (int)sizeof(Elem);
    fb[b] = ((na + ct - ca) * 64 + lane) * (int)sizeof(Elem);
  }
  Acc3 o[M];
#pragma unroll
  for (int b = 0; b < M; ++b) o[b].p1 = o[b].p2 = o[b].p3 = d4{0, 0, 0, 0};

  if (s0 < s1) {
    fetch();
    stash(0, 8 * s0);
    fetch();
    __syncthreads();
    int flip = kStage;
    const bool late = wave >= W / 2;
    // The next stage moves from registers to LDS, and the one after it starts
    // to load, in the middle of the MFMAs, half of the waves in each half of
    // the stage: the two waves of a SIMD then rarely leave the pipe together.
    // No branch around single loads (each would wait for the one before); the
    // last ones go unused.
    auto turn = [&](int s) {
      __builtin_amdgcn_s_setprio(3);
      stash(flip > 0 ? kStage : 0, 8 * s + 8);
      fetch();
      __builtin_amdgcn_s_setprio(0);
      __builtin_amdgcn_sched_barrier(0);
    };
    for (int s = s0; s < s1; ++s) {
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        if (AL && h == 1 && 8 * s + 4 >= d.K) break;   // K is a multiple of 4, this half is past it
        Elem x[2], v[2];
        x[0] = *(const Elem*)(lb + fa[0] + h * kHalf);
        v[0] = *(const Elem*)(lb + fb[0] + h * kHalf);
#pragma unroll
        for (int b = 0; b < M; ++b) {
          if (b + 1 < M) {                 // the next block's elements
            x[(b + 1) & 1] = *(const Elem*)(lb + fa[b + 1] + h * kHalf);
            v[(b + 1) & 1] = *(const Elem*)(lb + fb[b + 1] + h * kHalf);
          }
          o[b].p1 = __builtin_amdgcn_mfma_f64_16x16x4f64(x[b & 1].r, v[b & 1].r, o[b].p1, 0, 0, 0);
          o[b].p2 = __builtin_amdgcn_mfma_f64_16x16x4f64(x[b & 1].i, v[b & 1].i, o[b].p2, 0, 0, 0);
          o[b].p3 = __builtin_amdgcn_mfma_f64_16x16x4f64(x[b & 1].s, v[b & 1].s, o[b].p3, 0, 0, 0);
          __builtin_amdgcn_sched_barrier(0);   // keeps the live elements at two blocks
          if (b == M / 2 && late == (h == 1)) turn(s);
        }
      }
#pragma unroll
      for (int b = 0; b < M; ++b) {
        fa[b] += flip;
        fb[b] += flip;
      }
      flip = -flip;
      __syncthreads();
    }
  }
  // with V unconjugated in p2: re = p1 + p2, im = p3 - p1 + p2
  double2* out = d.part + (((long long)sp * d.nt + t) * d.nblk + p.g0 + wave * m) * 256 + lane;
#pragma unroll
  for (int b = 0; b < M; ++b)
    if (b < mine) {
#pragma unroll
      for (int q = 0; q < 4; ++q)
        out[b * 256 + q * 64] = double2{o[b].p1[q] + o[b].p2[q], o[b].p3[q] - o[b].p1[q] + o[b].p2[q]};
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
  // one wave up to 6 blocks, two up to 12, four up to 24 (12 fragment rows:
  // 74 KB of LDS, two workgroups per CU), otherwise eight and as many parts as
  // keep a wave at 7 blocks
  const int W = d.nblk <= 6 ? 1 : d.nblk <= 12 ? 2 : d.nblk <= 24 ? 4 : 8;
  const long long slots = W == 8 ? 256 : W == 1 ? 1024 : 512;
  const int steps = (d.K + 7) / 8;
  const long long room = part_elems / ((long long)d.nt * d.nblk * 256);
  // K parts: two waves per SIMD run at once; the count that ends its rounds
  // of workgroups soonest (a part costs about 12 steps of start and end).
  // Where that leaves half of the chip idle (a short K sum: few steps, and
  // room for few partial sums) the blocks are dealt to more workgroups, down to
  // one block per wave; a step costs about one block more than it has.
  int M = 1, split = 1;            // blocks of a wave, K parts
  long long wgs = 0;
  double cost = 0.0;
  for (int per = W == 8 ? kPartBlk : 6 * W;; per = per == kPartBlk ? 32 : per / 2) {
    int nparts = 0, m = 1;
    each_pair(d.nb, d.ns, d.tri != 0, [&](int, int, int rows, int cols, bool diag) {
      const int n = pair_blocks(rows, cols, diag), np = (n + per - 1) / per;
      nparts += np;
      m = std::max(m, ((n + np - 1) / np + W - 1) / W);
      return false;
    });
    const long long w = (long long)nparts * d.nt;
    for (int s = 1; s <= 64 && s <= room && s <= steps; ++s) {
      const double c = (double)((w * s + slots - 1) / slots) * ((steps + s - 1) / s + 12) * (m + 1);
      if (wgs == 0 || c < cost) {
        cost = c;
        split = s;
        M = m;
        wgs = w;
        d.per = per;
        d.nparts = nparts;
      }
    }
    if (W < 8 || per <= W || 2 * wgs * split > slots) break;
  }
  d.steps = (steps + split - 1) / split;
  d.nsplit = (steps + d.steps - 1) / d.steps;
  if (wgs * d.nsplit > 0x7fffffffLL) return hipErrorInvalidConfiguration;
  const dim3 grid((unsigned)(wgs * d.nsplit));
#define POL_CALL(W_, L_, M_)                                                    \
  do {                                                                          \
    if (d.n2 % 4 == 0) pol_acc_k<W_, L_, M_, true><<<grid, 64 * W_, 0, st>>>(d); \
    else pol_acc_k<W_, L_, M_, false><<<grid, 64 * W_, 0, st>>>(d);             \
  } while (0)
  if (W == 8) {
    if (M == 7) POL_CALL(8, 3, 7);
    else if (M == 6) POL_CALL(8, 3, 6);
    else if (M == 5) POL_CALL(8, 3, 5);
    else if (M > 2) POL_CALL(8, 3, 4);
    else if (M == 2) POL_CALL(8, 3, 2);
    else POL_CALL(8, 3, 1);
  } else if (W == 4) {
    if (M == 6) POL_CALL(4, 3, 6);
    else POL_CALL(4, 3, 4);
  } else if (W == 2) {
    POL_CALL(2, 4, 5);
  } else {
    if (M == 1) POL_CALL(1, 2, 1);
    else if (M <= 4) POL_CALL(1, 4, 4);
    else POL_CALL(1, 6, 6);
  }
#undef POL_CALL
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  pol_fin_k<<<dim3((unsigned)d.nblk, (unsigned)d.nt), 256, 0, st>>>(d);
  return hipGetLastError();
}
