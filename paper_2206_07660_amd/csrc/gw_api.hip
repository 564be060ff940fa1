// C ABI of the density-fitted GW hot path: context, argument checks, and the
// mapping of every equation onto the device kernels.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdio>
#include <algorithm>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <new>
#include <string>
#include <vector>

#include "../../include/gw.h"
#include "grids.h"
#include "gw_extents.h"
#include "gw_kernels.h"
#include "gw_mu.h"
#include "ir.h"

// Fixed scratch for gw_polarization_noalloc: a file-scope device array, one
// copy per GPU for the life of the process.  Host code never passes the
// array's name to a kernel (on the host it is only a stand-in symbol): the
// device address of each GPU's copy is looked up once per device with
// hipGetSymbolAddress and kept in g_scratch_dev.
static const size_t kScratchBytes = size_t(128) << 20;   // 128 MiB
static __device__ __align__(256) char scratch[kScratchBytes];
static const int kMaxDevices = 64;
static char* g_scratch_dev[kMaxDevices] = {};
static std::mutex g_scratch_mu;

struct gw_ctx {
  gw_dims d;
  int nk = 0;
  long long n2 = 0;      // nao^2
  long long sv = 0;      // complex elements of one V^{k,k+q} block: naux * nao^2
  hipStream_t st = nullptr;
  int device = 0;
  char* scratch = nullptr;   // this device's copy of the fixed scratch array (see below)
  bool grids = false;
  std::vector<double> tau, x, w;
  std::vector<long long> nF, nB;
  std::vector<gwgrid::cd> TF, TFp, TB, TBp, rrow;
  std::vector<int> plus;   // host copy of the k+q table
  std::vector<int> neg;    // neg[q] = index of -q
  bool check_bounds = false;
  int tile_cfg = -1;       // tile configuration of the large contractions (-1: default)
  int prod_tiles = 0;      // 1: fp32 producers on the tiled GEMM instead of the streaming kernel
  int split_cfg = -1;      // tile configuration of the split-bf16 contractions
  int split_group = 0;     // > 0: grouped workgroup order of the split contractions
  int herm = 0;            // gw_set_hermitian: GW_HERM_* bits
  // with symmetric bosonic tables: one q of each pair {q, -q} (reps), its
  // partner (negs) and the positions q nw_b + m of its matrices at Omega >= 0
  // (m >= mid); dsel holds reps, negs and these positions one after the other
  int nrep = 0, mid = 0;
  std::vector<int> sel;
  int* dsel = nullptr;
  bool sym_b = false;      // bosonic tables symmetric under Omega -> -Omega and tau -> beta - tau
  double mu_window = 0.0;  // gw_set_mu_window: electron-count window (0: exact root)
  // measurement: event pairs per kernel class while profiling is on
  bool prof = false;
  std::vector<std::pair<hipEvent_t, hipEvent_t>> ev[KC_COUNT];
  long long launches[KC_COUNT] = {};
  double flops[KC_COUNT] = {};
  double ms[KC_COUNT] = {};
  double2 *dTF = nullptr, *dTFp = nullptr, *dTB = nullptr, *dTBp = nullptr;
  double2 *dw = nullptr, *drrow = nullptr;
  double* dwF = nullptr;
  int *dplus = nullptr, *dminus = nullptr;
  int* dflag = nullptr;
  double* dpart = nullptr;   // nw_f * nk partials, then the reduced scalar at [nw_f*nk]
  MuCounts mu{1, 1};         // values of mu that one electron-count launch takes
  double* dcnt = nullptr;    // nw_f * nk partials of the electron counts of a launch
  double* hcnt = nullptr;    // pinned host memory: the counts
  double* dred = nullptr;    // 2 * 1024 partials + 2 results for gw_dot
  double* dphi = nullptr;    // Nk * nw_b per-matrix terms of Phi~, then their sum
  void* ws = nullptr;
  size_t ws_bytes = 0;
  int tc = 0;
  std::string err;
};

namespace {

gw_status fail(gw_ctx* c, gw_status s, const std::string& msg) {
  if (c) c->err = msg;
  return s;
}

#define HIPCHK(ctx, call)                                                              \
  do {                                                                                 \
    hipError_t e_ = (call);                                                            \
    if (e_ != hipSuccess)                                                              \
      return fail(ctx, GW_ERR_DEVICE, std::string(#call) + ": " + hipGetErrorString(e_)); \
  } while (0)

int mesh_index(const int* mesh, int a, int b, int c) {
  a = ((a % mesh[0]) + mesh[0]) % mesh[0];
  b = ((b % mesh[1]) + mesh[1]) % mesh[1];
  c = ((c % mesh[2]) + mesh[2]) % mesh[2];
  return (a * mesh[1] + b) * mesh[2] + c;
}

gw_status check_dims(const gw_dims* d, std::string& why) {
  if (!d) { why = "dims is NULL"; return GW_ERR_ARG; }
  for (int i = 0; i < 3; ++i)
    if (d->mesh[i] < 1 || d->mesh[i] > 64) { why = "mesh entries must be in 1..64"; return GW_ERR_ARG; }
  if (d->nao < 1 || d->nao > 60) { why = "nao must be in 1..60"; return GW_ERR_ARG; }
  if (d->naux < 1 || d->naux > 8192) { why = "naux must be in 1..8192"; return GW_ERR_ARG; }
  if (d->ntau < 2 || d->ntau > 512 || d->ntau % 2) { why = "ntau must be even, 2..512"; return GW_ERR_ARG; }
  if (d->nw_f < d->ntau || d->nw_f > 4 * d->ntau) { why = "nw_f must lie in ntau..4 ntau"; return GW_ERR_ARG; }
  if (d->nw_b < d->ntau || d->nw_b > 4 * d->ntau + 1) {
    why = "nw_b must lie in ntau..4 ntau + 1";
    return GW_ERR_ARG;
  }
  if (d->ns != 1 && d->ns != 2) { why = "ns must be 1 or 2"; return GW_ERR_ARG; }
  if (!(d->beta > 0.0) || !std::isfinite(d->beta)) { why = "beta must be positive"; return GW_ERR_ARG; }
  if (d->precision < GW_PREC_FP64 || d->precision > GW_PREC_BF16X6) {
    why = "unsupported precision";
    return GW_ERR_ARG;
  }
  const long long nk = (long long)d->mesh[0] * d->mesh[1] * d->mesh[2];
  if (nk * d->nao * (long long)d->nao * d->naux > (1LL << 31)) {
    why = "Nk * naux * nao^2 must stay below 2^31";
    return GW_ERR_ARG;
  }
  return GW_OK;
}

bool ready(gw_ctx* c) { return c && c->grids; }

size_t align256(size_t b) { return (b + 255) & ~size_t(255); }

template <class T>
gw_status upload(gw_ctx* c, T** dst, const void* src, size_t bytes) {
  HIPCHK(c, hipMalloc((void**)dst, bytes));
  HIPCHK(c, hipMemcpy(*dst, src, bytes, hipMemcpyHostToDevice));
  return GW_OK;
}

// Exact [min, max] of a mapped index over i in [0, n).
void map_range(const Map3& m, long long n, long long& lo, long long& hi) {
  lo = hi = 0;
  for (long long i = 0; i < n; ++i) {
    const unsigned a = (unsigned)(i % m.din);
    const unsigned r = (unsigned)(i / m.din);
    const long long o = (long long)(r / m.dmid) * m.sout + (long long)(r % m.dmid) * m.smid +
                        (long long)a * m.sin;
    if (i == 0 || o < lo) lo = (i == 0) ? o : std::min(lo, o);
    if (i == 0 || o > hi) hi = (i == 0) ? o : std::max(hi, o);
  }
}

// Host-side proof that a GEMM descriptor stays inside its operands: every
// touched offset of A, B and C lies in [0, ext).  Enabled by GW_DEBUG_BOUNDS.
struct Ext {
  long long lo, hi;   // valid element offsets [lo, hi) relative to the operand pointer
};

bool gemm_in_bounds(gw_ctx* c, const GemmDesc& g, Ext eA, Ext eB, Ext eC, std::string& why) {
  long long bl[3] = {0, 0, 0}, bh[3] = {0, 0, 0};
  const Map3* bm[3] = {&g.ba, &g.bb, &g.bc};
  const long long ts[3] = {g.tsA, g.tsB, g.tsC};
  for (int o = 0; o < 3; ++o)
    for (long long b = 0; b < g.batch; ++b) {
      const unsigned a = (unsigned)(b % bm[o]->din);
      const unsigned r = (unsigned)(b / bm[o]->din);
      long long off = (long long)(r / bm[o]->dmid) * bm[o]->sout +
                      (long long)(r % bm[o]->dmid) * bm[o]->smid + (long long)a * bm[o]->sin;
      if (ts[o] != 0) {
        // tables are rows of the k+q table or parts of the pair tables
        const bool pl = g.tab >= c->dplus && g.tab < c->dplus + c->plus.size();
        const int* th = pl ? c->plus.data() + (g.tab - c->dplus) : c->sel.data() + (g.tab - c->dsel);
        off += (long long)th[b % g.tmod] * ts[o];
      }
      if (b == 0 || off < bl[o]) bl[o] = (b == 0) ? off : std::min(bl[o], off);
      if (b == 0 || off > bh[o]) bh[o] = (b == 0) ? off : std::max(bh[o], off);
    }
  long long l1, h1, l2, h2;
  map_range(g.am, g.M, l1, h1);
  map_range(g.ak, g.K, l2, h2);
  if (bl[0] + l1 + l2 < eA.lo || bh[0] + h1 + h2 >= eA.hi) {
    why = "A out of bounds: [" + std::to_string(bl[0] + l1 + l2) + ", " + std::to_string(bh[0] + h1 + h2) +
          "] vs [" + std::to_string(eA.lo) + ", " + std::to_string(eA.hi) + ")";
    return false;
  }
  map_range(g.bk, g.K, l1, h1);
  map_range(g.bn, g.N, l2, h2);
  if (bl[1] + l1 + l2 < eB.lo || bh[1] + h1 + h2 >= eB.hi) {
    why = "B out of bounds: [" + std::to_string(bl[1] + l1 + l2) + ", " + std::to_string(bh[1] + h1 + h2) +
          "] vs [" + std::to_string(eB.lo) + ", " + std::to_string(eB.hi) + ")";
    return false;
  }
  map_range(g.cm, g.M, l1, h1);
  map_range(g.cn, g.N, l2, h2);
  if (bl[2] + l1 + l2 < eC.lo || bh[2] + h1 + h2 >= eC.hi) {
    why = "C out of bounds: [" + std::to_string(bl[2] + l1 + l2) + ", " + std::to_string(bh[2] + h1 + h2) +
          "] vs [" + std::to_string(eC.lo) + ", " + std::to_string(eC.hi) + ")";
    return false;
  }
  return true;
}

gw_status prof_begin(gw_ctx* c, int kc, hipEvent_t* e0) {
  if (!c->prof) return GW_OK;
  HIPCHK(c, hipEventCreate(e0));
  HIPCHK(c, hipEventRecord(*e0, c->st));
  (void)kc;
  return GW_OK;
}

gw_status prof_end(gw_ctx* c, int kc, hipEvent_t e0, double flops) {
  if (!c->prof) return GW_OK;
  hipEvent_t e1;
  HIPCHK(c, hipEventCreate(&e1));
  HIPCHK(c, hipEventRecord(e1, c->st));
  c->ev[kc].push_back({e0, e1});
  c->launches[kc] += 1;
  c->flops[kc] += flops;
  return GW_OK;
}

gw_status run(gw_ctx* c, const GemmDesc& g, Ext eA, Ext eB, Ext eC) {
  if (c->check_bounds) {
    std::string why;
    if (!gemm_in_bounds(c, g, eA, eB, eC, why))
      return fail(c, GW_ERR_ARG, "internal descriptor check: " + why);
  }
  hipEvent_t e0 = nullptr;
  gw_status s = prof_begin(c, g.tag, &e0);
  if (s != GW_OK) return s;
  GemmDesc gg = g;
  // tile shapes measured best on MI355X at naux = 250: 64x64 for the
  // polarization contraction, 64x96 on the three-product (Gauss) form for
  // the self-energy one, 32x192 where that executes less (few columns do not
  // fill its width: 3x3x3, one orbital, naux 220, 30 nodes: 68.6 vs 40.6 us)
  auto executed = [&](long long tm, long long tn) { return (g.M + tm - 1) / tm * tm * ((g.N + tn - 1) / tn * tn); };
  if (g.tag == KC_POL_PRODUCER || g.tag == KC_SE_PRODUCER) gg.cfg = c->prod_tiles;
  else if (c->tile_cfg >= 0) gg.cfg = c->tile_cfg;
  else if (g.tag == KC_SE_CONTRACT) gg.cfg = executed(32, 192) < executed(64, 96) ? 10 : 7;
  else gg.cfg = 0;
  hipError_t e = zgemm_launch(gg, c->st);
  if (e != hipSuccess) return fail(c, GW_ERR_DEVICE, std::string("zgemm: ") + hipGetErrorString(e));
  // MFMA flops executed: 8 real flops per complex multiply-add, 6 on the
  // three-product form; with g.tri only the entries on and above the diagonal
  const double outs = g.tri ? 0.5 * g.M * (g.M + 1.0) : (double)g.M * g.N;
  const double per = zgemm_three_product(gg) ? 6.0 : 8.0;
  return prof_end(c, g.tag, e0, per * outs * g.K * g.batch);
}

// Split-bf16 contraction: eA, eB, eC the valid element ranges of the
// operands; k_true the K that the algorithmic flops count.
gw_status run_split(gw_ctx* c, const SplitDesc& d, Ext eA, Ext eB, Ext eC) {
  if (c->check_bounds) {
    auto span = [&](const Map3& bm, const Map3& rm, int rows, long long ks, long long& lo, long long& hi) {
      long long l1, h1, l2, h2;
      map_range(bm, d.batch, l1, h1);
      map_range(rm, rows, l2, h2);
      lo = l1 + l2 + std::min(0LL, (long long)(d.K - 1) * ks);
      hi = h1 + h2 + std::max(0LL, (long long)(d.K - 1) * ks);
    };
    long long la, ha, lb, hb, lc, hc, l1, h1;
    span(d.ba, d.am, d.M, d.aks, la, ha);
    span(d.bb, d.bn, d.N, d.bks, lb, hb);
    span(d.bc, d.cm, d.M, 0, lc, hc);
    map_range(d.cn, d.N, l1, h1);
    lc += l1;
    hc += h1;
    if (la < eA.lo || ha >= eA.hi || lb < eB.lo || hb >= eB.hi || lc < eC.lo || hc >= eC.hi)
      return fail(c, GW_ERR_ARG, "internal descriptor check: split contraction out of bounds");
  }
  hipEvent_t e0 = nullptr;
  gw_status s = prof_begin(c, d.tag, &e0);
  if (s != GW_OK) return s;
  SplitDesc dd = d;
  dd.cfg = c->split_cfg;
  if (c->split_group > 0) {
    dd.batch_fastest = 2;
    dd.group = c->split_group;
  }
  hipError_t e = bsgemm_launch(dd, c->st);
  if (e != hipSuccess) return fail(c, GW_ERR_DEVICE, std::string("bsgemm: ") + hipGetErrorString(e));
  const double outs = d.tri ? 0.5 * d.M * (d.M + 1.0) : (double)d.M * d.N;
  return prof_end(c, d.tag, e0, 8.0 * outs * d.K * d.batch);
}

gw_status leaves(gw_ctx* c, const char* what, const char* operand) {
  return operand ? fail(c, GW_ERR_ARG, std::string("internal descriptor check: ") + what + ": " + operand + " out of bounds")
                 : GW_OK;
}
// host copy of a part of the k+q table, and its entries from there on
const int* host_tab(const gw_ctx* c, const int* tab) { return c->plus.data() + (tab - c->dplus); }
long long tab_left(const gw_ctx* c, const int* tab) { return (long long)c->plus.size() - (tab - c->dplus); }

// The triple products (nao x nao matrices) with their profiling class; 6 real
// flops per complex multiply-add (three real products).  The arrays that the
// operands lie in follow in the operands' order.
gw_status sand_prod(gw_ctx* c, SandProd d, int tag, Arr V, Arr L, Arr R, Arr Y) {
  d.nk = c->nk; d.naux = c->d.naux; d.nao = c->d.nao;
  d.svk = c->sv;
  gw_status s;
  if (c->check_bounds &&
      (s = leaves(c, "sand_prod", sand_prod_leaves(d, host_tab(c, d.tab), tab_left(c, d.tab), V, L, R, Y))) != GW_OK)
    return s;
  hipEvent_t e0 = nullptr;
  if ((s = prof_begin(c, tag, &e0)) != GW_OK) return s;
  hipError_t e = sand_prod_launch(d, c->st);
  if (e != hipSuccess) return fail(c, GW_ERR_DEVICE, std::string("sand_prod: ") + hipGetErrorString(e));
  return prof_end(c, tag, e0, 12.0 * d.nt * d.nk * c->sv * c->d.nao);
}

gw_status sand_sum(gw_ctx* c, SandSum d, int tag, Arr A, Arr B, Arr G, Arr O, Arr part) {
  d.nk = c->nk; d.naux = c->d.naux; d.nao = c->d.nao;
  gw_status s;
  if (c->check_bounds &&
      (s = leaves(c, "sand_sum", sand_sum_leaves(d, host_tab(c, d.tab), tab_left(c, d.tab), A, B, G, O, part))) != GW_OK)
    return s;
  hipEvent_t e0 = nullptr;
  if ((s = prof_begin(c, tag, &e0)) != GW_OK) return s;
  hipError_t e = sand_sum_launch(d, c->st);
  if (e != hipSuccess) return fail(c, GW_ERR_DEVICE, std::string("sand_sum: ") + hipGetErrorString(e));
  return prof_end(c, tag, e0, 12.0 * d.nt * d.nk * c->sv * c->d.nao);
}

gw_status read_flag(gw_ctx* c, const char* what) {
  int f = 0;
  HIPCHK(c, hipMemcpyAsync(&f, c->dflag, sizeof(int), hipMemcpyDeviceToHost, c->st));
  HIPCHK(c, hipStreamSynchronize(c->st));
  if (f) return fail(c, GW_ERR_SINGULAR, std::string(what) + ": zero pivot");
  return GW_OK;
}

// Dyson matrices at nmu values of mu: nao <= 32 on the wave-per-matrix kernel,
// larger ones (nmu = 1, see mu_counts) a workgroup each.
hipError_t dyson_any(gw_ctx* c, const DysonArgs& a, int nmu) {
  if (c->d.nao <= 32) return dyson_reg_launch(a, c->d.nw_f, nmu, c->st);
  return nmu == 1 ? dyson_launch(a, c->d.nw_f, c->st) : hipErrorInvalidValue;
}

// The electron count as a function of mu, for one set of Dyson inputs.
struct Count {
  gw_ctx* c;
  const gw_z *H0, *S, *Sinf, *Siw;

  // counts at n values in one launch (G written for n = 1, if given),
  // with a zero pivot left to count_status or to the flag
  gw_status at(const double* mu, int n, double* ne, gw_z* Gout = nullptr) const {
    DysonArgs a{};
    a.H0 = (const double2*)H0;
    a.S = (const double2*)S;
    a.Sinf = (const double2*)Sinf;
    a.Siw = (const double2*)Siw;
    a.wF = c->dwF;
    a.rrow = c->drrow;
    a.mu = mu[0];
    for (int i = 1; i < n; ++i) a.more[i - 1] = mu[i];
    a.nk = c->nk;
    a.nao = c->d.nao;
    a.G = (double2*)Gout;
    a.part = c->dcnt;
    a.flag = c->dflag;
    HIPCHK(c, dyson_any(c, a, n));
    // the sums go to pinned host memory: no copy to wait for
    HIPCHK(c, sum_rows_launch(c->dcnt, c->d.nw_f * c->nk, n, -(double)c->d.ns / c->nk, c->hcnt, c->st));
    HIPCHK(c, hipStreamSynchronize(c->st));
    for (int i = 0; i < n; ++i) ne[i] = c->hcnt[i];
    return GW_OK;
  }
  gw_status operator()(const double* mu, int n, double* ne) const { return at(mu, n, ne); }
  // one count that has to be finite
  gw_status one(double mu, double* n, gw_z* Gout = nullptr) const {
    const char* why = "";
    gw_status s = at(&mu, 1, n, Gout);
    if (s == GW_OK && (s = count_status(*n, &why)) != GW_OK) return fail(c, s, why);
    return s;
  }
};

}  // namespace

extern "C" {

const char* gw_status_string(gw_status s) {
  switch (s) {
    case GW_OK: return "ok";
    case GW_ERR_ARG: return "invalid argument";
    case GW_ERR_DEVICE: return "HIP runtime error";
    case GW_ERR_SINGULAR: return "singular matrix";
    case GW_ERR_NOCONV: return "no convergence";
    case GW_ERR_WORKSPACE: return "workspace missing or too small";
    case GW_ERR_STATE: return "grids not built";
    case GW_ERR_NONFINITE: return "non-finite value";
  }
  return "unknown status";
}

const char* gw_last_error(const gw_ctx* c) { return c ? c->err.c_str() : "NULL context"; }

gw_status gw_create(const gw_dims* d, void* hip_stream, gw_ctx** out) {
  if (!out) return GW_ERR_ARG;
  *out = nullptr;
  std::string why;
  if (check_dims(d, why) != GW_OK) return GW_ERR_ARG;
  gw_ctx* c = new (std::nothrow) gw_ctx();
  if (!c) return GW_ERR_DEVICE;
  c->d = *d;
  c->nk = d->mesh[0] * d->mesh[1] * d->mesh[2];
  c->n2 = (long long)d->nao * d->nao;
  c->sv = (long long)d->naux * c->n2;
  c->st = (hipStream_t)hip_stream;
  if (hipGetDevice(&c->device) != hipSuccess) { delete c; return GW_ERR_DEVICE; }
  if (c->device < 0 || c->device >= kMaxDevices) { delete c; return GW_ERR_DEVICE; }
  {
    // once per device, with that device current: the device address of its scratch copy
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (!g_scratch_dev[c->device]) {
      void* p = nullptr;
      if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) { delete c; return GW_ERR_DEVICE; }
      g_scratch_dev[c->device] = (char*)p;
    }
    c->scratch = g_scratch_dev[c->device];
  }
  std::vector<int> plus((size_t)c->nk * c->nk), minus((size_t)c->nk * c->nk);
  const int* m = d->mesh;
  for (int q = 0; q < c->nk; ++q)
    for (int k = 0; k < c->nk; ++k) {
      const int qa = q / (m[1] * m[2]), qb = (q / m[2]) % m[1], qc = q % m[2];
      const int ka = k / (m[1] * m[2]), kb = (k / m[2]) % m[1], kc = k % m[2];
      plus[(size_t)q * c->nk + k] = mesh_index(m, ka + qa, kb + qb, kc + qc);
      minus[(size_t)q * c->nk + k] = mesh_index(m, ka - qa, kb - qb, kc - qc);
    }
  c->plus = plus;
  c->neg.resize(c->nk);
  for (int q = 0; q < c->nk; ++q) c->neg[q] = minus[(size_t)q * c->nk];
  {
    const char* e = std::getenv("GW_DEBUG_BOUNDS");
    c->check_bounds = e && e[0] == '1';
    const char* t = std::getenv("GW_TILE_CFG");
    c->tile_cfg = t ? std::atoi(t) : -1;
    const char* pt = std::getenv("GW_PROD_TILES");
    c->prod_tiles = pt && pt[0] == '1' ? 1 : 0;
    const char* u = std::getenv("GW_SPLIT_CFG");
    c->split_cfg = u ? std::atoi(u) : -1;
    const char* gg = std::getenv("GW_SPLIT_GROUP");
    c->split_group = gg ? std::atoi(gg) : 0;
  }
  c->mu = mu_counts(d->nao, (long long)d->nw_f * c->nk);
  const size_t counts = (size_t)std::max(c->mu.batch, c->mu.ahead) * d->nw_f * c->nk;
  if (upload(c, &c->dplus, plus.data(), plus.size() * sizeof(int)) != GW_OK ||
      upload(c, &c->dminus, minus.data(), minus.size() * sizeof(int)) != GW_OK ||
      hipMalloc((void**)&c->dflag, sizeof(int)) != hipSuccess ||
      hipMemset(c->dflag, 0, sizeof(int)) != hipSuccess ||
      hipMalloc((void**)&c->dpart, ((size_t)d->nw_f * c->nk + 8) * sizeof(double)) != hipSuccess ||
      hipMalloc((void**)&c->dcnt, counts * sizeof(double)) != hipSuccess ||
      hipHostMalloc((void**)&c->hcnt, 16 * sizeof(double), hipHostMallocMapped) != hipSuccess ||
      hipMalloc((void**)&c->dred, (2 * 1024 + 8) * sizeof(double)) != hipSuccess ||
      hipMalloc((void**)&c->dphi, ((size_t)d->nw_b * c->nk + 8) * sizeof(double)) != hipSuccess) {
    gw_destroy(c);
    return GW_ERR_DEVICE;
  }
  *out = c;
  return GW_OK;
}

gw_status gw_destroy(gw_ctx* c) {
  if (!c) return GW_ERR_ARG;
  for (int k = 0; k < KC_COUNT; ++k)
    for (auto& p : c->ev[k]) {
      (void)hipEventDestroy(p.first);
      (void)hipEventDestroy(p.second);
    }
  void* ptrs[] = {c->dTF, c->dTFp, c->dTB, c->dTBp, c->dw, c->drrow, c->dwF,
                  c->dplus, c->dminus, c->dflag, c->dpart, c->dred, c->dphi, c->dcnt, c->dsel};
  for (void* p : ptrs)
    if (p) (void)hipFree(p);
  if (c->hcnt) (void)hipHostFree(c->hcnt);
  delete c;
  return GW_OK;
}

struct HostGrids {
  std::vector<double> tau, x, w;
  std::vector<long long> nF, nB;
  std::vector<gwgrid::cd> TF, TFp, TB, TBp, rrow;
  std::vector<double> wf;
};

// Derived tables: fermionic frequencies and the electron-count row r = w TFp.
static void finish_grids(double beta, HostGrids& g) {
  const int nt = (int)g.tau.size(), nwf = (int)g.nF.size();
  g.wf.assign(nwf, 0.0);
  for (int n = 0; n < nwf; ++n) g.wf[n] = gwgrid::matsubara(g.nF[n], beta, 0);
  g.rrow.assign(nwf, 0.0);
  for (int n = 0; n < nwf; ++n) {
    gwgrid::cd s = 0.0;
    for (int i = 0; i < nt; ++i) s += g.w[i] * g.TFp[(size_t)i * nwf + n];
    g.rrow[n] = s;
  }
}

static gw_status make_grids(double beta, int nt, const long long* nF, const long long* nB,
                            HostGrids& g, std::string& why) {
  if (!(beta > 0.0) || !std::isfinite(beta) || nt < 2 || nt > 512 || nt % 2) {
    why = "beta must be positive and ntau even in 2..512";
    return GW_ERR_ARG;
  }
  const int nwf = nt, nwb = nt + 1;
  try {
    g.tau.assign(nt, 0.0);
    g.x.assign(nt, 0.0);
    gwgrid::tau_nodes(beta, nt, g.tau.data(), g.x.data());
    if (nF) g.nF.assign(nF, nF + nwf); else g.nF = gwgrid::select_sparse(beta, nt, 0);
    if (nB) g.nB.assign(nB, nB + nwb); else g.nB = gwgrid::select_sparse(beta, nt, 1);
    for (size_t i = 1; i < g.nF.size(); ++i)
      if (g.nF[i] <= g.nF[i - 1]) { why = "nF must be strictly increasing"; return GW_ERR_ARG; }
    for (size_t i = 1; i < g.nB.size(); ++i)
      if (g.nB[i] <= g.nB[i - 1]) { why = "nB must be strictly increasing"; return GW_ERR_ARG; }
    std::vector<double> wf(nwf), wb(nwb);
    for (int n = 0; n < nwf; ++n) wf[n] = gwgrid::matsubara(g.nF[n], beta, 0);
    for (int n = 0; n < nwb; ++n) wb[n] = gwgrid::matsubara(g.nB[n], beta, 1);
    g.TF.assign((size_t)nwf * nt, 0.0);
    g.TB.assign((size_t)nwb * nt, 0.0);
    g.TFp.assign((size_t)nt * nwf, 0.0);
    g.TBp.assign((size_t)nt * nwb, 0.0);
    gwgrid::transform(beta, nt, g.x.data(), wf.data(), nwf, g.TF.data());
    gwgrid::transform(beta, nt, g.x.data(), wb.data(), nwb, g.TB.data());
    if (gwgrid::pinv_qr(g.TF.data(), nwf, nt, g.TFp.data()) ||
        gwgrid::pinv_qr(g.TB.data(), nwb, nt, g.TBp.data())) {
      why = "transform matrix is rank deficient for these frequencies";
      return GW_ERR_ARG;
    }
    g.w.assign(nt, 0.0);
    gwgrid::beta_row(nt, g.x.data(), g.w.data());
    finish_grids(beta, g);
  } catch (const std::exception& e) {
    why = e.what();
    return GW_ERR_ARG;
  }
  return GW_OK;
}

gw_status gw_grids_host(double beta, int ntau, const long long* nF, const long long* nB,
                        double* tau, long long* nF_out, long long* nB_out, gw_z* TF, gw_z* TFp,
                        gw_z* TB, gw_z* TBp, double* w) {
  HostGrids g;
  std::string why;
  gw_status s = make_grids(beta, ntau, nF, nB, g, why);
  if (s != GW_OK) return s;
  if (tau) std::memcpy(tau, g.tau.data(), g.tau.size() * 8);
  if (nF_out) std::memcpy(nF_out, g.nF.data(), g.nF.size() * 8);
  if (nB_out) std::memcpy(nB_out, g.nB.data(), g.nB.size() * 8);
  if (TF) std::memcpy(TF, g.TF.data(), g.TF.size() * 16);
  if (TFp) std::memcpy(TFp, g.TFp.data(), g.TFp.size() * 16);
  if (TB) std::memcpy(TB, g.TB.data(), g.TB.size() * 16);
  if (TBp) std::memcpy(TBp, g.TBp.data(), g.TBp.size() * 16);
  if (w) std::memcpy(w, g.w.data(), g.w.size() * 8);
  return GW_OK;
}

// Whether the bosonic tables keep the symmetries of the exact transforms,
// T(-Omega, tau) = conj T(Omega, tau) = T(Omega, beta - tau) and the same for
// the fit.  Chebyshev tables do to 3e-12 of their largest entry (200 nodes);
// IR tables of a small cutoff do not (1e-6 at lambda 500, eps 1e-12: their
// last basis functions are rounding), nor need caller tables.
static bool bosonic_symmetry(const gw_ctx* c) {
  const int nt = c->d.ntau, nw = c->d.nw_b;
  const double tol = 1e-11;
  for (int n = 0; n < nw; ++n)
    if (c->nB[n] != -c->nB[nw - 1 - n]) return false;
  double mT = 0.0, mP = 0.0, dT = 0.0, dP = 0.0;
  for (int n = 0; n < nw; ++n)
    for (int i = 0; i < nt; ++i) {
      const gwgrid::cd t = c->TB[(size_t)n * nt + i], q = c->TBp[(size_t)i * nw + n];
      mT = std::max(mT, std::abs(t));
      mP = std::max(mP, std::abs(q));
      dT = std::max({dT, std::abs(c->TB[(size_t)(nw - 1 - n) * nt + i] - std::conj(t)),
                     std::abs(c->TB[(size_t)n * nt + nt - 1 - i] - std::conj(t))});
      dP = std::max({dP, std::abs(c->TBp[(size_t)i * nw + nw - 1 - n] - std::conj(q)),
                     std::abs(c->TBp[(size_t)(nt - 1 - i) * nw + n] - std::conj(q))});
    }
  return dT <= tol * mT && dP <= tol * mP;
}

// Keep the host tables in the context and upload the device copies.
static gw_status install_grids(gw_ctx* c, HostGrids& g) {
  c->tau = g.tau; c->x = g.x; c->w = g.w; c->nF = g.nF; c->nB = g.nB;
  c->TF = g.TF; c->TFp = g.TFp; c->TB = g.TB; c->TBp = g.TBp; c->rrow = g.rrow;
  std::vector<gwgrid::cd> wz(c->w.begin(), c->w.end());
  void* olds[] = {c->dTF, c->dTFp, c->dTB, c->dTBp, c->dw, c->drrow, c->dwF, c->dsel};
  for (void* p : olds)
    if (p) (void)hipFree(p);
  c->dTF = c->dTFp = c->dTB = c->dTBp = c->dw = c->drrow = nullptr;
  c->dwF = nullptr;
  c->dsel = nullptr;
  c->grids = false;
  c->sym_b = bosonic_symmetry(c);
  gw_status s;
  c->sel.clear();
  c->nrep = 0;
  c->mid = c->d.nw_b / 2;
  if (c->sym_b) {
    for (int q = 0; q < c->nk; ++q)
      if (c->neg[q] >= q) c->sel.push_back(q);
    c->nrep = (int)c->sel.size();
    for (int i = 0; i < c->nrep; ++i) c->sel.push_back(c->neg[c->sel[i]]);
    for (int i = 0; i < c->nrep; ++i)
      for (int m = c->mid; m < c->d.nw_b; ++m) c->sel.push_back(c->sel[i] * c->d.nw_b + m);
    if ((s = upload(c, &c->dsel, c->sel.data(), c->sel.size() * sizeof(int))) != GW_OK) return s;
  }
  if ((s = upload(c, &c->dTF, c->TF.data(), c->TF.size() * 16)) != GW_OK) return s;
  if ((s = upload(c, &c->dTFp, c->TFp.data(), c->TFp.size() * 16)) != GW_OK) return s;
  if ((s = upload(c, &c->dTB, c->TB.data(), c->TB.size() * 16)) != GW_OK) return s;
  if ((s = upload(c, &c->dTBp, c->TBp.data(), c->TBp.size() * 16)) != GW_OK) return s;
  if ((s = upload(c, &c->dw, wz.data(), wz.size() * 16)) != GW_OK) return s;
  if ((s = upload(c, &c->drrow, c->rrow.data(), c->rrow.size() * 16)) != GW_OK) return s;
  if ((s = upload(c, &c->dwF, g.wf.data(), g.wf.size() * 8)) != GW_OK) return s;
  c->grids = true;
  return GW_OK;
}

gw_status gw_build_grids(gw_ctx* c, const long long* nF, const long long* nB) {
  if (!c) return GW_ERR_ARG;
  if (c->d.nw_f != c->d.ntau || c->d.nw_b != c->d.ntau + 1)
    return fail(c, GW_ERR_ARG, "gw_build_grids needs nw_f = ntau and nw_b = ntau + 1");
  HostGrids g;
  std::string why;
  gw_status s = make_grids(c->d.beta, c->d.ntau, nF, nB, g, why);
  if (s != GW_OK) return fail(c, s, why);
  return install_grids(c, g);
}

gw_status gw_set_grids(gw_ctx* c, const double* tau, const long long* nF, const long long* nB,
                       const gw_z* TF, const gw_z* TFp, const gw_z* TB, const gw_z* TBp,
                       const double* w) {
  if (!c) return GW_ERR_ARG;
  if (!tau || !nF || !nB || !TF || !TFp || !TB || !TBp || !w) return fail(c, GW_ERR_ARG, "NULL table");
  const int nt = c->d.ntau, nwf = c->d.nw_f, nwb = c->d.nw_b;
  const double beta = c->d.beta;
  for (int i = 0; i < nt; ++i) {
    if (!std::isfinite(tau[i]) || !(tau[i] > 0.0) || !(tau[i] < beta))
      return fail(c, GW_ERR_ARG, "tau nodes must lie in (0, beta)");
    if (i > 0 && !(tau[i] > tau[i - 1])) return fail(c, GW_ERR_ARG, "tau nodes must increase");
    if (std::fabs(tau[nt - 1 - i] - (beta - tau[i])) > 1e-12 * beta)
      return fail(c, GW_ERR_ARG, "tau nodes must be mirrored: tau[ntau-1-i] = beta - tau[i]");
    if (!std::isfinite(w[i])) return fail(c, GW_ERR_ARG, "density row is not finite");
  }
  for (int n = 1; n < nwf; ++n)
    if (nF[n] <= nF[n - 1]) return fail(c, GW_ERR_ARG, "nF must be strictly increasing");
  for (int n = 1; n < nwb; ++n)
    if (nB[n] <= nB[n - 1]) return fail(c, GW_ERR_ARG, "nB must be strictly increasing");
  auto finite = [](const gw_z* a, size_t n) {
    for (size_t i = 0; i < n; ++i)
      if (!std::isfinite(a[i].re) || !std::isfinite(a[i].im)) return false;
    return true;
  };
  const size_t nfT = (size_t)nwf * nt, nbT = (size_t)nwb * nt;
  if (!finite(TF, nfT) || !finite(TFp, nfT) || !finite(TB, nbT) || !finite(TBp, nbT))
    return fail(c, GW_ERR_ARG, "transform table is not finite");
  HostGrids g;
  try {
    g.tau.assign(tau, tau + nt);
    g.x.resize(nt);
    for (int i = 0; i < nt; ++i) g.x[i] = 2.0 * tau[i] / beta - 1.0;
    g.w.assign(w, w + nt);
    g.nF.assign(nF, nF + nwf);
    g.nB.assign(nB, nB + nwb);
    auto cz = [](const gw_z* a, size_t n) {
      std::vector<gwgrid::cd> v(n);
      for (size_t i = 0; i < n; ++i) v[i] = gwgrid::cd(a[i].re, a[i].im);
      return v;
    };
    g.TF = cz(TF, nfT); g.TFp = cz(TFp, nfT); g.TB = cz(TB, nbT); g.TBp = cz(TBp, nbT);
    finish_grids(beta, g);
  } catch (const std::exception& e) {
    return fail(c, GW_ERR_ARG, e.what());
  }
  return install_grids(c, g);
}

// ------------------------------------------------ IR grids (Sec. IV.C) ---
static gw_status check_ir(double lambda, double eps) {
  if (!(lambda >= 1.0 && lambda <= 1e5) || !(eps >= 1e-14 && eps <= 1e-2)) return GW_ERR_ARG;
  return GW_OK;
}

gw_status gw_ir_size(double lambda, double eps, int* ntau) {
  if (!ntau || check_ir(lambda, eps) != GW_OK) return GW_ERR_ARG;
  try {
    *ntau = gwir::ir_size(lambda, eps);
  } catch (const std::exception&) {
    return GW_ERR_ARG;
  }
  return GW_OK;
}

static gw_status make_ir(double beta, double lambda, double eps, int ntau, HostGrids& g, std::string& why) {
  if (!(beta > 0.0) || !std::isfinite(beta) || check_ir(lambda, eps) != GW_OK) {
    why = "beta must be positive, lambda in 1..1e5 and eps in 1e-14..1e-2";
    return GW_ERR_ARG;
  }
  try {
    gwir::IRTables t;
    if (gwir::ir_size(lambda, eps) != ntau) {
      why = "ntau differs from the IR basis size (gw_ir_size)";
      return GW_ERR_ARG;
    }
    gwir::ir_grids(beta, lambda, eps, t);
    g.tau = t.tau; g.x = t.x; g.w = t.w; g.nF = t.nF; g.nB = t.nB;
    g.TF = t.TF; g.TFp = t.TFp; g.TB = t.TB; g.TBp = t.TBp;
    finish_grids(beta, g);
  } catch (const std::exception& e) {
    why = e.what();
    return GW_ERR_ARG;
  }
  return GW_OK;
}

gw_status gw_ir_grids_host(double beta, double lambda, double eps, int ntau, double* tau, long long* nF,
                           long long* nB, gw_z* TF, gw_z* TFp, gw_z* TB, gw_z* TBp, double* w) {
  HostGrids g;
  std::string why;
  gw_status s = make_ir(beta, lambda, eps, ntau, g, why);
  if (s != GW_OK) return s;
  if (tau) std::memcpy(tau, g.tau.data(), g.tau.size() * 8);
  if (nF) std::memcpy(nF, g.nF.data(), g.nF.size() * 8);
  if (nB) std::memcpy(nB, g.nB.data(), g.nB.size() * 8);
  if (TF) std::memcpy(TF, g.TF.data(), g.TF.size() * 16);
  if (TFp) std::memcpy(TFp, g.TFp.data(), g.TFp.size() * 16);
  if (TB) std::memcpy(TB, g.TB.data(), g.TB.size() * 16);
  if (TBp) std::memcpy(TBp, g.TBp.data(), g.TBp.size() * 16);
  if (w) std::memcpy(w, g.w.data(), g.w.size() * 8);
  return GW_OK;
}

gw_status gw_build_ir_grids(gw_ctx* c, double lambda, double eps) {
  if (!c) return GW_ERR_ARG;
  const int nt = c->d.ntau;
  if (c->d.nw_f != nt || c->d.nw_b != nt + 1)
    return fail(c, GW_ERR_ARG, "IR grids need nw_f = ntau and nw_b = ntau + 1");
  HostGrids g;
  std::string why;
  gw_status s = make_ir(c->d.beta, lambda, eps, nt, g, why);
  if (s != GW_OK) return fail(c, s, why);
  return install_grids(c, g);
}

gw_status gw_get_grids(const gw_ctx* cc, double* tau, long long* nF, long long* nB, gw_z* TF,
                       gw_z* TFp, gw_z* TB, gw_z* TBp, double* w) {
  gw_ctx* c = const_cast<gw_ctx*>(cc);
  if (!c) return GW_ERR_ARG;
  if (!c->grids) return fail(c, GW_ERR_STATE, "grids not built (gw_build_grids or gw_set_grids)");
  if (tau) std::memcpy(tau, c->tau.data(), c->tau.size() * 8);
  if (nF) std::memcpy(nF, c->nF.data(), c->nF.size() * 8);
  if (nB) std::memcpy(nB, c->nB.data(), c->nB.size() * 8);
  if (TF) std::memcpy(TF, c->TF.data(), c->TF.size() * 16);
  if (TFp) std::memcpy(TFp, c->TFp.data(), c->TFp.size() * 16);
  if (TB) std::memcpy(TB, c->TB.data(), c->TB.size() * 16);
  if (TBp) std::memcpy(TBp, c->TBp.data(), c->TBp.size() * 16);
  if (w) std::memcpy(w, c->w.data(), c->w.size() * 8);
  return GW_OK;
}

// Bytes of the polarization / self-energy chains for a tau chunk: two
// intermediates of tc x Nk x naux x nao^2 (plus complex64 copies of two G
// arrays in mixed precision).
// complex64 V and chain intermediates (GW_PREC_FP32, GW_PREC_BF16X3, GW_PREC_BF16X6)
static bool lowp(const gw_ctx* c) { return c->d.precision != GW_PREC_FP64; }
// split-bf16 operands of the two large contractions (GW_PREC_BF16X3, GW_PREC_BF16X6)
static bool splitbf(const gw_ctx* c) {
  return c->d.precision == GW_PREC_BF16X3 || c->d.precision == GW_PREC_BF16X6;
}
static int nsplit(const gw_ctx* c) { return c->d.precision == GW_PREC_BF16X6 ? 3 : 2; }
// Chain workspace: two tau-chunk regions (X and Zt, or Vt and L); in the
// low-precision modes two complex64 copies of G after them.
static size_t region_bytes(const gw_ctx* c, int tc) {
  return align256((size_t)tc * c->nk * c->sv * (lowp(c) ? 8 : 16));
}
static size_t gslot_bytes(const gw_ctx* c) { return align256((size_t)c->d.ntau * c->nk * c->n2 * 8); }

// complex64 P~ of one tau chunk (split mode, after the G copies)
static size_t pchunk_bytes(const gw_ctx* c, int tc) {
  return align256((size_t)tc * c->d.naux * (size_t)c->d.naux * 8);
}

static size_t chain_bytes(const gw_ctx* c, int tc) {
  return 2 * region_bytes(c, tc) + (lowp(c) ? 2 * gslot_bytes(c) : 0) + (splitbf(c) ? pchunk_bytes(c, tc) : 0);
}

static size_t screened_bytes(const gw_ctx* c, int nq) {
  return align256((size_t)nq * c->d.nw_b * c->d.naux * (size_t)c->d.naux * 16);
}

static size_t hf_bytes(const gw_ctx* c) {
  return align256((size_t)c->nk * c->sv * 16) + align256((size_t)c->nk * c->n2 * 16) +
         align256((size_t)c->d.naux * 16);
}

// Per-q polarization buffers of the whole-chain calls (gw_sigma per q,
// gw_sigma_jvp, gw_sigma_vjp): two tau arrays and four frequency arrays of
// naux^2 complex numbers, at the end of the workspace.
static size_t perq_tau_bytes(const gw_ctx* c) {
  return align256((size_t)c->d.ntau * c->d.naux * (size_t)c->d.naux * 16);
}
static size_t perq_w_bytes(const gw_ctx* c) { return screened_bytes(c, 1); }
static size_t perq_bytes(const gw_ctx* c) { return 2 * perq_tau_bytes(c) + 4 * perq_w_bytes(c); }

// Front region the sub-calls of the whole-chain calls use.
static size_t sigma_front_bytes(const gw_ctx* c, int tc) {
  return std::max({chain_bytes(c, tc), screened_bytes(c, 1), hf_bytes(c)});
}

size_t gw_workspace_bytes(const gw_ctx* c, int op, int tau_chunk) {
  if (!c) return 0;
  switch (op) {
    case GW_OP_DYSON_JVP:
      return 2 * align256((size_t)c->d.nw_f * c->nk * c->n2 * 16);
    case GW_OP_POLARIZATION:
    case GW_OP_SELF_ENERGY:
      if (tau_chunk < 1 || tau_chunk > c->d.ntau) return 0;
      return chain_bytes(c, tau_chunk);
    case GW_OP_SCREENED_W:
      if (tau_chunk < 1) return 0;
      return screened_bytes(c, tau_chunk);
    case GW_OP_HF:
      return hf_bytes(c);
    case GW_OP_SIGMA:
      if (tau_chunk < 1 || tau_chunk > c->d.ntau) return 0;
      return sigma_front_bytes(c, tau_chunk) + perq_bytes(c);
    case GW_OP_THERMO: {
      const size_t nb = (size_t)c->d.nw_f * c->nk;
      return align256(nb * c->n2 * 16) + 3 * align256(nb * 8) + align256((size_t)c->nk * c->n2 * 16) +
             align256((size_t)c->d.nw_f * 16) + align256((size_t)c->nk * 3 * 8);
    }
  }
  return 0;
}

gw_status gw_set_workspace(gw_ctx* c, void* dev, size_t bytes, int tau_chunk) {
  if (!c) return GW_ERR_ARG;
  if (tau_chunk < 1 || tau_chunk > c->d.ntau)
    return fail(c, GW_ERR_ARG, "tau_chunk must be in 1..ntau");
  if (bytes && !dev) return fail(c, GW_ERR_ARG, "workspace pointer is NULL");
  if (((uintptr_t)dev) & 255) return fail(c, GW_ERR_ARG, "workspace must be 256-byte aligned");
  c->ws = dev;
  c->ws_bytes = bytes;
  c->tc = tau_chunk;
  return GW_OK;
}

gw_status gw_mix(gw_ctx* c, long long n, double alpha, const gw_z* X, gw_z* Y, double* maxdiff) {
  if (!c) return GW_ERR_ARG;
  if (!Y || n < 0) return fail(c, GW_ERR_ARG, "bad gw_mix arguments");
  if (!std::isfinite(alpha)) return fail(c, GW_ERR_ARG, "alpha is not finite");
  if (n == 0) {
    if (maxdiff) *maxdiff = 0.0;
    return GW_OK;
  }
  // partial maxima reuse the electron-count scratch (nw_f * nk + 8 doubles)
  const int cap = c->d.nw_f * c->nk + 7;
  const int nblk = (int)std::max(1LL, std::min<long long>({(n + 255) / 256, 2048LL, (long long)cap - 1}));
  HIPCHK(c, mix_launch(n, alpha, (const double2*)X, (double2*)Y, maxdiff ? c->dpart : nullptr, nblk,
                       c->st));
  if (maxdiff) {
    HIPCHK(c, hipMemcpyAsync(maxdiff, c->dpart + nblk, sizeof(double), hipMemcpyDeviceToHost, c->st));
    HIPCHK(c, hipStreamSynchronize(c->st));
    if (!std::isfinite(*maxdiff)) return fail(c, GW_ERR_NONFINITE, "gw_mix: non-finite element");
  }
  return GW_OK;
}

gw_status gw_profile_enable(gw_ctx* c, int on) {
  if (!c) return GW_ERR_ARG;
  HIPCHK(c, hipStreamSynchronize(c->st));
  for (int k = 0; k < KC_COUNT; ++k) {
    for (auto& p : c->ev[k]) {
      (void)hipEventDestroy(p.first);
      (void)hipEventDestroy(p.second);
    }
    c->ev[k].clear();
    if (on) {
      c->launches[k] = 0;
      c->flops[k] = 0.0;
      c->ms[k] = 0.0;
    }
  }
  c->prof = on != 0;
  return GW_OK;
}

gw_status gw_profile_read(gw_ctx* c, int kc, long long* launches, double* ms, double* flops) {
  if (!c) return GW_ERR_ARG;
  if (kc < 0 || kc >= KC_COUNT) return fail(c, GW_ERR_ARG, "kernel class out of range");
  HIPCHK(c, hipStreamSynchronize(c->st));
  for (auto& p : c->ev[kc]) {
    float t = 0.0f;
    HIPCHK(c, hipEventElapsedTime(&t, p.first, p.second));
    c->ms[kc] += t;
    (void)hipEventDestroy(p.first);
    (void)hipEventDestroy(p.second);
  }
  c->ev[kc].clear();
  if (launches) *launches = c->launches[kc];
  if (ms) *ms = c->ms[kc];
  if (flops) *flops = c->flops[kc];
  return GW_OK;
}

gw_status gw_synchronize(gw_ctx* c) {
  if (!c) return GW_ERR_ARG;
  HIPCHK(c, hipStreamSynchronize(c->st));
  return GW_OK;
}

// ------------------------------------------------------------- Eq. tilde_P0_tau
// Mixed-precision context: V and the chain intermediates are complex64, G is
// rounded to complex64 once per call, the MFMAs run in fp32 and the long
// contractions add each 512-element chunk of their K sum into fp64.
static const int kMixedChunk = 512;

// Scratch of one chain call: base pointer, bytes and tau chunk (the
// context's workspace, or another region of device memory).
struct Work {
  char* base;
  size_t bytes;
  int tc;
};
static Work ctx_work(gw_ctx* c) { return Work{(char*)c->ws, c->ws_bytes, c->tc}; }

// complex64 copy of G in slot 0 or 1 of the mixed-precision workspace
static gw_status g_to_c64(gw_ctx* c, const Work& w, const gw_z* G, void** Gc, int slot = 0) {
  const size_t off = 2 * region_bytes(c, w.tc) + (size_t)slot * gslot_bytes(c);
  *Gc = w.base + off;
  HIPCHK(c, to_c64_launch((const double2*)G, (float2*)*Gc, (long long)c->d.ntau * c->nk * c->n2, c->st));
  return GW_OK;
}

static gw_status pol_impl(gw_ctx* c, const Work& w, const void* V, const gw_z* G, const gw_z* Gb,
                          int q0, int nq, gw_z* P0, bool accumulate, bool two_slot);

gw_status gw_set_hermitian(gw_ctx* c, int mode) {
  if (!c) return GW_ERR_ARG;
  if (mode & ~(GW_HERM_FORWARD | GW_HERM_TWO_SLOT)) return fail(c, GW_ERR_ARG, "unknown Hermitian-mode bits");
  c->herm = mode;
  return GW_OK;
}

gw_status gw_set_mu_window(gw_ctx* c, double ne_tol) {
  if (!c) return GW_ERR_ARG;
  if (!std::isfinite(ne_tol) || ne_tol < 0.0) return fail(c, GW_ERR_ARG, "ne_tol must be finite and >= 0");
  c->mu_window = ne_tol;
  return GW_OK;
}

gw_status gw_polarization(gw_ctx* c, const void* V, const gw_z* G, int q0, int nq, gw_z* P0) {
  if (!c) return GW_ERR_ARG;
  return pol_impl(c, ctx_work(c), V, G, G, q0, nq, P0, false, false);
}

gw_status gw_polarization2(gw_ctx* c, const void* V, const gw_z* Ga, const gw_z* Gb, int q0, int nq,
                           int accumulate, gw_z* P0) {
  if (!c) return GW_ERR_ARG;
  return pol_impl(c, ctx_work(c), V, Ga, Gb, q0, nq, P0, accumulate != 0, true);
}

// gw_polarization on the fixed scratch array instead of the caller's
// workspace: the largest tau chunk whose intermediates fit is used.  Makes
// no allocation (profiling events are not recorded during the call).
gw_status gw_polarization_noalloc(gw_ctx* c, const void* V, const gw_z* G, int q0, int nq, gw_z* P0) {
  if (!c) return GW_ERR_ARG;
  if (!c->scratch) return fail(c, GW_ERR_DEVICE, "scratch address not set up");
  int tc = 0;
  for (int t = c->d.ntau; t >= 1; t = (t == 1) ? 0 : (t + 1) / 2)
    if (chain_bytes(c, t) <= kScratchBytes) { tc = t; break; }
  if (tc == 0)
    return fail(c, GW_ERR_WORKSPACE,
                "gw_polarization_noalloc: one tau slice of the intermediates needs " +
                    std::to_string(chain_bytes(c, 1)) + " bytes, above the fixed scratch of " +
                    std::to_string(kScratchBytes) + " bytes");
  const bool prof = c->prof;
  c->prof = false;
  const gw_status s = pol_impl(c, Work{c->scratch, kScratchBytes, tc}, V, G, G, q0, nq, P0, false, false);
  c->prof = prof;
  return s;
}

// One tau chunk of Eq. tilde_P0_tau in the split-bf16 modes (GW_PREC_BF16X3 / X6).
// The complex64 producers write X and Zt with K = (k, d, b) contiguous per
// row, so that the contraction's loader reads whole K-runs:
//   X2[tl][Q][k n2 + d nao + b]  = sum_a V[q][k][Q][d][a] G[t0+tl][k+q][a][b]
//   Z2[tl][Q'][k n2 + d nao + b] = sum_c G[nt-1-t0-tl][k][c][d] conj(V[q][k][Q'][c][b])
//   P0[iq][t0+tl][Q][Q'] (+)= -(ns/nk) sum_K X2[tl][Q][K] Z2[tl][Q'][K]   (bf16x3)
// Gd and Gbd are the complex64 copies of the two G slots.
static gw_status pol_split_chunk(gw_ctx* c, const char* Aq, const char* Gd, const char* Gbd, char* X, char* Z,
                                 int q, int iq, int t0, int tcur, int tc, gw_z* P0, bool accumulate,
                                 bool herm) {
  const int nk = c->nk, nao = c->d.nao, naux = c->d.naux, nt = c->d.ntau;
  const long long n2 = c->n2, sv = c->sv;
  const long long K = (long long)nk * n2, ldr = (long long)naux * K;
  GemmDesc g = gemm_desc();
  g.A = Aq; g.B = Gd + (size_t)t0 * nk * n2 * 8; g.C = X;
  g.M = naux * nao; g.N = tcur * nao; g.K = nao; g.batch = nk;
  g.am = aff(nao); g.ak = aff(1);
  g.bk = aff(nao); g.bn = two(nao, 1, (long long)nk * n2);
  g.cm = two(nao, nao, K); g.cn = two(nao, 1, ldr);
  g.ba = aff(sv); g.bb = aff(0); g.bc = aff(n2);
  g.tab = c->dplus + (size_t)q * nk; g.tmod = nk; g.tsB = n2;   // G^{k+q}
  g.ta = g.tb = g.tc = 1; g.f32 = 1;
  g.tag = KC_POL_PRODUCER;
  gw_status s = run(c, g, Ext{0, (long long)nk * sv}, Ext{0, (long long)tcur * nk * n2}, Ext{0, (long long)tc * ldr});
  if (s != GW_OK) return s;
  g = gemm_desc();
  // rows over tr = tcur-1-tl: G read with a positive stride (uniform-K loop)
  g.A = Gbd + (size_t)(nt - t0 - tcur) * nk * n2 * 8; g.B = Aq; g.C = Z + (size_t)(tcur - 1) * ldr * 8;
  g.M = tcur * nao; g.N = naux * nao; g.K = nao; g.batch = nk;
  g.am = two(nao, 1, (long long)nk * n2); g.ak = aff(nao);
  g.bk = aff(nao); g.bn = two(nao, 1, n2); g.conjB = 1;
  g.cm = two(nao, nao, -ldr); g.cn = two(nao, 1, K);
  g.ba = aff(n2); g.bb = aff(sv); g.bc = aff(n2);
  g.ta = g.tb = g.tc = 1; g.f32 = 1;
  g.tag = KC_POL_PRODUCER;
  if ((s = run(c, g, Ext{0, (long long)tcur * nk * n2}, Ext{0, (long long)nk * sv},
               Ext{-(long long)(tcur - 1) * ldr, (long long)(tc - tcur + 1) * ldr})) != GW_OK)
    return s;
  SplitDesc d = split_desc();
  d.A = X; d.B = Z; d.C = (double2*)P0 + ((long long)iq * nt + t0) * naux * naux;
  d.M = naux; d.N = naux; d.K = (int)K; d.batch = tcur;
  d.ta = d.tb = 1; d.tc = 0;
  d.am = aff(K); d.aks = 1; d.bn = aff(K); d.bks = 1;
  d.ba = d.bb = aff(ldr); d.bc = aff((long long)naux * naux);
  d.cm = aff(naux); d.cn = aff(1);
  d.alpha_r = -(double)c->d.ns / nk;
  if (accumulate) { d.beta_zero = 0; d.beta_r = 1.0; }
  d.tri = herm ? 1 : 0; d.kchunk = kMixedChunk; d.nsplit = nsplit(c);
  d.tag = KC_POL_CONTRACT;
  if ((s = run_split(c, d, Ext{0, (long long)tcur * ldr}, Ext{0, (long long)tcur * ldr},
                     Ext{0, (long long)tcur * naux * naux})) != GW_OK)
    return s;
  return GW_OK;
}

// The tau nodes [tb, te) of P0^q, written to P0, the [ntau][naux][naux] array
// of this q, and with M0 the mirrored nodes M0[ntau-1-i] = P0[i]^T of -q; Gd
// and Gbd are the two G slots in the chain's storage type.  herm: P0 is
// Hermitian, and only its upper half is contracted.  fp64: Gd2 and Gbd2 (may
// be NULL) are a second pair of slots, added to the first one's term before
// the long contraction.
static gw_status pol_nodes(gw_ctx* c, const Work& w, const char* Vd, const char* Gd, const char* Gbd, int q,
                           int tb, int te, gw_z* P0, gw_z* M0, bool accumulate, bool herm,
                           const char* Gd2 = nullptr, const char* Gbd2 = nullptr);

// Completes the nodes [tb, te) of one q: the lower triangle in Hermitian
// mode, and with M0 the mirrored nodes M0[ntau-1-i] = P0[i]^T of -q.
static gw_status pol_finish(gw_ctx* c, gw_z* P0, gw_z* M0, int tb, int te, bool herm) {
  if (!herm && !M0) return GW_OK;
  const long long nn = (long long)c->d.naux * c->d.naux;
  double2* src = (double2*)P0 + tb * nn;
  double2* dst = M0 ? (double2*)M0 + (long long)(c->d.ntau - 1 - tb) * nn : nullptr;
  HIPCHK(c, mirror_launch(src, dst, -nn, c->d.naux, te - tb, herm, c->st));
  return GW_OK;
}

// G fills the tau slot (G^{k+q}(tau_i)), Gb the mirrored slot (G^k(tau_{ntau-1-i})).
static gw_status pol_impl(gw_ctx* c, const Work& w, const void* V, const gw_z* G, const gw_z* Gb,
                          int q0, int nq, gw_z* P0, bool accumulate, bool two_slot) {
  if (!c) return GW_ERR_ARG;
  if (!ready(c)) return fail(c, GW_ERR_STATE, "grids not built");
  if (q0 < 0 || nq < 0 || q0 + nq > c->nk) return fail(c, GW_ERR_ARG, "q range outside the mesh");
  if (nq == 0) return GW_OK;
  if (!V || !G || !Gb || !P0) return fail(c, GW_ERR_ARG, "NULL array");
  const int tc = w.tc;
  if (!w.base || tc < 1 || tc > c->d.ntau || w.bytes < chain_bytes(c, tc))
    return fail(c, GW_ERR_WORKSPACE, "polarization workspace too small");
  const bool f32 = lowp(c);
  const char* Gd = (const char*)G;
  const char* Gbd = (const char*)Gb;
  if (f32) {
    void* Gc = nullptr;
    gw_status s = g_to_c64(c, w, G, &Gc);
    if (s != GW_OK) return s;
    Gd = Gbd = (const char*)Gc;
    if (Gb != G) {
      if ((s = g_to_c64(c, w, Gb, &Gc, 1)) != GW_OK) return s;
      Gbd = (const char*)Gc;
    }
  }
  // P0^q(tau) is Hermitian when G^k(tau) is and V^{k+q,k}(Q) = V^{k,k+q}(Q)^H,
  // and so is each two-slot term P0[Ga, Gb] for Hermitian Ga, Gb: then only
  // the tiles on and above the diagonal are contracted (accumulating into an
  // upper triangle and refilling the lower one keeps a Hermitian sum).
  const bool herm = (c->herm & (two_slot ? GW_HERM_TWO_SLOT : GW_HERM_FORWARD)) != 0;
  // With k -> k + q, the cyclic trace and the pair relation of V, Eq.
  // tilde_P0_tau with one G in both slots gives P0^{-q}(beta - tau) =
  // P0^q(tau)^T (nodes mirror each other), for any G.  So of two q-points q
  // and -q in the range only the first is contracted, and of a q = -q only
  // the lower half of the nodes; the rest are transposed copies.  fp64 only:
  // in the complex64 modes the other order of the sum over (k, a, b) would
  // move P0 by its own rounding (1e-8 relative).  Measured, whole evaluation
  // on a 3x3x3 mesh: 129 -> 99 ms (nao 16, naux 150, ntau 60) and 918 -> 721
  // ms (nao 26, naux 250, ntau 100).
  const bool pair = !f32 && !accumulate && !two_slot;
  const int nt = c->d.ntau;
  const long long per = (long long)nt * c->d.naux * c->d.naux;
  for (int q = q0; q < q0 + nq; ++q) {
    const int m = c->neg[q];
    const bool has = pair && m >= q0 && m < q0 + nq;
    if (has && m < q) continue;
    const int te = has && m == q ? nt / 2 : nt;
    gw_z* Pq = P0 + (q - q0) * per;
    gw_status s = pol_nodes(c, w, (const char*)V, Gd, Gbd, q, 0, te, Pq, has ? P0 + (m - q0) * per : nullptr,
                            accumulate, herm);
    if (s != GW_OK) return s;
  }
  return GW_OK;
}

// P[tl][Q][Q'] = alpha sum_{k,e} Y[tl][k][Q][e] conj(V[k][Q'][e]) of tcur nodes
// (added to P with accumulate), completed as pol_finish does; Z has room for
// the Y of tc nodes.  P and M lie in the arrays Pa and Ma.
static gw_status pol_contract(gw_ctx* c, const char* Y, char* Z, const char* Vq, int tcur, int tc, double2* P,
                              double2* M, double alpha, bool accumulate, bool herm, Arr Pa, Arr Ma) {
  const int nk = c->nk, naux = c->d.naux;
  const long long n2 = c->n2, sv = c->sv, S = (long long)nk * sv, nn = (long long)naux * naux;
  const long long room = (long long)tc * S;
  const double outs = herm ? 0.5 * naux * (naux + 1.0) : (double)nn;
  if (n2 >= 4 && c->tile_cfg < 0 && room >= tcur * pol_acc_blocks(naux, herm) * 256) {
    PolAcc a{};
    a.Y = (const double2*)Y; a.V = (const double2*)Vq;
    a.P = P; a.M = M; a.part = (double2*)Z;
    a.nt = tcur; a.naux = naux; a.n2 = (int)n2; a.K = nk * (int)n2;
    a.tsY = S; a.sv = sv; a.tri = herm; a.accumulate = accumulate;
    a.alpha = alpha;
    hipEvent_t e0 = nullptr;
    gw_status s;
    if (c->check_bounds &&
        (s = leaves(c, "pol_acc", pol_acc_leaves(a, room, Arr{Y, tcur * S}, Arr{Vq, S}, Pa, Ma, Arr{Z, room}))) != GW_OK)
      return s;
    if ((s = prof_begin(c, KC_POL_CONTRACT, &e0)) != GW_OK) return s;
    HIPCHK(c, pol_acc_launch(a, room, c->st));
    return prof_end(c, KC_POL_CONTRACT, e0, 6.0 * outs * a.K * tcur);
  }
  // matrices of one orbital, a chunk without room for the partial sums, or a
  // tile configuration asked for
  GemmDesc g = gemm_desc();
  g.A = Y; g.B = Vq; g.C = P;
  g.M = naux; g.N = naux; g.K = nk * (int)n2; g.batch = tcur;
  g.am = aff(n2); g.ak = two((unsigned)n2, 1, sv);
  g.bk = two((unsigned)n2, 1, sv); g.bn = aff(n2); g.conjB = 1;
  g.cm = aff(naux); g.cn = aff(1);
  g.ba = aff(S); g.bb = aff(0); g.bc = aff(nn);
  g.alpha_r = alpha;
  if (accumulate) { g.beta_zero = 0; g.beta_r = 1.0; }
  g.tri = herm ? 1 : 0;
  g.tag = KC_POL_CONTRACT;
  gw_status s = run(c, g, Ext{0, (long long)tcur * S}, Ext{0, S}, Ext{0, (long long)tcur * nn});
  if (s != GW_OK || (!herm && !M)) return s;
  HIPCHK(c, mirror_launch(P, M, -nn, naux, tcur, herm, c->st));
  return GW_OK;
}

static gw_status pol_nodes(gw_ctx* c, const Work& w, const char* Vd, const char* Gd, const char* Gbd, int q,
                           int tb, int te, gw_z* P0, gw_z* M0, bool accumulate, bool herm, const char* Gd2,
                           const char* Gbd2) {
  const int tc = w.tc;
  const int nk = c->nk, nao = c->d.nao, naux = c->d.naux, nt = c->d.ntau;
  const long long n2 = c->n2, sv = c->sv;
  const long long S = (long long)nk * sv;                // one tau slice of X or Zt
  const bool f32 = lowp(c);
  const bool sb = splitbf(c);
  const size_t ez = f32 ? 8 : 16;                        // bytes of V / X / Zt / G elements
  char* X = w.base;
  char* Z = w.base + region_bytes(c, tc);
  const char* Aq = Vd + (size_t)q * nk * sv * ez;
  for (int t0 = tb; t0 < te; t0 += tc) {
    const int tcur = std::min(tc, te - t0);
    if (sb) {
      gw_status s = pol_split_chunk(c, Aq, Gd, Gbd, X, Z, q, 0, t0, tcur, tc, P0, accumulate, herm);
      if (s != GW_OK) return s;
      continue;
    }
    if (!f32) {
      // Y[tl][k][Q][c][b] = sum_{d,a} Gb[nt-1-t0-tl][k][c][d] V[q][k][Q][d][a] G[t0+tl][k+q][a][b]
      // P0[t0+tl][Q][Q'] = -(ns/nk) sum_{k,c,b} Y[tl][k][Q][c][b] conj(V[q][k][Q'][c][b])
      // Both G on one side: one tau array is written and read instead of two
      // (V G and Gb conj(V)), and the other operand is the V slab that every
      // tau shares.
      const long long gs = (long long)nk * n2;
      SandProd p{};
      p.V = (const double2*)Aq; p.Y = (double2*)X; p.tab = c->dplus + (size_t)q * nk;
      p.nt = tcur; p.tsY = S; p.tabR = 1; p.tsL = -gs; p.tsR = gs;
      p.L = (const double2*)Gbd + (nt - 1 - t0) * gs;
      p.R = (const double2*)Gd + t0 * gs;
      const Arr slab{Aq, S}, y{X, tc * S};
      gw_status s = sand_prod(c, p, KC_POL_PRODUCER, slab, Arr{Gbd, nt * gs}, Arr{Gd, nt * gs}, y);
      if (s != GW_OK) return s;
      if (Gd2) {
        p.L = (const double2*)Gbd2 + (nt - 1 - t0) * gs;
        p.R = (const double2*)Gd2 + t0 * gs;
        p.accumulate = 1;
        if ((s = sand_prod(c, p, KC_POL_PRODUCER, slab, Arr{Gbd2, nt * gs}, Arr{Gd2, nt * gs}, y)) != GW_OK) return s;
      }
      const long long nn = (long long)naux * naux;
      if ((s = pol_contract(c, X, Z, Aq, tcur, tc, (double2*)P0 + t0 * nn,
                            M0 ? (double2*)M0 + (nt - 1 - t0) * nn : nullptr, -(double)c->d.ns / nk, accumulate,
                            herm, Arr{P0, nt * nn}, Arr{M0, nt * nn})) != GW_OK) return s;
      continue;
    }
    // X[tl][k][Q][d][b] = sum_a V[q][k][Q][d][a] G[t0+tl][k+q][a][b]
    GemmDesc g = gemm_desc();
    g.A = Aq; g.B = Gd + (size_t)t0 * nk * n2 * ez; g.C = X;
    g.M = naux * nao; g.N = tcur * nao; g.K = nao; g.batch = nk;
    g.am = aff(nao); g.ak = aff(1);
    g.bk = aff(nao); g.bn = two(nao, 1, (long long)nk * n2);
    g.cm = aff(nao); g.cn = two(nao, 1, S);
    g.ba = aff(sv); g.bb = aff(0); g.bc = aff(sv);
    g.tab = c->dplus + (size_t)q * nk; g.tmod = nk; g.tsB = n2;   // G^{k+q}
    g.ta = g.tb = g.tc = g.f32 = 1;
    g.tag = KC_POL_PRODUCER;
    gw_status s = run(c, g, Ext{0, (long long)nk * sv}, Ext{0, (long long)tcur * nk * n2}, Ext{0, (long long)tc * S});
    if (s != GW_OK) return s;
    // Zt[tl][k][Q'][d][b] = sum_c G[nt-1-t0-tl][k][c][d] conj(V[q][k][Q'][c][b])
    // Rows run over tr = tcur-1-tl, so that G is read with a positive
    // stride (the uniform-K loop needs non-negative operand strides) and
    // the rows are written backwards.
    g = gemm_desc();
    g.A = Gbd + (size_t)(nt - t0 - tcur) * nk * n2 * ez; g.B = Aq;
    g.C = Z + (size_t)(tcur - 1) * S * ez;
    g.M = tcur * nao; g.N = naux * nao; g.K = nao; g.batch = nk;
    g.am = two(nao, 1, (long long)nk * n2); g.ak = aff(nao);
    g.bk = aff(nao); g.bn = two(nao, 1, n2); g.conjB = 1;
    g.cm = two(nao, nao, -S); g.cn = two(nao, 1, n2);
    g.ba = aff(n2); g.bb = aff(sv); g.bc = aff(sv);
    g.ta = g.tb = g.tc = g.f32 = 1;
    g.tag = KC_POL_PRODUCER;
    if ((s = run(c, g, Ext{0, (long long)tcur * nk * n2}, Ext{0, (long long)nk * sv},
                 Ext{-(long long)(tcur - 1) * S, (long long)(tc - tcur + 1) * S})) != GW_OK) return s;
    // P0[t0+tl][Q][Q'] = -(ns/nk) sum_{k,e} X[tl][k][Q][e] Zt[tl][k][Q'][e]
    g = gemm_desc();
    g.A = X; g.B = Z; g.C = (double2*)P0 + (long long)t0 * naux * naux;
    g.M = naux; g.N = naux; g.K = nk * (int)n2; g.batch = tcur;
    g.am = aff(n2); g.ak = two((unsigned)n2, 1, sv);
    g.bk = two((unsigned)n2, 1, sv); g.bn = aff(n2);
    g.cm = aff(naux); g.cn = aff(1);
    g.ba = aff(S); g.bb = aff(S); g.bc = aff((long long)naux * naux);
    g.alpha_r = -(double)c->d.ns / nk;
    if (accumulate) { g.beta_zero = 0; g.beta_r = 1.0; }
    g.ta = g.tb = g.f32 = 1; g.tc = 0; g.kchunk = kMixedChunk;
    g.tag = KC_POL_CONTRACT;
    g.tri = herm ? 1 : 0;
    if ((s = run(c, g, Ext{0, (long long)tcur * S}, Ext{0, (long long)tcur * S}, Ext{0, (long long)tcur * naux * naux})) != GW_OK) return s;
  }
  return f32 ? pol_finish(c, P0, M0, tb, te, herm) : GW_OK;
}

// ------------------------------------------------------------- transforms
static gw_status transform(gw_ctx* c, int stat, const gw_z* Xin, long long batch, long long R,
                           gw_z* Xout, bool forward) {
  if (!c) return GW_ERR_ARG;
  if (!ready(c)) return fail(c, GW_ERR_STATE, "grids not built (gw_build_grids or gw_set_grids)");
  if (stat != GW_FERMION && stat != GW_BOSON) return fail(c, GW_ERR_ARG, "stat must be 0 or 1");
  if (batch < 0 || R < 0 || batch > 65535 || R > 0x7fffffffLL)
    return fail(c, GW_ERR_ARG, "batch or R out of range");
  if (batch == 0 || R == 0) return GW_OK;
  if (!Xin || !Xout) return fail(c, GW_ERR_ARG, "NULL array");
  const int nt = c->d.ntau;
  const int nw = stat == GW_FERMION ? c->d.nw_f : c->d.nw_b;
  const int rows = forward ? nw : nt, inner = forward ? nt : nw;
  GemmDesc g = gemm_desc();
  g.A = forward ? (stat == GW_FERMION ? c->dTF : c->dTB) : (stat == GW_FERMION ? c->dTFp : c->dTBp);
  g.B = (const double2*)Xin;
  g.C = (double2*)Xout;
  g.M = rows; g.N = (int)R; g.K = inner; g.batch = (int)batch;
  g.am = aff(inner); g.ak = aff(1);
  g.bk = aff(R); g.bn = aff(1);
  g.cm = aff(R); g.cn = aff(1);
  g.ba = aff(0); g.bb = aff((long long)inner * R); g.bc = aff((long long)rows * R);
  g.tag = KC_TRANSFORM;
  return run(c, g, Ext{0, (long long)rows * inner}, Ext{0, batch * inner * R}, Ext{0, batch * rows * R});
}

gw_status gw_tau_to_iw(gw_ctx* c, int stat, const gw_z* X_tau, long long batch, long long R,
                       gw_z* X_iw) {
  return transform(c, stat, X_tau, batch, R, X_iw, true);
}

gw_status gw_iw_to_tau(gw_ctx* c, int stat, const gw_z* X_iw, long long batch, long long R,
                       gw_z* X_tau) {
  return transform(c, stat, X_iw, batch, R, X_tau, false);
}

// ------------------------------------------------------------- Eq. tilde_P_omega
// Pt = (I - P0)^{-1} P0 of nmat matrices, whose LU factors stay in the
// workspace; matrix b of P0 and Pt is at position sel[b] (device table; b
// itself if NULL).
static gw_status solve_core(gw_ctx* c, const gw_z* P0, gw_z* Pt, const int* sel, long long nmat) {
  HIPCHK(c, zero_flag_launch(c->dflag, c->st));
  hipEvent_t e0 = nullptr;
  gw_status s = prof_begin(c, KC_WDYSON, &e0);
  if (s != GW_OK) return s;
  // Blocked right-looking LU with row pivoting inside each panel of kNb
  // columns; the trailing updates of A and of the right-hand side and the
  // blocked back substitution are batched GEMMs over all nq * nw_b matrices.
  const int n = c->d.naux, kNb = 32;
  const long long nn = (long long)n * n;
  double2* Am = (double2*)c->ws;
  double2* Bm = (double2*)Pt;
  if (c->check_bounds) {
    // the panel kernels take every matrix of A, and of P0 and Pt by position
    if ((size_t)nmat * nn * 16 > c->ws_bytes) return leaves(c, "solve", "A");
    if (sel && (sel < c->dsel || sel + nmat > c->dsel + c->sel.size())) return leaves(c, "solve", "table");
    for (long long b = 0; sel && b < nmat; ++b) {
      const int at = c->sel[(sel - c->dsel) + b];
      if (at < 0 || at >= c->nk * c->d.nw_b) return leaves(c, "solve", "B");
    }
  }
  HIPCHK(c, wlu_launch(0, (const double2*)P0, Am, Bm, sel, n, 0, kNb, nmat, c->dflag, c->st));
  auto gemm = [&](double2* X, long long xo, double2* Y, long long yo, double2* Z, long long zo, int M,
                  int N, int K) -> gw_status {
    if (M <= 0 || N <= 0 || K <= 0) return GW_OK;
    GemmDesc g = gemm_desc();
    g.A = X + xo; g.B = Y + yo; g.C = Z + zo;
    g.M = M; g.N = N; g.K = K; g.batch = (int)nmat;
    g.am = aff(n); g.ak = aff(1); g.bk = aff(n); g.bn = aff(1); g.cm = aff(n); g.cn = aff(1);
    g.ba = g.bb = g.bc = aff(nn);
    if (sel) {                        // matrices of B by position
      g.tab = sel; g.tmod = (int)nmat;
      if (Y == Bm) { g.bb = aff(0); g.tsB = nn; }
      if (Z == Bm) { g.bc = aff(0); g.tsC = nn; }
    }
    g.alpha_r = -1.0; g.beta_zero = 0; g.beta_r = 1.0;
    g.tag = KC_OTHER;                 // timed as part of the whole solve (KC_WDYSON)
    const long long span = nmat * nn, all = sel ? (long long)c->nk * c->d.nw_b * nn : span;
    return run(c, g, Ext{-xo, span - xo}, Ext{-yo, (Y == Bm ? all : span) - yo}, Ext{-zo, (Z == Bm ? all : span) - zo});
  };
  for (int j0 = 0; j0 < n;) {
    // Two panels per trailing update where both are register-resident: the
    // update reads and writes all of the trailing A and B and is bound by that
    // (404 matrices of order 250, with the back substitution by pairs of blocks:
    // 4.04 -> 3.30 ms)
    // (2624 matrices of order 4: 62 us a solve on the general panel, 70 on the
    // register-resident one, whose start costs more than so few columns)
    const bool small = n > 8 && n - j0 <= 512, two = small && n - j0 > 2 * kNb;
    const int j1 = std::min(j0 + (two ? 2 : 1) * kNb, n), w = j1 - j0, rest = n - j1;
    if (small) {
      HIPCHK(c, wlu_factor_launch(Am, Bm, sel, n, j0, false, nmat, c->dflag, c->st));
    } else {
      HIPCHK(c, wlu_launch(1, nullptr, Am, Bm, sel, n, j0, kNb, nmat, c->dflag, c->st));
      HIPCHK(c, wlu_launch(2, nullptr, Am, Bm, sel, n, j0, kNb, nmat, c->dflag, c->st));
    }
    if (two) {
      const int jm = j0 + kNb;
      // the second panel -= L21 U12 of the first
      if ((s = gemm(Am, (long long)jm * n + j0, Am, (long long)j0 * n + jm, Am, (long long)jm * n + jm, n - jm, kNb,
                    kNb)) != GW_OK) return s;
      HIPCHK(c, wlu_factor_launch(Am, Bm, sel, n, jm, true, nmat, c->dflag, c->st));
    }
    // A22 -= L21 U12 ;  B2 -= L21 B1
    if ((s = gemm(Am, (long long)j1 * n + j0, Am, (long long)j0 * n + j1, Am, (long long)j1 * n + j1,
                  rest, rest, w)) != GW_OK) return s;
    if ((s = gemm(Am, (long long)j1 * n + j0, Bm, (long long)j0 * n, Bm, (long long)j1 * n,
                  rest, n, w)) != GW_OK) return s;
    j0 = j1;
  }
  const int nblk = (n + kNb - 1) / kNb;
  // back substitution, two blocks per update of the rows above them
  for (int b = nblk - 1; b >= 0; b -= 2) {
    const int j0 = b * kNb, w = std::min(kNb, n - j0);
    HIPCHK(c, wlu_back_launch(Am, Bm, sel, n, j0, nmat, c->st));
    if (b == 0) break;
    // the block above: B[jm:j0] -= U[jm:j0, j0:j0+w] B[j0:j0+w], then solved
    const int jm = j0 - kNb;
    if ((s = gemm(Am, (long long)jm * n + j0, Bm, (long long)j0 * n, Bm, (long long)jm * n, kNb, n, w)) != GW_OK) return s;
    HIPCHK(c, wlu_back_launch(Am, Bm, sel, n, jm, nmat, c->st));
    // B[0:jm] -= U[0:jm, jm:j0+w] B[jm:j0+w]
    if ((s = gemm(Am, (long long)jm, Bm, (long long)jm * n, Bm, 0, jm, n, kNb + w)) != GW_OK) return s;
  }
  const double nd = n;
  if ((s = prof_end(c, KC_WDYSON, e0, (32.0 / 3.0) * nd * nd * nd * nmat)) != GW_OK) return s;
  return read_flag(c, "screened_W");
}

gw_status gw_screened_W(gw_ctx* c, const gw_z* P0, int nq, gw_z* Pt) {
  if (!c) return GW_ERR_ARG;
  if (!ready(c)) return fail(c, GW_ERR_STATE, "grids not built (gw_build_grids or gw_set_grids)");
  if (nq < 0 || nq > c->nk) return fail(c, GW_ERR_ARG, "nq out of range");
  if (nq == 0) return GW_OK;
  if (!P0 || !Pt) return fail(c, GW_ERR_ARG, "NULL array");
  if (P0 == Pt) return fail(c, GW_ERR_ARG, "Pt_iw may not alias P0_iw");
  if (!c->ws || c->ws_bytes < gw_workspace_bytes(c, GW_OP_SCREENED_W, nq))
    return fail(c, GW_ERR_WORKSPACE, "screened_W workspace too small");
  return solve_core(c, P0, Pt, nullptr, (long long)nq * c->d.nw_b);
}

// ------------------------------------------------------ Eq. tilde_Phi_GW
gw_status gw_screened_W_phi(gw_ctx* c, const gw_z* P0, int nq, gw_z* Pt, double* phi) {
  if (!c) return GW_ERR_ARG;
  if (!phi) return fail(c, GW_ERR_ARG, "NULL phi");
  *phi = 0.0;
  gw_status s = gw_screened_W(c, P0, nq, Pt);
  if (s != GW_OK || nq == 0) return s;
  // The LU of I - P0 is still packed in the workspace.  Weights of the
  // Matsubara sum: value at tau = 0 of the least-squares fit, i.e. the
  // beta^- row reversed (mirrored nodes) times TBp; real part, scaled by
  // 1 / (2 Nk).  dred[1..nw_b] holds the weights, dphi the per-matrix terms
  // and, after them, their sum.
  const int nt = c->d.ntau, nwb = c->d.nw_b;
  if (nwb + 1 > 2 * 1024 + 8) return fail(c, GW_ERR_ARG, "gw_screened_W_phi supports nw_b <= 2055");
  std::vector<double> up((size_t)nwb + 1, 0.0);
  for (int n = 0; n < nwb; ++n) {
    double r = 0.0;
    for (int i = 0; i < nt; ++i) r += c->w[nt - 1 - i] * c->TBp[(size_t)i * nwb + n].real();
    up[1 + n] = r / (2.0 * c->nk);
  }
  HIPCHK(c, hipMemcpyAsync(c->dred, up.data(), up.size() * sizeof(double), hipMemcpyHostToDevice, c->st));
  const long long nmat = (long long)nq * nwb;
  HIPCHK(c, phi_terms_launch((const double2*)c->ws, (const double2*)P0, c->d.naux, nmat, c->dred + 1,
                             nwb, c->dphi, c->dphi + nmat, c->st));
  HIPCHK(c, hipMemcpyAsync(phi, c->dphi + nmat, sizeof(double), hipMemcpyDeviceToHost, c->st));
  HIPCHK(c, hipStreamSynchronize(c->st));
  return GW_OK;
}

// ------------------------------------------------------------- Eq. tilde_sigma2
// Vt[tl][Q][k][b][j] = sum_Q' M[tl][Q][Q'] V[k][Q'][b][j] for n nodes (M^H
// with adjoint): the long contraction of the self-energy and of the adjoints.
static gw_status times_v(gw_ctx* c, const gw_z* M, const gw_z* Vq, char* Vt, int n, bool adjoint) {
  const int nk = c->nk, naux = c->d.naux;
  const long long n2 = c->n2, sv = c->sv, S = (long long)nk * sv;
  GemmDesc g = gemm_desc();
  g.A = M; g.B = Vq; g.C = Vt;
  g.M = naux; g.N = nk * (int)n2; g.K = naux; g.batch = n;
  if (adjoint) { g.am = aff(1); g.ak = aff(naux); g.conjA = 1; } else { g.am = aff(naux); g.ak = aff(1); }
  g.bk = aff(n2); g.bn = two((unsigned)n2, 1, sv);
  g.cm = aff((long long)nk * n2); g.cn = aff(1);
  g.ba = aff((long long)naux * naux); g.bb = aff(0); g.bc = aff(S);
  // groups of 8 tiles walk every tau: their V tiles and each tau's M
  // panels stay in L2 (measured at si-4x4x4: fetch 49 -> 29 GB per q,
  // 25.6 vs 25.9 ms; groups of 16: 21 GB, 26.1 ms)
  g.batch_fastest = 2;
  g.group = 8;
  g.tag = KC_SE_CONTRACT;
  return run(c, g, Ext{0, (long long)n * naux * naux}, Ext{0, S}, Ext{0, (long long)n * S});
}

// Contribution of one q at the tau nodes [tb, te); Gd is G in the chain's
// storage type, Pt the [ntau][naux][naux] array of this q.
// mirror (fp64): also the contribution of -q at the mirrored nodes, for P~ with
// P~^{-q}(beta - tau) = P~^q(tau)^T = conj(P~^q(tau)) (P~ of a Hermitian G).
// With V^{k+q,k} = V^{k,k+q}^H the long contraction of -q is then that of q,
//   Vt^{-q}(beta - tau)[Q][k+q][b][j] = conj(Vt^q(tau)[Q][k][j][b]),
// so only its producer and final contraction run:
//   Sig^k(beta - tau) += -(1/nk) sum_{Q,b} X[k][Q][i][b] conj(Vt^q(tau)[Q][k][j][b]),
//   X[k][Q][i][b] = sum_a V^{k,k+q}(Q)[i][a] G^{k+q}(beta - tau)[a][b].
static gw_status se_nodes(gw_ctx* c, const char* Vd, const char* Gd, const gw_z* Pt, int q, int tb, int te,
                          gw_z* Sig, bool mirror) {
  const int tc = c->tc;
  const int nk = c->nk, nao = c->d.nao, naux = c->d.naux, nt = c->d.ntau;
  const long long n2 = c->n2, sv = c->sv;
  const long long S = (long long)nk * sv;
  const bool f32 = lowp(c);
  const bool sb = splitbf(c);
  const size_t ez = f32 ? 8 : 16;
  char* Vt = (char*)c->ws;
  char* L = (char*)c->ws + region_bytes(c, tc);
  const int t = f32 ? 1 : 0;
  const char* Aq = Vd + (size_t)q * nk * sv * ez;
  for (int t0 = tb; t0 < te; t0 += tc) {
    const int tcur = std::min(tc, te - t0);
    // Vt[tl][Q][kk][b][j] = sum_Q' Pt[q][t0+tl][Q][Q'] V[q][kk][Q'][b][j]
    // (fp64), or Vt[tl][kk][Q][b][j] (mixed): see the final contraction
    if (sb) {
      // bf16x3: rows Q of P~ (complex64 copy, K = Q' contiguous), columns
      // (kk, b, j) of the V slab read in place (K = Q' with stride n2)
      float2* Pc = (float2*)((char*)c->ws + 2 * region_bytes(c, tc) + 2 * gslot_bytes(c));
      HIPCHK(c, to_c64_launch((const double2*)Pt + (long long)t0 * naux * naux, Pc,
                              (long long)tcur * naux * naux, c->st));
      SplitDesc d = split_desc();
      d.A = Pc;
      d.B = Aq; d.C = Vt;
      d.M = naux; d.N = nk * (int)n2; d.K = naux; d.batch = tcur;
      d.ta = 1; d.tb = 1; d.tc = 1;
      d.am = aff(naux); d.aks = 1; d.ba = aff((long long)naux * naux);
      d.bn = two((unsigned)n2, 1, sv); d.bks = n2; d.bb = aff(0);
      d.cm = aff(n2); d.cn = two((unsigned)n2, 1, sv); d.bc = aff(S);
      d.batch_fastest = 1;                    // every tau reads the same V slab
      d.kchunk = kMixedChunk; d.nsplit = nsplit(c);
      d.tag = KC_SE_CONTRACT;
      gw_status s = run_split(c, d, Ext{0, (long long)tcur * naux * naux}, Ext{0, (long long)nk * sv},
                              Ext{0, (long long)tcur * S});
      if (s != GW_OK) return s;
    } else if (!f32) {
      gw_status s = times_v(c, Pt + (long long)t0 * naux * naux, (const gw_z*)Aq, Vt, tcur, false);
      if (s != GW_OK) return s;
    } else {
      GemmDesc g = gemm_desc();
      g.A = (const double2*)Pt + (long long)t0 * naux * naux;
      g.B = Aq; g.C = Vt;
      g.M = naux; g.N = nk * (int)n2; g.K = naux; g.batch = tcur;
      g.am = aff(naux); g.ak = aff(1);
      g.bk = aff(n2); g.bn = two((unsigned)n2, 1, sv);
      g.cm = aff(n2); g.cn = two((unsigned)n2, 1, sv);
      g.ba = aff((long long)naux * naux); g.bb = aff(0); g.bc = aff(S);
      g.ta = 0; g.tb = g.tc = g.f32 = 1;
      g.batch_fastest = 2;   // as times_v
      g.group = 8;
      g.tag = KC_SE_CONTRACT;
      gw_status s = run(c, g, Ext{0, (long long)tcur * naux * naux}, Ext{0, (long long)nk * sv}, Ext{0, (long long)tcur * S});
      if (s != GW_OK) return s;
    }
    gw_status s;
    if (!f32) {
      // Sig[t0+tl][kk+q] += -(1/nk) sum_Q V[q][kk][Q]^H G[t0+tl][kk] Vt[tl][Q][kk]
      const long long gs = (long long)nk * n2;
      SandSum x{};
      x.A = Aq; x.skA = sv; x.sqA = n2;
      x.B = Vt; x.tsB = S; x.skB = n2; x.sqB = gs;
      x.tab = c->dplus + (size_t)q * nk;
      x.nt = tcur; x.alpha = -1.0 / nk; x.accumulate = 1;
      x.part = (double2*)L; x.part_elems = (long long)tc * S;
      x.G = (const double2*)Gd + t0 * gs; x.tsG = gs;
      x.O = (double2*)Sig + t0 * gs; x.tsO = gs; x.tabO = 1;
      const Arr slab{Aq, S}, vt{Vt, tc * S}, ga{Gd, nt * gs}, sa{Sig, nt * gs}, part{L, tc * S};
      if ((s = sand_sum(c, x, KC_SE_FINAL, slab, vt, ga, sa, part)) != GW_OK) return s;
      if (!mirror) continue;
      // -q at the mirrored nodes:
      // Sig[nt-1-t0-tl][kk] += -(1/nk) sum_Q V[q][kk][Q] G[nt-1-t0-tl][kk+q] Vt[tl][Q][kk]^H
      x.bh = 1;
      x.G = (const double2*)Gd + (nt - 1 - t0) * gs; x.tsG = -gs; x.tabG = 1;
      x.O = (double2*)Sig + (nt - 1 - t0) * gs; x.tsO = -gs; x.tabO = 0;
      if ((s = sand_sum(c, x, KC_SE_FINAL, slab, vt, ga, sa, part)) != GW_OK) return s;
      continue;
    }
    // L[tl][kk][i][Q][b] = sum_a conj(V[q][kk][Q][a][i]) G[t0+tl][kk][a][b]
    GemmDesc g = gemm_desc();
    g.A = Aq; g.B = Gd + (size_t)t0 * nk * n2 * ez; g.C = L;
    g.M = naux * nao; g.N = tcur * nao; g.K = nao; g.batch = nk;
    g.am = two(nao, 1, n2); g.ak = aff(nao); g.conjA = 1;
    g.bk = aff(nao); g.bn = two(nao, 1, (long long)nk * n2);
    g.cm = two(nao, (long long)naux * nao, nao);
    g.cn = two(nao, 1, S);
    g.ba = aff(sv); g.bb = aff(n2); g.bc = aff(sv);
    g.ta = g.tb = g.tc = g.f32 = 1;
    g.tag = KC_SE_PRODUCER;
    if ((s = run(c, g, Ext{0, (long long)nk * sv}, Ext{0, (long long)tcur * nk * n2}, Ext{0, (long long)tcur * S})) != GW_OK) return s;
    // Sig[t0+tl][kk+q][i][j] += -(1/nk) sum_{Q,b} L(i, (Q, b)) Vt((Q, b), j)
    // K = (Q, b) is contiguous in L and has stride nao in Vt, so the uniform-K
    // loop applies (fp32 MFMA steps are short enough for the per-lane index
    // carries of the fp64 layout to show: 6.6 vs 8.8 ms per q)
    g = gemm_desc();
    g.A = L; g.B = Vt; g.C = (double2*)Sig + (long long)t0 * nk * n2;
    g.M = nao; g.N = nao; g.K = naux * nao; g.batch = tcur * nk;
    g.am = aff((long long)naux * nao); g.ak = aff(1);
    g.bk = aff(nao); g.bn = aff(1);
    g.bb = two(nk, sv, S);
    g.cm = aff(nao); g.cn = aff(1);
    g.ba = two(nk, sv, S); g.bc = two(nk, 0, (long long)nk * n2);
    g.tab = c->dplus + (size_t)q * nk; g.tmod = nk; g.tsC = n2;
    g.alpha_r = -1.0 / nk;
    g.beta_zero = 0; g.beta_r = 1.0;
    g.ta = g.tb = g.f32 = 1; g.tc = 0; g.kchunk = kMixedChunk;
    g.tag = KC_SE_FINAL;
    if ((s = run(c, g, Ext{0, (long long)tcur * S}, Ext{0, (long long)tcur * S}, Ext{0, (long long)tcur * nk * n2})) != GW_OK) return s;
  }
  return GW_OK;
}

// The contribution of the pair {q, -q} (of q alone when q = -q): half of the
// nodes are enough for q = -q, whose mirrored nodes are its own.
static gw_status se_pair(gw_ctx* c, const void* V, const gw_z* G, const gw_z* Pt, int q, gw_z* Sig) {
  const int te = c->neg[q] == q ? c->d.ntau / 2 : c->d.ntau;
  return se_nodes(c, (const char*)V, (const char*)G, Pt, q, 0, te, Sig, true);
}

gw_status gw_self_energy(gw_ctx* c, const void* V, const gw_z* G, const gw_z* Pt, int q0, int nq,
                         gw_z* Sig) {
  if (!c) return GW_ERR_ARG;
  if (!ready(c)) return fail(c, GW_ERR_STATE, "grids not built (gw_build_grids or gw_set_grids)");
  if (q0 < 0 || nq < 0 || q0 + nq > c->nk) return fail(c, GW_ERR_ARG, "q range outside the mesh");
  if (nq == 0) return GW_OK;
  if (!V || !G || !Pt || !Sig) return fail(c, GW_ERR_ARG, "NULL array");
  if (!c->ws || c->ws_bytes < gw_workspace_bytes(c, GW_OP_SELF_ENERGY, c->tc))
    return fail(c, GW_ERR_WORKSPACE, "self-energy workspace too small");
  const char* Gd = (const char*)G;
  if (lowp(c)) {
    void* Gc = nullptr;
    gw_status s = g_to_c64(c, ctx_work(c), G, &Gc);
    if (s != GW_OK) return s;
    Gd = (const char*)Gc;
  }
  const long long per = (long long)c->d.ntau * c->d.naux * c->d.naux;
  for (int q = q0; q < q0 + nq; ++q) {
    gw_status s = se_nodes(c, (const char*)V, Gd, Pt + (q - q0) * per, q, 0, c->d.ntau, Sig, false);
    if (s != GW_OK) return s;
  }
  return GW_OK;
}

// ------------------------------------------------------------- density
static gw_status gamma_of(gw_ctx* c, const gw_z* G, double2* gamma) {
  GemmDesc g = gemm_desc();
  g.A = c->dw; g.B = (const double2*)G; g.C = gamma;
  g.M = 1; g.N = c->nk * (int)c->n2; g.K = c->d.ntau;
  g.am = aff(0); g.ak = aff(1); g.bk = aff((long long)c->nk * c->n2); g.bn = aff(1);
  g.cm = aff(0); g.cn = aff(1);
  g.alpha_r = -1.0;
  g.tag = KC_HF;
  return run(c, g, Ext{0, (long long)c->d.ntau}, Ext{0, (long long)c->d.ntau * c->nk * c->n2}, Ext{0, (long long)c->nk * c->n2});
}

gw_status gw_density(gw_ctx* c, const gw_z* G, const gw_z* S, gw_z* gamma, double* n_out) {
  if (!c) return GW_ERR_ARG;
  if (!ready(c)) return fail(c, GW_ERR_STATE, "grids not built (gw_build_grids or gw_set_grids)");
  if (!G || !gamma || (n_out && !S)) return fail(c, GW_ERR_ARG, "NULL array");
  gw_status s = gamma_of(c, G, (double2*)gamma);
  if (s != GW_OK || !n_out) return s;
  HIPCHK(c, trace_launch((const double2*)gamma, (const double2*)S, c->d.nao, c->nk, c->dpart, c->st));
  HIPCHK(c, sum_launch(c->dpart, c->nk, (double)c->d.ns / c->nk, c->dpart + c->nk, c->st));
  HIPCHK(c, hipMemcpyAsync(n_out, c->dpart + c->nk, sizeof(double), hipMemcpyDeviceToHost, c->st));
  HIPCHK(c, hipStreamSynchronize(c->st));
  return GW_OK;
}

// ------------------------------------------------------------- Eqs. HF_J, HF_K
// The exchange sums over q: with fold, O[k] += -(1/nk) sum_{q,Q} V^{k,k+q} X[k+q] V^H;
// otherwise O[k+q] += -(1/nk) sum_{q,Q} V^H X[k] V.  T holds nk naux nao^2
// numbers; as many q at once as leave room for their partial sums.
static gw_status exchange(gw_ctx* c, const char* Vd, const double2* X, double2* T, double2* O, bool fold) {
  const int nk = c->nk, tv = lowp(c) ? 1 : 0;
  const size_t ez = tv ? 8 : 16;
  const int qb = fold ? std::min(nk, c->d.naux) : 1;
  for (int q0 = 0; q0 < nk; q0 += qb) {
    SandSum x{};
    x.A = x.B = Vd + (size_t)q0 * nk * c->sv * ez;
    x.tsA = x.tsB = nk * c->sv; x.skA = x.skB = c->sv; x.sqA = x.sqB = c->n2;
    x.tv = tv; x.nt = std::min(qb, nk - q0); x.alpha = -1.0 / nk; x.accumulate = 1;
    x.tab = c->dplus + (size_t)q0 * nk; x.tstab = nk;
    x.G = X; x.O = O; x.part = T; x.part_elems = nk * c->sv;
    if (fold) { x.bh = 1; x.tabG = 1; x.fold_t = 1; }
    else x.tabO = 1;
    const Arr v{Vd, nk * (nk * c->sv)};
    gw_status s = sand_sum(c, x, KC_HF, v, v, Arr{X, nk * c->n2}, Arr{O, nk * c->n2}, Arr{T, nk * c->sv});
    if (s != GW_OK) return s;
  }
  return GW_OK;
}

gw_status gw_hf(gw_ctx* c, const void* V, const gw_z* G, gw_z* gamma_out, gw_z* Sinf) {
  if (!c) return GW_ERR_ARG;
  if (!ready(c)) return fail(c, GW_ERR_STATE, "grids not built (gw_build_grids or gw_set_grids)");
  if (!V || !G || !Sinf) return fail(c, GW_ERR_ARG, "NULL array");
  if (!c->ws || c->ws_bytes < gw_workspace_bytes(c, GW_OP_HF, 1))
    return fail(c, GW_ERR_WORKSPACE, "HF workspace too small");
  const int nk = c->nk, nao = c->d.nao, naux = c->d.naux;
  const long long n2 = c->n2, sv = c->sv;
  double2* T1 = (double2*)c->ws;
  double2* gam = (double2*)((char*)c->ws + align256((size_t)nk * sv * 16));
  double2* vq = (double2*)((char*)gam + align256((size_t)nk * n2 * 16));
  if (gamma_out) gam = (double2*)gamma_out;
  const char* Vd = (const char*)V;
  const int tv = lowp(c) ? 1 : 0;   // V storage type
  const size_t ez = tv ? 8 : 16;
  gw_status s = gamma_of(c, G, gam);
  if (s != GW_OK) return s;
  // v[Q] = (ns/nk) sum_{k',b,a} V[0][k'][Q][b][a] gamma[k'][a][b]
  hipEvent_t e0 = nullptr;
  if ((s = prof_begin(c, KC_HF, &e0)) != GW_OK) return s;
  HIPCHK(c, vdot_launch(Vd, tv, gam, vq, nk, naux, nao, (double)c->d.ns / nk, false, true, c->st));
  if ((s = prof_end(c, KC_HF, e0, 8.0 * nk * sv)) != GW_OK) return s;
  // J[k][e] = sum_Q v[Q] V[0][k][Q][e]
  GemmDesc g = gemm_desc();
  g.A = vq; g.B = Vd; g.C = (double2*)Sinf;
  g.M = 1; g.N = nk * (int)n2; g.K = naux;
  g.am = aff(0); g.ak = aff(1);
  g.bk = aff(n2); g.bn = two((unsigned)n2, 1, sv);
  g.cm = aff(0); g.cn = aff(1);
  g.tb = tv;
  g.tag = KC_HF;
  if ((s = run(c, g, Ext{0, (long long)naux}, Ext{0, (long long)nk * sv}, Ext{0, (long long)nk * n2})) != GW_OK) return s;
  // Sinf[k] += -(1/nk) sum_{q,Q} V[q][k][Q] gamma[k+q] V[q][k][Q]^H: one sum
  // over Q per (q, k), then the sum over q
  return exchange(c, Vd, gam, T1, (double2*)Sinf, true);
}

// ------------------------------------------------------------- Eq. Dyson
gw_status gw_dyson_G(gw_ctx* c, const gw_z* H0, const gw_z* S, const gw_z* Sinf, const gw_z* Siw,
                     double mu, gw_z* G) {
  if (!c) return GW_ERR_ARG;
  if (!ready(c)) return fail(c, GW_ERR_STATE, "grids not built (gw_build_grids or gw_set_grids)");
  if (!H0 || !S || !G) return fail(c, GW_ERR_ARG, "NULL array");
  if (!std::isfinite(mu)) return fail(c, GW_ERR_ARG, "mu is not finite");
  HIPCHK(c, zero_flag_launch(c->dflag, c->st));
  DysonArgs a{};
  a.H0 = (const double2*)H0; a.S = (const double2*)S;
  a.Sinf = (const double2*)Sinf; a.Siw = (const double2*)Siw;
  a.wF = c->dwF; a.rrow = c->drrow; a.mu = mu; a.nk = c->nk; a.nao = c->d.nao;
  a.G = (double2*)G; a.part = nullptr; a.flag = c->dflag;
  HIPCHK(c, dyson_any(c, a, 1));
  return read_flag(c, "dyson_G");
}

gw_status gw_find_mu(gw_ctx* c, const gw_z* H0, const gw_z* S, const gw_z* Sinf, const gw_z* Siw,
                     double n_target, double tol, double* mu_inout, gw_z* G_iw, gw_z* G_tau,
                     double* n_out) {
  if (!c) return GW_ERR_ARG;
  if (!ready(c)) return fail(c, GW_ERR_STATE, "grids not built (gw_build_grids or gw_set_grids)");
  if (!H0 || !S || !mu_inout) return fail(c, GW_ERR_ARG, "NULL array");
  if (G_tau && !G_iw) return fail(c, GW_ERR_ARG, "G_tau needs G_iw");
  if (!(n_target > 0.0) || !(n_target < (double)c->d.ns * c->d.nao))
    return fail(c, GW_ERR_ARG, "n_target must lie in (0, ns*nao)");
  if (!std::isfinite(*mu_inout)) return fail(c, GW_ERR_ARG, "initial mu is not finite");
  if (!(tol > 0.0)) tol = 1e-13;
  HIPCHK(c, zero_flag_launch(c->dflag, c->st));
  const double mu0 = *mu_inout;
  double n = 0.0;
  gw_status s;
  const Count count{c, H0, S, Sinf, Siw};
  auto root = [&](double target, double* out) {
    MuRoot<Count> r{count, c->mu.batch, c->mu.ahead, target, tol};
    const gw_status e = r.find(mu0, out);
    return e == GW_OK || !*r.why ? e : fail(c, e, r.why);
  };
  double mu = 0.0;
  if (c->mu_window > 0.0) {
    const double w = std::min(c->mu_window, 0.5 * std::min(n_target, (double)c->d.ns * c->d.nao - n_target));
    // keep mu0 when its count is inside the window, else the window's midpoint
    if ((s = count.one(mu0, &n)) != GW_OK) return s;
    if (std::fabs(n - n_target) <= w) {
      mu = mu0;
    } else {
      double m_lo = 0.0, m_hi = 0.0;
      if ((s = root(n_target - w, &m_lo)) != GW_OK) return s;
      if ((s = root(n_target + w, &m_hi)) != GW_OK) return s;
      mu = 0.5 * (m_lo + m_hi);
    }
  } else {
    if ((s = root(n_target, &mu)) != GW_OK) return s;
  }
  if ((s = count.one(mu, &n, G_iw)) != GW_OK) return s;
  if ((s = read_flag(c, "find_mu")) != GW_OK) return s;
  *mu_inout = mu;
  if (n_out) *n_out = n;
  if (G_tau) {
    if ((s = gw_iw_to_tau(c, GW_FERMION, G_iw, 1, (long long)c->nk * c->n2, G_tau)) != GW_OK)
      return s;
  }
  return GW_OK;
}


// =========================================================================
// Derivatives of G -> (Sigma_inf, Sigma~).  The map is holomorphic in G, so
// a vector-Jacobian product is the conjugate-transposed Jacobian applied to
// the cotangent (the convention of torch autograd for complex tensors).
// All of these need a GW_PREC_FP64 context.
// =========================================================================

// calls that never read V run in either precision
static gw_status need_grids(gw_ctx* c) {
  if (!c) return GW_ERR_ARG;
  if (!ready(c)) return fail(c, GW_ERR_STATE, "grids not built (gw_build_grids or gw_set_grids)");
  return GW_OK;
}

gw_status gw_screened_W_lin(gw_ctx* c, const gw_z* Pt, const gw_z* X, int nq, int adjoint, gw_z* Y) {
  gw_status s = need_grids(c);
  if (s != GW_OK) return s;
  if (nq < 0 || nq > c->nk) return fail(c, GW_ERR_ARG, "nq out of range");
  if (nq == 0) return GW_OK;
  if (!Pt || !X || !Y) return fail(c, GW_ERR_ARG, "NULL array");
  if (X == Y || Pt == Y) return fail(c, GW_ERR_ARG, "Y may not alias Pt or X");
  if (!c->ws || c->ws_bytes < gw_workspace_bytes(c, GW_OP_SCREENED_W, nq))
    return fail(c, GW_ERR_WORKSPACE, "screened_W workspace too small");
  const int n = c->d.naux;
  const long long nn = (long long)n * n, nmat = (long long)nq * c->d.nw_b;
  double2* T = (double2*)c->ws;
  // T = X + op(Pt) X, then Y = T + T op(Pt), op = identity (JVP) or ^H (VJP):
  // (I + Pt) X (I + Pt) is the derivative of (I - P0)^{-1} P0 = (I - P0)^{-1} - I.
  HIPCHK(c, mix_launch(nmat * nn, 1.0, (const double2*)X, T, nullptr, 2048, c->st));
  GemmDesc g = gemm_desc();
  g.A = Pt; g.B = X; g.C = T;
  g.M = n; g.N = n; g.K = n; g.batch = (int)nmat;
  if (adjoint) { g.am = aff(1); g.ak = aff(n); g.conjA = 1; } else { g.am = aff(n); g.ak = aff(1); }
  g.bk = aff(n); g.bn = aff(1); g.cm = aff(n); g.cn = aff(1);
  g.ba = g.bb = g.bc = aff(nn);
  g.beta_zero = 0; g.beta_r = 1.0;
  g.tag = KC_OTHER;
  if ((s = run(c, g, Ext{0, nmat * nn}, Ext{0, nmat * nn}, Ext{0, nmat * nn})) != GW_OK) return s;
  HIPCHK(c, mix_launch(nmat * nn, 1.0, T, (double2*)Y, nullptr, 2048, c->st));
  g = gemm_desc();
  g.A = T; g.B = Pt; g.C = Y;
  g.M = n; g.N = n; g.K = n; g.batch = (int)nmat;
  g.am = aff(n); g.ak = aff(1);
  if (adjoint) { g.bk = aff(1); g.bn = aff(n); g.conjB = 1; } else { g.bk = aff(n); g.bn = aff(1); }
  g.cm = aff(n); g.cn = aff(1);
  g.ba = g.bb = g.bc = aff(nn);
  g.beta_zero = 0; g.beta_r = 1.0;
  g.tag = KC_OTHER;
  return run(c, g, Ext{0, nmat * nn}, Ext{0, nmat * nn}, Ext{0, nmat * nn});
}

gw_status gw_transform_adjoint(gw_ctx* c, int stat, int inverse, const gw_z* Xin, long long batch,
                               long long R, gw_z* Xout) {
  gw_status s = need_grids(c);
  if (s != GW_OK) return s;
  if (stat != GW_FERMION && stat != GW_BOSON) return fail(c, GW_ERR_ARG, "stat must be 0 or 1");
  if (batch < 0 || R < 0 || batch > 65535 || R > 0x7fffffffLL)
    return fail(c, GW_ERR_ARG, "batch or R out of range");
  if (batch == 0 || R == 0) return GW_OK;
  if (!Xin || !Xout) return fail(c, GW_ERR_ARG, "NULL array");
  const int nt = c->d.ntau;
  const int nw = stat == GW_FERMION ? c->d.nw_f : c->d.nw_b;
  // inverse = 0: Xout[b][i][r] = sum_n conj(T[n][i]) Xin[b][n][r]  (adjoint of tau -> i w)
  // inverse = 1: Xout[b][n][r] = sum_i conj(Tp[i][n]) Xin[b][i][r] (adjoint of i w -> tau)
  const int rows = inverse ? nw : nt, inner = inverse ? nt : nw;
  GemmDesc g = gemm_desc();
  g.A = inverse ? (stat == GW_FERMION ? c->dTFp : c->dTBp) : (stat == GW_FERMION ? c->dTF : c->dTB);
  g.B = Xin; g.C = Xout;
  g.M = rows; g.N = (int)R; g.K = inner; g.batch = (int)batch;
  g.am = aff(1); g.ak = aff(rows); g.conjA = 1;
  g.bk = aff(R); g.bn = aff(1); g.cm = aff(R); g.cn = aff(1);
  g.ba = aff(0); g.bb = aff((long long)inner * R); g.bc = aff((long long)rows * R);
  g.tag = KC_TRANSFORM;
  return run(c, g, Ext{0, (long long)rows * inner}, Ext{0, batch * inner * R}, Ext{0, batch * rows * R});
}

// The fp64 adjoints, one q at a time, on the same kernels as the forward
// chain; the small matrices of a node meet in one triple product each:
//   Gbar(t)[k]   += -(1/nk) sum_Q V_Q Sbar(t)[k+q] Vt_Q^H,   Vt = P~(t) V
//   Ptbar(t)[Q][Q'] = -(1/nk) sum_{k,e} (G^H V_Q Sbar[k+q])[e] conj(V_Q'[e])
// pair: also the first of these for -q at the mirrored nodes, from the same Vt
// (see se_nodes):
//   Gbar(beta - t)[k+q] += -(1/nk) sum_Q V_Q^H Sbar(beta - t)[k] Vt_Q.
static gw_status se_vjp_g(gw_ctx* c, const gw_z* Vq, const gw_z* Pt, const gw_z* Sbar, int q, int te, gw_z* Gbar,
                          bool pair) {
  const int tc = c->tc, nk = c->nk, nt = c->d.ntau;
  const long long n2 = c->n2, sv = c->sv, S = (long long)nk * sv, gs = (long long)nk * n2;
  char* Vt = (char*)c->ws;
  for (int t0 = 0; t0 < te; t0 += tc) {
    const int tcur = std::min(tc, te - t0);
    gw_status s = times_v(c, Pt + (long long)t0 * c->d.naux * c->d.naux, Vq, Vt, tcur, false);
    if (s != GW_OK) return s;
    SandSum x{};
    x.A = Vq; x.skA = sv; x.sqA = n2;
    x.B = Vt; x.tsB = S; x.skB = n2; x.sqB = gs;
    x.tab = c->dplus + (size_t)q * nk;
    x.nt = tcur; x.alpha = -1.0 / nk; x.accumulate = 1;
    x.part = (double2*)((char*)c->ws + region_bytes(c, tc)); x.part_elems = (long long)tc * S;
    x.bh = 1;
    x.G = (const double2*)Sbar + t0 * gs; x.tsG = gs; x.tabG = 1;
    x.O = (double2*)Gbar + t0 * gs; x.tsO = gs;
    const Arr slab{Vq, S}, vt{Vt, tc * S}, sa{Sbar, nt * gs}, ga{Gbar, nt * gs}, part{x.part, tc * S};
    if ((s = sand_sum(c, x, KC_SE_FINAL, slab, vt, sa, ga, part)) != GW_OK) return s;
    if (!pair) continue;
    x.bh = 0;
    x.G = (const double2*)Sbar + (nt - 1 - t0) * gs; x.tsG = -gs; x.tabG = 0;
    x.O = (double2*)Gbar + (nt - 1 - t0) * gs; x.tsO = -gs; x.tabO = 1;
    if ((s = sand_sum(c, x, KC_SE_FINAL, slab, vt, sa, ga, part)) != GW_OK) return s;
  }
  return GW_OK;
}

static gw_status se_vjp_p(gw_ctx* c, const gw_z* Vq, const gw_z* G, const gw_z* Sbar, int q, gw_z* Ptbar) {
  const int tc = c->tc, nk = c->nk, nt = c->d.ntau;
  const long long gs = (long long)nk * c->n2, S = (long long)nk * c->sv;
  for (int t0 = 0; t0 < nt; t0 += tc) {
    const int tcur = std::min(tc, nt - t0);
    SandProd p{};
    p.V = (const double2*)Vq; p.Y = (double2*)c->ws; p.tab = c->dplus + (size_t)q * nk;
    p.nt = tcur; p.tsY = S;
    p.L = (const double2*)G + t0 * gs; p.tsL = gs; p.hermL = 1;
    p.R = (const double2*)Sbar + t0 * gs; p.tsR = gs; p.tabR = 1;
    gw_status s = sand_prod(c, p, KC_SE_PRODUCER, Arr{Vq, S}, Arr{G, nt * gs}, Arr{Sbar, nt * gs}, Arr{c->ws, tc * S});
    if (s != GW_OK) return s;
    const long long nn = (long long)c->d.naux * c->d.naux;
    if ((s = pol_contract(c, (char*)c->ws, (char*)c->ws + region_bytes(c, tc), (const char*)Vq, tcur, tc,
                          (double2*)Ptbar + t0 * nn, nullptr, -1.0 / nk, false, false, Arr{Ptbar, nt * nn}, Arr{})) != GW_OK)
      return s;
  }
  return GW_OK;
}

// Both slots of the polarization at the nodes [0, te):
//   Gbar(t)[k+q]        += sc sum_Q V_Q^H G(beta - t)[k]^H (P0bar V)_Q
//   Gbar(beta - t)[k]   += sc sum_Q V_Q G(t)[k+q]^H (P0bar^H V)_Q^H
static gw_status pol_vjp_q(gw_ctx* c, const gw_z* Vq, const gw_z* G, const gw_z* P0bar, int q, int te, gw_z* Gbar) {
  const int tc = c->tc, nk = c->nk, nt = c->d.ntau;
  const long long n2 = c->n2, sv = c->sv, S = (long long)nk * sv, gs = (long long)nk * n2;
  for (int t0 = 0; t0 < te; t0 += tc) {
    const int tcur = std::min(tc, te - t0);
    const gw_z* Pb = P0bar + (long long)t0 * c->d.naux * c->d.naux;
    gw_status s = times_v(c, Pb, Vq, (char*)c->ws, tcur, false);
    if (s != GW_OK) return s;
    SandSum x{};
    x.A = Vq; x.skA = sv; x.sqA = n2;
    x.B = c->ws; x.tsB = S; x.skB = n2; x.sqB = gs;
    x.tab = c->dplus + (size_t)q * nk;
    x.nt = tcur; x.alpha = -(double)c->d.ns / nk; x.accumulate = 1; x.hermG = 1;
    x.part = (double2*)((char*)c->ws + region_bytes(c, tc)); x.part_elems = (long long)tc * S;
    x.G = (const double2*)G + (nt - 1 - t0) * gs; x.tsG = -gs;
    x.O = (double2*)Gbar + t0 * gs; x.tsO = gs; x.tabO = 1;
    const Arr slab{Vq, S}, pv{c->ws, tc * S}, ga{G, nt * gs}, gb{Gbar, nt * gs}, part{x.part, tc * S};
    if ((s = sand_sum(c, x, KC_SE_FINAL, slab, pv, ga, gb, part)) != GW_OK) return s;
    if ((s = times_v(c, Pb, Vq, (char*)c->ws, tcur, true)) != GW_OK) return s;
    x.bh = 1;
    x.G = (const double2*)G + t0 * gs; x.tsG = gs; x.tabG = 1;
    x.O = (double2*)Gbar + (nt - 1 - t0) * gs; x.tsO = -gs; x.tabO = 0;
    if ((s = sand_sum(c, x, KC_SE_FINAL, slab, pv, ga, gb, part)) != GW_OK) return s;
  }
  return GW_OK;
}

gw_status gw_self_energy_vjp(gw_ctx* c, const void* V, const gw_z* G, const gw_z* Pt,
                             const gw_z* Sbar, int q0, int nq, gw_z* Gbar, gw_z* Ptbar) {
  gw_status s = need_grids(c);
  if (s != GW_OK) return s;
  if (q0 < 0 || nq < 0 || q0 + nq > c->nk) return fail(c, GW_ERR_ARG, "q range outside the mesh");
  if (nq == 0) return GW_OK;
  if (!V || !G || !Pt || !Sbar || !Gbar || !Ptbar) return fail(c, GW_ERR_ARG, "NULL array");
  const int tc = c->tc;
  if (!c->ws || c->ws_bytes < gw_workspace_bytes(c, GW_OP_SELF_ENERGY, tc))
    return fail(c, GW_ERR_WORKSPACE, "self-energy workspace too small");
  const int nk = c->nk, nao = c->d.nao, naux = c->d.naux, nt = c->d.ntau;
  const long long n2 = c->n2, sv = c->sv, S = (long long)nk * sv;
  if (!lowp(c)) {
    const long long per = (long long)nt * naux * naux;
    for (int q = q0; q < q0 + nq; ++q) {
      const gw_z* Vq = (const gw_z*)V + (size_t)q * S;
      if ((s = se_vjp_g(c, Vq, Pt + (q - q0) * per, Sbar, q, nt, Gbar, false)) != GW_OK) return s;
      if ((s = se_vjp_p(c, Vq, G, Sbar, q, Ptbar + (q - q0) * per)) != GW_OK) return s;
    }
    return GW_OK;
  }
  // the complex64 modes: complex64 intermediates, fp32 MFMA (operands rounded
  // on load) with fp64 sums of 512-term chunks for the long contractions
  char* R0 = (char*)c->ws;
  char* R1 = (char*)c->ws + region_bytes(c, tc);
  for (int q = q0; q < q0 + nq; ++q) {
    const char* Aq = (const char*)V + (size_t)q * S * 8;
    for (int t0 = 0; t0 < nt; t0 += tc) {
      const int tcur = std::min(tc, nt - t0);
      const gw_z* Ptq = Pt + ((long long)(q - q0) * nt + t0) * naux * naux;
      // R0 = Vt[tl][Q][kk][b][j] = sum_Q' Pt[Q][Q'] V[q][kk][Q'][b][j]
      GemmDesc g = gemm_desc();
      g.A = Ptq; g.B = Aq; g.C = R0;
      g.M = naux; g.N = nk * (int)n2; g.K = naux; g.batch = tcur;
      g.am = aff(naux); g.ak = aff(1); g.bk = aff(n2); g.bn = two((unsigned)n2, 1, sv);
      g.cm = aff((long long)nk * n2); g.cn = aff(1);
      g.ba = aff((long long)naux * naux); g.bb = aff(0); g.bc = aff(S);
      g.ta = 0; g.tb = g.tc = g.f32 = 1;
      g.batch_fastest = 1;
      g.tag = KC_SE_CONTRACT;
      if ((s = run(c, g, Ext{0, (long long)tcur * naux * naux}, Ext{0, (long long)nk * sv}, Ext{0, (long long)tcur * S})) != GW_OK) return s;
      // R1 = L'[tl][kk][Q][a][j] = sum_i V[q][kk][Q][a][i] Sbar[t][kk+q][i][j]
      g = gemm_desc();
      g.A = Aq; g.B = Sbar + (size_t)t0 * nk * n2; g.C = R1;
      g.M = naux * nao; g.N = tcur * nao; g.K = nao; g.batch = nk;
      g.am = aff(nao); g.ak = aff(1); g.bk = aff(nao); g.bn = two(nao, 1, (long long)nk * n2);
      g.cm = aff(nao); g.cn = two(nao, 1, S);
      g.ba = aff(sv); g.bb = aff(0); g.bc = aff(sv);
      g.tab = c->dplus + (size_t)q * nk; g.tmod = nk; g.tsB = n2;
      g.ta = g.tc = g.f32 = 1; g.tb = 0;
      g.tag = KC_SE_PRODUCER;
      if ((s = run(c, g, Ext{0, (long long)nk * sv}, Ext{0, (long long)tcur * nk * n2}, Ext{0, (long long)tcur * S})) != GW_OK) return s;
      // Gbar[t][kk][a][b] += -(1/nk) sum_{Q,j} L'[tl][kk][Q][a][j] conj(Vt[tl][Q][kk][b][j])
      g = gemm_desc();
      g.A = R1; g.B = R0; g.C = Gbar + (size_t)t0 * nk * n2;
      g.M = nao; g.N = nao; g.K = naux * nao; g.batch = tcur * nk;
      g.am = aff(nao); g.ak = two(nao, 1, n2);
      g.bk = two(nao, 1, (long long)nk * n2); g.bn = aff(nao); g.conjB = 1;
      g.cm = aff(nao); g.cn = aff(1);
      g.ba = two(nk, sv, S); g.bb = two(nk, n2, S); g.bc = two(nk, n2, (long long)nk * n2);
      g.alpha_r = -1.0 / nk; g.beta_zero = 0; g.beta_r = 1.0;
      g.ta = g.tb = g.f32 = 1; g.tc = 0; g.kchunk = kMixedChunk;
      g.tag = KC_SE_FINAL;
      if ((s = run(c, g, Ext{0, (long long)tcur * S}, Ext{0, (long long)tcur * S}, Ext{0, (long long)tcur * nk * n2})) != GW_OK) return s;
      // R0 = Y[tl][kk][Q'][a][j] = sum_b G[t][kk][a][b] V[q][kk][Q'][b][j]
      g = gemm_desc();
      g.A = G + (size_t)t0 * nk * n2; g.B = Aq; g.C = R0;
      g.M = tcur * nao; g.N = naux * nao; g.K = nao; g.batch = nk;
      g.am = two(nao, nao, (long long)nk * n2); g.ak = aff(1);
      g.bk = aff(nao); g.bn = two(nao, 1, n2);
      g.cm = two(nao, nao, S); g.cn = two(nao, 1, n2);
      g.ba = aff(n2); g.bb = aff(sv); g.bc = aff(sv);
      g.ta = 0; g.tb = g.tc = g.f32 = 1;
      g.tag = KC_SE_PRODUCER;
      if ((s = run(c, g, Ext{0, (long long)tcur * nk * n2}, Ext{0, (long long)nk * sv}, Ext{0, (long long)tcur * S})) != GW_OK) return s;
      // Ptbar[q][t][Q][Q'] = -(1/nk) sum_{kk,a,j} L'[tl][kk][Q][a][j] conj(Y[tl][kk][Q'][a][j])
      g = gemm_desc();
      g.A = R1; g.B = R0; g.C = Ptbar + ((long long)(q - q0) * nt + t0) * naux * naux;
      g.M = naux; g.N = naux; g.K = nk * (int)n2; g.batch = tcur;
      g.am = aff(n2); g.ak = two((unsigned)n2, 1, sv);
      g.bk = two((unsigned)n2, 1, sv); g.bn = aff(n2); g.conjB = 1;
      g.cm = aff(naux); g.cn = aff(1);
      g.ba = aff(S); g.bb = aff(S); g.bc = aff((long long)naux * naux);
      g.alpha_r = -1.0 / nk;
      g.ta = g.tb = g.f32 = 1; g.tc = 0; g.kchunk = kMixedChunk;
      g.tag = KC_POL_CONTRACT;
      if ((s = run(c, g, Ext{0, (long long)tcur * S}, Ext{0, (long long)tcur * S}, Ext{0, (long long)tcur * naux * naux})) != GW_OK) return s;
    }
  }
  return GW_OK;
}

gw_status gw_polarization_vjp(gw_ctx* c, const void* V, const gw_z* G, const gw_z* P0bar, int q0,
                              int nq, gw_z* Gbar) {
  gw_status s = need_grids(c);
  if (s != GW_OK) return s;
  if (q0 < 0 || nq < 0 || q0 + nq > c->nk) return fail(c, GW_ERR_ARG, "q range outside the mesh");
  if (nq == 0) return GW_OK;
  if (!V || !G || !P0bar || !Gbar) return fail(c, GW_ERR_ARG, "NULL array");
  const int tc = c->tc;
  if (!c->ws || c->ws_bytes < gw_workspace_bytes(c, GW_OP_POLARIZATION, tc))
    return fail(c, GW_ERR_WORKSPACE, "polarization workspace too small");
  const int nk = c->nk, nao = c->d.nao, naux = c->d.naux, nt = c->d.ntau;
  const long long n2 = c->n2, sv = c->sv, S = (long long)nk * sv;
  const double sc = -(double)c->d.ns / nk;
  if (!lowp(c)) {
    for (int q = q0; q < q0 + nq; ++q)
      if ((s = pol_vjp_q(c, (const gw_z*)V + (size_t)q * S, G, P0bar + (long long)(q - q0) * nt * naux * naux, q, nt,
                         Gbar)) != GW_OK) return s;
    return GW_OK;
  }
  // the complex64 modes: complex64 intermediates, fp32 MFMA (operands rounded
  // on load) with fp64 sums of 512-term chunks for the long contractions
  char* R0 = (char*)c->ws;
  char* R1 = (char*)c->ws + region_bytes(c, tc);
  for (int q = q0; q < q0 + nq; ++q) {
    const char* Aq = (const char*)V + (size_t)q * S * 8;
    for (int t0 = 0; t0 < nt; t0 += tc) {
      const int tcur = std::min(tc, nt - t0);
      const gw_z* Pb = P0bar + ((long long)(q - q0) * nt + t0) * naux * naux;
      // --- tau slot: Gbar[t][k+q] += sc sum_{Q,d} conj(V[q][k][Q][d][a]) U[Q][k][d][b]
      // R1 = W[tl][k][Q'][d][b] = sum_c conj(G[nt-1-t][k][c][d]) V[q][k][Q'][c][b]
      GemmDesc g = gemm_desc();
      g.A = G + (size_t)(nt - 1 - t0) * nk * n2; g.B = Aq; g.C = R1;
      g.M = tcur * nao; g.N = naux * nao; g.K = nao; g.batch = nk;
      g.am = two(nao, 1, -(long long)nk * n2); g.ak = aff(nao); g.conjA = 1;
      g.bk = aff(nao); g.bn = two(nao, 1, n2);
      g.cm = two(nao, nao, S); g.cn = two(nao, 1, n2);
      g.ba = aff(n2); g.bb = aff(sv); g.bc = aff(sv);
      g.ta = 0; g.tb = g.tc = g.f32 = 1;
      g.tag = KC_POL_PRODUCER;
      if ((s = run(c, g, Ext{-(long long)(tcur - 1) * nk * n2, (long long)nk * n2}, Ext{0, (long long)nk * sv}, Ext{0, (long long)tc * S})) != GW_OK) return s;
      // R0 = U[tl][Q][k][e] = sum_Q' Pbar[Q][Q'] W[tl][k][Q'][e]
      g = gemm_desc();
      g.A = Pb; g.B = R1; g.C = R0;
      g.M = naux; g.N = nk * (int)n2; g.K = naux; g.batch = tcur;
      g.am = aff(naux); g.ak = aff(1); g.bk = aff(n2); g.bn = two((unsigned)n2, 1, sv);
      g.cm = aff((long long)nk * n2); g.cn = aff(1);
      g.ba = aff((long long)naux * naux); g.bb = aff(S); g.bc = aff(S);
      g.ta = 0; g.tb = g.tc = g.f32 = 1;
      g.tag = KC_SE_CONTRACT;
      if ((s = run(c, g, Ext{0, (long long)tcur * naux * naux}, Ext{0, (long long)tcur * S}, Ext{0, (long long)tcur * S})) != GW_OK) return s;
      // Gbar[t0+tl][k+q][a][b] += sc sum_{Q,d} conj(V[q][k][Q][d][a]) U[tl][Q][k][d][b]
      g = gemm_desc();
      g.A = Aq; g.B = R0; g.C = Gbar + (size_t)t0 * nk * n2;
      g.M = nao; g.N = nao; g.K = naux * nao; g.batch = tcur * nk;
      g.am = aff(1); g.ak = two(nao, nao, n2); g.conjA = 1;
      g.bk = two(nao, nao, (long long)nk * n2); g.bn = aff(1);
      g.cm = aff(nao); g.cn = aff(1);
      g.ba = two(nk, sv, 0); g.bb = two(nk, n2, S); g.bc = two(nk, 0, (long long)nk * n2);
      g.tab = c->dplus + (size_t)q * nk; g.tmod = nk; g.tsC = n2;
      g.alpha_r = sc; g.beta_zero = 0; g.beta_r = 1.0;
      g.ta = g.tb = g.f32 = 1; g.tc = 0; g.kchunk = kMixedChunk;
      g.tag = KC_SE_FINAL;
      if ((s = run(c, g, Ext{0, (long long)nk * sv}, Ext{0, (long long)tcur * S}, Ext{0, (long long)tcur * nk * n2})) != GW_OK) return s;
      // --- mirrored slot: Gbar[nt-1-t][k] += sc sum_{Q',b} V[q][k][Q'][c][b] T[Q'][k][d][b]
      // R1 = X[tl][k][Q][d][b] = sum_a V[q][k][Q][d][a] G[t][k+q][a][b]
      g = gemm_desc();
      g.A = Aq; g.B = G + (size_t)t0 * nk * n2; g.C = R1;
      g.M = naux * nao; g.N = tcur * nao; g.K = nao; g.batch = nk;
      g.am = aff(nao); g.ak = aff(1); g.bk = aff(nao); g.bn = two(nao, 1, (long long)nk * n2);
      g.cm = aff(nao); g.cn = two(nao, 1, S);
      g.ba = aff(sv); g.bb = aff(0); g.bc = aff(sv);
      g.tab = c->dplus + (size_t)q * nk; g.tmod = nk; g.tsB = n2;
      g.ta = g.tc = g.f32 = 1; g.tb = 0;
      g.tag = KC_POL_PRODUCER;
      if ((s = run(c, g, Ext{0, (long long)nk * sv}, Ext{0, (long long)tcur * nk * n2}, Ext{0, (long long)tc * S})) != GW_OK) return s;
      // R0 = T[tl][Q'][k][e] = sum_Q Pbar[Q][Q'] conj(X[tl][k][Q][e])
      g = gemm_desc();
      g.A = Pb; g.B = R1; g.C = R0;
      g.M = naux; g.N = nk * (int)n2; g.K = naux; g.batch = tcur;
      g.am = aff(1); g.ak = aff(naux); g.bk = aff(n2); g.bn = two((unsigned)n2, 1, sv); g.conjB = 1;
      g.cm = aff((long long)nk * n2); g.cn = aff(1);
      g.ba = aff((long long)naux * naux); g.bb = aff(S); g.bc = aff(S);
      g.ta = 0; g.tb = g.tc = g.f32 = 1;
      g.tag = KC_SE_CONTRACT;
      if ((s = run(c, g, Ext{0, (long long)tcur * naux * naux}, Ext{0, (long long)tcur * S}, Ext{0, (long long)tcur * S})) != GW_OK) return s;
      // Gbar[nt-1-t0-tl][k][c][d] += sc sum_{Q',b} V[q][k][Q'][c][b] T[tl][Q'][k][d][b]
      g = gemm_desc();
      g.A = Aq; g.B = R0; g.C = Gbar + (size_t)(nt - 1 - t0) * nk * n2;
      g.M = nao; g.N = nao; g.K = naux * nao; g.batch = tcur * nk;
      g.am = aff(nao); g.ak = two(nao, 1, n2);
      g.bk = two(nao, 1, (long long)nk * n2); g.bn = aff(nao);
      g.cm = aff(nao); g.cn = aff(1);
      g.ba = two(nk, sv, 0); g.bb = two(nk, n2, S); g.bc = two(nk, n2, -(long long)nk * n2);
      g.alpha_r = sc; g.beta_zero = 0; g.beta_r = 1.0;
      g.ta = g.tb = g.f32 = 1; g.tc = 0; g.kchunk = kMixedChunk;
      g.tag = KC_SE_FINAL;
      if ((s = run(c, g, Ext{0, (long long)nk * sv}, Ext{0, (long long)tcur * S}, Ext{-(long long)(tcur - 1) * nk * n2, (long long)nk * n2})) != GW_OK) return s;
    }
  }
  return GW_OK;
}

gw_status gw_hf_vjp(gw_ctx* c, const void* V, const gw_z* Sbar, gw_z* Gbar) {
  gw_status s = need_grids(c);
  if (s != GW_OK) return s;
  if (!V || !Sbar || !Gbar) return fail(c, GW_ERR_ARG, "NULL array");
  if (!c->ws || c->ws_bytes < gw_workspace_bytes(c, GW_OP_HF, 1))
    return fail(c, GW_ERR_WORKSPACE, "HF workspace too small");
  const int nk = c->nk, nao = c->d.nao, naux = c->d.naux, nt = c->d.ntau;
  const long long n2 = c->n2, sv = c->sv;
  // complex64 V is read in fp64 arithmetic, as in gw_hf
  const int tv = lowp(c) ? 1 : 0;
  const size_t ez = tv ? 8 : 16;
  const char* Vd = (const char*)V;
  double2* T2 = (double2*)c->ws;
  double2* gb = (double2*)((char*)c->ws + align256((size_t)nk * sv * 16));
  double2* vb = (double2*)((char*)gb + align256((size_t)nk * n2 * 16));
  // vbar[Q] = sum_{k,e} conj(V[0][k][Q][e]) Sbar[k][e]
  hipEvent_t e0 = nullptr;
  if ((s = prof_begin(c, KC_HF, &e0)) != GW_OK) return s;
  HIPCHK(c, vdot_launch(Vd, tv, (const double2*)Sbar, vb, nk, naux, nao, 1.0, true, false, c->st));
  if ((s = prof_end(c, KC_HF, e0, 8.0 * nk * sv)) != GW_OK) return s;
  // gbar[k'][a][b] = (ns/nk) sum_Q conj(V[0][k'][Q][b][a]) vbar[Q]
  GemmDesc g = gemm_desc();
  g.A = vb; g.B = Vd; g.C = gb;
  g.M = 1; g.N = nk * (int)n2; g.K = naux;
  g.am = aff(0); g.ak = aff(1);
  g.bk = aff(n2); g.bn = three(nao, nao, nao, 1, sv); g.conjB = 1;
  g.cm = aff(0); g.cn = aff(1);
  g.alpha_r = (double)c->d.ns / nk;
  g.tb = tv;
  g.tag = KC_HF;
  if ((s = run(c, g, Ext{0, (long long)naux}, Ext{0, (long long)nk * sv}, Ext{0, (long long)nk * n2})) != GW_OK) return s;
  // gbar[k+q] += -(1/nk) sum_Q V[q][k][Q]^H Sbar[k] V[q][k][Q]: the adjoint of
  // X -> V X V^H; the targets of two q overlap, so one q after the other
  if ((s = exchange(c, Vd, (const double2*)Sbar, T2, gb, false)) != GW_OK) return s;
  // Gbar[t] += -w_t gbar   (gamma = -sum_t w_t G(t), w real)
  g = gemm_desc();
  g.A = c->dw; g.B = gb; g.C = Gbar;
  g.M = nt; g.N = nk * (int)n2; g.K = 1;
  g.am = aff(1); g.ak = aff(0); g.bk = aff(0); g.bn = aff(1);
  g.cm = aff((long long)nk * n2); g.cn = aff(1);
  g.alpha_r = -1.0; g.beta_zero = 0; g.beta_r = 1.0;
  g.tag = KC_HF;
  return run(c, g, Ext{0, (long long)nt}, Ext{0, (long long)nk * n2}, Ext{0, (long long)nt * nk * n2});
}


// ---------------------------------------------------------------- vectors
gw_status gw_axpby(gw_ctx* c, long long n, double ar, double ai, const gw_z* X, double br, double bi,
                   gw_z* Y) {
  if (!c) return GW_ERR_ARG;
  if (n < 0 || !Y) return fail(c, GW_ERR_ARG, "bad gw_axpby arguments");
  HIPCHK(c, axpby_launch(n, ar, ai, (const double2*)X, br, bi, (double2*)Y, c->st));
  return GW_OK;
}

gw_status gw_dot(gw_ctx* c, long long n, const gw_z* X, const gw_z* Y, double* out) {
  if (!c) return GW_ERR_ARG;
  if (n < 0 || !X || !Y || !out) return fail(c, GW_ERR_ARG, "bad gw_dot arguments");
  if (n == 0) {
    out[0] = out[1] = 0.0;
    return GW_OK;
  }
  const int nblk = (int)std::min<long long>((n + 255) / 256, 1024);
  HIPCHK(c, dot_launch(n, (const double2*)X, (const double2*)Y, c->dred, nblk, c->dred + 2 * 1024,
                       c->st));
  HIPCHK(c, hipMemcpyAsync(out, c->dred + 2 * 1024, 2 * sizeof(double), hipMemcpyDeviceToHost, c->st));
  HIPCHK(c, hipStreamSynchronize(c->st));
  return GW_OK;
}

gw_status gw_hermitize(gw_ctx* c, gw_z* X, int n, long long nmat) {
  if (!c) return GW_ERR_ARG;
  if (n < 1 || n > 8192 || nmat < 0 || nmat > 65535) return fail(c, GW_ERR_ARG, "bad gw_hermitize sizes");
  if (nmat == 0) return GW_OK;
  if (!X) return fail(c, GW_ERR_ARG, "NULL array");
  HIPCHK(c, herm_avg_launch((double2*)X, n, nmat, c->st));
  return GW_OK;
}

// ------------------------------------------------- finite-size corrections
gw_status gw_finite_size(gw_ctx* c, const gw_z* S, double chi, const gw_z* gamma, gw_z* Sig_inf,
                         const gw_z* G_tau, const double* head, gw_z* Sig_tau) {
  if (!c) return GW_ERR_ARG;
  const int nao = c->d.nao, nk = c->nk, nt = c->d.ntau;
  if (nao > 64) return fail(c, GW_ERR_ARG, "gw_finite_size needs nao <= 64");
  if (!std::isfinite(chi)) return fail(c, GW_ERR_ARG, "chi is not finite");
  if (!S) return fail(c, GW_ERR_ARG, "NULL S");
  if (!gamma != !Sig_inf) return fail(c, GW_ERR_ARG, "gamma and Sig_inf go together");
  if (!G_tau != !Sig_tau || (G_tau && !head))
    return fail(c, GW_ERR_ARG, "G_tau, head and Sig_tau go together");
  if (head)
    for (int i = 0; i < nt; ++i)
      if (!std::isfinite(head[i])) return fail(c, GW_ERR_ARG, "head is not finite");
  if (gamma)
    HIPCHK(c, sxs_add_launch((const double2*)S, (const double2*)gamma, (double2*)Sig_inf, nao, nk, nk,
                             -chi, c->st));
  if (G_tau) {
    // Sigma~(tau_i) += -chi head_i S G(tau_i) S: one launch per tau node
    const size_t slab = (size_t)nk * c->n2;
    for (int i = 0; i < nt; ++i) {
      if (head[i] == 0.0) continue;
      HIPCHK(c, sxs_add_launch((const double2*)S, (const double2*)G_tau + i * slab,
                               (double2*)Sig_tau + i * slab, nao, nk, nk, -chi * head[i], c->st));
    }
  }
  return GW_OK;
}

// ---------------------------------------------------------------- Dyson JVP
gw_status gw_dyson_jvp(gw_ctx* c, const gw_z* S, const gw_z* G_iw, const gw_z* dSinf,
                       const gw_z* dSig_iw, int fixed_mu, gw_z* dG_iw, double* dmu) {
  gw_status s = need_grids(c);
  if (s != GW_OK) return s;
  if (!S || !G_iw || !dG_iw) return fail(c, GW_ERR_ARG, "NULL array");
  if (!c->ws || c->ws_bytes < gw_workspace_bytes(c, GW_OP_DYSON_JVP, 1))
    return fail(c, GW_ERR_WORKSPACE, "dyson_jvp workspace too small");
  const int nk = c->nk, nao = c->d.nao, nw = c->d.nw_f;
  const long long n2 = c->n2, tot = (long long)nw * nk * n2;
  double2* T = (double2*)c->ws;
  double2* P2 = (double2*)((char*)c->ws + align256((size_t)tot * 16));
  const int nb = nw * nk;
  // one product X Y over all (n, k); Y's batch offset is given by its map
  auto prod = [&](const void* A, Map3 ba, const void* B, Map3 bb, void* C, bool acc) -> gw_status {
    GemmDesc g = gemm_desc();
    g.A = A; g.B = B; g.C = C;
    g.M = nao; g.N = nao; g.K = nao; g.batch = nb;
    g.am = aff(nao); g.ak = aff(1); g.bk = aff(nao); g.bn = aff(1);
    g.cm = aff(nao); g.cn = aff(1);
    g.ba = ba; g.bb = bb; g.bc = aff(n2);
    if (acc) { g.beta_zero = 0; g.beta_r = 1.0; }
    g.tag = KC_OTHER;
    const long long eb = bb.sin == n2 ? tot : (long long)nk * n2;
    return run(c, g, Ext{0, tot}, Ext{0, eb}, Ext{0, tot});
  };
  const Map3 per_nk = aff(n2);                  // batch b = n*nk + k -> b * n2
  const Map3 per_k = two(nk, n2, 0);            // -> k * n2
  // dG = G (dSinf + dSig(i w)) G - dmu G S G  (Eq. Dyson differentiated)
  bool have = false;
  if (dSig_iw) {
    if ((s = prod(G_iw, per_nk, dSig_iw, per_nk, T, false)) != GW_OK) return s;
    have = true;
  }
  if (dSinf) {
    if ((s = prod(G_iw, per_nk, dSinf, per_k, T, have)) != GW_OK) return s;
    have = true;
  }
  if (!have) HIPCHK(c, axpby_launch(tot, 0.0, 0.0, nullptr, 0.0, 0.0, T, c->st));
  if ((s = prod(T, per_nk, G_iw, per_nk, dG_iw, false)) != GW_OK) return s;
  double m = 0.0;
  if (!fixed_mu) {
    // dmu keeps N_e = -(ns/Nk) sum Re(r_n tr[G S]) fixed:
    // dmu = sum Re(r_n tr[G dSig G S]) / sum Re(r_n tr[G S G S])
    if ((s = prod(G_iw, per_nk, S, per_k, T, false)) != GW_OK) return s;
    if ((s = prod(T, per_nk, G_iw, per_nk, P2, false)) != GW_OK) return s;
    double t1 = 0.0, t2 = 0.0;
    HIPCHK(c, wtrace_launch((const double2*)dG_iw, (const double2*)S, c->drrow, nao, nk, nw, c->dpart, c->st));
    HIPCHK(c, sum_launch(c->dpart, nb, 1.0, c->dpart + nb, c->st));
    HIPCHK(c, hipMemcpyAsync(&t1, c->dpart + nb, sizeof(double), hipMemcpyDeviceToHost, c->st));
    HIPCHK(c, hipStreamSynchronize(c->st));
    HIPCHK(c, wtrace_launch(P2, (const double2*)S, c->drrow, nao, nk, nw, c->dpart, c->st));
    HIPCHK(c, sum_launch(c->dpart, nb, 1.0, c->dpart + nb, c->st));
    HIPCHK(c, hipMemcpyAsync(&t2, c->dpart + nb, sizeof(double), hipMemcpyDeviceToHost, c->st));
    HIPCHK(c, hipStreamSynchronize(c->st));
    if (!(t2 != 0.0)) return fail(c, GW_ERR_SINGULAR, "dyson_jvp: dN/dmu is zero");
    m = t1 / t2;
    HIPCHK(c, axpby_launch(tot, -m, 0.0, P2, 1.0, 0.0, (double2*)dG_iw, c->st));
  }
  if (dmu) *dmu = m;
  return GW_OK;
}

// =========================================================================
// Whole-chain calls: one Sigma[G] + Pi evaluation and its JVP / VJP, the
// composition of the calls above (Sec. III, Algorithm 1).
// =========================================================================

// Per-q buffers at the end of the workspace (the front is left to the
// sub-calls): two tau arrays and four frequency arrays of naux^2 numbers.
struct PerQ {
  gw_z *ta, *tb, *w0, *w1, *w2, *w3;
};

static gw_status perq_bufs(gw_ctx* c, PerQ& p) {
  if (!c->ws || c->ws_bytes < gw_workspace_bytes(c, GW_OP_SIGMA, c->tc))
    return fail(c, GW_ERR_WORKSPACE, "workspace too small for the whole-chain calls (GW_OP_SIGMA)");
  char* b = (char*)c->ws + ((c->ws_bytes - perq_bytes(c)) & ~size_t(255));
  const size_t tb = perq_tau_bytes(c), wb = perq_w_bytes(c);
  p.ta = (gw_z*)b;
  p.tb = (gw_z*)(b + tb);
  p.w0 = (gw_z*)(b + 2 * tb);
  p.w1 = (gw_z*)(b + 2 * tb + wb);
  p.w2 = (gw_z*)(b + 2 * tb + 2 * wb);
  p.w3 = (gw_z*)(b + 2 * tb + 3 * wb);
  return GW_OK;
}

static gw_status zero_z(gw_ctx* c, gw_z* Y, long long n) {
  HIPCHK(c, axpby_launch(n, 0.0, 0.0, nullptr, 0.0, 0.0, (double2*)Y, c->st));
  return GW_OK;
}

// P (P0^q(tau)) -> P0^q(i Omega) (p.w0) -> P~^q(i Omega) (p.w1) -> P~^q(tau),
// in place.  phi (may be NULL) accumulates this q's Phi~ term.
static gw_status pt_solve(gw_ctx* c, gw_z* P, const PerQ& p, double* phi) {
  gw_status s;
  const long long nn = (long long)c->d.naux * c->d.naux;
  if ((s = gw_tau_to_iw(c, GW_BOSON, P, 1, nn, p.w0)) != GW_OK) return s;
  if (phi) {
    double f = 0.0;
    if ((s = gw_screened_W_phi(c, p.w0, 1, p.w1, &f)) != GW_OK) return s;
    *phi += f;
  } else if ((s = gw_screened_W(c, p.w0, 1, p.w1)) != GW_OK) {
    return s;
  }
  return gw_iw_to_tau(c, GW_BOSON, p.w1, 1, nn, P);
}

// Whether P~ of a G declared Hermitian is Hermitian at every node and mirrors
// between q and -q, so that se_pair applies.  fp64 only (see pol_impl).
// Measured with the polarization pairs in both, whole evaluation on a 3x3x3
// mesh: 98.9 -> 83.3 ms (nao 16, naux 150, ntau 60), 721 -> 566 ms (nao 26,
// naux 250, ntau 100); gw_sigma_jvp at the first of them 241 -> 147 ms.
static bool pairs_ok(const gw_ctx* c, int bits) {
  return !lowp(c) && c->sym_b && (c->herm & bits) == bits;
}

// Boson transform of the matrices of nq q-points, tau -> i Omega at Omega >= 0
// only (forward), or back from all Omega.  reps (device): the q-points, as
// strides of both arrays; NULL for one q at the start of both.
static gw_status half_transform(gw_ctx* c, const gw_z* in, gw_z* out, const int* reps, int nq, bool forward) {
  const int nt = c->d.ntau, nw = c->d.nw_b, mid = c->mid;
  const long long nn = (long long)c->d.naux * c->d.naux;
  if (nn > 0x7fffffffLL) return fail(c, GW_ERR_ARG, "naux out of range");
  GemmDesc g = gemm_desc();
  g.A = forward ? c->dTB + (size_t)mid * nt : c->dTBp;
  g.B = in; g.C = (double2*)out + (forward ? mid * nn : 0);
  g.M = forward ? nw - mid : nt; g.N = (int)nn; g.K = forward ? nt : nw; g.batch = nq;
  g.am = aff(g.K); g.ak = aff(1);
  g.bk = aff(nn); g.bn = aff(1); g.cm = aff(nn); g.cn = aff(1);
  if (reps) {
    g.tab = reps; g.tmod = nq;
    g.tsB = (forward ? nt : nw) * nn; g.tsC = (forward ? nw : nt) * nn;
  }
  g.tag = KC_TRANSFORM;
  const long long all = reps ? c->nk : 1, cut = forward ? mid * nn : 0;
  return run(c, g, Ext{0, (long long)g.M * g.K}, Ext{0, all * g.K * nn},
             Ext{-cut, all * (forward ? nw : nt) * nn - cut});
}

// P~^q of G rebuilt for one q into p.ta and p.w1.  half: pairs_ok holds, so the
// solve at Omega >= 0 gives the rest by P~(-i Omega) = P~(i Omega)^H.
static gw_status pt_one_q(gw_ctx* c, const void* V, const gw_z* G, int q, const PerQ& p, double* phi, bool half) {
  gw_status s = pol_impl(c, ctx_work(c), V, G, G, q, 1, p.ta, false, false);
  if (s != GW_OK || !half || phi) return s != GW_OK ? s : pt_solve(c, p.ta, p, phi);
  const long long cut = (long long)c->mid * c->d.naux * c->d.naux;
  if ((s = half_transform(c, p.ta, p.w0, nullptr, 1, true)) != GW_OK) return s;
  if ((s = solve_core(c, p.w0 + cut, p.w1 + cut, nullptr, c->d.nw_b - c->mid)) != GW_OK) return s;
  HIPCHK(c, spread_launch((double2*)p.w1, nullptr, nullptr, 1, c->d.nw_b, c->mid, c->d.naux, c->st));
  return half_transform(c, p.w1, p.ta, nullptr, 1, false);
}

// P~ of every q with pairs_ok: P0 of one q of each pair, its solves at
// Omega >= 0, and everything else by P(-i Omega) = P(i Omega)^H,
// P^{-q}(i Omega) = conj(P^q(i Omega)), P^{-q}(beta - tau) = P^q(tau)^T: a
// quarter of the solves and half of the transforms.  Whole evaluation on a
// 3x3x3 mesh: 45.2 -> 39.8 ms (nao 16, naux 150), 455 -> 417 ms (nao 26, naux 250).
static gw_status pt_pairs(gw_ctx* c, const void* V, const gw_z* G, gw_z* P_tau, gw_z* P0_iw, gw_z* Pt_iw) {
  const int nt = c->d.ntau, nw = c->d.nw_b, n = c->d.naux, half = nw - c->mid, nrep = c->nrep;
  const long long nn = (long long)n * n, per = nt * nn;
  const int *reps = c->dsel, *negs = c->dsel + nrep, *pos = c->dsel + 2 * nrep;
  gw_status s;
  for (int i = 0; i < nrep; ++i) {
    const int q = c->sel[i];
    const bool self = c->neg[q] == q;
    gw_z* Pq = P_tau + q * per;
    if ((s = pol_nodes(c, ctx_work(c), (const char*)V, (const char*)G, (const char*)G, q, 0, self ? nt / 2 : nt, Pq,
                       self ? Pq : nullptr, false, true)) != GW_OK) return s;
  }
  if ((s = half_transform(c, P_tau, P0_iw, reps, nrep, true)) != GW_OK) return s;
  // as many matrices at once as the workspace holds
  const long long total = (long long)nrep * half;
  const long long mb = std::max(1LL, std::min<long long>(total, (long long)(c->ws_bytes / (nn * 16))));
  for (long long b = 0; b < total; b += mb)
    if ((s = solve_core(c, P0_iw, Pt_iw, pos + b, std::min(mb, total - b))) != GW_OK) return s;
  HIPCHK(c, spread_launch((double2*)P0_iw, reps, negs, nrep, nw, c->mid, n, c->st));
  HIPCHK(c, spread_launch((double2*)Pt_iw, reps, negs, nrep, nw, c->mid, n, c->st));
  if ((s = half_transform(c, Pt_iw, P_tau, reps, nrep, false)) != GW_OK) return s;
  for (int i = 0; i < nrep; ++i) {
    const int q = c->sel[i], m = c->neg[q];
    if (m != q)
      HIPCHK(c, mirror_launch((double2*)P_tau + q * per, (double2*)P_tau + m * per + (nt - 1) * nn, -nn, n, nt, false,
                              c->st));
  }
  return GW_OK;
}

gw_status gw_sigma(gw_ctx* c, const void* V, const gw_z* G, gw_z* gamma, gw_z* Sinf, gw_z* Stau,
                   gw_z* P_tau, gw_z* P0_iw, gw_z* Pt_iw, double* phi) {
  if (!c) return GW_ERR_ARG;
  if (!ready(c)) return fail(c, GW_ERR_STATE, "grids not built (gw_build_grids or gw_set_grids)");
  if (!V || !G || !Sinf || !Stau) return fail(c, GW_ERR_ARG, "NULL array");
  const bool stored = P_tau || P0_iw || Pt_iw;
  if (stored && !(P_tau && P0_iw && Pt_iw))
    return fail(c, GW_ERR_ARG, "P_tau, P0_iw and Pt_iw are given all together or not at all");
  if (stored && P0_iw == Pt_iw) return fail(c, GW_ERR_ARG, "Pt_iw may not alias P0_iw");
  if (phi) *phi = 0.0;
  const int nk = c->nk, naux = c->d.naux;
  const long long nn = (long long)naux * naux;
  PerQ p{};
  gw_status s;
  if (!stored && (s = perq_bufs(c, p)) != GW_OK) return s;
  if ((s = gw_hf(c, V, G, gamma, Sinf)) != GW_OK) return s;
  if ((s = zero_z(c, Stau, (long long)c->d.ntau * nk * c->n2)) != GW_OK) return s;
  double ph = 0.0;
  const bool pairs = pairs_ok(c, GW_HERM_FORWARD);
  if (stored && pairs && !phi) {
    if (!c->ws || c->tc < 1 || c->ws_bytes < chain_bytes(c, c->tc))
      return fail(c, GW_ERR_WORKSPACE, "polarization workspace too small");
    if (c->ws_bytes < screened_bytes(c, 1)) return fail(c, GW_ERR_WORKSPACE, "screened_W workspace too small");
    if ((s = pt_pairs(c, V, G, P_tau, P0_iw, Pt_iw)) != GW_OK) return s;
    for (int q = 0; q < nk; ++q)
      if (c->neg[q] >= q && (s = se_pair(c, V, G, P_tau + (size_t)q * c->d.ntau * nn, q, Stau)) != GW_OK)
        return s;
  } else if (stored) {
    if ((s = pol_impl(c, ctx_work(c), V, G, G, 0, nk, P_tau, false, false)) != GW_OK) return s;
    if ((s = gw_tau_to_iw(c, GW_BOSON, P_tau, nk, nn, P0_iw)) != GW_OK) return s;
    // screened-interaction solves in q-batches as large as the workspace holds
    const size_t per = screened_bytes(c, 1);
    const int qb = (int)std::max<size_t>(1, std::min<size_t>((size_t)nk, c->ws_bytes / per));
    for (int q0 = 0; q0 < nk; q0 += qb) {
      const int nq = std::min(qb, nk - q0);
      const size_t off = (size_t)q0 * c->d.nw_b * nn;
      if (phi) {
        double f = 0.0;
        if ((s = gw_screened_W_phi(c, P0_iw + off, nq, Pt_iw + off, &f)) != GW_OK) return s;
        ph += f;
      } else if ((s = gw_screened_W(c, P0_iw + off, nq, Pt_iw + off)) != GW_OK) {
        return s;
      }
    }
    if ((s = gw_iw_to_tau(c, GW_BOSON, Pt_iw, nk, nn, P_tau)) != GW_OK) return s;
    if (!pairs) {
      if ((s = gw_self_energy(c, V, G, P_tau, 0, nk, Stau)) != GW_OK) return s;
    } else {
      for (int q = 0; q < nk; ++q)
        if (c->neg[q] >= q && (s = se_pair(c, V, G, P_tau + (size_t)q * c->d.ntau * nn, q, Stau)) != GW_OK)
          return s;
    }
  } else if (lowp(c)) {
    for (int q = 0; q < nk; ++q) {
      if ((s = pt_one_q(c, V, G, q, p, phi ? &ph : nullptr, false)) != GW_OK) return s;
      if ((s = gw_self_energy(c, V, G, p.ta, q, 1, Stau)) != GW_OK) return s;
    }
  } else {
    const bool herm = (c->herm & GW_HERM_FORWARD) != 0;
    for (int q = 0; q < nk; ++q) {
      const int m = c->neg[q];
      if (m < q) continue;
      if (m == q || pairs) {
        double f = 0.0;
        if ((s = pt_one_q(c, V, G, q, p, phi ? &f : nullptr, pairs)) != GW_OK) return s;
        ph += m == q ? f : 2.0 * f;      // -q has the same Phi~ term
        s = pairs ? se_pair(c, V, G, p.ta, q, Stau) : gw_self_energy(c, V, G, p.ta, q, 1, Stau);
        if (s != GW_OK) return s;
        continue;
      }
      // P0^{-q} by transposition, then one q after the other
      if ((s = pol_nodes(c, ctx_work(c), (const char*)V, (const char*)G, (const char*)G, q, 0, c->d.ntau, p.ta,
                         p.tb, false, herm)) != GW_OK) return s;
      if ((s = pt_solve(c, p.ta, p, phi ? &ph : nullptr)) != GW_OK) return s;
      if ((s = gw_self_energy(c, V, G, p.ta, q, 1, Stau)) != GW_OK) return s;
      if ((s = pt_solve(c, p.tb, p, phi ? &ph : nullptr)) != GW_OK) return s;
      if ((s = gw_self_energy(c, V, G, p.tb, m, 1, Stau)) != GW_OK) return s;
    }
  }
  if (phi) {
    HIPCHK(c, hipStreamSynchronize(c->st));
    *phi = ph;
  }
  return GW_OK;
}

// Shared checks of the derivative calls; sets *stored.
static gw_status deriv_args(gw_ctx* c, const void* V, const gw_z* G, const gw_z* Pt_tau,
                            const gw_z* Pt_iw, bool* stored) {
  if (!V || !G) return fail(c, GW_ERR_ARG, "NULL array");
  if (!Pt_tau != !Pt_iw) return fail(c, GW_ERR_ARG, "Pt_tau and Pt_iw are given together or not at all");
  *stored = Pt_tau != nullptr;
  return GW_OK;
}

gw_status gw_sigma_jvp(gw_ctx* c, const void* V, const gw_z* G, const gw_z* Pt_tau, const gw_z* Pt_iw,
                       const gw_z* dG, gw_z* dSinf, gw_z* dStau) {
  gw_status s = need_grids(c);
  if (s != GW_OK) return s;
  bool stored = false;
  if ((s = deriv_args(c, V, G, Pt_tau, Pt_iw, &stored)) != GW_OK) return s;
  if (!dG || !dSinf || !dStau) return fail(c, GW_ERR_ARG, "NULL array");
  PerQ p{};
  if ((s = perq_bufs(c, p)) != GW_OK) return s;
  const int nk = c->nk, nt = c->d.ntau, nwb = c->d.nw_b;
  const long long nn = (long long)c->d.naux * c->d.naux;
  // dSigma_inf = HF[gamma(dG)] (linear in G)
  if ((s = gw_hf(c, V, dG, nullptr, dSinf)) != GW_OK) return s;
  if ((s = zero_z(c, dStau, (long long)nt * nk * c->n2)) != GW_OK) return s;
  const bool pairs = pairs_ok(c, GW_HERM_FORWARD | GW_HERM_TWO_SLOT);
  for (int q = 0; q < nk; ++q) {
    const gw_z* pt = stored ? Pt_tau + (size_t)q * nt * nn : p.ta;
    const gw_z* pw = stored ? Pt_iw + (size_t)q * nwb * nn : p.w1;
    if (pairs && c->neg[q] < q) continue;
    if (!stored && (s = pt_one_q(c, V, G, q, p, nullptr, pairs)) != GW_OK) return s;
    // dP0 = P0[dG, G] + P0[G, dG]
    if (pairs) {
      // the sum is symmetric in its slots, so it mirrors as P0[G, G] does
      const char *Vd = (const char*)V, *Gd = (const char*)G, *dGd = (const char*)dG;
      const bool self = c->neg[q] == q;
      const int te = self ? nt / 2 : nt;
      if ((s = pol_nodes(c, ctx_work(c), Vd, dGd, Gd, q, 0, te, p.tb, self ? p.tb : nullptr, false,
                         true, Gd, dGd)) != GW_OK) return s;
    } else if (!lowp(c)) {
      const bool herm = (c->herm & GW_HERM_TWO_SLOT) != 0;
      if ((s = pol_nodes(c, ctx_work(c), (const char*)V, (const char*)dG, (const char*)G, q, 0, nt, p.tb,
                         nullptr, false, herm, (const char*)G, (const char*)dG)) != GW_OK) return s;
    } else {
      if ((s = pol_impl(c, ctx_work(c), V, dG, G, q, 1, p.tb, false, true)) != GW_OK) return s;
      if ((s = pol_impl(c, ctx_work(c), V, G, dG, q, 1, p.tb, true, true)) != GW_OK) return s;
    }
    // dP~(i Omega) = (I + P~) dP0(i Omega) (I + P~)
    if ((s = gw_tau_to_iw(c, GW_BOSON, p.tb, 1, nn, p.w2)) != GW_OK) return s;
    if ((s = gw_screened_W_lin(c, pw, p.w2, 1, 0, p.w3)) != GW_OK) return s;
    if ((s = gw_iw_to_tau(c, GW_BOSON, p.w3, 1, nn, p.tb)) != GW_OK) return s;
    // dSigma~ += Sigma~[dP~, G] + Sigma~[P~, dG]
    if (pairs) {
      if ((s = se_pair(c, V, G, p.tb, q, dStau)) != GW_OK) return s;
      if ((s = se_pair(c, V, dG, pt, q, dStau)) != GW_OK) return s;
      continue;
    }
    if ((s = gw_self_energy(c, V, G, p.tb, q, 1, dStau)) != GW_OK) return s;
    if ((s = gw_self_energy(c, V, dG, pt, q, 1, dStau)) != GW_OK) return s;
  }
  return GW_OK;
}

gw_status gw_sigma_vjp(gw_ctx* c, const void* V, const gw_z* G, const gw_z* Pt_tau, const gw_z* Pt_iw,
                       const gw_z* Sinf_bar, const gw_z* Stau_bar, gw_z* G_bar) {
  gw_status s = need_grids(c);
  if (s != GW_OK) return s;
  bool stored = false;
  if ((s = deriv_args(c, V, G, Pt_tau, Pt_iw, &stored)) != GW_OK) return s;
  if (!Sinf_bar || !Stau_bar || !G_bar) return fail(c, GW_ERR_ARG, "NULL array");
  PerQ p{};
  if ((s = perq_bufs(c, p)) != GW_OK) return s;
  const int nk = c->nk, nt = c->d.ntau, nwb = c->d.nw_b;
  const long long nn = (long long)c->d.naux * c->d.naux;
  if ((s = zero_z(c, G_bar, (long long)nt * nk * c->n2)) != GW_OK) return s;
  if (!lowp(c)) {
    // P0^{-q}(beta - tau) = P0^q(tau)^T for any G (see pol_impl), so the
    // cotangents of q and -q add up, P0bar^q(tau) + P0bar^{-q}(beta - tau)^T,
    // before one polarization adjoint for both (half of the nodes for q = -q).
    // Measured with the triple products, 3x3x3, nao 16, naux 150: 251 -> 116 ms.
    // Where P~ is rebuilt here, from a G that is Hermitian by the mode's
    // statement, the P~ V of -q also comes from that of q as in se_nodes.  A
    // given P~ is read for every q: the mode states nothing of it or of its G
    // (taking its -q from q gave 103 ms, and a wrong gradient at a general G).
    const bool pairs = !stored && pairs_ok(c, GW_HERM_FORWARD);
    const long long per = nt * nn;
    // from P~bar(tau) in place to P0bar(tau)
    auto back = [&](gw_z* P, const gw_z* pw) -> gw_status {
      gw_status r;
      if ((r = gw_transform_adjoint(c, GW_BOSON, 1, P, 1, nn, p.w2)) != GW_OK) return r;
      if ((r = gw_screened_W_lin(c, pw, p.w2, 1, 1, p.w3)) != GW_OK) return r;
      return gw_transform_adjoint(c, GW_BOSON, 0, p.w3, 1, nn, P);
    };
    for (int q = 0; q < nk; ++q) {
      const int m = c->neg[q];
      if (m < q) continue;
      for (int half = 0; half < (m == q ? 1 : 2); ++half) {
        const int z = half ? m : q;
        const gw_z* Vz = (const gw_z*)V + (size_t)z * nk * c->sv;
        gw_z* Pb = half ? p.ta : p.tb;               // p.ta is free once P~ V is done
        if (!stored && (s = pt_one_q(c, V, G, z, p, nullptr, pairs)) != GW_OK) return s;
        const gw_z* pt = stored ? Pt_tau + (size_t)z * per : p.ta;
        const gw_z* pw = stored ? Pt_iw + (size_t)z * nwb * nn : p.w1;
        if (!half || !pairs) {
          const bool self = m == q;
          if ((s = se_vjp_g(c, Vz, pt, Stau_bar, z, pairs && self ? nt / 2 : nt, G_bar, pairs)) != GW_OK) return s;
        }
        if ((s = se_vjp_p(c, Vz, G, Stau_bar, z, Pb)) != GW_OK) return s;
        if ((s = back(Pb, pw)) != GW_OK) return s;
      }
      const gw_z* Vq = (const gw_z*)V + (size_t)q * nk * c->sv;
      const int te = m == q ? nt / 2 : nt;
      HIPCHK(c, add_transpose_launch((double2*)p.tb, (double2*)(m == q ? p.tb : p.ta) + (nt - 1) * nn, c->d.naux, te,
                                     c->st));
      if ((s = pol_vjp_q(c, Vq, G, p.tb, q, te, G_bar)) != GW_OK) return s;
    }
    return gw_hf_vjp(c, V, Sinf_bar, G_bar);
  }
  for (int q = 0; q < nk; ++q) {
    const gw_z* pt = stored ? Pt_tau + (size_t)q * nt * nn : p.ta;
    const gw_z* pw = stored ? Pt_iw + (size_t)q * nwb * nn : p.w1;
    if (!stored && (s = pt_one_q(c, V, G, q, p, nullptr, false)) != GW_OK) return s;
    // Sigma~ = SE[P~, G]: G part into G_bar, P~ part into P_bar (p.tb)
    if ((s = gw_self_energy_vjp(c, V, G, pt, Stau_bar, q, 1, G_bar, p.tb)) != GW_OK) return s;
    // back through i Omega -> tau, the screened-interaction solve, tau -> i Omega
    if ((s = gw_transform_adjoint(c, GW_BOSON, 1, p.tb, 1, nn, p.w2)) != GW_OK) return s;
    if ((s = gw_screened_W_lin(c, pw, p.w2, 1, 1, p.w3)) != GW_OK) return s;
    if ((s = gw_transform_adjoint(c, GW_BOSON, 0, p.w3, 1, nn, p.tb)) != GW_OK) return s;
    // both G slots of the polarization
    if ((s = gw_polarization_vjp(c, V, G, p.tb, q, 1, G_bar)) != GW_OK) return s;
  }
  return gw_hf_vjp(c, V, Sinf_bar, G_bar);
}

// ------------------------------------------- thermodynamics (Sec. III.C) ---
// Eigenvalues of the Hermitian pencil (H, S), S positive definite: Cholesky
// S = L L^H, A = L^{-1} H L^{-H}, cyclic complex Jacobi rotations on A.
static bool pencil_eigenvalues(const gwgrid::cd* H, const gwgrid::cd* S, int n, double* ev) {
  using cd = gwgrid::cd;
  std::vector<cd> L((size_t)n * n, 0.0), A((size_t)n * n), X((size_t)n * n);
  for (int j = 0; j < n; ++j) {
    double d = S[(size_t)j * n + j].real();
    for (int p = 0; p < j; ++p) d -= std::norm(L[(size_t)j * n + p]);
    if (!(d > 0.0)) return false;
    L[(size_t)j * n + j] = std::sqrt(d);
    for (int i = j + 1; i < n; ++i) {
      cd v = S[(size_t)i * n + j];
      for (int p = 0; p < j; ++p) v -= L[(size_t)i * n + p] * std::conj(L[(size_t)j * n + p]);
      L[(size_t)i * n + j] = v / L[(size_t)j * n + j];
    }
  }
  // X = L^{-1} M for a square M (forward substitution per column)
  auto lsolve = [&](const std::vector<cd>& M, std::vector<cd>& out) {
    for (int c = 0; c < n; ++c)
      for (int i = 0; i < n; ++i) {
        cd v = M[(size_t)i * n + c];
        for (int p = 0; p < i; ++p) v -= L[(size_t)i * n + p] * out[(size_t)p * n + c];
        out[(size_t)i * n + c] = v / L[(size_t)i * n + i];
      }
  };
  std::vector<cd> Hm(H, H + (size_t)n * n), Y((size_t)n * n);
  lsolve(Hm, X);                                       // X = L^{-1} H
  for (int i = 0; i < n; ++i)
    for (int j = 0; j < n; ++j) Y[(size_t)i * n + j] = std::conj(X[(size_t)j * n + i]);
  lsolve(Y, A);                                        // A = L^{-1} X^H = (X L^{-H})^H
  for (int i = 0; i < n; ++i)                          // A is Hermitian: make it exactly so
    for (int j = i; j < n; ++j) {
      const cd v = 0.5 * (A[(size_t)i * n + j] + std::conj(A[(size_t)j * n + i]));
      A[(size_t)i * n + j] = v;
      A[(size_t)j * n + i] = std::conj(v);
    }
  for (int sweep = 0; sweep < 100; ++sweep) {
    double off = 0.0, tot = 0.0;
    for (int i = 0; i < n; ++i)
      for (int j = 0; j < n; ++j) {
        tot += std::norm(A[(size_t)i * n + j]);
        if (i != j) off += std::norm(A[(size_t)i * n + j]);
      }
    if (off <= 1e-30 * tot) break;
    for (int p = 0; p < n; ++p)
      for (int q = p + 1; q < n; ++q) {
        const cd b = A[(size_t)p * n + q];
        const double ab = std::abs(b);
        if (ab == 0.0) continue;
        const cd ph = b / ab;                           // e^{i phi}
        const double a = A[(size_t)p * n + p].real(), d = A[(size_t)q * n + q].real();
        const double tau = (d - a) / (2.0 * ab);
        const double t = (tau >= 0.0 ? 1.0 : -1.0) / (std::fabs(tau) + std::sqrt(1.0 + tau * tau));
        const double c = 1.0 / std::sqrt(1.0 + t * t), sn = t * c;
        for (int k = 0; k < n; ++k) {                   // A <- A U
          const cd x = A[(size_t)k * n + p], y = A[(size_t)k * n + q];
          A[(size_t)k * n + p] = c * x - sn * std::conj(ph) * y;
          A[(size_t)k * n + q] = sn * x + c * std::conj(ph) * y;
        }
        for (int k = 0; k < n; ++k) {                   // A <- U^H A
          const cd x = A[(size_t)p * n + k], y = A[(size_t)q * n + k];
          A[(size_t)p * n + k] = c * x - sn * ph * y;
          A[(size_t)q * n + k] = sn * x + c * ph * y;
        }
      }
  }
  for (int i = 0; i < n; ++i) ev[i] = A[(size_t)i * n + i].real();
  return true;
}

gw_status gw_thermodynamics(gw_ctx* c, const gw_z* H0, const gw_z* S, const gw_z* Sinf, const gw_z* Siw,
                            double mu, double phi_tilde, gw_thermo* out) {
  gw_status s = need_grids(c);
  if (s != GW_OK) return s;
  if (!H0 || !S || !out) return fail(c, GW_ERR_ARG, "NULL array");
  if (!std::isfinite(mu) || !std::isfinite(phi_tilde)) return fail(c, GW_ERR_ARG, "mu or phi_tilde is not finite");
  if (!c->ws || c->ws_bytes < gw_workspace_bytes(c, GW_OP_THERMO, 1))
    return fail(c, GW_ERR_WORKSPACE, "thermodynamics workspace too small (GW_OP_THERMO)");
  const int nk = c->nk, nao = c->d.nao, nw = c->d.nw_f, ns = c->d.ns;
  const long long n2 = c->n2, nb = (long long)nw * nk;
  char* p = (char*)c->ws;
  double2* Giw = (double2*)p;                     // G(i w) [n][k][i][j]
  p += align256((size_t)nb * n2 * 16);
  double* ld = (double*)p;                        // ln|det M|
  p += align256((size_t)nb * 8);
  double* ldr = (double*)p;                       // ln|det M_ref|
  p += align256((size_t)nb * 8);
  double* tr = (double*)p;                        // per-(n, k) weighted traces
  p += align256((size_t)nb * 8);
  double2* gam = (double2*)p;                     // gamma [k][i][j]
  p += align256((size_t)nk * n2 * 16);
  double2* cw = (double2*)p;                      // (c_n, 0): c_n = -Re r_n
  p += align256((size_t)nw * 16);
  double* trk = (double*)p;                       // per-k traces
  // Dyson at mu with and without Sigma~ (log-determinants), G(i w) kept
  HIPCHK(c, zero_flag_launch(c->dflag, c->st));
  DysonArgs a{};
  a.H0 = (const double2*)H0; a.S = (const double2*)S; a.Sinf = (const double2*)Sinf;
  a.Siw = (const double2*)Siw; a.wF = c->dwF; a.rrow = c->drrow; a.mu = mu; a.nk = nk; a.nao = nao;
  a.flag = c->dflag; a.G = Giw; a.logdet = ld;
  HIPCHK(c, dyson_any(c, a, 1));
  a.Siw = nullptr; a.G = nullptr; a.logdet = ldr;
  HIPCHK(c, dyson_any(c, a, 1));
  if ((s = read_flag(c, "thermodynamics")) != GW_OK) return s;
  // gamma = -G(beta^-) = -sum_n r_n G(i w_n)
  GemmDesc g = gemm_desc();
  g.A = c->drrow; g.B = Giw; g.C = gam;
  g.M = 1; g.N = nk * (int)n2; g.K = nw;
  g.am = aff(0); g.ak = aff(1); g.bk = aff((long long)nk * n2); g.bn = aff(1);
  g.cm = aff(0); g.cn = aff(1);
  g.alpha_r = -1.0;
  g.tag = KC_OTHER;
  if ((s = run(c, g, Ext{0, (long long)nw}, Ext{0, nb * n2}, Ext{0, (long long)nk * n2})) != GW_OK) return s;
  // Matsubara-sum weights of decaying fermionic functions: c_n = -Re r_n
  std::vector<double2> cwh(nw);
  std::vector<double> cnh(nw);
  for (int n = 0; n < nw; ++n) {
    cnh[n] = -c->rrow[n].real();
    cwh[n] = double2{cnh[n], 0.0};
  }
  HIPCHK(c, hipMemcpyAsync(cw, cwh.data(), nw * sizeof(double2), hipMemcpyHostToDevice, c->st));
  if (Siw) HIPCHK(c, wtrace_launch((const double2*)Siw, Giw, cw, nao, nk, nw, tr, c->st, 1));
  // per-k traces tr[gamma X] for X = S, H0, Sigma_inf
  std::vector<double> t_s(nk), t_h(nk), t_x(nk, 0.0), t_dyn(nb, 0.0), lm(nb), lr(nb);
  HIPCHK(c, trace_launch(gam, (const double2*)S, nao, nk, trk, c->st));
  HIPCHK(c, hipMemcpyAsync(t_s.data(), trk, nk * sizeof(double), hipMemcpyDeviceToHost, c->st));
  HIPCHK(c, trace_launch(gam, (const double2*)H0, nao, nk, trk + nk, c->st));
  HIPCHK(c, hipMemcpyAsync(t_h.data(), trk + nk, nk * sizeof(double), hipMemcpyDeviceToHost, c->st));
  if (Sinf) {
    HIPCHK(c, trace_launch(gam, (const double2*)Sinf, nao, nk, trk + 2 * nk, c->st));
    HIPCHK(c, hipMemcpyAsync(t_x.data(), trk + 2 * nk, nk * sizeof(double), hipMemcpyDeviceToHost, c->st));
  }
  if (Siw) HIPCHK(c, hipMemcpyAsync(t_dyn.data(), tr, nb * sizeof(double), hipMemcpyDeviceToHost, c->st));
  HIPCHK(c, hipMemcpyAsync(lm.data(), ld, nb * sizeof(double), hipMemcpyDeviceToHost, c->st));
  HIPCHK(c, hipMemcpyAsync(lr.data(), ldr, nb * sizeof(double), hipMemcpyDeviceToHost, c->st));
  // the static pencil (H0 + Sigma_inf, S) on the host
  std::vector<gwgrid::cd> hh((size_t)nk * n2), ss((size_t)nk * n2), xx((size_t)nk * n2, 0.0);
  HIPCHK(c, hipMemcpyAsync(hh.data(), H0, hh.size() * 16, hipMemcpyDeviceToHost, c->st));
  HIPCHK(c, hipMemcpyAsync(ss.data(), S, ss.size() * 16, hipMemcpyDeviceToHost, c->st));
  if (Sinf) HIPCHK(c, hipMemcpyAsync(xx.data(), Sinf, xx.size() * 16, hipMemcpyDeviceToHost, c->st));
  HIPCHK(c, hipStreamSynchronize(c->st));
  const double beta = c->d.beta, pre = (double)ns / nk;
  double free_sum = 0.0;
  std::vector<double> ev(nao);
  for (int k = 0; k < nk; ++k) {
    std::vector<gwgrid::cd> hk(hh.begin() + (size_t)k * n2, hh.begin() + (size_t)(k + 1) * n2);
    for (long long e = 0; e < n2; ++e) hk[e] += xx[(size_t)k * n2 + e];
    if (!pencil_eigenvalues(hk.data(), &ss[(size_t)k * n2], nao, ev.data()))
      return fail(c, GW_ERR_ARG, "S is not positive definite");
    for (int i = 0; i < nao; ++i) {
      const double xi = ev[i] - mu;
      free_sum += std::max(-xi, 0.0) + std::log1p(std::exp(-beta * std::fabs(xi))) / beta;
    }
  }
  double ln_dyn = 0.0, sg_dyn = 0.0, ne = 0.0, e1 = 0.0, xs = 0.0;
  for (int n = 0; n < nw; ++n)
    for (int k = 0; k < nk; ++k) {
      const size_t i = (size_t)n * nk + k;
      ln_dyn += cnh[n] * (lm[i] - lr[i]);
      sg_dyn += t_dyn[i];
    }
  for (int k = 0; k < nk; ++k) {
    ne += t_s[k];
    e1 += t_h[k];
    xs += t_x[k];
  }
  gw_thermo o{};
  o.tr_ln = pre * (free_sum + ln_dyn);
  o.tr_sigma_g = pre * (xs + sg_dyn);
  o.phi_inf = 0.5 * pre * xs;
  o.phi_tilde = phi_tilde;
  o.omega = o.phi_inf + o.phi_tilde - o.tr_ln - o.tr_sigma_g;
  o.e_one_body = pre * e1;
  o.e_gm = o.e_one_body + 0.5 * o.tr_sigma_g;
  o.n_e = pre * ne;
  if (!std::isfinite(o.omega) || !std::isfinite(o.e_gm))
    return fail(c, GW_ERR_NONFINITE, "thermodynamics: non-finite result");
  *out = o;
  return GW_OK;
}

}  // extern "C"
