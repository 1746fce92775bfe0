// Depth-coupled acceptance loss with verify-gated masking, and its gradient in
// the head logits (Sec. "The Depth-Coupled Acceptance Loss", "Learning up to
// the First Rejection"; App. "DCA", Eqs. alpha, chain, dca, vgm, dca-partial,
// dca-tail, dca-coeff), over the cycle record's sparse support: the head
// distribution q = softmax(z) is normalised over the whole vocabulary and
// gathered at the record's ids S, and the mass outside S forms one residual
// bin (App. "Implementing Draft-Path Reconstruction in verl").
//
//  1. The row-statistics pass over the head logits (max and sum exp per chunk).
//  2. One block per cycle, one wave per draft position: q and p on S (float64),
//     alpha_k, the subgradient flags [q < p] of min, then the chain (one
//     thread): M = sum_{l<=L} prod_{i<=l} alpha_i, the loss -log M, and the
//     coefficient of position k, -(prod_{i<k} alpha_i) D_k / M (0 past L).
//  3. The gradient pass, one block per (row, 4096 ids): coef * q_x * (g_x - gbar)
//     with g_x the residual bin's flag; the block then rewrites the ids of S
//     that fall in its range with their own flags.
#include "common.h"
#include "forward.h"

namespace gm {

namespace {
struct DcaRow {          // per (cycle, position): what the gradient pass needs
  double coef, gbar, M, inv_s;
  int g_rest, pad;
};
constexpr int kDcaIds = 4096;   // ids per block of the gradient pass
// The gradient pass by the bytes of the gradient (as many logits are read):
//  up to the XCDs' L2s (8 x 4 MB)    DCA_SMALL   the row statistics have just brought the logits there
//  below the last-level cache        DCA_MEDIUM
//  from that on                      DCA_STREAM  stored past the caches (1.9 GB: 2% off the launch;
//                                                62 MB: 48 us past them, 43 through them)
// With rows a multiple of eight and without masking, where no row can be left unread, DCA_SMALL goes on to 96 MB
// (34 x 4 x 128256, 70 MB: 47.3 us, 48.9 DCA_MEDIUM; 64 x 3 x 151936, 117 MB: 70.2 and 68.4).
enum { DCA_SMALL, DCA_MEDIUM, DCA_STREAM };
constexpr size_t kDcaSmallBytes = size_t(32) << 20, kDcaRowBytes = size_t(96) << 20;
constexpr size_t kDcaStreamBytes = size_t(256) << 20;

__device__ __forceinline__ float bf16_to_f32(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

__global__ __launch_bounds__(1024) void dca_cycle_kernel(int K, int V, int topk, int vgm,
                                                         const float *__restrict__ z,
                                                         const RowStat *__restrict__ stats, int nch,
                                                         const uint16_t *__restrict__ rec_logp,
                                                         const int32_t *__restrict__ rec_ids,
                                                         const int32_t *__restrict__ n_accept,
                                                         float *__restrict__ loss, float *__restrict__ alpha_out,
                                                         DcaRow *__restrict__ rows, uint8_t *__restrict__ flags) {
  __shared__ double sh_alpha[16];
  const int n = blockIdx.x, k = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const long r = (long)n * K + k;
  // q's normaliser from the chunk statistics
  double M = 0.0, S = 1.0;
  int am = 0;
  {
    const RowStat *st = stats + r * nch;
    float m = -INFINITY;
    for (int c = 0; c < nch; ++c) m = fmaxf(m, st[c].max);
    double s = 0.0;
    for (int c = 0; c < nch; ++c) s += st[c].sum * exp((double)st[c].max - (double)m);
    M = (double)m;
    S = s;
    (void)am;
  }
  double p = 0.0, q = 0.0;
  if (lane < topk) {
    const int id = rec_ids[r * topk + lane];
    p = exp((double)bf16_to_f32(rec_logp[r * topk + lane]));
    q = (id >= 0 && id < V) ? exp((double)z[r * V + id] - M) / S : 0.0;
  }
  const double sum_p = wave_sum(p), sum_q = wave_sum(q), sum_min = wave_sum(fmin(p, q));
  const double pR = fmax(0.0, 1.0 - sum_p), qR = 1.0 - sum_q;
  const double alpha = sum_min + fmin(pR, qR);
  const int g = q < p, g_rest = qR < pR;
  const double gbar = wave_sum(lane < topk && g ? q : 0.0) + (g_rest ? qR : 0.0);
  if (lane < topk) flags[r * topk + lane] = (uint8_t)g;
  if (lane == 0) {
    sh_alpha[k] = alpha;
    alpha_out[r] = (float)alpha;
    rows[r].gbar = gbar;
    rows[r].M = M;
    rows[r].inv_s = 1.0 / S;
    rows[r].g_rest = g_rest;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    int L = K;
    if (vgm) {
      const int na = n_accept[n];
      L = na + 1 < K ? (na + 1 < 1 ? 1 : na + 1) : K;
    }
    double chain = 0.0, pre = 1.0;
    for (int l = 0; l < L; ++l) {
      pre *= sh_alpha[l];
      chain += pre;
    }
    loss[n] = (float)(-log(chain));
    double before = 1.0;
    for (int kk = 0; kk < K; ++kk) {
      double coef = 0.0;
      if (kk < L) {
        double D = 0.0, t = 1.0;   // D_k = sum_{l=k}^{L} prod_{i=k+1}^{l} alpha_i
        for (int l = kk; l < L; ++l) {
          if (l > kk) t *= sh_alpha[l];
          D += t;
        }
        coef = -before * D / chain;
      }
      rows[(long)n * K + kk].coef = coef;
      before *= sh_alpha[kk];
    }
  }
}

// kDcaIds ids of one row per block, 16 bytes per load and store where every row is aligned to them (VEC), else
// one id each.
//  DCA_MEDIUM, DCA_STREAM: nch blocks per row, neighbouring blocks on neighbouring ids, all loads of a thread
// issued before the first exponential.  A row past the first rejection has coefficient 0: its gradient is
// written without reading its logits (a quarter of the rows with accepted lengths uniform in 0..3).
//  DCA_SMALL: the logits of every row are loaded, not behind the load of the row's coefficient, by a grid of
// rows x nch, the row statistics' order: with rows a multiple of eight a row's logits are in the L2 of the
// XCD that reads them.  There a thread's 16-byte loads and stores alternate.
// Whole loss, us (cycles x positions x ids; every size row by row, in scalars off 16 bytes, -> here):
// 8 x 3 x 151936 19.0 -> 18.9 (DCA_MEDIUM 21.4), 16 x 4 x 128256 28.8 -> 29.3 (all loads first 30.1), 64 x 3 x 151936
// 67.9 -> 64.0 (DCA_SMALL 68.1), 100 x 3 x 50257 58.7 -> 42.8 (45.7), 500 x 3 x 50257 332 -> 187, 1024 x 3 x 151936
// 1069 -> 882.
template <bool VEC, int MODE>
__global__ __launch_bounds__(256) void dca_grad_kernel(int V, int topk, int nch, const float *__restrict__ z,
                                                       const DcaRow *__restrict__ rows,
                                                       const int32_t *__restrict__ rec_ids,
                                                       const uint8_t *__restrict__ flags, float *__restrict__ grad) {
  const bool flat = gridDim.y == 1;
  const long r = flat ? blockIdx.x / (unsigned)nch : blockIdx.x;
  const int lo = (int)(flat ? blockIdx.x % (unsigned)nch : blockIdx.y) * kDcaIds, hi = min(V, lo + kDcaIds);
  const float *zr = z + r * V;
  float *gr = grad + r * V;
  const bool want = MODE == DCA_SMALL || rows[r].coef != 0.0;
  // the record's ids in this range carry their own flags; read beside the row's logits
  int own_id = -1;
  if (want && (int)threadIdx.x < topk) own_id = rec_ids[r * topk + threadIdx.x];
  constexpr int kVec = kDcaIds / (4 * 256);
  auto load = [&](int u, float (&v)[4]) {
    if constexpr (VEC) {
      const int x = lo + 4 * ((int)threadIdx.x + 256 * u);
      const floatx4_t f = want && x < hi ? *reinterpret_cast<const floatx4_t *>(zr + x) : floatx4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int q = 0; q < 4; ++q) v[q] = f[q];
    } else {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int x = lo + (int)threadIdx.x + 256 * (4 * u + q);
        v[q] = want && x < hi ? zr[x] : 0.f;
      }
    }
  };
  constexpr bool kAhead = !(VEC && MODE == DCA_SMALL);
  float v[kAhead ? kVec : 1][4];
  if constexpr (kAhead) {
#pragma unroll
    for (int u = 0; u < kVec; ++u) load(u, v[u]);
  }
  const DcaRow d = rows[r];
  const float coef = (float)d.coef, M = (float)d.M, inv_s = (float)d.inv_s;
  const float rest = (float)((double)d.g_rest - d.gbar);
  const bool zero = d.coef == 0.0;
  float own_z = 0.f;
  int own_flag = 0;
  auto load_own = [&]() {
    if (zero || own_id < lo || own_id >= hi) own_id = -1;
    if (own_id < 0) return;
    own_z = zr[own_id];
    own_flag = flags[r * topk + threadIdx.x];
  };
  auto store = [&](int u, const float (&w)[4]) {
    floatx4_t o = {0.f, 0.f, 0.f, 0.f};
    if (!zero) {
#pragma unroll
      for (int q = 0; q < 4; ++q) o[q] = coef * (expf(w[q] - M) * inv_s) * rest;
    }
    if constexpr (VEC) {
      const int x = lo + 4 * ((int)threadIdx.x + 256 * u);
      if (x >= hi) return;
      if (MODE == DCA_STREAM) __builtin_nontemporal_store(o, reinterpret_cast<floatx4_t *>(gr + x));
      else *reinterpret_cast<floatx4_t *>(gr + x) = o;
    } else {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int x = lo + (int)threadIdx.x + 256 * (4 * u + q);
        if (x < hi) gr[x] = o[q];
      }
    }
  };
  if constexpr (kAhead) {
    load_own();
#pragma unroll
    for (int u = 0; u < kVec; ++u) store(u, v[u]);
  } else {
#pragma unroll 1
    for (int u = 0; u < kVec; ++u) {
      load(u, v[0]);
      store(u, v[0]);
    }
    load_own();   // (behind the logits, which need not wait for the record's ids)
  }
  // written over the rest's, behind the block's stores above; those past the caches are waited for
  if (MODE == DCA_STREAM) {
    if (!__syncthreads_or(own_id >= 0)) return;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  }
  __syncthreads();
  if (own_id >= 0) gr[own_id] = coef * (expf(own_z - M) * inv_s) * (float)((double)own_flag - d.gbar);
}
}  // namespace

size_t dca_workspace(int N, int K, int V) {
  Carve c;
  c.take(sizeof(RowStat) * (size_t)N * K * stat_chunks(V));
  c.take(sizeof(DcaRow) * (size_t)N * K);
  c.take((size_t)N * K * kRecMaxTopk);
  return c.off;
}

void run_dca_loss(int N, int K, int V, int topk, const float *head_logits, const uint16_t *rec_logp,
                  const int32_t *rec_ids, const int32_t *n_accept, int vgm, float *loss, float *alpha, float *grad,
                  char *ws, hipStream_t s) {
  Carve c;
  RowStat *stats = (RowStat *)(ws + c.take(sizeof(RowStat) * (size_t)N * K * stat_chunks(V)));
  DcaRow *rows = (DcaRow *)(ws + c.take(sizeof(DcaRow) * (size_t)N * K));
  uint8_t *flags = (uint8_t *)(ws + c.take((size_t)N * K * kRecMaxTopk));
  launch_row_stats("dca_row_stats", head_logits, V, N * K, V, 1.0f, stats, s);
  {
    TraceScope ts("dca_cycle", s);
    hipLaunchKernelGGL(dca_cycle_kernel, dim3(N), dim3(64 * K), 0, s, K, V, topk, vgm, head_logits, stats,
                       stat_chunks(V), rec_logp, rec_ids, n_accept, loss, alpha, rows, flags);
  }
  if (grad) {
    TraceScope ts("dca_grad", s);
    const int nch = (V + kDcaIds - 1) / kDcaIds;
    const size_t bytes = (size_t)N * K * V * sizeof(float);
    const bool small = bytes <= kDcaSmallBytes || (!vgm && (long)N * K % 8 == 0 && bytes <= kDcaRowBytes);
    const int mode = small ? DCA_SMALL : bytes < kDcaStreamBytes ? DCA_MEDIUM : DCA_STREAM;
    const bool vec = (V & 3) == 0 && (((uintptr_t)head_logits | (uintptr_t)grad) & 15) == 0;
    // (a grid's dimension holds less than 2^32 threads)
    const bool flat = nch == 1 || (mode != DCA_SMALL && (size_t)N * K * nch < (size_t(1) << 24));
    const dim3 grid = flat ? dim3((unsigned)N * K * nch) : dim3(N * K, nch);
    auto launch = [&](auto kernel) {
      hipLaunchKernelGGL(kernel, grid, dim3(256), 0, s, V, topk, nch, head_logits, rows, rec_ids, flags, grad);
    };
    if (mode == DCA_SMALL) launch(vec ? dca_grad_kernel<true, DCA_SMALL> : dca_grad_kernel<false, DCA_SMALL>);
    else if (mode == DCA_MEDIUM) launch(vec ? dca_grad_kernel<true, DCA_MEDIUM> : dca_grad_kernel<false, DCA_MEDIUM>);
    else launch(vec ? dca_grad_kernel<true, DCA_STREAM> : dca_grad_kernel<false, DCA_STREAM>);
  }
}

}  // namespace gm
