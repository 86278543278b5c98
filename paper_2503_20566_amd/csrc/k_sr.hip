// Stochastic-reconfiguration build over a batch (SM S-1 eq. gradient, read as the covariance
// <O E> - <O><E>; SM S-3 S_mn = <O_m O_n> - <O_m><O_n>; plain means over the valid samples).
//
// O arrives block-sparse: per sample and site only the selected block is nonzero, stored in the
// projected layout with its block index.  Every kernel here reduces over samples in a fixed
// order (no atomics; k_sr_blocks by lane groups, the dense forms in index order), so results are bitwise
// reproducible.
//   k_sr_blocks : per site and block: <O> and F, or S v = <O (O v)> - <O> (<O> . v), or the vjp
//   k_sr_ov     : (O v)_b per sample (gathers v through the block index)
//   k_cg_*      : the vector steps of the conjugate gradients, their dot products in block partials
//   k_sr_dense  : dense S for small parameter counts
//   k_sr_rows   : rows of the dense S for any parameter count (block-sparse scatter per sample)
#include <algorithm>

#include "dev_common.h"
#include "internal.h"

namespace gipeps {

namespace {

struct SiteShape {
  int nb, bs;  // blocks and block size of the site
};

__device__ SiteShape site_shape(const Dims& d, int s) {
  const int x = s % d.L, y = s / d.L;
  const int np = (x > 0) + (x < d.L - 1) + (y > 0) + (y < d.L - 1);
  SiteShape r{1, 1};
  for (int i = 0; i < np; ++i) r.bs *= d.Dk;
  for (int i = 0; i < np - 1; ++i) r.nb *= d.N;
  return r;
}

// Number of valid samples and the mean local energy over them (every thread gets both).
__device__ void valid_stats(const uint8_t* valid, const double* e, int B, double* red, double* nv,
                            double* emean) {
  double c = 0.0, s = 0.0;
  for (int b = threadIdx.x; b < B; b += blockDim.x)
    if (valid[b]) {
      c += 1.0;
      s += e ? e[b] : 0.0;
    }
  *nv = block_sum(c, red);
  const double tot = block_sum(s, red);
  *emean = (*nv > 0.0) ? tot / *nv : 0.0;
}

}  // namespace

// Sums over the samples that select each block of a site.  One workgroup per (site, 16 blocks), one
// wave per block (several when the site has few): the site's block ids of a chunk of samples are
// staged in LDS, each wave lists its block's samples in order (a ballot per 64 samples), and the
// list is split over the wave's lane groups (one lane per entry of the block, so a sample's entries
// are one coalesced read), whose partial sums are added in lane-group order: no atomics, the
// same bits on every run.  Each O entry is read by one lane exactly once per pass, so what bounds it
// is the read of O (67 MB at Z3 16 x 16, B = 2048).  One workgroup per site whose threads, one per
// parameter, each scanned every sample's block id took 1471 us per pass there; this takes 24 us (2.8 TB/s).
//   kSums: om = <O>, F = <O E> - <O><E>;  kMatvec: S v = <O (O v)> - <O> (<O> . v), with <O> given;
//   kVjp: sum_b w_b O_b (w null: all ones; valid samples)
namespace {
constexpr int kBlkThreads = 1024, kBlkWaves = kBlkThreads / 64;  // blocks of one workgroup: kBlkWaves
constexpr int kChunk = 1024;                                     // samples staged at a time
enum { kSums = 0, kMatvec = 1, kVjp = 2 };
}  // namespace

template <int MODE>
__global__ void __launch_bounds__(kBlkThreads)
k_sr_blocks(Dims d, const int64_t* __restrict__ site_offset, const int32_t* __restrict__ block_id,
            const uint8_t* __restrict__ valid, const double* __restrict__ O, const double* __restrict__ e_loc,
            const double* __restrict__ x, int B, const double* __restrict__ omean_in, double* __restrict__ out,
            double* __restrict__ omean_out) {
  __shared__ int32_t ids[kChunk];
  __shared__ uint16_t list[kBlkWaves][kChunk];
  __shared__ double part[2][kBlkThreads];
  __shared__ double red[kBlkWaves];
  const int s = blockIdx.x, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int bs = site_shape(d, s).bs;
  const int nb = (int)((site_offset[s + 1] - site_offset[s]) / bs);  // both occupations' blocks with matter
  const int j0 = (int)blockIdx.y * kBlkWaves;
  if (j0 >= nb) return;
  // the samples' count and the means that the sums are centred with (every thread)
  double inv = 0.0, mean = 0.0;  // 1 / count; <E> (kSums) or <O v> = <O> . v (kMatvec)
  if (MODE != kVjp) {
    double nv;
    valid_stats(valid, MODE == kSums ? e_loc : x, B, red, &nv, &mean);
    inv = nv > 0.0 ? 1.0 / nv : 0.0;
  }
  const int nj = nb - j0 < kBlkWaves ? nb - j0 : kBlkWaves;
  const int parts = kBlkWaves / nj;                 // waves per block
  const int j = j0 + wave % nj, pt = wave / nj;     // waves with pt >= parts idle
  const int nsub = 64 / bs, e = lane % bs, sub = lane / bs;
  double a0 = 0.0, a1 = 0.0;
  for (int c0 = 0; c0 < B; c0 += kChunk) {
    const int nc = B - c0 < kChunk ? B - c0 : kChunk;
    __syncthreads();  // the previous chunk's ids are no longer read
    for (int i = threadIdx.x; i < nc; i += kBlkThreads)
      ids[i] = valid[c0 + i] ? block_id[(size_t)(c0 + i) * d.n_sites + s] : -1;
    __syncthreads();
    if (pt >= parts) continue;
    int n = 0;  // samples of block j in the chunk, in order
    for (int i0 = 0; i0 < nc; i0 += 64) {
      const bool mine = i0 + lane < nc && ids[i0 + lane] == j;
      const unsigned long long m = __ballot(mine);
      if (mine) list[wave][n + __popcll(m & ((1ull << lane) - 1))] = (uint16_t)(i0 + lane);
      n += __popcll(m);
    }
    __builtin_amdgcn_wave_barrier();  // the list is read by the wave that wrote it
    const double* Oc = O + ((size_t)c0 * d.n_sites + s) * d.P4 + e;
    const size_t row = (size_t)d.n_sites * d.P4;
    const int first = pt * nsub + sub, step = parts * nsub;
    constexpr int U = 4;  // samples in flight per lane
    for (int q = first; q < n; q += U * step) {
      double o[U], w[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const bool in = q + u * step < n;
        const int b = list[wave][in ? q + u * step : q];
        o[u] = in ? Oc[(size_t)b * row] : 0.0;
        w[u] = MODE == kSums ? e_loc[c0 + b] : (MODE == kMatvec || x) ? x[c0 + b] : 1.0;
        w[u] = in ? w[u] : 0.0;
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        a0 = fma(o[u], w[u], a0);
        if (MODE == kSums) a1 += o[u];
      }
    }
  }
  part[0][threadIdx.x] = a0;
  if (MODE == kSums) part[1][threadIdx.x] = a1;
  __syncthreads();
  for (int i = threadIdx.x; i < nj * bs; i += kBlkThreads) {
    const int jj = i / bs, ee = i % bs;
    double t0 = 0.0, t1 = 0.0;
    for (int p = 0; p < parts; ++p)
      for (int u = 0; u < nsub; ++u) {
        const int at = (p * nj + jj) * 64 + u * bs + ee;
        t0 += part[0][at];
        if (MODE == kSums) t1 += part[1][at];
      }
    const int64_t m = site_offset[s] + (int64_t)(j0 + jj) * bs + ee;
    if (MODE == kSums) {
      const double om = t1 * inv;
      omean_out[m] = om;
      out[m] = t0 * inv - om * mean;
    } else if (MODE == kMatvec) {
      out[m] = t0 * inv - omean_in[m] * mean;
    } else {
      out[m] = t0;
    }
  }
}

__global__ void k_sr_ov(Dims d, const int64_t* __restrict__ site_offset,
                        const int32_t* __restrict__ block_id, const uint8_t* __restrict__ valid,
                        const double* __restrict__ O, const double* __restrict__ v,
                        double* __restrict__ ov) {
  __shared__ double red[16];
  const int b = blockIdx.x;
  double acc = 0.0;
  if (valid[b]) {
    for (int idx = threadIdx.x; idx < d.n_sites * d.P4; idx += blockDim.x) {
      const int s = idx / d.P4, e = idx % d.P4;
      const SiteShape sh = site_shape(d, s);
      if (e >= sh.bs) continue;
      const int blk = block_id[(size_t)b * d.n_sites + s];
      acc += O[(size_t)b * d.n_sites * d.P4 + idx] * v[site_offset[s] + (int64_t)blk * sh.bs + e];
    }
  }
  acc = block_sum(acc, red);
  if (threadIdx.x == 0) ov[b] = acc;
}

// Dense S (row m per workgroup): S_mn = <O_m O_n> - <O_m><O_n>.
__global__ void k_sr_dense(Dims d, const int64_t* __restrict__ site_offset,
                           const int32_t* __restrict__ block_id, const uint8_t* __restrict__ valid,
                           const double* __restrict__ O, const double* __restrict__ omean, int B,
                           int64_t n_params, double* __restrict__ S) {
  __shared__ double red[16];
  __shared__ int sm_site, sm_blk, sm_e;
  const int64_t m = blockIdx.x;
  if (threadIdx.x == 0) {
    int s = 0;
    while (site_offset[s + 1] <= m) ++s;
    const SiteShape sh = site_shape(d, s);
    const int64_t r = m - site_offset[s];
    sm_site = s;
    sm_blk = (int)(r / sh.bs);
    sm_e = (int)(r % sh.bs);
  }
  double nv, em;
  valid_stats(valid, nullptr, B, red, &nv, &em);
  const double inv = nv > 0.0 ? 1.0 / nv : 0.0;
  const int s1 = sm_site, b1 = sm_blk, e1 = sm_e;
  for (int64_t n = threadIdx.x; n < n_params; n += blockDim.x) {
    int s2 = 0;
    while (site_offset[s2 + 1] <= n) ++s2;
    const SiteShape sh = site_shape(d, s2);
    const int64_t r = n - site_offset[s2];
    const int b2 = (int)(r / sh.bs), e2 = (int)(r % sh.bs);
    double acc = 0.0;
    for (int b = 0; b < B; ++b) {
      if (!valid[b]) continue;
      if (block_id[(size_t)b * d.n_sites + s1] != b1 || block_id[(size_t)b * d.n_sites + s2] != b2) continue;
      acc += O[((size_t)b * d.n_sites + s1) * d.P4 + e1] * O[((size_t)b * d.n_sites + s2) * d.P4 + e2];
    }
    S[m * n_params + n] = acc * inv - omean[m] * omean[n];
  }
}

// Rows row0 .. row0 + gridDim.x - 1 of S (one workgroup per row m): the row is cleared, then every
// valid sample whose selected block holds m adds O_bm times its own nonzeros (one block per site);
// an entry n is always updated by the thread that owns its (site, entry) pair, so the samples are
// added in index order without atomics, as k_sr_dense adds them.
__global__ void k_sr_rows(Dims d, const int64_t* __restrict__ site_offset,
                          const int32_t* __restrict__ block_id, const uint8_t* __restrict__ valid,
                          const double* __restrict__ O, const double* __restrict__ omean, int B,
                          int64_t n_params, int64_t row0, double* __restrict__ S) {
  __shared__ double red[16];
  __shared__ int sm_site, sm_blk, sm_e;
  const int64_t m = row0 + blockIdx.x;
  double* row = S + (size_t)blockIdx.x * (size_t)n_params;
  if (threadIdx.x == 0) {
    int s = 0;
    while (site_offset[s + 1] <= m) ++s;
    const SiteShape sh = site_shape(d, s);
    const int64_t r = m - site_offset[s];
    sm_site = s;
    sm_blk = (int)(r / sh.bs);
    sm_e = (int)(r % sh.bs);
  }
  double nv, em;
  valid_stats(valid, nullptr, B, red, &nv, &em);  // its barriers also publish sm_*
  const double inv = nv > 0.0 ? 1.0 / nv : 0.0;
  const int s1 = sm_site, b1 = sm_blk, e1 = sm_e;
  for (int64_t n = threadIdx.x; n < n_params; n += blockDim.x) row[n] = 0.0;
  __syncthreads();
  const int nse = d.n_sites * d.P4;
  for (int b = 0; b < B; ++b) {
    if (!valid[b] || block_id[(size_t)b * d.n_sites + s1] != b1) continue;  // same in every thread
    const double w = O[((size_t)b * d.n_sites + s1) * d.P4 + e1];
    for (int idx = threadIdx.x; idx < nse; idx += blockDim.x) {
      const int s = idx / d.P4, e = idx % d.P4;
      const SiteShape sh = site_shape(d, s);
      if (e >= sh.bs) continue;
      const int64_t n = site_offset[s] + (int64_t)block_id[(size_t)b * d.n_sites + s] * sh.bs + e;
      row[n] += w * O[((size_t)b * d.n_sites + s) * d.P4 + e];
    }
  }
  __syncthreads();
  for (int64_t n = threadIdx.x; n < n_params; n += blockDim.x) row[n] = row[n] * inv - omean[m] * omean[n];
}

// Conjugate-gradient vector steps of sr_solve ((S + shift I) x = F).  A dot product is left as one
// partial sum per block (at most kCgBlocks, each over a fixed set of entries) and added up, in the same
// order by every block, in the kernel that needs it: five launches per iteration and no kernel of a
// single workgroup (the dot products of 88,752 entries took 28 us each in one).
// sc: [k & 1] r.r before iteration k, [2] its p.q, then two arrays of kCgBlocks partials: r.r and p.q.
namespace {
constexpr int kCgBlocks = 1024;
__device__ __forceinline__ double* rr_part(double* sc) { return sc + 8; }
__device__ __forceinline__ double* pq_part(double* sc) { return sc + 8 + kCgBlocks; }
__device__ double add_parts(const double* part, int n, double* red) {
  double v = 0.0;
  for (int i = threadIdx.x; i < n; i += blockDim.x) v += part[i];
  return block_sum(v, red);
}
}  // namespace

__global__ void k_cg_init(const double* __restrict__ F, double* __restrict__ x, double* __restrict__ r,
                          double* __restrict__ p, double* __restrict__ sc, int64_t n) {
  __shared__ double red[4];
  double acc = 0.0;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
    x[i] = 0.0;
    r[i] = F[i];
    p[i] = F[i];
    acc = fma(F[i], F[i], acc);
  }
  acc = block_sum(acc, red);
  if (threadIdx.x == 0) rr_part(sc)[blockIdx.x] = acc;
}

// r.r of the start (one workgroup)
__global__ void k_cg_first(double* __restrict__ sc, int nblk) {
  __shared__ double red[4];
  const double rr = add_parts(rr_part(sc), nblk, red);
  if (threadIdx.x == 0) sc[0] = rr;
}

// q = S p + shift p, p.q
__global__ void k_cg_shift(double* __restrict__ q, const double* __restrict__ p, double shift,
                           double* __restrict__ sc, int64_t n) {
  __shared__ double red[4];
  double acc = 0.0;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
    const double v = q[i] + shift * p[i];
    q[i] = v;
    acc = fma(p[i], v, acc);
  }
  acc = block_sum(acc, red);
  if (threadIdx.x == 0) pq_part(sc)[blockIdx.x] = acc;
}

// x += alpha p, r -= alpha q with alpha = r.r / p.q, and the new r.r; x and r keep their values when
// p.q <= 0 (breakdown)
__global__ void k_cg_step(double* __restrict__ x, double* __restrict__ r, const double* __restrict__ p,
                          const double* __restrict__ q, double* __restrict__ sc, int nblk, int k, int64_t n) {
  __shared__ double red[4];
  const double pq = add_parts(pq_part(sc), nblk, red);
  if (blockIdx.x == 0 && threadIdx.x == 0) sc[2] = pq;
  if (!(pq > 0.0)) return;  // the same in every thread
  const double alpha = sc[k & 1] / pq;
  double acc = 0.0;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
    x[i] += alpha * p[i];
    const double v = r[i] - alpha * q[i];
    r[i] = v;
    acc = fma(v, v, acc);
  }
  acc = block_sum(acc, red);
  if (threadIdx.x == 0) rr_part(sc)[blockIdx.x] = acc;
}

// the r.r after iteration k, then p = r + beta p with beta = it over the r.r before
__global__ void k_cg_dir(double* __restrict__ p, const double* __restrict__ r, double* __restrict__ sc, int nblk,
                         int k, int64_t n) {
  __shared__ double red[4];
  if (!(sc[2] > 0.0)) return;
  const double rr = add_parts(rr_part(sc), nblk, red);
  if (blockIdx.x == 0 && threadIdx.x == 0) sc[(k + 1) & 1] = rr;
  const double beta = rr / sc[k & 1];
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    p[i] = r[i] + beta * p[i];
}

namespace {
int cg_blocks(int64_t n) { return (int)std::min<int64_t>((n + 255) / 256, kCgBlocks); }

template <int MODE>
hipError_t launch_blocks(const Dims& d, const DeviceTables& t, const int32_t* block_id, const uint8_t* valid,
                         const double* O, const double* e_loc, const double* x, int B, const double* omean_in,
                         double* out, double* omean_out, hipStream_t s) {
  const int nb = d.N * d.N * d.N * (d.matter ? 2 : 1);  // blocks of an inner site
  hipLaunchKernelGGL(k_sr_blocks<MODE>, dim3(d.n_sites, (nb + kBlkWaves - 1) / kBlkWaves), dim3(kBlkThreads), 0, s, d,
                     t.site_offset, block_id, valid, O, e_loc, x, B, omean_in, out, omean_out);
  return hipGetLastError();
}
}  // namespace

hipError_t launch_vjp(const Dims& d, const DeviceTables& t, const int32_t* block_id, const uint8_t* valid,
                      const double* w, const double* O, int B, double* vjp, hipStream_t s) {
  return launch_blocks<kVjp>(d, t, block_id, valid, O, nullptr, w, B, nullptr, vjp, nullptr, s);
}

hipError_t launch_sr_sums(const Dims& d, const DeviceTables& t, const int32_t* block_id, const uint8_t* valid,
                          const double* O, const double* e_loc, int B, double* F, double* omean, hipStream_t s) {
  return launch_blocks<kSums>(d, t, block_id, valid, O, e_loc, nullptr, B, nullptr, F, omean, s);
}

hipError_t launch_sr_matvec(const Dims& d, const DeviceTables& t, const int32_t* block_id, const uint8_t* valid,
                            const double* O, int B, const double* omean, const double* v, double* ov, double* out,
                            hipStream_t s) {
  hipLaunchKernelGGL(k_sr_ov, dim3(B), dim3(256), 0, s, d, t.site_offset, block_id, valid, O, v, ov);
  if (hipError_t e = hipGetLastError()) return e;
  return launch_blocks<kMatvec>(d, t, block_id, valid, O, nullptr, ov, B, omean, out, nullptr, s);
}

hipError_t launch_sr_dense(const Dims& d, const DeviceTables& t, int64_t n_params, const int32_t* block_id,
                           const uint8_t* valid, const double* O, int B, const double* omean, double* S,
                           hipStream_t s) {
  hipLaunchKernelGGL(k_sr_dense, dim3((unsigned)n_params), dim3(256), 0, s, d, t.site_offset, block_id, valid, O,
                     omean, B, n_params, S);
  return hipGetLastError();
}

hipError_t launch_cg_start(int64_t n, double* x, double* r, double* p, const double* F, double* sc, hipStream_t s) {
  const int g = cg_blocks(n);
  hipLaunchKernelGGL(k_cg_init, dim3(g), dim3(256), 0, s, F, x, r, p, sc, n);
  if (hipError_t e = hipGetLastError()) return e;
  hipLaunchKernelGGL(k_cg_first, dim3(1), dim3(256), 0, s, sc, g);
  return hipGetLastError();
}

hipError_t launch_cg_iteration(int64_t n, double* x, double* r, double* p, double* q, double* sc, int k, double shift,
                               hipStream_t s) {
  const int g = cg_blocks(n);
  hipLaunchKernelGGL(k_cg_shift, dim3(g), dim3(256), 0, s, q, p, shift, sc, n);
  if (hipError_t e = hipGetLastError()) return e;
  hipLaunchKernelGGL(k_cg_step, dim3(g), dim3(256), 0, s, x, r, p, q, sc, g, k, n);
  if (hipError_t e = hipGetLastError()) return e;
  hipLaunchKernelGGL(k_cg_dir, dim3(g), dim3(256), 0, s, p, r, sc, g, k, n);
  return hipGetLastError();
}

hipError_t launch_sr_rows(const Dims& d, const DeviceTables& t, int64_t n_params, const int32_t* block_id,
                          const uint8_t* valid, const double* O, const double* omean, int B, int64_t row0,
                          int64_t nrows, double* S, hipStream_t s) {
  if (nrows == 0 || B == 0) return hipSuccess;
  hipLaunchKernelGGL(k_sr_rows, dim3((unsigned)nrows), dim3(256), 0, s, d, t.site_offset, block_id, valid,
                     O, omean, B, n_params, row0, S);
  return hipGetLastError();
}

}  // namespace gipeps
