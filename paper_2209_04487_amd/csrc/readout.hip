// Readouts beside the molecular step.
//  - Dipole, norm and yield of every wavepacket (m = 0 and (j, m) bases).
//  - Excited-state radial moments of every wavepacket (Eq. (8)): per molecule
//    <chi_e|R|chi_e> = sum_{J,k} r_k |psi_e,J(r_k)|^2 dr and <chi_e|chi_e>,
//    accumulated in FP64, plus the ensemble sums over molecules and their
//    ratio in a fixed order.
//  - Ensemble sums of per-molecule FP64 values (dipole, norm, yield) in a
//    fixed two-stage order.
//  - Transmission, reflection and absorption spectra from monitor fluxes.
//
// The per-molecule readouts read each wavepacket once and are bound by HBM.  One
// wavefront per molecule: a lane owns 16 bytes of every line (two complex64 or
// one complex128 radial point), so the lines of a molecule, which lie n_r
// elements apart, are read whole and in order, the sum over J stays in the lane,
// and the sums over r are shuffles.  Nothing goes through LDS and no barrier
// stands between a molecule's loads and the next molecule's.
#include <hip/hip_runtime.h>

#include "mol.h"
#include "mol_jmg.h"
#include "readout.h"

namespace msqd {

constexpr int kRdThreads = 256;
constexpr int kRdWaves = kRdThreads / 64;
constexpr int kRdMaxNr = 512;

namespace {

// 16 bytes of a line: V radial points
template <typename T>
struct RdVec {
  static constexpr int V = 16 / static_cast<int>(sizeof(cx<T>));
  cx<T> p[V];
};
// (one load of 16 bytes on the elements' own alignment: excited_r_readout takes any)
typedef unsigned RdRaw __attribute__((ext_vector_type(4), aligned(4)));
template <typename T>
__device__ __forceinline__ RdVec<T> rd_load(const cx<T>* p) {
  RdVec<T> v;
  *reinterpret_cast<RdRaw*>(&v) = *reinterpret_cast<const RdRaw*>(p);
  return v;
}

__device__ __forceinline__ double rd_wave_sum(double v) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}

}  // namespace

// d = 2 dr sum_r mu(r) sum_J c_J Re[conj(g_J) e_{J+1} + conj(g_{J+1}) e_J], the J
// sum in the working precision and the r sum in FP64 as in the step's own
// dipole; the norm also when no dipole is asked for, as the finiteness check.
// 100,000 molecules of n_r = 256, J <= 10 in complex64 (4.5 GB): 1221 us when the
// step's kernel did this (lines through LDS, barriers), 734 us here (6.1 TB/s).
// SPLIT: the four wavefronts of a workgroup take a molecule's points in turn and the
// first one adds their terms up from LDS, where lines hold a load for each of them
// (n_r = 256 in complex128, 512 in complex64): a wavefront alone goes through four or
// eight loads of every line one after another, which is what a small batch waits for,
// and streams less well in a large one.  us, one wavefront / four: complex128, n_r = 256,
// J <= 15: 8 molecules 9.1 / 5.2 (6.1 in the step's kernel), 333 17.7 / 10.1 (13.6),
// 30,000 644 / 636; J <= 10, 50,000: 825 / 745; complex64, n_r = 512, J <= 8: 8 6.5 /
// 4.2, 60,000 771 / 704.  Shorter lines lose by it in large batches (complex64, n_r =
// 256, J <= 10, 100,000: 737 / 746; complex128, n_r = 128, J = 0, 200,000: 156 / 165).
template <typename T, bool SPLIT>
__global__ __launch_bounds__(kRdThreads) void mol_readout_kernel(MolArgs a, int n_r) {
  constexpr int V = RdVec<T>::V, kUnroll = SPLIT ? 8 : 4;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int mol = SPLIT ? static_cast<int>(blockIdx.x) : static_cast<int>(blockIdx.x) * kRdWaves + wave;
  if (mol >= a.n_mol) return;
  const int nj = a.nj;
  const double* mu = reinterpret_cast<const double*>(a.ws + a.lay.mu_d);
  const double* cj = reinterpret_cast<const double*>(a.ws + a.lay.cj_d);
  const cx<T>* g = static_cast<const cx<T>*>(a.psi) + static_cast<size_t>(mol) * 2 * nj * n_r;
  const cx<T>* e = g + static_cast<size_t>(nj) * n_r;
  __shared__ double terms[2][SPLIT ? kRdMaxNr : 1];
  double nrm = 0.0, yld = 0.0, dd = 0.0;
  auto add = [&](int r, double acc, double n2) {
    dd += mu[r] * acc;
    nrm += n2;
    if (r >= a.kdiss) yld += n2;
  };
  for (int r = (SPLIT ? static_cast<int>(threadIdx.x) : lane) * V; r < n_r; r += (SPLIT ? kRdThreads : 64) * V) {
    RdVec<T> g0 = rd_load(g + r), e0 = rd_load(e + r);
    T acc[V];
    double n2[V];
#pragma unroll
    for (int i = 0; i < V; ++i) {
      acc[i] = T(0);
      n2[i] = static_cast<double>(norm2(g0.p[i])) + static_cast<double>(norm2(e0.p[i]));
    }
#pragma unroll kUnroll
    for (int J = 0; J + 1 < nj; ++J) {
      const RdVec<T> g1 = rd_load(g + (J + 1) * n_r + r), e1 = rd_load(e + (J + 1) * n_r + r);
      const T c = static_cast<T>(cj[J]);
#pragma unroll
      for (int i = 0; i < V; ++i) {
        const T t = g0.p[i].x * e1.p[i].x + g0.p[i].y * e1.p[i].y + g1.p[i].x * e0.p[i].x + g1.p[i].y * e0.p[i].y;
        acc[i] += c * t;
        n2[i] += static_cast<double>(norm2(g1.p[i])) + static_cast<double>(norm2(e1.p[i]));
      }
      g0 = g1;
      e0 = e1;
    }
#pragma unroll
    for (int i = 0; i < V; ++i) {
      if constexpr (SPLIT) {
        terms[0][r + i] = static_cast<double>(acc[i]);
        terms[1][r + i] = n2[i];
      } else {
        add(r + i, static_cast<double>(acc[i]), n2[i]);
      }
    }
  }
  if constexpr (SPLIT) {
    __syncthreads();
    if (wave > 0) return;
    for (int r = lane * V; r < n_r; r += 64 * V) {
#pragma unroll
      for (int i = 0; i < V; ++i) add(r + i, terms[0][r + i], terms[1][r + i]);
    }
  }
  nrm = rd_wave_sum(nrm);
  yld = rd_wave_sum(yld);
  dd = rd_wave_sum(dd);
  if (lane == 0) {
    const double absorbed = a.absorbed[mol];
    const double d = a.want_d ? 2.0 * a.dr * dd : 0.0;
    if (a.want_d) a.d_mol[mol] = d;
    if (a.want_norm) a.norm_mol[mol] = nrm * a.dr;
    if (a.want_yield) a.yield_mol[mol] = yld * a.dr + absorbed;
    const bool check_n = a.want_norm || !a.want_d || a.want_yield;
    if (!isfinite(d) || (check_n && !isfinite(nrm)) || !isfinite(absorbed)) atomicOr(a.status, 1);
  }
}

// The same in the (j, m) basis, three dipole components: a lane owns one radial
// point, holds the states of one j of both electronic states (converted once) and
// reads those of j + 1.  With the terms Re<g|D_z|e>, P = <g|D_+|e> and P' =
// <e|D_+|g>, D_+ = D_x + i D_y, d_x and d_y are Re (P + P') / 2 and Im (P + P') / 2.
// dip: per state <j+1,m|cos|j,m>, <j+1,m+1|sin e^{i ph}|j,m>, <j-1,m+1|sin e^{i ph}|j,m>.
// When the steps' kernels did this (lines through LDS, one workgroup per molecule)
// -> here, us: 389 -> 265 (100,000 molecules, n_r = 256, j_max = 1, complex64), 1009 ->
// 354 (60,000, j_max = 2), 1072 -> 415 (40,000, j_max = 3), 1644 -> 676 (20,000, j_max
// = 5), 1041 -> 489 (8,000, n_r = 512, j_max = 4); complex128 662 -> 336 (15,000, n_r =
// 256, j_max = 3), 1197 -> 537 (20,000, n_r = 128, j_max = 5).
// SPLIT: the wavefronts of a workgroup share a molecule's radial points, for launches
// that leave the card idle otherwise; the first one adds their terms up from LDS in the
// order in which a single wavefront meets them.  The products are stated as fused, so
// that both forms round alike and a molecule's readouts do not depend on the batch.
template <typename T, int JM, bool SPLIT>
__global__ __launch_bounds__(kRdThreads) void jm_readout_kernel(MolArgs a, int n_r) {
  constexpr int NB = (JM + 1) * (JM + 1), NM = 2 * JM + 1;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int mol = SPLIT ? static_cast<int>(blockIdx.x) : static_cast<int>(blockIdx.x) * kRdWaves + wave;
  if (mol >= a.n_mol) return;
  const double* mu = reinterpret_cast<const double*>(a.ws + a.lay.mu_d);
  // j_max = 1 has no tables in the workspace
  const double one[12] = {0.57735026918962576451, -0.81649658092772603273, 0.0, 0.0, 0.0, 0.81649658092772603273};
  const double* __restrict__ dip =
      JM == 1 ? one : reinterpret_cast<const double*>(a.ws + a.lay.total) + jmg_tab(JM).dip;
  const cx<T>* g = static_cast<const cx<T>*>(a.psi) + static_cast<size_t>(mol) * 2 * NB * n_r;
  const cx<T>* e = g + static_cast<size_t>(NB) * n_r;
  __shared__ double terms[4][SPLIT ? kRdMaxNr : 1];
  double nrm = 0.0, yld = 0.0, dx = 0.0, dy = 0.0, dz = 0.0;
  auto add = [&](int r, double n2, double pr, double pi, double z) {
    const double m = mu[r];
    dx = fma(m, 0.5 * pr, dx);
    dy = fma(m, 0.5 * pi, dy);
    dz = fma(m, z, dz);
    nrm += n2;
    if (r >= a.kdiss) yld += n2;
  };
#pragma unroll 1
  for (int r = SPLIT ? static_cast<int>(threadIdx.x) : lane; r < n_r; r += SPLIT ? kRdThreads : 64) {
    double n2 = 0.0, z = 0.0, pr = 0.0, pi = 0.0;
    cx<double> g0[NM], e0[NM], g1[NM], e1[NM];
#pragma unroll
    for (int j = 0; j <= JM; ++j) {
#pragma unroll
      for (int i = 0; i < 2 * j + 1; ++i) {
        const cx<T> u = g[(j * j + i) * n_r + r], w = e[(j * j + i) * n_r + r];
        n2 += static_cast<double>(fma(u.x, u.x, u.y * u.y)) + static_cast<double>(fma(w.x, w.x, w.y * w.y));
        g1[i] = {static_cast<double>(u.x), static_cast<double>(u.y)};
        e1[i] = {static_cast<double>(w.x), static_cast<double>(w.y)};
      }
      // c (conj(p_g) b_e + conj(p_e) b_g)
      auto link = [&](double c, const cx<double>& pg, const cx<double>& pe, const cx<double>& bg, const cx<double>& be) {
        pr = fma(c, fma(pg.x, be.x, fma(pg.y, be.y, fma(pe.x, bg.x, pe.y * bg.y))), pr);
        pi = fma(c, fma(pg.x, be.y, fma(-pg.y, be.x, fma(pe.x, bg.y, -pe.y * bg.x))), pi);
      };
      if (j > 0) {
        // state (j - 1, m) = [i] with (j, m) = [i + 1] and (j, m + 1) = [i + 2]
#pragma unroll
        for (int i = 0; i < 2 * j - 1; ++i) {
          const double* c = dip + 3 * ((j - 1) * (j - 1) + i);
          z = fma(c[0], fma(g1[i + 1].x, e0[i].x, fma(g1[i + 1].y, e0[i].y,
                                                      fma(g0[i].x, e1[i + 1].x, g0[i].y * e1[i + 1].y))), z);
          link(c[1], g1[i + 2], e1[i + 2], g0[i], e0[i]);
        }
        // state (j, m) = [i] with (j - 1, m + 1) = [i]
#pragma unroll
        for (int i = 0; i < 2 * j - 1; ++i) link(dip[3 * (j * j + i) + 2], g0[i], e0[i], g1[i], e1[i]);
      }
#pragma unroll
      for (int i = 0; i < 2 * j + 1; ++i) {
        g0[i] = g1[i];
        e0[i] = e1[i];
      }
    }
    if constexpr (SPLIT) {
      terms[0][r] = n2;
      terms[1][r] = pr;
      terms[2][r] = pi;
      terms[3][r] = z;
    } else {
      add(r, n2, pr, pi, z);
    }
  }
  if constexpr (SPLIT) {
    __syncthreads();
    if (wave > 0) return;
    for (int r = lane; r < n_r; r += 64) add(r, terms[0][r], terms[1][r], terms[2][r], terms[3][r]);
  }
  const double sum[5] = {rd_wave_sum(nrm), rd_wave_sum(yld), rd_wave_sum(dx), rd_wave_sum(dy), rd_wave_sum(dz)};
  if (lane == 0) {
    const double* d = sum + 2;
    nrm = sum[0];
    yld = sum[1];
    const double absorbed = a.absorbed[mol];
    bool ok = isfinite(nrm) && isfinite(absorbed);
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      if (!a.want_d) continue;
      a.d_mol[3 * mol + k] = 2.0 * a.dr * d[k];
      ok = ok && isfinite(d[k]);
    }
    if (a.want_norm) a.norm_mol[mol] = nrm * a.dr;
    if (a.want_yield) a.yield_mol[mol] = yld * a.dr + absorbed;
    if (!ok) atomicOr(a.status, 1);
  }
}

// The moments of Eq. (8), with the wavefronts of a workgroup sharing long lines as in
// mol_readout_kernel (us with the ensemble sums, one wavefront / four, and one pass of a
// workgroup over all lines before: complex128, n_r = 256, J <= 15, 10,000 molecules 156 /
// 120, 131; J <= 10, 64 molecules 7.6 / 6.1, 6.9; complex64, n_r = 512, J <= 8, 30,000
// 224 / 196, 268).
template <typename T, bool SPLIT>
__global__ __launch_bounds__(kRdThreads) void excited_r_kernel(RdArgs a) {
  constexpr int V = RdVec<T>::V;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int mol = SPLIT ? static_cast<int>(blockIdx.x) : static_cast<int>(blockIdx.x) * kRdWaves + wave;
  if (mol >= a.n_mol) return;
  const cx<T>* e = static_cast<const cx<T>*>(a.psi) + (static_cast<size_t>(mol) * 2 + 1) * a.nj * a.n_r;
  __shared__ double terms[SPLIT ? kRdMaxNr : 1];
  double num = 0.0, pop = 0.0;
  auto add = [&](int r, double p2) {
    pop += p2;
    num += (a.r_min + r * a.dr) * p2;
  };
  for (int r = (SPLIT ? static_cast<int>(threadIdx.x) : lane) * V; r < a.n_r; r += (SPLIT ? kRdThreads : 64) * V) {
    double p2[V];
#pragma unroll
    for (int i = 0; i < V; ++i) p2[i] = 0.0;
#pragma unroll 4
    for (int J = 0; J < a.nj; ++J) {
      const RdVec<T> v = rd_load(e + static_cast<size_t>(J) * a.n_r + r);
#pragma unroll
      for (int i = 0; i < V; ++i) {
        const double re = static_cast<double>(v.p[i].x), im = static_cast<double>(v.p[i].y);
        p2[i] += re * re + im * im;
      }
    }
#pragma unroll
    for (int i = 0; i < V; ++i) {
      if constexpr (SPLIT)
        terms[r + i] = p2[i];
      else
        add(r + i, p2[i]);
    }
  }
  if constexpr (SPLIT) {
    __syncthreads();
    if (wave > 0) return;
    for (int r = lane * V; r < a.n_r; r += 64 * V) {
#pragma unroll
      for (int i = 0; i < V; ++i) add(r + i, terms[r + i]);
    }
  }
  num = rd_wave_sum(num);
  pop = rd_wave_sum(pop);
  if (lane == 0) {
    a.r_num[mol] = num * a.dr;
    a.pop[mol] = pop * a.dr;
  }
}

// ensemble sums over molecules (one workgroup, an order fixed by their number) and
// their ratio: a single CU's read of 16 bytes per molecule, kept busy by 1,024 threads
// with eight independent loads each (100,000 molecules: 164 us with 256 threads and one
// load in flight each), one wavefront where that is one pass (0.5 us less at 64 molecules)
constexpr int kPairThreads = 1024, kPairLoads = 8;
template <int THREADS>
__global__ __launch_bounds__(THREADS) void pair_sum_kernel(const double* x, const double* y, int n, double* out) {
  __shared__ double sx[THREADS / 64], sy[THREADS / 64];
  const int tid = threadIdx.x;
  double ax[kPairLoads] = {}, ay[kPairLoads] = {};
  for (int i0 = tid; i0 < n; i0 += kPairLoads * THREADS) {
#pragma unroll
    for (int u = 0; u < kPairLoads; ++u) {
      const int i = i0 + u * THREADS;
      ax[u] += i < n ? x[i] : 0.0;
      ay[u] += i < n ? y[i] : 0.0;
    }
  }
#pragma unroll
  for (int u = 1; u < kPairLoads; ++u) {
    ax[0] += ax[u];
    ay[0] += ay[u];
  }
  const double vx = rd_wave_sum(ax[0]), vy = rd_wave_sum(ay[0]);
  if ((tid & 63) == 0) {
    sx[tid >> 6] = vx;
    sy[tid >> 6] = vy;
  }
  __syncthreads();
  if (tid == 0) {
    double tx = 0.0, ty = 0.0;
    for (int w = 0; w < THREADS / 64; ++w) {
      tx += sx[w];
      ty += sy[w];
    }
    out[0] = tx;
    out[1] = ty;
    out[2] = tx / ty;   // NaN while the excited population is exactly zero
  }
}

// stage one: block b sums molecules [b kSumBlock, (b+1) kSumBlock), thread t
// taking b kSumBlock + t + kRdThreads q, q = 0..3, then a fixed tree
__global__ __launch_bounds__(kRdThreads) void block_sums_kernel(SumArgs a) {
  __shared__ double sh[kMaxSumVecs][kRdThreads];
  const int tid = threadIdx.x;
  const int base = blockIdx.x * kSumBlock;
  for (int v = 0; v < a.nv; ++v) {
    double acc = 0.0;
    for (int q = 0; q < kSumBlock / kRdThreads; ++q) {
      const int i = base + tid + q * kRdThreads;
      if (i < a.n) acc += a.src[v][static_cast<size_t>(i) * a.stride[v]];
    }
    sh[v][tid] = acc;
  }
  __syncthreads();
  for (int w = kRdThreads / 2; w > 0; w >>= 1) {
    if (tid < w)
      for (int v = 0; v < a.nv; ++v) sh[v][tid] += sh[v][tid + w];
    __syncthreads();
  }
  if (tid < a.nv) a.partial[static_cast<size_t>(blockIdx.x) * a.nv + tid] = sh[tid][0];
}

// stage two: one workgroup over the partials, thread t taking blocks
// t, t + kRdThreads, ..., then the same tree
__global__ __launch_bounds__(kRdThreads) void partial_sums_kernel(SumArgs a, int nblk) {
  __shared__ double sh[kMaxSumVecs][kRdThreads];
  const int tid = threadIdx.x;
  for (int v = 0; v < a.nv; ++v) {
    double acc = 0.0;
    for (int b = tid; b < nblk; b += kRdThreads) acc += a.partial[static_cast<size_t>(b) * a.nv + v];
    sh[v][tid] = acc;
  }
  __syncthreads();
  for (int w = kRdThreads / 2; w > 0; w >>= 1) {
    if (tid < w)
      for (int v = 0; v < a.nv; ++v) sh[v][tid] += sh[v][tid + w];
    __syncthreads();
  }
  if (tid < a.nv) a.out[tid] = sh[tid][0];
}

__global__ void spectra_kernel(const double* st, const double* si, const double* sr, int n, double* tra) {
  const int f = blockIdx.x * blockDim.x + threadIdx.x;
  if (f >= n) return;
  const double ref = sr[f];
  tra[f] = st[f] / ref;
  tra[n + f] = (ref - si[f]) / ref;
  tra[2 * n + f] = (si[f] - st[f]) / ref;
}

// Small batches give each molecule a workgroup (us, a wavefront / a workgroup; j_max =
// 5, n_r = 256, complex64: 1 molecule 20.7 / 8.9, 1,000 44.0 / 32.9, 2,000 71.2 / 80.2;
// j_max = 3: 1,000 17.3 / 15.0, 2,000 23.6 / 23.6, 40,000 415 / 455; j_max = 4, n_r =
// 128, complex128: 1 10.1 / 7.1, 333 20.1 / 13.2, 1,000 22.7 / 25.2; at n_r = 64 a line
// has points for one wavefront).
static bool jm_split(int n_mol, int n_r) { return n_mol <= (n_r >= 256 ? 1024 : 512) && n_r >= 128; }
template <typename T, int JM>
static int launch_jm_readout_j(const MolArgs& a, int n_r, hipStream_t s) {
  if (jm_split(a.n_mol, n_r))
    hipLaunchKernelGGL((jm_readout_kernel<T, JM, true>), dim3(a.n_mol), dim3(kRdThreads), 0, s, a, n_r);
  else
    hipLaunchKernelGGL((jm_readout_kernel<T, JM, false>), dim3((a.n_mol + kRdWaves - 1) / kRdWaves), dim3(kRdThreads), 0, s,
                       a, n_r);
  return static_cast<int>(hipGetLastError());
}

template <typename T>
static int launch_jm_readout_t(const MolArgs& a, int n_r, hipStream_t s) {
  switch (a.nj - 1) {
    case 1: return launch_jm_readout_j<T, 1>(a, n_r, s);
    case 2: return launch_jm_readout_j<T, 2>(a, n_r, s);
    case 3: return launch_jm_readout_j<T, 3>(a, n_r, s);
    case 4: return launch_jm_readout_j<T, 4>(a, n_r, s);
    case 5: return launch_jm_readout_j<T, 5>(a, n_r, s);
    default: return static_cast<int>(hipErrorInvalidValue);
  }
}

int launch_jm_readout(const MolArgs& a, int n_r, bool f32, hipStream_t s) {
  if (a.n_mol <= 0) return 0;
  return f32 ? launch_jm_readout_t<float>(a, n_r, s) : launch_jm_readout_t<double>(a, n_r, s);
}

template <typename T>
static int launch_mol_readout_t(const MolArgs& a, int n_r, hipStream_t s) {
  if (n_r >= kRdThreads * RdVec<T>::V)
    hipLaunchKernelGGL((mol_readout_kernel<T, true>), dim3(a.n_mol), dim3(kRdThreads), 0, s, a, n_r);
  else
    hipLaunchKernelGGL((mol_readout_kernel<T, false>), dim3((a.n_mol + kRdWaves - 1) / kRdWaves), dim3(kRdThreads), 0, s, a,
                       n_r);
  return static_cast<int>(hipGetLastError());
}

int launch_mol_readout(const MolArgs& a, int n_r, bool f32, hipStream_t s) {
  if (a.n_mol <= 0) return 0;
  return f32 ? launch_mol_readout_t<float>(a, n_r, s) : launch_mol_readout_t<double>(a, n_r, s);
}

template <typename T>
static void launch_excited_r_t(const RdArgs& a, hipStream_t s) {
  if (a.n_r >= kRdThreads * RdVec<T>::V)
    hipLaunchKernelGGL((excited_r_kernel<T, true>), dim3(a.n_mol), dim3(kRdThreads), 0, s, a);
  else
    hipLaunchKernelGGL((excited_r_kernel<T, false>), dim3((a.n_mol + kRdWaves - 1) / kRdWaves), dim3(kRdThreads), 0, s, a);
}

int launch_excited_r(const RdArgs& a, bool f32, hipStream_t s) {
  if (a.n_mol <= 0) return 0;
  if (f32)
    launch_excited_r_t<float>(a, s);
  else
    launch_excited_r_t<double>(a, s);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || a.sums == nullptr) return static_cast<int>(e);
  if (a.n_mol <= 64 * kPairLoads)
    hipLaunchKernelGGL(pair_sum_kernel<64>, dim3(1), dim3(64), 0, s, a.r_num, a.pop, a.n_mol, a.sums);
  else
    hipLaunchKernelGGL(pair_sum_kernel<kPairThreads>, dim3(1), dim3(kPairThreads), 0, s, a.r_num, a.pop, a.n_mol, a.sums);
  return static_cast<int>(hipGetLastError());
}

int launch_ensemble_sums(const SumArgs& a, hipStream_t s) {
  const int nblk = sum_blocks(a.n);
  if (nblk > 0) {
    hipLaunchKernelGGL(block_sums_kernel, dim3(nblk), dim3(kRdThreads), 0, s, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return static_cast<int>(e);
  }
  hipLaunchKernelGGL(partial_sums_kernel, dim3(1), dim3(kRdThreads), 0, s, a, nblk);
  return static_cast<int>(hipGetLastError());
}

int launch_spectra(const double* s_trans, const double* s_inc, const double* s_ref, int n_freq, double* tra,
                   hipStream_t s) {
  if (n_freq <= 0) return 0;
  hipLaunchKernelGGL(spectra_kernel, dim3((n_freq + 255) / 256), dim3(256), 0, s, s_trans, s_inc, s_ref, n_freq,
                     tra);
  return static_cast<int>(hipGetLastError());
}

}  // namespace msqd
