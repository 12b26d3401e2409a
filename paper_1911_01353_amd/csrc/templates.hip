// Template bank generation on the GPU, in FP64.
//
// Each tap is the response of a tone with constant fdot and fddot (paper,
// section "Implementation": one filter per (z, w)), evaluated as
//   T(qbar; zbar, w) = R(qbar - zbar/2 + w/12; zbar - w/2, w),
//   R(q; z, w)       = integral_0^1 exp(2 pi i (q u + z u^2/2 + w u^3/6)) du,
// by composite 16-point Gauss-Legendre quadrature. The phase turns at
// |qbar| + |zbar|/2 + |w|/12 cycles per unit u at most (the sweep's end points
// bound it), which is at most K/2 + (K/2 - margin) for the taps inside a
// template's window, K the group's taps; panels of at most two such cycles
// leave a quadrature error of (2 pi)^32 2.7e-45 ~ 1e-19.
//
// All taps of a width group use the same nodes u_k, so the integrand separates:
//   T_t(qbar) = sum_k E_k(qbar) g_t,k,   E_k(qbar) = exp(2 pi i qbar u_k),
//   g_t,k = weight_k exp(2 pi i u_k (-zbar/2 + w/12 + u_k ((zbar - w/2)/2 + u_k w/6))),
// a complex FP64 matrix product over the nodes on the matrix cores
// (v_mfma_f64_16x16x4), with one sincospi per (template, node) instead of one
// per (tap, node).
//
// The FP64 taps are kept in the bank; the path-specific banks are derived
// from them:
//   FFT path  - spectra H[f] = (1/S) sum_j c_j exp(+2 pi i f j / S), f < S,
//               so that IFFT(FFT(segment) * H) is the circular correlation of
//               the segment with the taps (the overlap-save identity).
//   MFMA path - tap fragments (gemm_correlate.hip).
#include <algorithm>
#include <cmath>

#include "jerk_internal.h"

namespace jerk {
namespace {

typedef double d4vec __attribute__((ext_vector_type(4)));

constexpr int kTapRows = 16;      // templates per workgroup
constexpr int kTapWaves = 8;      // waves per workgroup, 16 columns (half-bin steps of qbar) each
constexpr int kTapCols = 16 * kTapWaves;
constexpr int kTapNodes = 64;     // quadrature nodes per step
constexpr int kMaxJobs = 32;      // width groups per launch

struct TapJob {
  const int32_t* members;
  double2* out;        // [n][2][taps]
  int32_t n, taps, panels;
  int32_t tile_begin;  // first workgroup of the job
};
struct TapJobs {
  TapJob job[kMaxJobs];
  double gl_x[16], gl_w[16];
  double zmax, dz, dw;
  int32_t n_jobs, n_z, J, margin;
};

// Nodes are kept in two parts, u = x + y: a phase of hundreds of cycles magnifies the rounding of u.
// exp(i pi n u) for an integer n; the product is reduced before it is rounded.
__device__ __forceinline__ double2 unit_int(int32_t n, double2 u) {
  const double x = (double)n * u.x;
  const double lo = fma((double)n, u.y, fma((double)n, u.x, -x));
  double s, c;
  sincospi((x - 2.0 * rint(0.5 * x)) + lo, &s, &c);
  return make_double2(c, s);
}

// u (a + u (b + u c)) modulo 1, by a compensated Horner scheme.
__device__ __forceinline__ double phase_cycles(double2 node, double a, double b, double c) {
#pragma clang fp contract(off)
  const double u = node.x;
  const double p1 = c * u, e1 = __builtin_fma(c, u, -p1);
  const double s1 = p1 + b, z1 = s1 - p1, d1 = (p1 - (s1 - z1)) + (b - z1);
  const double p2 = s1 * u, e2 = __builtin_fma(s1, u, -p2);
  const double s2 = p2 + a, z2 = s2 - p2, d2 = (p2 - (s2 - z2)) + (a - z2);
  const double p3 = s2 * u, e3 = __builtin_fma(s2, u, -p3);
  const double err = ((e1 + d1) * u + (e2 + d2)) * u + e3 + (a + u * (2.0 * b + 3.0 * c * u)) * node.y;
  return (p3 - rint(p3)) + err;
}

// A workgroup forms 16 templates x 128 columns of one group; column c is qbar = hg - 1/2 - c/2,
// that is tap j = c/2 and phase 1 - c%2. Per step of 64 nodes the threads put g (16 templates) and
// the factors of E (a base per node and wave, a step per node and column offset) into LDS; each
// lane multiplies its E together and the wave runs 16 k-steps of four products (real and imaginary
// parts). Bound by FP64 arithmetic: the products' matrix time and about as much for the sincospi of
// g. The 3131 templates of zmax 100 and wmax 300 (32 to 192 taps): 0.23 ms; one thread per tap with a
// sincospi per tap and node, on panels of one cycle of |q| + |z| + |w|/2, took 9.0 ms. Error against
// extended precision 2e-17 to 6e-16 RMS, where that kernel had 1e-16 to 9e-16.
__global__ void __launch_bounds__(64 * kTapWaves) tap_quadrature_kernel(TapJobs a) {
  __shared__ double2 g[kTapNodes][kTapRows];
  __shared__ double2 step[kTapNodes][16];
  __shared__ double2 base[kTapNodes][kTapWaves];
  __shared__ double cf[kTapRows][3];
  __shared__ int32_t half[kTapRows];
  __shared__ double glx[16], glw[16];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, col = lane & 15, quad = lane >> 4;
  int k = 0;
  while (k + 1 < a.n_jobs && (int32_t)blockIdx.x >= a.job[k + 1].tile_begin) ++k;
  const TapJob& j = a.job[k];
  const int32_t K = j.taps, local = (int32_t)blockIdx.x - j.tile_begin;
  const int32_t ncb = (2 * K + kTapCols - 1) / kTapCols;
  const int32_t row0 = local / ncb * kTapRows, col0 = local % ncb * kTapCols;
  if (tid < kTapRows) {
    const int32_t t = j.members[min(row0 + tid, j.n - 1)];
    const double zb = -a.zmax + (t % a.n_z) * a.dz;
    const double w = (t / a.n_z - a.J) * a.dw;
    cf[tid][0] = -0.5 * zb + w / 12.0;
    cf[tid][1] = 0.5 * (zb - 0.5 * w);
    cf[tid][2] = w / 6.0;
    half[tid] = (int32_t)ceil(fabs(zb) * 0.5 + fabs(w) / 12.0) + a.margin;
    glx[tid] = a.gl_x[tid];
    glw[tid] = a.gl_w[tid];
  }
  const int32_t nodes = 16 * j.panels;
  const double hw = 0.5 / j.panels;  // half panel width
  const int32_t wcol = col0 + 16 * wave;
  const bool busy = wcol < 2 * K;  // wave-uniform (K is a multiple of 16)
  d4vec sum_re = {0.0, 0.0, 0.0, 0.0}, sum_im = {0.0, 0.0, 0.0, 0.0};
  for (int32_t n0 = 0; n0 < nodes; n0 += kTapNodes) {
    __syncthreads();
    // (2 panel + 1 + x) / (2 panels) and the part lost to rounding
    auto node = [&](int32_t n) {
      const double m = (double)(2 * (n >> 4) + 1), x = glx[n & 15];
      const double h = m + x, l = x - (h - m);  // |x| < m
      const double u = h * hw;
      return make_double2(u, (fma(-u, (double)(2 * j.panels), h) + l) * hw);
    };
    for (int e = tid; e < kTapNodes * 16; e += 64 * kTapWaves) {
      const int kk = e >> 4, i = e & 15;
      const int32_t n = n0 + kk;
      const double2 u = node(n);
      const double wt = n < nodes ? glw[n & 15] : 0.0;  // times hw at the end
      double sn, c;
      sincospi(2.0 * phase_cycles(u, cf[i][0], cf[i][1], cf[i][2]), &sn, &c);
      g[kk][i] = make_double2(wt * c, wt * sn);
      step[kk][i] = unit_int(-i, u);
    }
    {
      const int kk = tid >> 3, w = tid & 7;
      base[kk][w] = unit_int(K - 1 - (col0 + 16 * w), node(n0 + kk));
    }
    __syncthreads();
    if (busy) {
      d4vec re = {0.0, 0.0, 0.0, 0.0}, im = {0.0, 0.0, 0.0, 0.0};  // per step, so that no sum grows long
#pragma unroll 4
      for (int ks = 0; ks < kTapNodes / 4; ++ks) {
        const int kk = 4 * ks + quad;
        const double2 gv = g[kk][col], st = step[kk][col], ba = base[kk][wave];
        const double ex = fma(ba.x, st.x, -ba.y * st.y), ey = fma(ba.x, st.y, ba.y * st.x);
        re = __builtin_amdgcn_mfma_f64_16x16x4f64(gv.x, ex, re, 0, 0, 0);
        im = __builtin_amdgcn_mfma_f64_16x16x4f64(gv.x, ey, im, 0, 0, 0);
        re = __builtin_amdgcn_mfma_f64_16x16x4f64(-gv.y, ey, re, 0, 0, 0);
        im = __builtin_amdgcn_mfma_f64_16x16x4f64(gv.y, ex, im, 0, 0, 0);
      }
      sum_re += re;
      sum_im += im;
    }
  }
  if (!busy) return;
  // register r of lane l holds row l/16 + 4 r, column l%16
  const int32_t c = wcol + col, jj = c >> 1, phase = 1 - (c & 1), hg = K / 2;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int i = quad + 4 * r;
    if (row0 + i >= j.n) continue;
    // tap j multiplies bin k0 - hg + 1 + j; conjugated: the correlation multiplies conj(T); zero
    // outside the template's own window
    const bool in = jj >= hg - half[i] && jj < hg + half[i];
    j.out[((int64_t)(row0 + i) * 2 + phase) * K + jj] = in ? make_double2(sum_re[r] * hw, -(sum_im[r] * hw)) : make_double2(0.0, 0.0);
  }
}

struct SpecJob {
  const double2* taps;  // [rows][K]
  float2* out;          // [rows][S]
  int32_t rows, K;      // rows: 2 per template
  int32_t tile_begin;
  int32_t pad;
};
struct SpecJobs {
  SpecJob job[kMaxJobs];
  int32_t n_jobs;
};
constexpr int kSpecRows = 8;  // rows per workgroup (they share the register twiddles)

// Spectra of one segment length: an FP64 Stockham FFT of each row's zero-padded taps in LDS,
// radix-4 passes and a last radix-2 one when log2 S is odd, rounded once to complex64.
// S/4 threads, one radix-4 butterfly each per pass. In place of the direct sum (one sincospi per
// tap and frequency) the work falls from K S to 2.5 S log2 S operations a row: 35 us instead of
// 2.2 ms for the 6262 rows of 1024 points of that grid, 51 MB written.
template <int S>
__global__ void __launch_bounds__(S / 4) tap_spectra_kernel(SpecJobs a) {
  constexpr int LOG = S == 512 ? 9 : S == 1024 ? 10 : S == 2048 ? 11 : 12;
  constexpr int P4 = LOG / 2;  // radix-4 passes
  __shared__ double2 x[S];
  const int tid = threadIdx.x;
  int k = 0;
  while (k + 1 < a.n_jobs && (int32_t)blockIdx.x >= a.job[k + 1].tile_begin) ++k;
  const SpecJob& j = a.job[k];
  const int32_t row0 = ((int32_t)blockIdx.x - j.tile_begin) * kSpecRows;
  const int32_t row1 = min(row0 + kSpecRows, j.rows);
  double2 w[P4][3];  // exp(+2 pi i r (tid mod L) / (4 L)) of the pass with span L = 4^p
#pragma unroll
  for (int p = 1; p < P4; ++p) {
    const int L = 1 << (2 * p);
#pragma unroll
    for (int r = 1; r < 4; ++r) {
      double s, c;
      sincospi((double)(r * (tid & (L - 1))) / (double)(2 * L), &s, &c);
      w[p][r - 1] = make_double2(c, s);
    }
  }
  auto mul = [](double2 u, double2 v) { return make_double2(fma(u.x, v.x, -u.y * v.y), fma(u.x, v.y, u.y * v.x)); };
  const double inv = 1.0 / (double)S;
  for (int32_t row = row0; row < row1; ++row) {
    const double2* c = j.taps + (int64_t)row * j.K;
    float2* out = j.out + (int64_t)row * S;
    auto put = [&](int f, double2 v) { out[f] = make_float2((float)(v.x * inv), (float)(v.y * inv)); };
#pragma unroll
    for (int p = 0; p < P4; ++p) {
      const int L = 1 << (2 * p);
      double2 v[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int i = tid + r * (S / 4);
        if (p == 0) v[r] = i < j.K ? c[i] : make_double2(0.0, 0.0);
        else v[r] = x[i];
      }
      __syncthreads();
      if (p > 0) {
#pragma unroll
        for (int r = 1; r < 4; ++r) v[r] = mul(v[r], w[p][r - 1]);
      }
      const double2 s0 = make_double2(v[0].x + v[2].x, v[0].y + v[2].y), d0 = make_double2(v[0].x - v[2].x, v[0].y - v[2].y);
      const double2 s1 = make_double2(v[1].x + v[3].x, v[1].y + v[3].y), d1 = make_double2(v[1].x - v[3].x, v[1].y - v[3].y);
      const double2 o[4] = {make_double2(s0.x + s1.x, s0.y + s1.y), make_double2(d0.x - d1.y, d0.y + d1.x),
                            make_double2(s0.x - s1.x, s0.y - s1.y), make_double2(d0.x + d1.y, d0.y - d1.x)};
      const int jj = tid & (L - 1);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int f = (tid - jj) * 4 + jj + L * r;
        if (LOG % 2 == 0 && p == P4 - 1) put(f, o[r]);
        else x[f] = o[r];
      }
      __syncthreads();
    }
    if (LOG % 2) {
#pragma unroll
      for (int m = 0; m < 2; ++m) {
        const int b = tid + m * (S / 4);
        double s, co;
        sincospi((double)b / (double)(S / 2), &s, &co);
        const double2 e = x[b], o = mul(x[b + S / 2], make_double2(co, s));
        put(b, make_double2(e.x + o.x, e.y + o.y));
        put(b + S / 2, make_double2(e.x - o.x, e.y - o.y));
      }
      __syncthreads();
    }
  }
}

// exp(-2 pi i k / n), k < n, from FP64 and rounded once to complex64; table y holds n = n0 << y.
struct TwiddleTables {
  float2* out[4];
};
__global__ void gen_twiddles_kernel(TwiddleTables a, int32_t n0) {
  const int32_t k = blockIdx.x * blockDim.x + threadIdx.x;
  const int32_t n = n0 << blockIdx.y;
  if (k >= n) return;
  double s, c;
  sincospi(-2.0 * (double)k / (double)n, &s, &c);
  a.out[blockIdx.y][k] = make_float2((float)c, (float)s);
}

// Everything of a job but its tile_begin; returns its workgroups.
int32_t tap_job(const Plan& p, TapJob& j, const int32_t* d_members, int32_t n, int32_t taps, double2* out) {
  const int32_t half = taps / 2;
  const int32_t cycles = half + std::max(0, half - p.desc.margin_bins);  // over u in [0, 1]
  j.members = d_members;
  j.out = out;
  j.n = n;
  j.taps = taps;
  j.panels = (cycles + 1) / 2 + 1;
  return (n + kTapRows - 1) / kTapRows * ((2 * taps + kTapCols - 1) / kTapCols);
}

void taps_enqueue(const Plan& p, TapJobs& a, int32_t tiles, hipStream_t stream) {
  for (int k = 0; k < 16; ++k) {
    a.gl_x[k] = p.gl_x[k];
    a.gl_w[k] = p.gl_w[k];
  }
  a.zmax = p.desc.zmax;
  a.dz = p.desc.dz;
  a.dw = p.desc.dw;
  a.n_z = p.n_z;
  a.J = p.J;
  a.margin = p.desc.margin_bins;
  hipLaunchKernelGGL(tap_quadrature_kernel, dim3((unsigned)tiles), dim3(64 * kTapWaves), 0, stream, a);
  JERK_HIP_CHECK(hipGetLastError());
}

void spectra_enqueue(const SpecJobs& a, int32_t S, int32_t tiles, hipStream_t stream) {
  switch (S) {
    case 512: hipLaunchKernelGGL(tap_spectra_kernel<512>, dim3((unsigned)tiles), dim3(128), 0, stream, a); break;
    case 1024: hipLaunchKernelGGL(tap_spectra_kernel<1024>, dim3((unsigned)tiles), dim3(256), 0, stream, a); break;
    case 2048: hipLaunchKernelGGL(tap_spectra_kernel<2048>, dim3((unsigned)tiles), dim3(512), 0, stream, a); break;
    case 4096: hipLaunchKernelGGL(tap_spectra_kernel<4096>, dim3((unsigned)tiles), dim3(1024), 0, stream, a); break;
    default: throw Error(JERK_EINTERNAL, "unsupported segment length");
  }
  JERK_HIP_CHECK(hipGetLastError());
}

int32_t spectra_tiles(int32_t n) { return (2 * n + kSpecRows - 1) / kSpecRows; }

}  // namespace

void gen_twiddles(float2* out, int32_t n, hipStream_t stream) {
  TwiddleTables t{{out, nullptr, nullptr, nullptr}};
  hipLaunchKernelGGL(gen_twiddles_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, stream, t, n);
  JERK_HIP_CHECK(hipGetLastError());
}

void gemm_bank_build(const Plan& p, const Group& g, const double2* taps, void* out, hipStream_t stream);

void taps_launch(const Plan& p, int32_t taps, const int32_t* d_members, int32_t n, double2* out, hipStream_t stream) {
  if (n <= 0) return;
  TapJobs a{};
  a.n_jobs = 1;
  const int32_t tiles = tap_job(p, a.job[0], d_members, n, taps, out);
  taps_enqueue(p, a, tiles, stream);
}

void fft_spectra_launch(const double2* taps, int32_t n, int32_t K, int32_t S, float2* out, hipStream_t stream) {
  if (n <= 0) return;
  SpecJobs a{};
  a.n_jobs = 1;
  a.job[0] = SpecJob{taps, out, 2 * n, K, 0, 0};
  spectra_enqueue(a, S, spectra_tiles(n), stream);
}

void bank_build(Plan& p, void* d_bank, hipStream_t stream) {
  if (!p.pinned_members) {
    void* h = nullptr;
    JERK_HIP_CHECK(hipHostMalloc(&h, sizeof(int32_t) * (size_t)p.T, hipHostMallocDefault));
    p.pinned_members = static_cast<int32_t*>(h);
    int32_t k = 0;
    for (const auto& g : p.groups)
      for (int32_t t : g.members) p.pinned_members[k++] = t;
  }
  char* bank = static_cast<char*>(d_bank);
  JERK_HIP_CHECK(hipMemcpyAsync(bank + p.off_members, p.pinned_members, sizeof(int32_t) * (size_t)p.T,
                                hipMemcpyHostToDevice, stream));
  TwiddleTables t;
  for (int i = 0; i < 4; ++i) t.out[i] = reinterpret_cast<float2*>(bank + p.off_tw[i]);
  hipLaunchKernelGGL(gen_twiddles_kernel, dim3(4096 / 256, 4), dim3(256), 0, stream, t, 512);
  JERK_HIP_CHECK(hipGetLastError());
  templates_build(p, d_bank, stream);
}

// Taps of all groups in one launch (widest groups first: theirs are the longest workgroups), then
// the spectra of all FFT-path groups of a segment length in one launch each; 32 groups a launch.
void templates_build(const Plan& p, void* d_bank, hipStream_t stream) {
  char* bank = static_cast<char*>(d_bank);
  const int32_t* d_members = reinterpret_cast<const int32_t*>(bank + p.off_members);
  auto taps_of = [&](const Group& g) { return reinterpret_cast<double2*>(bank + g.off_taps); };
  {
    TapJobs a{};
    int64_t tiles = 0;
    for (auto g = p.groups.rbegin(); g != p.groups.rend(); ++g) {
      const int32_t n = (int32_t)g->members.size();
      if (n == 0) continue;
      TapJob& j = a.job[a.n_jobs++];
      j.tile_begin = (int32_t)tiles;
      tiles += tap_job(p, j, d_members + g->first_member, n, g->taps, taps_of(*g));
      if (a.n_jobs == kMaxJobs) {
        taps_enqueue(p, a, (int32_t)tiles, stream);
        a.n_jobs = 0;
        tiles = 0;
      }
    }
    if (a.n_jobs > 0) taps_enqueue(p, a, (int32_t)tiles, stream);
  }
  for (int32_t S = 512; S <= 4096; S *= 2) {
    SpecJobs a{};
    int32_t tiles = 0;
    for (const Group& g : p.groups) {
      const int32_t n = (int32_t)g.members.size();
      if (n == 0 || g.path != JERK_PATH_FFT_FP32 || g.seg_len != S) continue;
      a.job[a.n_jobs++] = SpecJob{taps_of(g), reinterpret_cast<float2*>(bank + g.off_fft), 2 * n, g.taps, tiles, 0};
      tiles += spectra_tiles(n);
      if (a.n_jobs == kMaxJobs) {
        spectra_enqueue(a, S, tiles, stream);
        a.n_jobs = 0;
        tiles = 0;
      }
    }
    if (a.n_jobs > 0) spectra_enqueue(a, S, tiles, stream);
  }
  for (const Group& g : p.groups)
    if (!g.members.empty() && g.path != JERK_PATH_FFT_FP32) gemm_bank_build(p, g, taps_of(g), bank + g.off_gemm, stream);
}

}  // namespace jerk
