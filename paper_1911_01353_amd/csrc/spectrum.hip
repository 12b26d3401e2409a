// Spectrum preparation on the GPU: N real float32 samples -> N/2 complex64
// bins, DC zeroed and scaled to unit mean power above DC (the search's input
// contract), with every step in FP64.
//
// The N real samples are read as M = N/2 complex points z[m] = x[2m] + i x[2m+1].
// Their length-M DFT Z comes from self-sorting Stockham passes in global memory.
// A pass with sub-transform length L and radix R reads in[b + r M/R], r < R,
// multiplies by the twiddle w_{LR}^{r j} (j = b mod L) and writes the R-point DFT
// to out[j + L (r' + R q)], b = j + L q: after the last pass the result is in
// natural order. Radices run from 16 to 256 (a workgroup holds 4096 points in
// LDS, each thread 16 of them in registers), the last one 128, so 2^22 points
// take three passes over memory. The R-point DFTs are radix-2 butterflies, so a
// constant input gives exact zeros above DC (as a butterfly FFT in FP64 on the
// host does) rather than rounding noise that the normalisation would then blow up.
//
// The real spectrum follows from E[k] = (Z[k] + conj Z[M-k]) / 2 (even samples),
// O[k] = (Z[k] - conj Z[M-k]) / (2i) (odd samples), X[k] = E[k] + e^{-2 pi i k / N} O[k]
// and X[M-k] = conj(E[k] - e^{-2 pi i k / N} O[k]), inside the last pass, whose
// workgroups hold a run of columns and the mirrored run. The power sum above DC is
// reduced in a fixed order (per-block trees, then one tree over the blocks), so the
// result does not depend on scheduling. Up to 2^11 points one workgroup does it all.
#include "jerk_internal.h"

namespace jerk {
namespace {

constexpr int kThreads = 256;
constexpr int kPoints = 16 * kThreads;   // points of a workgroup in LDS (64 KB)
constexpr int kLastRadix = 128;          // of the pass that also splits
constexpr int kLastCols = kPoints / kLastRadix / 2;  // columns of its run (and of the mirrored one)
constexpr int kSmallMax = 2048;          // points of the one-workgroup transform
constexpr int64_t kMaxParts = 2048;      // partial power sums every block of the last step adds up

__device__ __forceinline__ double2 cmul(double2 a, double2 b) {
  return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
__device__ __forceinline__ double2 unit(double turns_times_two) {  // exp(i pi t)
  double s, c;
  sincospi(turns_times_two, &s, &c);
  return make_double2(c, s);
}

// In-register FP64 DFT of size R by radix-2 decimation in time.
template <int R>
struct DftD {
  __device__ __forceinline__ static void run(double2* x) {
    double2 e[R / 2], o[R / 2];
#pragma unroll
    for (int i = 0; i < R / 2; ++i) {
      e[i] = x[2 * i];
      o[i] = x[2 * i + 1];
    }
    DftD<R / 2>::run(e);
    DftD<R / 2>::run(o);
#pragma unroll
    for (int k = 0; k < R / 2; ++k) {
      const double2 t = k == 0 ? o[k] : cmul(o[k], unit(-2.0 * (double)k / (double)R));
      x[k] = make_double2(e[k].x + t.x, e[k].y + t.y);
      x[k + R / 2] = make_double2(e[k].x - t.x, e[k].y - t.y);
    }
  }
};
template <>
struct DftD<1> {
  __device__ __forceinline__ static void run(double2*) {}
};

// x[i] *= w^i, i < 16, the powers formed in a tree (four roundings at most).
__device__ __forceinline__ void mul_powers(double2 (&x)[16], double2 w) {
  double2 p[16];
  p[1] = w;
#pragma unroll
  for (int i = 2; i < 16; ++i) p[i] = cmul(p[i / 2], p[i - i / 2]);
#pragma unroll
  for (int i = 1; i < 16; ++i) x[i] = cmul(x[i], p[i]);
}

// 16 R2-point DFT of a column over the R2 threads that hold it: thread t2 enters with elements
// t2 + R2 i in x[i] and leaves with outputs i + 16 s in x[m R2 + s], i = t2 (16 / R2) + m. cols
// columns a workgroup; c: this thread's. The first barrier also orders an earlier use of lds.
template <int R2>
__device__ __forceinline__ void column_dft(double2 (&x)[16], double2* lds, int cols, int c, int t2) {
  DftD<16>::run(x);
  if constexpr (R2 > 1) {
    if (t2 > 0) mul_powers(x, unit(-2.0 * (double)t2 / (double)(16 * R2)));
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 16; ++i) lds[(i * R2 + t2) * cols + c] = x[i];
    __syncthreads();
#pragma unroll
    for (int m = 0; m < 16 / R2; ++m) {
#pragma unroll
      for (int t = 0; t < R2; ++t) x[m * R2 + t] = lds[((t2 * (16 / R2) + m) * R2 + t) * cols + c];
      DftD<R2>::run(&x[m * R2]);
    }
  }
}

// One pass of radix R = 16 R2 over a tile of 4096 / R consecutive butterflies. FIRST: the input is
// the series and L = 1; the tile's output is then one run of 4096 points, put in order through LDS
// (thread-contiguous stores made this pass three times as long as the others). Bound by memory:
// 16 bytes read and written a point at 2^22 points; see spectrum_prepare for the times.
template <int R2, bool FIRST>
__global__ void __launch_bounds__(kThreads) stockham_pass_fp64(const void* __restrict__ in_v, double2* __restrict__ out,
                                                               int64_t M, int32_t log_l) {
  constexpr int R = 16 * R2;
  const int64_t L = int64_t(1) << log_l;
  constexpr int C = kPoints / R;
  __shared__ double2 lds[kPoints];
  const int c = threadIdx.x % C, t2 = threadIdx.x / C;
  const int64_t b = (int64_t)blockIdx.x * C + c;
  const int64_t stride = M / R;
  double2 x[16];
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const int64_t at = b + (t2 + R2 * i) * stride;
    if constexpr (FIRST) {
      const float2 v = static_cast<const float2*>(in_v)[at];
      x[i] = make_double2((double)v.x, (double)v.y);
    } else {
      x[i] = static_cast<const double2*>(in_v)[at];
    }
  }
  const int64_t j = FIRST ? 0 : b & (L - 1);
  const int64_t q = FIRST ? b : b >> log_l;
  if constexpr (!FIRST) {  // w_{LR}^{(t2 + R2 i) j}
    mul_powers(x, unit(-2.0 * (double)j / (double)(16 * L)));
    if (t2 > 0) {
      const double2 w = unit(-2.0 * (double)(t2 * j) / (double)(L * R));
#pragma unroll
      for (int i = 0; i < 16; ++i) x[i] = cmul(x[i], w);
    }
  }
  column_dft<R2>(x, lds, C, c, t2);
  if constexpr (FIRST) {
    // [column][output], the output index's low bits turned by the column: 16 lanes on 16 bank groups
    __syncthreads();
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const int r = t2 * (16 / R2) + e / R2 + 16 * (e % R2);
      lds[c * R + (r ^ (c & 15))] = x[e];
    }
    __syncthreads();
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const int at = threadIdx.x + kThreads * e;
      const int cc = at / R;
      out[(int64_t)blockIdx.x * kPoints + at] = lds[at ^ (cc & 15)];
    }
  } else {
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const int r = t2 * (16 / R2) + e / R2 + 16 * (e % R2);
      out[j + L * (r + (int64_t)R * q)] = x[e];
    }
  }
}

__device__ __forceinline__ double block_sum(double v, double* red) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  double s = 0.0;
  for (int i = 0; i < (int)blockDim.x / 64; ++i) s += red[i];
  __syncthreads();
  return s;
}

// E and O of Z[k] and Z[M-k], O already times its twiddle w.
__device__ __forceinline__ void split(double2 zk, double2 zc, double2 w, double2& e, double2& t) {
  e = make_double2(0.5 * (zk.x + zc.x), 0.5 * (zk.y - zc.y));
  // (zk - conj zc) / (2i) = ((zk.y + zc.y) - i (zk.x - zc.x)) / 2
  t = cmul(make_double2(0.5 * (zk.y + zc.y), -0.5 * (zk.x - zc.x)), w);
}

// The last pass (R = 128, L = M / 128) of columns j = 16 T + i and their mirrors L - j, i < 16, and
// the real split of both: bins k = j + L r and M - k = (L - j) + L (127 - r). Column 0 is its own
// mirror (k = L r and L (128 - r)), and so is column L/2, which takes the mirrored column's place in
// that slot. X[k] for k < M (X[0] = 0) and the per-block sum of |X[k]|^2. Splitting here saves
// reading and writing 16 bytes a point once more.
__global__ void __launch_bounds__(kThreads) last_pass_kernel(const double2* __restrict__ in, int64_t M,
                                                             double2* __restrict__ X, double* __restrict__ part) {
  constexpr int R = kLastRadix, R2 = R / 16, C = 2 * kLastCols;
  __shared__ double2 lds[kPoints];
  const int64_t L = M / R;
  const int64_t j0 = (int64_t)blockIdx.x * kLastCols;
  const int c = threadIdx.x % C, t2 = threadIdx.x / C;
  const bool own = j0 == 0 && c % kLastCols == 0;
  const int64_t j = c < kLastCols ? j0 + c : own ? L / 2 : L - j0 - (c - kLastCols);
  double2 x[16];
#pragma unroll
  for (int i = 0; i < 16; ++i) x[i] = in[j + (t2 + R2 * i) * L];
  mul_powers(x, unit(-2.0 * (double)j / (double)(16 * L)));
  if (t2 > 0) {
    const double2 w = unit(-2.0 * (double)(t2 * j) / (double)M);
#pragma unroll
    for (int i = 0; i < 16; ++i) x[i] = cmul(x[i], w);
  }
  column_dft<R2>(x, lds, C, c, t2);
  __syncthreads();
#pragma unroll
  for (int e = 0; e < 16; ++e) {
    const int r = t2 * (16 / R2) + e / R2 + 16 * (e % R2);
    lds[r * C + c] = x[e];
  }
  __syncthreads();
  // thread: column i of the run, outputs r0 + 16 m
  const int i = threadIdx.x % kLastCols, r0 = threadIdx.x / kLastCols;
  double p = 0.0;
  auto add = [&](int64_t k, double2 v) {
    X[k] = v;
    p += v.x * v.x + v.y * v.y;
  };
  if (j0 == 0 && i == 0) {
    for (int m = 0; m < R / 16; ++m) {
      const int r = r0 + 16 * m;
      double2 e, t;
      split(lds[r * C], lds[(R - r) % R * C], unit(-(double)r / (double)R), e, t);
      add(L * r, r == 0 ? make_double2(0.0, 0.0) : make_double2(e.x + t.x, e.y + t.y));
      split(lds[r * C + kLastCols], lds[(R - 1 - r) * C + kLastCols], unit(-((double)r + 0.5) / (double)R), e, t);
      add(L / 2 + L * r, make_double2(e.x + t.x, e.y + t.y));
    }
  } else {
    const double2 w0 = unit(-(double)(j0 + i + L * r0) / (double)M);  // exp(-2 pi i k / N), N = 2 M
#pragma unroll
    for (int m = 0; m < R / 16; ++m) {
      const int r = r0 + 16 * m;
      const int64_t k = j0 + i + L * r;
      double2 e, t;
      split(lds[r * C + i], lds[(R - 1 - r) * C + kLastCols + i], m == 0 ? w0 : cmul(w0, unit(-(double)m / 8.0)), e, t);
      add(k, make_double2(e.x + t.x, e.y + t.y));
      add(M - k, make_double2(e.x - t.x, -(e.y - t.y)));
    }
  }
  __syncthreads();
  const double s = block_sum(p, reinterpret_cast<double*>(lds));
  if (threadIdx.x == 0) part[blockIdx.x] = s;
}

// Partial sums folded to gridDim.x of them, each over a run of the given ones.
__global__ void __launch_bounds__(kThreads) fold_parts_kernel(const double* __restrict__ part, int64_t n,
                                                              double* __restrict__ out) {
  __shared__ double red[kThreads / 64];
  const int64_t run = (n + gridDim.x - 1) / gridDim.x;
  const int64_t lo = blockIdx.x * run, hi = lo + run < n ? lo + run : n;
  double v = 0.0;
  for (int64_t i = lo + threadIdx.x; i < hi; i += kThreads) v += part[i];
  const double s = block_sum(v, red);
  if (threadIdx.x == 0) out[blockIdx.x] = s;
}

// scale = 1 / sqrt(mean power above DC), or 0 when that power is 0
__device__ __forceinline__ double power_scale(double sum, int64_t M) {
  const double mean = sum / (double)(M - 1);
  return mean > 0.0 ? 1.0 / sqrt(mean) : 0.0;
}

// Every block adds up the partial sums itself (the same order in each), then scales and rounds its
// run: no launch for the sum, which took 17 us over 2^14 sums in one block.
__global__ void __launch_bounds__(kThreads) scale_round_kernel(const double2* __restrict__ X, int64_t M,
                                                               const double* __restrict__ part, int32_t nparts,
                                                               float2* __restrict__ spec) {
  __shared__ double red[kThreads / 64];
  double v = 0.0;
  for (int32_t i = threadIdx.x; i < nparts; i += kThreads) v += part[i];
  const double s = power_scale(block_sum(v, red), M);
  for (int64_t k = (int64_t)blockIdx.x * kThreads + threadIdx.x; k < M; k += (int64_t)gridDim.x * kThreads) {
    const double2 x = X[k];
    spec[k] = make_float2((float)(x.x * s), (float)(x.y * s));
  }
}

// Everything for M <= 2048 points in one workgroup: radix-4 passes (and a radix-2 one) in LDS with
// a twiddle table, the split, the power and the scaling. Bound by its serial passes; it replaces up
// to six launches.
__global__ void __launch_bounds__(kSmallMax / 4) small_spectrum_kernel(const float2* __restrict__ z, int32_t M,
                                                                       float2* __restrict__ spec) {
  __shared__ double2 x[kSmallMax];
  __shared__ double2 tw[kSmallMax - kSmallMax / 4];  // exp(-2 pi i k / M), k < 3 M / 4
  const int tid = threadIdx.x, threads = blockDim.x;
  for (int k = tid; k < M; k += threads) {
    const float2 v = z[k];
    x[k] = make_double2((double)v.x, (double)v.y);
    if (4 * k < 3 * M) tw[k] = unit(-2.0 * (double)k / (double)M);
  }
  __syncthreads();
  int L = 1;
  for (; 4 * L <= M; L *= 4) {  // one butterfly a thread: M / 4 <= threads
    const int j = tid & (L - 1);
    double2 v[4];
    if (tid < M / 4) {
#pragma unroll
      for (int r = 0; r < 4; ++r) v[r] = x[tid + r * (M / 4)];
      if (L > 1) {
#pragma unroll
        for (int r = 1; r < 4; ++r) v[r] = cmul(v[r], tw[r * j * (M / (4 * L))]);
      }
      DftD<4>::run(v);
    }
    __syncthreads();
    if (tid < M / 4) {
#pragma unroll
      for (int r = 0; r < 4; ++r) x[(tid - j) * 4 + j + L * r] = v[r];
    }
    __syncthreads();
  }
  if (L < M) {  // radix 2, L = M / 2
    for (int b = tid; b < M / 2; b += threads) {
      const double2 e = x[b], o = b == 0 ? x[M / 2] : cmul(x[b + M / 2], tw[b]);
      x[b] = make_double2(e.x + o.x, e.y + o.y);
      x[b + M / 2] = make_double2(e.x - o.x, e.y - o.y);
    }
    __syncthreads();
  }
  constexpr int kMost = 4;  // bins of a thread: M <= 4 threads
  double2 X[kMost];
  double p = 0.0;
#pragma unroll
  for (int m = 0; m < kMost; ++m) {
    const int k = tid + m * threads;
    X[m] = make_double2(0.0, 0.0);
    if (k > 0 && k < M) {
      double2 e, t;
      split(x[k], x[M - k], unit(-(double)k / (double)M), e, t);
      X[m] = make_double2(e.x + t.x, e.y + t.y);
      p += X[m].x * X[m].x + X[m].y * X[m].y;
    }
  }
  __syncthreads();
  const double s = power_scale(block_sum(p, reinterpret_cast<double*>(tw)), M);
#pragma unroll
  for (int m = 0; m < kMost; ++m) {
    const int k = tid + m * threads;
    if (k < M) spec[k] = make_float2((float)(X[m].x * s), (float)(X[m].y * s));
  }
}

struct WsLayout {
  size_t a, b, part, fold, total;
};

int64_t last_pass_blocks(int64_t M) { return M / kPoints; }  // kLastCols columns and their mirrors each

WsLayout ws_layout(int64_t M) {
  WsLayout w{};
  w.a = 0;
  w.b = align_up((size_t)M * sizeof(double2));
  w.part = w.b + align_up((size_t)M * sizeof(double2));               // last_pass_blocks sums
  w.fold = w.part + align_up((size_t)last_pass_blocks(M) * sizeof(double));  // kMaxParts of them, if there are more
  // one sum per kThreads points and a value: the size callers have been told, more than both take
  w.total = w.part + align_up((size_t)((M + kThreads - 1) / kThreads) * sizeof(double)) + kAlign;
  return w;
}

template <bool FIRST>
void launch_pass(int bits, const void* in, double2* out, int64_t M, int32_t log_l, hipStream_t stream) {
  const dim3 grid((unsigned)(M / kPoints)), block(kThreads);
  switch (bits) {
    case 4: hipLaunchKernelGGL((stockham_pass_fp64<1, FIRST>), grid, block, 0, stream, in, out, M, log_l); break;
    case 5: hipLaunchKernelGGL((stockham_pass_fp64<2, FIRST>), grid, block, 0, stream, in, out, M, log_l); break;
    case 6: hipLaunchKernelGGL((stockham_pass_fp64<4, FIRST>), grid, block, 0, stream, in, out, M, log_l); break;
    case 7: hipLaunchKernelGGL((stockham_pass_fp64<8, FIRST>), grid, block, 0, stream, in, out, M, log_l); break;
    case 8: hipLaunchKernelGGL((stockham_pass_fp64<16, FIRST>), grid, block, 0, stream, in, out, M, log_l); break;
    default: throw Error(JERK_EINTERNAL, "no FFT pass of this radix");
  }
  JERK_HIP_CHECK(hipGetLastError());
}

}  // namespace

size_t spectrum_workspace_bytes(int64_t n_samples) { return ws_layout(n_samples / 2).total; }

void spectrum_prepare(const float* series, int64_t n_samples, float2* spec, void* ws, size_t ws_bytes,
                      hipStream_t stream) {
  const int64_t M = n_samples / 2;
  const WsLayout w = ws_layout(M);
  require(ws_bytes >= w.total, JERK_ENOMEM, "spectrum workspace too small");
  if (M <= kSmallMax) {
    const unsigned threads = (unsigned)(M / 4 < 64 ? 64 : M / 4);
    hipLaunchKernelGGL(small_spectrum_kernel, dim3(1), dim3(threads), 0, stream,
                       reinterpret_cast<const float2*>(series), (int32_t)M, spec);
    JERK_HIP_CHECK(hipGetLastError());
    return;
  }
  char* base = static_cast<char*>(ws);
  double2* buf[2] = {reinterpret_cast<double2*>(base + w.a), reinterpret_cast<double2*>(base + w.b)};
  double* part = reinterpret_cast<double*>(base + w.part);
  // log2 M - 7 >= 5 bits before the last pass, in as few passes of at most 8 bits as hold them,
  // the bits shared out evenly (each pass costs a read and a write of 16 bytes a point). 2^22 bins:
  // 19 + 25 + 29 us for the passes of radix 256, 128 and 128 (the last with the split) and 18 us for
  // the scaling, 90 us with the gaps; five passes of radix 16, one of 4, the split and the power sum by
  // themselves took 222 us. 2^16 bins 33 -> 25 us, 2^11 bins and fewer 20 -> 9 us.
  int log_m = 0;
  while ((int64_t(1) << log_m) < M) ++log_m;
  int rest = log_m - 7, passes = (rest + 7) / 8;
  const void* in = series;
  int log_l = 0, cur = 0;
  for (; passes > 0; --passes) {
    const int bits = (rest + passes - 1) / passes;
    if (log_l == 0) launch_pass<true>(bits, in, buf[cur], M, log_l, stream);
    else launch_pass<false>(bits, in, buf[cur], M, log_l, stream);
    in = buf[cur];
    cur ^= 1;
    log_l += bits;
    rest -= bits;
  }
  double2* X = buf[cur];
  int64_t nparts = last_pass_blocks(M);
  hipLaunchKernelGGL(last_pass_kernel, dim3((unsigned)nparts), dim3(kThreads), 0, stream,
                     static_cast<const double2*>(in), M, X, part);
  JERK_HIP_CHECK(hipGetLastError());
  if (nparts > kMaxParts) {  // M > 2^23
    double* const folded = reinterpret_cast<double*>(base + w.fold);
    require(w.fold + (size_t)kMaxParts * sizeof(double) <= w.total, JERK_EINTERNAL, "folded sums outside the workspace");
    hipLaunchKernelGGL(fold_parts_kernel, dim3((unsigned)kMaxParts), dim3(kThreads), 0, stream, part, nparts, folded);
    JERK_HIP_CHECK(hipGetLastError());
    part = folded;
    nparts = kMaxParts;
  }
  const int64_t blocks = M / 1024;
  hipLaunchKernelGGL(scale_round_kernel, dim3((unsigned)(blocks < 2048 ? blocks : 2048)), dim3(kThreads), 0, stream, X, M,
                     part, (int32_t)nparts, spec);
  JERK_HIP_CHECK(hipGetLastError());
}

}  // namespace jerk
