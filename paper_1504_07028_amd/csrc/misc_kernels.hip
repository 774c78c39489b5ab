// Set-up, initialisation, layout conversion and read-out kernels.
#include <cstring>
#include "segsalsa_internal.h"
#include "segsalsa_kernels.h"

namespace segsalsa {

// Twiddle tables exp(-2 pi i t / N) and the 1-D symbols 4 sin^2(pi t / N) of
// D^T D (periodic forward difference), in FP64 then rounded to T, and the fold
// lists.  One table per block row (blockIdx.y + first): the launch lasts one
// table's chain of FP64 sines or divisions instead of all of them (24x37 FP64:
// 11.1 -> 6.3 us).
enum SetupJob : int { kJobRows, kJobCols, kJobTwW, kJobTwH, kJobSym, kJobTwMW, kJobTwMH, kJobCh, kSetupJobs };

template <typename T>
__device__ inline C2<T> unit_root(double turns) {   // exp(-i pi turns)
  double s, c;
  sincospi(turns, &s, &c);
  return C2<T>{T(c), T(-s)};
}

template <typename T>
__global__ void setup_kernel(const SetupArgs<T> a) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  const double dt = (double)t, dW = (double)a.W, dH = (double)a.H;
  const uint32_t plane = a.g.ER * a.g.EC;
  switch (blockIdx.y) {
    case kJobRows: {   // (the host checked that no list overflows)
      if (t == 0) {
        *a.form_first = *a.form;
        if (a.form_after >= 0) *a.form = a.form_after;
      }
      if (t >= a.H) return;
      FoldEnt e = {fold_list(a.g, t, true, a.frow + a.H + t, a.H), {0u, 0u}, 0};
      a.frow[t] = e.n;
      if (!a.wrow) return;
      for (int i = 0; i < 2 && i < e.n; ++i) {   // byte offsets of the first two entries of the list just written
        const int f = a.frow[(size_t)(1 + i) * a.H + t];
        e.off[i] = 4u * ((uint32_t)(f >> kFoldShift) * a.g.ntc * a.K * plane + (uint32_t)(f & kFoldMask) * a.g.EC);
      }
      a.wrow[t] = e;
      return;
    }
    case kJobCols: {
      if (t >= a.W) return;
      FoldEnt e = {fold_list(a.g, t, false, a.fcol + a.W + t, a.W), {0u, 0u}, 0};
      a.fcol[t] = e.n;
      if (!a.wcol) return;
      for (int i = 0; i < 2 && i < e.n; ++i) {
        const int f = a.fcol[(size_t)(1 + i) * a.W + t];
        e.off[i] = 4u * ((uint32_t)(f >> kFoldShift) * a.K * plane + (uint32_t)(f & kFoldMask));
      }
      a.wcol[t] = e;
      return;
    }
    case kJobTwW:
      if (t < a.W) a.twW[t] = unit_root<T>(2.0 * dt / dW);
      return;
    case kJobTwH:
      if (t < a.H) a.twH[t] = unit_root<T>(2.0 * dt / dH);
      return;
    case kJobSym: {
      if (t < a.W) {
        const double h = sinpi(dt / dW);
        a.sx[t] = 4.0 * h * h;
      }
      if (t < a.H) {
        const double h = sinpi(dt / dH);
        a.sy[t] = 4.0 * h * h;
      }
      return;
    }
    case kJobTwMW:
      if (t < a.MW) a.twMW[t] = unit_root<T>(2.0 * dt / (double)a.MW);
      return;
    case kJobTwMH:
      if (t < a.MH) a.twMH[t] = unit_root<T>(2.0 * dt / (double)a.MH);
      return;
    case kJobCh:   // Bluestein chirps, angle pi (t^2 mod 2N) / N (t < 2^12)
      if (a.MW && t < a.W) a.chW[t] = unit_root<T>((double)(((uint32_t)t * t) % (2u * a.W)) / dW);
      if (a.MH && t < a.H) a.chH[t] = unit_root<T>((double)(((uint32_t)t * t) % (2u * a.H)) / dH);
      return;
  }
}

template <typename T>
hipError_t launch_setup_t(const SetupArgs<T>& a, hipStream_t st) {
  int n = a.W > a.H ? a.W : a.H;
  n = n > a.MW ? n : a.MW;
  n = n > a.MH ? n : a.MH;
  // the window solve takes the fold lists only; the last jobs are Bluestein's
  const int jobs = a.wrow ? kJobTwW : (a.MW || a.MH) ? kSetupJobs : kJobTwMW;
  hipLaunchKernelGGL(setup_kernel<T>, dim3((n + 63) / 64, jobs), dim3(64), 0, st, a);
  return hipGetLastError();
}
hipError_t launch_setup(const SetupArgs<float>& a, hipStream_t st) { return launch_setup_t(a, st); }
hipError_t launch_setup(const SetupArgs<double>& a, hipStream_t st) { return launch_setup_t(a, st); }

// Initial state: p_hat = p / 1^T p (or softmax of logits), z = p_hat, d3 = 0, and
// the per-pixel gain and d4 are 0, which makes d1 = d4 = 0.
template <typename T>
__global__ void init_kernel(const InitArgs<T> a) {
  const int H = a.g.H, W = a.g.W, K = a.K;
  const size_t n = (size_t)H * W;
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const int r = (int)(i / W), c = (int)(i - (size_t)r * W);
  int flags = 0;
  double mx = -1.0 / 0.0;
  double sum = 0.0;
  if (a.is_logits) {
    for (int k = 0; k < K; ++k) {
      const double x = (double)a.input[(size_t)k * n + i];
      if (!isfinite(x)) flags |= 1;
      mx = fmax(mx, x);
    }
    for (int k = 0; k < K; ++k) sum += exp((double)a.input[(size_t)k * n + i] - mx);
  } else {
    for (int k = 0; k < K; ++k) {
      const double x = (double)a.input[(size_t)k * n + i];
      if (!isfinite(x)) flags |= 1;
      if (x < 0.0) flags |= 2;
      sum += x;
    }
  }
  if (!(sum > 0.0)) flags |= 4;
  const double inv = 1.0 / sum;
  int tile, step, lane;
  tile_pos(a.g, r, c, tile, step, lane);
  const size_t st = (size_t)tile * a.g.steps + step, sb = st * K;
  char* px = a.px + st * a.px_stride;
  reinterpret_cast<double*>(px)[lane] = 0.0;
  reinterpret_cast<T*>(px + 512)[lane] = T(0);
  for (int k = 0; k < K; ++k) {
    const double x = (double)a.input[(size_t)k * n + i];
    const T ph = T(a.is_logits ? exp(x - mx) * inv : x * inv);
    a.z[(size_t)k * n + i] = ph;
    a.phat[(sb + k) * 64 + lane] = ph;
    a.d3[(sb + k) * 64 + lane] = T(0);
  }
  if (flags) atomicOr(a.flags, flags);
}

template <typename T>
hipError_t launch_init_t(const InitArgs<T>& a, hipStream_t st) {
  const size_t n = (size_t)a.g.H * a.g.W;
  hipLaunchKernelGGL(init_kernel<T>, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, a);
  return hipGetLastError();
}
hipError_t launch_init(const InitArgs<float>& a, hipStream_t st) { return launch_init_t(a, st); }
hipError_t launch_init(const InitArgs<double>& a, hipStream_t st) { return launch_init_t(a, st); }

__global__ void fill_zero_kernel(uint4* p, size_t n16, unsigned char* tail, size_t ntail) {
  const size_t stride = (size_t)gridDim.x * blockDim.x;
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n16; i += stride) p[i] = make_uint4(0, 0, 0, 0);
  if (blockIdx.x == 0 && threadIdx.x < ntail) tail[threadIdx.x] = 0;
}

hipError_t launch_fill_zero(void* p, size_t bytes, hipStream_t st) {
  if (bytes == 0) return hipSuccess;
  const size_t n16 = bytes / 16;
  const size_t ntail = bytes - n16 * 16;
  size_t blocks = (n16 + 255) / 256;
  if (blocks > 65536) blocks = 65536;
  if (blocks == 0) blocks = 1;
  hipLaunchKernelGGL(fill_zero_kernel, dim3((unsigned)blocks), dim3(256), 0, st, reinterpret_cast<uint4*>(p), n16,
                     reinterpret_cast<unsigned char*>(p) + n16 * 16, ntail);
  return hipGetLastError();
}

// Several host blocks in as few launches as their bytes need (kernel arguments
// hold about 4 KB).
struct StoreBlob {
  static constexpr int kSegs = 8, kWords = 896;
  unsigned* dst[kSegs];
  int first[kSegs + 1];   // word ranges of the segments
  unsigned w[kWords];
};

__global__ void store_kernel(StoreBlob blob, int segs) {
  for (int q = 0; q < segs; ++q)
    for (int i = blob.first[q] + threadIdx.x; i < blob.first[q + 1]; i += blockDim.x)
      blob.dst[q][i - blob.first[q]] = blob.w[i];
}

hipError_t launch_store(const StorePart* parts, int n, hipStream_t st) {
  StoreBlob blob;
  int segs = 0, used = 0;
  auto flush = [&]() {
    if (segs == 0) return hipSuccess;
    blob.first[segs] = used;
    hipLaunchKernelGGL(store_kernel, dim3(1), dim3(256), 0, st, blob, segs);
    segs = used = 0;
    return hipGetLastError();
  };
  for (int p = 0; p < n; ++p) {
    const unsigned char* src = reinterpret_cast<const unsigned char*>(parts[p].src);
    int left = (int)(parts[p].bytes / 4);
    unsigned* dst = reinterpret_cast<unsigned*>(parts[p].dst);
    while (left > 0) {
      if (segs == StoreBlob::kSegs || used == StoreBlob::kWords) {
        hipError_t e = flush();
        if (e != hipSuccess) return e;
      }
      const int m = left < StoreBlob::kWords - used ? left : StoreBlob::kWords - used;
      blob.dst[segs] = dst;
      blob.first[segs] = used;
      std::memcpy(blob.w + used, src, 4 * (size_t)m);
      ++segs;
      used += m;
      dst += m;
      src += 4 * (size_t)m;
      left -= m;
    }
  }
  return flush();
}

struct StorePair {
  unsigned char* dst[2];
  int n[2];
  unsigned char b[2][kStorePairMax];
};

__global__ void store_pair_kernel(StorePair sp) {
  for (int q = 0; q < 2; ++q)
    for (int i = threadIdx.x; i < sp.n[q]; i += blockDim.x) sp.dst[q][i] = sp.b[q][i];
}

hipError_t launch_store_pair(void* dst0, const void* src0, size_t n0, void* dst1, const void* src1, size_t n1,
                             hipStream_t st) {
  if (n0 > (size_t)kStorePairMax || n1 > (size_t)kStorePairMax) return hipErrorInvalidValue;
  StorePair sp;
  sp.dst[0] = reinterpret_cast<unsigned char*>(dst0);
  sp.dst[1] = reinterpret_cast<unsigned char*>(dst1);
  sp.n[0] = (int)n0;
  sp.n[1] = (int)n1;
  std::memcpy(sp.b[0], src0, n0);
  std::memcpy(sp.b[1], src1, n1);
  hipLaunchKernelGGL(store_pair_kernel, dim3(1), dim3(64), 0, st, sp);
  return hipGetLastError();
}

// Tile layout <-> canonical layouts, one thread per (pixel, class).
template <typename T>
__global__ void state_kernel(const StateArgs<T> a) {
  const int H = a.g.H, W = a.g.W, K = a.K, L = a.L;
  const size_t n = (size_t)H * W;
  const size_t gid = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (gid >= n * K) return;
  const int k = (int)(gid / n);
  const size_t i = gid - (size_t)k * n;
  const int r = (int)(i / W), c = (int)(i - (size_t)r * W);
  int tile, step, lane;
  tile_pos(a.g, r, c, tile, step, lane);
  const size_t st = (size_t)tile * a.g.steps + step, kb = st * K + k;
  const size_t e1 = (st * 2 * K + k) * 64 + lane, e4 = e1 + (size_t)K * 64;   // d1, d4 in dfull
  const size_t ci = (size_t)k * n + i;
  if (a.to_canonical) {
    const int form = *a.form;
    const char* px = a.px_t + st * a.px_stride;
    const T ph = a.phat_t[kb * 64 + lane];
    if (a.phat) a.phat[ci] = ph;
    if (a.d1)
      a.d1[ci] = form & kFormD1 ? a.dfull_t[e1] : T((double)ph * reinterpret_cast<const double*>(px)[lane]);
    if (a.d3) a.d3[ci] = a.d3_t[kb * 64 + lane];
    if (a.d4) a.d4[ci] = form & kFormD4 ? a.dfull_t[e4] : reinterpret_cast<const T*>(px + 512)[lane];
    if (a.d2) {
      for (int j = 0; j < L; ++j) {
        const C2<T> v = reinterpret_cast<const C2<T>*>(a.d2_t)[(kb * L + j) * 64 + lane];
        a.d2[((size_t)(j * 2 + 0) * K + k) * n + i] = v.x;
        a.d2[((size_t)(j * 2 + 1) * K + k) * n + i] = v.y;
      }
    }
  } else {
    a.phat_t[kb * 64 + lane] = a.phat[ci];
    if (gid == 0) *a.form = kFormD1 | kFormD4;
    a.dfull_t[e1] = a.d1[ci];
    a.d3_t[kb * 64 + lane] = a.d3[ci];
    a.dfull_t[e4] = a.d4[ci];
    for (int j = 0; j < L; ++j) {
      C2<T> v;
      v.x = a.d2[((size_t)(j * 2 + 0) * K + k) * n + i];
      v.y = a.d2[((size_t)(j * 2 + 1) * K + k) * n + i];
      reinterpret_cast<C2<T>*>(a.d2_t)[(kb * L + j) * 64 + lane] = v;
    }
  }
}

template <typename T>
hipError_t launch_state_t(const StateArgs<T>& a, hipStream_t st) {
  const size_t tot = (size_t)a.g.H * a.g.W * a.K;
  hipLaunchKernelGGL(state_kernel<T>, dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, st, a);
  return hipGetLastError();
}
hipError_t launch_state(const StateArgs<float>& a, hipStream_t st) { return launch_state_t(a, st); }
hipError_t launch_state(const StateArgs<double>& a, hipStream_t st) { return launch_state_t(a, st); }

// Segmentation read-out: argmax over classes, lowest class on ties.
template <typename T>
__global__ void labels_kernel(int K, size_t n, const T* __restrict__ z, int32_t* __restrict__ lab) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  T best = z[i];
  int arg = 0;
  for (int k = 1; k < K; ++k) {
    const T v = z[(size_t)k * n + i];
    if (v > best) {
      best = v;
      arg = k;
    }
  }
  lab[i] = arg;
}

template <typename T>
hipError_t launch_labels_t(int K, int H, int W, const T* z, int32_t* lab, hipStream_t st) {
  const size_t n = (size_t)H * W;
  hipLaunchKernelGGL(labels_kernel<T>, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, K, n, z, lab);
  return hipGetLastError();
}
hipError_t launch_labels(int K, int H, int W, const float* z, int32_t* lab, hipStream_t st) {
  return launch_labels_t(K, H, W, z, lab, st);
}
hipError_t launch_labels(int K, int H, int W, const double* z, int32_t* lab, hipStream_t st) {
  return launch_labels_t(K, H, W, z, lab, st);
}

}  // namespace segsalsa
