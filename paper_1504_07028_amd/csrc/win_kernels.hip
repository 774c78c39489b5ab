// z-update solve (eq. (12)) of FP32 images in one launch, by overlapping windows.
//
// A = 3 I + Wsum (D_h^T D_h + D_v^T D_v) is diagonally dominant, so its
// inverse decays geometrically: summed over one direction it is the 1-D
// Green's function rho^(|r| + 1) / (Wsum (1 - rho^2)) with rho the root below
// 1 of rho + 1/rho = 3 / Wsum + 2 (rho = 0.2087 at Wsum = 1, the paper's
// normalised weights).  A window that holds the right-hand side R pixels
// beyond the pixels it is solved for therefore gives them to within
//   2 rho^(R + 2) / (Wsum (1 - rho^2) (1 - rho)) x max |rhs change|,
// 8e-10 at R = 12, whatever is assumed beyond the window (per direction).  The
// host takes the smallest R that holds this below 2^-28, a sixteenth of the
// FP32 rounding unit (win_halo), and solves larger weights, FP64, the
// differentiable solve and tuned entries that ask for particular DFT kernels
// by the three passes over the whole image.
//
// A window is 64 rows x NX columns of one pair of classes (real and imaginary
// part), solved as the three passes solve the image: a DFT along one
// direction (here the 64 rows, periodic in the window), then for every
// frequency the constant-coefficient tridiagonal system along the other, then
// the inverse DFT.  The tridiagonal inverse is the sum of a forward and a
// backward first-order recursion,
//   1 / ((1 - rho S)(1 - rho S^-1)) = [1 / (1 - rho S) + 1 / (1 - rho S^-1) - 1] / (1 - rho^2),
// with nothing assumed before the first and after the last column.
//
// Layout: wavefront (t, xh) takes rows t + 4 q (q < 16), lane = column, so
// that the gather and the stores run along image rows and a row's fold entry
// is wavefront-uniform (a scalar offset of buffer loads).  The 64-point DFT is
// two radix-8 stages with one exchange through LDS between the four
// wavefronts; its twiddles are uniform per wavefront.  For the
// recursions lane = frequency and a wavefront takes 16 columns: it runs the
// recursions from 0 for its chunk's carries, and then from the carries of the
// two chunks before it (rho^32 of anything further).  Every stage writes the LDS slots that it has
// read, so five barriers order the whole solve.  The LDS row pitch NX + 1 is
// odd: no bank conflicts in either orientation.
//
// Rounding: z is rounded alike in every round once the iterates settle, and
// the multipliers add up what the solve does to a field each time, so errors
// that do not average out count most.  The recursions' gain makes the response
// to values constant along a row exact for the rounded rho, the gain and the
// DFT's 1 / sqrt(2) are each the sum of two FP32 numbers, the twiddles have
// |w|^2 close to 1 (kW64), and a value passes one rounding per recursion.
// Relative to FP64 (root mean square over 8 to 16 images, 20 rounds), rounded
// gain, twiddles and separate carries -> here (three passes): 64x64 K = 4
// 2.3e-7 -> 1.45e-7 (1.65e-7), 64x64 K = 8 5x5 2.6e-7 -> 1.6e-7 (1.8e-7),
// 110x60 K = 11 2.5e-7 -> 1.4e-7 (1.5e-7), 128x64 K = 4 1.8e-7 -> 1.4e-7
// (1.6e-7), below the three passes at all 29 shapes tried; same times.
//
// What bounds it: up to 200x311 its time hardly depends on the size (8.7 to
// 9.7 us): a chain of dependent reads (descriptor, fold entries, partial sums)
// and five barriers.  At large sizes it grows with the window pixels, 2.56
// (NX = 64) or 1.97 (NX = 128) per pixel solved at R = 12; at 2048x2048 its
// wavefronts issue VALU instructions in 16 % of their cycles, wait in 30 % and
// are ready but not issued in 42 %, and it moves 0.81 GB at 3.4 TB/s.  One
// launch instead of three and two round trips of the spectrum less; us per
// round, three passes -> windows (rocprofv3): 64x64 K=4 19.0 -> 9.6, 97x131 K=9
// 27.8 -> 9.7, 145x145 K=16 26.3 -> 8.7, 200x311 K=6 41.1 -> 8.9, 610x340 K=9
// 46.9 -> 15.6, 64 images of 96..512 733 -> 272, 2048x2048 K=16 433 -> 236 (on
// 20x32 tiles; 289 on 20x16 ones, whose grown tiles overlap more).
#include "segsalsa_internal.h"
#include "segsalsa_kernels.h"
#include "fft_math.h"

namespace segsalsa {

// exp(-2 pi i m / 64) for m = s k, s < 8, k < 8: the twiddles between the
// DFT's two stages.  Each part is the nearest FP32 number or one beside it, the
// pair whose |w|^2 is closest to 1: the forward and the inverse transform
// multiply by w and its conjugate, so what |w|^2 misses is a gain error of the
// frequency in every round, which the multipliers add up.
static __device__ const C2<float> kW64[50] = {
    {1.0f, 0.0f}, {0.99518472f, -0.0980171487f}, {0.980785251f, -0.195090339f}, {0.956940353f, -0.290284634f},
    {0.923879564f, -0.382683396f}, {0.881921232f, -0.471396774f}, {0.831469595f, -0.555570245f}, {0.773010433f, -0.634393334f},
    {0.707106769f, -0.707106769f}, {0.634393334f, -0.773010433f}, {0.555570245f, -0.831469595f}, {0.471396774f, -0.881921232f},
    {0.382683396f, -0.923879564f}, {0.290284634f, -0.956940353f}, {0.195090339f, -0.980785251f}, {0.0980171487f, -0.99518472f},
    {0.0f, -1.0f}, {-0.0980171487f, -0.99518472f}, {-0.195090339f, -0.980785251f}, {-0.290284634f, -0.956940353f},
    {-0.382683396f, -0.923879564f}, {-0.471396774f, -0.881921232f}, {-0.555570245f, -0.831469595f}, {-0.634393334f, -0.773010433f},
    {-0.707106769f, -0.707106769f}, {-0.773010433f, -0.634393334f}, {-0.831469595f, -0.555570245f}, {-0.881921232f, -0.471396774f},
    {-0.923879564f, -0.382683396f}, {-0.956940353f, -0.290284634f}, {-0.980785251f, -0.195090339f}, {-0.99518472f, -0.0980171487f},
    {-1.0f, 0.0f}, {-0.99518472f, 0.0980171487f}, {-0.980785251f, 0.195090339f}, {-0.956940353f, 0.290284634f},
    {-0.923879564f, 0.382683396f}, {-0.881921232f, 0.471396774f}, {-0.831469595f, 0.555570245f}, {-0.773010433f, 0.634393334f},
    {-0.707106769f, 0.707106769f}, {-0.634393334f, 0.773010433f}, {-0.555570245f, 0.831469595f}, {-0.471396774f, 0.881921232f},
    {-0.382683396f, 0.923879564f}, {-0.290284634f, 0.956940353f}, {-0.195090339f, 0.980785251f}, {-0.0980171487f, 0.99518472f},
    {0.0f, 1.0f}, {0.0980171487f, 0.99518472f},
};

// The DFT of 8 values as Bfly<float, 8>, with 1 / sqrt(2) as the sum of two
// FP32 numbers, for the same reason.
__device__ __forceinline__ void bfly8(C2<float>* v, float sg) {
  using C = C2<float>;
  auto half = [](float t) { return 0.707106769f * t + 1.21016175e-8f * t; };
  C e[4] = {v[0], v[2], v[4], v[6]}, o[4] = {v[1], v[3], v[5], v[7]};
  Bfly<float, 4>::run(e, sg);
  Bfly<float, 4>::run(o, sg);
  const C r[4] = {o[0], C{half(o[1].x - sg * o[1].y), half(o[1].y + sg * o[1].x)}, cmuli(o[2], sg),
                  C{half(-o[3].x - sg * o[3].y), half(-o[3].y + sg * o[3].x)}};
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    v[q] = cadd(e[q], r[q]);
    v[q + 4] = csub(e[q], r[q]);
  }
}

__device__ __forceinline__ FoldEnt ldf(gptr<const FoldEnt> p) { return FoldEnt{p->n, {p->off[0], p->off[1]}, 0}; }

// floor(n / d) with m = ceil(2^32 / d), or n with m = 0 (d = 1); exact while n d < 2^32
__device__ __forceinline__ uint32_t udiv(uint32_t n, uint32_t m) { return m ? __umulhi(n, m) : n; }
__device__ __forceinline__ int wrap(uint32_t n, uint32_t d, uint32_t m) { return (int)(n - udiv(n, m) * d); }

// Raw buffer accesses of FP32 words (byte offsets: lane + scalar).
__device__ __forceinline__ auto buffer(const void* p, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, (int)bytes, 0x00027000);
}
template <typename Rsrc>
__device__ __forceinline__ float bload(Rsrc r, uint32_t lane, uint32_t scalar) {
  return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, (int)lane, (int)scalar, 0));
}
template <typename Rsrc>
__device__ __forceinline__ void bstore(Rsrc r, float v, uint32_t lane, uint32_t scalar) {
  __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), r, (int)lane, (int)scalar, 0);
}

template <int NX, bool NARROW>
__global__ void __launch_bounds__(4 * NX, 4) win_solve_kernel(const WinArgs* __restrict__ descs, int ndesc) {
  constexpr int PX = NX + 1;
  constexpr int NC = NX / 16;   // 16-column chunks
  using C = C2<float>;
  extern __shared__ __align__(16) unsigned char smem[];
  const lptr<C> buf = (lptr<C>)smem;            // [64][PX]
  const lptr<C> carry = buf + kWinRows * PX;    // [2][NC][64]
  const int blk = xcd_block();
  const WinArgs& a = descs[find_desc(descs, ndesc, blk)];
  const int bid = blk - a.block0;
  const int H = a.g.H, W = a.g.W, K = a.K, R = a.R;
  const int plane = a.g.ER * a.g.EC;
  const int nwin = a.nwy * a.nwx;
  const int m = bid / nwin;
  int win = bid - m * nwin;
  // windows in bands of four window rows, walked column by column: the runs of
  // 16 consecutive workgroups that share an XCD's L2 then cover 4 x 4 windows,
  // whose halos overlap in both directions
  const int band = (int)udiv(win, a.m4x);
  win -= band * 4 * a.nwx;
  const int bh = min(4, a.nwy - 4 * band);
  const int wx = bh == 4 ? win >> 2 : bh == 3 ? win / 3 : bh == 2 ? win >> 1 : win;
  const int wy = 4 * band + win - wx * bh;
  const int y0 = udiv(wy * H, a.my), hb = udiv((wy + 1) * H, a.my) - y0;   // rows solved for
  const int x0 = udiv(wx * W, a.mx), wb = udiv((wx + 1) * W, a.mx) - x0;   // columns solved for
  const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int t = wid & 3, x = (wid >> 2) * 64 + lane;
  const int k0 = 2 * m;
  const bool has1 = k0 + 1 < K;
  // Everything that the gather and the transforms look up comes in one round
  // of vector loads: the fold entry of the lane's column, in lane q that of
  // row t + 4 q, in lane i the twiddle exp(-2 pi i i / 64) and the recursion
  // coefficients of frequency i (uniform values are read back lane by lane).
  const FoldEnt ce = ldf(glob(a.wcol) + wrap(x0 + a.offW - R + x, W, a.mW));
  const FoldEnt rl = ldf(glob(a.wrow) + wrap(y0 + a.offH - R + t + 4 * (lane & 15), H, a.mH));
  const C twl = kW64[min(lane, 49)];
  const float rho = a.rho[lane], gain = a.gain[lane], gain_lo = a.gain_lo[lane];
  auto lane_i = [](int v, int l) { return __builtin_amdgcn_readlane(v, l); };
  auto lane_f = [](float v, int l) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l)); };
  auto tw = [&](int i) { return C{lane_f(twl.x, i), lane_f(twl.y, i)}; };

  // Right-hand side: rows t + 4 q of the window, the sum of the grown-tile
  // partial sums covering each pixel.  Rows and columns past the halo are read
  // like the others (any value serves there), and without a second class the
  // first is read twice, so that the loads of the first entries need no
  // branches; second entries are read where they are.  Eight rows at a time
  // have all their loads in flight together.
  C v[16];
  {
    // buffer loads: scalar row offset + lane offset, no address arithmetic per load
    const auto acc = buffer(a.acc, a.acc_bytes);
    const uint32_t kb = 4u * (uint32_t)k0 * plane, p4 = has1 ? 4u * plane : 0u;
    auto ld = [&](uint32_t row, uint32_t col) { return C{bload(acc, kb + col, row), bload(acc, kb + p4 + col, row)}; };
    const bool c1 = ce.n > 1;
#pragma unroll
    for (int h = 0; h < 16; h += 8) {
      C vc[8], vr[8], vd[8];
      int n[8];
      uint32_t o0[8], o1[8];
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        n[q] = lane_i(rl.n, h + q);
        o0[q] = lane_i(rl.off[0], h + q);
        o1[q] = lane_i(rl.off[1], h + q);
        vc[q] = vr[q] = vd[q] = C{0.f, 0.f};
      }
#pragma unroll
      for (int q = 0; q < 8; ++q) v[h + q] = ld(o0[q], ce.off[0]);
#pragma unroll
      for (int q = 0; q < 8; ++q)
        if (n[q] > 1) vr[q] = ld(o1[q], ce.off[0]);
      if (c1) {
#pragma unroll
        for (int q = 0; q < 8; ++q) vc[q] = ld(o0[q], ce.off[1]);
#pragma unroll
        for (int q = 0; q < 8; ++q)
          if (n[q] > 1) vd[q] = ld(o1[q], ce.off[1]);
      }
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        v[h + q].x = (v[h + q].x + vr[q].x) + (vc[q].x + vd[q].x);
        v[h + q].y = (v[h + q].y + vr[q].y) + (vc[q].y + vd[q].y);
      }
    }
    // tiles narrower than the halo: the rest of the fold lists, one pair of
    // entries at a time, with the loads of all sixteen rows in flight together
    if (NARROW && __any(rl.n > 2 || ce.n > 2)) {
      int mr = rl.n, mc = ce.n;
      for (int o = 32; o > 0; o >>= 1) {
        mr = max(mr, __shfl_xor(mr, o));
        mc = max(mc, __shfl_xor(mc, o));
      }
      mr = __builtin_amdgcn_readfirstlane(mr);
      mc = __builtin_amdgcn_readfirstlane(mc);
      const gptr<const int> frow = glob(a.frow), fcol = glob(a.fcol);
      const int gx = wrap(x0 + a.offW - R + x, W, a.mW);
      const int gr = wrap(y0 + a.offH - R + t + 4 * (lane & 15), H, a.mH);
      for (int i = 0; i < mr; ++i) {
        uint32_t ro = rl.off[i < 2 ? i : 0];
        if (i >= 2 && i < rl.n) {
          const int e = frow[(size_t)(1 + i) * H + gr];
          ro = 4u * ((uint32_t)(e >> kFoldShift) * a.g.ntc * K * plane + (uint32_t)(e & kFoldMask) * a.g.EC);
        }
        for (int j = i < 2 ? 2 : 0; j < mc; ++j) {
          uint32_t co = ce.off[j < 2 ? j : 0];
          const bool in = j < ce.n;
          if (j >= 2 && in) {
            const int e = fcol[(size_t)(1 + j) * W + gx];
            co = 4u * ((uint32_t)(e >> kFoldShift) * K * plane + (uint32_t)(e & kFoldMask));
          }
          C vx[16];
#pragma unroll
          for (int q = 0; q < 16; ++q) {
            vx[q] = C{0.f, 0.f};
            if (i < lane_i(rl.n, q) && in) vx[q] = ld(lane_i(ro, q), co);
          }
#pragma unroll
          for (int q = 0; q < 16; ++q) v[q] = cadd(v[q], vx[q]);
        }
      }
    }
  }

  // DFT along the 64 rows: X[k + 8 j] = sum_s w8^(s j) w64^(s k) sum_p w8^(p k) x[s + 8 p].
  // The wavefront's rows t + 4 q are the residues s = t (q even) and t + 4 (q odd).
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int s = t + 4 * h;
    C y[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) y[i] = v[2 * i + h];
    bfly8(y, -1.f);
#pragma unroll
    for (int k = 0; k < 8; ++k) stc(buf + (8 * s + k) * PX + x, k ? twmul(y[k], tw(s * k), false) : y[k]);
  }
  __syncthreads();
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const lptr<C> col = buf + (t + 4 * h) * PX + x;
    C y[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) y[i] = ldc(col + 8 * i * PX);
    bfly8(y, -1.f);
#pragma unroll
    for (int i = 0; i < 8; ++i) stc(col + 8 * i * PX, y[i]);
  }
  __syncthreads();

  // the tridiagonal systems: frequency `lane`, columns 16 wid .. 16 wid + 15
  {
    const lptr<C> row = buf + lane * PX + 16 * wid;
    C r[16], b[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) r[i] = ldc(row + i);
    auto step = [&](C x, C y) { return C{x.x + rho * y.x, x.y + rho * y.y}; };
    // the chunk's sums from 0 at its last and first column
    C s = {0.f, 0.f}, w = {0.f, 0.f};
#pragma unroll
    for (int i = 0; i < 16; ++i) s = step(r[i], s);
#pragma unroll
    for (int i = 15; i >= 0; --i) w = step(r[i], w);
    stc(carry + wid * 64 + lane, s);
    stc(carry + (NC + wid) * 64 + lane, w);
    const float rho2 = rho * rho, rho4 = rho2 * rho2, rho8 = rho4 * rho4, pw = rho8 * rho8;
    __syncthreads();
    // the recursions again from the two chunks before (after) this one
    s = w = C{0.f, 0.f};
    if (wid > 0) s = ldc(carry + (wid - 1) * 64 + lane);
    if (wid > 1) {
      const C s2 = ldc(carry + (wid - 2) * 64 + lane);
      s = C{s.x + pw * s2.x, s.y + pw * s2.y};
    }
    if (wid < NC - 1) w = ldc(carry + (NC + wid + 1) * 64 + lane);
    if (wid < NC - 2) {
      const C w2 = ldc(carry + (NC + wid + 2) * 64 + lane);
      w = C{w.x + pw * w2.x, w.y + pw * w2.y};
    }
#pragma unroll
    for (int i = 15; i >= 0; --i) {
      b[i] = w;   // sum_(d > 0) rho^(d - 1) r[i + d]
      w = step(r[i], w);
    }
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      s = step(r[i], s);
      const C t = step(s, b[i]);
      stc(row + i, C{gain * t.x + gain_lo * t.x, gain * t.y + gain_lo * t.y});
    }
  }
  __syncthreads();

  // inverse DFT along the rows
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int k = t + 4 * h;
    const lptr<C> col = buf + k * PX + x;
    C y[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) y[i] = ldc(col + 8 * i * PX);
    bfly8(y, 1.f);
#pragma unroll
    for (int i = 0; i < 8; ++i) stc(col + 8 * i * PX, i ? twmul(y[i], tw(i * k), true) : y[i]);
  }
  __syncthreads();
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    C y[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) y[k] = ldc(buf + (8 * (t + 4 * h) + k) * PX + x);
    bfly8(y, 1.f);
#pragma unroll
    for (int i = 0; i < 8; ++i) v[2 * i + h] = y[i];
  }
  if (x >= R && x < R + wb) {
    const uint32_t hw = 4u * (uint32_t)(H * W);
    const auto z = buffer(a.z + (size_t)k0 * H * W, has1 ? 2 * hw : hw);
    const uint32_t col = 4u * (uint32_t)(x0 + x - R);
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      const int r = t + 4 * q - R;
      if (r >= 0 && r < hb) {
        const uint32_t row = 4u * (uint32_t)((y0 + r) * W);
        bstore(z, v[q].x, col, row);
        if (has1) bstore(z, v[q].y, col + hw, row);
      }
    }
  }
}

template <int NX, bool NARROW>
static hipError_t launch_win_t(const WinArgs* d, int n, int blocks, hipStream_t st) {
  static bool lds_set = false;  // idempotent, so a racing second call is harmless
  if (!lds_set) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(win_solve_kernel<NX, NARROW>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, kLdsMax);
    if (e != hipSuccess) return e;
    lds_set = true;
  }
  hipLaunchKernelGGL((win_solve_kernel<NX, NARROW>), dim3(blocks), dim3(4 * NX), win_lds(NX), st, d, n);
  return hipGetLastError();
}

hipError_t launch_win(const WinArgs* d, int n, int blocks, int nx, bool narrow, hipStream_t st) {
  if (nx == 64) return narrow ? launch_win_t<64, true>(d, n, blocks, st) : launch_win_t<64, false>(d, n, blocks, st);
  if (nx == 128) return narrow ? launch_win_t<128, true>(d, n, blocks, st) : launch_win_t<128, false>(d, n, blocks, st);
  return hipErrorInvalidValue;
}

}  // namespace segsalsa
