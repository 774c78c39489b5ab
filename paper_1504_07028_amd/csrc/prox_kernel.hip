// Fused per-pixel proximity kernel of one SALSA round (SegSALSA-STR, Sec. 4).
//
// One workgroup owns one tile of the image.  Wavefront w handles classes
// k = w, w + nw, ... for 64 pixels at a time (one pixel per lane).  Per pixel
// and round it computes, from z and the scaled multipliers d:
//   g1 (data term, eq. (10)):   u1 = prox_{g1/mu}(z - d1): closed-form root
//                               of mu t^2 - mu (p^T v) t - ||p||^2 = 0
//   g2 (Schatten prior):        u2 = prox_{(lambda/mu)||.||_{S_p}}(J z - d2),
//                               reduced to the 2x2 structure tensor (eq. (5))
//   g3 (positivity):            u3 = max(z - d3, 0)
//   g4 (sum to one):            u4 = (z - d4) - (1^T (z - d4) - 1) / K, or, with
//                               g4s, the projection of z - d4 onto the probability
//                               simplex: u4 = max(v4 - theta, 0) with 1^T u4 = 1
// the multiplier update d_j <- u_j - (H_j z - d_j) (eq. (14)), and scatters
// u_j + d_j through H_j^T into a per-tile accumulator: the right-hand side
// G^T (u + d) of the normal equations of the z-update (eq. (12)).
//
// The J^T scatter of a pixel reaches pixels up to (M, M+1) away, so every
// tile accumulates over its tile grown by that margin in LDS; the row FFT
// pass sums the overlapping grown tiles.  A class's accumulator is written by
// one wavefront only and, within one instruction, lanes hit distinct
// addresses, so plain LDS read-modify-writes (in program order) are free of
// races and their summation order is fixed.
#include "segsalsa_internal.h"
#include "segsalsa_kernels.h"
#include "prox_math.h"

namespace segsalsa {

// VAR (ProxVariant bits) compiles in the primal-residual accumulation of
// checked rounds and the method's variants (simplex g4, general Schatten p with
// either g4); the plain instantiation (p in {1, 2, inf}, affine g4, no
// residuals) stays lean.  One build for all of them keeps the residual's sum
// and the Newton solve's temporaries next to the class block for everyone
// (FP64 3x3, one class per wavefront: 60 spilled registers; 0 with the
// residuals or the simplex alone, 1 with both, 45 with the Newton solve).
// us per round in one build -> here, FP64: 145x145 K = 16 5x5, simplex 127 ->
// 111, p = 3 147 -> 141, residuals 185 -> 177; 209x795 K = 9 3x3, simplex 267
// -> 206, p = 3 415 -> 390, residuals 314 -> 257, simplex with residuals 341 ->
// 278.
//
// PF (prefetch): the loads of step s + 1 (p_hat, d3 and the raw d2
// pairs of the wavefront's classes) are issued into a second register set at
// the start of step s's multiplier/scatter phase, so that they stream while
// that phase computes and stores.  All wavefronts of a workgroup run each
// step's phases in lockstep (three barriers per step), and without it the
// loads of a step only start once the previous step's work is done, so the
// memory and the arithmetic of a step never overlap.  It doubles the per-lane
// state, hence fewer (and fuller) wavefronts.
//
// SY (streamed Y, patches of 9x9 and larger): the 2L values of Y = J z - d2
// of a pixel and class are not kept in registers between the structure-tensor
// sums and the update; the update phase rebuilds each offset's pair from z in
// LDS and the old d2 (read again, just before its new value overwrites it).
// The registers then do not grow with L, so these patches keep the wavefront
// count and the ordered FP32 scatter of the smaller ones, at the price of a
// second read of d2 (mostly served by the caches).  Both phases load the pairs
// NA offsets ahead: in the update the compiler has to leave a load behind the
// stores before it (for all it knows they may meet), and in the sums it
// overlaps as many as the registers of the occupancy that it aims at allow, so
// that each offset waited for most of a memory latency.  us per round without
// -> with: FP32 145x145 K = 16 9x9 162 -> 137, 507x716 K = 9 11x11 3098 ->
// 1680, FP64 65x102 K = 13 11x11 139 -> 124; over 115 shapes and options 0.72
// times the time.  Twice the distance gains nothing more (0.72) and spills in
// FP64.
//
// d1 and d4 are not stored per class: after a round d1 = p_hat * gain with the
// pixel's FP64 gain, and with the affine g4 all classes share one d4, so the
// round keeps those two per pixel (px) and forms d1 again exactly as it was
// rounded.  That is 4 words of the 4L + 9 per pixel and class that the kernel
// would otherwise stream; 2048x2048 K = 16 5x5 FP32, bound by the HBM, 5478 ->
// 5152 us per launch (28.6 GB, 5.55 TB/s), 145x145 32.8 -> 31 us.  States with other d1 and d4 (imported ones, and the
// d4 of the simplex g4) are per class in dfull; `form` says which.
//
// NT (streaming, plain instantiation only): p_hat, d3 and d2 are
// loaded and stored nontemporally, and so are the grown-tile partial sums
// written at the end (measured: the fold that reads them next runs as fast or
// faster).  A round touches the state once, so when the state of all images
// of a launch far exceeds the L2s and the 256 MB MALL, caching it only evicts
// what the next kernels read again (z, the spectrum); when it fits, the
// cached accesses keep it resident from round to round.  The host chooses per
// round from the state's size.
template <typename T, int M, int KPW, int VAR, bool PF, bool NT>
__global__ void __launch_bounds__((prox_max_threads<T, M, KPW, PF>()), (prox_min_waves<T, M, KPW, VAR, PF>()))
prox_rhs_kernel(const ProxArgs<T>* __restrict__ descs, int ndesc, bool first) {
  constexpr int D = 2 * M + 1;
  constexpr int L = D * D;
  constexpr bool SY = prox_streams_y<M>();
  constexpr int NA = sizeof(T) == 4 ? 4 : 2;   // offsets that SY loads ahead
  constexpr int LY = SY ? 1 : L;
  const int blk = xcd_block();   // neighbouring tiles (shared halo rows) on one XCD
  const ProxArgs<T>& a = descs[find_desc(descs, ndesc, blk)];
  const TileGeom& g = a.g;
  const int tile = blk - a.block0;
  const int tr = tile / g.ntc;
  const int tc = tile - tr * g.ntc;
  const int r0 = g.r0(tr), c0 = g.c0(tc);
  const int th = g.th(tr), tw = g.tw(tc);
  const int ER = th + 2 * M + 1, EC = tw + 2 * M + 1;
  const int plane = ER * EC;
  const int K = a.K, nw = a.nw;
  const int wid = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int H = g.H, W = g.W;
  constexpr bool GEN = (VAR & kProxGeneralP) != 0, want_res = (VAR & kProxResiduals) != 0;
  const bool g4s = (VAR & kProxSimplex) != 0 || (GEN && a.g4s);
  const gptr<const T> gz = glob(a.z);
  const gptr<const T> gphat = glob(a.phat);
  const gptr<const T> gd3_in = glob(a.d3_in);
  const gptr<const char> gpx_in = glob(a.px_in);
  const size_t pxs = a.px_stride;
  const int form = first ? *glob(a.form_in) : a.form;
  const gptr<const T> gd2_in = glob(a.d2_in);   // (h, v) pairs
  const gptr<T> gd3 = glob(a.d3);
  const gptr<char> gpx = glob(a.px);
  const gptr<T> gd2 = glob(a.d2);
  // NT: the per-pixel state streams past the caches (nontemporal loads and
  // stores), for rounds whose state is far larger than the caches
  auto sld = [](gptr<const T> p) -> T {
    if constexpr (NT) return __builtin_nontemporal_load(p);
    else return *p;
  };
  auto sst = [](gptr<T> p, T v) {
    if constexpr (NT) __builtin_nontemporal_store(v, p);
    else *p = v;
  };

  extern __shared__ __align__(16) unsigned char smem[];
  T* zt = reinterpret_cast<T*>(smem);  // [K][ER][EC] z over the grown tile (periodic)
  T* acc = zt + K * plane;             // [K][ER][EC] G^T(u + d) partial sums
  // [6][ns][64] sums of a step, per class, or per wavefront where classes
  // would take too much LDS (prox_slots), 16-byte aligned (also read as
  // doubles); with g4s also v4 of every class, [K][64]: the classes' slots of
  // its sum, or after the FP64 sums and coefficients where the slots are the
  // wavefronts'.  (A step's are read before its last barrier, the next step's
  // written after.)
  const int ns = prox_slots(K, nw);
  // (offsets from smem, not integer casts of pointers: the compiler then keeps
  // these accesses as LDS instructions instead of generic FLAT ones, which
  // would also wait for outstanding global memory operations)
  T* part = reinterpret_cast<T*>(smem + (((size_t)2 * K * plane * sizeof(T) + 15) & ~size_t(15)));
  // [6][64] FP64 per-pixel class sums and [5][64] FP64 per-pixel coefficients
  double* tot = reinterpret_cast<double*>(part + 6 * ns * 64);
  double* coef = tot + 6 * 64;
  T* v4buf = ns == K ? part + 2 * ns * 64 : reinterpret_cast<T*>(coef + 5 * 64);

  const int P = th * tw;
  const int nsteps = (P + 63) >> 6;
  double rp_acc = 0.0;
  // Inputs of one step: p_hat, d3 and the raw d2 pairs (turned into Y in place)
  // of the wavefront's classes, and the pixel's gain and d4 (every wavefront
  // reads these: cached loads).  The first step's are issued before z is
  // staged, so that their latency passes under the staging.  (FP64
  // 7x7 with four classes, whose block of 3136 bytes is several times the
  // registers, reads each class's where they are used: raw values that spill
  // are moved twice, 376 -> 1834 spills and 129 -> 147 us per round at 60x61,
  // K = 11.  Blocks up to 1600 bytes gain: FP64 300x301 7x7 292 -> 272 us.  Nor
  // does it pay next to the Newton solve in FP64 with two classes of a 3x3 patch
  // on a wavefront, 139 -> 95 spills without: p = 3, 287x317 K = 24 450 -> 440;
  // with one class, or 5x5 patches, it does: 476x188 K = 13 265 -> 246.)
  constexpr bool EARLY = !PF && !(GEN && sizeof(T) == 8 && M == 1 && KPW == 2) && KPW * LY * 2 * (int)sizeof(T) <= 1600;
  T Y[KPW][LY][2];
  T pk[KPW], r3[KPW];
  double gain_in = 0.0;
  T d4_in = T(0);
  auto load = [&](int s) {
    if ((s << 6) + lane >= P) return;
    const size_t step = (size_t)tile * g.steps + s;
#pragma unroll
    for (int kk = 0; EARLY && kk < KPW; ++kk) {
      const int k = wid + kk * nw;
      if (k < K) {
        const size_t kb = step * K + k;
        pk[kk] = sld(gphat + kb * 64 + lane);
        r3[kk] = sld(gd3_in + kb * 64 + lane);
        if constexpr (!SY) {
          const gptr<const T> d2p = gd2_in + 2 * (kb * (size_t)(L * 64) + lane);
#pragma unroll
          for (int j = 0; j < L; ++j) {
            Y[kk][j][0] = sld(d2p + j * 128);
            Y[kk][j][1] = sld(d2p + j * 128 + 1);
          }
        }
      }
    }
    gain_in = ((gptr<const double>)(gpx_in + step * pxs))[lane];
    d4_in = ((gptr<const T>)(gpx_in + step * pxs + 512))[lane];
  };
  // prefetched inputs of the next step (PF)
  constexpr int KP = PF ? KPW : 1, LP = PF ? L : 1;
  T Pp[KP], P3[KP], Pd[KP][LP][2];
  // class kk's inputs of step sn (one class at a time, so that in the update
  // phase the next step's block of a class only becomes live as the current
  // step's block of the class before it dies)
  auto prefetch = [&](int sn, int kk) {
    const bool vn = (sn << 6) + lane < P;
    const int k = wid + kk * nw;
    if (k < K && vn) {
      const size_t kb = ((size_t)tile * g.steps + sn) * K + k;
      Pp[kk] = gphat[kb * 64 + lane];
      P3[kk] = gd3_in[kb * 64 + lane];
      const gptr<const T> d2p = gd2_in + 2 * (kb * (size_t)(L * 64) + lane);
#pragma unroll
      for (int j = 0; j < LP; ++j) {
        Pd[kk][j][0] = d2p[j * 128];
        Pd[kk][j][1] = d2p[j * 128 + 1];
      }
    }
  };
  if constexpr (PF) {
#pragma unroll
    for (int kk = 0; kk < KP; ++kk) prefetch(0, kk);
  } else if constexpr (EARLY) {
    load(0);
  }
  const FastDiv fER = FastDiv::uniform(ER), ftw = FastDiv::uniform(tw);
  // z over the grown tile: rows (class, grown row) of EC columns, as many rows
  // side by side in a wavefront as fit its lanes, four of them per lane in flight
  tile_rows<4>(K * ER, EC, nw, [&](int row, int ec) {
    const int k = (int)fER.div(row), er = row - k * ER;
    return gz[(k * H + wrap_near(r0 - M + er, H)) * W + wrap_near(c0 - M + ec, W)];
  }, [&](int row, int ec, T v) {
    zt[row * EC + ec] = v;
    acc[row * EC + ec] = T(0);
  });
  __syncthreads();
  for (int s = 0; s < nsteps; ++s) {
    const int f = (s << 6) + lane;
    const bool valid = f < P;
    const int lr = valid ? (int)ftw.div(f) : 0;
    const int lc = valid ? f - lr * tw : 0;
    const size_t step = (size_t)tile * g.steps + s;
    const size_t stepbase = step * K;
    if (!EARLY) {
      if (valid) {
        gain_in = ((gptr<const double>)(gpx_in + step * pxs))[lane];
        d4_in = ((gptr<const T>)(gpx_in + step * pxs + 512))[lane];
      }
    } else if (s > 0) {
      load(s);
    }

    T v1[KPW], v3[KPW], v4[KPW];
#pragma unroll
    for (int kk = 0; kk < KPW; ++kk) {
      const int k = wid + kk * nw;
      if constexpr (!EARLY) pk[kk] = T(0);
      v1[kk] = v3[kk] = v4[kk] = T(0);
      if (k < K && valid) {
        const size_t kb = stepbase + k;
        if constexpr (PF) {
          pk[kk] = Pp[kk];
          r3[kk] = P3[kk];
        } else if constexpr (!EARLY) {
          pk[kk] = sld(gphat + kb * 64 + lane);
          r3[kk] = sld(gd3_in + kb * 64 + lane);
        }
        const T d3 = r3[kk];
        // d1 and d4 as the previous round formed them, or (form) per class
        T d1 = T((double)pk[kk] * gain_in), d4 = d4_in;
        // (indexed from kb, whose registers are there: four VGPRs less than from the step)
        if (form & kFormD1) d1 = glob(a.dfull)[(kb + stepbase) * 64 + lane];
        if (form & kFormD4) d4 = glob(a.dfull)[(kb + stepbase + K) * 64 + lane];
        const T* zk = zt + k * plane + (lr + M) * EC + (lc + M);
        const T zc = zk[0];
        v1[kk] = zc - d1;
        v3[kk] = zc - d3;
        v4[kk] = zc - d4;
        T pa = T(0), pb = T(0), pc = T(0);
        if (g4s && ns != K) v4buf[k * 64 + lane] = v4[kk];
        [[maybe_unused]] const gptr<const T> d2p = gd2_in + 2 * (kb * (size_t)(L * 64) + lane);
        [[maybe_unused]] C2<T> ahead[NA];
#pragma unroll
        for (int j = 0; SY && j < NA; ++j) ahead[j] = C2<T>{d2p[j * 128], d2p[j * 128 + 1]};
#pragma unroll
        for (int j = 0; j < L; ++j) {
          const int dy = j / D - M, dx = j % D - M;
          const T* zr = zk + dy * EC + dx;
          const T z00 = zr[0], z01 = zr[1], z10 = zr[EC];
          C2<T> dd;
          if constexpr (PF) {
            dd.x = Pd[kk][j < LP ? j : 0][0];
            dd.y = Pd[kk][j < LP ? j : 0][1];
          } else if constexpr (SY) {   // (read again in the update: cached)
            dd = ahead[j % NA];
            if (j + NA < L) ahead[j % NA] = C2<T>{d2p[(j + NA) * 128], d2p[(j + NA) * 128 + 1]};
          } else if constexpr (!EARLY) {
            dd.x = sld(d2p + j * 128);
            dd.y = sld(d2p + j * 128 + 1);
          } else {
            dd.x = Y[kk][j][0];
            dd.y = Y[kk][j][1];
          }
          const T yh = a.c[j] * (z01 - z00) - dd.x;
          const T yv = a.c[j] * (z10 - z00) - dd.y;
          if constexpr (!SY) {
            Y[kk][j][0] = yh;
            Y[kk][j][1] = yv;
          }
          pa += yh * yh;
          pb += yh * yv;
          pc += yv * yv;
        }
        // the class's terms of the pixel's six sums over the classes
        T six[6] = {pk[kk] * v1[kk], pk[kk] * pk[kk], v4[kk], pa, pb, pc};
        T* sl = part + (ns == K ? k : wid) * 64 + lane;
        if (kk > 0 && ns != K) {
#pragma unroll
          for (int q = 0; q < 6; ++q) six[q] = sl[q * ns * 64] + six[q];
        }
#pragma unroll
        for (int q = 0; q < 6; ++q) sl[q * ns * 64] = six[q];
      }
    }
    // Per-pixel sums over the classes and the per-pixel coefficients, each
    // computed once per step: waves q < 6 reduce the q-th sum over the
    // classes in FP64 (class by class up to 16 of them, so that the sums do not
    // depend on whether a wavefront holds one or two), then waves 0 and 1 evaluate the two
    // FP64 closed forms and share them through LDS (the other wavefronts would
    // only repeat them).
    __syncthreads();
#pragma unroll 1
    for (int q = wid; q < 6; q += nw) {
      double t = 0.0;  // fixed order; unrolled so the LDS reads overlap
#pragma unroll 4
      for (int w = 0; w < ns; ++w) t += (double)part[(q * ns + w) * 64 + lane];
      tot[q * 64 + lane] = t;
    }
    __syncthreads();
    // the two FP64 closed forms on two different wavefronts (each keeps its
    // own class block live, so splitting them keeps the register peak down)
    const int wn = nw > 1 ? 1 : 0;
    if (wid == 0 && valid) {
      const double S = tot[0 * 64 + lane], Q = tot[1 * 64 + lane], SV = tot[2 * 64 + lane];
      double g4c = -(SV - 1.0) / (double)K;  // affine g4: the shared d4 of the pixel
      if (g4s) {
        // simplex g4: threshold theta with sum_k max(v4_k - theta, 0) = 1, by
        // Michelot's active-set iteration (theta rises, the active set
        // shrinks, at most K passes over the pixel's K values)
        const T* vb = v4buf + lane;
        double theta = (SV - 1.0) / (double)K;
        int cnt = K;
        for (int it = 0; it < K; ++it) {
          double sum = 0.0;
          int c2 = 0;
          for (int k = 0; k < K; ++k) {
            const double v = (double)vb[k * 64];
            if (v > theta) {
              sum += v;
              ++c2;
            }
          }
          if (c2 == cnt || c2 == 0) break;
          cnt = c2;
          theta = (sum - 1.0) / (double)c2;
        }
        g4c = theta;
      }
      const double gain = data_prox_gain(S, Q, a.mu);
      coef[0 * 64 + lane] = gain;
      coef[1 * 64 + lane] = g4c;
      ((gptr<double>)(gpx + step * pxs))[lane] = gain;
      if (!g4s) ((gptr<T>)(gpx + step * pxs + 512))[lane] = T(g4c);
    }
    if (wid == wn && valid) {
      const double A = tot[3 * 64 + lane], B = tot[4 * 64 + lane], C = tot[5 * 64 + lane];
      double n11, n12, n22;
      schatten_multiplier<GEN>(A, B, C, a.tau, a.pkind, a.pval, n11, n12, n22);
      coef[2 * 64 + lane] = n11 - 1.0;
      coef[3 * 64 + lane] = n12;
      coef[4 * 64 + lane] = n22 - 1.0;
    }
    __syncthreads();
    // (with PF, the next step's loads are issued class by class below: a step
    // other than the last has all its lanes valid, so they are issued by every lane)
    if (valid) {
    const double gain = coef[0 * 64 + lane];
    const double g4c = coef[1 * 64 + lane];
    const T d4a = T(g4c);
    const double theta = g4c;
    const T m11 = T(coef[2 * 64 + lane]), m12 = T(coef[3 * 64 + lane]), m22 = T(coef[4 * 64 + lane]);

#pragma unroll
    for (int kk = 0; kk < KPW; ++kk) {
      const int k = wid + kk * nw;
      if constexpr (PF) {
        if (s + 1 < nsteps) prefetch(s + 1, kk);   // streams while this class's updates compute and store
      }
      if (k < K) {
        const size_t kb = stepbase + k;
        const T d1n = T((double)pk[kk] * gain);
        const T d3n = v3[kk] < T(0) ? -v3[kk] : T(0);
        const T d4n = g4s ? T(fmax((double)v4[kk] - theta, 0.0) - (double)v4[kk]) : d4a;
        const T own = (v1[kk] + T(2) * d1n) + (v3[kk] < T(0) ? -v3[kk] : v3[kk]) + (v4[kk] + T(2) * d4n);
        sst(gd3 + kb * 64 + lane, d3n);
        if (g4s) glob(a.dfull)[(kb + stepbase + K) * 64 + lane] = d4n;
        if (want_res) {  // primal residual: d_new - d_old = u - H z (eq. (14))
          const T zc = zt[k * plane + (lr + M) * EC + (lc + M)];
          const double e1 = (double)d1n - (double)(zc - v1[kk]);
          const double e3 = (double)d3n - (double)(zc - v3[kk]);
          const double e4 = (double)d4n - (double)(zc - v4[kk]);
          rp_acc += e1 * e1 + e3 * e3 + e4 * e4;
        }
        const gptr<T> d2o = gd2 + 2 * (kb * (size_t)(L * 64) + lane);
        // SY: the old d2 and z of this pixel and class, to rebuild Y offset by offset
        [[maybe_unused]] const gptr<const T> d2i = gd2_in + 2 * (kb * (size_t)(L * 64) + lane);
        [[maybe_unused]] const T* zk0 = zt + k * plane + (lr + M) * EC + (lc + M);
        [[maybe_unused]] C2<T> ahead[NA];
#pragma unroll
        for (int j = 0; SY && j < NA; ++j) ahead[j] = C2<T>{d2i[j * 128], d2i[j * 128 + 1]};
        // New d2 = u2 - Y = Y (N - I) and the J^T scatter of c_j (u2 + d2).
        // The h part of offset (dy, dx) lands at (dy, dx + 1) with + and at
        // (dy, dx) with -, the v part at (dy + 1, dx) with + and at (dy, dx)
        // with -.  Walking the destinations (da, db) in row-major order, each
        // one sums its (up to three) terms in registers: the h part of the
        // previous column and the v part of the previous row are carried.
        // Neighbouring lanes reach the same address through different
        // offsets, so the read-modify-writes stay in program order: volatile
        // keeps the compiler from hoisting a later read above an earlier
        // write (LDS executes one wavefront's accesses in order).
        T* ak = acc + k * plane + (lr + M) * EC + (lc + M);
        T vprev[D + 1];
#pragma unroll
        for (int q = 0; q <= D; ++q) vprev[q] = T(0);
#pragma unroll
        for (int da = -M; da <= M + 1; ++da) {
          T hprev = T(0);
#pragma unroll
          for (int db = -M; db <= M + 1; ++db) {
            const bool in0 = da <= M && db <= M;
            T ah = T(0), av = T(0);
            if (in0) {
              const int jj = (da + M) * D + (db + M);
              T yh, yv;
              if constexpr (SY) {   // Y of this offset again, from z in LDS and the old d2
                const T* zr = zk0 + da * EC + db;
                const C2<T> dd = ahead[jj % NA];
                if (jj + NA < L) ahead[jj % NA] = C2<T>{d2i[(jj + NA) * 128], d2i[(jj + NA) * 128 + 1]};
                yh = a.c[jj] * (zr[1] - zr[0]) - dd.x;
                yv = a.c[jj] * (zr[EC] - zr[0]) - dd.y;
              } else {
                yh = Y[kk][jj][0];
                yv = Y[kk][jj][1];
              }
              const T nh = yh * m11 + yv * m12;
              const T nv = yh * m12 + yv * m22;
              C2<T> o;
              o.x = nh;
              o.y = nv;
              sst(d2o + jj * 128, o.x);
              sst(d2o + jj * 128 + 1, o.y);
              if (want_res) {  // old d2 = c_j grad z - Y, rebuilt from the LDS tile
                const T* zr = zt + k * plane + (lr + M + da) * EC + (lc + M + db);
                const double oh = (double)(a.c[jj] * (zr[1] - zr[0]) - yh);
                const double ov = (double)(a.c[jj] * (zr[EC] - zr[0]) - yv);
                rp_acc += ((double)nh - oh) * ((double)nh - oh) + ((double)nv - ov) * ((double)nv - ov);
              }
              ah = a.c[jj] * (T(2) * nh + yh);
              av = a.c[jj] * (T(2) * nv + yv);
            }
            const bool inh = da <= M && db - 1 >= -M;
            const bool inv = da - 1 >= -M && db <= M;
            const bool own_here = da == 0 && db == 0;
            const int q = db + M;
            if (in0 || inh || inv || own_here) {
              T gsum = own_here ? own : T(0);
              if (in0) gsum -= ah + av;
              if (inh) gsum += hprev;
              if (inv) gsum += vprev[q];
              if constexpr (sizeof(T) == 4 && (M <= 3 || SY)) {
                volatile __attribute__((address_space(3))) T* at =
                    (volatile __attribute__((address_space(3))) T*)(ak + da * EC + db);
                *at = *at + gsum;
              } else {
                // FP64: the LDS atomic add is fast and keeps register pressure down.
                atomicAdd(ak + da * EC + db, gsum);
              }
            }
            hprev = ah;
            if (q <= D) vprev[q] = av;
          }
        }
      }
    }
    }  // valid
  }
  __syncthreads();
  if (want_res) {  // fixed-order reduction of the tile's primal-residual partial sums
    double v = rp_acc;
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    double* red = reinterpret_cast<double*>(part);
    if (lane == 0) red[wid] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
      double t = 0.0;
      for (int w = 0; w < nw; ++w) t += red[w];
      glob(a.res_tile)[tile] = t;
    }
  }
  const gptr<T> out = glob(a.acc) + (size_t)tile * K * g.ER * g.EC;
  tile_rows<4>(K * ER, EC, nw, [&](int row, int ec) { return acc[row * EC + ec]; }, [&](int row, int ec, T v) {
    const int k = (int)fER.div(row);
    sst(out + (k * g.ER + (row - k * ER)) * g.EC + ec, v);
  });
}

template <typename T, int M, int KPW, int VAR, bool PF, bool NT = false>
static hipError_t launch_prox_t(const ProxArgs<T>* descs, int ndesc, int blocks, int threads, size_t lds,
                                bool first, hipStream_t st) {
  auto fn = prox_rhs_kernel<T, M, KPW, VAR, PF, NT>;
  static bool lds_set = false;  // idempotent, so a racing second call is harmless
  if (!lds_set) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(fn),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, kLdsMax);
    if (e != hipSuccess) return e;
    lds_set = true;
  }
  hipLaunchKernelGGL(fn, dim3(blocks), dim3(threads), lds, st, descs, ndesc, first);
  return hipGetLastError();
}

template <typename T, int M, int VAR>
static hipError_t launch_prox_m(const ProxArgs<T>* d, int n, int blocks, int threads, int kpw, bool pf, bool nt,
                                size_t lds, bool first, hipStream_t st) {
  if (pf) {   // built for the plain FP32 kernel with two classes per wavefront and M <= 2 only
    if constexpr (prox_has_prefetch<T, M, 2, VAR>()) {
      if (kpw == 2) return launch_prox_t<T, M, 2, VAR, true>(d, n, blocks, threads, lds, first, st);
    }
    return hipErrorInvalidValue;
  }
  if constexpr (VAR == 0) {   // the streaming build: plain instantiation only
    if (nt) {
      switch (kpw) {
        case 1: return launch_prox_t<T, M, 1, 0, false, true>(d, n, blocks, threads, lds, first, st);
        case 2: return launch_prox_t<T, M, 2, 0, false, true>(d, n, blocks, threads, lds, first, st);
        case 4: return launch_prox_t<T, M, 4, 0, false, true>(d, n, blocks, threads, lds, first, st);
        default: return hipErrorInvalidValue;
      }
    }
  }
  switch (kpw) {
    case 1: return launch_prox_t<T, M, 1, VAR, false>(d, n, blocks, threads, lds, first, st);
    case 2: return launch_prox_t<T, M, 2, VAR, false>(d, n, blocks, threads, lds, first, st);
    case 4: return launch_prox_t<T, M, 4, VAR, false>(d, n, blocks, threads, lds, first, st);
    default: return hipErrorInvalidValue;
  }
}

template <typename T, int VAR>
hipError_t launch_prox_v(const ProxArgs<T>* d, int n, int blocks, int threads, int M, int kpw, bool pf,
                                bool nt, size_t lds, bool first, hipStream_t st) {
  switch (M) {
    case 0: return launch_prox_m<T, 0, VAR>(d, n, blocks, threads, kpw, pf, nt, lds, first, st);
    case 1: return launch_prox_m<T, 1, VAR>(d, n, blocks, threads, kpw, pf, nt, lds, first, st);
    case 2: return launch_prox_m<T, 2, VAR>(d, n, blocks, threads, kpw, pf, nt, lds, first, st);
    case 3: return launch_prox_m<T, 3, VAR>(d, n, blocks, threads, kpw, pf, nt, lds, first, st);
    case 4: return launch_prox_m<T, 4, VAR>(d, n, blocks, threads, kpw, pf, nt, lds, first, st);
    case 5: return launch_prox_m<T, 5, VAR>(d, n, blocks, threads, kpw, pf, nt, lds, first, st);
    default: return hipErrorInvalidValue;
  }
}

// The whole file, or (SEGSALSA_PROX_BITS, SEGSALSA_PROX_PART) one precision's
// builds PART and PART + 1, part 0 with the choice among all: they compile side
// by side.
#ifdef SEGSALSA_PROX_PART
#if SEGSALSA_PROX_BITS == 32
using PartT = float;
#else
using PartT = double;
#endif
#define SEGSALSA_PROX_BUILD(VAR)                                                                                     \
  template hipError_t launch_prox_v<PartT, VAR>(const ProxArgs<PartT>*, int, int, int, int, int, bool, bool, size_t, \
                                                bool, hipStream_t)
SEGSALSA_PROX_BUILD(SEGSALSA_PROX_PART);
SEGSALSA_PROX_BUILD(SEGSALSA_PROX_PART + 1);
#if SEGSALSA_PROX_PART == 0
extern SEGSALSA_PROX_BUILD(2);
extern SEGSALSA_PROX_BUILD(3);
extern SEGSALSA_PROX_BUILD(4);
extern SEGSALSA_PROX_BUILD(5);
#endif
#endif

#if !defined(SEGSALSA_PROX_PART) || SEGSALSA_PROX_PART == 0
template <typename T>
static hipError_t launch_prox_any(const ProxArgs<T>* d, int n, int blocks, int threads, int M, int kpw, bool pf, bool nt,
                                  size_t lds, int variant, bool first, hipStream_t st) {
  switch (variant) {
    case 0: return launch_prox_v<T, 0>(d, n, blocks, threads, M, kpw, pf, nt, lds, first, st);
    case 1: return launch_prox_v<T, 1>(d, n, blocks, threads, M, kpw, pf, nt, lds, first, st);
    case 2: return launch_prox_v<T, 2>(d, n, blocks, threads, M, kpw, pf, nt, lds, first, st);
    case 3: return launch_prox_v<T, 3>(d, n, blocks, threads, M, kpw, pf, nt, lds, first, st);
    case 4: return launch_prox_v<T, 4>(d, n, blocks, threads, M, kpw, pf, nt, lds, first, st);
    case 5: return launch_prox_v<T, 5>(d, n, blocks, threads, M, kpw, pf, nt, lds, first, st);
    default: return hipErrorInvalidValue;
  }
}
#if !defined(SEGSALSA_PROX_BITS) || SEGSALSA_PROX_BITS == 32
hipError_t launch_prox(const ProxArgs<float>* d, int n, int blocks, int threads, int M, int kpw, bool pf, bool nt,
                       size_t lds, int variant, bool first, hipStream_t st) {
  return launch_prox_any(d, n, blocks, threads, M, kpw, pf, nt, lds, variant, first, st);
}
#endif
#if !defined(SEGSALSA_PROX_BITS) || SEGSALSA_PROX_BITS == 64
hipError_t launch_prox(const ProxArgs<double>* d, int n, int blocks, int threads, int M, int kpw, bool pf, bool nt,
                       size_t lds, int variant, bool first, hipStream_t st) {
  return launch_prox_any(d, n, blocks, threads, M, kpw, pf, nt, lds, variant, first, st);
}
#endif
#endif

}  // namespace segsalsa
