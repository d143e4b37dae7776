// Hyperuniformity diagnostics (Sec. II.A): the local variance of Eq. (1) over a spherical window,
// in its Fourier form
//   sigma^2(R) = sum_{m != 0} |X(m)|^2 / N^2 W(|k_m| R)^2,   W = 2 J_1(u)/u (2D), 3 (sin u - u cos u)/u^3 (3D),
// evaluated on the half spectrum with the multiplicities w_m in the axis-0 pass (the last forward
// axis, after the same row and y passes as the power spectrum), and the host-side exponent fit
// and class table.
#include <cmath>

#include "hu_common.hpp"

namespace hu {

// words per column of the power values in LDS: the lanes of a half wave (C columns of 32 / C modes)
// on distinct banks
template <int L>
struct WvarLds {
  static constexpr int C = ColTile<L, 0>::C;
  static constexpr int PS = (L + 31) / 32 * 32 + (C >= 32 ? 1 : C >= 16 ? 2 : C >= 8 ? 4 : 8);
};

// W^2 at u = |k| R in FP32.
// 2D: J_1 by the polynomial approximations of Abramowitz & Stegun (Handbook of Mathematical
// Functions, 9.4.4 for u <= 3: J_1(u)/u as a polynomial in (u/3)^2, |error| < 1.3e-8; 9.4.6 for
// u > 3: J_1(u) = u^(-1/2) f_1 cos(theta_1), f_1 and theta_1 - u polynomials in 3/u, absolute error
// of J_1 below 1e-7), so W = 2 J_1(u) / u costs a few fused multiply-adds and three hardware
// transcendentals.
// 3D: below u = 1 the closed form loses digits to cancellation, so the Taylor series
// 3 sum_{n>=1} (-1)^(n+1) 2n u^(2n-2) / (2n+1)! (through u^10; the next term is below 3.3e-11 at
// u = 1) is used there; above, the closed form with the hardware sine and cosine.
template <int NDIM>
__device__ __forceinline__ float window_w2(float u) {
  float w;
  if constexpr (NDIM == 2) {
    if (u <= 3.0f) {
      const float t = (u * (1.0f / 3.0f)) * (u * (1.0f / 3.0f));
      w = 2.0f * (0.5f + t * (-0.56249985f + t * (0.21093573f + t * (-0.03954289f +
                                     t * (0.00443319f + t * (-0.00031761f + t * 0.00001109f))))));
    } else {
      const float y = 3.0f * __builtin_amdgcn_rcpf(u);
      const float f1 = 0.79788456f + y * (0.00000156f + y * (0.01659667f + y * (0.00017105f +
                                     y * (-0.00249511f + y * (0.00113653f + y * (-0.00020033f))))));
      const float th = (u - 2.35619449f) + y * (0.12499612f + y * (0.00005650f + y * (-0.00637879f +
                                     y * (0.00074348f + y * (0.00079824f + y * (-0.00029166f))))));
      const float ru = __builtin_amdgcn_rsqf(u);
      w = 2.0f * f1 * __cosf(th) * ru * ru * ru;
    }
  } else {
    if (u < 1.0f) {
      const float t = u * u;
      w = 1.0f + t * (-1.0f / 10.0f + t * (1.0f / 280.0f + t * (-1.0f / 15120.0f +
                                              t * (1.0f / 1330560.0f + t * (-1.0f / 172972800.0f)))));
    } else {
      float s, c;
      __sincosf(u, &s, &c);           // hardware sin / cos: ~1e-7 absolute, W is O(u^-2) beyond
      const float ri = __builtin_amdgcn_rcpf(u);
      w = 3.0f * (s - u * c) * (ri * ri * ri);
    }
  }
  return w * w;
}

// |k| of the modes q and n0 - q of a column (kappa enters squared): FP32, the same for every field
__device__ __forceinline__ float mode_k(const Axis0Geom& gm, const ColCoord& cc, int q) {
  constexpr float PI = 3.14159265358979323846f;
  const float kfix2 = gm.ndim == 3 ? cc.kx_c * cc.kx_c + cc.ky * cc.ky : cc.kx_c * cc.kx_c;
  const float k0 = (float)q * gm.kap0;
  return PI * sqrtf(fmaf(k0, k0, kfix2));
}

// The squared form factors of a launch's radii, in the order in which the threads of the axis-0 pass use
// them: [radius][tile][pair][thread].  One workgroup: 256 threads of a tile, one of the pairs.
template <int NDIM>
__global__ void __launch_bounds__(256) k_wvar_table(WvarTabArgs a) {
  const int nbt = (a.T + 255) / 256;
  const int tile = (int)blockIdx.x / nbt, tid = ((int)blockIdx.x - tile * nbt) * 256 + (int)threadIdx.x;
  if (tid >= a.T) return;
  const int k = blockIdx.y, p = tid / a.C, c = tid - p * a.C;
  const int g = tile * a.C + c;
  const int q = k < a.H ? p + a.P * k : a.gm.n0 / 2;
  const float kk = mode_k(a.gm, col_coord(a.gm, g < a.gm.ncol ? g : 0), q);
  for (int j = 0; j < a.nr; ++j)
    a.tab[(((long long)j * a.ntiles + tile) * (a.H + 1) + k) * a.T + tid] = window_w2<NDIM>(kk * a.radii[j]);
}

// Forward transform along axis 0, then sum w_m |X|^2 W(|k| R)^2 of the tile's modes for each radius.
// The modes q and n0 - q of a column share |k|, so their powers meet in LDS and a thread takes pairs
// (q = p + P k, k < E/2; thread p = 0 of a column also q = n0 / 2; q = 0 and q = n0 / 2 stand alone): half
// the form factors.  Those, not memory, bound the pass (about 50 instructions each): evaluated per
// mode it took 290 us for 16 x 2048^2 and 8 radii.  TAB: read from a table instead, evaluated once for
// the fields of the launch; the fields of a tile run on one XCD, whose L2 then serves the table (both
// kernels 113 us).  Otherwise all pairs of a radius in flight at once: two at a time left the transcendentals'
// latency open (3 x 128^3 57 -> 51 us a call, 512^2 31 -> 27, 48 x 64^2 28.2 -> 24.6).
template <int L, int NDIM, bool TAB>
__global__ void __launch_bounds__((ColTile<L, 0>::T)) k_cols_wvar(WvarArgs a) {
  constexpr int P = Plan<L>::P, E = Plan<L>::E, C = ColTile<L, 0>::C, T = ColTile<L, 0>::T, H = E / 2;
  constexpr int PS = WvarLds<L>::PS;
  using Rad = typename Plan<L>::fwd;
  constexpr int R1 = RadInfo<Rad>::first, RL = RadInfo<Rad>::last;
  extern __shared__ float2 lds[];
  __shared__ double red[HU_MAX_RADII][T / 64];
  int b;
  long long tile;
  if (!map_tile(a.sc, b, tile)) return;
  const int tid = threadIdx.x;
  const int c = tid % C, p = tid / C;
  const int g = (int)tile * C + c;
  const bool valid = g < a.gm.ncol;
  const ColIO io = col_io<L>(a.spec + (long long)b * a.Nh, a.Nh, a.gm.inner0, g, p);
  float2 v[E];
  col_load<L, R1, P, E>(v, io);
  fft_run<L, P, E, false>(Rad{}, v, col_region<L, 0, (L >= 64)>(lds, c), p, a.tw);
  // w_m |X|^2 (0 for the mean mode and for columns past the end) to LDS, [column][mode]
  const ColCoord cc = col_coord(a.gm, valid ? g : 0);
  const bool col0 = cc.mx == 0 && (NDIM == 2 || cc.my == 0);
  float* pc = reinterpret_cast<float*>(lds) + c * PS;
  __syncthreads();                                  // the exchange buffer is free from here
#pragma unroll
  for (int s = 0; s < E; ++s) {
    const int e = slot_index<L, RL, P>(s, p);
    pc[e] = (valid && !(col0 && e == 0)) ? cc.wm * (v[s].x * v[s].x + v[s].y * v[s].y) : 0.0f;
  }
  __syncthreads();
  float xa[H + 1], xb[H], kk[TAB ? 1 : H + 1];
#pragma unroll
  for (int k = 0; k < H; ++k) {
    const int q = p + P * k;
    xa[k] = pc[q];
    xb[k] = q == 0 ? 0.0f : pc[L - q];
    if constexpr (!TAB) kk[k] = mode_k(a.gm, cc, q);
  }
  xa[H] = p == 0 ? pc[L / 2] : 0.0f;
  if constexpr (!TAB) kk[H] = mode_k(a.gm, cc, L / 2);
  float w[H + 1];
  auto table = [&](int j) {                         // the form factors of radius j
    const float* t = a.tab + ((long long)j * a.sc.ntiles + tile) * ((H + 1) * T) + tid;
#pragma unroll
    for (int k = 0; k < H; ++k) w[k] = t[k * T];
    if (p == 0) w[H] = t[H * T];
  };
  w[H] = 0.0f;
  if constexpr (TAB) table(0);
  for (int j = 0; j < a.nr; ++j) {
    double acc = 0.0;
    if constexpr (TAB) {
      float wc[H + 1];
#pragma unroll
      for (int k = 0; k <= H; ++k) wc[k] = w[k];
      if (j + 1 < a.nr) table(j + 1);               // in flight during this radius
#pragma unroll
      for (int k = 0; k < H; ++k) acc += (double)(xa[k] * wc[k]) + (double)(xb[k] * wc[k]);
      acc += (double)(xa[H] * wc[H]);
    } else {
      const float R = a.radii[j];
#pragma unroll
      for (int k = 0; k < H; ++k) {
        const float w2 = window_w2<NDIM>(kk[k] * R);
        acc += (double)(xa[k] * w2) + (double)(xb[k] * w2);
      }
      if (p == 0) acc += (double)(xa[H] * window_w2<NDIM>(kk[H] * R));
    }
    acc = wave_sum(acc);
    if ((tid & 63) == 0) red[j][tid >> 6] = acc;
  }
  __syncthreads();
  if (tid < a.nr) {
    double s = 0.0;
    for (int w2 = 0; w2 < T / 64; ++w2) s += red[tid][w2];
    a.partials[((long long)b * a.sc.ntiles + tile) * a.nr_all + a.j0 + tid] = s;
  }
}

template <int L, int NDIM>
static hipError_t launch_cols_wvar_N(const WvarArgs& a, hipStream_t st) {
  constexpr int T = ColTile<L, 0>::T, C = ColTile<L, 0>::C;
  constexpr size_t x = col_xchg_bytes<L, 0, (L >= 64)>(), pw = (size_t)C * WvarLds<L>::PS * 4, lds = x > pw ? x : pw;
  if (a.tab) {
    WvarTabArgs t{};
    t.gm = a.gm;
    t.C = C;
    t.P = Plan<L>::P;
    t.H = Plan<L>::E / 2;
    t.T = T;
    t.ntiles = a.sc.ntiles;
    t.nr = a.nr;
    for (int j = 0; j < a.nr; ++j) t.radii[j] = a.radii[j];
    t.tab = const_cast<float*>(a.tab);
    hipLaunchKernelGGL((k_wvar_table<NDIM>), dim3((unsigned)t.ntiles * ((T + 255) / 256), t.H + 1), dim3(256), 0, st, t);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((k_cols_wvar<L, NDIM, true>), dim3(sched_blocks(a.sc)), dim3(T), lds, st, a);
  } else {
    hipLaunchKernelGGL((k_cols_wvar<L, NDIM, false>), dim3(sched_blocks(a.sc)), dim3(T), lds, st, a);
  }
  return hipGetLastError();
}

hipError_t launch_cols_wvar(int L, const WvarArgs& a, hipStream_t st) {
  switch (L) {
#define X(LL) case LL: return a.gm.ndim == 2 ? launch_cols_wvar_N<LL, 2>(a, st) : launch_cols_wvar_N<LL, 3>(a, st);
    HU_COL_LENGTHS(X)
#undef X
    default: return hipErrorInvalidValue;
  }
}

size_t wvar_table_bytes(int L, int ntiles) {
  switch (L) {
#define X(LL) case LL: return (size_t)WVAR_TAB_RADII * ntiles * (Plan<LL>::E / 2 + 1) * ColTile<LL, 0>::T * sizeof(float);
    HU_COL_LENGTHS(X)
#undef X
    default: return 0;
  }
}

// out[b][j] = scale * (sum over the tiles of field b, in tile order, of partial j): one workgroup
// per field; thread t sums tiles t, t + 256, ... for every radius, then waves and the workgroup
// reduce in a fixed order
__global__ void __launch_bounds__(256) k_wvar_final(WvarFinalArgs a) {
  __shared__ double red[HU_MAX_RADII][4];
  const int b = blockIdx.x, tid = threadIdx.x;
  const double* part = a.partials + (long long)b * a.ntiles * a.nr;
  for (int j = 0; j < a.nr; ++j) {
    double s = 0.0;
    for (int t = tid; t < a.ntiles; t += 256) s += part[(long long)t * a.nr + j];
    s = wave_sum(s);
    if ((tid & 63) == 0) red[j][tid >> 6] = s;
  }
  __syncthreads();
  if (tid < a.nr) a.out[(long long)b * a.nr + tid] = a.scale * (((red[tid][0] + red[tid][1]) + red[tid][2]) + red[tid][3]);
}

hipError_t launch_wvar_final(const WvarFinalArgs& a, int batch, hipStream_t st) {
  hipLaunchKernelGGL(k_wvar_final, dim3(batch), dim3(256), 0, st, a);
  return hipGetLastError();
}

}  // namespace hu
