// The fused axis-0 pass of the generator: forward FFT along the slowest axis, multiplication by
// the symmetrised amplitude H_sym = sqrt(chi) (Eq. (8) with Eqs. (12)-(13)), the FP64 Parseval
// statistics of Eq. (15), the continuous-field spectrum bins, and the inverse FFT along the same
// axis -- one read and one write of the half spectrum.  Each workgroup leaves its partial sums
// and its tile's bin partials; k_finalize turns the sums into (mu, var, scale, offset) in a fixed
// order, and k_spec_final assembles the bins of the normalised field.
#include "hu_common.hpp"

namespace hu {

// where the filter pass takes the amplitudes from: evaluated per mode in FP32, evaluated in the
// general form (tabulated radial form or FP64), or read from the call's table (k_amp)
enum { AMP_FP32 = 0, AMP_GENERAL = 1, AMP_TABLE = 2 };

// Waves per SIMD asked of the compiler.  A tile of five waves (384 and 768, 24 elements a thread) doubles up on
// one SIMD, so two workgroups are resident only where four waves fit: 128 registers.  Left alone the FP32 form
// takes 132-143 of them (384 x 128 x 256 x 3: 217 us against 165; 768 x 128^2 x 4: 330 against 259); the 2 and 4
// waves of 96 and 192 lose by the same cap (66 -> 68, 126 -> 129).
template <int L, int V, int AMP>
constexpr int filter_waves() { return AMP == AMP_FP32 && Plan<L>::E > 16 && ColTile<L, V>::T > 256 ? 4 : 1; }

// One tile of C columns of one field per workgroup.
template <int L, int NDIM, int V, int AMP, int RV, bool SPLIT>
__global__ void __launch_bounds__((ColTile<L, V>::T)) __attribute__((amdgpu_waves_per_eu(filter_waves<L, V, AMP>())))
k_cols_filter(FilterArgs a) {
  constexpr int P = Plan<L>::P, E = Plan<L>::E, C = ColTile<L, V>::C, T = ColTile<L, V>::T;
  constexpr int LP = ColTile<L, V>::LP;
  using Rad = typename Plan<L, RV>::fwd;
  using RadI = Reverse<Rad>;
  constexpr int R1 = RadInfo<Rad>::first, RL = RadInfo<Rad>::last;
  extern __shared__ __align__(16) float2 lds[];
  __shared__ double red_d[T / 64], red_d0[T / 64];
  __shared__ float red_f[T / 64];
  int b;
  long long tile;
  if (!map_tile(a.sc, b, tile)) return;
  const int tid = threadIdx.x;
  const int c = tid % C, p = tid / C;
  const int g = (int)tile * C + c;
  const bool valid = g < a.gm.ncol;
  // the filter's view of the column and the amplitude of its mode e
  ColCoord cc;
  FiltDev filt{};
  Col3 c3a{}, c3b{};
  // the lattice maximum of ln(chi_rel + offset) is at least ln offset
  float lmax = -1.0e30f;
  auto column = [&]() {
    cc = col_coord(a.gm, valid ? g : 0);
    if constexpr (AMP != AMP_TABLE) {
      filt = a.io ? a.io[b].filt : a.filt;
      lmax = filt.lnoffset;
      if constexpr (NDIM == 3) {                   // the column's x / y terms of the filter
        c3a = col3(filt, cc.kx_c, cc.ky);
        c3b = (filt.rotated && (cc.nyq_x || cc.nyq_y))
                  ? col3(filt, cc.nyq_x ? -cc.kx_c : cc.kx_c, cc.nyq_y ? -cc.ky : cc.ky) : c3a;
      }
    }
  };
  auto amplitude = [&](int e) {
    float lnc;
    const float h = NDIM == 3 ? amp_sym3<AMP == AMP_GENERAL>(filt, a.gm, cc, c3a, c3b, e, lnc)
                              : amp_sym<NDIM, AMP == AMP_GENERAL>(filt, a.gm, cc, e, lnc);
    if (valid) lmax = fmaxf(lmax, lnc);
    return h;
  };
  float* pw = reinterpret_cast<float*>(lds);
  float H[E];
  if constexpr (AMP == AMP_GENERAL) {
    // Before the columns are loaded: one register per amplitude crosses the transform instead of two per
    // column value crossing the FP64 evaluation, and the pass keeps four waves per SIMD (186-230 registers and two
    // waves the other way round; alpha 20: 16 x 2048^2 730 -> 483 us, 512^3 1709 -> 1214, 512^2 x 20 98 -> 81).  A
    // rolled loop that leaves the amplitudes in LDS: unrolled it is tens of kilobytes of code (1024^2 68 us for 43)
    column();
#pragma unroll 1
    for (int s = 0; s < E; ++s) pw[s * T + tid] = amplitude(slot_index<L, RL, P>(s, p));
#pragma unroll
    for (int s = 0; s < E; ++s) H[s] = pw[s * T + tid];
  }
  const ColIO io = col_io<L>(a.spec + (long long)b * a.Nh, a.Nh, a.gm.inner0, g, p);
  float2 v[E];
  col_load<L, R1, P, E>(v, io);
  const bool do_bins = a.parts != nullptr;
  const TileBinPre pre = do_bins ? tile_bins_pre<T>(a.tb, (int)tile, tid) : TileBinPre{};
  fft_run<L, P, E, false, false, RV>(Rad{}, v, col_region<L, V, SPLIT>(lds, c), p, a.tw);
  // ---- filter and per-thread statistics
  if constexpr (AMP != AMP_GENERAL) column();
  double gsum = 0.0, f0 = 0.0;
  // the exchange buffer is free once every thread has its transform in registers: the power
  // values of the continuous spectrum go to LDS as they are computed
  if constexpr (AMP == AMP_TABLE) {                // all loads at once (in groups of four the pass took 8 % longer)
    const rsrc_t ar = make_rsrc(a.amp + tile * (long long)(E * T), (unsigned)(E * T * 4));
#pragma unroll
    for (int s = 0; s < E; ++s)
      H[s] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(ar, (unsigned)tid * 4u, (unsigned)(s * T * 4), 0));
  }
  if (do_bins) __syncthreads();
#pragma unroll
  for (int s = 0; s < E; ++s) {
    const int e = slot_index<L, RL, P>(s, p);
    const float2 F = cscale(v[s], AMP == AMP_FP32 ? amplitude(e) : H[s]);
    v[s] = F;
    const float m2 = cc.wm * (F.x * F.x + F.y * F.y);
    if (do_bins) pw[c * LP + pw_index(e)] = valid ? m2 : 0.0f;
    if (valid) {
      gsum += (double)m2;
      if (g == 0 && e == 0) f0 = (double)F.x;
    }
  }
  // ---- workgroup statistics -> partials[b][tile] (reduced by k_finalize after this kernel)
  gsum = wave_sum(gsum);
  lmax = wave_max(lmax);
  f0 = wave_sum(f0);
  if ((tid & 63) == 0) { red_d[tid >> 6] = gsum; red_f[tid >> 6] = lmax; red_d0[tid >> 6] = f0; }
  __syncthreads();
  if (tid == 0) {
    double gs = 0.0, fz = 0.0;
    float lm = -1.0e30f;
    for (int w = 0; w < T / 64; ++w) { gs += red_d[w]; fz += red_d0[w]; lm = fmaxf(lm, red_f[w]); }
    double* part = a.partials + ((long long)b * a.sc.ntiles + tile) * 4;
    part[0] = gs;
    part[1] = fz;
    part[2] = (double)lm;
    part[3] = 0.0;
  }
  // ---- continuous-spectrum bins of the tile -> its partials in parts[b] (deterministic)
  if (do_bins) {
    tile_bins<L, E, C, LP, T, ColTile<L, V>::PWV, (NDIM == 2)>(lds, a.tb, pre, (int)tile, a.gm.ncol, a.parts + (long long)b * a.tb.M, tid);
  }

  if (a.read_only) return;                       // uniform

  // ---- inverse transform along axis 0 (first radix = last forward radix: no exchange needed)
  fft_run<L, P, E, true, false, RV>(RadI{}, v, col_region<L, V, SPLIT>(lds, c), p, a.tw);
  __builtin_amdgcn_s_setprio(2);                 // the stores out ahead of other workgroups' transforms
  if (valid) col_store<L, R1, P, E>(v, io);
  __builtin_amdgcn_s_setprio(0);
}

// ---------------------------------------------------------------------------------------------
// The symmetrised amplitudes of one filter for every mode, in the order in which the threads of the
// filter pass hold them ([tile][slot][thread]: a wave reads 256 consecutive bytes), and the maximum of
// ln chi over the modes of each workgroup.  A workgroup: 256 threads of a tile, AMP_SLOTS of the slots
// (one 1024^2 field still gives every SIMD two waves), then the next tiles.
// ---------------------------------------------------------------------------------------------
template <int NDIM, bool GEN>
__global__ void __launch_bounds__(256) k_amp(AmpArgs a) {
  __shared__ float red[4];
  float lmax = a.filt.lnoffset;
  const int nbt = (a.T + 255) / 256;
  for (int blk = blockIdx.x; blk < a.ntiles * nbt; blk += gridDim.x) {
    const int tile = blk / nbt, tid = (blk - tile * nbt) * 256 + (int)threadIdx.x;
    if (tid >= a.T) continue;
    const int p = tid / a.C, c = tid - p * a.C;
    const int g = tile * a.C + c;
    const bool valid = g < a.gm.ncol;
    const ColCoord cc = col_coord(a.gm, valid ? g : 0);
    Col3 c3a{}, c3b{};
    if constexpr (NDIM == 3) {
      c3a = col3(a.filt, cc.kx_c, cc.ky);
      c3b = (a.filt.rotated && (cc.nyq_x || cc.nyq_y))
                ? col3(a.filt, cc.nyq_x ? -cc.kx_c : cc.kx_c, cc.nyq_y ? -cc.ky : cc.ky) : c3a;
    }
    float* out = a.amp + (long long)tile * (a.E * a.T) + tid;
#pragma unroll GEN ? 1 : AMP_SLOTS
    for (int u = 0; u < AMP_SLOTS; ++u) {
      const int s = (int)blockIdx.y * AMP_SLOTS + u;
      if (s >= a.E) break;                         // uniform
      const int e = p + a.P * (s / a.R) + (s % a.R) * (a.gm.n0 / a.R);   // slot_index
      float lnc;
      const float H = NDIM == 3 ? amp_sym3<GEN>(a.filt, a.gm, cc, c3a, c3b, e, lnc) : amp_sym<NDIM, GEN>(a.filt, a.gm, cc, e, lnc);
      out[(long long)s * a.T] = H;
      if (valid) lmax = fmaxf(lmax, lnc);
    }
  }
  lmax = wave_max(lmax);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = lmax;
  __syncthreads();
  if (threadIdx.x == 0)
    a.amax[blockIdx.y * gridDim.x + blockIdx.x] = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
}

hipError_t launch_amp(AmpArgs a, int L, int radix, int general, hipStream_t st, int* blocks) {
  switch (L) {
#define X(LL) case LL: a.R = radix ? RadInfo<Plan<LL, 1>::fwd>::last : RadInfo<Plan<LL, 0>::fwd>::last; break;
    HU_COL_LENGTHS(X)
#undef X
    default: return hipErrorInvalidValue;
  }
  a.E = col_elems(L);
  a.P = L / a.E;
  a.T = a.C * a.P;
  const long long n = (long long)a.ntiles * ((a.T + 255) / 256);
  const dim3 grid((unsigned)(n < AMP_MAX_BLOCKS ? n : AMP_MAX_BLOCKS), (unsigned)((a.E + AMP_SLOTS - 1) / AMP_SLOTS));
  *blocks = (int)(grid.x * grid.y);
  auto go = [&](auto kern) { hipLaunchKernelGGL(kern, grid, dim3(256), 0, st, a); };
  if (a.gm.ndim == 2) general ? go(k_amp<2, true>) : go(k_amp<2, false>);
  else general ? go(k_amp<3, true>) : go(k_amp<3, false>);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------------------
// finalize: one workgroup per field turns the filter pass's partials into mu, var and the
// normalisation constants (Eq. (15) via Parseval) with a fixed-order reduction, and the factor
// that turns the continuous-field bins into the spectrum of the normalised field.
// ---------------------------------------------------------------------------------------------
__global__ void __launch_bounds__(256) k_finalize(FinalizeArgs a) {
  __shared__ double sg[256], sf[256];
  __shared__ float sm[256];
  const int b = blockIdx.x, tid = threadIdx.x;
  const double* part = a.partials + (long long)b * a.ntiles * 4;
  double G = 0.0, F0 = 0.0;
  float lm = -1.0e30f;
#pragma unroll 4
  for (int w = tid; w < a.ntiles; w += 256) {
    G += part[4 * w + 0];
    F0 += part[4 * w + 1];
    lm = fmaxf(lm, (float)part[4 * w + 2]);
  }
  for (int w = tid; w < a.namax; w += 256) lm = fmaxf(lm, a.amax[w]);   // the table's maxima
  sg[tid] = G;
  sf[tid] = F0;
  sm[tid] = lm;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if (tid < o) {
      sg[tid] += sg[tid + o];
      sf[tid] += sf[tid + o];
      sm[tid] = fmaxf(sm[tid], sm[tid + o]);
    }
    __syncthreads();
  }
  if (tid == 0) {
    float scale, offset;
    finalize_field(a, b, sg[0], sf[0], (double)sm[0], true, scale, offset);
  }
}

hipError_t launch_finalize(const FinalizeArgs& a, int batch, hipStream_t st) {
  hipLaunchKernelGGL(k_finalize, dim3(batch), dim3(256), 0, st, a);
  return hipGetLastError();
}

template <int L, int V, int RV, bool SPLIT>
static hipError_t launch_cols_filter_L(FilterArgs a, hipStream_t st) {
  constexpr int T = ColTile<L, V>::T;
  size_t lds = col_xchg_bytes<L, V, SPLIT>();
  if (a.parts) lds = col_bin_bytes<L, V, SPLIT>(a.tb);
  // with a table the pass does not depend on the dimension; the general form only in the instantiation
  // launched when a field may use it (complex exchange alone: the exchange does not change the bits)
  if constexpr (SPLIT) {
    if (!a.amp && a.any_gen) return launch_cols_filter_L<L, V, RV, false>(a, st);
  }
  const dim3 grid(sched_blocks(a.sc));
  auto go = [&](auto kern) { hipLaunchKernelGGL(kern, grid, dim3(T), lds, st, a); };
  auto evaluated = [&](auto amp) {
    constexpr int AMP = decltype(amp)::value;
    if (a.gm.ndim == 3) go(k_cols_filter<L, 3, V, AMP, RV, SPLIT>);
    else if constexpr (V == 1 || !half_tile_length(L)) go(k_cols_filter<L, 2, V, AMP, RV, SPLIT>);
    else return hipErrorInvalidValue;
    return hipGetLastError();
  };
  if (a.amp) go(k_cols_filter<L, 2, V, AMP_TABLE, RV, SPLIT>);
  else if (!a.any_gen) return evaluated(std::integral_constant<int, AMP_FP32>{});
  else if constexpr (!SPLIT) return evaluated(std::integral_constant<int, AMP_GENERAL>{});
  return hipGetLastError();
}

int col_width(int L, int variant) {
  switch (L) {
#define X(LL) case LL: return variant ? ColTile<LL, 1>::C : ColTile<LL, 0>::C;
    HU_COL_LENGTHS(X)
#undef X
    default: return 0;
  }
}

int col_elems(int L) {
  switch (L) {
#define X(LL) case LL: return Plan<LL>::E;
    HU_COL_LENGTHS(X)
#undef X
    default: return 0;
  }
}

hipError_t launch_cols_filter(int L, int variant, const FilterArgs& a, hipStream_t st, int radix, int split) {
  switch (L) {
#define X(LL)                                                                                             \
  case LL:                                                                                                \
    return with_choices3<LL>(variant, radix, split, [&](auto v, auto r, auto s) {                         \
      return launch_cols_filter_L<LL, decltype(v)::value, decltype(r)::value, decltype(s)::value>(a, st); \
    });
    HU_COL_LENGTHS(X)
#undef X
    default: return hipErrorInvalidValue;
  }
}

}  // namespace hu
