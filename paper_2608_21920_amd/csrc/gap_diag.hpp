// gap_diag.hpp -- discharge diagnostics of libgap (gfx950, wave64): the
// quantities the paper reads off its simulations (Sect. 5, Figs. 3, 5, 7).
//
//  * Profile (Fig. 3, rows 5-7): per bin of B cells and per group -- e- and
//    e+ moving up (u > 0) and down, photons with |x| > 2 moving up (x > 0)
//    and down -- the multiplicity m = n / n_co = sum |w| / (B ppc_ref) (a
//    weight-w macro-particle stands for w dx / ppc_ref particles per unit
//    area), the mean Lorentz factor <gamma> (photons: <|x|>) and the
//    plasma-inertia measure <gamma^-3> = n^-1 sum w gamma^-3 (its definition
//    with eq. omega_osc, Sect. 3).
//  * Peak (Fig. 5): the largest pair multiplicity m_+- (e- plus e+, both
//    directions) over the bins inside the gap zone h < H, the height of that
//    bin, <gamma^-3> of the pairs there, the photon multiplicity there, and
//    the extremes of E over the cells.
//  * Return spectrum (Fig. 7): the weight of the leptons absorbed at the
//    surface, binned in log10 gamma, filled by the lepton passes (gap_kernels).
//  * Waterfall (Fig. 4): the space-time diagram of E^2, the mean of E^2 over
//    bins of cells recorded after the field update of every k-th step.
//  * Power spectrum of E along the gap: the field zero-padded to M, the next
//    power of two >= N, transformed by a radix-4 Stockham FFT in FP64,
//    P_k = |X_k|^2 / M for k = 0 .. M/2.
#pragma once
#include "gap_kernels.hpp"

namespace gap {

constexpr int PROF_G = 6;   // groups: e- up, e- down, e+ up, e+ down, photons (|x| > 2) up, down
constexpr int PROF_M = 3;   // moments per group: sum |w|, sum |w| gamma (photons |x|), sum |w| gamma^-3

// Adds (v0, v1, v2) to acc[key * 3 + m] for every lane with key >= 0, one
// atomic per distinct key of the wave.
__device__ __forceinline__ void prof_wave_add(int key, double v0, double v1, double v2, double* acc) {
  while (true) {
    const uint64_t m = __ballot(key >= 0);
    if (!m) break;
    const int lead = __ffsll((long long)m) - 1;
    const int kk = __shfl(key, lead);
    double a = key == kk ? v0 : 0.0, b = key == kk ? v1 : 0.0, c = key == kk ? v2 : 0.0;
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) {
      a += __shfl_xor(a, d);
      b += __shfl_xor(b, d);
      c += __shfl_xor(c, d);
    }
    if (lane_id() == lead) {
      atomicAdd(&acc[(size_t)kk * PROF_M + 0], a);
      atomicAdd(&acc[(size_t)kk * PROF_M + 1], b);
      if (c != 0.0) atomicAdd(&acc[(size_t)kk * PROF_M + 2], c);
    }
    if (key == kk) key = -1;
  }
}

// Profile moments of one particle of tube T: key = bin * PROF_G + group (-1:
// none).  a: lepton weight or photon energy (0: no particle); u: lepton
// momentum; pw: photon weight.
__device__ __forceinline__ int prof_moments(const Tube& T, bool lep, int base, uint32_t pos, float a, float u, float pw,
                                            int B, double* v0, double* v1, double* v2) {
  *v0 = *v1 = *v2 = 0.0;
  if (a == 0.0f) return -1;
  int cell = base + (int)(pos >> FRAC);
  if (T.flags & F_PERIODIC) cell = wrap_cell(cell, T.N);
  const int bin = min(max(cell, 0), T.N - 1) / B;
  if (lep) {
    const double ud = (double)u;
    const double w = fabs((double)a);
    const double g = sqrt(1.0 + ud * ud);
    *v0 = w;
    *v1 = w * g;
    *v2 = w / (g * g * g);
    return bin * PROF_G + (a < 0.0f ? 0 : 2) + (ud > 0.0 ? 0 : 1);
  }
  if (!(fabsf(a) > 2.0f)) return -1;
  const double w = (double)pw;
  *v0 = w;
  *v1 = w * fabs((double)a);
  return bin * PROF_G + 4 + (a > 0.0f ? 0 : 1);
}

// The sorted part of one store, for the diagnostics of one tube: workgroup bx
// of G takes a contiguous range of chunks, VEC slots per thread in 16-byte
// loads, and calls enter(tile) (block-uniform) when the tile changes and
// slot(tile base, position, w or x, u or 0, 0 or photon w) for every slot.
template <class Enter, class Slot>
__device__ __forceinline__ void diag_sorted(const Ctx& cx, bool lep, int tube, Enter enter, Slot each) {
  long long c0, c1;
  chunk_range((lep ? cx.lc : cx.pc)->n_sorted_chunks, gridDim.x, blockIdx.x, &c0, &c1);
  const CPtr<int32_t> chunk = cptr(lep ? cx.lchunk : cx.pchunk);
  const float* const fa = lep ? cx.L.w : cx.P.x;
  const float* const fb = lep ? cx.L.u : cx.P.w;
  const uint32_t* const fp = lep ? cx.L.pos : cx.P.pos;
  int held = -1, base = 0;
  bool mine = false;
  for (long long c = c0; c < c1; ++c) {
    const int tile = chunk[c];
    if (tile != held) {
      held = tile;
      const Tile tl = cx.tiles[tile];
      base = tl.base;
      mine = tl.tube == tube;
      if (mine) enter(base);
    }
    if (!mine) continue;
    const long long s0 = c * CHUNK + VEC * (int)threadIdx.x;
    float a[VEC], b[VEC];
    uint32_t p[VEC];
    rec_get(rec_load<float, VEC>(fa + s0), a);
    rec_get(rec_load<float, VEC>(fb + s0), b);
    rec_get(rec_load<uint32_t, VEC>(fp + s0), p);
#pragma unroll
    for (int j = 0; j < VEC; ++j) each(base, p[j], a[j], b[j]);
  }
}
// The tail of one store, strided over all workgroups: one slot per lane (the
// lanes of a wave go together; a lane without a particle of the tube has a = 0).
template <class Slot>
__device__ __forceinline__ void diag_tail(const Ctx& cx, bool lep, int tube, Slot each) {
  const Ctl* ctl = lep ? cx.lc : cx.pc;
  const long long S = ctl->n_sorted_chunks * CHUNK, tail = ctl->tail;
  const long long nsq = S / TPB, nq = nsq + (tail + TPB - 1) / TPB;
  for (long long q = nsq + blockIdx.x; q < nq; q += gridDim.x) {
    uint32_t slot;
    int tile;
    piece_slot(q, nsq, S, tail, lep ? cx.lchunk : cx.pchunk, lep ? cx.ltt : cx.ptt, &slot, &tile);
    const Tile tl = cx.tiles[tile >= 0 ? tile : 0];
    const bool in = tile >= 0 && tl.tube == tube;
    each(tl.base, lep ? cx.L.pos[slot] : cx.P.pos[slot], in ? (lep ? cx.L.w[slot] : cx.P.x[slot]) : 0.0f,
         lep ? cx.L.u[slot] : cx.P.w[slot]);
  }
}

constexpr int PROF_LDS = 80 * PROF_G * PROF_M;   // LDS sums of a workgroup

// Moments of tube `tube`'s particles into acc[nb][PROF_G][PROF_M], which the
// caller has zeroed.  The particles of a sorted chunk lie within its tile's
// 256-cell window, so with bins of at least 4 cells they are summed into an
// LDS window of bins (FP64 LDS atomics), flushed to acc when the tile changes
// and at the end; tail rows (and narrower bins) add to acc directly, one
// atomic per distinct key of a wave.  Few bins in the window mean many lanes
// on one word, served one at a time: the window is kept in as many copies as
// the LDS holds (up to 16), a lane's copy by its index (4.0e6 particles, bins
// of 64 cells: 37 us with one copy and one slot per thread).
__global__ __launch_bounds__(TPB) void k_profile(Ctx cx, int tube, int B, int nb, double* acc) {
  __shared__ double s_w[PROF_LDS];
  const bool win = B >= 4;
  const int lw = win ? (WIN - 1) / B + 2 : 1;            // bins a tile's window can reach
  const int stride = lw * PROF_G * PROF_M;
  int copies = 1;
  while (copies < 16 && 2 * copies * stride <= PROF_LDS) copies *= 2;
  const Tube& T = cx.tubes[tube];
  for (int j = threadIdx.x; j < PROF_LDS; j += blockDim.x) s_w[j] = 0.0;
  int lo = -1;                              // first bin of the LDS window (block-uniform)
  __syncthreads();
  auto flush = [&]() {
    __syncthreads();
    if (lo >= 0)
      for (int j = threadIdx.x; j < stride; j += blockDim.x) {
        double v = 0.0;
        for (int r = 0; r < copies; ++r) {
          v += s_w[r * stride + j];
          s_w[r * stride + j] = 0.0;
        }
        if (v != 0.0 && lo + j / (PROF_G * PROF_M) < nb) atomicAdd(&acc[(size_t)lo * PROF_G * PROF_M + j], v);
      }
    __syncthreads();
  };
  for (int sp = 0; sp < 2; ++sp) {
    const bool lep = sp == 0;
    diag_sorted(
        cx, lep, tube,
        [&](int base) {
          const int wl = max(base, 0) / B;
          if (win && wl != lo) {
            flush();
            lo = wl;
          }
        },
        [&](int base, uint32_t pos, float a, float b) {
          double v0, v1, v2;
          const int key = prof_moments(T, lep, base, pos, a, b, b, B, &v0, &v1, &v2);
          const int kb = win && key >= 0 ? key / PROF_G - lo : -1;
          const bool in = kb >= 0 && kb < lw;
          if (in) {
            double* e = &s_w[(lane_id() & (copies - 1)) * stride + (kb * PROF_G + key % PROF_G) * PROF_M];
            atomicAdd(&e[0], v0);
            atomicAdd(&e[1], v1);
            if (v2 != 0.0) atomicAdd(&e[2], v2);
          }
          if (__ballot(key >= 0 && !in)) prof_wave_add(in ? -1 : key, v0, v1, v2, acc);   // (every lane takes part)
        });
    diag_tail(cx, lep, tube, [&](int base, uint32_t pos, float a, float b) {
      double v0, v1, v2;
      const int key = prof_moments(T, lep, base, pos, a, b, b, B, &v0, &v1, &v2);
      prof_wave_add(key, v0, v1, v2, acc);
    });
  }
  flush();
}

// Sums to the profile: out[nb][PROF_G][3] = multiplicity, <gamma> (photons
// <|x|>), <gamma^-3> (0 for photons and for empty groups).
__global__ void k_profile_finish(const double* acc, int nb, double bppc, double* out) {
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < nb * PROF_G; i += gridDim.x * blockDim.x) {
    const double w = acc[(size_t)i * PROF_M], wg = acc[(size_t)i * PROF_M + 1], wg3 = acc[(size_t)i * PROF_M + 2];
    out[(size_t)i * 3 + 0] = w / bppc;
    out[(size_t)i * 3 + 1] = w > 0.0 ? wg / w : 0.0;
    out[(size_t)i * 3 + 2] = w > 0.0 ? wg3 / w : 0.0;
  }
}

// Peak of the pair multiplicity over the bins whose centre lies in the gap
// zone (h < H), with ties to the lowest bin, and the field's extremes; one
// workgroup.  out: m_+- at the peak, the peak bin's centre height, <gamma^-3>
// of the pairs there, the photon multiplicity (|x| > 2) there, min E, max E.
constexpr int PEAK_T = 1024;   // one workgroup of 1024 threads

__global__ __launch_bounds__(PEAK_T) void k_profile_peak(const double* acc, int nb, int B, double dx, double H,
                                                         double bppc, const float* E, int N, double* out) {
  __shared__ double s_v[PEAK_T];
  __shared__ int s_i[PEAK_T];
  __shared__ double s_lo[PEAK_T], s_hi[PEAK_T];
  double best = -1.0;
  int arg = -1;
  for (int b = threadIdx.x; b < nb; b += blockDim.x) {
    if (!(((double)b + 0.5) * B * dx < H)) continue;
    double m = 0.0;
    for (int g = 0; g < 4; ++g) m += acc[((size_t)b * PROF_G + g) * PROF_M];
    if (m > best) { best = m; arg = b; }   // (b grows within a thread: the first of equal values stays)
  }
  // four independent loads per round
  double lo = 1e300, hi = -1e300;
  const int bd = blockDim.x;
  for (int k = threadIdx.x; k < N; k += 4 * bd) {
    float v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) v[u] = k + u * bd < N ? E[k + u * bd] : E[k];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      lo = fmin(lo, (double)v[u]);
      hi = fmax(hi, (double)v[u]);
    }
  }
  s_v[threadIdx.x] = best;
  s_i[threadIdx.x] = arg;
  s_lo[threadIdx.x] = lo;
  s_hi[threadIdx.x] = hi;
  __syncthreads();
  for (int d = blockDim.x / 2; d >= 1; d >>= 1) {
    if ((int)threadIdx.x < d) {
      const double v = s_v[threadIdx.x + d];
      const int i = s_i[threadIdx.x + d];
      if (v > s_v[threadIdx.x] || (v == s_v[threadIdx.x] && i >= 0 && (s_i[threadIdx.x] < 0 || i < s_i[threadIdx.x]))) {
        s_v[threadIdx.x] = v;
        s_i[threadIdx.x] = i;
      }
      s_lo[threadIdx.x] = fmin(s_lo[threadIdx.x], s_lo[threadIdx.x + d]);
      s_hi[threadIdx.x] = fmax(s_hi[threadIdx.x], s_hi[threadIdx.x + d]);
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    const int b = s_i[0];
    double m = 0.0, g3 = 0.0, mx = 0.0;
    if (b >= 0) {
      double w = 0.0;
      for (int g = 0; g < 4; ++g) {
        w += acc[((size_t)b * PROF_G + g) * PROF_M];
        g3 += acc[((size_t)b * PROF_G + g) * PROF_M + 2];
      }
      m = w / bppc;
      g3 = w > 0.0 ? g3 / w : 0.0;
      mx = (acc[((size_t)b * PROF_G + 4) * PROF_M] + acc[((size_t)b * PROF_G + 5) * PROF_M]) / bppc;
    }
    out[0] = m;
    out[1] = b >= 0 ? ((double)b + 0.5) * B * dx : -1.0;
    out[2] = g3;
    out[3] = mx;
    out[4] = N > 0 ? s_lo[0] : 0.0;
    out[5] = N > 0 ? s_hi[0] : 0.0;
  }
}

// Waterfall record of the step that the field update just counted, when
// its index is a multiple of `every`: the mean of E^2 over each bin of B
// cells (the last bin ragged) goes to ring slot (step / every) mod cap of
// the tube, and the step index beside it.  One wave per bin, FP64 sums of
// squares of the FP32 field; grid (ceil(nbmax / waves per block), tubes).
struct WfCtx {
  const Tube* tubes;
  const float* E;
  double* ring;        // [tube][cap][nbmax]
  long long* steps;    // [tube][cap], -1 for an empty slot
  int every, B, cap, nbmax;
};

__global__ __launch_bounds__(TPB) void k_waterfall(WfCtx w) {
  const int t = blockIdx.y;
  const Tube& T = w.tubes[t];
  const long long step = T.step;
  if (step < 0 || step % w.every != 0) return;
  const int N = T.N;
  const int nb = (N + w.B - 1) / w.B;
  const long long slot = (step / w.every) % w.cap;
  const int bin = blockIdx.x * (TPB / WAVE) + (int)(threadIdx.x / WAVE);
  if (bin < nb) {
    const int c0 = bin * w.B, c1 = min(N, c0 + w.B);
    double s = 0.0;
    for (int c = c0 + lane_id(); c < c1; c += WAVE) {
      const double e = (double)w.E[T.cell_off + c];
      s += e * e;
    }
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) s += __shfl_xor(s, d);
    if (lane_id() == 0) w.ring[((size_t)t * w.cap + slot) * w.nbmax + bin] = s / (double)(c1 - c0);
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) w.steps[(size_t)t * w.cap + slot] = step;
}

// Power spectrum of E: load (zero-padded), Stockham stages of radix 4 and, for
// an odd power of two, one of radix 2 (output in natural order after the
// last), |X|^2 / M.  One thread per butterfly of the stage; every index is
// below M (M a power of two).
__global__ void k_fft_load(const float* E, int N, int M, double2* x) {
  for (int j = blockIdx.x * blockDim.x + threadIdx.x; j < M; j += gridDim.x * blockDim.x)
    x[j] = make_double2(j < N ? (double)E[j] : 0.0, 0.0);
}

// Stage with sub-transforms of length Ns (1, 2, 4, ..., M/2): pair j takes
// in[j] and in[j + M/2], turns the second by exp(-i pi k / Ns) with
// k = j mod Ns, and writes the sum and difference Ns apart at 2 (j - k) + k.
__global__ void k_fft_stage(const double2* in, double2* out, int M, int Ns) {
  const int h = M / 2;
  for (int j = blockIdx.x * blockDim.x + threadIdx.x; j < h; j += gridDim.x * blockDim.x) {
    const int k = j & (Ns - 1);
    double s, c;
    sincospi(-(double)k / (double)Ns, &s, &c);
    const double2 a = in[j], b = in[j + h];
    const double2 t = make_double2(b.x * c - b.y * s, b.x * s + b.y * c);
    const int o = 2 * (j - k) + k;
    out[o] = make_double2(a.x + t.x, a.y + t.y);
    out[o + Ns] = make_double2(a.x - t.x, a.y - t.y);
  }
}

// Two of those stages in one: sub-transforms of length Ns to 4 Ns.  Butterfly j
// of M/4 takes in[j + q M/4], q = 0 .. 3, turns them by exp(-i pi q k / (2
// Ns)) with k = j mod Ns, and writes their 4-point transform Ns apart at
// 4 (j - k) + k.  (A stage is a launch and a trip through L2 more than it is
// arithmetic: 14 of them for 16384 cells.  With 7 of these in their place all
// diagnostics of a snapshot on 16384 cells took 443 us, from 465.)
__global__ void k_fft_stage4(const double2* in, double2* out, int M, int Ns) {
  const int h = M / 4;
  for (int j = blockIdx.x * blockDim.x + threadIdx.x; j < h; j += gridDim.x * blockDim.x) {
    const int k = j & (Ns - 1);
    double2 v[4];
    v[0] = in[j];
#pragma unroll
    for (int q = 1; q < 4; ++q) {
      double s, c;
      sincospi(-(double)(q * k) / (double)(2 * Ns), &s, &c);
      const double2 b = in[j + q * h];
      v[q] = make_double2(b.x * c - b.y * s, b.x * s + b.y * c);
    }
    const double2 p = make_double2(v[0].x + v[2].x, v[0].y + v[2].y), m = make_double2(v[0].x - v[2].x, v[0].y - v[2].y);
    const double2 r = make_double2(v[1].x + v[3].x, v[1].y + v[3].y), d = make_double2(v[1].x - v[3].x, v[1].y - v[3].y);
    const int o = 4 * (j - k) + k;
    out[o] = make_double2(p.x + r.x, p.y + r.y);
    out[o + Ns] = make_double2(m.x + d.y, m.y - d.x);       // m - i d
    out[o + 2 * Ns] = make_double2(p.x - r.x, p.y - r.y);
    out[o + 3 * Ns] = make_double2(m.x - d.y, m.y + d.x);   // m + i d
  }
}

__global__ void k_fft_power(const double2* X, int M, double* P) {
  for (int k = blockIdx.x * blockDim.x + threadIdx.x; k <= M / 2; k += gridDim.x * blockDim.x)
    P[k] = (X[k].x * X[k].x + X[k].y * X[k].y) / (double)M;
}

// Momentum spectra (Fig. 3, row 1): the weight of electrons and positrons
// per 1/8 decade of |u| and of photons per 1/8 decade of |x|, from 1e-2 to
// 1e9, with an underflow and an overflow bin.  A value's bin is the number of
// edges 10^(-2 + b/8) (b = 0 .. 88) whose square its square reaches, taken
// in FP64 against a host-computed table of the squares (spec_bin).  Each
// workgroup sums a contiguous range of each store's sorted chunks, and its
// share of the tails, into an LDS histogram and adds it to acc[3][SPEC_NB]
// once.
constexpr int SPEC_EDGES = 89;
constexpr int SPEC_NB = SPEC_EDGES + 1;

// Edges at or below |p| by its FP32 logarithm, at least one: edge b is at
// log2 |p| = (b - 16) log2(10) / 8.  (Clamped before the conversion: an
// infinite |p| has every edge below it.)
__host__ __device__ __forceinline__ int spec_guess(float log2p) {
  return (int)fminf(fmaxf(floorf(log2p * (8.0f * 0.30102999566398120f)) + 17.0f, 1.0f), (float)SPEC_EDGES);
}
// (The guess is off by at most one bin, settled by the exact comparisons with
// its two edges.)
__device__ __forceinline__ int spec_bin(const double* thr, float p) {
  const double p2 = (double)p * (double)p;
  if (!(p2 >= thr[0])) return 0;
  int n = spec_guess(__log2f(fabsf(p)));
  if (n < SPEC_EDGES && thr[n] <= p2) ++n;
  else if (thr[n - 1] > p2) --n;
  return n;
}

__global__ __launch_bounds__(TPB) void k_spectra(Ctx cx, int tube, const double* thr, double* acc) {
  __shared__ double s_h[3 * SPEC_NB];
  __shared__ double s_thr[SPEC_EDGES];
  for (int j = threadIdx.x; j < 3 * SPEC_NB; j += blockDim.x) s_h[j] = 0.0;
  for (int j = threadIdx.x; j < SPEC_EDGES; j += blockDim.x) s_thr[j] = thr[j];
  __syncthreads();
  for (int sp = 0; sp < 2; ++sp) {
    const bool lep = sp == 0;
    auto add = [&](int, uint32_t, float a, float b) {
      if (a == 0.0f) return;
      const int s3 = lep ? (a < 0.0f ? 0 : 1) : 2;
      atomicAdd(&s_h[s3 * SPEC_NB + spec_bin(s_thr, lep ? b : a)], (double)(lep ? fabsf(a) : b));
    };
    diag_sorted(cx, lep, tube, [](int) {}, add);
    diag_tail(cx, lep, tube, add);
  }
  __syncthreads();
  for (int j = threadIdx.x; j < 3 * SPEC_NB; j += blockDim.x)
    if (s_h[j] != 0.0) atomicAdd(&acc[j], s_h[j]);
}

// Phase space (Fig. 3, rows 1-4): the weights of the momentum spectra, per
// bin of B cells and signed momentum column (column SPEC_NB + b for p > 0,
// SPEC_NB - 1 - b for p <= 0, b the spectrum bin of |p|), added to
// acc[3][nb][2 SPEC_NB].  Sorted chunks go through an LDS window of the lw
// bins their tile can reach (2 lepton species or the photons), flushed when
// the tile changes; the tails, and bins too narrow for the LDS (lw = 0), add
// to acc directly, equal keys of a wave together (phase_wave_add).  (One
// global atomic per distinct key of a wave for all of them, found one after
// the other, took 545 us for 4.0e6 particles.)
constexpr int PHASE_NP = 2 * SPEC_NB;
constexpr int PHASE_LDS = 60 * 1024;
// Bins of the LDS window for bins of B cells (0: too many).
inline int phase_window(int B) {
  const int lw = (WIN - 1) / B + 2;
  return 2 * lw * PHASE_NP * (int)sizeof(double) <= PHASE_LDS ? lw : 0;
}

// Adds v to acc[key] for every lane with key >= 0 (every lane takes part).
// Lanes that share a key are added together, key after key, until two keys in
// a row have fewer than PHASE_FEW lanes: additions to one word are served one
// after the other, and rounds for keys of a lane or two cost more than they
// save.  (1.9e6 photons of one energy in one cell and 4.1e5 new pairs beside
// them: 0.51 ms with bins of 8 cells and 0.16 with bins of 64; with an
// addition per particle 23.5 and 2.3, with a round per key 0.54 and 0.56.  A
// discharge mix of 4.0e6 with bins of 8: 0.98, 0.96 and 1.44 ms.)
constexpr int PHASE_FEW = 4;
__device__ __forceinline__ void phase_wave_add(long long key, double v, double* acc) {
  for (int few = 0; few < 2;) {
    const uint64_t m = __ballot(key >= 0);
    if (!m) return;
    const int lead = __ffsll((long long)m) - 1;
    const long long kk = __shfl(key, lead);
    const bool mine = key == kk;
    if (__popcll(__ballot(mine)) < PHASE_FEW) {
      if (mine) atomicAdd(&acc[kk], v);
      ++few;
    } else {
      double a = mine ? v : 0.0;
#pragma unroll
      for (int d = 32; d >= 1; d >>= 1) a += __shfl_xor(a, d);
      if (lane_id() == lead) atomicAdd(&acc[kk], a);
      few = 0;
    }
    if (mine) key = -1;
  }
  if (key >= 0) atomicAdd(&acc[key], v);
}

__global__ __launch_bounds__(TPB) void k_phase(Ctx cx, int tube, int B, int nb, const double* thr, double* acc, int lw) {
  extern __shared__ double s_h[];           // [2][lw][PHASE_NP]
  __shared__ double s_thr[SPEC_EDGES];
  for (int j = threadIdx.x; j < SPEC_EDGES; j += blockDim.x) s_thr[j] = thr[j];
  const int n = lw * PHASE_NP;
  for (int j = threadIdx.x; j < 2 * n; j += blockDim.x) s_h[j] = 0.0;
  __syncthreads();
  const Tube& T = cx.tubes[tube];
  for (int sp = 0; sp < 2; ++sp) {
    const bool lep = sp == 0;
    int lo = -1;                            // first bin of the LDS window (block-uniform)
    auto flush = [&]() {
      __syncthreads();
      if (lo >= 0)
        for (int j = threadIdx.x; j < (lep ? 2 : 1) * n; j += blockDim.x) {
          const double v = s_h[j];
          if (v != 0.0) {
            const int s = j >= n ? 1 : 0, r = j - s * n;
            atomicAdd(&acc[((size_t)(lep ? s : 2) * nb + lo) * PHASE_NP + r], v);
            s_h[j] = 0.0;
          }
        }
      __syncthreads();
    };
    auto add = [&](bool window, int base, uint32_t pos, float a, float b) {
      int cell = base + (int)(pos >> FRAC);
      if (T.flags & F_PERIODIC) cell = wrap_cell(cell, T.N);
      cell = min(max(cell, 0), T.N - 1);
      const float p = lep ? b : a;
      const int m = spec_bin(s_thr, p);
      const int col = p > 0.0f ? SPEC_NB + m : SPEC_NB - 1 - m;
      const int s = lep && a > 0.0f ? 1 : 0, bin = cell / B;
      const double v = (double)(lep ? fabsf(a) : b);
      const bool in = window && bin >= lo && bin - lo < lw;
      if (in && a != 0.0f) atomicAdd(&s_h[s * n + (bin - lo) * PHASE_NP + col], v);
      const bool out = !in && a != 0.0f;
      if (__ballot(out)) phase_wave_add(out ? ((long long)(lep ? s : 2) * nb + bin) * PHASE_NP + col : -1, v, acc);
    };
    diag_sorted(
        cx, lep, tube,
        [&](int base) {
          const int wl = max(base, 0) / B;
          if (lw > 0 && wl != lo) {
            flush();
            lo = wl;
          }
        },
        [&](int base, uint32_t pos, float a, float b) { add(lw > 0, base, pos, a, b); });
    diag_tail(cx, lep, tube, [&](int base, uint32_t pos, float a, float b) { add(false, base, pos, a, b); });
    flush();
  }
}

}  // namespace gap
