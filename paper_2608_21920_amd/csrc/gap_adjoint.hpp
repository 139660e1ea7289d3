// gap_adjoint.hpp -- reverse pass of the particle loop over a window with the
// QED realisation frozen: every emission is a constant recoil offset on its
// lepton, and photons and pairs born inside the window are constants.  The
// differentiated map is the push and the field of one step (Sect. 4 kick and
// drift, Sect. 2.2 Gauss integration from the surface field E_s, which the
// Ampere drive alpha j_co advances):
//   E_{j+1/2} = E_s + w0 sum_{i<=j} rho_i - background,  rho from the
//   first-order split (w (1 - xi) on node k, w xi on node k + 1);
//   u' = u + sign(w) E_p dt, E_p = (1 - xi) Eb_k + xi Eb_{k+1};
//   u'' = u' - x (recorded recoil);  xi' = xi + cfl u'' / sqrt(1 + u''^2);
//   E_s' = E_s + w0 (absorbed w + injected |w|) + alpha s_co dt.
// The fixed-point rounding of the deposit and drift is taken as the identity.
//
// Within a checkpoint segment no re-sort runs, so a lepton keeps its slot;
// the tape holds each slot's position and momentum at the start of every
// step (TAPE_DEAD for empty or dead slots) and the node field each step used.
#pragma once
#include "gap_kernels.hpp"

namespace gap {

constexpr uint32_t TAPE_DEAD = 0xFFFFFFFFu;

struct AdjTube {            // per tube (device)
  double lamEs;             // adjoint of the surface field
  double dalpha;            // dL/dalpha
  double dinjw;             // dL/d(weight of one injected electron)
  // w0 sum_k lamE_k summed over the reverse steps taken so far: the part of
  // every live lepton's weight adjoint that does not depend on its cell.
  // The slots hold their weight adjoints less this sum (FP32 then keeps the
  // small cell-dependent rest, and an injected electron's -lam_w + lamEs w0,
  // a near cancellation of two large sums, is formed in FP64).
  double cw;
  double w0, s_co, dt, cfl, lossw;   // lossw = 2 / (window steps * N)
  int32_t N, cell_off, node_off, pad;
};

struct TapeMeta {           // lepton store at one tape point
  int64_t S;                // sorted-region slots
  int64_t tail_pre;         // tail before this step's injection
  int64_t tail_post;        // tail after it
  int64_t used;             // slots taped: S + tail_post
};

struct AdjCtx {
  const Tile* tiles;
  const int32_t* chunk;     // lepton chunk -> tile (layout of the segment)
  const int32_t* tt;        // lepton tail slot -> tile
  const float* wlast;       // weight of each slot while alive
  const uint32_t* pos0;     // tape at the start of step j
  const float* u0;
  const uint32_t* pos1;     // tape at the start of step j + 1
  const float* u1;
  const TapeMeta* meta0;
  const float* eb0;         // node field used by step j
  float* lxi;
  float* lu;
  float* lw;
  const double* lamE;       // adjoint of the cell field after step j
  const double* suf;        // suffix sums of lamE per tube node: suf_k = sum_{m>=k} lamE_m
  double* lamEb;            // adjoint of the node field of step j (accumulated)
  AdjTube* at;
};

// ------------------------------------------------------------------ tape
// Copy the lepton positions and momenta of slots [0, S + tail) into one tape
// point; `final` marks the point after a segment's last step (no injection).
__global__ __launch_bounds__(TPB) void k_tape(LepBuf L, const Ctl* lc, uint32_t* tpos, float* tu, float* wlast,
                                              TapeMeta* meta, long long M, int final_point, int* err) {
  const long long S = lc->n_sorted_chunks * CHUNK;
  long long used = S + lc->tail;
  if (used > M) {
    if (blockIdx.x == 0 && threadIdx.x == 0) atomicOr(err, E_CAP);
    used = M;
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    TapeMeta m;
    m.S = S;
    m.tail_post = lc->tail;
    m.tail_pre = final_point ? lc->tail : lc->tail_pre;
    m.used = used;
    *meta = m;
  }
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < used; i += (long long)gridDim.x * blockDim.x) {
    const float w = L.w[i];
    const bool alive = w != 0.0f;
    tpos[i] = alive ? L.pos[i] : TAPE_DEAD;
    tu[i] = L.u[i];
    if (alive) wlast[i] = w;
  }
}

// ------------------------------------------------------------------ reverse
// The field of one step in reverse, one launch: the node-field adjoints of
// the step after it (nb) become cell-field adjoints (and E_s's share), the
// loss term of the field is added, and the suffix sums of the cell-field
// adjoints are formed for the weights; E_s receives their total and alpha
// enters it as alpha s_co dt.  At the window's last field there is no step
// after it (nb null).
//
// Blocks of FB_NODES cells, one tube's from its top down, find the sum over
// the cells above them by looking back over the records of lower-indexed
// blocks, as k_field_1p does (same records, termination and bounded wait).
// The former form, one workgroup per tube in two launches, took 48 us per
// step at 16384 cells; this one 8.
struct AdjFieldCtx {
  const FBlk* fb;
  unsigned long long* rec;   // a four-word record per block, then an epoch per tube
  double* lamE;
  double* suf;
  const double* nb;          // node-field adjoints of the step after (null: none)
  double* nb_clear;          // the other buffer, cleared for the step before
  const float* E;            // the field whose loss term is added (null: outside the window)
  AdjTube* at;
  int* err;
};

__global__ __launch_bounds__(FB_THREADS) void k_adj_field(AdjFieldCtx f) {
  constexpr int NW = FB_THREADS / WAVE;
  __shared__ double sh[NW];
  __shared__ double s_above;
  __shared__ unsigned long long s_ep;
  const FBlk b = load_fblk(f.fb, (int)blockIdx.x);
  AdjTube& a = f.at[b.tube];
  const int N = b.N;
  const int bx = (int)blockIdx.x;
  const int q = b.nblk - 1 - (bx - b.first_blk);   // the tube's top block comes first
  const int k = q * FB_NODES + (int)threadIdx.x * FB_PER;
  unsigned long long* epoch = f.rec + 4 * gridDim.x + b.tube;
  const double* nb = f.nb ? f.nb + b.node_off : nullptr;
  double v[FB_PER], loc = 0.0;
#pragma unroll
  for (int i = FB_PER - 1; i >= 0; --i) {
    v[i] = 0.0;
    if (k + i < N) {
      if (nb) v[i] = k + i < N - 1 ? 0.5 * (nb[k + i] + nb[k + i + 1]) : 0.5 * nb[N - 1] + nb[N];
      if (f.E) v[i] += a.lossw * (double)f.E[b.cell_off + k + i];
      f.lamE[b.cell_off + k + i] = v[i];
      f.nb_clear[b.node_off + k + i] = 0.0;
      if (k + i == N - 1) f.nb_clear[b.node_off + N] = 0.0;
    }
    loc += v[i];
  }
  // inclusive suffix over the wave's lanes, then over the waves
  double incl = loc;
#pragma unroll
  for (int d = 1; d < WAVE; d <<= 1) {
    const double o = __shfl_down(incl, d);
    if (lane_id() + d < WAVE) incl += o;
  }
  const int wv = threadIdx.x / WAVE;
  if (lane_id() == 0) sh[wv] = incl;
  if (threadIdx.x == 0) s_ep = __hip_atomic_load(epoch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __syncthreads();
  if (threadIdx.x < WAVE) {
    double tot = 0.0;
    for (int w = NW - 1; w >= 0; --w) tot += sh[w];
    const uint32_t cur = (uint32_t)(s_ep + 1) << 2;
    double above = 0.0;
    if (bx == b.first_blk) {
      if (lane_id() == 0) fs_put(f.rec + 4 * bx, cur | FS_INCL, 0, tot);
    } else {
      if (lane_id() == 0) fs_put(f.rec + 4 * bx, cur | FS_AGG, 0, tot);
      for (int top = bx - 1; top >= b.first_blk; top -= WAVE) {
        const int p = top - lane_id();
        const bool in = p >= b.first_blk;
        uint32_t t = 0;
        long long pv = 0;
        double pe = 0.0;
        if (in) {
          int spin = 0;
          t = fs_get(f.rec + 4 * p, &pv, &pe);
          while ((t & ~3u) != cur && ++spin < FS_SPIN) {
            __builtin_amdgcn_s_sleep(2);
            t = fs_get(f.rec + 4 * p, &pv, &pe);
          }
          if ((t & ~3u) != cur) atomicOr(f.err, E_SCAN);
        }
        const unsigned long long im = __ballot(in && t == (cur | FS_INCL));
        const int stop = im ? __ffsll((long long)im) - 1 : WAVE;
        double x = (in && lane_id() <= stop && (t & ~3u) == cur) ? pe : 0.0;
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) x += __shfl_xor(x, d);
        above += x;
        if (im) break;
      }
      if (lane_id() == 0) fs_put(f.rec + 4 * bx, cur | FS_INCL, 0, above + tot);
    }
    if (lane_id() == 0) {
      s_above = above;
      if (q == 0) {                     // every cell of the tube is in
        const double total = above + tot;
        a.lamEs += (nb ? 0.5 * nb[0] : 0.0) + total;
        a.cw += a.w0 * total;
        a.dalpha += a.lamEs * a.s_co * a.dt;
      }
    }
  }
  __syncthreads();
  double s = s_above + (incl - loc);
  for (int w = NW - 1; w > wv; --w) s += sh[w];
#pragma unroll
  for (int i = FB_PER - 1; i >= 0; --i) {
    if (k + i >= N) continue;
    s += v[i];
    f.suf[b.node_off + k + i] = s;
    if (k + i == N - 1) f.suf[b.node_off + N] = 0.0;
  }
  // (the look-back is over: every block of the tube has read the epoch)
  if (threadIdx.x == 0 && bx == b.first_blk + b.nblk - 1)
    __hip_atomic_store(epoch, s_ep + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// One live lepton, step j in reverse: field term at the post-step position,
// drift, recoil (identity), kick.  e, sd: the adjoint of its cell's field
// after the step and the sum of those above it, less the tube's total (dead
// after the step: unused); e0, e1: the node field around it before.  Gives
// the adjoint of the field it was kicked by.
__device__ __forceinline__ float adj_push(const AdjTube& a, uint32_t p0, uint32_t p1, float u1, float w, int cell0,
                                          double e, double sd, float e0, float e1, float* lxi, float* lu, float* lw) {
  const float dt = (float)a.dt, cfl = (float)a.cfl;
  const double w0 = a.w0;
  if (p1 != TAPE_DEAD) {
    const double xi1 = (double)(p1 & 0xFFFFFFu) * 5.9604644775390625e-8;
    *lxi += (float)(-w0 * (double)w * e);
    // w0 ((1 - xi) lamE_k + sum_{m>k} lamE_m), less the common w0 sum_m lamE_m
    *lw += (float)(w0 * ((1.0 - xi1) * e + sd));
    const float g = sqrtf(1.0f + u1 * u1);
    *lu += *lxi * cfl / (g * g * g);
  } else {
    // gone during step j: absorbed below the surface (its charge enters E_s)
    // or out of the top of the box
    *lxi = 0.0f;
    *lu = 0.0f;
    *lw = (float)((cell0 < a.N / 2 ? a.lamEs * w0 : 0.0) - a.cw);
  }
  const float lEp = (w < 0.0f ? -1.0f : 1.0f) * dt * *lu;
  *lxi += lEp * (e1 - e0);
  return lEp;
}

// A slot of the tail: global memory for the field adjoints.
__device__ __forceinline__ void adj_tail(const AdjCtx& c, long long slot, int tile, long long inj0, long long inj1) {
  const uint32_t p0 = c.pos0[slot];
  if (p0 == TAPE_DEAD) return;
  const Tile tl = c.tiles[tile];
  AdjTube& a = c.at[tl.tube];
  const float w = c.wlast[slot];
  const int cell0 = tl.base + (int)(p0 >> FRAC);
  const float xi0 = (float)(p0 & 0xFFFFFFu) * 5.9604645e-8f;
  float lxi = c.lxi[slot], lu = c.lu[slot], lw = c.lw[slot];
  const uint32_t p1 = c.pos1[slot];
  double e = 0.0, sd = 0.0;
  if (p1 != TAPE_DEAD) {
    const int cell1 = tl.base + (int)(p1 >> FRAC);
    e = c.lamE[a.cell_off + cell1];
    sd = c.suf[a.node_off + cell1 + 1] - c.suf[a.node_off];
  }
  const float lEp = adj_push(a, p0, p1, c.u1[slot], w, cell0, e, sd, c.eb0[a.node_off + cell0],
                             c.eb0[a.node_off + cell0 + 1], &lxi, &lu, &lw);
  atomicAdd(&c.lamEb[a.node_off + cell0], (double)((1.0f - xi0) * lEp));
  atomicAdd(&c.lamEb[a.node_off + cell0 + 1], (double)(xi0 * lEp));
  if (slot >= inj0 && slot < inj1) {
    // injected at the start of step j with weight -inj_w; its injection also
    // raised E_s by inj_w w0
    atomicAdd(&a.dinjw, -(double)lw + (a.lamEs * a.w0 - a.cw));
    lxi = 0.0f;
    lu = 0.0f;
    lw = 0.0f;
  }
  c.lxi[slot] = lxi;
  c.lu[slot] = lu;
  c.lw[slot] = lw;
}

// The leptons of step j in reverse.  Sorted slots: a contiguous range of
// chunks per workgroup, VEC slots per thread in 16-byte accesses, and the
// tile's field adjoints, suffix sums and node field in an LDS window beside
// the one that collects the node-field adjoints (injected electrons are in
// the tail).  Tail slots go through global memory.
// Bound by HBM: both ends of the step (12 B of the tape), the weight, and
// three adjoints in and out, 40 B a slot: 4.0e6 slots take 38 us, 56 with a
// chunk and a window per workgroup and gathers from global memory.
constexpr int ADJ_GRID = 1024;

__global__ __launch_bounds__(TPB) void k_adj_leptons(AdjCtx c) {
  __shared__ double s_acc[WIN + 2];
  __shared__ double s_lam[WIN], s_sd[WIN];
  __shared__ float s_e0[WIN + 2];
  const TapeMeta m = *c.meta0;
  const long long S = m.S, used = m.used;
  const long long nsc = S / CHUNK, ntp = (used - S + TPB - 1) / TPB;
  const int j0 = (int)threadIdx.x;
  long long q0, q1;
  chunk_range(nsc, gridDim.x, blockIdx.x, &q0, &q1);
  int held = -1;
  Tile tl{};
  for (int j = j0; j < WIN + 2; j += TPB) s_acc[j] = 0.0;
  auto flush = [&](const AdjTube& a) {
    for (int j = j0; j <= WIN; j += TPB) {
      const double v = s_acc[j];
      if (v != 0.0) {
        atomicAdd(&c.lamEb[a.node_off + tl.base + j], v);
        s_acc[j] = 0.0;
      }
    }
  };
  for (long long q = q0; q < q1; ++q) {
    const long long s0 = q * CHUNK + VEC * j0;
    const uint4 p0 = *reinterpret_cast<const uint4*>(c.pos0 + s0), p1 = *reinterpret_cast<const uint4*>(c.pos1 + s0);
    const float4 u1 = *reinterpret_cast<const float4*>(c.u1 + s0), w = *reinterpret_cast<const float4*>(c.wlast + s0);
    float4 lxi = *reinterpret_cast<const float4*>(c.lxi + s0), lu = *reinterpret_cast<const float4*>(c.lu + s0),
           lw = *reinterpret_cast<const float4*>(c.lw + s0);
    const int tile = cptr(c.chunk)[q];
    if (tile != held) {
      __syncthreads();
      if (held >= 0) flush(c.at[tl.tube]);
      held = tile;
      tl = c.tiles[tile];
      const AdjTube& a = c.at[tl.tube];
      const int cell = tl.base + j0;
      const bool in = cell >= 0 && cell < a.N;
      s_lam[j0] = in ? c.lamE[a.cell_off + cell] : 0.0;
      s_sd[j0] = in ? c.suf[a.node_off + cell + 1] - c.suf[a.node_off] : 0.0;
      for (int j = j0; j <= WIN; j += TPB) {
        const int node = tl.base + j;
        s_e0[j] = node >= 0 && node <= a.N ? c.eb0[a.node_off + node] : 0.0f;
      }
      __syncthreads();
    }
    const AdjTube& a = c.at[tl.tube];
    auto one = [&](uint32_t x0, uint32_t x1, float uu, float ww, float& gx, float& gu, float& gw) {
      if (x0 == TAPE_DEAD) return;
      const int off0 = (int)(x0 >> FRAC), off1 = (int)(x1 >> FRAC);
      const float xi0 = (float)(x0 & 0xFFFFFFu) * 5.9604645e-8f;
      const float lEp = adj_push(a, x0, x1, uu, ww, tl.base + off0, s_lam[off1], s_sd[off1], s_e0[off0], s_e0[off0 + 1],
                                 &gx, &gu, &gw);
      atomicAdd(&s_acc[off0], (double)((1.0f - xi0) * lEp));
      atomicAdd(&s_acc[off0 + 1], (double)(xi0 * lEp));
    };
    one(p0.x, p1.x, u1.x, w.x, lxi.x, lu.x, lw.x);
    one(p0.y, p1.y, u1.y, w.y, lxi.y, lu.y, lw.y);
    one(p0.z, p1.z, u1.z, w.z, lxi.z, lu.z, lw.z);
    one(p0.w, p1.w, u1.w, w.w, lxi.w, lu.w, lw.w);
    *reinterpret_cast<float4*>(c.lxi + s0) = lxi;
    *reinterpret_cast<float4*>(c.lu + s0) = lu;
    *reinterpret_cast<float4*>(c.lw + s0) = lw;
  }
  __syncthreads();
  if (held >= 0) flush(c.at[tl.tube]);
  for (long long q = blockIdx.x; q < ntp; q += gridDim.x) {
    const long long slot = S + q * TPB + j0;
    if (slot < used) adj_tail(c, slot, c.tt[slot], S + m.tail_pre, S + m.tail_post);
  }
}

// ------------------------------------------------------------------ id map
__device__ __forceinline__ uint64_t mix64(uint64_t x) {
  // splitmix64 finaliser (Steele, Lea & Flood, OOPSLA 2014)
  x ^= x >> 30;
  x *= 0xBF58476D1CE4E5B9ull;
  x ^= x >> 27;
  x *= 0x94D049BB133111EBull;
  x ^= x >> 31;
  return x;
}

// The table holds slots of a saved layout (HASH_EMPTY32 = free); a particle
// is found by (tube, id), read back through the saved arrays.
constexpr uint32_t HASH_EMPTY32 = 0xFFFFFFFFu;

__device__ __forceinline__ uint64_t hkey(uint64_t id, int tube) {
  return mix64(id ^ mix64((uint64_t)tube + 0x632BE59BD9B4E019ull));
}

__global__ void k_hash_clear(uint32_t* vals, long long n) {
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long long)gridDim.x * blockDim.x)
    vals[i] = HASH_EMPTY32;
}

// Insert the live slots [0, n) of a saved lepton store (sorted region only).
__global__ void k_hash_insert(const uint64_t* ids, const float* w, const int32_t* chunk, const Tile* tiles, long long n,
                              uint32_t* vals, uint64_t mask) {
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long long)gridDim.x * blockDim.x) {
    if (w[i] == 0.0f) continue;
    const int tube = tiles[chunk[i / CHUNK]].tube;
    uint64_t h = hkey(ids[i], tube) & mask;
    for (uint64_t probe = 0; probe <= mask; ++probe) {
      if (atomicCAS(&vals[h], HASH_EMPTY32, (uint32_t)i) == HASH_EMPTY32) break;
      h = (h + 1) & mask;
    }
  }
}

// The adjoint of every live slot of the current lepton store, taken from the
// slot of the same particle (same tube and id) in the saved layout (zero for
// dead slots).
__global__ void k_lam_map(LepBuf L, const Ctl* lc, const int32_t* chunk, const int32_t* tt, const Tile* tiles,
                          const uint64_t* sid, const int32_t* schunk, const uint32_t* vals, uint64_t mask,
                          const float* sxi, const float* su, const float* sw, float* dxi, float* du, float* dw,
                          long long M, int* err) {
  const long long S = lc->n_sorted_chunks * CHUNK;
  long long used = S + lc->tail;
  if (used > M) {
    if (blockIdx.x == 0 && threadIdx.x == 0) atomicOr(err, E_CAP);
    used = M;
  }
  for (long long r = (long long)blockIdx.x * blockDim.x + threadIdx.x; r < used; r += (long long)gridDim.x * blockDim.x) {
    float a = 0.0f, b = 0.0f, c = 0.0f;
    if (L.w[r] != 0.0f) {
      const uint64_t id = L.id[r];
      const int tube = tiles[r < S ? chunk[r / CHUNK] : tt[r]].tube;
      uint64_t h = hkey(id, tube) & mask;
      bool found = false;
      for (uint64_t probe = 0; probe <= mask; ++probe) {
        const uint32_t q = vals[h];
        if (q == HASH_EMPTY32) break;
        if (sid[q] == id && tiles[schunk[q / CHUNK]].tube == tube) {
          a = sxi[q]; b = su[q]; c = sw[q];
          found = true;
          break;
        }
        h = (h + 1) & mask;
      }
      if (!found) atomicOr(err, E_TILE);
    }
    dxi[r] = a;
    du[r] = b;
    dw[r] = c;
  }
}

}  // namespace gap
