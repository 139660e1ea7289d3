// gap_records.hpp -- a store's particles to and from the records of the C ABI
// (GAP_DIAG_LEPTONS, GAP_DIAG_PHOTONS, GAP_STATE_PARTICLES), on the device: the
// records of one tube are packed in slot order into a staging buffer, a piece
// at a time, and loaded ones are unpacked from it.  Bound by the copies between
// the device and pageable host memory.  (With every array of the store copied
// out and the records put together by the host, twice because the caller asks
// for the size first, saving and reloading 1e6 particles took 100 ms; it takes
// 67, of which some 55 are the sorting of the ids in that measurement.)
#pragma once
#include "gap_kernels.hpp"

namespace gap {

constexpr int REC_LEP = 24, REC_PHO = 32;   // bytes of a record
constexpr int REC_BLOCK = CHUNK;            // slots per workgroup

struct RecCtx {
  Ctx cx;
  int tube, n_tiles;
  int lep;               // leptons (1) or photons (0)
  int64_t* count;        // per block of REC_BLOCK slots: its records, then the records before it
  long long* total;
};

// Whether slot i of the store holds a record of the tube, and its cell.
__device__ __forceinline__ bool rec_of(const RecCtx& r, long long i, long long S, long long n, int* cell) {
  if (i >= n) return false;
  const Ctx& cx = r.cx;
  const int tile = i < S ? (r.lep ? cx.lchunk : cx.pchunk)[i / CHUNK] : (r.lep ? cx.ltt : cx.ptt)[i];
  if (tile < 0 || tile >= r.n_tiles) return false;
  const Tile tl = cx.tiles[tile];
  if (tl.tube != r.tube || (r.lep ? cx.L.w[i] : cx.P.x[i]) == 0.0f) return false;
  const Tube& T = cx.tubes[tl.tube];
  *cell = tl.base + (int)((r.lep ? cx.L.pos[i] : cx.P.pos[i]) >> FRAC);
  if (T.flags & F_PERIODIC) *cell = wrap_cell(*cell, T.N);
  return true;
}

__global__ __launch_bounds__(TPB) void k_rec_count(RecCtx r) {
  __shared__ int s_n;
  const Ctl* c = r.lep ? r.cx.lc : r.cx.pc;
  const long long S = c->n_sorted_chunks * CHUNK, n = S + c->tail, nb = (n + REC_BLOCK - 1) / REC_BLOCK;
  for (long long b = blockIdx.x; b < nb; b += gridDim.x) {
    if (threadIdx.x == 0) s_n = 0;
    __syncthreads();
    for (int j = 0; j < REC_BLOCK / TPB; ++j) {
      int cell;
      const uint64_t m = __ballot(rec_of(r, b * REC_BLOCK + j * TPB + threadIdx.x, S, n, &cell));
      if (lane_id() == 0 && m) atomicAdd(&s_n, (int)__popcll(m));
    }
    __syncthreads();
    if (threadIdx.x == 0) r.count[b] = s_n;
    __syncthreads();
  }
}

// The blocks' counts to the records before each (one workgroup, four blocks
// per thread and round).
constexpr int REC_SCAN_T = 1024;
__global__ __launch_bounds__(REC_SCAN_T) void k_rec_scan(RecCtx r) {
  __shared__ long long sh[REC_SCAN_T / WAVE];
  const Ctl* c = r.lep ? r.cx.lc : r.cx.pc;
  const long long nb = (c->n_sorted_chunks * CHUNK + c->tail + REC_BLOCK - 1) / REC_BLOCK;
  long long carry = 0;
  for (long long b0 = 0; b0 < nb; b0 += 4 * REC_SCAN_T) {
    const long long b = b0 + 4 * (long long)threadIdx.x;
    long long v[4];
    long long sum = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      v[j] = b + j < nb ? r.count[b + j] : 0;
      sum += v[j];
    }
    long long incl = sum;
#pragma unroll
    for (int d = 1; d < WAVE; d <<= 1) {
      const long long o = __shfl_up(incl, d);
      if (lane_id() >= d) incl += o;
    }
    const int wv = threadIdx.x / WAVE;
    if (lane_id() == WAVE - 1) sh[wv] = incl;
    __syncthreads();
    long long before = carry, tot = carry;
    for (int w = 0; w < REC_SCAN_T / WAVE; ++w) {
      if (w < wv) before += sh[w];
      tot += sh[w];
    }
    long long ex = before + incl - sum;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      if (b + j < nb) r.count[b + j] = ex;
      ex += v[j];
    }
    carry = tot;
    __syncthreads();
  }
  if (threadIdx.x == 0) *r.total = carry;
}

// Records [lo, hi) of the tube to out[0, hi - lo).
__global__ __launch_bounds__(TPB) void k_rec_pack(RecCtx r, long long lo, long long hi, uint2* out) {
  __shared__ int s_w[TPB / WAVE];
  const Ctl* c = r.lep ? r.cx.lc : r.cx.pc;
  const long long S = c->n_sorted_chunks * CHUNK, n = S + c->tail, nb = (n + REC_BLOCK - 1) / REC_BLOCK;
  for (long long b = blockIdx.x; b < nb; b += gridDim.x) {
    long long first = r.count[b];
    if (first >= hi || (b + 1 < nb && r.count[b + 1] <= lo)) continue;
    for (int j = 0; j < REC_BLOCK / TPB; ++j) {
      const long long i = b * REC_BLOCK + j * TPB + threadIdx.x;
      int cell = 0;
      const bool has = rec_of(r, i, S, n, &cell);
      const uint64_t m = __ballot(has);
      __syncthreads();
      if (lane_id() == 0) s_w[threadIdx.x / WAVE] = (int)__popcll(m);
      __syncthreads();
      long long at = first + rank_in(m);
      for (int w = 0; w < TPB / WAVE; ++w) {
        if (w < (int)threadIdx.x / WAVE) at += s_w[w];
        first += s_w[w];
      }
      if (!has || at < lo || at >= hi) continue;
      const Ctx& cx = r.cx;
      const uint32_t frac = (r.lep ? cx.L.pos[i] : cx.P.pos[i]) & 0xFFFFFFu;
      const uint64_t id = r.lep ? cx.L.id[i] : cx.P.id[i];
      uint2* o = out + (at - lo) * (r.lep ? REC_LEP / 8 : REC_PHO / 8);
      *o++ = make_uint2((uint32_t)cell, frac);
      *o++ = r.lep ? make_uint2(__float_as_uint(cx.L.u[i]), __float_as_uint(cx.L.w[i]))
                   : make_uint2(__float_as_uint(cx.P.x[i]), __float_as_uint(cx.P.w[i]));
      if (!r.lep) *o++ = make_uint2((uint32_t)cx.P.n0[i], 0u);
      *o = make_uint2((uint32_t)id, (uint32_t)(id >> 32));
    }
  }
}

// Loaded records lo .. lo + n - 1 (checked by the host) to slots of the same
// index, as a tail of the tube whose first tile is tile0.
__global__ __launch_bounds__(TPB) void k_rec_unpack(Ctx cx, int lep, int tile0, const uint2* in, long long lo, long long n) {
  for (long long j = (long long)blockIdx.x * TPB + threadIdx.x; j < n; j += (long long)gridDim.x * TPB) {
    const uint2* r = in + j * (lep ? REC_LEP / 8 : REC_PHO / 8);
    const uint2 place = r[0], vals = r[1], id = r[lep ? 2 : 3];
    const int t = (int)place.x / TILE;
    const uint32_t pos = (uint32_t)((int)place.x - (t * TILE - MARGIN)) << FRAC | place.y;
    const long long i = lo + j;
    const uint64_t id64 = (uint64_t)id.y << 32 | id.x;
    if (lep) {
      cx.L.pos[i] = pos;
      cx.L.u[i] = __uint_as_float(vals.x);
      cx.L.w[i] = __uint_as_float(vals.y);
      cx.L.id[i] = id64;
      cx.ltt[i] = tile0 + t;
    } else {
      cx.P.pos[i] = pos;
      cx.P.x[i] = __uint_as_float(vals.x);
      cx.P.w[i] = __uint_as_float(vals.y);
      cx.P.n0[i] = (int32_t)r[2].x;
      cx.P.id[i] = id64;
      cx.ptt[i] = tile0 + t;
    }
  }
}

}  // namespace gap
