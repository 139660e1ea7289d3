// gap_fused.hpp -- the particle passes of a step in two launches, for handles
// whose photon store is small.
//
// The general step runs its photon side (prologue, sorted photon pass,
// conversion draws) on a second stream beside the lepton side, which pays
// when both sides fill the chip.  With few photons that side is launches and
// waits: a step of the production gap's start state (2.1e5 leptons, 65536
// cells) took 52 us, of which the kernels' critical path is about half and
// the rest is two cross-stream waits of about 5 us each and the issue of six
// launches and three event calls.  Here the same work is two launches on one
// stream:
//   k_sorted   the prologue, both sorted passes
//   k_rest     the queued photon births and conversions' pairs, both tail
//              passes, the protons
// and the field update is the third: the same steps took 35 us then, and take
// 25 to 30 now; one step of the 1024-cell gap with a read of its field and
// charge 62 us instead of 137, 64 steps of a 1000-cell periodic box 1.34 ms
// instead of 3.35.  The roles inside a launch touch
// disjoint data for the reasons the two streams do: each pass reads its own
// store up to a tail snapshot, births go past the snapshots, only leptons
// and protons deposit charge, and the prologue changes the surface charge
// only atomically.  What the photon pass took from the prologue it takes from
// the state the prologue starts from (the tubes' own step index, the cold
// guarantee before it is counted down), and k_rest counts the guarantee down.
// No result depends on which form ran.
#pragma once
#include "gap_protons.hpp"

namespace gap {

constexpr int FUSED_PRE = 8;   // workgroups before the passes (one XCD round; the first is the prologue)

// Workgroups [0, FUSED_PRE): the prologue (n_tubes < 0: already done); then gp of the photon pass; then gl
// of the lepton pass (gp and gl multiples of 8, for the XCD-aware ranges).
// The short roles come first so that a lepton pass of several rounds does
// not keep them waiting.
template <bool Q, bool A, int V>
__global__ __launch_bounds__(TPB, 6) void k_sorted(Ctx cx, int n_tubes, int gp, int gl) {
  const int bx = (int)blockIdx.x;
  if (bx < FUSED_PRE) {
    if (bx == 0 && n_tubes >= 0) prologue<A>(cx, n_tubes, false);
  } else if (bx < FUSED_PRE + gp) {
    photons_sorted<V, true>(cx, bx - FUSED_PRE, gp);
  } else {
    leptons_sorted<Q, A, V>(cx, bx - FUSED_PRE - gp, gl);
  }
}

// Workgroups of k_rest by role, in dispatch order.
struct RestGrid { int births, conv, tails, protons; };

template <bool Q, bool A>
__global__ __launch_bounds__(TPB) void k_rest(Ctx cx, RestGrid n) {
  int bx = (int)blockIdx.x;
  if (bx == 0 && threadIdx.x == 0 && cx.pc->cold_steps >= 0) cx.pc->cold_steps -= 1;
  if (bx < n.births) { births_queue<Q>(cx, bx, n.births); return; }
  bx -= n.births;
  if (bx < n.conv) { pairs_queue<Q>(cx, bx, n.conv); return; }
  bx -= n.conv;
  if (bx < n.tails) { both_tails<Q, A>(cx, bx, n.tails); return; }
  protons_pass(cx, bx - n.tails, n.protons);
}

}  // namespace gap
