// Select kernel: the phase-2 argmin of Algorithm 1 (section 4).
//
// At a step t with N_att - 1 <= t <= N_r - 2 every KV head appends one skip
// entry: the kept window key with the lowest softmax weight.  The window
// softmax is taken over the kept decode keys only (the prompt is not part of
// K[idx]).  With several query heads per KV head, the weights of the group
// are summed; with one, the argmin is taken on the logits themselves, which
// the softmax orders identically.  Ties go to the first (oldest) key.  The
// entry is stored as the offset t - idx[j*] at list slot k = t - N_att + 1,
// so running the same step twice rewrites the same slot.
//
// With S sinks the steps that select are N_att - 1 <= t <= N_r + S - 2 (the
// phase-2 range of the positions after the sinks), the sinks are the first
// S kept positions and never candidates, and k = t - N_att + 1 still holds.
#include "device.h"
#include "internal.h"

namespace dsa {
namespace {

// One wave per (request, KV head), or for long windows of several heads
// (GROUP, sel_lds_bytes) a workgroup whose waves take the heads.  Bound by
// latency.  Long windows (LONG, over kSelectShort keys) in launches of at most
// kSelectAhead pairs (AHEAD) load the logits and the plan row with the position
// and the counts, before those say how many there are; the others after them,
// since most requests select nothing and then need none.
template <int G, bool GROUP, bool LONG, bool AHEAD>
__global__ __launch_bounds__(kBlock) void select_kernel(SelectArgs a) {
  extern __shared__ __attribute__((aligned(16))) float terms[];  // GROUP: [window key][G]
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int pair = GROUP ? blockIdx.x : blockIdx.x * kWaves + wave;
  if (pair >= a.pairs) return;
  const int b = pair / a.Hkv;
  const int kvh = pair % a.Hkv;
  const int plan_cap = a.plan_cap;
  const float* wl = a.wlog + (static_cast<size_t>(b) * a.Hq + kvh * G) * plan_cap + a.Ns;
  const int32_t* kept_pos = a.idx + static_cast<size_t>(pair) * plan_cap + a.Ns;
  int t = a.pos[b];
  const int cnt = a.st_count[pair];
  const int n = min(max(a.count[pair], 0), plan_cap);
  float v[kRowRegs];
  int32_t kp[kRowRegs];
  if constexpr (AHEAD) {
    load_row(wl + (GROUP ? wave : 0) * plan_cap, lane, plan_cap - a.Ns, v);
    load_row(kept_pos, lane, plan_cap - a.Ns, kp);
  }
  if (t < 0) return;
  t = min(t, a.Ldec - 1);
  if (t < a.Natt - 1 || t > a.Nr + a.Ns - 2) return;
  const int k = t - (a.Natt - 1);
  if (k >= a.state_cap) return;
  if (cnt < k) {
    if ((!GROUP || wave == 0) && lane == 0) a.st_flags[pair] |= DSA_FLAG_STATE_BEHIND;
    return;
  }
  const int nw = n - a.Ns;  // kept window keys after the sinks
  if (nw <= 0) return;
  if constexpr (LONG && !AHEAD) load_row(wl + (GROUP ? wave : 0) * plan_cap, lane, nw, v);
  int jbest;
  if constexpr (GROUP) {
    head_terms_row<G>(lane, nw, wl + wave * plan_cap, v, terms + wave);
    for (int g = wave + select_waves(G); g < G; g += select_waves(G)) {
      load_row(wl + g * plan_cap, lane, nw, v);
      head_terms_row<G>(lane, nw, wl + g * plan_cap, v, terms + g);
    }
    __syncthreads();
    if (wave > 0) return;
    jbest = terms_argmin<G>(lane, nw, [&](int g, int j) { return terms[j * G + g]; });
  } else if constexpr (G == 1 && LONG) {
    jbest = row_argmin(lane, nw, wl, v);
  } else {
    jbest = window_argmin<G>(lane, nw, [&](int g, int j) { return wl[g * plan_cap + j]; });
  }
  if (jbest < 0 || jbest >= nw) jbest = 0;  // only for NaN logits
  int pos = 0;
  if (AHEAD && jbest < 64 * kRowRegs) {
#pragma unroll
    for (int c = 0; c < kRowRegs; ++c)
      if (jbest >> 6 == c) pos = __shfl(kp[c], jbest & 63, 64);
  } else {
    pos = kept_pos[jbest];
  }
  if (lane == 0) {
    const int d = min(max(t - pos, 0), a.Nr - 2);
    a.st_off[static_cast<size_t>(pair) * a.state_cap + k] = static_cast<uint16_t>(d);
    a.st_count[pair] = k + 1;
  }
  if (a.kept_on && nw == a.kept_cap) {
    const int sl = (k + 1) & 1;
    write_kept_list(lane, nw, jbest, t, a.Natt - a.Ns + k, [&](int r) { return kept_pos[r]; },
                    a.st_kept + (static_cast<size_t>(pair) * 2 + sl) * a.kept_stride,
                    a.st_kc + 2 * pair + sl, k + 1);
  }
}

template <int G>
void launch_g(const SelectArgs& a, hipStream_t st) {
  constexpr bool kGroup = G > 1;
  const int grid = (a.pairs + kWaves - 1) / kWaves;
  if (kGroup ? a.lds == 0 : a.plan_cap - a.Ns <= kSelectShort) {
    select_kernel<G, false, false, false><<<grid, kBlock, 0, st>>>(a);
    return;
  }
  const auto kernel = a.pairs <= kSelectAhead ? select_kernel<G, kGroup, true, true>
                                              : select_kernel<G, kGroup, true, false>;
  if (kGroup)
    kernel<<<a.pairs, 64 * select_waves(G), a.lds, st>>>(a);
  else
    kernel<<<grid, kBlock, 0, st>>>(a);
}

}  // namespace

hipError_t launch_select(const Derived& d, const SelectArgs& a, hipStream_t st) {
  switch (d.G) {
    case 1: launch_g<1>(a, st); break;
    case 2: launch_g<2>(a, st); break;
    case 4: launch_g<4>(a, st); break;
    default: launch_g<8>(a, st); break;
  }
  return hipGetLastError();
}

}  // namespace dsa
