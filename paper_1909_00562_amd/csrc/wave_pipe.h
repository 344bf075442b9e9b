// A reduction split over the waves of a block, every wave with fragments in flight in registers.
#pragma once
#include <hip/hip_runtime.h>

namespace asx {

// steps w, w + KS, ... of a list of nsteps
template <int KS> __device__ __forceinline__ int own_steps(int nsteps, int wave) {
  return nsteps > wave ? (nsteps - wave + KS - 1) / KS : 0;
}

// schedule of a region: load v of NL after (v + 1) / NL of its NM matrix instructions
template <int v, int NL, int NM> __device__ __forceinline__ void spread_loads() {
  if constexpr (v < NL) {
    constexpr int nm = (v + 1) * NM / NL - v * NM / NL;
    if constexpr (nm > 0) __builtin_amdgcn_sched_group_barrier(0x008, nm, 0);
    __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
    spread_loads<v + 1, NL, NM>();
  }
}

struct NoRest {
  __device__ __forceinline__ void operator()(int, int) const {}
};
struct NoMeanwhile {
  __device__ __forceinline__ void operator()() const {}
};

// A wave's n reduction steps, slot i % PF of the fragment registers holding step i.  load(slot, i) must be free of
// branches and valid for 0 <= i < n; past the last step it is called with the last one again, so that the number of
// loads in flight is the same on every path and a wait covers just the fragments it needs.
// The NL loads of a step are spread over the NM matrix instructions of an earlier one.  Issued in one run they hold the
// wave at the address unit while its matrix pipe idles: forward wavefronts of 4 layers x 1024 units x 128 sentences
// then took the sum of their load and matrix times.
// rest(slot, i): products of step i that may need a branch, behind the region that the loads are spread over.
// meanwhile(): other work of the wave, done while the first loads are on their way.
template <int PF, int NL, int NM, typename Load, typename Mul, typename Rest = NoRest, typename Meanwhile = NoMeanwhile>
__device__ __forceinline__ void wave_reduce(int n, Load load, Mul mul, Rest rest = Rest(),
                                            Meanwhile meanwhile = Meanwhile()) {
  if (n <= 0) {
    meanwhile();
    return;
  }
  auto at = [&](int i) { return i < n ? i : n - 1; };
#pragma unroll
  for (int u = 0; u + 1 < PF; ++u) load(u, at(u));
  __builtin_amdgcn_sched_barrier(0);
  meanwhile();
  __builtin_amdgcn_sched_barrier(0);
  int i = 0;
  for (; i + PF <= n; i += PF) {
#pragma unroll
    for (int u = 0; u < PF; ++u) {
      mul(u, at(i + u));
      load((u + PF - 1) % PF, at(i + u + PF - 1));
      spread_loads<0, NL, NM>();
      __builtin_amdgcn_sched_barrier(0);
      rest(u, at(i + u));
    }
  }
#pragma unroll
  for (int u = 0; u + 1 < PF; ++u)
    if (i + u < n) {
      mul(u, at(i + u));
      rest(u, at(i + u));
    }
}

}  // namespace asx
