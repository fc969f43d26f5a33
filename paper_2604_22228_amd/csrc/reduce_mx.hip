// MX blocks (e4m3 codes, one E8M0 scale per 32 elements): sum (plain or
// Sum2).
#include "reduce_impl.hpp"

namespace pcoll {
template <class Args>
hipError_t launch_reduce_mx(const Args& a, bool comp, int nranks, const Launch& l) {
  using namespace dev;
  if (comp) return launch_ranks<MxTile<true>>(a, nranks, l);
  return launch_ranks<MxTile<false>>(a, nranks, l);
}

template hipError_t launch_reduce_mx(const ReduceArgs&, bool, int,
                                     const Launch&);
template hipError_t launch_reduce_mx(const DirectArgs&, bool, int,
                                     const Launch&);
}  // namespace pcoll
