// How the persistent PCG (pcg.hip) deals a block's rows, and the clearing of
// an exchange buffer, over its workgroups.  Plain C++, so that a CPU test can
// check it.
#pragma once

namespace rg {

// Of a block of c rows, workgroup w of `active` has rows [w rpw, (w+1) rpw)
// and clears entries [w per, (w+1) per) of a buffer of cap.  P, the workgroups
// that are there, comes from the block's capacity, c only from the device:
// those that are left without a row (6 of 256 at c = 4000, nearly all when
// few weights are positive) take no part in the exchange, for nobody would
// wait for them.  An empty block is one workgroup's.
struct PqShare {
  int rpw, active, per;
};
constexpr PqShare pq_share(int c, int cap, int P) {
  const int rpw = (c + P - 1) / P;
  const int active = c > 0 ? (c + rpw - 1) / rpw : 1;
  return {rpw, active, (cap + active - 1) / active};
}

}  // namespace rg
