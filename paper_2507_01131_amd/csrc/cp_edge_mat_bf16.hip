// The L = 4 edge pass through per-edge matrices, bf16 features.
#include "cp_edge_mat_impl.hpp"

#define TDN_MAT(RS, NT) \
  template hipError_t tdn::mat_detail::launch_mat<RS, NT, true, false>(const tdn::EdgeArgs&, hipStream_t);
TDN_MAT(6, 8)
TDN_MAT(8, 4)
TDN_MAT(8, 8)
