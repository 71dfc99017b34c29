// The L = 4 edge pass through per-edge matrices, fp32 features.
#include "cp_edge_mat_impl.hpp"

#define TDN_MAT(RS, NT)                                                                                         \
  template hipError_t tdn::mat_detail::launch_mat<RS, NT, false, false>(const tdn::EdgeArgs&, hipStream_t); \
  template hipError_t tdn::mat_detail::launch_mat<RS, NT, false, true>(const tdn::EdgeArgs&, hipStream_t); \
  template hipError_t tdn::mat_detail::launch_mat<RS, NT, false, false, true>(const tdn::EdgeArgs&, hipStream_t);
TDN_MAT(6, 3)
TDN_MAT(6, 4)
TDN_MAT(8, 3)
TDN_MAT(8, 4)
