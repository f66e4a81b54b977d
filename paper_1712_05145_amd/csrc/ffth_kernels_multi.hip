// Multi-size launches of the FP32 inner iteration (grouped z-pass with the
// Green operator, fused three-term CG x-pass): the kernels in ffth_kernels.h
// take each load's grid from its descriptor.
#include "ffth_kernels.h"
#include "ffth_launch.h"

namespace ffth {

bool multi_grid(const int n[3]) { return multi_size(n[0]) && multi_size(n[1]) && multi_size(n[2]); }

void multi_blocks(const int n[3], int out[2], int lds[2]) {
  out[0] = multi_z_blocks(n);
  out[1] = multi_x_blocks(n);
  lds[0] = multi_z_lds(n);
  lds[1] = multi_x_lds(n);
}

hipError_t multi_gz(const MultiSegs& sg, int lds, hipStream_t s, const Desc* d, int op, bool h16, int fin) {
  const dim3 grid(sg.off[sg.n] + (fin >= 0 ? sg.nload : 0));
  if (h16) hipLaunchKernelGGL(k_gz_multi<H2>, grid, dim3(MULTI_NT), lds, s, d, op, sg, fin);
  else hipLaunchKernelGGL(k_gz_multi<C2<float>>, grid, dim3(MULTI_NT), lds, s, d, op, sg, fin);
  return hipGetLastError();
}

hipError_t multi_xcg3(const MultiSegs& sg, int lds, hipStream_t s, const Desc* d, bool iso, bool h16) {
  const dim3 grid(sg.off[sg.n]);
  if (iso) {
    if (h16) hipLaunchKernelGGL((k_xcg3_multi<true, H2>), grid, dim3(MULTI_NT), lds, s, d, sg);
    else hipLaunchKernelGGL((k_xcg3_multi<true, C2<float>>), grid, dim3(MULTI_NT), lds, s, d, sg);
  } else {
    if (h16) hipLaunchKernelGGL((k_xcg3_multi<false, H2>), grid, dim3(MULTI_NT), lds, s, d, sg);
    else hipLaunchKernelGGL((k_xcg3_multi<false, C2<float>>), grid, dim3(MULTI_NT), lds, s, d, sg);
  }
  return hipGetLastError();
}

}  // namespace ffth
