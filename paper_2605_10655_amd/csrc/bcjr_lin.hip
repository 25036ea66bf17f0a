// bcjr_lin.hip -- the linear-domain kernels of bcjr_lin_kernels.h (trellises
// below 65536 states) in their own translation unit; the dispatcher in
// bcjr_capi.hip reaches them through these functions.
#include <hip/hip_runtime.h>

#include "bcjr_lin_kernels.h"

namespace bcjr {

namespace {

template <int KB, int n>
LinShape group_shape(bool vjp, bool dc) {
  LinShape s;
  s.fn = !vjp ? (const void*)lin_group_kernel<KB, n, false, false>
         : dc ? (const void*)lin_group_kernel<KB, n, true, true> : (const void*)lin_group_kernel<KB, n, true, false>;
  s.nt = 64;
  s.bpw = 64 >> (n - KB);
  return s;
}

template <int KB, int n, int SGT>
LinShape sg_form(const void* fn, bool vjp) {
  constexpr int tpb = (1 << (n - 2 * KB)) / SGT;
  LinShape s;
  s.fn = fn;
  s.nt = lin::sg_threads(n, KB, SGT);
  s.bpw = tpb > 64 ? 1 : 64 / tpb;
  s.lds = lin::sg_lds(n, KB, SGT, vjp);
  return s;
}

// SGT super-groups per lane, with dCodebook SDC
template <int KB, int n, int SGT, int SDC = SGT>
LinShape sg_shape(bool vjp, bool dc) {
  if (!vjp) return sg_form<KB, n, SGT>((const void*)lin_sg_kernel<KB, n, SGT, false, false>, false);
  if (!dc) return sg_form<KB, n, SGT>((const void*)lin_sg_kernel<KB, n, SGT, true, false>, true);
  return sg_form<KB, n, SDC>((const void*)lin_sg_kernel<KB, n, SDC, true, true>, true);
}

}  // namespace

// The state bits are compiled in (every LDS and history offset folds into its
// instruction).  One lane per group while a block's groups fit one wave;
// above, 16 states per lane (64 at k = 3), more where the block would need
// over 512 threads.
LinShape lin_shape(int n, int k, bool vjp, bool dc) {
  switch (16 * k + n) {
    case 16 + 2: return group_shape<1, 2>(vjp, dc);
    case 16 + 3: return group_shape<1, 3>(vjp, dc);
    case 16 + 4: return group_shape<1, 4>(vjp, dc);
    case 16 + 5: return group_shape<1, 5>(vjp, dc);
    case 16 + 6: return group_shape<1, 6>(vjp, dc);
    case 16 + 7: return group_shape<1, 7>(vjp, dc);
    case 16 + 8: return sg_shape<1, 8, 4>(vjp, dc);
    case 16 + 9: return sg_shape<1, 9, 4>(vjp, dc);
    case 16 + 10: return sg_shape<1, 10, 4>(vjp, dc);
    case 16 + 11: return sg_shape<1, 11, 4>(vjp, dc);
    case 16 + 12: return sg_shape<1, 12, 4>(vjp, dc);
    case 16 + 13: return sg_shape<1, 13, 4>(vjp, dc);
    case 16 + 14: return sg_shape<1, 14, 8>(vjp, dc);
    case 32 + 4: return group_shape<2, 4>(vjp, dc);
    case 32 + 5: return group_shape<2, 5>(vjp, dc);
    case 32 + 6: return group_shape<2, 6>(vjp, dc);
    case 32 + 7: return group_shape<2, 7>(vjp, dc);
    case 32 + 8: return group_shape<2, 8>(vjp, dc);
    case 32 + 9: return sg_shape<2, 9, 1>(vjp, dc);
    case 32 + 10: return sg_shape<2, 10, 1>(vjp, dc);
    case 32 + 11: return sg_shape<2, 11, 1>(vjp, dc);
    case 32 + 12: return sg_shape<2, 12, 1>(vjp, dc);
    case 32 + 13: return sg_shape<2, 13, 1>(vjp, dc);
    case 32 + 14: return sg_shape<2, 14, 2, 1>(vjp, dc);
    case 32 + 15: return sg_shape<2, 15, 4>(vjp, dc);
    case 48 + 6: return group_shape<3, 6>(vjp, dc);
    case 48 + 7: return group_shape<3, 7>(vjp, dc);
    case 48 + 8: return group_shape<3, 8>(vjp, dc);
    case 48 + 9: return group_shape<3, 9>(vjp, dc);
    case 48 + 10: return sg_shape<3, 10, 1>(vjp, dc);
    case 48 + 11: return sg_shape<3, 11, 1>(vjp, dc);
    case 48 + 12: return sg_shape<3, 12, 1>(vjp, dc);
    case 48 + 13: return sg_shape<3, 13, 1>(vjp, dc);
    case 48 + 14: return sg_shape<3, 14, 1>(vjp, dc);
    default: return LinShape();
  }
}

// 0 on success, -1 when the launch reports a HIP error
int lin_launch(const LinShape& s, unsigned grid, hipStream_t stream, LinArgs a) {
  void* args[] = {&a};
  if (hipLaunchKernel(s.fn, dim3(grid), dim3(s.nt), args, s.lds, stream) != hipSuccess) return -1;
  return hipGetLastError() == hipSuccess ? 0 : -1;
}

}  // namespace bcjr
