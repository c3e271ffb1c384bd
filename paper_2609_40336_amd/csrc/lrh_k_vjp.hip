// Adjoint (Daleckii-Krein VJP) cluster kernels: launcher and instantiations.
#include "lrh_device.h"

namespace lrh {

hipError_t launch_cluster_vjp(const ClusterArgs<double>& a, bool cplx, int mode, hipStream_t s) {
  if (a.n == 0) return hipSuccess;
  const dim3 b(64);
  // lanes per cluster: one per column up to D = 16 (the eigensolver in registers), else a whole wave
#define VJP_LAUNCH(DE, CPLX, W)                                                                             \
  {                                                                                                         \
    const dim3 g((unsigned)((a.n + 64 / W - 1) / (64 / W)));                                                \
    if (mode == MODE_GIBBS) hipLaunchKernelGGL((k_cluster_vjp<double, CPLX, DE, MODE_GIBBS, W>), g, b, 0, s, a); \
    else hipLaunchKernelGGL((k_cluster_vjp<double, CPLX, DE, MODE_GROUND, W>), g, b, 0, s, a);              \
    return hipGetLastError();                                                                               \
  }
#define VJP_CASE(DE, W)                    \
  if (a.De == DE) {                        \
    if (cplx) VJP_LAUNCH(DE, true, W)      \
    else VJP_LAUNCH(DE, false, W)          \
  }
  VJP_CASE(2, 2)
  VJP_CASE(4, 4)
  VJP_CASE(8, 8)
  // Complex, up to a wave per SIMD of the chip, a wave per cluster with the solver in LDS: its products are
  // four times as wide, and the code of the solver in registers (15 000 instructions) does not fit the instruction
  // cache.  A call on two-level windows of 4 sites, us, beta = 0 / 3: 100 clusters 185 / 200 (16 lanes 211 /
  // 247), 1000 clusters 205 / 220 (237 / 272); 1400 clusters 287 / 301 (237 / 273).  Real, 16 lanes are the faster.
  if (a.De == 16 && cplx && a.n <= 1024) VJP_LAUNCH(16, true, 64)
  VJP_CASE(16, 16)
  VJP_CASE(32, 64)
  if (a.De == 64 && !cplx) VJP_LAUNCH(64, false, 64)
#undef VJP_CASE
#undef VJP_LAUNCH
  return hipErrorInvalidValue;
}

hipError_t launch_cluster_vjp_group(const ClusterArgs<double>& a8, const ClusterArgs<double>& a4,
                                    const ClusterArgs<double>& a2, bool cplx, int mode, hipStream_t s) {
  const int n8 = (int)((a8.n + 7) / 8), n4 = (int)((a4.n + 15) / 16), n2 = (int)((a2.n + 31) / 32);
  const dim3 g((unsigned)(n8 + n4 + n2)), b(64);
#define VJP_GROUP(CPLX, MODE) \
  hipLaunchKernelGGL((k_cluster_vjp_group<CPLX, MODE>), g, b, 0, s, a8, a4, a2, n8, n4, n2)
  if (cplx) {
    if (mode == MODE_GIBBS) VJP_GROUP(true, MODE_GIBBS);
    else VJP_GROUP(true, MODE_GROUND);
  } else {
    if (mode == MODE_GIBBS) VJP_GROUP(false, MODE_GIBBS);
    else VJP_GROUP(false, MODE_GROUND);
  }
#undef VJP_GROUP
  return hipGetLastError();
}

// blocks of launch_cluster_vjp_group that the 256 CUs hold at once, by their 160 KiB of LDS
int64_t vjp_group_resident(bool cplx) {
  return 256 * (163840 / (cplx ? vjp_group_lds<true>() : vjp_group_lds<false>()));
}

}  // namespace lrh
