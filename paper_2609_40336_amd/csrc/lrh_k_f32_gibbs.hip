// Cluster kernels instantiated for float iterations, MODE_GIBBS.
#include "lrh_device.h"

namespace lrh {
template hipError_t launch_cluster_mode<float, false, MODE_GIBBS>(const ClusterArgs<float>&, int, int, hipStream_t);
template hipError_t launch_cluster_mode<float, true, MODE_GIBBS>(const ClusterArgs<float>&, int, int, hipStream_t);
template hipError_t launch_expm16_pair<float, false>(const ClusterArgs<float>&, const ClusterArgs<float>&,
                                                     const ClusterArgs<float>&, hipStream_t);
template hipError_t launch_expm16_pair<float, true>(const ClusterArgs<float>&, const ClusterArgs<float>&,
                                                    const ClusterArgs<float>&, hipStream_t);
template hipError_t launch_lds8_pair<float, false, MODE_GIBBS>(const ClusterArgs<float>&, const ClusterArgs<float>&,
    const ClusterArgs<float>&, int, hipStream_t);
template hipError_t launch_lds8_pair<float, true, MODE_GIBBS>(const ClusterArgs<float>&, const ClusterArgs<float>&,
    const ClusterArgs<float>&, int, hipStream_t);
}  // namespace lrh
