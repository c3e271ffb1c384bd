// Cluster kernels instantiated for double iterations, MODE_GROUND.
#include "lrh_device.h"

namespace lrh {
template hipError_t launch_cluster_mode<double, false, MODE_GROUND>(const ClusterArgs<double>&, int, int, hipStream_t);
template hipError_t launch_cluster_mode<double, true, MODE_GROUND>(const ClusterArgs<double>&, int, int, hipStream_t);
template hipError_t launch_lds8_pair<double, false, MODE_GROUND>(const ClusterArgs<double>&, const ClusterArgs<double>&,
    const ClusterArgs<double>&, int, hipStream_t);
template hipError_t launch_lds8_pair<double, true, MODE_GROUND>(const ClusterArgs<double>&, const ClusterArgs<double>&,
    const ClusterArgs<double>&, int, hipStream_t);
}  // namespace lrh
