// Cluster kernels instantiated for double iterations, MODE_GIBBS.
#include "lrh_device.h"

namespace lrh {
template hipError_t launch_cluster_mode<double, false, MODE_GIBBS>(const ClusterArgs<double>&, int, int, hipStream_t);
template hipError_t launch_cluster_mode<double, true, MODE_GIBBS>(const ClusterArgs<double>&, int, int, hipStream_t);
template hipError_t launch_lds8_pair<double, false, MODE_GIBBS>(const ClusterArgs<double>&, const ClusterArgs<double>&,
    const ClusterArgs<double>&, int, hipStream_t);
template hipError_t launch_lds8_pair<double, true, MODE_GIBBS>(const ClusterArgs<double>&, const ClusterArgs<double>&,
    const ClusterArgs<double>&, int, hipStream_t);
}  // namespace lrh
