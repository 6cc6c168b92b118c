// 3D pass kernels, float, 1 and 2 cells per lane.
#include "sweep3d.h"

template hipError_t launch_sweep3<float, 1>(const GeomDev*, const Item*, int, int, PassParams, size_t, hipStream_t, int);
template hipError_t launch_sweep3<float, 2>(const GeomDev*, const Item*, int, int, PassParams, size_t, hipStream_t, int);
