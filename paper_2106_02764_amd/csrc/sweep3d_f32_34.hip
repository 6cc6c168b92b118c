// 3D pass kernels, float, 3 and 4 cells per lane.
#include "sweep3d.h"

template hipError_t launch_sweep3<float, 3>(const GeomDev*, const Item*, int, int, PassParams, size_t, hipStream_t, int);
template hipError_t launch_sweep3<float, 4>(const GeomDev*, const Item*, int, int, PassParams, size_t, hipStream_t, int);
