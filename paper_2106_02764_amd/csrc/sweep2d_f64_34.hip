// 2D pass kernels, double, 3 and 4 cells per lane.
#include "sweep2d.h"

template hipError_t launch_sweep2<double, 3>(const GeomDev*, const Item*, int, int, PassParams, size_t, hipStream_t, int);
template hipError_t launch_sweep2<double, 4>(const GeomDev*, const Item*, int, int, PassParams, size_t, hipStream_t, int);
