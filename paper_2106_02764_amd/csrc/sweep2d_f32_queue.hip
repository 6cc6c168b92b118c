// The persistent 2D pass over every work item of a batch, float.
#include "sweep2d.h"

template hipError_t launch_queue2<float>(const GeomDev*, const Item*, int, int, PassParams, size_t, hipStream_t, int*);
