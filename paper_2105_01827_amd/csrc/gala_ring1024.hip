// The kernels of gala_ring_impl.h for rings of 1024 slots.
#define GALA_LOGN 10
#include "gala_ring_impl.h"
