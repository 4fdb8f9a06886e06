// The kernels of gala_ring_impl.h for rings of 2048 slots.
#define GALA_LOGN 11
#include "gala_ring_impl.h"
