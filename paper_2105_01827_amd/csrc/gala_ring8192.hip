// The kernels of gala_ring_impl.h for rings of 8192 slots.
#define GALA_LOGN 13
#include "gala_ring_impl.h"
