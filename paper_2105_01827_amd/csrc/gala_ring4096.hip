// The kernels of gala_ring_impl.h for rings of 4096 slots.
#define GALA_LOGN 12
#include "gala_ring_impl.h"
