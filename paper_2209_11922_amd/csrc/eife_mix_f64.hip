// The mixed-radix passes of FP64 grids, plans without prime stages.
#define EIFE_T double
#define EIFE_PRIME false
#include "eife_mix_launch.hpp"
