// The mixed-radix passes of FP32 grids, plans without prime stages.
#define EIFE_T float
#define EIFE_PRIME false
#include "eife_mix_launch.hpp"
