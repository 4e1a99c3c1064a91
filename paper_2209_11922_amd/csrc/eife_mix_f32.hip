// The mixed-radix passes of FP32 grids.
#define EIFE_T float
#include "eife_mix_launch.hpp"
