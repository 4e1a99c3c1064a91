// The mixed-radix passes of FP32 grids, plans with prime stages.
#define EIFE_T float
#define EIFE_PRIME true
#include "eife_mix_launch.hpp"
