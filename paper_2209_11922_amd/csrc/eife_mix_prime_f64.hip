// The mixed-radix passes of FP64 grids, plans with prime stages.
#define EIFE_T double
#define EIFE_PRIME true
#include "eife_mix_launch.hpp"
