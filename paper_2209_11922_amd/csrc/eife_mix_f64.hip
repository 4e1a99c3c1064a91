// The mixed-radix passes of FP64 grids.
#define EIFE_T double
#include "eife_mix_launch.hpp"
