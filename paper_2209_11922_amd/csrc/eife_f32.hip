// The specialised passes of FP32 grids.
#define EIFE_T float
#include "eife_special.hpp"
