// The specialised passes of FP64 grids.
#define EIFE_T double
#include "eife_special.hpp"
