// Part 4 of rda_kernels.inl: turn-free strips and half-storage kernels.
#define SAR_PART 4
#include "rda_kernels.inl"
