// Included before the runtime's sources when they are built for the CPU with
// the test doubles of fake_hip.cpp in place of the HIP runtime and the kernels.
#pragma once
#define __align__(n) __attribute__((aligned(n)))
#define HIP_SYMBOL(x) ((const void *)&(x))
