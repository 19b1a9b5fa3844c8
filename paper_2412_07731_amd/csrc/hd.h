// AHLP_HD marks functions of the device code that are plain C++ as well, so that a host
// program can check them.
#pragma once

#if defined(__HIPCC__)
#define AHLP_HD __host__ __device__ inline
#else
#define AHLP_HD inline
#endif
