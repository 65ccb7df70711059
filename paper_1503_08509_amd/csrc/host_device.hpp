// Functions compiled for the kernels and for the host.
#pragma once

#ifdef __HIPCC__
#define FEP3M_HOST_DEVICE __host__ __device__
#else
#define FEP3M_HOST_DEVICE
#endif
