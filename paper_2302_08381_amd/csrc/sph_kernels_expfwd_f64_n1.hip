// compile-time radial expansion, double, normalised harmonics
#define SPH_T double
#define SPH_SUFFIX f64
#define SPH_NORM 1
#include "sph_expfwd_instances.inl"
