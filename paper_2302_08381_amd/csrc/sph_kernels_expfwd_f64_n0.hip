// compile-time radial expansion, double, scaled harmonics
#define SPH_T double
#define SPH_SUFFIX f64
#define SPH_NORM 0
#include "sph_expfwd_instances.inl"
