// compile-time radial expansion, float, scaled harmonics
#define SPH_T float
#define SPH_SUFFIX f32
#define SPH_NORM 0
#include "sph_expfwd_instances.inl"
