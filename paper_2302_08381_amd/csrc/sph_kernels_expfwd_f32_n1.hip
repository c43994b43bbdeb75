// compile-time radial expansion, float, normalised harmonics
#define SPH_T float
#define SPH_SUFFIX f32
#define SPH_NORM 1
#include "sph_expfwd_instances.inl"
