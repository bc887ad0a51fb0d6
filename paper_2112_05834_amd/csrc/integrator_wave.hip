// The integrator's variants with one cell per wave (G = 64), as a unit of their
// own: they are compiled with other options than those with several cells per
// wave (the reason and both sides' times stand at the variants' list).
#define CHEM_WAVE_UNIT
#include "integrator.hip"
