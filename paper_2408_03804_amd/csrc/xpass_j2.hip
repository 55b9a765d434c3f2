// x passes of J2 plasticity.
#define FH_XPASS xpass_j2
#define FH_XPASS_LAWS(X) X(6, MAT_J2, 2) X(7, MAT_J2, 3)
#include "xpass_law.h"
