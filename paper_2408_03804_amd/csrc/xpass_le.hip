// x passes of linear elasticity.
#define FH_XPASS xpass_le
#define FH_XPASS_LAWS(X) X(0, MAT_LE, 2) X(1, MAT_LE, 3)
#include "xpass_law.h"
