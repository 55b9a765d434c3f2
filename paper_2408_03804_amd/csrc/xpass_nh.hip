// x passes of the Neo-Hookean law.
#define FH_XPASS xpass_nh
#define FH_XPASS_LAWS(X) X(2, MAT_NH, 2) X(3, MAT_NH, 3)
#include "xpass_law.h"
