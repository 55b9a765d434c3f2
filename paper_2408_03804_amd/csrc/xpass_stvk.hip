// x passes of the St. Venant-Kirchhoff law.
#define FH_XPASS xpass_stvk
#define FH_XPASS_LAWS(X) X(4, MAT_STVK, 2) X(5, MAT_STVK, 3)
#include "xpass_law.h"
