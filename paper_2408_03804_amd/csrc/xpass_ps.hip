// x passes of the laws with their own plane-stress form.
#define FH_XPASS xpass_ps
#define FH_XPASS_LAWS(X) X(8, MAT_NH_PS, 2) X(9, MAT_J2_PS, 2)
#include "xpass_law.h"
