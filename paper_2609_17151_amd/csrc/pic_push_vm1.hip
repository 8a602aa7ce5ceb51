// Push kernels that carry the velocity components x and y.
#define PIC_PUSH_VM 1
#include "pic_push_inst.h"
