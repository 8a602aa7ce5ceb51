// Push kernels that carry the velocity components x, y and z.
#define PIC_PUSH_VM 3
#include "pic_push_inst.h"
