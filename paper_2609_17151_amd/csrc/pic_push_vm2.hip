// Push kernels that carry the velocity components x and z.
#define PIC_PUSH_VM 2
#include "pic_push_inst.h"
