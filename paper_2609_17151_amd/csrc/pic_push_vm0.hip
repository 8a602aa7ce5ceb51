// Push kernels that carry the velocity components x only.
#define PIC_PUSH_VM 0
#include "pic_push_inst.h"
