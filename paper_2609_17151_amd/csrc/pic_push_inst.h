// The push kernels of one set of velocity components (PIC_PUSH_VM), with their
// launch and occupancy: one source file per set, so that they compile side by
// side.
#include "pic_push_kernel.h"

namespace pic {

#define PIC_KERNELS(X)        \
    X(1, 256, false, false)   \
    X(2, 256, false, false)   \
    X(4, 256, false, false)   \
    X(8, 256, false, false)   \
    X(4, 512, false, false)   \
    X(4, 1024, false, false)  \
    X(1, 256, true, false)    \
    X(2, 256, true, false)    \
    X(4, 256, true, false)    \
    X(4, 512, true, false)    \
    X(4, 1024, true, false)   \
    X(8, 256, true, false)    \
    X(8, 512, true, false)    \
    X(1, 256, true, true)     \
    X(2, 256, true, true)     \
    X(4, 256, true, true)

template <>
hipError_t launch_push_vm<PIC_PUSH_VM>(const PushArgs& a, int ppt, int threads, bool general, bool fuse, int64_t grid,
                                       hipStream_t st)
{
    const size_t lds = push_lds_bytes(a.nodes_max_dyn, a.cells_max_dyn, a.diag);
    const dim3 g((unsigned)grid);
#define PIC_LAUNCH(P, B, G, F)                                                                       \
    if (ppt == P && threads == B && general == G && fuse == F) {                                     \
        if (a.diag) hipLaunchKernelGGL((push_kernel<P, B, G, F, PIC_PUSH_VM, true, false>), g, dim3(B), lds, st, a); \
        else if (!G && a.acc_in)                                                                             \
            hipLaunchKernelGGL((push_kernel<P, B, G, F, PIC_PUSH_VM, false, !G>), g, dim3(B), lds, st, a);    \
        else hipLaunchKernelGGL((push_kernel<P, B, G, F, PIC_PUSH_VM, false, false>), g, dim3(B), lds, st, a); \
        return hipGetLastError();                                                                    \
    }
    PIC_KERNELS(PIC_LAUNCH)
#undef PIC_LAUNCH
    return hipErrorInvalidValue;
}

template <>
int push_occupancy_vm<PIC_PUSH_VM>(int ppt, int threads, bool general, bool fuse, bool diag, size_t lds)
{
    int nb = 0;
#define PIC_OCC(P, B, G, F)                                                                                  \
    if (ppt == P && threads == B && general == G && fuse == F) {                                             \
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(                                                    \
                &nb,                                                                                         \
                diag ? reinterpret_cast<const void*>(push_kernel<P, B, G, F, PIC_PUSH_VM, true, false>)      \
                     : reinterpret_cast<const void*>(push_kernel<P, B, G, F, PIC_PUSH_VM, false, !G>),       \
                B, lds) != hipSuccess)                                                                       \
            nb = 0;                                                                                          \
    }
    PIC_KERNELS(PIC_OCC)
#undef PIC_OCC
    return nb > 0 ? nb : 1;
}

}  // namespace pic
