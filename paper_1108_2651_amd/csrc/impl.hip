// impl.hip -- instantiations of the kernel dispatch.  The build compiles this
// file once per unit (LBEM_UNIT), the units in parallel.
#include "impl.h"

#if LBEM_UNIT == 0
Impl* make_plain2d(int prec)
{
    switch (prec) {
        case LBEM_F64: return new (std::nothrow) PlainImpl<2, double>();
        case LBEM_F32: return new (std::nothrow) PlainImpl<2, float>();
        default: return new (std::nothrow) PlainImpl<2, float, __half>();
    }
}
#elif LBEM_UNIT == 1
Impl* make_dev2d(int prec)
{
    switch (prec) {
        case LBEM_F16DEV: return new (std::nothrow) DevImpl<2, __half, false>();
        case LBEM_BF16DEV: return new (std::nothrow) DevImpl<2, __hip_bfloat16, false>();
        case LBEM_F16GHOST: return new (std::nothrow) DevImpl<2, __half, true>();
        default: return new (std::nothrow) DevImpl<2, __hip_bfloat16, true>();
    }
}
#elif LBEM_UNIT == 2
Impl* make_plain3d(int prec)
{
    switch (prec) {
        case LBEM_F64: return new (std::nothrow) PlainImpl<3, double>();
        case LBEM_F32: return new (std::nothrow) PlainImpl<3, float>();
        default: return new (std::nothrow) PlainImpl<3, float, __half>();
    }
}
#elif LBEM_UNIT == 3
Impl* make_dev3d_f16(int prec)
{
    if (prec == LBEM_F16DEV) return new (std::nothrow) DevImpl<3, __half, false>();
    return new (std::nothrow) DevImpl<3, __half, true>();
}
#elif LBEM_UNIT == 4
Impl* make_dev3d_bf16(int prec)
{
    if (prec == LBEM_BF16DEV) return new (std::nothrow) DevImpl<3, __hip_bfloat16, false>();
    return new (std::nothrow) DevImpl<3, __hip_bfloat16, true>();
}
#else
#error "LBEM_UNIT names no unit"
#endif
