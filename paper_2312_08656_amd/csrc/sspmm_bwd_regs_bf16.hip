#include "sspmm_bwd_regs_impl.hpp"

namespace maxk {
template maxk_status launch_regs_format<MAXK_VALUE_BF16>(const RegsSet&, const void*, const void*, int, int64_t, int, int, float*, hipStream_t);
}
