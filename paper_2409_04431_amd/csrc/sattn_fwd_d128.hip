// Forward bf16 kernels for head dimension 128.
#include "sattn_fwd_launch.hpp"
#include "sattn_fwd_short.hpp"

template int sattn::launch_fwd_bf16<128>(sattn::FwdParams, int, int, bool, bool, int, bool, hipStream_t);
template int sattn::launch_fwd_few<128>(sattn::FwdParams, int, bool, hipStream_t);
template int sattn::launch_fwd_short<128>(const sattn::FwdParams&, int, hipStream_t);
