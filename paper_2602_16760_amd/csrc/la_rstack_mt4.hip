// The register-streaming persistent kernel (la_rstack.h) for blocks of 49..64 rows (4 row tiles).
#include "la_rstack.h"
namespace la {
namespace rs {
template int launch_rstack_kernel<4, 4, false>(const StackArgs &, int, hipStream_t);
template int prepare_rstack_kernel<4, 4, false>(int, int);
template int launch_rstack_kernel<4, 4, true>(const StackArgs &, int, hipStream_t);
template int prepare_rstack_kernel<4, 4, true>(int, int);
}
}  // namespace la
