// The register-streaming persistent kernel (la_rstack.h) for blocks of 33..48 rows (3 row tiles).
#include "la_rstack.h"
namespace la {
namespace rs {
template int launch_rstack_kernel<3, 4, false>(const StackArgs &, int, hipStream_t);
template int prepare_rstack_kernel<3, 4, false>(int, int);
template int launch_rstack_kernel<3, 4, true>(const StackArgs &, int, hipStream_t);
template int prepare_rstack_kernel<3, 4, true>(int, int);
}
}  // namespace la
