// The instances of gemm_bf16_resident.h for more than 128 columns (a source of their own: they compile side by side).
#include "gemm_bf16_resident.h"

namespace cofree {

bool launch_resident_wide(int nb, int nch, int end, dim3 grid, hipStream_t stream, const ResidentK& p) {
  switch (nb) {
    case 5: return launch_resident_pieces<5, 6>(nch, end, grid, stream, p);
    case 6: return launch_resident_pieces<6, 5>(nch, end, grid, stream, p);
    case 7: return launch_resident_pieces<7, 4>(nch, end, grid, stream, p);
    case 8: return launch_resident_pieces<8, 4>(nch, end, grid, stream, p);
    default: return false;
  }
}

}  // namespace cofree
