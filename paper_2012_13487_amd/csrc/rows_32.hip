// Row kernels of FP32 storage (rows_kernel.hpp).
#include "rows_kernel.hpp"

namespace dgbgk {

hipError_t launch_rows32_plain(int p, int kind, const RowArgs<float> &a, size_t lds, hipStream_t st) {
  using namespace rows;
  switch (p) {
    case 1: return launch_kind<1, float, false>(kind, a, lds, st);
    case 2: return launch_kind<2, float, false>(kind, a, lds, st);
    case 3: return launch_kind<3, float, false>(kind, a, lds, st);
    case 4: return launch_kind<4, float, false>(kind, a, lds, st);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_rows_sums32(int p, const RowArgs<float> &a, size_t lds, hipStream_t st) {
  using namespace rows;
  switch (p) {
    case 1: return launch_one<kKindSums, 1, float, 0, false>(a, lds, st);
    case 2: return launch_one<kKindSums, 2, float, 0, false>(a, lds, st);
    case 3: return launch_one<kKindSums, 3, float, 0, false>(a, lds, st);
    case 4: return launch_one<kKindSums, 4, float, 0, false>(a, lds, st);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_batch_rows32_plain(int p, int stage, const RowArgs<float> *descs, const int2 *items,
                                     int nitems, size_t lds, hipStream_t st) {
  if (nitems <= 0) return hipSuccess;
  return rows::launch_batch_any<float, false>(p, stage, descs, items, nitems, lds, st);
}

}  // namespace dgbgk
