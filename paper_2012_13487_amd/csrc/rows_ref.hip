// Row kernels of the reference form (rows_kernel.hpp).
#include "rows_kernel.hpp"

namespace dgbgk {

hipError_t launch_rows32_plain(int p, int kind, const RowArgs<float> &a, size_t lds, hipStream_t st);
hipError_t launch_batch_rows32_plain(int p, int stage, const RowArgs<float> *descs, const int2 *items,
                                     int nitems, size_t lds, hipStream_t st);

hipError_t launch_rows32(int p, int kind, int ref, const RowArgs<float> &a, size_t lds, hipStream_t st) {
  using namespace rows;
  if (!ref) return launch_rows32_plain(p, kind, a, lds, st);
  if (!a.rref || !a.mref) return hipErrorInvalidValue;
  switch (p) {
    case 1: return launch_kind<1, float, true>(kind, a, lds, st);
    case 2: return launch_kind<2, float, true>(kind, a, lds, st);
    case 3: return launch_kind<3, float, true>(kind, a, lds, st);
    case 4: return launch_kind<4, float, true>(kind, a, lds, st);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_batch_rows32(int p, int ref, int stage, const RowArgs<float> *descs, const int2 *items,
                               int nitems, size_t lds, hipStream_t st) {
  if (nitems <= 0) return hipSuccess;
  if (!ref) return launch_batch_rows32_plain(p, stage, descs, items, nitems, lds, st);
  return rows::launch_batch_any<float, true>(p, stage, descs, items, nitems, lds, st);
}

}  // namespace dgbgk
