// Dispatch of the general kernels that are built per block shape (pbz_brick.h): the parts are asked in turn.
#include "pbz_brick.h"

namespace pbz {

int try_compress_brick(const pbz_codec* c, const Geom& g, const DeviceTables* t, const void* x, int xtype, void* N, void* F,
                       hipStream_t s, bool dry_run) {
  int r = 0;
#define PBZ_ASK(PART) if (r == 0) r = brick::PART##_compress(c, g, t, x, xtype, N, F, s, dry_run);
  PBZ_BRICK_PARTS(PBZ_ASK)
#undef PBZ_ASK
  return r;
}

int try_decompress_brick(const pbz_codec* c, const Geom& g, const DeviceTables* t, const void* N, const void* F, void* y,
                         int ytype, hipStream_t s, bool dry_run) {
  int r = 0;
#define PBZ_ASK(PART) if (r == 0) r = brick::PART##_decompress(c, g, t, N, F, y, ytype, s, dry_run);
  PBZ_BRICK_PARTS(PBZ_ASK)
#undef PBZ_ASK
  return r;
}

}  // namespace pbz
