// Block shapes of pbz_brick.h, a translation unit of their own.
#include "pbz_brick.h"

namespace pbz {
namespace brick {

#define PBZ_SHAPES(X) X(2, 4, 8, 8) X(2, 2, 8, 8)
PBZ_DEFINE_BRICK_PART(long_tesseracts, PBZ_SHAPES)

}  // namespace brick
}  // namespace pbz
