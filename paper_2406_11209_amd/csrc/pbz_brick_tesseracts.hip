// Block shapes of pbz_brick.h, a translation unit of their own.
#include "pbz_brick.h"

namespace pbz {
namespace brick {

#define PBZ_SHAPES(X) X(2, 4, 4, 4) X(4, 4, 4, 4)
PBZ_DEFINE_BRICK_PART(tesseracts, PBZ_SHAPES)

}  // namespace brick
}  // namespace pbz
