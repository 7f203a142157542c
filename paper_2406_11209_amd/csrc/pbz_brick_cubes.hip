// Block shapes of pbz_brick.h, a translation unit of their own.
#include "pbz_brick.h"

namespace pbz {
namespace brick {

#define PBZ_SHAPES(X) X(1, 4, 4, 4) X(1, 8, 8, 8) X(2, 2, 4, 4)
PBZ_DEFINE_BRICK_PART(cubes, PBZ_SHAPES)

}  // namespace brick
}  // namespace pbz
