// Block shapes of pbz_brick.h, a translation unit of their own.
#include "pbz_brick.h"

namespace pbz {
namespace brick {

#define PBZ_SHAPES(X) X(1, 1, 8, 8) X(1, 1, 8, 16) X(1, 1, 16, 8)
PBZ_DEFINE_BRICK_PART(flat, PBZ_SHAPES)

}  // namespace brick
}  // namespace pbz
