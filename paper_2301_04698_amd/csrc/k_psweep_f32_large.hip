// Resident sweep kernels (les_resident.h): FP32, large boxes.
#include "les_resident.h"

namespace lesmi {
namespace resident {

LES_RESIDENT(Shapes<float>::L, true, true)
LES_RESIDENT(Shapes<float>::L, true, false)

}  // namespace resident
}  // namespace lesmi
