// Resident sweep kernels (les_resident.h): FP32, medium and small boxes.
#include "les_resident.h"

namespace lesmi {
namespace resident {

LES_RESIDENT(Shapes<float>::M, true, true)
LES_RESIDENT(Shapes<float>::M, true, false)
LES_RESIDENT(Shapes<float>::M, false, true)
LES_RESIDENT(Shapes<float>::M, false, false)
LES_RESIDENT(Shapes<float>::S, true, true)
LES_RESIDENT(Shapes<float>::S, true, false)
LES_RESIDENT(Shapes<float>::S, false, true)
LES_RESIDENT(Shapes<float>::S, false, false)

}  // namespace resident
}  // namespace lesmi
