// Resident sweep kernels (les_resident.h): FP32, small boxes.
#include "les_resident.h"

namespace lesmi {
namespace resident {

LES_RESIDENT(Shapes<float>::S, true, true)
LES_RESIDENT(Shapes<float>::S, true, false)
LES_RESIDENT(Shapes<float>::S, false, true)
LES_RESIDENT(Shapes<float>::S, false, false)
LES_RESIDENT(Shapes<float>::M1, true, true)
LES_RESIDENT(Shapes<float>::M1, true, false)
LES_RESIDENT(Shapes<float>::M1, false, true)
LES_RESIDENT(Shapes<float>::M1, false, false)

}  // namespace resident
}  // namespace lesmi
