// Resident sweep kernels (les_resident.h): FP32, medium boxes.
#include "les_resident.h"

namespace lesmi {
namespace resident {

LES_RESIDENT(Shapes<float>::M2, true, true)
LES_RESIDENT(Shapes<float>::M2, true, false)
LES_RESIDENT(Shapes<float>::M2, false, true)
LES_RESIDENT(Shapes<float>::M2, false, false)
LES_RESIDENT(Shapes<float>::M3Rag, true, true)
LES_RESIDENT(Shapes<float>::M3, true, false)

}  // namespace resident
}  // namespace lesmi
