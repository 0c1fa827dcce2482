// Resident sweep kernels (les_resident.h): FP64, medium boxes.
#include "les_resident.h"

namespace lesmi {
namespace resident {

LES_RESIDENT(Shapes<double>::M2, true, true)
LES_RESIDENT(Shapes<double>::M2, true, false)
LES_RESIDENT(Shapes<double>::M2, false, true)
LES_RESIDENT(Shapes<double>::M2, false, false)

}  // namespace resident
}  // namespace lesmi
