// Resident sweep kernels (les_resident.h): FP64, medium and small boxes.
#include "les_resident.h"

namespace lesmi {
namespace resident {

LES_RESIDENT(Shapes<double>::M, true, true)
LES_RESIDENT(Shapes<double>::M, true, false)
LES_RESIDENT(Shapes<double>::M, false, true)
LES_RESIDENT(Shapes<double>::M, false, false)
LES_RESIDENT(Shapes<double>::S, true, true)
LES_RESIDENT(Shapes<double>::S, true, false)
LES_RESIDENT(Shapes<double>::S, false, true)
LES_RESIDENT(Shapes<double>::S, false, false)

}  // namespace resident
}  // namespace lesmi
