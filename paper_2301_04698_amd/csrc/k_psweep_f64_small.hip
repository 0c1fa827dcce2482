// Resident sweep kernels (les_resident.h): FP64, small boxes.
#include "les_resident.h"

namespace lesmi {
namespace resident {

LES_RESIDENT(Shapes<double>::S, true, true)
LES_RESIDENT(Shapes<double>::S, true, false)
LES_RESIDENT(Shapes<double>::S, false, true)
LES_RESIDENT(Shapes<double>::S, false, false)
LES_RESIDENT(Shapes<double>::M1, true, true)
LES_RESIDENT(Shapes<double>::M1, true, false)
LES_RESIDENT(Shapes<double>::M1, false, true)
LES_RESIDENT(Shapes<double>::M1, false, false)

}  // namespace resident
}  // namespace lesmi
