// Resident sweep kernels (les_resident.h): FP64, one-row boxes.
#include "les_resident.h"

namespace lesmi {
namespace resident {

LES_RESIDENT(Shapes<double>::RowL, true, true)
LES_RESIDENT(Shapes<double>::RowL, true, false)
LES_RESIDENT(Shapes<double>::RowL, false, true)
LES_RESIDENT(Shapes<double>::RowL, false, false)
LES_RESIDENT(Shapes<double>::RowS, true, true)
LES_RESIDENT(Shapes<double>::RowS, true, false)
LES_RESIDENT(Shapes<double>::RowS, false, true)
LES_RESIDENT(Shapes<double>::RowS, false, false)

}  // namespace resident
}  // namespace lesmi
