// Resident sweep kernels (les_resident.h): FP32, one-row boxes.
#include "les_resident.h"

namespace lesmi {
namespace resident {

LES_RESIDENT(Shapes<float>::RowL, true, true)
LES_RESIDENT(Shapes<float>::RowL, true, false)
LES_RESIDENT(Shapes<float>::RowL, false, true)
LES_RESIDENT(Shapes<float>::RowL, false, false)
LES_RESIDENT(Shapes<float>::RowS, true, true)
LES_RESIDENT(Shapes<float>::RowS, true, false)
LES_RESIDENT(Shapes<float>::RowS, false, true)
LES_RESIDENT(Shapes<float>::RowS, false, false)

}  // namespace resident
}  // namespace lesmi
