// Resident sweep kernels (les_resident.h): FP64, large boxes.
#include "les_resident.h"

namespace lesmi {
namespace resident {

LES_RESIDENT(Shapes<double>::M3Rag, true, true)
LES_RESIDENT(Shapes<double>::M3, true, false)

}  // namespace resident
}  // namespace lesmi
