// Instances of the LM-head tile kernel (several sources, compiled in parallel).
#include "lmhead_tile.h"

namespace al {

AL_LM_INSTANCE(5, 2)
AL_LM_INSTANCE(6, 6)
AL_LM_INSTANCE(8, 2)

}  // namespace al
