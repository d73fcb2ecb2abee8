// Instances of the LM-head tile kernel (several sources, compiled in parallel).
#include "lmhead_tile.h"

namespace al {

AL_LM_INSTANCE(5, 4)
AL_LM_INSTANCE(5, 6)
AL_LM_INSTANCE(5, 8)
AL_LM_INSTANCE(5, 9)
AL_LM_INSTANCE(5, 10)

}  // namespace al
