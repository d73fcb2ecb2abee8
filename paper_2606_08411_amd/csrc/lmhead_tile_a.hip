// Instances of the LM-head tile kernel (several sources, compiled in parallel).
#include "lmhead_tile.h"

namespace al {

AL_LM_INSTANCE(1, 2)
AL_LM_INSTANCE(1, 4)
AL_LM_INSTANCE(1, 6)
AL_LM_INSTANCE(1, 10)
AL_LM_INSTANCE(2, 2)
AL_LM_INSTANCE(2, 4)
AL_LM_INSTANCE(2, 6)

}  // namespace al
