// Instances of the LM-head tile kernel (several sources, compiled in parallel).
#include "lmhead_tile.h"

namespace al {

AL_LM_INSTANCE(2, 8)
AL_LM_INSTANCE(2, 10)
AL_LM_INSTANCE(2, 13)
AL_LM_INSTANCE(4, 2)
AL_LM_INSTANCE(4, 4)

}  // namespace al
