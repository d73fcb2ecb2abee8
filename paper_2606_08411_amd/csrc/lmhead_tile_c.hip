// Instances of the LM-head tile kernel (several sources, compiled in parallel).
#include "lmhead_tile.h"

namespace al {

AL_LM_INSTANCE(4, 6)
AL_LM_INSTANCE(4, 8)
AL_LM_INSTANCE(4, 9)
AL_LM_INSTANCE(4, 10)

}  // namespace al
