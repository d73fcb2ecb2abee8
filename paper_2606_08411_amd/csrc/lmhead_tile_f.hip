// Instances of the LM-head tile kernel (several sources, compiled in parallel).
#include "lmhead_tile.h"

namespace al {

AL_LM_INSTANCE(4, 15)
AL_LM_INSTANCE(4, 16)

}  // namespace al
