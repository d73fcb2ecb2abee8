// Instances of the LM-head tile kernel (several sources, compiled in parallel).
#include "lmhead_tile.h"

namespace al {

AL_LM_INSTANCE(5, 11)
AL_LM_INSTANCE(5, 12)
AL_LM_INSTANCE(5, 13)

}  // namespace al
