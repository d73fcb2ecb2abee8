// Instances of the LM-head tile kernel (several sources, compiled in parallel).
#include "lmhead_tile.h"

namespace al {

AL_LM_INSTANCE(4, 11)
AL_LM_INSTANCE(4, 12)

}  // namespace al
