// One size class of the wave engine (SFRDE_PART, set by the build).
#include "wave_parts.h"
