// The strip form of the split members, all its instantiations.
#include "wpk_strip.h"
