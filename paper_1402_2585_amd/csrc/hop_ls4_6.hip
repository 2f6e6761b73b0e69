// The hop stage for Ls = 4 and 6.
#include "hop_ls.h"

namespace hdk {
HDCG_HOP_SPLIT(4)
HDCG_HOP_SPLIT(6)
}  // namespace hdk
