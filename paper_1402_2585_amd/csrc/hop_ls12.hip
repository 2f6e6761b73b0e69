// The hop stage for Ls = 12.
#include "hop_ls.h"

namespace hdk {
HDCG_HOP_SPLIT(12)
HDCG_HOP_MARCH(12)
}  // namespace hdk
