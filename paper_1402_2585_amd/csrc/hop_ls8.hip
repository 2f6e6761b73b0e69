// The hop stage for Ls = 8.
#include "hop_ls.h"

namespace hdk {
HDCG_HOP_SPLIT(8)
HDCG_HOP_MARCH(8)
}  // namespace hdk
