// The hop stage for Ls = 16.
#include "hop_ls.h"

namespace hdk {
HDCG_HOP_SPLIT(16)
HDCG_HOP_MARCH(16)
}  // namespace hdk
