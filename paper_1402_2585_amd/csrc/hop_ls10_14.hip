// The hop stage for Ls = 10 and 14.
#include "hop_ls.h"

namespace hdk {
HDCG_HOP_SPLIT(10)
HDCG_HOP_SPLIT(14)
}  // namespace hdk
