// The hop stage for the Ls <= 16 that have no file of their own (at run time).
#include "hop_ls.h"

namespace hdk {
HDCG_HOP_SPLIT(0)
}  // namespace hdk
