// The split kernel's instances for small calls (a team of waves per page range),
// compiled apart from the others; the kernel source is the same file.
#define OSCAR_SPLIT_TEAM_UNIT
#include "decode_mfma.hip"
