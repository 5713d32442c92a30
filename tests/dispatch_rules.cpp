// Which kernels a table of sizes takes: the library's rules (lamb_internal.h)
// at sizes on both sides of their lines, checked at compile time.
#include "lamb_internal.h"

using namespace lamb_mi355x;

// Finalize: one kernel whose workgroups hold no more teams than the widest
// tensor has segments; two for a wide tensor, or where teams would idle on many
// narrow ones.
static_assert(direct_teams(1, 1) == 1 && direct_teams(40000, 1) == 1, "tensors of one segment");
static_assert(direct_teams(161, 5) == 4 && direct_teams(391, 8) == 4, "ResNet-50, BERT-Large / 8");
static_assert(direct_teams(1280, 2) == 2 && direct_teams(1281, 2) == 0, "idle teams");
static_assert(direct_teams(426, 4) == 4 && direct_teams(427, 4) == 0, "idle teams");
static_assert(direct_teams(4096, 4) == 0 && direct_teams(1, 9) == 0, "many tensors, a wide one");

int main() { return 0; }
