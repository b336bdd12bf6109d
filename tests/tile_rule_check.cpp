// C entry point to default_tile_elems of csrc/sw_layout.h for
// tests/test_tile_rule.py.
#include "sw_layout.h"

extern "C" int tile_elems(long long n_tets) { return sw::default_tile_elems(n_tets); }
