// Column-kernel instances of the first iteration of a sparse call: element type double.
#define MAM_INST_T double
#define MAM_INST_KC -1
#include "mam_sparse.hpp"
#include "mam_instances.hpp"
