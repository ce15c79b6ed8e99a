// Column-kernel instances of the first iteration of a sparse call: element type float.
#define MAM_INST_T float
#define MAM_INST_KC -1
#include "mam_sparse.hpp"
#include "mam_instances.hpp"
