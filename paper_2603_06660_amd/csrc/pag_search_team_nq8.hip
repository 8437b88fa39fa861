// Instantiations of the search kernel with several waves per query, 8 chunks of a stored vector per lane.
#include "pag_search_kernel.h"

PAG_SEARCH_TEAM_INSTANCES(8)
