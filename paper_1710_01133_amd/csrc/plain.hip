// K1 in double: the instantiations of plain_block.h for abm_solve and
// abm_solve_noalloc.
#include "plain_block.h"

namespace abm {

size_t plain_chain_lds(int d, bool per_comp, int64_t chunks, bool alone)
{
    return plainblk::chain_lds<double>(d, per_comp, chunks, alone);
}

int plain_worker_chunks(int d) { return plainblk::worker_chunks<double>(d); }

hipError_t launch_plain(const PlainArgs& A, int kind, hipStream_t st)
{
    return plainblk::launch_kind<double>(A, kind, st);
}

}  // namespace abm
