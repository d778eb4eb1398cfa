// bca_block_f16.hip -- the matrix-core layer kernels of bca_block_kernels.hpp for StoreF16 rows.
#include "bca_block_kernels.hpp"

namespace rdfft {

BcaBlockTables bca_block_tables_f16() { return make_block_tables<StoreF16>(std::make_integer_sequence<int, kBlockPlans>{}); }

}  // namespace rdfft
