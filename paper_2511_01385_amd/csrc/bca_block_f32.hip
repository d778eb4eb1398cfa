// bca_block_f32.hip -- the matrix-core layer kernels of bca_block_kernels.hpp for StoreF32 rows.
#include "bca_block_kernels.hpp"

namespace rdfft {

BcaBlockTables bca_block_tables_f32() { return make_block_tables<StoreF32>(std::make_integer_sequence<int, kBlockPlans>{}); }

}  // namespace rdfft
