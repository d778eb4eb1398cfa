// bca_block_bf16.hip -- the matrix-core layer kernels of bca_block_kernels.hpp for StoreBF16 rows.
#include "bca_block_kernels.hpp"

namespace rdfft {

BcaBlockTables bca_block_tables_bf16() { return make_block_tables<StoreBF16>(std::make_integer_sequence<int, kBlockPlans>{}); }

}  // namespace rdfft
