// Instances of the Gaussian kernels whose state fills the registers: quad, block, the largest of the band and element-wise
// kernels.  A translation unit of their own for the compiler flags that they are built with (build.py): constants and addresses
// are not hoisted out of the loops, where they would hold registers that the state then has to leave.  Same instructions on the same
// numbers, the same bits.  Time without the flags over time with: quad 1.01 to 1.05, block 1.01 to 1.24, band 1.13 to 2.9,
// element-wise (d = 2000, binary64) 1.4 to 1.7.  Kernels with room to spare are slower with them (tile 0.98, wide in
// binary32 0.95, dense 0.99, element-wise at d = 1000 0.94 to 0.98).
#include "nuts_band.h"
#include "nuts_block.h"
#include "nuts_elem.h"
#include "nuts_quad.h"

namespace nuts {

hipError_t quad_launch(const QuadArgs& qa, const DevSample& sa, int blocks, size_t lds_bytes, hipStream_t stream)
{
    switch (qa.n_r) {
    case 1: return quad_launch_inst<1>(qa, sa, blocks, lds_bytes, stream);
    case 2: return quad_launch_inst<2>(qa, sa, blocks, lds_bytes, stream);
    case 3: return quad_launch_inst<3>(qa, sa, blocks, lds_bytes, stream);
    case 4: return quad_launch_inst<4>(qa, sa, blocks, lds_bytes, stream);
    case 5: return quad_launch_inst<5>(qa, sa, blocks, lds_bytes, stream);
    case 6: return quad_launch_inst<6>(qa, sa, blocks, lds_bytes, stream);
    case 7: return quad_launch_inst<7>(qa, sa, blocks, lds_bytes, stream);
    default: return quad_launch_inst<8>(qa, sa, blocks, lds_bytes, stream);
    }
}

template hipError_t block_launch<float>(const BlockData&, const DevSample&, const BlockPlan&, hipStream_t);
template hipError_t block_launch<double>(const BlockData&, const DevSample&, const BlockPlan&, hipStream_t);

NUTS_BAND_INSTANCES()
NUTS_ELEM_INSTANCE(double, 16, false)

}  // namespace nuts
