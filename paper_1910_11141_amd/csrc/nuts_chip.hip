// Instances of the chip kernel.
#include "nuts_chip.h"

namespace nuts {

void chip_lds(int mt, int max_depth, ChipPlan* cp)
{
    switch (mt) {
    case 1: return chip_lds_inst<1>(max_depth, cp);
    case 2: return chip_lds_inst<2>(max_depth, cp);
    case 3: return chip_lds_inst<3>(max_depth, cp);
    case 4: return chip_lds_inst<4>(max_depth, cp);
    case 5: return chip_lds_inst<5>(max_depth, cp);
    case 6: return chip_lds_inst<6>(max_depth, cp);
    case 7: return chip_lds_inst<7>(max_depth, cp);
    default: return chip_lds_inst<8>(max_depth, cp);
    }
}

hipError_t chip_launch(int mt, const ChipArgs& ca, const DevSample& sa, const ChipPlan& cp, hipStream_t stream)
{
    switch (mt) {
    case 1: return chip_launch_inst<1>(ca, sa, cp, stream);
    case 2: return chip_launch_inst<2>(ca, sa, cp, stream);
    case 3: return chip_launch_inst<3>(ca, sa, cp, stream);
    case 4: return chip_launch_inst<4>(ca, sa, cp, stream);
    case 5: return chip_launch_inst<5>(ca, sa, cp, stream);
    case 6: return chip_launch_inst<6>(ca, sa, cp, stream);
    case 7: return chip_launch_inst<7>(ca, sa, cp, stream);
    default: return chip_launch_inst<8>(ca, sa, cp, stream);
    }
}

}  // namespace nuts
