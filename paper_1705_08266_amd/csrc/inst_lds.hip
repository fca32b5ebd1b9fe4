// Kernel instantiations: the exchange ablation (every neighbour exchange
// through LDS), FP32 level kernels.
#include "dwt2_table.hpp"

namespace dwt2 {
namespace {

template <int WV, int SCH, int T>
hipError_t launch_fwd_lds(const FwdParams &p, hipStream_t s) {
    return launch_fwd<WV, SCH, T, float, float, float>(p, s);
}
template <int WV, int SCH, int T>
hipError_t launch_inv_lds(const InvParams &p, hipStream_t s) {
    return launch_inv<WV, SCH, T, float, float, float>(p, s);
}
template <int WV, int SCH, int... I>
constexpr std::array<FwdLauncher, kNumTiles> fwd_lds_tiles(std::integer_sequence<int, I...>) {
    return {&launch_fwd_lds<WV, SCH, I>...};
}
template <int WV, int SCH, int... I>
constexpr std::array<InvLauncher, kNumTiles> inv_lds_tiles(std::integer_sequence<int, I...>) {
    return {&launch_inv_lds<WV, SCH, I>...};
}
constexpr FwdLdsTable make_fwd_lds_table() {
    using S = std::make_integer_sequence<int, kNumTiles>;
    return {{{fwd_lds_tiles<CDF97, NONSEP_LDS>(S{}), fwd_lds_tiles<CDF97, SEP_LDS>(S{})},
             {fwd_lds_tiles<CDF53, NONSEP_LDS>(S{}), fwd_lds_tiles<CDF53, SEP_LDS>(S{})}}};
}
constexpr InvLdsTable make_inv_lds_table() {
    using S = std::make_integer_sequence<int, kNumTiles>;
    return {{{inv_lds_tiles<CDF97, NONSEP_LDS>(S{}), inv_lds_tiles<CDF97, SEP_LDS>(S{})},
             {inv_lds_tiles<CDF53, NONSEP_LDS>(S{}), inv_lds_tiles<CDF53, SEP_LDS>(S{})}}};
}

}  // namespace

FwdLdsTable kFwdLds = make_fwd_lds_table();
InvLdsTable kInvLds = make_inv_lds_table();
}  // namespace dwt2
