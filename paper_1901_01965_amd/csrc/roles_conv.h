// The role-specialised single-kernel forms (transform and products on separate waves): what a launch is given, and the
// launches.  They read channels-last activations with C % 4 = 0 through 4-byte loads and write any K in either layout.
#pragma once
#include "input_transform_core.h"

namespace wg {

struct RolesCall {
    const int8_t* x;             // channels-last, pixel stride p.C
    const ZeroPointU8* zero;     // null: signed int8 activations and filters; else uint8 (p.Cf <= kMaxChannelsInt9, q8.out null)
    const uint8_t* blob;
    BlobLayout bl;
    int32_t* y;
    Problem p;
    int layout;                  // of the outputs
    Int8Epilogue q8;
};

// One tile block of 16 tiles per workgroup.  wide: 64 filters per workgroup (eight product waves), else 32.
hipError_t launch_roles_lossless(const RolesCall& c, bool wide, hipStream_t s);
hipError_t launch_roles_scaled(const RolesCall& c, bool wide, hipStream_t s);
inline hipError_t launch_roles(const RolesCall& c, int mode, bool wide, hipStream_t s) {
    return mode == WG_LOSSLESS ? launch_roles_lossless(c, wide, s) : launch_roles_scaled(c, wide, s);
}
// Second kernel of a convolution with split channels: adds, finishes and stores what launch_scaled_sums /
// launch_lossless_pair_sums left.
hipError_t launch_split_finish(const RolesCall& c, const int32_t* partial, int splits, hipStream_t s);
hipError_t launch_sums_finish(const RolesCall& c, const int32_t* sums, int splits, hipStream_t s);
// A workgroup's sums lie together (what one XCD writes would otherwise fall into a few of its L2's channels: rows of Kp filters,
// 592 -> 240 at 33x33, N = 1, scaled: 16.5 us): `values` numbers of 16 tiles x 32 filters from here on.
__host__ __device__ inline size_t split_sums_offset(int values, int split, int tile_block, int filter_block, int tile_blocks, int Kp) {
    return (((size_t)split * tile_blocks + tile_block) * (Kp >> 5) + filter_block) * (size_t)(values * 16 * 32);
}
inline size_t split_partial_bytes(const Problem& p, int mode, int splits) {
    return (size_t)splits * (mode == WG_LOSSLESS ? 16 : kAccPlanes) * 16 * ceil_div(p.T, 16) * p.Kp * sizeof(int32_t);
}
// A workgroup walks over many tile blocks of one filter block (see stream_kernel.h for the forms): 32 filters or, kStreamWhole
// (lossless mode, or one channel block), kStreamEight and kStreamPairs (lossless mode and one channel block), 64.
enum StreamForm { kStreamHalves, kStreamWhole, kStreamEight, kStreamPairs };
hipError_t launch_stream_lossless(const RolesCall& c, StreamForm form, hipStream_t s);
hipError_t launch_stream_scaled(const RolesCall& c, StreamForm form, hipStream_t s);
inline hipError_t launch_stream(const RolesCall& c, int mode, StreamForm form, hipStream_t s) {
    return mode == WG_LOSSLESS ? launch_stream_lossless(c, form, s) : launch_stream_scaled(c, form, s);
}
// Activations scaled per tile as well (WG_SCALED blob, signed int8): the factors of every tile into factors (uint32 [T][26],
// act_factor_bytes; act_table: null or the exported int32 [T][26][4]), then the convolution with them.
inline size_t act_factor_bytes(const Problem& p) { return round_up((size_t)p.T * kEntries * sizeof(uint32_t), 256); }
hipError_t launch_act_factors(const RolesCall& c, uint32_t* factors, int32_t* act_table, hipStream_t s);
hipError_t launch_act_scaled_roles(const RolesCall& c, const uint32_t* factors, hipStream_t s);
// Workgroups per filter block of the streaming kernel: about one workgroup per compute unit in total (a test hook can set
// a smaller number, so that small problems stream, too).
int stream_workgroups(int tile_blocks, int filter_blocks);

}  // namespace wg
