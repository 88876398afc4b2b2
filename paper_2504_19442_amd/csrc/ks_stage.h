// What the loads of one stage of K address.  Plain C++ (constexpr functions are device functions as well), so that every
// access can be checked without a GPU.
#pragma once

namespace agg {

struct KsStage {
    unsigned bytes;       // size in the buffer descriptor
    int k_off;            // scalar offset of the loads
};

// Stage s of KC, `step` bytes of a row each, of an operand of `bytes`.  Nothing of a stage past the end may be loaded.  Its size
// is its scalar offset: whether the bounds check adds that offset to the lane's or takes it from the size, every lane is
// outside.  (A size of zero beside the offset would wrap in the second reading; making both zero costs one more scalar select
// per stage, 0.2 us of a 25 us call.)
constexpr KsStage ks_stage(int s, int KC, int step, unsigned bytes)
{
    return KsStage{s < KC ? bytes : (unsigned)(s * step), s * step};
}

}  // namespace agg
