// What the loads of one stage of K address.  Plain C++ (constexpr functions are device functions as well), so that every
// access can be checked without a GPU.
#pragma once

namespace agg {

struct KsStage {
    unsigned bytes;       // size in the buffer descriptor
    int k_off;            // scalar offset of the loads
};

// Stage s of KC, `step` bytes of a row each, of an operand of `bytes`.  A stage past the end has an empty descriptor and no
// scalar offset: the bounds check may compare a lane's offset with the size less the scalar offset, which must not wrap.
constexpr KsStage ks_stage(int s, int KC, int step, unsigned bytes)
{
    return s < KC ? KsStage{bytes, s * step} : KsStage{0u, 0};
}

}  // namespace agg
