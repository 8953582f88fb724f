// Attention forward for few query rows per key/value head (internal to
// libtileattn; attn_decode.hip).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace tileattn_detail {

// Query rows per key/value head (heads of the group times queries) the
// decode kernel takes.
constexpr int DECODE_MAX_ROWS = 16;

struct DecodeArgs {
    const uint16_t *Q, *K, *V;
    // O fp32 or bf16 and LSE, or with splits the partial results of split 0;
    // split s adds s * o_split / s * l_split elements
    void *O;
    float *LSE;
    size_t o_split, l_split;
    int B, Hkv, Sq, Sk;
    int rows;        // Hq / Hkv * Sq
    int causal;
    int n_split;
    int split_keys;  // keys per split
    float c;         // scale * log2(e)
};

// D = 64 or 128; rows <= DECODE_MAX_ROWS
hipError_t launch_attn_decode(const DecodeArgs &a, int D, bool o_bf16, hipStream_t stream);

}  // namespace tileattn_detail
