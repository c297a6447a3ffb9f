// Codes as exact bf16 operands in units that keep sums small (gemm_w4_rescale.hip, w4_tile.hip).
#pragma once
#include "common.hpp"

namespace dmr {

// One word of a lane's codes -> the 8 bf16 values (16 + q) / 2 = 8 + q / 2 of an MFMA B operand.  Each nibble goes to
// mantissa bits [3, 7) of a bf16 whose high byte is 0x41 and whose exponent's lowest bit (the top bit of the low byte)
// stays clear: 2^3 (1 + q / 16).  (With that bit set the value would be 16 + q; leaving it saves an OR per four
// weights.  The decode kernels' 128 + q would carry an offset eight times larger into the cancellation with the
// zero-point term.)  In the streaming layout word w of a lane's unit holds the 8 codes of k = 8 w .. 8 w + 7 of its k
// step, the nibbles in the order 0, 4, 1, 5, 2, 6, 3, 7 that the four permutes below undo.
__device__ __forceinline__ void unpack4_word(uint32_t w, Frag &f) {
    const uint32_t even = (w << 3) & 0x78787878u;     // nibbles 0, 2, 4, 6 as low bytes
    const uint32_t odd = (w >> 1) & 0x78787878u;      // nibbles 1, 3, 5, 7
    const uint32_t exp = 0x41414141u;
    f.w[0] = __builtin_amdgcn_perm(even, exp, 0x00060004u);
    f.w[1] = __builtin_amdgcn_perm(odd, exp, 0x00060004u);
    f.w[2] = __builtin_amdgcn_perm(even, exp, 0x00070005u);
    f.w[3] = __builtin_amdgcn_perm(odd, exp, 0x00070005u);
}

// The 3-bit unit (three words per weight row and k step): chunk c < 3 of the row's 32 k is the two 3-bit fields of
// the bytes of word c, chunk 3 the spare top bits of all three words (bit 6 + h of word 2 is the third bit of a code
// in half h of the chunk, the top two bits of word h its low two).  Codes land in mantissa bits [3, 6): values
// (16 + q) / 2 as for four bits.
__device__ __forceinline__ void unpack3_chunk(const u32x4_t &u, int c, Frag &f) {
    const uint32_t exp = 0x41414141u, m38 = 0x38383838u;
    const uint32_t sel_a = 0x00060004u, sel_b = 0x00070005u;
    uint32_t f0, f1;
    if (c < 3) {
        const uint32_t v = u[c];
        f0 = (v << 3) & m38;
        f1 = v & m38;
    } else {
        f0 = (((u[2] >> 6) & 0x01010101u) << 5) | (((u[0] >> 6) & 0x03030303u) << 3);
        f1 = (((u[2] >> 7) & 0x01010101u) << 5) | (((u[1] >> 6) & 0x03030303u) << 3);
    }
    f.w[0] = __builtin_amdgcn_perm(f0, exp, sel_a);
    f.w[1] = __builtin_amdgcn_perm(f0, exp, sel_b);
    f.w[2] = __builtin_amdgcn_perm(f1, exp, sel_a);
    f.w[3] = __builtin_amdgcn_perm(f1, exp, sel_b);
}

}  // namespace dmr
