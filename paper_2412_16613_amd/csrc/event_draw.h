// The threshold planes of one event of a 32-replica word.
#pragma once

#include "bitops.h"
#include "bwg_internal.h"

namespace bwg {

// EVENT planes of one event of a word: the NQ Philox calls differ in one
// counter word only, so the first rounds share work.  Round 1's products and
// the product on counter word 0 of round 2 depend on the word and the call,
// not on the event (up to its high bits): ha, la hold the latter.  The other
// products of rounds 1 and 2 and one of round 3 are the same for all calls:
// 5 + 32 NQ instructions an event instead of 40 NQ.  set_word has to be called
// for the word (G) and again where bits 32 to 47 of the event index change.
// Plane p goes to x[OFF + p].
template <int NQ, int OFF = 0>
struct EventDraw {
    uint32_t k0, k1, net_id, G;
    uint32_t ha[NQ], la[NQ];

    __device__ __forceinline__ void set_word(uint32_t hi)
    {
        const uint32_t h = (uint32_t)(((uint64_t)0xCD9E8D57u * G) >> 32);
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            const uint32_t c1 = (DOM_EVENT << 24) | ((uint32_t)q << 16) | hi;
            const uint64_t p = (uint64_t)0xD2511F53u * (uint32_t)BWG_OP3(h, c1, k0, L_XOR3);
            ha[q] = (uint32_t)(p >> 32);
            la[q] = (uint32_t)p;
        }
    }
    template <int W>
    __device__ __forceinline__ void draw(uint32_t e_lo, uint32_t (&x)[W]) const
    {
        constexpr uint32_t W0 = 0x9E3779B9u, W1 = 0xBB67AE85u;
        constexpr uint64_t M0 = 0xD2511F53u, M1 = 0xCD9E8D57u;
        static_assert(OFF + 4 * NQ <= W, "planes");
        // shared by the calls
        const uint64_t a0 = M0 * e_lo;                                           // round 1
        const uint64_t a1 = M1 * (uint32_t)BWG_OP3((uint32_t)(a0 >> 32), net_id, k1, L_XOR3);  // round 2
        const uint32_t lg = (uint32_t)(M1 * G);
        const uint64_t a2 = M0 * (uint32_t)BWG_OP3((uint32_t)(a1 >> 32), lg, k0 + W0, L_XOR3);  // round 3
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            // counter word 2 after round 2, then round 3
            const uint64_t b = M1 * (uint32_t)BWG_OP3(ha[q], (uint32_t)a0, k1 + W1, L_XOR3);
            uint32_t c0 = BWG_OP3((uint32_t)(b >> 32), (uint32_t)a1, k0 + 2 * W0, L_XOR3);
            uint32_t c1 = (uint32_t)b;
            uint32_t c2 = BWG_OP3((uint32_t)(a2 >> 32), la[q], k1 + 2 * W1, L_XOR3);
            uint32_t c3 = (uint32_t)a2;
#pragma unroll
            for (int r = 3; r < 10; ++r) {
                const uint64_t p0 = M0 * c0, p1 = M1 * c2;
                c0 = BWG_OP3((uint32_t)(p1 >> 32), c1, k0 + (uint32_t)r * W0, L_XOR3);
                c2 = BWG_OP3((uint32_t)(p0 >> 32), c3, k1 + (uint32_t)r * W1, L_XOR3);
                c1 = (uint32_t)p1;
                c3 = (uint32_t)p0;
            }
            x[OFF + 4 * q] = c0;
            x[OFF + 4 * q + 1] = c1;
            x[OFF + 4 * q + 2] = c2;
            x[OFF + 4 * q + 3] = c3;
        }
    }
};

}  // namespace bwg
