// The "lanes" event loop: one replica per thread on the bit-plane state,
// shared by the per-ensemble kernel, the batch's persistent kernel and the
// kernels compiled per network.  Results are bit for bit those of the
// bit-sliced word (wm_device.h): every event uses the same EVENT planes.
//
// The 32 threads of one half of a wave hold a word's 32 replicas as int32
// counts.  A window of 32 events goes in three steps:
//   draw       thread t makes the Philox calls of event e0 + t for the word,
//              transposes its planes in registers in blocks of 8 x 8 bits, so
//              that byte b of row r belongs to replica 8 b + r, and stores the
//              rows in LDS (one octet of planes: 8 words);
//   candidates each thread compares the top bytes of its replica's 32
//              thresholds with that of a bound of its total weight and keeps
//              the events below it as a bit mask.  Most events of a
//              uniformised chain are null (94 % on the N_tot = 1024 Frank
//              network) and change nothing, so they cost no more than that;
//   apply      each thread takes its own candidates in order: threshold from
//              its bytes, first crossing of the current cumulative weights,
//              count change, new weights.  Where the total weight has passed
//              the bound, the rest of the window is compared again.
//
// Bound by VALU issue on large ensembles: on the N_tot = 1024 workload (2^20
// replicas, 23 planes) a wave issues about 670 instructions per 64 word-events
// -- 197 for the draws, 144 for the transposition, 64 per comparison of the
// window and 34 per round of the last step (5 rounds: the busiest of 64
// replicas) -- against the bit-sliced word's 800, and unlike that word's one
// long chain they fill the chip: one instruction per 4.2 cycles and SIMD.  29 ms
// for the workload with every event drawn, where drawing, transposing and
// testing all 32 thresholds in order took 75.8 ms; 15.2 ms now that waves whose
// replicas have all ended stop.  Bound by a round's chain of dependent
// instructions, about 7 cycles each, where a SIMD holds a wave or none: 3.6 ms
// against 11.9 for 2^17 replicas, 4.1 against 6.2 for 16523 replicas of 4 10^4
// events of which 42 % are real.  (Measured there and not kept: a candidate's
// bytes read a full round ahead, 4.6 to 4.8 ms; A in a register of its own, 4.3
// ms.)
#pragma once

#include "event_draw.h"
#include "wm_device.h"

namespace bwg {

// LDS of one half wave: 32 event rows of 8 words per octet of planes, padded
// so that the 16-byte row stores of consecutive threads meet all banks.
template <int NQ>
struct LanesRow {
    static constexpr int NO = (NQ + 1) / 2;      // octets of planes, bytes of a threshold
    static constexpr int SH = (NQ & 1) ? 4 : 0;  // the lowest octet is half empty
    static constexpr int WORDS = 8 * NO + 4;
    static constexpr int HALF = 32 * WORDS;
};
constexpr int kLanesHalfWords = LanesRow<8>::HALF;  // the largest

// m = 2 m + [v < s] for v, s < 2^31 by the sign of the difference: two
// instructions, neither of which waits for a scalar register.
__device__ __forceinline__ uint32_t push_lt(uint32_t m, uint32_t v, uint32_t s)
{
    return __builtin_amdgcn_alignbit(m, v - s, 31);
}

// Transposes the 8 x 8 bit blocks of eight planes, byte column by byte
// column: afterwards bit q of byte b of x[r] is bit r of byte b of the
// original x[q].  HALF: only planes 4 .. 7 are given, the others are zero.
template <bool HALF>
__device__ __forceinline__ void transpose8(uint32_t *x)
{
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const uint32_t hi = x[k + 4];
        if (HALF) {
            x[k] = (hi << 4) & 0xF0F0F0F0u;
            x[k + 4] = hi & 0xF0F0F0F0u;
        } else {
            const uint32_t lo = x[k];
            x[k] = (lo & 0x0F0F0F0Fu) | ((hi << 4) & 0xF0F0F0F0u);
            x[k + 4] = ((lo >> 4) & 0x0F0F0F0Fu) | (hi & 0xF0F0F0F0u);
        }
    }
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        if (k & 2) continue;
        const uint32_t lo = x[k], hi = x[k + 2];
        x[k] = (lo & 0x33333333u) | ((hi << 2) & 0xCCCCCCCCu);
        x[k + 2] = ((lo >> 2) & 0x33333333u) | (hi & 0xCCCCCCCCu);
    }
#pragma unroll
    for (int k = 0; k < 8; k += 2) {
        const uint32_t lo = x[k], hi = x[k + 1];
        x[k] = (lo & 0x55555555u) | ((hi << 1) & 0xAAAAAAAAu);
        x[k + 1] = ((lo >> 1) & 0x55555555u) | (hi & 0xAAAAAAAAu);
    }
}

__device__ __forceinline__ uint64_t ballot(bool v) { return __builtin_amdgcn_ballot_w64(v); }
__device__ __forceinline__ bool wave_any(bool v) { return ballot(v) != 0; }

// Low 32 bits of a product of numbers below 2^24, at full rate.
__device__ __forceinline__ uint32_t mul24(uint32_t x, uint32_t y)
{
    return (x & 0xFFFFFFu) * (y & 0xFFFFFFu);
}

// A Frank-family replica: the counts of L and D in one register (A is what
// the conserved total leaves) and the cumulative weights of its state,
// S_1 = U, S_2 = 2U, S_3 = 2U + 2^fa A L, S_4 = 2U + 2^fa A (L + D),
// S_5 = S_4 + 2^fi L D with U = cu A, all below 2^32 (the host refuses larger
// totals).  FULL: the network has both bimolecular kinds and cu < 2^16.
template <bool FULL>
struct FrankReplica {
    static constexpr int S = 3;  // species in the planes' order L, D, A
    uint32_t ld, nt;
    uint32_t s1, s2, s3, s4, s5;
    uint32_t cu, step;
    int fa, fi;
    bool has_a, has_i;

    __device__ __forceinline__ explicit FrankReplica(const WmArgs &a)
    {
        cu = a.cu;
        has_a = a.fa >= 0;
        has_i = a.fi >= 0;
        fa = has_a ? a.fa : 0;
        fi = has_i ? a.fi : 0;
        step = (1u << fa) + (1u << fi);
    }
    __device__ __forceinline__ void set_counts(const uint32_t (&N)[S])
    {
        ld = N[0] | N[1] << 16;
        nt = N[0] + N[1] + N[2];
        weigh();
    }
    __device__ __forceinline__ void get_counts(uint32_t (&N)[S]) const
    {
        N[0] = ld & 0xFFFFu;
        N[1] = ld >> 16;
        N[2] = nt - N[0] - N[1];
    }
    __device__ __forceinline__ void weigh()
    {
        // counts have at most 14 bits: the products of 16-bit numbers are
        // 24-bit multiplications, at full rate (a 32-bit low product issues
        // at a quarter of it)
        const uint32_t L = ld & 0xFFFFu, D = ld >> 16, B = L + D, A = (nt - B) & 0xFFFFu;
        s1 = (cu & 0xFFFFu) * A;
        if (!FULL) s1 += ((cu >> 16) * A) << 16;
        s2 = 2 * s1;
        const uint32_t Aa = FULL || has_a ? A : 0u, Li = FULL || has_i ? L : 0u;
        s3 = s2 + ((Aa * L) << fa);
        s4 = s2 + ((Aa * (B & 0xFFFFu)) << fa);
        s5 = s4 + ((Li * D) << fi);
    }
    __device__ __forceinline__ uint32_t total() const { return s5; }
    // A bound that the total weight rarely passes within a window: a quarter
    // more plus about two events' change of the pair counts.  A state of
    // weight zero is left by no event.
    __device__ __forceinline__ uint32_t bound() const
    {
        const uint32_t slack = (s5 >> 2) + step * nt;
        return s5 ? __builtin_elementwise_add_sat(s5, slack) : 0u;
    }
    // The reaction whose cumulative weight first exceeds n (A -> L, A -> D,
    // A + L -> 2L, A + D -> 2D, L + D -> 2A) if on and n < s5, without
    // branches; returns the lanes whose state changed.  A tree of selections:
    // a wave alone on its SIMD waits for every instruction of a round's chain
    // (N_tot = 200, 100003 replicas: 592 us a pass with the comparisons
    // combined in turn, 554 with the tree).
    __device__ __forceinline__ uint64_t fire(uint32_t n, bool on, uint64_t)
    {
        const uint32_t m = on ? n : ~0u;
        const uint32_t lo = m < s1 ? 1u : 0x10000u, hi = m < s3 ? 1u : 0x10000u;
        const uint32_t a = m < s2 ? lo : hi, b = m < s5 ? 0xFFFEFFFFu : 0u;
        const uint64_t fired = ballot(m < s5);
        ld += m < s4 ? a : b;
        weigh();
        return fired;
    }
};

// Low k bits set, k in 0 .. 32.
__device__ __forceinline__ uint32_t low_bits(uint32_t k)
{
    return k >= 32 ? ~0u : (1u << k) - 1u;
}
__device__ __forceinline__ uint32_t clamp32(int32_t k)
{
    return k < 0 ? 0u : (k > 32 ? 32u : (uint32_t)k);
}

// Event range of a word's thread: its own pending events [E0, T0), and the
// word's window [lo, hi) over its pending lanes, as in wm_word.
struct LaneWindow {
    uint64_t E0, T0, lo, hi;
    bool live, mine;
};

__device__ __forceinline__ LaneWindow lane_window(const WmArgs &a, uint64_t i)
{
    LaneWindow v;
    v.live = i < a.M;
    v.E0 = v.live ? a.E[i] : 0;
    v.T0 = v.live ? a.Etgt[i] : 0;
    v.mine = v.live && v.E0 < v.T0;
    v.lo = v.mine ? v.E0 : ~0ull;
    v.hi = v.mine ? v.T0 : 0;
    for (int o = 16; o; o >>= 1) {
        const uint64_t lo2 =
            (uint64_t)(uint32_t)__shfl_xor((int)(uint32_t)v.lo, o, 32) |
            ((uint64_t)(uint32_t)__shfl_xor((int)(uint32_t)(v.lo >> 32), o, 32) << 32);
        const uint64_t hi2 =
            (uint64_t)(uint32_t)__shfl_xor((int)(uint32_t)v.hi, o, 32) |
            ((uint64_t)(uint32_t)__shfl_xor((int)(uint32_t)(v.hi >> 32), o, 32) << 32);
        v.lo = lo2 < v.lo ? lo2 : v.lo;
        v.hi = hi2 > v.hi ? hi2 : v.hi;
    }
    if (v.hi == 0) v.lo = 0;
    if (a.max_events && v.hi > v.lo + a.max_events) v.hi = v.lo + a.max_events;
    return v;
}

// Counts of lane l of word w from its planes; every plane's load is in flight
// at once (14 planes at most).
template <int S>
__device__ __forceinline__ void unpack_counts(const WmArgs &a, uint64_t w, int l,
                                              uint32_t (&N)[S])
{
    const int nbm = a.nb_mem;
#pragma unroll
    for (int x = 0; x < S; ++x) {
        uint32_t v = 0;
#pragma unroll
        for (int q = 0; q < 14; ++q) {
            const int qq = q < nbm ? q : 0;
            const uint32_t bit = (a.planes[((uint64_t)x * nbm + qq) * a.wp + w] >> l) & 1u;
            v |= q < nbm ? bit << q : 0u;
        }
        N[x] = v;
    }
}

// Counts back into the planes (lane q of the half stores plane q), the
// replica's event counter and the word's real events; a word past the end
// stores nothing.
template <int S>
__device__ __forceinline__ void pack_counts(const WmArgs &a, uint64_t w, int l, int hv,
                                            const LaneWindow &v, const uint32_t (&N)[S],
                                            uint32_t nreal)
{
    const int nbm = a.nb_mem;
    const bool valid = w < a.n_words;
#pragma unroll
    for (int x = 0; x < S; ++x) {
        uint32_t own = 0;
        for (int q = 0; q < nbm; ++q) {
            const uint32_t bits = (uint32_t)(__ballot((int)((N[x] >> q) & 1u)) >> (32 * hv));
            own = l == q ? bits : own;
        }
        if (l < nbm && valid) a.planes[((uint64_t)x * nbm + l) * a.wp + w] = own;
    }
    if (v.live) a.E[32 * w + l] = v.hi < v.E0 ? v.E0 : (v.hi > v.T0 ? v.T0 : v.hi);
    if (l == 0 && valid) a.real[w] += nreal;
}

// Every pending event of word w (one half wave), NQ quads of threshold
// planes; sq: the half's LanesRow<NQ>::HALF words of LDS.  Both halves of a
// wave take every loop together (words past the end and words without
// pending events with empty masks), so the loops are the wave's own and cost
// no lane masking.
//
// PAIR: two waves of one workgroup take the same two words; the one that
// draws is a window ahead of the one that keeps the replicas, each in another
// of two buffers (2 HALF words apart).  `ended` is two words of LDS: for every
// window the replicas' wave writes whether the chain ended there into the word
// of the window's parity before the barrier that closes it, and the drawing
// wave reads it after that barrier.  That word is written again only after the
// next barrier, so both waves leave at the same one.
template <int NQ, class Replica, bool PAIR = false>
__device__ __forceinline__ void wm_lanes(const WmArgs &a, uint64_t w, uint32_t *sq,
                                         bool draws = false, volatile uint32_t *ended = nullptr)
{
    constexpr int NO = LanesRow<NQ>::NO, SH = LanesRow<NQ>::SH, ROW = LanesRow<NQ>::WORDS;
    const int l = threadIdx.x & 31;
    const int hv = (threadIdx.x >> 5) & 1;
    const bool valid = w < a.n_words;
    const LaneWindow v = lane_window(a, valid ? 32 * w + (uint64_t)l : ~0ull);
    Replica rep(a);
    {
        uint32_t N[Replica::S] = {};
        if (valid && !draws) unpack_counts(a, w, l, N);
        rep.set_counts(N);
    }

    EventDraw<NQ, SH> dr;
    dr.k0 = (uint32_t)a.seed;
    dr.k1 = (uint32_t)(a.seed >> 32);
    dr.net_id = a.net_id;
    dr.G = (uint32_t)w;
    const int last = a.B - 4 * (NQ - 1);  // planes of the last quad, 1 .. 4
    const uint32_t m1 = last > 1 ? ~0u : 0u, m2 = last > 2 ? ~0u : 0u, m3 = last > 3 ? ~0u : 0u;
    // this replica's place in a row: byte l / 8 of word l mod 8 of each octet
    const uint32_t *word = sq + (l & 7);
    const uint32_t top_at = 32 * (NO - 1) + (l >> 3);
    const uint32_t sel = (uint32_t)(l >> 3);
    const uint32_t sel2 = 0x0C0C0400u + sel * 0x0101u, sel3 = 0x0C040100u + (sel << 16);
    const uint32_t sel4 = 0x04020100u + (sel << 24);
    auto threshold = [&](int g) -> uint32_t {
        const uint32_t *p = word + ROW * g;
        uint32_t n;
        if constexpr (NO == 1) {
            n = (p[0] >> (8 * sel)) & 0xFFu;
        } else {
            n = __builtin_amdgcn_perm(p[8], p[0], sel2);
            if constexpr (NO >= 3) n = __builtin_amdgcn_perm(p[16], n, sel3);
            if constexpr (NO >= 4) n = __builtin_amdgcn_perm(p[24], n, sel4);
        }
        return n >> SH;
    };
    const uint64_t Ts = v.mine ? (v.T0 < v.hi ? v.T0 : v.hi) : 0;
    // real events of the wave's two words: a launch runs at most kLanesEvents
    // of a replica, so that 32 bits hold them
    uint32_t real0 = 0, real1 = 0;
    // runs of events that share their index's bits 32 and up
    bool done = false;
    for (uint64_t base = v.lo; !done && wave_any(base < v.hi);) {
        const uint64_t room = (base | 0x3FFFFFFFull) + 1;
        const uint64_t stop = v.hi < room ? v.hi : room;
        const uint32_t span = base < stop ? (uint32_t)(stop - base) : 0u;
        // this replica's events of the run: [from, to)
        const int32_t to = Ts > base ? (int32_t)((Ts < stop ? Ts : stop) - base) : 0;
        const int32_t from = v.E0 > base ? (int32_t)(v.E0 < stop ? v.E0 - base : span) : 0;
        const uint32_t sp0 = (uint32_t)__builtin_amdgcn_readlane((int)span, 0);
        const uint32_t sp1 = (uint32_t)__builtin_amdgcn_readlane((int)span, 32);
        const int32_t most = (int32_t)(sp0 > sp1 ? sp0 : sp1);
        dr.set_word((uint32_t)(base >> 32) & 0xFFFFu);
        const uint32_t e_lo = (uint32_t)base + (uint32_t)l;
        // this thread's event k + l of the window at k
        auto draw = [&](int32_t k, uint32_t *rows) {
            uint32_t x[32];
            dr.draw(e_lo + (uint32_t)k, x);
            x[8 * NO - 3] &= m1;
            x[8 * NO - 2] &= m2;
            x[8 * NO - 1] &= m3;
#pragma unroll
            for (int o = 0; o < NO; ++o) {
                if (o == 0 && SH)
                    transpose8<true>(x);
                else
                    transpose8<false>(x + 8 * o);
            }
            uint4 *row = reinterpret_cast<uint4 *>(rows + ROW * l);
#pragma unroll
            for (int c = 0; c < 2 * NO; ++c)
                row[c] = make_uint4(x[4 * c], x[4 * c + 1], x[4 * c + 2], x[4 * c + 3]);
        };
        // the window's events of this thread's replica, from the rows at word
        auto take = [&](int32_t k) {
            const uint8_t *top = reinterpret_cast<const uint8_t *>(word) + top_at;
            // this replica's events of the window
            uint32_t ends = ~0u, rem = ~0u;
            if (wave_any(to - k < 32 || from > k)) {
                ends = low_bits(clamp32(to - k));
                rem = ends & ~low_bits(clamp32(from - k));
            }
            do {
                const uint32_t bound = rep.bound();
                const uint32_t most_t =
                    NO == 1 ? ((bound < 256u ? bound : 256u) - 1u) << SH
                            : (bound - 1u) >> (NO == 1 ? 0 : 8 * (NO - 1) - SH);
                uint32_t cut = most_t < 255u ? most_t + 1u : 256u;
                if (!bound) cut = 0;
                uint32_t cm = 0;
#pragma unroll
                for (int g = 31; g >= 0; --g) cm = push_lt(cm, top[4 * ROW * g], cut);
                cm &= rem;
                const uint32_t cm0 = cm;
                // one candidate of every replica a round, until no replica
                // has one left whose total is within its bound (a round
                // without any changes nothing); the next candidate's bytes
                // are read while this one runs
                uint32_t n = threshold(__builtin_ctz(cm | 0x80000000u));
                bool on = cm != 0;
                uint64_t onm = ballot(cm != 0);
                do {
                    const uint32_t left = cm & (cm - 1);
                    cm = on ? left : cm;
                    const uint32_t nn = threshold(__builtin_ctz(cm | 0x80000000u));
                    const uint64_t fired = rep.fire(n, on, onm);
                    real0 += (uint32_t)__builtin_popcount((uint32_t)fired);
                    real1 += (uint32_t)__builtin_popcount((uint32_t)(fired >> 32));
                    onm = ballot(cm != 0) & ballot(rep.total() <= bound);
#if __has_builtin(__builtin_amdgcn_inverse_ballot_w64)
                    // the mask itself, which the ballots have formed
                    on = __builtin_amdgcn_inverse_ballot_w64(onm);
#else
                    on = cm != 0 && rep.total() <= bound;
#endif
                    n = nn;
                } while (onm);
                // past the bound: the events after the last candidate taken
                // may lie between the bound and the total
                const uint32_t taken = cm0 ^ cm;
                rem = rep.total() > bound && taken
                          ? ~((2u << (31 - __builtin_clz(taken))) - 1u) & ends
                          : 0u;
            } while (wave_any(rem != 0));
        };
        if constexpr (PAIR) {
            if (draws) {
                if (most > 0) draw(0, sq);
                __syncthreads();
                for (int32_t k = 0; k < most && !done; k += 32) {
                    const uint32_t to_buf = k & 32 ? 0 : 2 * LanesRow<NQ>::HALF;
                    if (k + 32 < most) draw(k + 32, sq + to_buf);
                    __syncthreads();
                    done = ended[(k >> 5) & 1] != 0;
                }
            } else {
                __syncthreads();
                for (int32_t k = 0; k < most && !done; k += 32) {
                    word = sq + (k & 32 ? 2 * LanesRow<NQ>::HALF : 0) + (l & 7);
                    done = !wave_any(rep.total() != 0);
                    ended[(k >> 5) & 1] = done;
                    if (!done) take(k);
                    __syncthreads();
                }
            }
        } else {
            for (int32_t k = 0; k < most; k += 32) {
                // a state of total weight zero (one enantiomer and no A) is
                // left by no event: nothing to draw once all replicas of the
                // wave have reached one (N_tot = 1024, t = 100: 29.0 -> 15.2 ms)
                done = !wave_any(rep.total() != 0);
                if (done) break;
                draw(k, sq);
                // the half's LDS operations run in program order: the reads
                // see every lane's stores, and the next window's stores
                // follow them
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                __builtin_amdgcn_wave_barrier();
                take(k);
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                __builtin_amdgcn_wave_barrier();
            }
        }
        base = base < stop ? stop : base;
    }
    if (draws) return;
    uint32_t N[Replica::S];
    rep.get_counts(N);
    pack_counts(a, valid ? w : ~0ull, l, hv, v, N, hv ? real1 : real0);
}

// The same for shared thresholds: at every event all replicas compare the n
// that the table holds (one event counter for all of them, kept by the host).
template <class Replica>
__device__ __forceinline__ void wm_lanes_shared(const WmArgs &a, uint64_t w)
{
    const int l = threadIdx.x & 31;
    const int hv = (threadIdx.x >> 5) & 1;
    if (w >= a.n_words) return;
    const bool live = 32 * w + (uint64_t)l < a.M;
    LaneWindow v{};  // not live: no counter is stored
    Replica rep(a);
    uint32_t N[Replica::S];
    unpack_counts(a, w, l, N);
    rep.set_counts(N);
    uint32_t nreal = 0;
    for (uint64_t e = a.zbase; e < a.zbase + a.zlen; ++e) {
        const uint32_t n = shared_at(a, e);
        nreal += live && n < rep.total() ? 1u : 0u;
        rep.fire(n, live, 0);
    }
    for (int o = 16; o; o >>= 1) nreal += (uint32_t)__shfl_xor((int)nreal, o, 32);
    rep.get_counts(N);
    pack_counts(a, w, l, hv, v, N, nreal);
}

}  // namespace bwg
