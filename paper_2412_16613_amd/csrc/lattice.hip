// Compartment (lattice) kernels: initial site states, the component schedule
// of each 2048-replica group, the layered event kernel and the readouts.
//
// The paper presents the bitwise method for one well-mixed reactor and names
// ensembles of small compartments as what it is meant for (Sec. 1, Sec. 6).
// Here every replica is a periodic lx x ly lattice of Frank reactors (site
// counts L, D, A in P bit planes each, site total at most T = 2^P - 1) whose
// molecules hop to the 4 neighbours.  The uniformised chain draws, per event,
// one component shared by the replicas of a group -- the reaction of a site,
// or a hop out of a site in one direction -- and per replica a threshold
// (reaction: B_r planes, first crossing of the site's cumulative weights, the
// Sec. 4 comparator) or a hop index j in [0, T] (A if j < n_A, L if
// j < n_A + n_L, D if j < n_site; blocked when the destination is full).
//
// Events of one group that touch disjoint sites commute, so the schedule
// kernel sorts each chunk of the group's component sequence into greedy
// layers of pairwise disjoint events; the event kernel runs one layer at a
// time, every event of a layer in its own thread, on the planes of one word
// (32 replicas).  Each replica still applies exactly its own events, in an
// order that only permutes commuting events.

#include "bitops.h"
#include "bwg.h"
#include "bwg_internal.h"
#include "event_draw.h"

namespace bwg {

// ---- draws -------------------------------------------------------------------

// Component of event e of a group: uniform in [0, C) from 64-bit COMPONENT
// draws by Lemire's multiply-and-reject (thresh = 2^64 mod C); the attempt
// index is part of the counter, and the 256th attempt is taken as it is.
__device__ __forceinline__ uint64_t lat_component(uint64_t seed, uint32_t net_id, uint32_t group,
                                                  uint64_t e, uint64_t C, uint64_t thresh)
{
    uint64_t u = 0;
    for (uint32_t attempt = 0; attempt < 256; ++attempt) {
        uint32_t o0, o1, o2, o3;
        philox4x32_10((uint32_t)e,
                      (DOM_COMPONENT << 24) | (attempt << 16) | ((uint32_t)(e >> 32) & 0xFFFFu),
                      group, net_id, (uint32_t)seed, (uint32_t)(seed >> 32), o0, o1, o2, o3);
        u = (uint64_t)o0 | ((uint64_t)o1 << 32);
        if (u * C >= thresh) break;
    }
    return __umul64hi(u, C);
}

// A uniform in {lo..hi} for (replica i, site s): 32-bit Lemire with rejection
// over the four outputs of successive INIT draws; R = hi - lo + 1, thresh =
// 2^32 mod R.  Nearly always the first output is taken, so it is formed by
// itself (the last rounds' other products fall away).
__device__ __forceinline__ int32_t lat_init_count(uint64_t seed, uint32_t net_id, uint64_t i,
                                                  uint32_t s, int32_t lo, uint32_t R,
                                                  uint32_t thresh)
{
    uint32_t f, u0, u1, u2;
    philox4x32_10(s, (DOM_INIT << 24) | (1u << 23), (uint32_t)i, net_id, (uint32_t)seed,
                  (uint32_t)(seed >> 32), f, u0, u1, u2);
    const uint64_t m0 = (uint64_t)f * R;
    if (__builtin_expect((uint32_t)m0 >= thresh, 1)) return lo + (int32_t)(m0 >> 32);
    for (uint32_t attempt = 0; attempt < 65536; ++attempt) {
        uint32_t o[4];
        philox4x32_10(s, (DOM_INIT << 24) | (1u << 23) | attempt, (uint32_t)i, net_id,
                      (uint32_t)seed, (uint32_t)(seed >> 32), o[0], o[1], o[2], o[3]);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const uint64_t m = (uint64_t)o[k] * R;
            if ((uint32_t)m >= thresh) return lo + (int32_t)(m >> 32);
        }
    }
    return lo;
}

__device__ __forceinline__ uint32_t lat_neighbour(const LatShape &sh, uint32_t s, uint32_t dir)
{
    // s / lx by the reciprocal 2^24 / lx, rounded up: exact for s, lx <= 4096
    uint32_t y = (uint32_t)(((uint64_t)s * sh.inv_lx) >> 24), x = s - y * (uint32_t)sh.lx;
    if (dir == 0)
        x = x + 1 == (uint32_t)sh.lx ? 0 : x + 1;
    else if (dir == 1)
        x = x == 0 ? sh.lx - 1 : x - 1;
    else if (dir == 2)
        y = y + 1 == (uint32_t)sh.ly ? 0 : y + 1;
    else
        y = y == 0 ? sh.ly - 1 : y - 1;
    return y * (uint32_t)sh.lx + x;
}

// ---- layout ----------------------------------------------------------------
// Site planes of word w in group g = w / 64: a group stores, site by site, the
// 3P planes of each of its 64 words (padded), so the planes of one site of
// consecutive words are contiguous:
//   planes[((g S + s) 64 + (w mod 64)) 3P + x P + q],  species x in (L, D, A).
__device__ __forceinline__ uint32_t *site_planes(uint32_t *planes, uint64_t w, uint32_t s,
                                                 int S, int NP)
{
    return planes + (((w >> 6) * (uint64_t)S + s) * 64 + (w & 63)) * (uint64_t)NP;
}
__device__ __forceinline__ const uint32_t *site_planes(const uint32_t *planes, uint64_t w,
                                                       uint32_t s, int S, int NP)
{
    return planes + (((w >> 6) * (uint64_t)S + s) * 64 + (w & 63)) * (uint64_t)NP;
}

// ---- initial states -------------------------------------------------------------

// mode 0: every site of every replica holds site[s] (sites = null: site0 for
// all sites); one thread per (word, site).
__global__ void lat_init_fixed_kernel(uint32_t *planes, uint64_t words, uint64_t M, int S, int P,
                                      const int32_t *sites, int32_t l0, int32_t d0, int32_t a0,
                                      uint64_t *E, uint64_t *Et, uint64_t *real, uint64_t *blocked)
{
    const uint64_t w = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const uint32_t s = blockIdx.y;
    if (w >= words) return;
    const uint64_t rem = M - 32 * w;
    const uint32_t live = rem >= 32 ? 0xFFFFFFFFu : ((1u << rem) - 1u);
    int32_t c[3] = {l0, d0, a0};
    if (sites) {
        c[0] = sites[3 * s];
        c[1] = sites[3 * s + 1];
        c[2] = sites[3 * s + 2];
    }
    uint32_t *p = site_planes(planes, w, s, S, 3 * P);
    for (int x = 0; x < 3; ++x)
        for (int q = 0; q < P; ++q) p[x * P + q] = ((c[x] >> q) & 1) ? live : 0u;
    if (s == 0) {
        for (int l = 0; l < 32; ++l) {
            E[32 * w + l] = 0;
            Et[32 * w + l] = 0;
        }
        real[w] = 0;
        blocked[w] = 0;
    }
}

// mode 1: A uniform in {lo..hi} per (replica, site), L = D = 0.  A wave holds
// 64 replicas (two words) of one site at a time and packs their counts with
// ballots; it takes LAT_INIT_SITES sites, so that the products of the first
// two Philox rounds, which depend on the replica or on the site alone, are
// formed once or by the scalar unit.  Bound by the draws' multiplications:
// 509 us for 64 x 64 sites of 2^16 replicas (985 with a site per thread and
// every output formed).
constexpr int LAT_INIT_SITES = 8;

__global__ __launch_bounds__(256) void lat_init_uniform_kernel(
    uint32_t *planes, uint64_t words, uint64_t M, int S, int P, int32_t lo, int32_t hi,
    uint64_t seed, uint32_t net_id, uint64_t *E, uint64_t *Et, uint64_t *real, uint64_t *blocked)
{
    // blockDim.x is a multiple of 64; grid.x covers 64 * ceil(words / 2) replicas
    const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const uint32_t s0 = blockIdx.y * LAT_INIT_SITES;
    const uint32_t s1 = min(s0 + LAT_INIT_SITES, (uint32_t)S);
    const bool ok = i < M;
    const uint64_t w = i >> 5;
    const int lane = threadIdx.x & 63;
    const bool stores = (lane & 31) == 0 && w < words;
    const uint32_t R = (uint32_t)(hi - lo + 1);
    const uint32_t thresh = (0u - R) % R;
    for (uint32_t s = s0; s < s1; ++s) {
        int32_t a = 0;
        if (ok) a = lat_init_count(seed, net_id, i, s, lo, R, thresh);
        uint32_t *p = site_planes(planes, w, s, S, 3 * P);
        if (P == 4) {
            uint32_t b[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const uint64_t bits = __ballot((a & (1 << q)) != 0);
                b[q] = lane & 32 ? (uint32_t)(bits >> 32) : (uint32_t)bits;
            }
            if (stores) {
                uint4 *v = reinterpret_cast<uint4 *>(p);
                v[0] = v[1] = make_uint4(0u, 0u, 0u, 0u);
                v[2] = make_uint4(b[0], b[1], b[2], b[3]);
            }
            continue;
        }
        for (int q = 0; q < P; ++q) {
            const uint64_t bits = __ballot((a >> q) & 1);
            if (stores) {
                p[q] = 0u;
                p[P + q] = 0u;
                p[2 * P + q] = lane ? (uint32_t)(bits >> 32) : (uint32_t)bits;
            }
        }
    }
    if (s0 == 0 && w < words) {
        E[i] = 0;
        Et[i] = 0;
        if ((i & 31) == 0) {
            real[w] = 0;
            blocked[w] = 0;
        }
    }
}

// ---- schedule -------------------------------------------------------------------
// One workgroup per (group, chunk of LAT_CH events).  Slot layout (uint32):
//   recs[LAT_CH]   events in layer order: (offset in chunk) << 16 | site << 3 | kind
//                  (within a layer in any order)
//   tmp[LAT_CH]    per event: other site << 16 | site << 3 | kind (~0: outside),
//                  then layer << 16 | site << 3 | kind (0: outside)
//   offs[0]        number of layers; the low half of offs[1 + L] is the first
//                  event of layer L (L = 0 .. layers), so layer L is
//                  recs[offs[1+L] .. offs[2+L]); the high half its first hop.
// kind 0 is the site's reaction component, 1 + d a hop in direction d.
//
// The layers are a serial chain over the chunk's batches of 64 events, walked
// by one wave; the draws before it and the sort after it are shared by
// LAT_SCHED_BLOCK threads, and the chain's LDS traffic is one round trip a
// round (a stamp that grows from round to round needs no clearing between
// them).  A launch of 32 groups by 32 chunks over 64 x 64 sites takes 114 us
// (316 with one wave a workgroup, three barriers a round and 56 KB of LDS, of
// which two workgroups fit a CU).
constexpr int LAT_SCHED_BLOCK = 256;

__device__ __forceinline__ uint32_t wave_max_u32(uint32_t v)
{
    for (int o = 32; o; o >>= 1) v = max(v, (uint32_t)__shfl_xor((int)v, o, 64));
    return v;
}
__device__ __forceinline__ uint64_t wave_min_u64(uint64_t v)
{
    for (int o = 32; o; o >>= 1) {
        const uint32_t lo = __shfl_xor((int)(uint32_t)v, o, 64);
        const uint32_t hi = __shfl_xor((int)(uint32_t)(v >> 32), o, 64);
        v = min(v, (uint64_t)lo | ((uint64_t)hi << 32));
    }
    return v;
}
__device__ __forceinline__ uint64_t wave_max_u64(uint64_t v)
{
    for (int o = 32; o; o >>= 1) {
        const uint32_t lo = __shfl_xor((int)(uint32_t)v, o, 64);
        const uint32_t hi = __shfl_xor((int)(uint32_t)(v >> 32), o, 64);
        v = max(v, (uint64_t)lo | ((uint64_t)hi << 32));
    }
    return v;
}
__device__ __forceinline__ uint32_t wave_incl_scan(uint32_t v, int lane)
{
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t t = __shfl_up((int)v, o, 64);
        if (lane >= o) v += t;
    }
    return v;
}

__global__ __launch_bounds__(LAT_SCHED_BLOCK) void lat_schedule_kernel(LatArgs a)
{
    constexpr int NW = LAT_SCHED_BLOCK / 64;
    // the sort's counters take the place of the chain's site tables: two
    // 16-bit counters per word, key = 2 layer + hop
    __shared__ uint32_t lds[LAT_CH];
    static_assert(LAT_MAX_SITES * 3 / 2 <= LAT_CH, "site tables");
    uint32_t *const hist = lds;
    uint32_t *const first = lds;
    uint16_t *const last = reinterpret_cast<uint16_t *>(lds + LAT_MAX_SITES);
    __shared__ uint64_t wlo[NW], whi[NW];
    __shared__ uint32_t s_nl;

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const uint32_t ci = blockIdx.x % a.n_chunks;
    const uint32_t g = blockIdx.x / a.n_chunks;
    uint32_t *slot = a.sched + ((uint64_t)g * LAT_NCB + ci) * LAT_SLOT;
    uint32_t *recs = slot, *tmp = slot + LAT_CH, *offs = slot + 2 * LAT_CH;
    const LatShape &sh = a.sh;

    // events of this chunk that some pending replica of the group runs
    const uint64_t r0 = (uint64_t)g * LAT_GROUP_WORDS * 32;
    const uint64_t r1 = min(a.M, r0 + LAT_GROUP_WORDS * 32);
    uint64_t lo = ~0ull, hi = 0;
#pragma unroll 4
    for (uint64_t i = r0 + tid; i < r1; i += LAT_SCHED_BLOCK) {
        const uint64_t e0 = a.E[i], e1 = a.Et[i];
        if (e0 < e1) {
            lo = min(lo, e0);
            hi = max(hi, e1);
        }
    }
    lo = wave_min_u64(lo);
    hi = wave_max_u64(hi);
    if (lane == 0) {
        wlo[wave] = lo;
        whi[wave] = hi;
    }
    for (int k = tid; k < LAT_MAX_SITES * 3 / 2; k += LAT_SCHED_BLOCK) lds[k] = 0;
    __syncthreads();
    for (int k = 0; k < NW; ++k) {
        lo = min(lo, wlo[k]);
        hi = max(hi, whi[k]);
    }
    const uint64_t cbase = a.base + (uint64_t)(a.chunk0 + ci) * LAT_CH;
    const uint64_t clo = max(cbase, lo), chi = min(cbase + LAT_CH, hi);
    if (clo >= chi) {
        if (tid == 0) offs[0] = 0;
        return;
    }

    for (uint32_t off = tid; off < LAT_CH; off += LAT_SCHED_BLOCK) {
        const uint64_t e = cbase + off;
        uint32_t v = ~0u;
        if (e >= clo && e < chi) {
            const uint64_t comp = lat_component(a.seed, a.net_id, g, e, sh.C, sh.thresh);
            const uint64_t q = comp / sh.Wsite;
            const uint64_t r = comp - q * sh.Wsite;
            const uint32_t s = (uint32_t)q;
            const uint32_t kind = r < sh.W_R ? 0u : 1u + (uint32_t)((r - sh.W_R) / sh.W_H);
            v = ((kind ? lat_neighbour(sh, s, kind - 1) : s) << 16) | (s << 3) | kind;
        }
        tmp[off] = v;
    }
    __syncthreads();

    // greedy layers: an event's layer is one more than the last layer that
    // touched either of its sites; within a batch of 64 events, a lane is
    // settled in the round where it is the earliest unsettled lane at both
    // of its sites, so settled lanes of one round touch disjoint sites.  The
    // sites' entries of first[] hold the round's stamp and 63 - lane of the
    // earliest lane; a wave's LDS operations keep their order.
    if (wave == 0) {
        uint32_t maxlay = 0, stamp = 0, next = tmp[lane];
        for (uint32_t b = 0; b < LAT_CH; b += 64) {
            const uint32_t v = next;
            if (b + 64 < LAT_CH) next = tmp[b + 64 + lane];
            const bool in = v != ~0u;
            const uint32_t s = (v >> 3) & 0x1FFFu, s2 = v >> 16;
            bool pend = in;
            uint32_t lay = 0;
            while (__any(pend)) {
                stamp += 64;
                const uint32_t key = stamp | (63u - (uint32_t)lane);
                if (pend) {
                    atomicMax(&first[s], key);
                    atomicMax(&first[s2], key);
                }
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                __builtin_amdgcn_wave_barrier();
                if (pend) {
                    const uint32_t f1 = first[s], f2 = first[s2], l1 = last[s], l2 = last[s2];
                    if (f1 == key && f2 == key) {
                        lay = 1u + max(l1, l2);
                        last[s] = (uint16_t)lay;
                        last[s2] = (uint16_t)lay;
                        pend = false;
                    }
                }
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                __builtin_amdgcn_wave_barrier();
            }
            maxlay = max(maxlay, lay);
            tmp[b + lane] = in ? (lay << 16) | (v & 0xFFFFu) : 0u;
        }
        const uint32_t nl = wave_max_u32(maxlay);
        if (lane == 0) s_nl = nl;
    }
    __syncthreads();
    const uint32_t nl = s_nl;

    // sort by key: count, exclusive prefix over keys 0 .. 2 nl - 1, written
    // back as cursors, then place
    for (uint32_t k = tid; k < nl; k += LAT_SCHED_BLOCK) hist[k] = 0;
    __syncthreads();
#pragma unroll 4
    for (uint32_t off = tid; off < LAT_CH; off += LAT_SCHED_BLOCK) {
        const uint32_t t = tmp[off], lay = t >> 16;
        if (lay) atomicAdd(&hist[lay - 1], (t & 7u) != 0 ? 0x10000u : 1u);
    }
    __syncthreads();
    if (wave == 0) {
        uint32_t run = 0;
        for (uint32_t kb = 0; kb < nl; kb += 64) {
            const uint32_t k = kb + lane;
            const uint32_t h = k < nl ? hist[k] : 0u;
            const uint32_t cnt = (h & 0xFFFFu) + (h >> 16);
            const uint32_t incl = wave_incl_scan(cnt, lane);
            const uint32_t excl = run + incl - cnt;
            if (k < nl) {
                hist[k] = excl | ((excl + (h & 0xFFFFu)) << 16);
                offs[1 + k] = hist[k];
            }
            run += __shfl((int)incl, 63, 64);
        }
        if (lane == 0) {
            offs[0] = nl;
            offs[1 + nl] = run;
        }
    }
    __syncthreads();
#pragma unroll 4
    for (uint32_t off = tid; off < LAT_CH; off += LAT_SCHED_BLOCK) {
        const uint32_t t = tmp[off], lay = t >> 16;
        if (lay) {
            const uint32_t sh16 = (t & 7u) != 0 ? 16 : 0;
            const uint32_t old = atomicAdd(&hist[lay - 1], 1u << sh16);
            recs[(old >> sh16) & 0xFFFFu] = (off << 16) | (t & 0xFFFFu);
        }
    }
}

// ---- event kernel ------------------------------------------------------------

// acc (BC planes) += p << SH over planes [SH, BC).
template <int BC, int WP, int SH>
__device__ __forceinline__ void add_shifted(uint32_t (&acc)[BC], const uint32_t (&p)[WP])
{
    uint32_t cy = 0;
#pragma unroll
    for (int q = SH; q < BC; ++q) {
        const uint32_t v = (q - SH < WP) ? p[q - SH] : 0u;
        const uint32_t s = BWG_OP3(acc[q], v, cy, L_XOR3);
        if (q + 1 < BC) cy = BWG_OP3(acc[q], v, cy, L_MAJ);
        acc[q] = s;
    }
}

// Run-time shift: one compile-time addition is taken (wave-uniform branch).
template <int BC, int WP, int SH = 0>
__device__ __forceinline__ void add_dispatch(int sh, uint32_t (&acc)[BC], const uint32_t (&p)[WP])
{
    if constexpr (SH < BC) {
        if (sh == SH) {
            add_shifted<BC, WP, SH>(acc, p);
            return;
        }
        add_dispatch<BC, WP, SH + 1>(sh, acc, p);
    }
}

template <int BC, int WP, int64_t K, int k = 0>
__device__ __forceinline__ void add_bits(uint32_t (&acc)[BC], const uint32_t (&p)[WP])
{
    if constexpr (k < BC) {
        if constexpr ((K >> k) & 1) add_shifted<BC, WP, k>(acc, p);
        add_bits<BC, WP, K, k + 1>(acc, p);
    }
}

// acc += c * p: K >= 0 is the constant at compile time, else c at run time
// (one shifted addition per set bit).
template <int BC, int WP, int64_t K>
__device__ __forceinline__ void add_const_mul(uint32_t (&acc)[BC], const uint32_t (&p)[WP],
                                              uint64_t c)
{
    if constexpr (K >= 0) {
        add_bits<BC, WP, K>(acc, p);
    } else {
        for (uint64_t cc = c; cc; cc &= cc - 1) add_dispatch<BC, WP>(__builtin_ctzll(cc), acc, p);
    }
}

// [n < S] per lane over BC planes.
template <int BC>
__device__ __forceinline__ uint32_t less_than(const uint32_t (&n)[BC], const uint32_t (&S)[BC])
{
    uint32_t br = 0;
#pragma unroll
    for (int q = 0; q < BC; ++q) br = BWG_OP3(n[q], S[q], br, L_BORROW);
    return br;
}

template <int W>
__device__ __forceinline__ uint32_t less_than_w(const uint32_t (&j)[W], const uint32_t (&x)[W])
{
    uint32_t br = 0;
#pragma unroll
    for (int q = 0; q < W; ++q) br = BWG_OP3(j[q], x[q], br, L_BORROW);
    return br;
}

template <int P>
__device__ __forceinline__ void load_site(const uint32_t *p, uint32_t (&l)[P], uint32_t (&d)[P],
                                          uint32_t (&a)[P])
{
    if constexpr (P == 4) {
        const uint4 *v = reinterpret_cast<const uint4 *>(p);
        const uint4 x = v[0], y = v[1], z = v[2];
        l[0] = x.x; l[1] = x.y; l[2] = x.z; l[3] = x.w;
        d[0] = y.x; d[1] = y.y; d[2] = y.z; d[3] = y.w;
        a[0] = z.x; a[1] = z.y; a[2] = z.z; a[3] = z.w;
    } else {
#pragma unroll
        for (int q = 0; q < P; ++q) {
            l[q] = p[q];
            d[q] = p[P + q];
            a[q] = p[2 * P + q];
        }
    }
}

template <int P>
__device__ __forceinline__ void store_site(uint32_t *p, const uint32_t (&l)[P],
                                           const uint32_t (&d)[P], const uint32_t (&a)[P])
{
    if constexpr (P == 4) {
        uint4 *v = reinterpret_cast<uint4 *>(p);
        v[0] = make_uint4(l[0], l[1], l[2], l[3]);
        v[1] = make_uint4(d[0], d[1], d[2], d[3]);
        v[2] = make_uint4(a[0], a[1], a[2], a[3]);
    } else {
#pragma unroll
        for (int q = 0; q < P; ++q) {
            p[q] = l[q];
            p[P + q] = d[q];
            p[2 * P + q] = a[q];
        }
    }
}

// ---- a site's reaction with weights known at compile time -------------------
// Every quantity in exactly the planes its largest value over a site's states
// (at most T = 2^P - 1 molecules) needs, and no plane that is known to be zero.

constexpr int lat_bits(uint64_t v) { return v ? 1 + lat_bits(v >> 1) : 0; }
constexpr int lat_ctz(uint64_t v) { return v & 1 ? 0 : 1 + lat_ctz(v >> 1); }

// out (WO planes) = a (WA planes) + b (WB planes), the sum known to fit.
template <int WO, int WA, int WB>
__device__ __forceinline__ void add_planes(uint32_t (&out)[WO], const uint32_t (&a)[WA],
                                           const uint32_t (&b)[WB])
{
    constexpr int WMIN = WA < WB ? WA : WB, WMAX = WA < WB ? WB : WA;
    uint32_t c = 0;
#pragma unroll
    for (int q = 0; q < WO; ++q) {
        if (q >= WMAX) {
            out[q] = c;  // the last carry
            continue;
        }
        const uint32_t u = q < WMIN || WA > WB ? a[q < WA ? q : 0] : b[q < WB ? q : 0];
        const uint32_t v = q < WMIN ? b[q < WB ? q : 0] : c;
        if (q > 0 && q < WMIN) {
            out[q] = BWG_OP3(u, v, c, L_XOR3);
            c = BWG_OP3(u, v, c, L_MAJ);
        } else {
            out[q] = u ^ v;
            c = u & v;
        }
    }
}

// x * y of two 4-plane numbers with x + y <= 15: at most 56, six planes.
__device__ __forceinline__ void mul_6(uint32_t (&p)[6], const uint32_t (&x)[4],
                                      const uint32_t (&y)[4])
{
    constexpr uint32_t L_AND3 = lut(TA & TB & TC);
    uint32_t t, c;
    p[0] = x[0] & y[0];
    t = x[0] & y[1];
    p[1] = BWG_OP3(x[1], y[0], t, L_ANDXOR);
    c = BWG_OP3(x[1], y[0], t, L_AND3);
    uint32_t u = x[2] & y[0];
    t = x[1] & y[1];
    p[2] = BWG_OP3(u, t, c, L_XOR3);
    c = BWG_OP3(u, t, c, L_MAJ);
    u = x[3] & y[0];
    t = x[2] & y[1];
    p[3] = BWG_OP3(u, t, c, L_XOR3);
    c = BWG_OP3(u, t, c, L_MAJ);
    p[4] = BWG_OP3(x[3], y[1], c, L_ANDXOR);
    p[5] = BWG_OP3(x[3], y[1], c, L_AND3);
    // + x y_2 2^2
    c = BWG_OP3(x[0], y[2], p[2], L_AND3);
    p[2] = BWG_OP3(x[0], y[2], p[2], L_ANDXOR);
    t = x[1] & y[2];
    u = BWG_OP3(p[3], t, c, L_MAJ);
    p[3] = BWG_OP3(p[3], t, c, L_XOR3);
    t = x[2] & y[2];
    c = BWG_OP3(p[4], t, u, L_MAJ);
    p[4] = BWG_OP3(p[4], t, u, L_XOR3);
    t = x[3] & y[2];
    p[5] = BWG_OP3(p[5], t, c, L_XOR3);
    // + x y_3 2^3
    c = BWG_OP3(x[0], y[3], p[3], L_AND3);
    p[3] = BWG_OP3(x[0], y[3], p[3], L_ANDXOR);
    t = x[1] & y[3];
    u = BWG_OP3(p[4], t, c, L_MAJ);
    p[4] = BWG_OP3(p[4], t, c, L_XOR3);
    t = x[2] & y[3];
    p[5] = BWG_OP3(p[5], t, u, L_XOR3);
}

// acc (W planes, in planes [0, top) so far) +- x << SH.
template <int W, int P, int SH, bool NEG>
__device__ __forceinline__ void acc_digit(uint32_t (&acc)[W], const uint32_t (&x)[P])
{
    uint32_t c = 0;
#pragma unroll
    for (int q = SH; q < W; ++q) {
        const bool in = q - SH < P;
        const uint32_t v = in ? x[q - SH < P ? q - SH : 0] : 0u, o = acc[q];
        if (q == SH) {
            acc[q] = o ^ v;
            c = NEG ? ~o & v : o & v;
        } else if (in) {
            acc[q] = BWG_OP3(o, v, c, L_XOR3);
            c = NEG ? BWG_OP3(o, v, c, L_BORROW) : BWG_OP3(o, v, c, L_MAJ);
        } else {
            acc[q] = o ^ c;
            c = NEG ? ~o & c : o & c;
        }
    }
}

// acc = K x over the signed digits of K (no two neighbouring ones), the
// highest first.
template <int W, int P, int64_t K, int k = 40>
__device__ __forceinline__ void times_const(uint32_t (&acc)[W], const uint32_t (&x)[P])
{
    constexpr int64_t pos = (3 * K & ~K) >> 1, neg = (K & ~(3 * K)) >> 1;
    if constexpr (k >= 0) {
        if constexpr (k < W && ((pos >> k) & 1)) acc_digit<W, P, k, false>(acc, x);
        if constexpr (k < W && ((neg >> k) & 1)) acc_digit<W, P, k, true>(acc, x);
        times_const<W, P, K, k - 1>(acc, x);
    }
}

// Borrow of n[0 .. WN) - s[0 .. WS) (WS <= WN) from the borrow in.
template <int WN, int WS>
__device__ __forceinline__ uint32_t borrow_of(const uint32_t *n, const uint32_t (&s)[WS],
                                              uint32_t br)
{
#pragma unroll
    for (int q = 0; q < WN; ++q)
        br = q < WS ? BWG_OP3(n[q], s[q < WS ? q : 0], br, L_BORROW) : ~n[q] & br;
    return br;
}

// Widths of the weights c_u, c_a = c_i = 2^F (F planes of S_3 .. S_5 are those
// of S_2 = 2 U, so the comparisons share one borrow below them).
template <int P, int64_t CU, int64_t CA, int64_t CI>
struct LatWidths {
    static constexpr bool CT = P == 4 && CU > 0 && CA > 0 && CA == CI && (CA & (CA - 1)) == 0;
    static constexpr int T = (1 << P) - 1;
    static constexpr int F = CT ? lat_ctz((uint64_t)CA) : 0;
    static constexpr int UW = CT ? lat_bits((uint64_t)CU * T) : 1;         // U = c_u A
    static constexpr int64_t most()
    {
        int64_t m = 0;
        for (int64_t a = 0; a <= T; ++a)
            for (int64_t l = 0; a + l <= T; ++l)
                for (int64_t d = 0; a + l + d <= T; ++d) {
                    const int64_t w = 2 * CU * a + CA * (a * l + a * d) + CI * l * d;
                    m = w > m ? w : m;
                }
        return m;
    }
    static constexpr int64_t MOST = CT ? most() : 1;
    static constexpr int SW = lat_bits((uint64_t)MOST);                     // selection planes
    static constexpr int HU = UW + 1 - F;                                   // 2 U >> F
    static constexpr int H3 = lat_bits(((uint64_t)(2 * CU * T) >> F) + 56);
    static constexpr bool SPLIT = CT && HU > 0 && HU <= 6 && UW > 1 && F > 1;
};

// The event's changers from its threshold planes n (SW planes): lanes of
// A -> L or A + L -> 2L (mL), A -> D or A + D -> 2D (mD), L + D -> 2A (mI).
// 240 instructions for c = (246, 246, 2048, 2048, 2048), where forming every
// S_r in 19 planes and comparing each over all of them took 480.
template <int64_t CU, int64_t CA, int64_t CI>
__device__ __forceinline__ void lat_select(const uint32_t *n, const uint32_t (&l)[4],
                                           const uint32_t (&d)[4], const uint32_t (&x)[4],
                                           uint32_t &mL, uint32_t &mD, uint32_t &mI)
{
    using Wd = LatWidths<4, CU, CA, CI>;
    constexpr int F = Wd::F, UW = Wd::UW, SW = Wd::SW, HU = Wd::HU, HW = SW - F;
    uint32_t U[UW];
#pragma unroll
    for (int q = 0; q < UW; ++q) U[q] = 0;
    times_const<UW, 4, CU>(U, x);
    // S_1 = U and S_2 = 2 U
    const uint32_t lt1 = borrow_of<SW, UW>(n, U, 0u);
    uint32_t low = 0;  // borrow of n - 2 U below plane F
#pragma unroll
    for (int q = 1; q < F; ++q)
        low = q - 1 < UW ? BWG_OP3(n[q], U[q - 1 < UW ? q - 1 : 0], low, L_BORROW) : ~n[q] & low;
    uint32_t h2[HU];
#pragma unroll
    for (int q = 0; q < HU; ++q) h2[q] = U[F - 1 + q];
    const uint32_t lt2 = borrow_of<HW, HU>(n + F, h2, low);
    // S_r >> F for r = 3, 4, 5 (A L + A D and their sum with the rest of 2 U
    // stay below 64, with L D below 128: checked by the widths)
    uint32_t p[6], h3[6], h4[6], h5[HW];
    static_assert(Wd::H3 <= 6 && HW >= 6, "site weights beyond the planes below");
    static_assert((Wd::MOST & (Wd::MOST - 1)) != 0, "2^B_r equal to the largest weight");
    mul_6(p, x, l);
    add_planes<6, HU, 6>(h3, h2, p);
    const uint32_t lt3 = borrow_of<HW, 6>(n + F, h3, low);
    mul_6(p, x, d);
    add_planes<6, 6, 6>(h4, h3, p);
    const uint32_t lt4 = borrow_of<HW, 6>(n + F, h4, low);
    mul_6(p, l, d);
    if constexpr (HW == 6) {
        add_planes<6, 6, 6>(h5, h4, p);
    } else {
        uint32_t t[7];
        add_planes<7, 6, 6>(t, h4, p);
#pragma unroll
        for (int q = 0; q < HW; ++q) h5[q] = q < 7 ? t[q < 7 ? q : 0] : 0u;
    }
    const uint32_t lt5 = borrow_of<HW, HW>(n + F, h5, low);
    mL = lt1 | (lt3 & ~lt2);
    mD = (lt2 & ~lt1) | (lt4 & ~lt3);
    mI = lt5 & ~lt4;
}

// Reaction component of a site (planes l, d, x already loaded, updated in
// place) for the lanes in act, n the event's threshold planes (4 NQ of them,
// those from B_r on still drawn); returns the lanes whose state changed (the
// caller stores the planes if any did).
template <int P, int BC, int NQ, int64_t CU, int64_t CA, int64_t CI>
__device__ __forceinline__ uint32_t lat_reaction(uint32_t (&l)[P], uint32_t (&d)[P],
                                                 uint32_t (&x)[P], const LatArgs &a,
                                                 uint32_t (&n)[4 * NQ], uint32_t act)
{
    constexpr int WP = 2 * P;
    using Wd = LatWidths<P, CU, CA, CI>;
    const LatShape &sh = a.sh;
    uint32_t mL, mD, mI;
    if constexpr (Wd::SPLIT) {
        lat_select<CU, CA, CI>(n, l, d, x, mL, mD, mI);
    } else {
        static_assert(BC <= 4 * NQ, "threshold planes");
        uint32_t t[BC];
#pragma unroll
        for (int q = 0; q < BC; ++q) t[q] = q < sh.B_r ? n[q] : 0u;
        // S_1 = cu A, S_2 = 2 cu A, S_3 = S_2 + c_a A L, S_4 = S_3 + c_a A D,
        // S_5 = S_4 + c_i L D (table order A->L, A->D, A+L->2L, A+D->2D, L+D->2A)
        uint32_t X[BC];
#pragma unroll
        for (int q = 0; q < BC; ++q) X[q] = 0;
        add_const_mul<BC, P, CU>(X, x, sh.cu);
        const uint32_t lt1 = less_than<BC>(t, X);
        uint32_t S[BC];
        S[0] = 0;
#pragma unroll
        for (int q = 1; q < BC; ++q) S[q] = X[q - 1];
        const uint32_t lt2 = less_than<BC>(t, S);
        uint32_t pr[WP];
        mul_planes<P, WP>(pr, x, l);
        add_const_mul<BC, WP, CA>(S, pr, sh.ca);
        const uint32_t lt3 = less_than<BC>(t, S);
        mul_planes<P, WP>(pr, x, d);
        add_const_mul<BC, WP, CA>(S, pr, sh.ca);
        const uint32_t lt4 = less_than<BC>(t, S);
        mul_planes<P, WP>(pr, l, d);
        add_const_mul<BC, WP, CI>(S, pr, sh.ci);
        const uint32_t lt5 = less_than<BC>(t, S);
        mL = lt1 | (lt3 & ~lt2);
        mD = (lt2 & ~lt1) | (lt4 & ~lt3);
        mI = lt5 & ~lt4;
    }
    mL &= act;
    mD &= act;
    mI &= act;
    const uint32_t ch = mL | mD | mI;
    if (ch) {
        add_pm1<P>(l, mL, mI);
        add_pm1<P>(d, mD, mI);
        add_m1_p2<P>(x, mL | mD, mI);
    }
    return ch;
}

// Hop component out of one site into another (planes already loaded,
// updated in place; self: the lattice is one site wide along that axis and
// the hop changes nothing).  Sets the lanes that moved (the caller stores
// both sites' planes if any did) and the lanes blocked by a full
// destination.
template <int P>
__device__ __forceinline__ void lat_hop(bool self, uint32_t (&l)[P],
                                        uint32_t (&d)[P], uint32_t (&x)[P], uint32_t (&l2)[P],
                                        uint32_t (&d2)[P], uint32_t (&x2)[P],
                                        const uint32_t (&o)[4], uint32_t act, uint32_t &moved,
                                        uint32_t &blocked)
{
    static_assert(P <= 4, "hop index from one Philox quad");
    uint32_t j[P];
#pragma unroll
    for (int q = 0; q < P; ++q) j[q] = o[q];
    uint32_t al[P], tot[P];
    add_planes<P, P, P>(al, x, l);  // site totals are at most T = 2^P - 1: no carry out
    add_planes<P, P, P>(tot, al, d);
    const uint32_t hA = less_than_w<P>(j, x);
    const uint32_t cAL = less_than_w<P>(j, al);
    const uint32_t any = less_than_w<P>(j, tot) & act;
    const uint32_t sA = hA & act, sL = cAL & ~hA & act, sD = any & ~cAL;
    uint32_t t1[P], t2[P], full = ~0u;
    add_planes<P, P, P>(t1, x2, l2);
    add_planes<P, P, P>(t2, t1, d2);
#pragma unroll
    for (int q = 0; q < P; ++q) full &= t2[q];
    const uint32_t mv = any & ~full;
    blocked = any & full;
    moved = self ? 0u : mv;
    if (self || !mv) return;
    add_pm1<P>(x, 0u, sA & mv);
    add_pm1<P>(l, 0u, sL & mv);
    add_pm1<P>(d, 0u, sD & mv);
    add_pm1<P>(x2, sA & mv, 0u);
    add_pm1<P>(l2, sL & mv, 0u);
    add_pm1<P>(d2, sD & mv, 0u);
}

// The 4 NQ threshold planes of event e for the lanes of word G.
template <int NQ>
__device__ __forceinline__ void event_draw(const LatArgs &a, uint32_t G, uint64_t e,
                                           uint32_t (&n)[4 * NQ])
{
    EventDraw<NQ> dr;
    dr.k0 = (uint32_t)a.seed;
    dr.k1 = (uint32_t)(a.seed >> 32);
    dr.net_id = a.net_id;
    dr.G = G;
    asm volatile("" : "+v"(dr.G));  // not hoisted out of the event loop
    dr.set_word((uint32_t)(e >> 32) & 0xFFFFu);
    dr.draw((uint32_t)e, n);
}

// Lanes of a word that run event e (E_l <= e < Et_l); kept out of line so the
// 64 window bounds are not held in registers across the event loop.
__device__ __noinline__ uint32_t lanes_at(const uint64_t *sE, const uint64_t *sEt, uint32_t pend,
                                          uint64_t e)
{
    uint32_t act = 0;
    for (int l = 0; l < 32; ++l)
        if (((pend >> l) & 1u) && sE[l] <= e && e < sEt[l]) act |= 1u << l;
    return act;
}

// One workgroup per slice of WS consecutive words of a group, BLOCK
// threads: thread t works on word t mod WS of the slice and on every
// (BLOCK / WS)-th event of a layer, so the WS words of one event read
// WS * 12 contiguous planes.  A launch covers the band of groups
// [a.g0, a.g0 + a.ng): the host sizes bands so that their site planes fit the
// last-level (infinity) cache.  Slices are spread so that the slices of a
// group run on one XCD (workgroups go to the 8 XCDs in turn), where they
// share the group's schedule in L2.  Runs the events of chunks chunk0 ..
// chunk0+n_chunks-1 layer by layer.
//
// ST > 0 (P = 4): the planes of sites 0 .. ST/WS - 1 of the slice's words
// are copied into LDS when the launch starts and back when it ends, and
// every event on those sites reads and writes LDS instead of memory.  LDS
// holds ST = 3360 (site, word) pairs (158 KB of the CU's 160 KB): with 4-word
// slices the first 840 sites of each word, a fifth of a 64 x 64 lattice.
// Within a layer no two events share a site, so the LDS copy needs no more
// ordering than the memory planes do.  (One word per workgroup would hold
// 3392 sites, 83 % of a 64 x 64 lattice, but a word's layers hold ~550
// independent events on average, half of the 1024 threads a CU needs to
// hide latency: measured slower.)
//
// Bound by the latency of a layer: schedule record, then planes, then about
// 150 (hop) or 430 (reaction) instructions, then the barrier, at one
// workgroup of 16 waves a CU.  The next event's loads overlap the current
// event's arithmetic only as long as nothing spills (a scratch load waits in
// order behind them), hence two register sets that trade places instead of a
// copied one, the windows in LDS, 32-bit plane offsets and draws whose
// per-word part is formed again for each event.  A launch of the 64 x 64
// lattice at 2^16 replicas takes 3102 us (3344 before, with the run-time
// selection and copied registers; 3435 with 17 spilled registers, 3847 with
// the records read a further event ahead); a pass of the 21 x 17 one at 1000
// replicas 1681 us (2042).  The staged kernel sits on the edge: 126 registers
// with layer bounds of their own, 128 and two spilled (32 bytes of scratch a
// lane) since a bound shares its word with the layer's first hop, which
// lat_word_kernel needs; a pass of the 64 x 64 lattice did not change by it.
template <int P, int BC, int64_t CU, int64_t CA, int64_t CI, int WS, int BLOCK, int ST>
__global__ __launch_bounds__(BLOCK, 1) void lat_event_kernel(LatArgs a)
{
    static_assert(ST == 0 || P == 4, "staging holds 12 planes per site and word");
    constexpr int NP = 3 * P;
    constexpr int NSL = LAT_GROUP_WORDS / WS;   // slices per group
    constexpr int EV = BLOCK / WS;              // events in flight per workgroup
    const uint32_t nwg = a.ng * NSL;
    const uint32_t per_xcd = (nwg + 7) / 8;
    const uint32_t v = (blockIdx.x % 8) * per_xcd + blockIdx.x / 8;
    if (v >= nwg) return;
    const uint32_t g = a.g0 + v / NSL;
    const uint64_t w0 = (uint64_t)g * LAT_GROUP_WORDS + (v % NSL) * WS;
    const uint64_t words = (a.M + 31) / 32;
    if (w0 >= words) return;
    const uint32_t tid = threadIdx.x, lw = tid % WS, slot = tid / WS;
    const uint64_t w = w0 + lw;
    __shared__ uint64_t sE[WS][32], sEt[WS][32];
    __shared__ uint32_t sred[2][WS];

    for (uint32_t i = tid; i < WS * 32; i += BLOCK) {
        const uint64_t r = 32 * w0 + i;
        const bool ok = r < a.M;
        sE[i / 32][i % 32] = ok ? a.E[r] : 0;
        sEt[i / 32][i % 32] = ok ? a.Et[r] : 0;
    }
    if (tid < 2 * WS) sred[tid / WS][tid % WS] = 0;
    __syncthreads();
    // window of each word over its pending lanes (E < Et): [lo, hi) holds every
    // event of the word, [blo, bhi) the events every pending lane runs; kept in
    // LDS, since only the start of a chunk needs them
    __shared__ uint64_t win[WS][4];
    __shared__ uint32_t spend[WS];
    if (tid < WS) {
        uint64_t lo = ~0ull, hi = 0, blo = 0, bhi = ~0ull;
        uint32_t p = 0;
        for (int l = 0; l < 32; ++l) {
            const uint64_t e0 = sE[tid][l], e1 = sEt[tid][l];
            if (e0 < e1) {
                p |= 1u << l;
                lo = min(lo, e0);
                hi = max(hi, e1);
                blo = max(blo, e0);
                bhi = min(bhi, e1);
            }
        }
        win[tid][0] = lo;
        win[tid][1] = hi;
        win[tid][2] = blo;
        win[tid][3] = bhi;
        spend[tid] = p;
    }
    __syncthreads();
    const uint32_t pend = spend[lw];
    // the union of the slice's windows
    uint64_t wlo = ~0ull, whi = 0;
    for (int k = 0; k < WS; ++k) {
        wlo = min(wlo, win[k][0]);
        whi = max(whi, win[k][1]);
    }
    const int S = a.sh.S;
    uint32_t n_real = 0, n_blocked = 0;
    // the launch's events of this slice: [wlo, whi) within its chunks
    const uint64_t c_lo = a.base + (uint64_t)a.chunk0 * LAT_CH;
    const uint64_t c_hi = c_lo + (uint64_t)a.n_chunks * LAT_CH;
    const bool runs = whi > wlo && wlo < c_hi && whi > c_lo;
    // stage[(st WS + word) 3 + part]: the slice's WS words of site st
    __shared__ uint4 stage[ST > 0 ? 3 * ST : 1];
    const uint32_t nst = ST > 0 ? min((uint32_t)S, (uint32_t)(ST / WS)) : 0u;
    if (ST > 0 && runs) {
        for (uint32_t k = tid; k < 3 * WS * nst; k += BLOCK)
            stage[k] = reinterpret_cast<const uint4 *>(
                site_planes(a.planes, w0 + (k / 3) % WS, k / (3 * WS), S, NP))[k % 3];
        __syncthreads();
    }
    // planes of site st of this thread's word: LDS for staged sites.  The two
    // cases stay separate instructions (LDS and memory loads wait on their own
    // counters, so the next event's memory loads still overlap this event).
    // A group's planes start at a wave-uniform address, the rest is a 32-bit
    // offset (4096 sites of 64 words).
    uint32_t *const gplanes = a.planes + (uint64_t)g * S * LAT_GROUP_WORDS * NP;
    const uint32_t wofs = (uint32_t)(w % LAT_GROUP_WORDS);
    auto load_at = [&](uint32_t st, uint32_t (&l_)[P], uint32_t (&d_)[P], uint32_t (&x_)[P]) {
        if (ST > 0 && st < nst)
            load_site<P>(reinterpret_cast<const uint32_t *>(&stage[3 * (st * WS + lw)]), l_, d_, x_);
        else
            load_site<P>(gplanes + (st * LAT_GROUP_WORDS + wofs) * NP, l_, d_, x_);
    };
    auto store_at = [&](uint32_t st, const uint32_t (&l_)[P], const uint32_t (&d_)[P],
                        const uint32_t (&x_)[P]) {
        if (ST > 0 && st < nst)
            store_site<P>(reinterpret_cast<uint32_t *>(&stage[3 * (st * WS + lw)]), l_, d_, x_);
        else
            store_site<P>(gplanes + (st * LAT_GROUP_WORDS + wofs) * NP, l_, d_, x_);
    };
    if (runs) {
        // the draws' per-word part is formed again for every event: kept in
        // registers it spilled others to scratch, whose loads wait in order
        // behind the next event's planes
        constexpr int NQ = (BC + 3) / 4;
        for (uint32_t c = 0; c < a.n_chunks; ++c) {
            const uint32_t *slotp = a.sched + ((uint64_t)g * LAT_NCB + c) * LAT_SLOT;
            const uint32_t *recs = slotp;
            const uint32_t *offs = slotp + 2 * LAT_CH;
            const uint64_t cbase = a.base + (uint64_t)(a.chunk0 + c) * LAT_CH;
            if (cbase >= whi || cbase + LAT_CH <= wlo) continue;
            const uint32_t nl = offs[0];
            // whether every pending lane of every word runs the whole chunk
            bool full = true;
            for (int k = 0; k < WS; ++k)
                full = full && (win[k][0] > win[k][1] ||
                                (win[k][2] <= cbase && win[k][3] >= cbase + LAT_CH));
            full = __builtin_amdgcn_readfirstlane(full);
            // one event with the planes of its sites
            struct Fetched {
                uint32_t rec, s2, act;
                uint32_t l[P], d[P], x[P], l2[P], d2[P], x2[P];
            };
            auto fetch = [&](Fetched &f, uint32_t i) {
                f.rec = recs[i];
                const uint32_t off = f.rec >> 16, st = (f.rec >> 3) & 0x1FFFu, kind = f.rec & 7u;
                f.act = pend;
                if (!full) {
                    const uint64_t e = cbase + off;
                    if (e < win[lw][0] || e >= win[lw][1])
                        f.act = 0;
                    else if (e < win[lw][2] || e >= win[lw][3])
                        f.act = lanes_at(sE[lw], sEt[lw], pend, e);
                }
                f.s2 = kind ? lat_neighbour(a.sh, st, kind - 1) : st;
                if (f.act) {
                    load_at(st, f.l, f.d, f.x);
                    if (kind) load_at(f.s2, f.l2, f.d2, f.x2);
                }
            };
            auto apply = [&](Fetched &f) {
                if (!f.act) return;
                const uint64_t e = cbase + (f.rec >> 16);
                const uint32_t st = (f.rec >> 3) & 0x1FFFu;
                if ((f.rec & 7u) == 0) {
                    uint32_t n[4 * NQ];
                    event_draw<NQ>(a, (uint32_t)w, e, n);
                    const uint32_t ch =
                        lat_reaction<P, BC, NQ, CU, CA, CI>(f.l, f.d, f.x, a, n, f.act);
                    if (ch) store_at(st, f.l, f.d, f.x);
                    n_real += __popc(ch);
                } else {
                    uint32_t o[4], mv, bl;
                    event_draw<1>(a, (uint32_t)w, e, o);
                    lat_hop<P>(f.s2 == st, f.l, f.d, f.x, f.l2, f.d2, f.x2, o, f.act, mv, bl);
                    if (mv) {
                        store_at(st, f.l, f.d, f.x);
                        store_at(f.s2, f.l2, f.d2, f.x2);
                    }
                    n_real += __popc(mv);
                    n_blocked += __popc(bl);
                }
            };
            for (uint32_t L = 0; L < nl; ++L) {
                const uint32_t end = offs[2 + L] & 0xFFFFu;
                // the planes of this thread's next event of the layer are
                // loaded while the current one computes (events of a layer
                // touch disjoint sites, so nothing else writes them
                // meanwhile), in two sets of registers that trade places
                uint32_t idx = (offs[1 + L] & 0xFFFFu) + slot;
                Fetched f0, f1;
                if (idx < end) fetch(f0, idx);
                while (idx < end) {
                    idx += EV;
                    if (idx < end) fetch(f1, idx);
                    apply(f0);
                    if (idx >= end) break;
                    idx += EV;
                    if (idx < end) fetch(f0, idx);
                    apply(f1);
                }
                __syncthreads();
            }
        }
    }
    if (ST > 0 && runs) {
        __syncthreads();
        for (uint32_t k = tid; k < 3 * WS * nst; k += BLOCK)
            reinterpret_cast<uint4 *>(
                site_planes(a.planes, w0 + (k / 3) % WS, k / (3 * WS), S, NP))[k % 3] = stage[k];
    }
    // per-word totals of real events and blocked hops
    if (n_real) atomicAdd(&sred[0][lw], n_real);
    if (n_blocked) atomicAdd(&sred[1][lw], n_blocked);
    __syncthreads();
    if (tid < WS && w < words) {
        a.real[w] += sred[0][tid];
        a.blocked[w] += sred[1][tid];
    }
}

// One workgroup per word, all of the word's sites (S <= ST) in LDS: for
// ensembles of fewer words than fill the chip with 4-word slices, where a
// layer of a small lattice holds fewer events than a workgroup has threads and
// its latency is all that counts.  A chunk's schedule is copied to LDS as
// well.  The two halves of the workgroup take the layers in turn: while one
// half reads planes, selects and writes them back, the other draws the
// thresholds of the next layer's events, which depend on nothing but the
// record.  In a half, the first waves take a layer's reactions and the others
// its hops, so that no wave runs both paths.  512 threads: with 1024 a layer's
// barrier costs more than the further events in flight give (793 us instead of
// 664).  Bound by the instructions of one wave, selection on one side and draws
// on the other, with 40 % of the issue slots used: 599 us for 60000 events of
// 1000 replicas on 21 x 17 sites, 549 layers (1401 in the kernel above).
template <int P, int BC, int64_t CU, int64_t CA, int64_t CI, int BLOCK, int ST>
__global__ __launch_bounds__(BLOCK, 1) void lat_word_kernel(LatArgs a)
{
    static_assert(P == 4, "staging holds 12 planes per site");
    constexpr int NP = 3 * P, NQ = (BC + 3) / 4, HALF = BLOCK / 2, HW = HALF / 64;
    const uint64_t w = (uint64_t)a.g0 * LAT_GROUP_WORDS + blockIdx.x;
    const uint32_t g = (uint32_t)(w / LAT_GROUP_WORDS);
    if (w >= (a.M + 31) / 32 || g >= a.g0 + a.ng) return;
    const uint32_t tid = threadIdx.x;
    const int S = a.sh.S;
    __shared__ uint4 stage[3 * ST];
    __shared__ uint4 recs4[LAT_CH / 4], offs[LAT_CH / 4 + 1];
    const uint32_t *const recs = reinterpret_cast<const uint32_t *>(recs4);
    const uint32_t *const bounds = reinterpret_cast<const uint32_t *>(offs) + 1;
    __shared__ uint4 window[8];
    __shared__ uint32_t sred[2];

    // the windows of the word's pending lanes (E < Et): [lo, hi) holds every
    // event, [blo, bhi) the events every pending lane runs
    const uint64_t r = 32 * w + (tid & 31);
    const uint64_t e0 = r < a.M ? a.E[r] : 0, e1 = r < a.M ? a.Et[r] : 0;
    const uint32_t pend = (uint32_t)__ballot(e0 < e1);
    const uint64_t lo = wave_min_u64(e0 < e1 ? e0 : ~0ull), hi = wave_max_u64(e0 < e1 ? e1 : 0);
    const uint64_t blo = wave_max_u64(e0 < e1 ? e0 : 0), bhi = wave_min_u64(e0 < e1 ? e1 : ~0ull);
    if (tid < 2) sred[tid] = 0;
    // the launch's events of this word: [lo, hi) within its chunks
    const uint64_t c_lo = a.base + (uint64_t)a.chunk0 * LAT_CH;
    const uint64_t c_hi = c_lo + (uint64_t)a.n_chunks * LAT_CH;
    if (hi <= lo || lo >= c_hi || hi <= c_lo) return;

    for (uint32_t k = tid; k < 3u * S; k += BLOCK)
        stage[k] = reinterpret_cast<const uint4 *>(site_planes(a.planes, w, k / 3, S, NP))[k % 3];
    uint32_t n_real = 0, n_blocked = 0;
    // the second half numbers its waves backwards: waves go to the four SIMDs
    // in turn, and so one half's selections meet the other half's hops there,
    // not its reactions' draws
    const uint32_t half = tid / HALF;
    const uint32_t ht = half ? (tid % HALF) ^ (HALF - 64) : tid;
    // waves of a half that take reactions, by their share of the events
    const uint32_t rw = min(
        max((uint32_t)((float)HW * (float)a.sh.W_R / (float)a.sh.Wsite + 0.5f), 1u),
        (uint32_t)HW - 1);
    const bool hops = __builtin_amdgcn_readfirstlane(ht >= 64 * rw);
    const uint32_t first = hops ? ht - 64 * rw : ht;
    const uint32_t stride = hops ? HALF - 64 * rw : 64 * rw;

    for (uint32_t c = 0; c < a.n_chunks; ++c) {
        const uint64_t cbase = a.base + (uint64_t)(a.chunk0 + c) * LAT_CH;
        if (cbase >= hi || cbase + LAT_CH <= lo) continue;
        const uint32_t *slotp = a.sched + ((uint64_t)g * LAT_NCB + c) * LAT_SLOT;
        const uint32_t nl = slotp[2 * LAT_CH];
        if (nl == 0) continue;
        const bool full = blo <= cbase && bhi >= cbase + LAT_CH;
        // the whole slot of records, so that no load waits for their number
        static_assert(LAT_CH % (4 * BLOCK) == 0 && LAT_SLOT % 4 == 0, "copies of 16 bytes");
        uint4 t[LAT_CH / (4 * BLOCK)];
#pragma unroll
        for (int j = 0; j < LAT_CH / (4 * BLOCK); ++j)
            t[j] = reinterpret_cast<const uint4 *>(slotp)[tid + j * BLOCK];
        // each lane's events of the chunk: the first and their number
        if (!full && tid < 32) {
            const uint64_t b = min(max(e0, cbase), cbase + LAT_CH);
            const uint64_t n = max(min(e1, cbase + LAT_CH), b) - b;
            reinterpret_cast<uint32_t *>(window)[tid] =
                e0 < e1 ? (uint32_t)(b - cbase) | ((uint32_t)n << 16) : 0u;
        }
        for (uint32_t k = tid; k <= (nl + 1) / 4; k += BLOCK)
            offs[k] = reinterpret_cast<const uint4 *>(slotp + 2 * LAT_CH)[k];
#pragma unroll
        for (int j = 0; j < LAT_CH / (4 * BLOCK); ++j) recs4[tid + j * BLOCK] = t[j];
        __syncthreads();

        uint32_t idx = 0, end = 0, rec = 0, act = 0, n[4 * NQ];
        // the drawn planes of this thread's event idx
        auto draw = [&]() {
            act = 0;
            if (idx >= end) return;
            rec = recs[idx];
            const uint32_t off = rec >> 16;
            const uint64_t e = cbase + off;
            if (full) {
                act = pend;
            } else {
                for (int k = 0; k < 8; ++k) {
                    const uint4 v = window[k];
                    const uint32_t m = (uint32_t)(off - (v.x & 0xFFFFu) < v.x >> 16) |
                                       (uint32_t)(off - (v.y & 0xFFFFu) < v.y >> 16) << 1 |
                                       (uint32_t)(off - (v.z & 0xFFFFu) < v.z >> 16) << 2 |
                                       (uint32_t)(off - (v.w & 0xFFFFu) < v.w >> 16) << 3;
                    act |= m << (4 * k);
                }
            }
            if (!act) return;
            if (hops) {
                uint32_t o[4];
                event_draw<1>(a, (uint32_t)w, e, o);
#pragma unroll
                for (int q = 0; q < 4; ++q) n[q] = o[q];
            } else {
                event_draw<NQ>(a, (uint32_t)w, e, n);
            }
        };
        auto prepare = [&](uint32_t L) {
            idx = end = 0;
            if (L < nl) {
                const uint32_t o0 = bounds[L];
                idx = (hops ? o0 >> 16 : o0 & 0xFFFFu) + first;
                end = hops ? bounds[L + 1] & 0xFFFFu : o0 >> 16;
            }
            draw();
        };
        auto apply = [&]() {
            if (!act) return;
            const uint32_t st = (rec >> 3) & 0x1FFFu;
            uint32_t *p = reinterpret_cast<uint32_t *>(&stage[3 * st]);
            uint32_t l[P], d[P], x[P];
            load_site<P>(p, l, d, x);
            if (!hops) {
                const uint32_t ch = lat_reaction<P, BC, NQ, CU, CA, CI>(l, d, x, a, n, act);
                if (ch) store_site<P>(p, l, d, x);
                n_real += __popc(ch);
            } else {
                const uint32_t s2 = lat_neighbour(a.sh, st, (rec & 7u) - 1);
                uint32_t *p2 = reinterpret_cast<uint32_t *>(&stage[3 * s2]);
                uint32_t l2[P], d2[P], x2[P], mv, bl;
                load_site<P>(p2, l2, d2, x2);
                const uint32_t o[4] = {n[0], n[1], n[2], n[3]};
                lat_hop<P>(s2 == st, l, d, x, l2, d2, x2, o, act, mv, bl);
                if (mv) {
                    store_site<P>(p, l, d, x);
                    store_site<P>(p2, l2, d2, x2);
                }
                n_real += __popc(mv);
                n_blocked += __popc(bl);
            }
        };
        if (half == 0) prepare(0);
        for (uint32_t L = 0; L < nl; ++L) {
            if ((L & 1) == half) {
                apply();
                for (idx += stride; idx < end; idx += stride) {
                    draw();
                    apply();
                }
            } else {
                prepare(L + 1);
            }
            __syncthreads();
        }
    }
    if (n_real) atomicAdd(&sred[0], n_real);
    if (n_blocked) atomicAdd(&sred[1], n_blocked);
    __syncthreads();
    for (uint32_t k = tid; k < 3u * S; k += BLOCK)
        reinterpret_cast<uint4 *>(site_planes(a.planes, w, k / 3, S, NP))[k % 3] = stage[k];
    if (tid == 0) {
        a.real[w] += sred[0];
        a.blocked[w] += sred[1];
    }
}

// ---- readouts --------------------------------------------------------------

// Species totals over sites of every replica: dst[i*3 + x].  A workgroup takes
// LAT_TOT_WORDS consecutive words (the piece of the launch starts at word w0):
// thread t adds the planes of word t mod 8 on every LAT_TOT_SUBS-th site to
// bit-sliced counters, so 32 replicas share an addition and the kernel is bound
// by reading the planes.  Counters meet over the 8 sites of a wave by shuffles
// and over the waves in LDS, where each (species, replica) picks out its bits.
// 97 us for the 402 MB of 64 x 64 sites of 2^16 replicas, 4.1 TB/s (450 with a
// thread per replica), with 71 of the counters' registers spilled.
constexpr int LAT_TOT_WORDS = 8, LAT_TOT_SUBS = 128;
constexpr int LAT_TOT_BLOCK = LAT_TOT_WORDS * LAT_TOT_SUBS;

template <int P>
__global__ __launch_bounds__(LAT_TOT_BLOCK) void lat_totals_kernel(const uint32_t *planes,
                                                                   uint64_t M, int S,
                                                                   int32_t *dst, uint64_t w0)
{
    // planes of a wave's sum over its 8 threads a word
    constexpr int PT = P + 8, NW = LAT_TOT_BLOCK / 64;
    static_assert((int64_t)LAT_MAX_SITES / LAT_TOT_SUBS * 8 * ((1 << P) - 1) < (1 << PT),
                  "counter planes");
    __shared__ uint32_t part[NW][3][PT][LAT_TOT_WORDS];
    const uint32_t t = threadIdx.x, lw = t % LAT_TOT_WORDS, sub = t / LAT_TOT_WORDS;
    const uint64_t wb = w0 + (uint64_t)blockIdx.x * LAT_TOT_WORDS;
    uint32_t c[3][PT];
#pragma unroll
    for (int k = 0; k < 3; ++k)
#pragma unroll
        for (int q = 0; q < PT; ++q) c[k][q] = 0;
    // several sites' loads in flight per thread
#pragma unroll 2
    for (uint32_t s = sub; s < (uint32_t)S; s += LAT_TOT_SUBS) {
        uint32_t l[P], d[P], x[P];
        load_site<P>(site_planes(planes, wb + lw, s, S, 3 * P), l, d, x);
        acc_digit<PT, P, 0, false>(c[0], l);
        acc_digit<PT, P, 0, false>(c[1], d);
        acc_digit<PT, P, 0, false>(c[2], x);
    }
#pragma unroll
    for (int o = LAT_TOT_WORDS; o < 64; o *= 2)
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            uint32_t y[PT];
#pragma unroll
            for (int q = 0; q < PT; ++q) y[q] = (uint32_t)__shfl_xor((int)c[k][q], o, 64);
            acc_digit<PT, PT, 0, false>(c[k], y);
        }
    if (t % 64 < LAT_TOT_WORDS)
#pragma unroll
        for (int k = 0; k < 3; ++k)
#pragma unroll
            for (int q = 0; q < PT; ++q) part[t / 64][k][q][lw] = c[k][q];
    __syncthreads();
    for (uint32_t o = t; o < 3 * 32 * LAT_TOT_WORDS; o += LAT_TOT_BLOCK) {
        const uint32_t r = o / 3, k = o % 3;
        int32_t v = 0;
        for (int j = 0; j < NW; ++j)
#pragma unroll
            for (int q = 0; q < PT; ++q)
                v += (int32_t)((part[j][k][q][r / 32] >> (r % 32)) & 1u) << q;
        const uint64_t i = 32 * wb + r;
        if (i < M) dst[3 * i + k] = v;
    }
}

// Site counts of replicas first .. first+count-1: dst[(k S + s) 3 + x].
__global__ void lat_sites_kernel(const uint32_t *planes, int S, int P, uint64_t first,
                                 uint64_t count, int32_t *dst)
{
    const uint64_t k = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const uint32_t s = blockIdx.y;
    if (k >= count) return;
    const uint64_t i = first + k;
    const uint64_t w = i >> 5;
    const uint32_t lane = i & 31;
    const uint32_t *p = site_planes(planes, w, s, S, 3 * P);
    for (int x = 0; x < 3; ++x) {
        int32_t v = 0;
        for (int q = 0; q < P; ++q) v |= (int32_t)((p[x * P + q] >> lane) & 1u) << q;
        dst[(k * S + s) * 3 + x] = v;
    }
}

// ee histogram from per-replica totals: n = L + D + A of the replica,
// bin = min(n_bins - 1, (L - D + n) n_bins / (2 n)), n = 0 in bin n_bins / 2.
__global__ void lat_histogram_kernel(const int32_t *tot, uint64_t M, int n_bins, uint64_t *dst)
{
    extern __shared__ uint32_t h[];
    for (int b = threadIdx.x; b < n_bins; b += blockDim.x) h[b] = 0;
    __syncthreads();
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < M;
         i += (uint64_t)gridDim.x * blockDim.x) {
        const int64_t L = tot[3 * i], D = tot[3 * i + 1], A = tot[3 * i + 2];
        const int64_t n = L + D + A;
        int64_t b = n_bins / 2;
        if (n > 0) b = min((int64_t)n_bins - 1, ((L - D + n) * n_bins) / (2 * n));
        atomicAdd(&h[b], 1u);
    }
    __syncthreads();
    for (int b = threadIdx.x; b < n_bins; b += blockDim.x)
        if (h[b]) atomicAdd((unsigned long long *)&dst[b], (unsigned long long)h[b]);
}

// ---- launchers ---------------------------------------------------------------

hipError_t launch_lat_init(uint32_t *planes, uint64_t words, uint64_t M, int S, int P, int mode,
                           const int32_t *sites_dev, const int32_t c3[3], int32_t lo, int32_t hi,
                           uint64_t seed, uint32_t net_id, uint64_t *E, uint64_t *Et,
                           uint64_t *real, uint64_t *blocked, hipStream_t s)
{
    if (mode == 0) {
        dim3 grid((unsigned)((words + 255) / 256), (unsigned)S);
        hipLaunchKernelGGL(lat_init_fixed_kernel, grid, dim3(256), 0, s, planes, words, M, S, P,
                           sites_dev, c3[0], c3[1], c3[2], E, Et, real, blocked);
    } else {
        const uint64_t reps = 64 * ((words + 1) / 2);
        dim3 grid((unsigned)((reps + 255) / 256),
                  (unsigned)((S + LAT_INIT_SITES - 1) / LAT_INIT_SITES));
        hipLaunchKernelGGL(lat_init_uniform_kernel, grid, dim3(256), 0, s, planes, words, M, S, P,
                           lo, hi, seed, net_id, E, Et, real, blocked);
    }
    return hipGetLastError();
}

hipError_t launch_lat_schedule(const LatArgs &a, uint32_t n_groups, hipStream_t s)
{
    hipLaunchKernelGGL(lat_schedule_kernel, dim3(n_groups * a.n_chunks),
                       dim3(LAT_SCHED_BLOCK), 0, s, a);
    return hipGetLastError();
}

// (id, P, BC, CU, CA, CI, WS, BLOCK, ST): species planes, threshold-plane
// capacity, the weights of A -> L / A -> D, A + L -> 2L / A + D -> 2D and
// L + D -> 2A (-1: taken at run time), words per slice, threads per
// workgroup (512 for the run-time weights, which need more registers) and
// (site, word) pairs staged in LDS (0: none; with one word per slice, the
// lattices that lat_word_kernel takes).
#define BWG_LAT_VARIANTS(X)                                                                   \
    X(0, 4, 19, 246, 2048, 2048, 4, 1024, 0) X(1, 4, 19, 246, 2048, 2048, 1, 1024, 0)          \
    X(2, 4, 19, -1, -1, -1, 4, 512, 0) X(3, 4, 19, -1, -1, -1, 1, 512, 0)                      \
    X(4, 4, 24, -1, -1, -1, 4, 512, 0) X(5, 4, 24, -1, -1, -1, 1, 512, 0)                      \
    X(6, 4, 19, 246, 2048, 2048, 4, 1024, 4 * BWG_LAT_STAGE_SITES)                             \
    X(7, 4, 19, 246, 2048, 2048, 1, 512, LAT_WORD_SITES)                                   \
    X(8, 4, 19, -1, -1, -1, 1, 512, LAT_WORD_SITES_RT19)                                   \
    X(9, 4, 24, -1, -1, -1, 1, 512, LAT_WORD_SITES_RT24)

// grid: the slices of the band's groups, rounded up to a multiple of the 8 XCDs
#define BWG_LAT_LAUNCH(ID, P_, BC_, CU_, CA_, CI_, WS_, BL_, ST_)                             \
    static hipError_t lat_launch_##ID(const LatArgs &a, uint64_t words, hipStream_t s)       \
    {                                                                                         \
        const uint64_t nwg = (uint64_t)a.ng * (LAT_GROUP_WORDS / WS_);                        \
        if constexpr (WS_ == 1 && ST_ > 0) {                                                  \
            const uint64_t left = words - (uint64_t)a.g0 * LAT_GROUP_WORDS;                   \
            hipLaunchKernelGGL((lat_word_kernel<P_, BC_, CU_, CA_, CI_, BL_, ST_>),           \
                               dim3((unsigned)(left < nwg ? left : nwg)), dim3(BL_), 0, s, a); \
        } else {                                                                              \
            hipLaunchKernelGGL((lat_event_kernel<P_, BC_, CU_, CA_, CI_, WS_, BL_, ST_>),     \
                               dim3((unsigned)(8 * ((nwg + 7) / 8))), dim3(BL_), 0, s, a);    \
        }                                                                                     \
        return hipGetLastError();                                                             \
    }
BWG_LAT_VARIANTS(BWG_LAT_LAUNCH)

#ifndef __HIP_DEVICE_COMPILE__
#define BWG_LAT_ROW(ID, P_, BC_, CU_, CA_, CI_, WS_, BL_, ST_) {P_, BC_, CU_, CA_, CI_, WS_, BL_, ST_, lat_launch_##ID},
const LatVariant kLatVariants[] = {BWG_LAT_VARIANTS(BWG_LAT_ROW)};
const int kLatVariantCount = sizeof(kLatVariants) / sizeof(kLatVariants[0]);
#endif

hipError_t launch_lat_totals(const uint32_t *planes, uint64_t M, int S, int P, int32_t *dst,
                             hipStream_t s)
{
    if (P != 4) return hipErrorInvalidValue;
    const uint64_t n = ((M + 31) / 32 + LAT_TOT_WORDS - 1) / LAT_TOT_WORDS;
    return launch_pieces(n * LAT_TOT_BLOCK, LAT_TOT_BLOCK, [&](uint64_t i0, dim3 g) {
        hipLaunchKernelGGL(lat_totals_kernel<4>, g, dim3(LAT_TOT_BLOCK), 0, s, planes, M, S, dst,
                           i0 / LAT_TOT_BLOCK * LAT_TOT_WORDS);
    });
}

hipError_t launch_lat_sites(const uint32_t *planes, int S, int P, uint64_t first, uint64_t count,
                            int32_t *dst, hipStream_t s)
{
    dim3 grid((unsigned)((count + 255) / 256), (unsigned)S);
    hipLaunchKernelGGL(lat_sites_kernel, grid, dim3(256), 0, s, planes, S, P, first, count, dst);
    return hipGetLastError();
}

hipError_t launch_lat_histogram(const int32_t *tot, uint64_t M, int n_bins, uint64_t *dst,
                                hipStream_t s)
{
    hipError_t err = launch_fill_u64(dst, (uint64_t)n_bins, 0, s);
    if (err != hipSuccess) return err;
    const unsigned blocks = (unsigned)std::min<uint64_t>(1024, (M + 255) / 256);
    hipLaunchKernelGGL(lat_histogram_kernel, dim3(blocks), dim3(256), n_bins * 4, s, tot, M,
                       n_bins, dst);
    return hipGetLastError();
}

}  // namespace bwg
