// Simulation preparation on the GPU:
//  1. build the 64-bit sort key of every connection, (source prefix, target,
//     delay), with the digit histograms of every radix pass in the same
//     read; the source prefix is the local id of a local source, and
//     M_local + (alpha+1) G + global id of a remote one (global id = host
//     base + local id), an order that agrees with (alpha+1, sigma, source);
//     where every call gives each target a run of connections the keys are
//     written in target order, and the source bits alone remain to be sorted;
//  2. source-major radix sort to the unpacked arrays;
//  3. with remote sources, one scan over the sorted prefixes numbers the
//     images: the first connection of every distinct remote prefix starts the
//     next image after the local neurons (the sorted-unique map R of every
//     (alpha+1, sigma) and the remap of the paper's flag/compact/sort/search/
//     append steps in one pass);
//  4. R, its per-(alpha+1, sigma) offsets and a bit set of the images;
//  5. first-index array from the sorted sources;
//  6. point-to-point send lists: regenerate alpha = -1 draws per target host,
//     bit rows of the local sources they use, their compaction (S) and the
//     per-source transpose (T/P);
//  7. collective arrays H, I, G/Q from the source ranges of each group.
#include <algorithm>
#include <numeric>

#include "device_common.h"
#include "internal.h"

namespace snnc {

namespace {

constexpr int PNT = 256;

struct CallD {
    uint64_t gen_begin;
    SetRef S;
    uint32_t a;      // alpha + 1
    uint32_t order;  // position of the call in call order
    uint32_t flag;   // 1: only the sources its local connections use get images
    uint32_t uniform;   // 1: all source segments have the same length (segment = ordinal / length)
    FastDiv seg_div;
};

// segment lookup by division when every source segment of the call has the same length
CallD make_calld(const Call& cl, uint32_t order, uint32_t flag) {
    CallD d{cl.gen_begin, set_ref(cl.S, cl.dS), (uint32_t)(cl.alpha + 1), order, flag, 0, FastDiv{}};
    const auto& seg = cl.S.seg;
    bool uniform = seg.size() > 1 && seg[0].n > 0 && cl.S.total < (1ull << 31);
    for (const auto& g : seg) uniform = uniform && g.n == seg[0].n;
    if (uniform) {
        d.uniform = 1;
        d.seg_div = make_fastdiv(seg[0].n);
    }
    return d;
}

struct Lookup {
    const CallD* calls;
    uint32_t ncalls;
    const uint64_t* host_base;   // [P + 1]
    uint32_t P, PL;
    uint64_t G;                  // neurons over all hosts
};

__device__ __forceinline__ uint32_t find_call(const CallD* calls, uint32_t n, uint64_t i) {
    uint32_t a = 0, b = n;
    while (b - a > 1) {
        const uint32_t m = (a + b) >> 1;
        if (calls[m].gen_begin <= i) a = m; else b = m;
    }
    return a;
}

// Source of connection i (host, local id and bit index (alpha+1) G + global
// id), with a per-thread cache of the current call and source segment:
// a thread walks increasing positions, so the binary searches run only when
// the position leaves the cached call or the ordinal leaves the cached segment.
struct SourceCursor {
    uint64_t call_lo = 1, call_hi = 0;   // cached call covers [call_lo, call_hi)
    CallD call{};
    uint64_t seg_lo = 1, seg_hi = 0;     // cached segment covers ordinals [seg_lo, seg_hi)
    uint32_t seg_host = 0, seg_first = 0;
    uint64_t bit_base = 0;               // a G + host_base[seg_host] + seg_first - seg_lo

    __device__ __forceinline__ const CallD& call_at(const Lookup& L, uint64_t i) {
        if (i < call_lo || i >= call_hi) {
            const uint32_t k = find_call(L.calls, L.ncalls, i);
            call = L.calls[k];
            call_lo = call.gen_begin;
            call_hi = k + 1 < L.ncalls ? L.calls[k + 1].gen_begin : ~0ull;
            seg_lo = 1;
            seg_hi = 0;
        }
        return call;
    }

    __device__ __forceinline__ void at(const Lookup& L, uint64_t i, uint32_t ord, uint32_t& host, uint32_t& local,
                                       uint64_t& bit) {
        call_at(L, i);
        if (ord < seg_lo || ord >= seg_hi) {
            const bool inl = call.S.n <= SEG_INLINE;
            uint32_t a = 0, b = call.S.n;
            if (inl) {
                a = b > 1 && call.S.in[1].ord_begin <= ord ? 1 : 0;
            } else if (call.uniform) {
                a = fastdiv(ord, call.seg_div);
            } else {
                while (b - a > 1) {
                    const uint32_t m = (a + b) >> 1;
                    if (call.S.d[m].ord_begin <= ord) a = m; else b = m;
                }
            }
            const SegD s = !inl ? call.S.d[a] : a ? call.S.in[1] : call.S.in[0];
            seg_lo = s.ord_begin;
            seg_hi = a + 1 >= call.S.n ? ~0ull : inl ? call.S.in[1].ord_begin : call.S.d[a + 1].ord_begin;
            seg_host = s.host;
            seg_first = s.first;
            bit_base = (uint64_t)call.a * L.G + L.host_base[s.host] + s.first - s.ord_begin;
        }
        host = seg_host;
        local = seg_first + (uint32_t)(ord - seg_lo);
        bit = bit_base + ord;
    }
};

// contiguous range of positions for workgroup b of g over n (multiple of the block size)
__device__ __forceinline__ void block_range(uint64_t n, uint64_t& lo, uint64_t& hi) {
    const uint64_t per = ((n + gridDim.x - 1) / gridDim.x + PNT - 1) / PNT * PNT;
    lo = (uint64_t)blockIdx.x * per;
    hi = lo + per < n ? lo + per : n;
}

// Source ordinal of a call -> sort prefix (local id, or M_local + (alpha+1) G +
// global id of a remote source): prefix = ordinal + addend of its segment.
struct SrcMap {
    int64_t add;             // the only segment's addend (nS == 1)
    const int64_t* seg_add;  // per segment
    const uint64_t* seg_ord; // first ordinal per segment
    uint64_t div_m;          // equal segment lengths: segment = ordinal * div_m >> div_shift; else 0
    uint32_t div_shift;
    uint32_t nS;
};

// Target-major order.  When every call gives each of its targets a run of K
// consecutive connections (fixed in-degree, one-to-one), the connections in
// order of (target, call, element) are known in closed form: the targets fall
// into intervals covered by the same calls, and inside an interval every
// target has the same D connections.  With the keys written in that order, a
// stable sort by the source alone gives the order by (source, target,
// generation): the target's bits take no passes.
struct TInterval {
    uint64_t q0, q1;         // target-major positions [q0, q1)
    uint32_t first, D;       // first target, connections per target
    FastDiv div;             // by D (q1 - q0 < 2^31)
    uint32_t e0, ne;         // its entries
};

struct TEntry {              // a call's share of an interval: offsets [o, end) of each target's D
    uint32_t o, end, K, call;
    int64_t base;            // generation index = base + (target - first) K + offset
    int64_t add, add2;       // one or two source segments: the addends of ordinals below `split` and from it on
    uint32_t split;          // 0: more segments; `add` is their div_m if they are of equal length, else 0
    uint32_t seg;            // place of the call's segments among all calls' << 6 | div_shift
};

struct GenSource {
    const uint32_t* src;
    const uint32_t* tgt;
    const uint16_t* delay;
    const uint32_t* weight;
    const SrcMap* maps;            // per call with connections
    const uint64_t* call_begin;    // [ncalls + 1], the last one N
    const int64_t* seg_add;        // of all calls
    uint32_t n_seg;
    uint32_t ncalls;
    uint32_t n_iv;
    const TInterval* iv;
    const TEntry* ent;
    const uint32_t* bits;          // images numbered before the sort: their bit set, ranks and indices
    const uint64_t* word_rank;
    const int32_t* Lmap;
    uint32_t M_local, tgt_shift;
};

// the last of n ascending values at or below x (v[0] <= x)
__device__ __forceinline__ uint32_t last_at_or_below(const uint64_t* v, uint32_t n, uint64_t x) {
    uint32_t a = 0, b = n;
    while (b - a > 1) {
        const uint32_t m = (a + b) >> 1;
        if (v[m] <= x) a = m; else b = m;
    }
    return a;
}

__device__ __forceinline__ uint64_t rank_of(const uint32_t* bits, const uint64_t* word_rank, uint64_t bit) {
    const uint64_t w = bit >> 5;
    return word_rank[w] + (uint64_t)__popc(bits[w] & ((1u << (bit & 31)) - 1u));
}

__device__ __forceinline__ int64_t segment_add(const SrcMap& m, uint32_t ord) {
    if (m.nS == 1) return m.add;
    uint32_t j;
    if (m.div_m) {
        j = (uint32_t)(((uint64_t)ord * m.div_m) >> m.div_shift);
    } else {
        uint32_t a = 0, b = m.nS;
        while (b - a > 1) {
            const uint32_t x = (a + b) >> 1;
            if (m.seg_ord[x] <= ord) a = x; else b = x;
        }
        j = a;
    }
    return m.seg_add[j];
}

// sort key (source' << tgt_shift | target << 16 | delay).  Remote sources: the
// image index L when the images were numbered before the sort, else the global
// prefix (images are numbered after the sort).
__device__ __forceinline__ uint64_t conn_key(const GenSource& g, int64_t add, uint32_t ord, uint32_t tgt, uint32_t delay) {
    uint64_t p = (uint64_t)(add + (int64_t)ord);
    if (g.bits && p >= g.M_local) p = (uint64_t)g.Lmap[rank_of(g.bits, g.word_rank, p - g.M_local)];
    return (p << g.tgt_shift) | ((uint64_t)tgt << 16) | delay;
}

// the digits of one key per lane (valid lanes) into the workgroup's histograms; bits above the key's top are zero
__device__ __forceinline__ void key_digits(uint32_t* h, uint64_t key, bool valid, uint32_t bit_lo, const Digits& dg) {
    for (uint32_t p = 0; p < dg.passes; ++p)
        wave_hist_add(&h[p * dg.stride], (uint32_t)(key >> dg.shift(bit_lo, p)) & ((1u << dg.width(p)) - 1), valid);
}

// Sort keys in generation order, with the digit histograms of all radix
// passes: 10 B read and 8 B written per connection.
constexpr int KNT = 512;   // few, large workgroups: see hist_grid

__global__ __launch_bounds__(KNT) void k_keys(GenSource g, uint64_t n, uint32_t bit_lo, Digits dg,
                                              uint64_t* keys, uint64_t* hist) {
    extern __shared__ uint32_t h[];   // a histogram a pass
    for (uint32_t i = threadIdx.x; i < dg.passes * dg.stride; i += KNT) h[i] = 0;
    __syncthreads();
    uint64_t lo, hi;
    block_range(n, lo, hi);
    constexpr int KU = 4;   // independent elements per thread per step: their table loads overlap
    uint64_t call_end = 0;  // end of the call that holds the step's first element
    SrcMap m{};
    for (uint64_t base = lo; base < hi; base += (uint64_t)KNT * KU) {
        uint32_t ord[KU], tg[KU], dl[KU];
#pragma unroll
        for (int u = 0; u < KU; ++u) {
            const uint64_t i = base + (uint64_t)u * KNT + threadIdx.x;
            ord[u] = tg[u] = dl[u] = 0;
            if (i < hi) {
                ord[u] = g.src[i];
                tg[u] = g.tgt[i];
                dl[u] = g.delay[i];
            }
        }
        if (base >= call_end) {   // the same in every thread
            const uint32_t c = last_at_or_below(g.call_begin, g.ncalls, base);
            call_end = g.call_begin[c + 1];
            m = g.maps[c];
        }
        uint64_t key[KU];
#pragma unroll
        for (int u = 0; u < KU; ++u) {
            const uint64_t i = base + (uint64_t)u * KNT + threadIdx.x;
            key[u] = 0;
            if (i >= hi) continue;
            const int64_t add = i < call_end ? segment_add(m, ord[u])
                                             : segment_add(g.maps[last_at_or_below(g.call_begin, g.ncalls, i)], ord[u]);
            key[u] = conn_key(g, add, ord[u], tg[u], dl[u]);
            keys[i] = key[u];
        }
#pragma unroll
        for (int u = 0; u < KU; ++u)
            key_digits(h, key[u], base + (uint64_t)u * KNT + threadIdx.x < hi, bit_lo, dg);
    }
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < dg.passes * dg.stride; i += KNT)
        if (h[i]) atomicAdd((unsigned long long*)&hist[i], (unsigned long long)h[i]);
}

// The same in target-major order, with the weights moved along: 10 B read
// (source, delay, weight) and 12 B written per connection.  A wave takes
// `unit` consecutive positions; it walks the runs of a call in them one after
// another (all their parameters the same in every lane, so scalar) and each
// run by 64 lanes x 4, loading one step ahead.  Everything a step needs of its
// call comes with the run's table entry: looked up per key through the call's
// own table, the scalar loads stood in every key's way.  2.25e9 connections from
// 1,024 hosts 14.9 -> 9.6 ms (5.2 TB/s), 6.3e8 from 32 areas 4.1 -> 3.7.
// The alternative of letting the first radix pass gather its own connections
// was slower: the pass ranks 16 keys a lane at 16 waves a compute unit, and
// waits for the gather (6.3e8 connections: first pass 10.3 ms instead of 4.1).
constexpr uint32_t TM_UNIT = 2048;   // at most; fewer (whole steps of a wave) where 2048 would leave compute units idle:
                                     // 1e5 connections 53.6 us with units of 2048, 10.6 with units of 128

// Segment addends are read from LDS where they and the histograms fit a sixth of
// a compute unit's 160 KB: the kernel's 78 registers allow six workgroups.  A gather
// from memory takes a cycle a lane in the address unit (2.25e9 connections, 2 x 1,024
// segments: 11.3 ms through memory, 10.0 through LDS).
constexpr uint32_t TM_LDS = 26 << 10;

__host__ __device__ __forceinline__ bool adds_in_lds(const Digits& dg, uint32_t n_seg) {
    return (uint64_t)dg.passes * dg.stride * 4 + (uint64_t)n_seg * 8 <= TM_LDS;
}

uint32_t tm_unit(uint64_t n) {
    return (uint32_t)std::min<uint64_t>(std::max<uint64_t>(n / 8192 / 64 * 64, 128), TM_UNIT);
}

__global__ __launch_bounds__(PNT) void k_keys_tmajor(GenSource g, uint64_t n, uint32_t bit_lo, Digits dg,
                                                     uint32_t unit_size, uint64_t* keys, uint32_t* vals,
                                                     uint64_t* hist) {
    extern __shared__ __align__(8) uint32_t h[];   // a histogram a pass, then the segments' addends if they are few
    for (uint32_t i = threadIdx.x; i < dg.passes * dg.stride; i += PNT) h[i] = 0;
    int64_t* adds = nullptr;
    if (adds_in_lds(dg, g.n_seg)) {
        adds = reinterpret_cast<int64_t*>(h + dg.passes * dg.stride);
        for (uint32_t i = threadIdx.x; i < g.n_seg; i += PNT) adds[i] = g.seg_add[i];
    }
    __syncthreads();
    const uint32_t lane = threadIdx.x & 63;
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    constexpr int KU = 4;
    for (uint64_t unit = (uint64_t)blockIdx.x * (PNT / 64) + wave; unit * unit_size < n;
         unit += (uint64_t)gridDim.x * (PNT / 64)) {
        uint64_t q = unit * unit_size;
        const uint64_t end = q + unit_size < n ? q + unit_size : n;
        uint32_t a = 0, b = g.n_iv;
        while (b - a > 1) {
            const uint32_t m = (a + b) >> 1;
            if (g.iv[m].q0 <= q) a = m; else b = m;
        }
        TInterval v = g.iv[a];
        uint32_t t = fastdiv((uint32_t)(q - v.q0), v.div);
        uint32_t r = (uint32_t)(q - v.q0) - t * v.D;
        uint32_t e = v.e0, f = v.e0 + v.ne;
        while (f - e > 1) {
            const uint32_t m = (e + f) >> 1;
            if (g.ent[m].o <= r) e = m; else f = m;
        }
        // Steps of at most 64 KU connections of one call's run of one target; a step's connections are
        // loaded, and the step after it worked out, while the one before it is written.
        struct Step {
            uint64_t i, q;           // generation index and position of its first connection
            uint32_t cnt, tgt, split, seg, call;
            int64_t add, add2;
        };
        TEntry en{};
        uint64_t i0 = 0;
        uint32_t len = 0, x0 = 0;    // the run (or what of it lies in the unit) and how far it is stepped through
        auto next = [&]() {
            Step st{};
            if (q >= end) return st;
            if (!x0) {
                en = g.ent[e];
                len = (uint32_t)min((uint64_t)(en.end - r), end - q);
                i0 = (uint64_t)(en.base + (int64_t)((uint64_t)t * en.K) + r);
            }
            st = Step{i0 + x0, q + x0, len - x0 < 64u * KU ? len - x0 : 64u * KU, v.first + t, en.split, en.seg, en.call,
                      en.add, en.add2};
            x0 += 64 * KU;
            if (x0 >= len) {
                x0 = 0;
                q += len;
                r += len;
                ++e;
                if (r == v.D) {   // next target, or the next interval's first
                    r = 0;
                    ++t;
                    if (q == v.q1 && q < end) {
                        v = g.iv[++a];
                        t = 0;
                    }
                    e = v.e0;
                }
            }
            return st;
        };
        auto load = [&](const Step& st, uint32_t (&ord)[KU], uint32_t (&dl)[KU], uint32_t (&w)[KU]) {
#pragma unroll
            for (int u = 0; u < KU; ++u) {
                const uint32_t x = u * 64 + lane;
                ord[u] = dl[u] = w[u] = 0;
                if (x < st.cnt) {
                    ord[u] = g.src[st.i + x];
                    dl[u] = g.delay[st.i + x];
                    w[u] = g.weight[st.i + x];
                }
            }
        };
        Step cur = next();
        uint32_t ord[KU], dl[KU], w[KU];
        load(cur, ord, dl, w);
        while (cur.cnt) {
            const Step nxt = next();
            uint32_t ord1[KU], dl1[KU], w1[KU];
            load(nxt, ord1, dl1, w1);
#pragma unroll
            for (int u = 0; u < KU; ++u) {
                if (u * 64u >= cur.cnt) break;   // the same in every lane
                const uint32_t x = u * 64 + lane;
                uint64_t key = 0;
                if (x < cur.cnt) {
                    int64_t add;
                    if (cur.split) {
                        add = ord[u] < cur.split ? cur.add : cur.add2;
                    } else if (cur.add) {
                        const uint32_t j =
                            (cur.seg >> 6) + (uint32_t)(((uint64_t)ord[u] * (uint64_t)cur.add) >> (cur.seg & 63));
                        add = adds ? adds[j] : g.seg_add[j];
                    } else {
                        add = segment_add(g.maps[cur.call], ord[u]);
                    }
                    key = conn_key(g, add, ord[u], cur.tgt, dl[u]);
                    keys[cur.q + x] = key;
                    vals[cur.q + x] = w[u];
                }
                key_digits(h, key, x < cur.cnt, bit_lo, dg);
            }
            cur = nxt;
#pragma unroll
            for (int u = 0; u < KU; ++u) {
                ord[u] = ord1[u];
                dl[u] = dl1[u];
                w[u] = w1[u];
            }
        }
    }
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < dg.passes * dg.stride; i += PNT)
        if (h[i]) atomicAdd((unsigned long long*)&hist[i], (unsigned long long)h[i]);
}

// ---- image numbering after the sort (networks with remote sources)
// The connections were sorted with source prefix p = local id (local source)
// or M_local + (alpha+1) G + global id (remote source); both orders agree with
// (alpha+1, sigma, s).  One pass over the sorted prefixes numbers the images:
// the first connection of every distinct remote prefix starts a new image, and
// a scan of these flags (decoupled look-back across tiles) gives each
// connection its source'.  The same pass records each image's prefix and writes
// the first-index array.  4 B read and written per connection (the last radix
// pass has written the other arrays).
// Tile shapes: threads, items per thread.  The settings 0 and 9, 1 and 3, 2 and 4
// stand for the same shape (they once differed in when a payload was loaded).
struct NumberShape {
    int nt, ipt;
};
constexpr NumberShape NUMBER_SHAPES[] = {{1024, 12}, {512, 12}, {256, 12}, {512, 12}, {256, 12}, {256, 16},
                                         {256, 8}, {256, 6}, {512, 8}, {1024, 12}, {1024, 10}, {1024, 8}};
constexpr int NUMBER_VARIANTS = (int)(sizeof(NUMBER_SHAPES) / sizeof(NUMBER_SHAPES[0]));
constexpr uint64_t XFLAG_AGG = 1ull << 62, XFLAG_INC = 2ull << 62, XVALUE = (1ull << 40) - 1;
constexpr uint32_t XEPOCH_MASK = (1u << 22) - 1;

template <class P>
__device__ __forceinline__ P last_lane(P v) {   // lane 63's value
    if constexpr (sizeof(P) == 8)
        return ((P)(uint32_t)__builtin_amdgcn_readlane((int)(v >> 32), 63) << 32) |
               (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, 63);
    else
        return (P)__builtin_amdgcn_readlane((int)v, 63);
}

template <int XNT, int XIPT, class P>
__global__ __launch_bounds__(XNT) void k_number(const P* __restrict__ prefix, uint64_t n, uint32_t M_local,
                                                uint64_t* lookback, uint32_t epoch, uint32_t taken_epoch,
                                                uint32_t spin_limit, int32_t* o_src, uint64_t* img_key,
                                                uint64_t* row_ptr, uint64_t* n_img_out) {
    __shared__ uint64_t wave_tot[XNT / 64];
    __shared__ uint64_t s_excl;
    const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const uint64_t tile = blockIdx.x;
    constexpr uint64_t XTILE = (uint64_t)XNT * XIPT;
    const uint64_t wbase = tile * XTILE + (uint64_t)wave * 64 * XIPT;
    // element of item k on this lane: wbase + k*64 + lane (wave-striped, so loads and stores coalesce)
    P key[XIPT];
    uint32_t incl[XIPT];          // flags up to and including the item, within the wave
    uint32_t fl = 0;              // bit k: item k starts a new image
    const P before_wave = wbase > 0 && wbase - 1 < n ? prefix[wbase - 1] : ~(P)0;
    uint32_t carry = 0;
#pragma unroll
    for (int k = 0; k < XIPT; ++k) {
        const uint64_t i = wbase + (uint64_t)k * 64 + lane;
        key[k] = i < n ? prefix[i] : ~(P)0;
    }
    const uint64_t upto = ~0ull >> (63 - lane);   // lanes up to and including this one
    uint32_t bl = 0;              // bit k: item k starts a row
#pragma unroll
    for (int k = 0; k < XIPT; ++k) {
        const uint64_t i = wbase + (uint64_t)k * 64 + lane;
        P prev = __shfl_up(key[k], 1, 64);
        if (lane == 0) prev = k ? last_lane(key[k ? k - 1 : 0]) : before_wave;
        const bool b = i < n && (i == 0 || key[k] != prev);
        const bool f = b && key[k] >= M_local;
        bl |= (b ? 1u : 0u) << k;
        fl |= (f ? 1u : 0u) << k;
        const uint64_t m = __ballot(f);
        incl[k] = carry + (uint32_t)__popcll(m & upto);
        carry += (uint32_t)__popcll(m);
    }
    if (lane == 63) wave_tot[wave] = carry;
    __syncthreads();
    uint64_t wave_excl = 0, tile_tot = 0;
#pragma unroll
    for (int w = 0; w < XNT / 64; ++w) {
        if (w < (int)wave) wave_excl += wave_tot[w];
        tile_tot += wave_tot[w];
    }
    if (wave == 0) {
        uint64_t* my = lookback + tile;
        const uint64_t ep = (uint64_t)epoch << 40;
        uint64_t excl = 0;
        if (lane == 0)
            __hip_atomic_store(my, (tile == 0 ? XFLAG_INC : XFLAG_AGG) | ep | tile_tot, __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
        // the wave reads 64 earlier tiles at a time, nearest first, up to one with its inclusive count
        int64_t pred = (int64_t)tile - 1;
        uint32_t spins = 0;
        while (pred >= 0) {
            const int64_t t = pred - lane;
            const uint64_t st = t >= 0 ? __hip_atomic_load(lookback + t, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)
                                       : XFLAG_INC | (uint64_t)taken_epoch << 40;
            const bool ready = (st >> 62) != 0 && ((st >> 40) & XEPOCH_MASK) == taken_epoch;
            const uint64_t m_ready = __ballot(ready), m_inc = __ballot(ready && (st >> 62) == 2);
            const uint32_t stop = m_inc ? (uint32_t)__ffsll((unsigned long long)m_inc) : 64u;   // lanes to take
            const uint64_t need = ~0ull >> (64 - stop);
            const uint64_t missing = need & ~m_ready;
            if (missing && spins++ < spin_limit) {
                __builtin_amdgcn_s_sleep(1);
                continue;
            }
            // a tile that stays without counts (its workgroup may not have started): the wave counts it
            const uint32_t take = missing ? (uint32_t)__ffsll((unsigned long long)missing) - 1 : stop;
            uint64_t v = lane < take ? st & XVALUE : 0;
            for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
            excl += v;
            pred -= take;
            if (!missing) {
                if (m_inc) break;
                continue;
            }
            for (uint64_t i0 = (uint64_t)pred * XTILE; i0 < ((uint64_t)pred + 1) * XTILE; i0 += 64) {
                const uint64_t i = i0 + lane;   // every tile before the last is full
                excl += (uint64_t)__popcll(__ballot(prefix[i] >= M_local && (i == 0 || prefix[i] != prefix[i - 1])));
            }
            --pred;
        }
        if (lane == 0) {
            if (tile)
                __hip_atomic_store(my, XFLAG_INC | ep | (excl + tile_tot), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            s_excl = excl;
        }
    }
    __syncthreads();
    const uint64_t before = s_excl + wave_excl;   // images started before this wave
    // past the local rows every row is an image's, starts at its flag and has connections: one
    // store per image; among the local rows runs of empty ones are filled as well
    const bool images_only = wbase > 0 && before_wave >= M_local;   // the same in every lane
#pragma unroll
    for (int k = 0; k < XIPT; ++k) {
        const uint64_t i = wbase + (uint64_t)k * 64 + lane;
        const uint64_t rank = before + incl[k];                 // images started up to and including i
        const bool flag_here = (fl >> k) & 1u;
        const int64_t src2 = key[k] < M_local ? (int64_t)key[k] : (int64_t)(M_local + rank - 1);
        if (i < n) o_src[i] = (int32_t)src2;
        if (flag_here) img_key[rank - 1] = (uint64_t)key[k] - M_local;
        if (images_only) {
            if (flag_here) row_ptr[src2] = i;
        } else if (__ballot((bl >> k) & 1u)) {
            P pp = __shfl_up(key[k], 1, 64);     // prefix of the previous connection
            if (lane == 0) pp = k ? last_lane(key[k ? k - 1 : 0]) : before_wave;
            int64_t lo = 0, hi = -1;
            if ((bl >> k) & 1u) {   // the previous row: a local one, or the image before this one
                lo = i == 0 ? 0 : pp < M_local ? (int64_t)pp + 1 : src2;
                hi = src2;
            }
            fill_rows(row_ptr, lo, hi, i);
        }
        if (i + 1 == n) *n_img_out = rank;
        const bool ends = i + 1 == n;
        if (__ballot(ends))   // rows after the last connection
            fill_rows(row_ptr, ends ? src2 + 1 : 0, ends ? (int64_t)M_local + (int64_t)rank : -1, n);
    }
}

// R value and (alpha+1, sigma) boundaries from the image prefixes a G + gid.
// Each thread takes RV_RUN consecutive images (sorted): the map slot a and the
// host are found for the first and kept while the next ones stay inside them.
constexpr int RV_RUN = 8;

__global__ void k_rvals_sorted(const uint64_t* img_key, uint64_t n_img, const uint64_t* host_base, uint32_t P,
                               uint64_t G, int32_t* R) {
    const uint64_t j0 = ((uint64_t)blockIdx.x * blockDim.x + threadIdx.x) * RV_RUN;
    if (j0 >= n_img) return;
    const uint64_t j1 = j0 + RV_RUN < n_img ? j0 + RV_RUN : n_img;
    uint64_t base = 0;             // a G of the current slot
    uint64_t hlo = 1, hhi = 0;     // [host_base[h], host_base[h + 1]) of the current host (empty: none yet)
    for (uint64_t j = j0; j < j1; ++j) {
        const uint64_t key = img_key[j];
        if (key < base || key - base >= G) base = key / G * G;
        const uint64_t gid = key - base;
        if (gid < hlo || gid >= hhi) {
            uint32_t lo = 0, hi = P;
            while (hi - lo > 1) {
                const uint32_t m = (lo + hi) >> 1;
                if (host_base[m] <= gid) lo = m; else hi = m;
            }
            hlo = host_base[lo];
            hhi = host_base[lo + 1];
        }
        R[j] = (int32_t)(gid - hlo);
    }
}

__global__ void k_bounds_sorted(const uint64_t* img_key, uint64_t n_img, const uint64_t* host_base, uint32_t P,
                                uint32_t n_a, uint64_t G, uint32_t M_local, uint64_t* r_off, int64_t* img_base) {
    const uint64_t k = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const uint64_t nk = (uint64_t)n_a * P;
    if (k > nk) return;
    const uint64_t x = k == nk ? (uint64_t)n_a * G : (k / P) * G + host_base[k % P];
    uint64_t a = 0, b = n_img;   // lower_bound of x
    while (a < b) {
        const uint64_t m = (a + b) >> 1;
        if (img_key[m] < x) a = m + 1; else b = m;
    }
    r_off[k] = a;
    if (k < nk) img_base[k] = (int64_t)M_local + (int64_t)a;
}

// Bit of every image prefix (bits is zero before).  The prefixes are sorted,
// so the lanes of one word are contiguous in a wave: a segmented OR across
// them leaves the word's bits in its last lane, which sets them with one
// atomic (a word can continue in the next wave).
__global__ void k_bits_sorted(const uint64_t* img_key, uint64_t n_img, uint32_t* bits) {
    const uint64_t j = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int lane = threadIdx.x & 63;
    const bool valid = j < n_img;
    const uint64_t key = valid ? img_key[j] : ~0ull;
    const uint64_t w = key >> 5;
    uint32_t acc = valid ? 1u << (key & 31) : 0u;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t a = __shfl_up(acc, o, 64);
        const uint64_t wo = __shfl_up(w, o, 64);
        if (lane >= o && wo == w) acc |= a;
    }
    const uint64_t wn = __shfl_down(w, 1, 64);
    if (valid && (lane == 63 || wn != w)) atomicOr(bits + w, acc);
}

// ---- images numbered before the sort (map policies other than the default)
// fc[(alpha+1) G + gid] = first call (in call order) that gives the source an
// image; ~0 = none.  Flagged calls: the sources their local connections use.
__global__ __launch_bounds__(PNT) void k_first_use(Lookup L, const uint32_t* g_src, uint64_t n, uint32_t* fc) {
    uint64_t lo, hi;
    block_range(n, lo, hi);
    SourceCursor cur;
    for (uint64_t i = lo + threadIdx.x; i < hi; i += PNT) {
        if (!cur.call_at(L, i).flag) continue;
        uint32_t host, local;
        uint64_t bit;
        cur.at(L, i, g_src[i], host, local, bit);
        if (host == L.PL) continue;
        const uint32_t ord = cur.call.order;
        if (fc[bit] > ord) atomicMin(&fc[bit], ord);   // fc only decreases: a stale read never skips wrongly
    }
}

// Unflagged calls: every source passed to them (bit ranges, concatenated)
struct FRange {
    uint64_t begin;   // first position in the concatenation
    uint64_t bit;     // bit of the range's first source
    uint32_t order;   // call order
    uint32_t pad;
};

__global__ __launch_bounds__(PNT) void k_first_pass(const FRange* rg, uint32_t n_rg, uint64_t total, uint32_t* fc) {
    for (uint64_t j = (uint64_t)blockIdx.x * PNT + threadIdx.x; j < total; j += (uint64_t)gridDim.x * PNT) {
        uint32_t a = 0, b = n_rg;
        while (b - a > 1) {
            const uint32_t m = (a + b) >> 1;
            if (rg[m].begin <= j) a = m; else b = m;
        }
        const uint64_t bit = rg[a].bit + (j - rg[a].begin);
        const uint32_t ord = rg[a].order;
        if (fc[bit] > ord) atomicMin(&fc[bit], ord);
    }
}

// bit set of the sources with an image: one ballot per wave covers 64 bits
__global__ __launch_bounds__(PNT) void k_fc_bits(const uint32_t* fc, uint64_t n_bits, uint64_t n_words, uint32_t* bits) {
    for (uint64_t base = (uint64_t)blockIdx.x * PNT; base < n_bits; base += (uint64_t)gridDim.x * PNT) {
        const uint64_t b = base + threadIdx.x;   // the loop bound is uniform per workgroup: whole waves ballot
        const uint64_t m = __ballot(b < n_bits && fc[b] != ~0u);
        if ((threadIdx.x & 63) == 0) {
            const uint64_t w = (b >> 6) * 2;
            if (w < n_words) bits[w] = (uint32_t)m;
            if (w + 1 < n_words) bits[w + 1] = (uint32_t)(m >> 32);
        }
    }
}

// images in canonical order: R value, and (first call << 16, canonical index)
// pairs for the numbering in call order
__global__ __launch_bounds__(PNT) void k_img_list(const uint32_t* bits, const uint64_t* word_rank, uint64_t n_words,
                                                  const uint32_t* fc, const uint64_t* host_base, uint32_t P, uint64_t G,
                                                  int32_t* R, uint64_t* okey, uint32_t* oval) {
    for (uint64_t w = (uint64_t)blockIdx.x * PNT + threadIdx.x; w < n_words; w += (uint64_t)gridDim.x * PNT) {
        uint32_t word = bits[w];
        uint64_t pos = word_rank[w];
        while (word) {
            const uint32_t bb = __ffs(word) - 1;
            word &= word - 1;
            const uint64_t bit = w * 32 + bb;
            const uint64_t gid = bit % G;
            uint32_t lo = 0, hi = P;
            while (hi - lo > 1) {
                const uint32_t m = (lo + hi) >> 1;
                if (host_base[m] <= gid) lo = m; else hi = m;
            }
            R[pos] = (int32_t)(gid - host_base[lo]);
            if (okey) {
                okey[pos] = (uint64_t)fc[bit] << 16;
                oval[pos] = (uint32_t)pos;
            }
            ++pos;
        }
    }
}

// L[j] = M_local + j (canonical numbering)
__global__ void k_iota_l(int32_t* Lv, uint64_t n, uint32_t M_local) {
    const uint64_t j = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (j < n) Lv[j] = (int32_t)((uint64_t)M_local + j);
}

// L[canonical index] = M_local + position in call order
__global__ void k_scatter_l(const uint32_t* canon, uint64_t n, uint32_t M_local, int32_t* Lv) {
    const uint64_t k = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k < n) Lv[canon[k]] = (int32_t)((uint64_t)M_local + k);
}

// R offsets per (alpha+1, sigma) from the bit set ranks
__global__ void k_bounds_bits(const uint32_t* bits, const uint64_t* word_rank, const uint64_t* host_base, uint32_t P,
                              uint32_t n_a, uint64_t G, uint32_t M_local, int canonical, uint64_t* r_off,
                              int64_t* img_base) {
    const uint64_t k = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const uint64_t nk = (uint64_t)n_a * P;
    if (k > nk) return;
    const uint64_t x = k == nk ? (uint64_t)n_a * G : (k / P) * G + host_base[k % P];
    const uint64_t r = rank_of(bits, word_rank, x);
    r_off[k] = r;
    if (k < nk) img_base[k] = canonical ? (int64_t)M_local + (int64_t)r : -1;
}

// point-to-point rows: set the bits of local-id ranges (unflagged calls)
struct WRange {
    uint64_t begin;   // first position in the concatenation of word counts
    uint64_t row;     // first word of the row
    uint32_t lo, hi;  // local ids [lo, hi)
};

__global__ __launch_bounds__(PNT) void k_set_ranges(const WRange* rg, uint32_t n_rg, uint64_t total, uint32_t* rows) {
    for (uint64_t j = (uint64_t)blockIdx.x * PNT + threadIdx.x; j < total; j += (uint64_t)gridDim.x * PNT) {
        uint32_t a = 0, b = n_rg;
        while (b - a > 1) {
            const uint32_t m = (a + b) >> 1;
            if (rg[m].begin <= j) a = m; else b = m;
        }
        const WRange r = rg[a];
        const uint32_t w = (r.lo >> 5) + (uint32_t)(j - r.begin);
        const uint32_t first = max(r.lo, w * 32), last = min(r.hi, w * 32 + 32);   // [first, last) in this word
        const uint32_t nb = last - first;
        const uint32_t mask = (nb == 32 ? ~0u : ((1u << nb) - 1u)) << (first & 31);
        atomicOr(&rows[r.row + w], mask);
    }
}

// first-index array: row_ptr[r] = first position with source >= r
// Each thread takes 4 consecutive positions with one 16-byte load; position
// i closes the rows (src[i-1], src[i]] (position n closes the rest; lanes past
// it close none).  Whole waves stay in the loop: long runs of rows without
// connections are filled by the wave together.
__global__ __launch_bounds__(PNT) void k_csr(const int32_t* src, uint64_t n, uint64_t n_rows, uint64_t* row_ptr) {
    const uint64_t quads = n / 4 + 1;   // the last quad holds the tail and position n
    for (uint64_t q0 = (uint64_t)blockIdx.x * PNT; q0 < quads; q0 += (uint64_t)gridDim.x * PNT) {
        const uint64_t i0 = (q0 + threadIdx.x) * 4;
        int64_t v[4], prev = (int64_t)n_rows;
        if (i0 + 4 <= n) {
            const int4 x = *reinterpret_cast<const int4*>(src + i0);
            v[0] = x.x; v[1] = x.y; v[2] = x.z; v[3] = x.w;
        } else {
            for (int k = 0; k < 4; ++k) v[k] = i0 + k < n ? (int64_t)src[i0 + k] : (int64_t)n_rows;
        }
        if (i0 <= n) prev = i0 == 0 ? -1 : (int64_t)src[i0 - 1];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            fill_rows(row_ptr, prev + 1, v[k], i0 + k);   // nothing past position n: prev == v[k] == n_rows
            prev = v[k];
        }
    }
}

// The same by a binary search per row: a search reads about log2(n) positions
// where the pass above reads all n, and no row waits for its neighbours.
__global__ void k_csr_search(const int32_t* src, uint64_t n, uint64_t n_rows, uint64_t* row_ptr) {
    const uint64_t r = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (r > n_rows) return;
    uint64_t lo = 0, hi = n;
    while (lo < hi) {
        const uint64_t mid = (lo + hi) >> 1;
        if ((int64_t)src[mid] < (int64_t)r) lo = mid + 1; else hi = mid;
    }
    row_ptr[r] = lo;
}

// Constant result arrays (no image, no send list, no group), all in one launch.
struct Fills {
    static constexpr int MAX = 8;
    uint64_t* p[MAX];
    uint64_t n[MAX], v[MAX];
    int count = 0;
    void add(uint64_t* ptr, uint64_t len, uint64_t value) {
        p[count] = ptr;
        n[count] = len;
        v[count] = value;
        ++count;
    }
};

__global__ __launch_bounds__(PNT) void k_fills(Fills f) {
    for (int k = 0; k < f.count; ++k)
        for (uint64_t i = (uint64_t)blockIdx.x * PNT + threadIdx.x; i < f.n[k]; i += (uint64_t)gridDim.x * PNT)
            f.p[k][i] = f.v[k];
}

// offsets of the send rows: rank of every row's first word
__global__ void k_row_offsets(const uint64_t* row_rank, uint32_t P, uint32_t words_per_row, uint64_t* s_off) {
    const uint32_t tau = blockIdx.x * blockDim.x + threadIdx.x;
    if (tau <= P) s_off[tau] = row_rank[(uint64_t)tau * words_per_row];
}

// ---- point-to-point lists
// S values: set bits of row tau as local ids, at their rank
__global__ __launch_bounds__(PNT) void k_s_vals(const uint32_t* rows, const uint64_t* word_rank, uint64_t n_words,
                                                uint32_t words_per_row, int32_t* S) {
    for (uint64_t w = (uint64_t)blockIdx.x * PNT + threadIdx.x; w < n_words; w += (uint64_t)gridDim.x * PNT) {
        uint32_t word = rows[w];
        uint64_t pos = word_rank[w];
        const uint32_t s0 = (uint32_t)(w % words_per_row) * 32;
        while (word) {
            const uint32_t b = __ffs(word) - 1;
            word &= word - 1;
            S[pos++] = (int32_t)(s0 + b);
        }
    }
}

// per local source: number of target hosts whose row has its bit
__global__ __launch_bounds__(PNT) void k_tp_count(const uint32_t* rows, uint32_t P, uint32_t words_per_row,
                                                  uint32_t M, uint32_t* cnt) {
    const uint32_t s = blockIdx.x * PNT + threadIdx.x;
    if (s >= M) return;
    uint32_t c = 0;
    for (uint32_t tau = 0; tau < P; ++tau) c += (rows[(uint64_t)tau * words_per_row + (s >> 5)] >> (s & 31)) & 1u;
    cnt[s] = c;
}

__global__ __launch_bounds__(PNT) void k_tp_fill(const uint32_t* rows, const uint64_t* word_rank, const uint64_t* s_off,
                                                 uint32_t P, uint32_t words_per_row, uint32_t M, const uint64_t* tp_ptr,
                                                 uint32_t* T, uint32_t* Pos) {
    const uint32_t s = blockIdx.x * PNT + threadIdx.x;
    if (s >= M) return;
    uint64_t o = tp_ptr[s];
    for (uint32_t tau = 0; tau < P; ++tau) {
        const uint64_t w = (uint64_t)tau * words_per_row + (s >> 5);
        const uint32_t word = rows[w];
        if ((word >> (s & 31)) & 1u) {
            T[o] = tau;
            Pos[o] = (uint32_t)(word_rank[w] + (uint64_t)__popc(word & ((1u << (s & 31)) - 1u)) - s_off[tau]);
            ++o;
        }
    }
}

// ---- collective arrays
struct HRange {
    uint64_t h_begin;   // first position in H
    uint32_t lo, len;   // source ids [lo, lo + len)
    uint32_t a, sigma;  // map index alpha + 1 and host
};

// H and I: a workgroup takes PNT * HI_RUN consecutive entries at a time and finds
// the range of its first one once (the ranges are long: a host's population);
// only entries past that range search for their own.  canonical: images are
// numbered in the order of their bits, so L is the rank and is not read.
// Bound by the two written arrays and the random reads of the bit set; 1,024
// hosts with 2.3e8 entries: 0.70 ms, one entry a thread with a search each 2.5 ms.
constexpr int HI_RUN = 8;

__global__ __launch_bounds__(PNT) void k_hi(const HRange* rg, uint32_t n_rg, uint64_t n_h, const uint32_t* bits,
                                            const uint64_t* word_rank, const int32_t* Lmap, int canonical,
                                            uint32_t M_local, const uint64_t* host_base, uint64_t G, uint32_t PL,
                                            int32_t* H, int32_t* I) {
    for (uint64_t j0 = (uint64_t)blockIdx.x * PNT * HI_RUN; j0 < n_h; j0 += (uint64_t)gridDim.x * PNT * HI_RUN) {
        auto range_of = [&](uint64_t j) {
            uint32_t a = 0, b = n_rg;
            while (b - a > 1) {
                const uint32_t m = (a + b) >> 1;
                if (rg[m].h_begin <= j) a = m; else b = m;
            }
            return a;
        };
        const HRange first = rg[range_of(j0)];
        const uint64_t first_end = first.h_begin + first.len;
        const uint64_t first_bit = (uint64_t)first.a * G + host_base[first.sigma];
#pragma unroll
        for (int k = 0; k < HI_RUN; ++k) {
            const uint64_t j = j0 + (uint64_t)k * PNT + threadIdx.x;
            if (j >= n_h) break;
            HRange r = first;
            uint64_t bit0 = first_bit;
            if (j >= first_end) {
                r = rg[range_of(j)];
                bit0 = (uint64_t)r.a * G + host_base[r.sigma];
            }
            const uint32_t s = r.lo + (uint32_t)(j - r.h_begin);
            H[j] = (int32_t)s;
            int32_t img = -1;
            if (r.sigma != PL) {
                const uint64_t bit = bit0 + s;
                const uint32_t word = bits[bit >> 5];
                if ((word >> (bit & 31)) & 1u) {
                    const uint64_t rank = word_rank[bit >> 5] + (uint64_t)__popc(word & ((1u << (bit & 31)) - 1u));
                    img = canonical ? (int32_t)(M_local + rank) : Lmap[rank];
                }
            }
            I[j] = img;
        }
    }
}

// G/Q of local source s: groups (ascending) whose H on P_local contains s
struct LRange {
    uint32_t lo, hi;    // [lo, hi)
    uint64_t pos;       // position of lo in H_{g, P_local}
};

__global__ __launch_bounds__(PNT) void k_gq(const LRange* lr, const uint32_t* g_first, uint32_t n_groups,
                                            const int32_t* groups, uint32_t M, const uint64_t* gq_ptr, uint32_t* cnt,
                                            int32_t* Gv, uint32_t* Qv) {
    const uint32_t s = blockIdx.x * PNT + threadIdx.x;
    if (s >= M) return;
    uint64_t o = gq_ptr ? gq_ptr[s] : 0;
    uint32_t c = 0;
    for (uint32_t g = 0; g < n_groups; ++g) {
        uint32_t a = g_first[g], b = g_first[g + 1];
        if (a == b) continue;
        while (b - a > 1) {   // last range with lo <= s
            const uint32_t m = (a + b) >> 1;
            if (lr[m].lo <= s) a = m; else b = m;
        }
        const LRange r = lr[a];
        if (s >= r.lo && s < r.hi) {
            if (gq_ptr) {
                Gv[o] = groups[g];
                Qv[o] = (uint32_t)(r.pos + (s - r.lo));
                ++o;
            }
            ++c;
        }
    }
    if (!gq_ptr) cnt[s] = c;
}

uint64_t count_on(const HostSet& s, uint32_t host) {
    uint64_t n = 0;
    for (auto& g : s.seg)
        if (g.host == host) n += g.n;
    return n;
}

// Map policy: does call cl give images on host tau only to the sources its
// connections there use (flagging)?  The threshold heuristic flags rules that
// draw their sources at random (and assigned pairs) when the estimated
// connections on tau per source fall below xi; out-degree and one-to-one calls
// use every source.
bool flag_sources(const Ctx& c, const Call& cl, uint32_t tau) {
    if (c.img_sources == 0) return true;
    if (c.img_sources == 2) return false;
    if (cl.S.total == 0) return true;
    const double n_s = (double)cl.S.total, n_t = (double)count_on(cl.T, tau);
    double est;
    switch (cl.rule) {
        case SNNC_FIXED_INDEGREE: est = (double)cl.n * n_t; break;
        case SNNC_FIXED_TOTAL_NUMBER: est = (double)cl.n * n_t / (double)cl.T.total; break;
        case SNNC_PAIRWISE_BERNOULLI: est = cl.p * n_s * n_t; break;
        case SNNC_ASSIGNED_NODES: {
            auto it = cl.pairs_on.find(tau);
            est = it == cl.pairs_on.end() ? 0.0 : (double)it->second;
            break;
        }
        default: return false;
    }
    return est / n_s < c.xi;
}

template <class T>
T* result(Ctx& c, int32_t id, uint64_t n) {
    auto& a = c.arrays[id];
    dfree(c, a.p);
    a.p = dalloc(c, (size_t)std::max<uint64_t>(n, 1) * sizeof(T));
    a.bytes = (size_t)n * sizeof(T);
    c.counts[id] = n;
    return static_cast<T*>(a.p);
}

unsigned grid_for(uint64_t n, uint64_t cap = 1u << 20) {
    return (unsigned)std::max<uint64_t>(1, std::min<uint64_t>((n + PNT - 1) / PNT, cap));
}

uint32_t bits_for(uint64_t n_values) {   // bits to hold 0 .. n_values - 1
    uint32_t b = 0;
    while (b < 64 && (n_values > 0 ? (n_values - 1) >> b : 0)) ++b;
    return b;
}

}  // namespace

namespace {

// first index and count of the image rows [M_local, M_local + n_img)
__global__ void k_img_rows(const uint64_t* row_ptr, uint32_t M_local, uint64_t n_img, uint64_t* first,
                           uint32_t* count) {
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n_img; i += (uint64_t)gridDim.x * blockDim.x) {
        const uint64_t a = row_ptr[(uint64_t)M_local + i], b = row_ptr[(uint64_t)M_local + i + 1];
        if (first) first[i] = a;
        if (count) count[i] = (uint32_t)(b - a);
    }
}

// Moves result arrays into pinned host memory that kernels can read: one
// block for all (pinning costs 30 us a call and more with its pages), all the
// copies, then one wait.
void to_host(Ctx& c, std::initializer_list<int32_t> ids) {
    auto up = [](size_t b) { return (b + 255) & ~(size_t)255; };
    size_t total = 0;
    for (int32_t id : ids) {
        auto it = c.arrays.find(id);
        if (it != c.arrays.end()) total += up(std::max<size_t>(it->second.bytes, 1));
    }
    if (!total) return;
    c.host_block = result_pinned_take(c.device, total, &c.host_block_bytes);
    char* h = static_cast<char*>(c.host_block);
    void* dev = nullptr;
    if (hipHostGetDevicePointer(&dev, h, 0) != hipSuccess) {
        (void)hipGetLastError();
        raise(SNNC_EDEVICE, "pinned host memory without a device address");
    }
    char* d = static_cast<char*>(dev);
    std::vector<void*> old;
    for (int32_t id : ids) {
        auto it = c.arrays.find(id);
        if (it == c.arrays.end()) continue;
        DevArray& a = it->second;
        old.push_back(a.p);
        const void* from = a.p;
        a.p = h;
        a.dev = d;
        a.host = true;
        h += up(std::max<size_t>(a.bytes, 1));
        d += up(std::max<size_t>(a.bytes, 1));
        if (a.bytes) HIPCHK(hipMemcpyAsync(a.p, from, a.bytes, hipMemcpyDeviceToHost, c.stream));
    }
    sync(c);
    for (void* p : old) dfree(c, p);
}

// GPU memory levels (Methods, GPU memory levels subsection).  Levels 0 and 1:
// the maps of the remote sources to their images (R, L, img_base and their
// offsets; H and I of the collective layout) and the first index and count
// of every image row live in pinned host memory, the device keeps the
// first-index array of the local rows only.  Level 2: everything in device
// memory, the count of a row from two first-index entries.  Level 3: level 2
// plus the counts of the image rows as an array.  (Images of every passed
// source from level 1 on: set with the level.)
void place_memory_level(Ctx& c, uint32_t M_local) {
    const int L = c.mem_level;
    if (L != 0 && L != 1 && L != 3) return;
    const uint64_t n_img = c.n_img;
    const uint64_t* rp = static_cast<const uint64_t*>(c.arrays[SNNC_ROW_PTR].p);
    uint64_t* first = (L <= 1) ? result<uint64_t>(c, SNNC_IMG_FIRST, n_img) : nullptr;
    uint32_t* count = result<uint32_t>(c, SNNC_IMG_COUNT, n_img);
    if (n_img) {
        tstart(c, "prep_img_rows");
        hipLaunchKernelGGL(k_img_rows, dim3(grid_for(n_img)), dim3(PNT), 0, c.stream, rp, M_local, n_img, first, count);
        tstop(c);
        HIPCHK(hipGetLastError());
    }
    if (L == 3) return;
    // the device keeps the local rows of the first-index array
    const uint64_t keep = (uint64_t)M_local + 1;
    DevArray old = c.arrays[SNNC_ROW_PTR];
    c.arrays[SNNC_ROW_PTR] = DevArray{};
    uint64_t* nrp = result<uint64_t>(c, SNNC_ROW_PTR, keep);
    HIPCHK(hipMemcpyAsync(nrp, old.p, keep * 8, hipMemcpyDeviceToDevice, c.stream));
    free_array(c, old);
    to_host(c, {SNNC_IMG_FIRST, SNNC_IMG_COUNT, SNNC_R_OFF, SNNC_R_VAL, SNNC_IMG_BASE, SNNC_L_VAL, SNNC_H_OFF,
                SNNC_H_VAL, SNNC_I_VAL});
}

// Intervals of targets covered by the same calls, and the calls' entries in
// them (see TInterval), from the calls' runs (in call order).  False when some
// call has no such runs, or they are short (fewer than 16 connections a run on
// average: a run takes at least one step of a wave), or the entries are many for
// the connections.  An entry takes the host 50 ns; the passes saved (two over 65,536
// targets) are worth 10 us up to 1e6 connections, 38 us at 5.2e6 and 205 us at 2.1e7.
// Prepare of 3.3e5 connections to targets in 1, 256, 1,024, 16,384 segments: 82, 99, 130,
// 880 us in target order, 96 otherwise; of 2.1e7: 453, 476, 505, 1,269 and 663.
bool target_major(const Ctx& c, const std::vector<uint32_t>& with_conns, const std::vector<SrcMap>& maps,
                  const std::vector<size_t>& seg_at, const std::vector<int64_t>& seg_add,
                  const std::vector<uint64_t>& seg_ord, std::vector<TInterval>& iv, std::vector<TEntry>& ent) {
    const size_t max_entries = (size_t)std::min<uint64_t>(128 + c.n_gen / 8192, 1u << 16);
    size_t n_seg = 0;   // each of them a run at least: no need to look further where they are too many
    for (uint32_t k : with_conns) {
        for (auto& g : c.calls[k].T.seg) n_seg += g.host == c.P_local ? 1 : 0;
        if (n_seg > max_entries) return false;
    }
    struct Run {
        TargetRun r;
        uint32_t call;
    };
    std::vector<Run> runs;
    std::vector<TargetRun> tmp;
    for (uint32_t k = 0; k < with_conns.size(); ++k) {
        tmp.clear();
        if (!target_runs(c, c.calls[with_conns[k]], tmp)) return false;
        for (auto& r : tmp)
            if (r.n && r.K) runs.push_back(Run{r, k});
        if (runs.size() > max_entries) return false;
    }
    std::vector<uint64_t> cuts;
    for (auto& x : runs) {
        cuts.push_back(x.r.first);
        cuts.push_back((uint64_t)x.r.first + x.r.n);
    }
    std::sort(cuts.begin(), cuts.end());
    cuts.erase(std::unique(cuts.begin(), cuts.end()), cuts.end());
    std::sort(runs.begin(), runs.end(), [](const Run& a, const Run& b) { return a.r.first < b.r.first; });
    std::map<uint32_t, TargetRun> active;   // by call: a set lists a neuron once, so one run per call
    size_t next = 0;
    uint64_t q = 0, n_runs = 0;
    for (size_t i = 0; i + 1 < cuts.size(); ++i) {
        for (auto it = active.begin(); it != active.end();)
            it = (uint64_t)it->second.first + it->second.n <= cuts[i] ? active.erase(it) : std::next(it);
        for (; next < runs.size() && runs[next].r.first <= cuts[i]; ++next) active[runs[next].call] = runs[next].r;
        if (active.empty()) continue;
        if (ent.size() + active.size() > max_entries) return false;
        uint64_t D = 0;
        for (auto& kv : active) D += kv.second.K;
        if (D > 0x7fffffffull) return false;
        const uint64_t max_n = 0x7fffffffull / D;   // positions inside an interval stay below 2^31
        for (uint64_t t = cuts[i]; t < cuts[i + 1];) {
            const uint64_t n = std::min(max_n, cuts[i + 1] - t);
            if (ent.size() + active.size() > max_entries) return false;
            TInterval v{};
            v.q0 = q;
            v.q1 = q + n * D;
            v.first = (uint32_t)t;
            v.D = (uint32_t)D;
            v.div = make_fastdiv((uint32_t)D);
            v.e0 = (uint32_t)ent.size();
            v.ne = (uint32_t)active.size();
            uint64_t o = 0;
            for (auto& kv : active) {
                const TargetRun& r = kv.second;
                TEntry e{};
                e.o = (uint32_t)o;
                e.end = (uint32_t)(o + r.K);
                e.K = r.K;
                e.call = kv.first;
                e.base = (int64_t)(r.begin + (t - r.first) * r.K) - (int64_t)o;
                const SrcMap& m = maps[kv.first];
                const size_t at = seg_at[kv.first];
                if (m.nS == 1) {
                    e.split = 1;
                    e.add = e.add2 = m.add;
                } else if (m.nS == 2 && seg_ord[at + 1]) {
                    e.split = (uint32_t)seg_ord[at + 1];
                    e.add = seg_add[at];
                    e.add2 = seg_add[at + 1];
                } else if (at < (1u << 26)) {
                    e.add = (int64_t)m.div_m;
                    e.seg = (uint32_t)at << 6 | m.div_shift;
                }
                ent.push_back(e);
                o += r.K;
            }
            iv.push_back(v);
            q = v.q1;
            n_runs += n * active.size();
            t += n;
        }
    }
    return q == c.n_gen && n_runs * 16 <= q;
}

}  // namespace

int number_variant_count() { return NUMBER_VARIANTS; }

void prepare_all(Ctx& c) {
    const uint32_t P = c.P, PL = c.P_local;
    const uint64_t N = c.n_gen;
    const uint32_t M_local = c.M[PL];
    std::vector<void*> temps;
    auto tmp = [&](size_t bytes) {
        void* p = dalloc(c, bytes);
        temps.push_back(p);
        return p;
    };
    auto cleanup = [&] {
        for (void* p : temps) dfree(c, p);
        temps.clear();
    };
    try {
        // ---------------------------------------------------------- layout tables
        std::vector<uint64_t> host_base(P + 1, 0);
        for (uint32_t h = 0; h < P; ++h) host_base[h + 1] = host_base[h] + c.M[h];
        const uint64_t G = std::max<uint64_t>(host_base[P], 1);
        int32_t amax = -1;
        for (auto& cl : c.calls) amax = std::max(amax, cl.alpha);
        const uint32_t n_a = (uint32_t)(amax + 2);
        const uint32_t n_calls = (uint32_t)c.calls.size();
        std::vector<uint8_t> flag_local(n_calls);
        for (uint32_t k = 0; k < n_calls; ++k) flag_local[k] = flag_sources(c, c.calls[k], PL) ? 1 : 0;
        std::vector<CallD> calls;
        std::vector<uint32_t> with_conns;   // calls with connections on this host
        std::vector<SrcMap> maps;
        std::vector<uint64_t> call_begin;
        std::vector<int64_t> seg_add;       // all calls' segment tables, concatenated
        std::vector<uint64_t> seg_ord;
        std::vector<size_t> seg_at;
        for (uint32_t k = 0; k < n_calls; ++k) {
            const Call& cl = c.calls[k];
            if (!cl.gen_count) continue;
            const CallD d = make_calld(cl, k, flag_local[k]);
            calls.push_back(d);
            const uint64_t a = (uint64_t)(cl.alpha + 1);
            seg_at.push_back(seg_add.size());
            for (size_t j = 0; j < cl.S.seg.size(); ++j) {
                const snnc_segment& g = cl.S.seg[j];
                const uint64_t remote = M_local + a * G + host_base[g.host] + g.first;
                seg_add.push_back((int64_t)(g.host == PL ? g.first : remote) - (int64_t)cl.S.ord_begin[j]);
                seg_ord.push_back(cl.S.ord_begin[j]);
            }
            maps.push_back(SrcMap{seg_add[seg_at.back()], nullptr, nullptr, d.uniform ? d.seg_div.m : 0, d.seg_div.shift, d.S.n});
            with_conns.push_back(k);
            call_begin.push_back(cl.gen_begin);
        }
        call_begin.push_back(N);
        Fills fills;

        // ---------------------------------------------------------- 1-5 image map, keys, sort, first index
        // Default policy: without remote sources the keys hold final sources and
        // the last radix pass unpacks; with remote sources the keys hold global
        // source ids and the images are numbered by a scan over the sorted keys.
        // Other policies (or "map_path"): the images are numbered first (first
        // call of every image source, its order), the keys hold image indices
        // and the last pass unpacks.
        bool remote_net = false;
        for (auto& cl : c.calls)
            for (auto& g : cl.S.seg) remote_net |= (g.host != PL && cl.gen_count > 0);
        const bool mapped = c.numbering != 0 || c.img_sources != 0 || c.force_map_path;
        const uint64_t n_bits = (uint64_t)n_a * G;
        const uint64_t n_words = n_bits / 32 + 1;    // one spare word: rank of the end bit
        const bool need_bits = mapped || amax >= 0;  // the image bit set: numbering before the sort, collective arrays
        uint32_t* bits = nullptr;
        uint64_t* word_rank = nullptr;
        uint64_t* d_hb = nullptr;
        if (need_bits || remote_net) {
            d_hb = static_cast<uint64_t*>(tmp((P + 1) * 8));
            upload(c, d_hb, host_base.data(), (P + 1) * 8);
        }
        if (need_bits) {
            bits = static_cast<uint32_t*>(tmp(n_words * 4));
            HIPCHK(hipMemsetAsync(bits, 0, n_words * 4, c.stream));
            word_rank = static_cast<uint64_t*>(tmp((n_words + 1) * 8));
        }
        uint64_t n_img = 0;
        int32_t* Lmap = nullptr;
        if (mapped) {
            uint32_t* fc = static_cast<uint32_t*>(dalloc(c, n_bits * 4));
            try {
                HIPCHK(hipMemsetAsync(fc, 0xff, n_bits * 4, c.stream));
                bool any_flagged = false;
                for (auto& cd : calls) any_flagged |= (cd.flag && cd.S.n > 0);
                if (N && remote_net && any_flagged) {
                    CallD* d_calls = static_cast<CallD*>(tmp(calls.size() * sizeof(CallD)));
                    upload(c, d_calls, calls.data(), calls.size() * sizeof(CallD));
                    const Lookup L{d_calls, (uint32_t)calls.size(), d_hb, P, PL, G};
                    tstart(c, "prep_first_use");
                    hipLaunchKernelGGL(k_first_use, dim3(grid_for(N, 8192)), dim3(PNT), 0, c.stream, L, c.g_src, N, fc);
                    tstop(c);
                    HIPCHK(hipGetLastError());
                }
                std::vector<FRange> fr;
                uint64_t f_total = 0;
                for (uint32_t k = 0; k < n_calls; ++k) {
                    const Call& cl = c.calls[k];
                    if (flag_local[k] || count_on(cl.T, PL) == 0) continue;
                    for (auto& g : cl.S.seg)
                        if (g.host != PL && g.n) {
                            fr.push_back(FRange{f_total, (uint64_t)(cl.alpha + 1) * G + host_base[g.host] + g.first, k, 0});
                            f_total += g.n;
                        }
                }
                if (f_total) {
                    FRange* d_fr = static_cast<FRange*>(tmp(fr.size() * sizeof(FRange)));
                    upload(c, d_fr, fr.data(), fr.size() * sizeof(FRange));
                    tstart(c, "prep_first_pass");
                    hipLaunchKernelGGL(k_first_pass, dim3(grid_for(f_total)), dim3(PNT), 0, c.stream, d_fr,
                                       (uint32_t)fr.size(), f_total, fc);
                    tstop(c);
                    HIPCHK(hipGetLastError());
                }
                tstart(c, "prep_fc_bits");
                hipLaunchKernelGGL(k_fc_bits, dim3(grid_for(n_bits)), dim3(PNT), 0, c.stream, fc, n_bits, n_words, bits);
                tstop(c);
                HIPCHK(hipGetLastError());
                n_img = scan_popc_u64(c, bits, word_rank, n_words, true);
                if ((uint64_t)M_local + n_img > 0x7fffffffull)
                    raise(SNNC_EUNSUPPORTED, "more than 2^31-1 local and image neurons");
                int32_t* R = result<int32_t>(c, SNNC_R_VAL, n_img);
                Lmap = result<int32_t>(c, SNNC_L_VAL, n_img);
                const uint32_t call_bits = bits_for(n_calls);
                const bool by_call = c.numbering == 1 && call_bits > 0;
                uint64_t* ik0 = nullptr;
                uint32_t* iv0 = nullptr;
                if (by_call && n_img) {
                    ik0 = static_cast<uint64_t*>(tmp(n_img * 8));
                    iv0 = static_cast<uint32_t*>(tmp(n_img * 4));
                }
                if (n_img) {
                    tstart(c, "prep_img_list");
                    hipLaunchKernelGGL(k_img_list, dim3(grid_for(n_words)), dim3(PNT), 0, c.stream, bits, word_rank,
                                       n_words, fc, d_hb, P, G, R, ik0, iv0);
                    tstop(c);
                    HIPCHK(hipGetLastError());
                }
                dfree(c, fc);
                fc = nullptr;
                if (n_img && by_call) {
                    // stable sort of the canonical indices by first call: the paper's order
                    uint64_t* ik1 = static_cast<uint64_t*>(tmp(n_img * 8));
                    uint32_t* iv1 = static_cast<uint32_t*>(tmp(n_img * 4));
                    struct Tag {   // its passes are not the connections'
                        Ctx& c;
                        explicit Tag(Ctx& ctx) : c(ctx) { c.sort_tag = "prep_first_sort"; }
                        ~Tag() { c.sort_tag = nullptr; }
                    } tag(c);
                    const int w = radix_sort(c, ik0, iv0, ik1, iv1, n_img, 16, 16 + call_bits, nullptr, nullptr);
                    tstart(c, "prep_number_calls");
                    hipLaunchKernelGGL(k_scatter_l, dim3((unsigned)((n_img + 255) / 256)), dim3(256), 0, c.stream,
                                       w ? iv1 : iv0, n_img, M_local, Lmap);
                    tstop(c);
                    HIPCHK(hipGetLastError());
                } else if (n_img) {
                    hipLaunchKernelGGL(k_iota_l, dim3((unsigned)((n_img + 255) / 256)), dim3(256), 0, c.stream, Lmap,
                                       n_img, M_local);
                    HIPCHK(hipGetLastError());
                }
                uint64_t* r_off = result<uint64_t>(c, SNNC_R_OFF, (uint64_t)n_a * P + 1);
                int64_t* img_base = result<int64_t>(c, SNNC_IMG_BASE, (uint64_t)n_a * P);
                const uint64_t nk = (uint64_t)n_a * P + 1;
                hipLaunchKernelGGL(k_bounds_bits, dim3((unsigned)((nk + 255) / 256)), dim3(256), 0, c.stream, bits,
                                   word_rank, d_hb, P, n_a, G, M_local, c.numbering == 0 ? 1 : 0, r_off, img_base);
                HIPCHK(hipGetLastError());
            } catch (...) {
                if (fc) dfree(c, fc);
                throw;
            }
        }
        const uint32_t tbits = bits_for(M_local);
        const uint64_t prefix_span = mapped       ? (uint64_t)M_local + n_img
                                     : remote_net ? (uint64_t)M_local + n_bits
                                                  : (uint64_t)M_local;
        const uint32_t sbits = bits_for(prefix_span);
        c.key_bits = sbits + tbits;
        if (sbits + tbits > 48) raise(SNNC_EUNSUPPORTED, "source and target ids need more than 48 key bits");
        int32_t* o_src = nullptr;
        uint64_t* row_ptr = nullptr;
        if (N) {
            // the source maps and, where it exists, the target-major order: one block, one copy
            std::vector<TInterval> iv;
            std::vector<TEntry> ent;
            const bool by_source = target_major(c, with_conns, maps, seg_at, seg_add, seg_ord, iv, ent);
            if (!by_source) {
                iv.clear();
                ent.clear();
            }
            auto up16 = [](size_t b) { return (b + 15) & ~(size_t)15; };
            const size_t b_maps = up16(maps.size() * sizeof(SrcMap)), b_call = up16(call_begin.size() * 8);
            const size_t b_seg = up16(seg_add.size() * 8), b_iv = up16(iv.size() * sizeof(TInterval));
            const size_t b_ent = up16(ent.size() * sizeof(TEntry));
            std::vector<char> tab(b_maps + b_call + 2 * b_seg + b_iv + b_ent);
            char* d_tab = static_cast<char*>(tmp(tab.size()));
            const int64_t* d_seg = reinterpret_cast<const int64_t*>(d_tab + b_maps + b_call);
            const uint64_t* d_ord = reinterpret_cast<const uint64_t*>(d_tab + b_maps + b_call + b_seg);
            for (size_t k = 0; k < maps.size(); ++k) {
                maps[k].seg_add = d_seg + seg_at[k];
                maps[k].seg_ord = d_ord + seg_at[k];
            }
            memcpy(tab.data(), maps.data(), maps.size() * sizeof(SrcMap));
            memcpy(tab.data() + b_maps, call_begin.data(), call_begin.size() * 8);
            memcpy(tab.data() + b_maps + b_call, seg_add.data(), seg_add.size() * 8);
            memcpy(tab.data() + b_maps + b_call + b_seg, seg_ord.data(), seg_ord.size() * 8);
            if (!iv.empty()) {
                memcpy(tab.data() + b_maps + b_call + 2 * b_seg, iv.data(), iv.size() * sizeof(TInterval));
                memcpy(tab.data() + b_maps + b_call + 2 * b_seg + b_iv, ent.data(), ent.size() * sizeof(TEntry));
            }
            upload(c, d_tab, tab.data(), tab.size());
            GenSource gs{};
            gs.src = c.g_src;
            gs.tgt = c.g_tgt;
            gs.delay = c.g_delay;
            gs.weight = reinterpret_cast<const uint32_t*>(c.g_weight);
            gs.maps = reinterpret_cast<const SrcMap*>(d_tab);
            gs.call_begin = reinterpret_cast<const uint64_t*>(d_tab + b_maps);
            gs.ncalls = (uint32_t)maps.size();
            gs.seg_add = d_seg;
            gs.n_seg = (uint32_t)seg_add.size();
            if (by_source) {
                gs.n_iv = (uint32_t)iv.size();
                gs.iv = reinterpret_cast<const TInterval*>(d_tab + b_maps + b_call + 2 * b_seg);
                gs.ent = reinterpret_cast<const TEntry*>(d_tab + b_maps + b_call + 2 * b_seg + b_iv);
            }
            gs.bits = mapped ? bits : nullptr;
            gs.word_rank = mapped ? word_rank : nullptr;
            gs.Lmap = Lmap;
            gs.M_local = M_local;
            gs.tgt_shift = 16 + tbits;
            const uint32_t bit_lo = by_source ? 16 + tbits : 16, bit_hi = 16 + sbits + tbits;
            const Digits dg = plan_sort(c, N, bit_hi - bit_lo).d;   // the sort below takes the same plan
            uint64_t* keys0 = static_cast<uint64_t*>(tmp(N * 8));
            uint32_t* weights = reinterpret_cast<uint32_t*>(c.g_weight);
            uint32_t* moved = by_source ? static_cast<uint32_t*>(tmp(N * 4)) : nullptr;
            const size_t n_hist = (size_t)dg.passes * dg.stride;
            uint64_t* hist = static_cast<uint64_t*>(tmp(std::max<size_t>(n_hist, 1) * 8));
            HIPCHK(hipMemsetAsync(hist, 0, std::max<size_t>(n_hist, 1) * 8, c.stream));
            tstart(c, "prep_keys");
            const uint32_t unit = tm_unit(N);
            if (by_source)
                hipLaunchKernelGGL(k_keys_tmajor,
                                   dim3((unsigned)std::min<uint64_t>((N + unit * 4 - 1) / (unit * 4), 8192)), dim3(PNT),
                                   n_hist * 4 + (adds_in_lds(dg, gs.n_seg) ? gs.n_seg * 8 : 0), c.stream, gs, N, bit_lo, dg, unit,
                                   keys0, moved, hist);
            else
                hipLaunchKernelGGL(k_keys, dim3(hist_grid(N)), dim3(KNT), n_hist * 4, c.stream, gs, N, bit_lo, dg, keys0,
                                   hist);
            tstop(c);
            HIPCHK(hipGetLastError());
            // the source ordinals, targets and delays now live in the keys (released in stream order)
            if (!c.gen_vmm) {   // block store: handed back after Prepare's final wait
                dfree(c, c.g_src); c.g_src = nullptr;
                dfree(c, c.g_tgt); c.g_tgt = nullptr;
                dfree(c, c.g_delay); c.g_delay = nullptr;
            }
            uint64_t* keys1 = static_cast<uint64_t*>(tmp(N * 8));
            uint32_t* vals0 = by_source ? moved : weights;
            uint32_t* vals1 = by_source ? weights : static_cast<uint32_t*>(tmp(N * 4));
            // outputs allocated only now, so they reuse the memory just released.  With images still to be
            // numbered the last pass writes the source prefixes, into the key buffer it does not read,
            // in place of the sources
            o_src = result<int32_t>(c, SNNC_SRC, N);
            FinalOut fo{o_src, nullptr, result<int32_t>(c, SNNC_TGT, N), result<uint16_t>(c, SNNC_DELAY, N),
                        result<float>(c, SNNC_WEIGHT, N), 16 + tbits, tbits ? (1ull << tbits) - 1 : 0};
            const bool unpack_in_sort = !remote_net || mapped;
            const bool wide_prefix = !unpack_in_sort && sbits > 32;
            uint64_t* prefix = nullptr;
            radix_sort(
                c, keys0, vals0, keys1, vals1, N, bit_lo, bit_hi, hist,
                [&](int in) {
                    if (unpack_in_sort) return fo;
                    prefix = in ? keys0 : keys1;
                    if (wide_prefix) fo.prefix64 = prefix;
                    else fo.src = reinterpret_cast<int32_t*>(prefix);
                    return fo;
                },
                N > (1u << 22));   // the wait for the histograms pays where a skipped pass would be long
            if (c.budget) release_lookback(c);   // room for what follows, which needs a small table at most
            if (unpack_in_sort) {
                const uint64_t n_rows = (uint64_t)M_local + n_img;
                row_ptr = result<uint64_t>(c, SNNC_ROW_PTR, n_rows + 1);
                tstart(c, "prep_csr");
                if (n_rows * 64 < N || n_rows > N)   // rows few against connections, or mostly empty: search
                    hipLaunchKernelGGL(k_csr_search, dim3((unsigned)((n_rows + 1 + 255) / 256)), dim3(256), 0,
                                       c.stream, o_src, N, n_rows, row_ptr);
                else
                    hipLaunchKernelGGL(k_csr, dim3(grid_for(N / 4 + 1, 16384)), dim3(PNT), 0, c.stream, o_src, N,
                                       n_rows, row_ptr);
                tstop(c);
                HIPCHK(hipGetLastError());
            } else {
                const uint64_t max_img = std::min<uint64_t>(N, n_bits);
                uint64_t* img_key = static_cast<uint64_t*>(tmp(max_img * 8 + 8));
                row_ptr = result<uint64_t>(c, SNNC_ROW_PTR, (uint64_t)M_local + max_img + 1);
                uint64_t* d_nimg = static_cast<uint64_t*>(tmp(8));
                const NumberShape shape = NUMBER_SHAPES[c.number_variant];
                const uint64_t xtile = (uint64_t)shape.nt * shape.ipt;
                const uint64_t tiles = (N + xtile - 1) / xtile;
                ensure_lookback(c, tiles * 8);
                next_epoch(c);
                tstart(c, "prep_number");
                const uint32_t taken = c.lookback_recount ? 0u : c.sort_epoch;
                auto number = [&](auto kern32, auto kern64, int nt) {
                    if (wide_prefix)
                        hipLaunchKernelGGL(kern64, dim3((unsigned)tiles), dim3(nt), 0, c.stream,
                                           (const uint64_t*)prefix, N, M_local, (uint64_t*)c.lookback,
                                           c.sort_epoch, taken, c.lookback_spins, o_src, img_key, row_ptr, d_nimg);
                    else
                        hipLaunchKernelGGL(kern32, dim3((unsigned)tiles), dim3(nt), 0, c.stream,
                                           reinterpret_cast<const uint32_t*>(prefix), N, M_local, (uint64_t*)c.lookback,
                                           c.sort_epoch, taken, c.lookback_spins, o_src, img_key, row_ptr, d_nimg);
                };
#define NUMBER(nt, ipt) number(k_number<nt, ipt, uint32_t>, k_number<nt, ipt, uint64_t>, nt)
                switch (shape.nt * 100 + shape.ipt) {
                case 102412: NUMBER(1024, 12); break;
                case 51212: NUMBER(512, 12); break;
                case 25612: NUMBER(256, 12); break;
                case 25616: NUMBER(256, 16); break;
                case 25608: NUMBER(256, 8); break;
                case 25606: NUMBER(256, 6); break;
                case 51208: NUMBER(512, 8); break;
                case 102410: NUMBER(1024, 10); break;
                default: NUMBER(1024, 8); break;
                }
#undef NUMBER
                tstop(c);
                HIPCHK(hipGetLastError());
                download(c, &n_img, d_nimg, 8);
                c.counts[SNNC_ROW_PTR] = (uint64_t)M_local + n_img + 1;
                if ((uint64_t)M_local + n_img > 0x7fffffffull)
                    raise(SNNC_EUNSUPPORTED, "more than 2^31-1 local and image neurons");
                int32_t* R = result<int32_t>(c, SNNC_R_VAL, n_img);
                Lmap = result<int32_t>(c, SNNC_L_VAL, n_img);
                uint64_t* r_off = result<uint64_t>(c, SNNC_R_OFF, (uint64_t)n_a * P + 1);
                int64_t* img_base = result<int64_t>(c, SNNC_IMG_BASE, (uint64_t)n_a * P);
                if (n_img) {
                    tstart(c, "prep_rvals");
                    hipLaunchKernelGGL(k_rvals_sorted, dim3((unsigned)((n_img + 256 * RV_RUN - 1) / (256 * RV_RUN))),
                                       dim3(256), 0, c.stream,
                                       img_key, n_img, d_hb, P, G, R);
                    tstop(c);
                    HIPCHK(hipGetLastError());
                    if (need_bits) {
                        tstart(c, "prep_bits");
                        hipLaunchKernelGGL(k_bits_sorted, dim3((unsigned)((n_img + 255) / 256)), dim3(256), 0, c.stream,
                                           img_key, n_img, bits);
                        tstop(c);
                        HIPCHK(hipGetLastError());
                    }
                    hipLaunchKernelGGL(k_iota_l, dim3((unsigned)((n_img + 255) / 256)), dim3(256), 0, c.stream, Lmap,
                                       n_img, M_local);
                    HIPCHK(hipGetLastError());
                }
                const uint64_t nk = (uint64_t)n_a * P + 1;
                tstart(c, "prep_bounds");
                hipLaunchKernelGGL(k_bounds_sorted, dim3((unsigned)((nk + 255) / 256)), dim3(256), 0, c.stream, img_key,
                                   n_img, d_hb, P, n_a, G, M_local, r_off, img_base);
                tstop(c);
                HIPCHK(hipGetLastError());
            }
        } else {
            o_src = result<int32_t>(c, SNNC_SRC, 0);
            result<int32_t>(c, SNNC_TGT, 0);
            result<uint16_t>(c, SNNC_DELAY, 0);
            result<float>(c, SNNC_WEIGHT, 0);
            const uint64_t n_rows = (uint64_t)M_local + n_img;
            row_ptr = result<uint64_t>(c, SNNC_ROW_PTR, n_rows + 1);
            fills.add(row_ptr, n_rows + 1, 0);
        }
        if (!mapped && (!remote_net || !N)) {
            result<int32_t>(c, SNNC_R_VAL, 0);
            result<int32_t>(c, SNNC_L_VAL, 0);
            fills.add(result<uint64_t>(c, SNNC_R_OFF, (uint64_t)n_a * P + 1), (uint64_t)n_a * P + 1, 0);
            fills.add(reinterpret_cast<uint64_t*>(result<int64_t>(c, SNNC_IMG_BASE, (uint64_t)n_a * P)), (uint64_t)n_a * P,
                      M_local);
        }
        c.n_img = n_img;
        // word ranks of the image bit set (the collective arrays look images up by bit)
        if (need_bits && !mapped) scan_popc_u64(c, bits, word_rank, n_words, false);
        if (!c.gen_vmm) {   // block store: unmapped after the final wait of Prepare
            dfree(c, c.g_weight);
            c.g_weight = nullptr;
            c.cap_gen = 0;
        }
        (void)row_ptr;

        // ---------------------------------------------------------- 6 point-to-point lists
        const uint32_t wpr = (M_local + 31) / 32 + 1;     // words per row (+1 spare)
        const uint64_t n_rw = (uint64_t)P * wpr;
        uint32_t* rows = nullptr;   // allocated when some call has an entry to make
        auto row_of = [&](uint32_t tau) {
            if (!rows) {
                rows = static_cast<uint32_t*>(tmp(n_rw * 4));
                HIPCHK(hipMemsetAsync(rows, 0, n_rw * 4, c.stream));
            }
            return rows + (uint64_t)tau * wpr;
        };
        std::vector<WRange> wr;
        uint64_t w_total = 0;
        for (auto& cl : c.calls) {
            if (cl.alpha != -1) continue;
            bool has_local_source = false;
            for (auto& g : cl.S.seg) has_local_source |= (g.host == PL && g.n > 0);
            if (!has_local_source) continue;
            for (uint32_t tau = 0; tau < P; ++tau) {
                if (tau == PL || count_on(cl.T, tau) == 0) continue;
                if (flag_sources(c, cl, tau)) {   // regenerate tau's draws, keep the local sources they use
                    gen_mark(c, cl, tau, row_of(tau));
                    continue;
                }
                for (auto& g : cl.S.seg)          // not flagged: every local source of the call
                    if (g.host == PL && g.n) {
                        wr.push_back(WRange{w_total, (uint64_t)tau * wpr, g.first, g.first + g.n});
                        w_total += ((g.first + g.n - 1) >> 5) - (g.first >> 5) + 1;
                    }
            }
        }
        if (w_total) {
            row_of(0);
            WRange* d_wr = static_cast<WRange*>(tmp(wr.size() * sizeof(WRange)));
            upload(c, d_wr, wr.data(), wr.size() * sizeof(WRange));
            tstart(c, "prep_s_ranges");
            hipLaunchKernelGGL(k_set_ranges, dim3(grid_for(w_total)), dim3(PNT), 0, c.stream, d_wr, (uint32_t)wr.size(),
                               w_total, rows);
            tstop(c);
            HIPCHK(hipGetLastError());
        }
        uint64_t* s_off = result<uint64_t>(c, SNNC_S_OFF, P + 1);
        uint64_t* tp_ptr = result<uint64_t>(c, SNNC_TP_PTR, (uint64_t)M_local + 1);
        uint64_t* row_rank = nullptr;
        uint64_t n_s = 0;
        if (rows) {
            row_rank = static_cast<uint64_t*>(tmp((n_rw + 1) * 8));
            n_s = scan_popc_u64(c, rows, row_rank, n_rw, true);
            hipLaunchKernelGGL(k_row_offsets, dim3((P + 1 + 255) / 256), dim3(256), 0, c.stream, row_rank, P, wpr, s_off);
            HIPCHK(hipGetLastError());
        } else {
            fills.add(s_off, P + 1, 0);
        }
        int32_t* S = result<int32_t>(c, SNNC_S_VAL, n_s);
        uint32_t* Tv = result<uint32_t>(c, SNNC_T_VAL, n_s);
        uint32_t* Pv = result<uint32_t>(c, SNNC_P_VAL, n_s);
        if (n_s) {
            tstart(c, "prep_s_vals");
            hipLaunchKernelGGL(k_s_vals, dim3(grid_for(n_rw)), dim3(PNT), 0, c.stream, rows, row_rank, n_rw, wpr, S);
            tstop(c);
            HIPCHK(hipGetLastError());
            uint32_t* cnt = static_cast<uint32_t*>(tmp((size_t)M_local * 4));
            tstart(c, "prep_tp");
            hipLaunchKernelGGL(k_tp_count, dim3((M_local + PNT - 1) / PNT), dim3(PNT), 0, c.stream, rows, P, wpr,
                               M_local, cnt);
            tstop(c);
            HIPCHK(hipGetLastError());
            scan_u32_u64(c, cnt, tp_ptr, M_local, false);
            tstart(c, "prep_tp");
            hipLaunchKernelGGL(k_tp_fill, dim3((M_local + PNT - 1) / PNT), dim3(PNT), 0, c.stream, rows, row_rank, s_off,
                               P, wpr, M_local, tp_ptr, Tv, Pv);
            tstop(c);
            HIPCHK(hipGetLastError());
        } else {
            fills.add(tp_ptr, (uint64_t)M_local + 1, 0);
        }

        // ---------------------------------------------------------- 7 collective arrays
        std::vector<int32_t> groups;
        for (auto& cl : c.calls)
            if (cl.alpha >= 0) groups.push_back(cl.alpha);
        std::sort(groups.begin(), groups.end());
        groups.erase(std::unique(groups.begin(), groups.end()), groups.end());
        const uint32_t NG = (uint32_t)groups.size();
        std::vector<HRange> ranges;
        std::vector<uint64_t> h_off_h((size_t)NG * P + 1, 0);
        std::vector<LRange> lranges;
        std::vector<uint32_t> g_first(NG + 1, 0);
        uint64_t h_total = 0;
        for (uint32_t g = 0; g < NG; ++g) {
            std::vector<std::vector<std::pair<uint32_t, uint32_t>>> per(P);
            for (auto& cl : c.calls)
                if (cl.alpha == groups[g])
                    for (auto& sg : cl.S.seg) per[sg.host].push_back({sg.first, sg.first + sg.n});
            g_first[g] = (uint32_t)lranges.size();
            for (uint32_t sigma = 0; sigma < P; ++sigma) {
                auto& v = per[sigma];
                std::sort(v.begin(), v.end());
                std::vector<std::pair<uint32_t, uint32_t>> merged;
                for (auto& r : v) {
                    if (!merged.empty() && r.first <= merged.back().second) merged.back().second = std::max(merged.back().second, r.second);
                    else merged.push_back(r);
                }
                h_off_h[(size_t)g * P + sigma] = h_total;
                uint64_t pos = 0;
                for (auto& r : merged) {
                    ranges.push_back(HRange{h_total, r.first, r.second - r.first, (uint32_t)(groups[g] + 1), sigma});
                    if (sigma == PL) lranges.push_back(LRange{r.first, r.second, pos});
                    h_total += r.second - r.first;
                    pos += r.second - r.first;
                }
            }
        }
        g_first[NG] = (uint32_t)lranges.size();
        h_off_h[(size_t)NG * P] = h_total;
        int32_t* d_groups = result<int32_t>(c, SNNC_GROUPS, NG);
        upload(c, d_groups, groups.data(), NG * 4);
        uint64_t* h_off = result<uint64_t>(c, SNNC_H_OFF, (uint64_t)NG * P + 1);
        if (NG) upload(c, h_off, h_off_h.data(), h_off_h.size() * 8);
        else fills.add(h_off, 1, 0);
        int32_t* Hv = result<int32_t>(c, SNNC_H_VAL, h_total);
        int32_t* Iv = result<int32_t>(c, SNNC_I_VAL, h_total);
        if (h_total) {
            HRange* d_rg = static_cast<HRange*>(tmp(ranges.size() * sizeof(HRange)));
            upload(c, d_rg, ranges.data(), ranges.size() * sizeof(HRange));
            tstart(c, "prep_hi");
            hipLaunchKernelGGL(k_hi, dim3(grid_for((h_total + HI_RUN - 1) / HI_RUN)), dim3(PNT), 0, c.stream, d_rg,
                               (uint32_t)ranges.size(), h_total, bits, word_rank, Lmap, c.numbering == 0 ? 1 : 0, M_local,
                               d_hb, G, PL, Hv, Iv);
            tstop(c);
            HIPCHK(hipGetLastError());
        }
        uint64_t* gq_ptr = result<uint64_t>(c, SNNC_GQ_PTR, (uint64_t)M_local + 1);
        uint64_t n_gq = 0;
        if (M_local && !lranges.empty()) {
            LRange* d_lr = static_cast<LRange*>(tmp(lranges.size() * sizeof(LRange)));
            upload(c, d_lr, lranges.data(), lranges.size() * sizeof(LRange));
            uint32_t* d_gf = static_cast<uint32_t*>(tmp((NG + 1) * 4));
            upload(c, d_gf, g_first.data(), (NG + 1) * 4);
            uint32_t* cnt = static_cast<uint32_t*>(tmp((size_t)M_local * 4));
            tstart(c, "prep_gq");
            hipLaunchKernelGGL(k_gq, dim3((M_local + PNT - 1) / PNT), dim3(PNT), 0, c.stream, d_lr, d_gf, NG, d_groups,
                               M_local, (const uint64_t*)nullptr, cnt, (int32_t*)nullptr, (uint32_t*)nullptr);
            tstop(c);
            HIPCHK(hipGetLastError());
            n_gq = scan_u32_u64(c, cnt, gq_ptr, M_local, true);
            int32_t* Gv = result<int32_t>(c, SNNC_G_VAL, n_gq);
            uint32_t* Qv = result<uint32_t>(c, SNNC_Q_VAL, n_gq);
            if (n_gq) {
                tstart(c, "prep_gq");
                hipLaunchKernelGGL(k_gq, dim3((M_local + PNT - 1) / PNT), dim3(PNT), 0, c.stream, d_lr, d_gf, NG,
                                   d_groups, M_local, (const uint64_t*)gq_ptr, cnt, Gv, Qv);
                tstop(c);
                HIPCHK(hipGetLastError());
            }
        } else {
            fills.add(gq_ptr, (uint64_t)M_local + 1, 0);
            result<int32_t>(c, SNNC_G_VAL, 0);
            result<uint32_t>(c, SNNC_Q_VAL, 0);
        }
        if (fills.count) {
            uint64_t most = 0;
            for (int k = 0; k < fills.count; ++k) most = std::max(most, fills.n[k]);
            tstart(c, "prep_fills");
            hipLaunchKernelGGL(k_fills, dim3(grid_for(most, 4096)), dim3(PNT), 0, c.stream, fills);
            tstop(c);
            HIPCHK(hipGetLastError());
        }
        place_memory_level(c, M_local);
    } catch (...) {
        cleanup();
        throw;
    }
    cleanup();
}

void free_array(Ctx& c, DevArray& a) {
    if (!a.host) dfree(c, a.p);   // host arrays lie in the context's pinned block
    a = DevArray{};
}

}  // namespace snnc
