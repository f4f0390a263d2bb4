// The whole policy search (Alg. 2, Sec. IV-F, one frequency interval per pack) as one kernel, for
// searches that set the packs in the order the evaluators visit them.
//
// A stage-by-stage search evaluates every stored policy times every level from the first node to
// the last.  But when packs are set in visiting order, the policies of stage q differ only in
// packs 0 .. q: everything after pack q still runs at the top level, with durations that no policy
// changes.  A stored policy is therefore kept as what the rest of the graph reads of it:
//   live[k]  the finish times of visited nodes that an unvisited node follows (a few values),
//   m        the latest finish among visited nodes without successors (and constant nodes),
//   ed, eb   the closed fp32 energy blocks' fp64 sum and the open fp32 block,
// and extending it by pack q at level f costs a table entry instead of a pass over the graph:
//   EFT  = max(cst_q, live predecessors) + t[q][f]
//   T    = max(R, EFT + tail_q),   R = max(m, C_q, live[k] + outw_q[k])
// where tail_q is the longest path after pack q, outw_q[k] the longest path that leaves node k by
// an unvisited successor other than q, and C_q the longest path from a constant start floor of a
// node after q, all with packs at the top level (host constants).  With exact time sums (every sum
// along a path an exact fp32 number, whatever the order) T is bit for bit the evaluators' makespan.
// The energy is accumulated as they do: the open block goes on with the top-level energies of its
// remaining packs one by one (in fp32), and the later blocks, which hold only top-level packs, are one
// constant: the host checks that every fp64 sum of block sums is exact, so their order is free.
//
// One workgroup runs every stage: one pass over the (state, level) candidates with a 64-bit LDS
// minimum per makespan bucket, then one thread per bucket writes the winner's state (the other half
// of a double buffer) and its back pointer; two LDS barriers a stage and no launch between stages.
// The records of stage q + 2 are on their way while stage q runs.  At the end the best policy is
// read off the back pointers, staged through LDS so that the chain of dependent reads is an LDS
// chain.
//
// What bounds it is the instructions and latency of a stage on one compute unit, not bytes: about 40
// fp32 additions a candidate for the rest of its energy block (a row of 16 lanes holds 16 of the
// block's energies and each is added with one broadcast-operand instruction: with LDS reads 2.60 us a
// stage, with scalar loads 2.48, this way 1.95, on 512 packs), then the winner's chain of LDS reads.
// Searches of 64 buckets, 16 levels: 512 packs on 4 streams 15.1 -> 1.00 ms, 4,096 packs on 8 streams
// 88.2 -> 9.2 ms against the search by stages, which needs three to four launches a stage.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <climits>
#include <cmath>
#include <cstring>
#include <type_traits>

#include "emo_internal.h"

namespace emo {
namespace {

constexpr int kThreads = 1024;
constexpr unsigned long long kEmptyKey = ~0ull;
constexpr size_t kSearchLds = 150 * 1024;

// Words of a stage record: a header, then (outw, predw)[L] (spare slots weigh -inf, and so does the
// slot of the previous stage's pack, whose weights are kRecEftOutw and kRecEftPredw).
enum { kRecLater = 0 /* fp64: energy of the later blocks */, kRecTail = 2, kRecBlkPos /* place in the energy block */,
       kRecCst, kRecFloor, kRecEftOutw, kRecEftPredw,
       kRecOut, kRecFlags, kRecFixBegin, kRecFixCount, kRecHdr };
constexpr uint32_t kRecSink = 1u, kRecCloses = 2u;   // flags: no successors; the last pack of its energy block
// Words of a fixed step's record: a header, then predw[L].
enum { kFixCst = 0, kFixDur, kFixOut, kFixSink, kFixHdr = 4 };

struct Lds {
    uint32_t ring_words;         // a stage's record and table row
    uint32_t keys;               // u64 [NB]
    uint32_t kstate;             // [2] blocks of states: float4 {R, est, eb, m} [NB], ed f64 [NB], live f32 [L][NB]
    uint32_t state_bytes;        // one of them
    uint32_t tst;                // f32 [NB]
    uint32_t total;
};

__host__ __device__ inline Lds search_lds(int F, int L, int NB) {
    Lds o;
    const uint32_t n = static_cast<uint32_t>(NB);
    o.ring_words = (kRecHdr + 2u * static_cast<uint32_t>(L + F) + 3u) & ~3u;
    o.kstate = (3u * o.ring_words * 4u + 15u) & ~15u;          // (the ring is at 0)
    o.state_bytes = (n * (24u + 4u * static_cast<uint32_t>(L)) + 15u) & ~15u;
    o.keys = o.kstate + 2u * o.state_bytes;
    o.tst = o.keys + 8u * n;
    o.total = o.tst + 4u * n;
    return o;
}

struct State {
    float4 *a;     // R, est, eb, m
    double *ed;
    float *live;   // [L][NB]
};

__device__ __forceinline__ State state_at(char *lds, const Lds &l, int half, int NB) {
    State s;
    s.a = reinterpret_cast<float4 *>(lds + l.kstate + static_cast<uint32_t>(half) * l.state_bytes);
    s.ed = reinterpret_cast<double *>(s.a + NB);
    s.live = reinterpret_cast<float *>(s.ed + NB);
    return s;
}

// Barrier for LDS traffic only: the records in flight and the back pointers stay in flight.
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// floor(T / q) - bmin with the quotient rounded as a division rounds it: the product with the
// reciprocal decides it unless it lies next to a whole number (its error is below 2^-50 of it).
// Callers take results in [0, NB) only: the conversion saturates.
__device__ __forceinline__ int bucket_of(float T, double q, double rq, double bmin) {
    const double d = static_cast<double>(T) * rq;
    double k = floor(d);
    const double frac = d - k;
    if (!(frac > 1e-6 && frac < 1.0 - 1e-6 && d < 268435456.0)) k = floor(static_cast<double>(T) / q);
    return static_cast<int>(k - bmin);
}

// x of lane J of the lane's row of 16 lanes (every lane active)
template <int J>
__device__ __forceinline__ float row_bcast(float x) {
    return __uint_as_float(static_cast<uint32_t>(__builtin_amdgcn_update_dpp(
        0, static_cast<int>(__float_as_uint(x)), 0x150 + J, 0xf, 0xf, true)));
}

// Adds the 16 values that the rows hold in x, lane by lane, to N sums.
template <int N, int J = 0>
__device__ __forceinline__ void add_row(float (&sum)[N], float x) {
    const float v = row_bcast<J>(x);
#pragma unroll
    for (int i = 0; i < N; ++i) sum[i] += v;
    if constexpr (J < 15) add_row<N, J + 1>(sum, x);
}

template <int L>
__global__ void __launch_bounds__(kThreads)
dp_search_kernel(SearchProg g, const float2 *__restrict__ tab, float tmax, double q, double bmin, int NB,
                 uint32_t *__restrict__ bp, uint8_t *__restrict__ best, emo_selection *__restrict__ res) {
    extern __shared__ double2 smem[];
    char *lds = reinterpret_cast<char *>(smem);
    const int t = threadIdx.x;
    const int P = g.P, F = g.F;
    const Lds l = search_lds(F, L, NB);
    unsigned long long *keys = reinterpret_cast<unsigned long long *>(lds + l.keys);
    float *tst = reinterpret_cast<float *>(lds + l.tst);
    const int nw = static_cast<int>(l.ring_words);   // at most kThreads (checked by the host)
    constexpr int kRec = kRecHdr + 2 * L;            // words of a record
    const float inf = __builtin_inff();

    // ring word t of stage s: its record, its table row (stages past the last repeat it; the words that
    // round the ring up read on into the table or its spare entries)
    const uint32_t *src = t < kRec ? g.recs + t : reinterpret_cast<const uint32_t *>(tab) + (t - kRec);
    const int src_pitch = t < kRec ? kRec : 2 * F;
    auto ring_word = [&](int s) -> uint32_t {
        return t < nw ? src[static_cast<int64_t>(s < P ? s : P - 1) * src_pitch] : 0u;
    };
    uint32_t *r0 = reinterpret_cast<uint32_t *>(lds), *r1 = r0 + nw, *r2 = r1 + nw;   // stages st, st + 1, st + 2
    if (t < nw) {
        r0[t] = ring_word(0);
        r1[t] = ring_word(1);
    }
    // candidate t of a pass over the candidates: state t / F, level t % F; and the step to the next
    const int b0 = t / F, f0 = t - b0 * F;
    const int db = kThreads / F, df = kThreads - db * F;
    const double rq = 1.0 / q;
    State cur = state_at(lds, l, 0, NB), nxt = state_at(lds, l, 1, NB);
    // (until its record arrives, the first stage's floor and start come from memory)
    for (int b = t; b < NB; b += kThreads) {   // P_0 is the only state
        keys[b] = kEmptyKey;
        cur.a[b] = make_float4(b == 0 ? fmaxf(g.t_const, __uint_as_float(g.recs[kRecFloor])) : inf,
                               __uint_as_float(g.recs[kRecCst]), 0.f, g.t_const);
        cur.ed[b] = 0.0;
        for (int k = 0; k < L; ++k) cur.live[k * NB + b] = 0.f;
    }
    // every row of 16 lanes holds the open energy block at the top level, lane j packs j, j + 16, ..; packs
    // up to the stage's are zeros (adding zero changes nothing)
    float rest[kEnergyBlock / 16], coming[kEnergyBlock / 16];
    const float *etop = g.etop + (t & 15);
#pragma unroll
    for (int k = 0; k < kEnergyBlock / 16; ++k) coming[k] = rest[k] = etop[16 * k];
    lds_barrier();
    const int ncand = NB * F;
    for (int st = 0; st < P; ++st) {
        const float2 *row = reinterpret_cast<const float2 *>(r0 + kRec);
        const uint32_t pre = ring_word(st + 2);
        const float tail = __uint_as_float(r0[kRecTail]);
        const int pos = __builtin_amdgcn_readfirstlane(static_cast<int>(r0[kRecBlkPos]));
        const double later = *reinterpret_cast<const double *>(r0 + kRecLater);
        if (pos == 0) {   // a block opens: the next one's energies are asked for
            etop += kEnergyBlock;
#pragma unroll
            for (int k = 0; k < kEnergyBlock / 16; ++k) {
                rest[k] = coming[k];
                coming[k] = etop[16 * k];   // (past the last block: a row of zeros)
            }
        }
#pragma unroll
        for (int k = 0; k < kEnergyBlock / 16; ++k) rest[k] = 16 * k + (t & 15) == pos ? 0.f : rest[k];
        // N candidates (b[i], f[i]) side by side: state b with pack st at level f.  A key's low word
        // b << 8 | f orders like the candidate's number b * F + f, and is its back pointer.
        auto candidates = [&](auto n, const int *b, const int *f, const bool *in) {
            constexpr int N = decltype(n)::value;
            float T[N], eb[N];
            double ed[N];
#pragma unroll
            for (int i = 0; i < N; ++i) {
                const float4 a = cur.a[b[i]];
                const float2 te = row[f[i]];
                T[i] = fmaxf(a.x, a.y + te.x + tail);   // (an empty state has R = +inf)
                eb[i] = a.z + te.y;
                ed[i] = cur.ed[b[i]];
            }
            if (pos < 15) add_row<N>(eb, rest[0]);
            if (pos < 31) add_row<N>(eb, rest[1]);
            if (pos < 47) add_row<N>(eb, rest[2]);
            if (pos < 63) add_row<N>(eb, rest[3]);
#pragma unroll
            for (int i = 0; i < N; ++i) {
                if (!(in[i] && T[i] <= tmax)) continue;
                const int k = bucket_of(T[i], q, rq, bmin);
                const double e = ed[i] + static_cast<double>(eb[i]) + later;
                const float E = static_cast<float>(e + static_cast<double>(g.static_power) * static_cast<double>(T[i]));
                const unsigned long long key = (static_cast<unsigned long long>(__float_as_uint(E)) << 32) |
                                               static_cast<unsigned>(b[i] << 8 | f[i]);
                if (static_cast<unsigned>(k) < static_cast<unsigned>(NB)) atomicMin(&keys[k], key);
            }
        };
        // (whole waves stay in the loop: lanes past the candidates repeat state 0 and propose nothing)
        int b = b0, f = f0;
        for (int c = t; (c & ~63) < ncand; c += 2 * kThreads) {
            int bb[2] = {b, b + db}, ff[2] = {f, f + df};
            if (ff[1] >= F) {
                ff[1] -= F;
                ++bb[1];
            }
            b = bb[1] + db;
            f = ff[1] + df;
            if (f >= F) {
                f -= F;
                ++b;
            }
            const bool in[2] = {c < ncand, c + kThreads < ncand};
            if (!in[0]) bb[0] = 0;
            if (!in[1]) bb[1] = 0;
            if ((c & ~63) + kThreads < ncand) candidates(std::integral_constant<int, 2>(), bb, ff, in);
            else candidates(std::integral_constant<int, 1>(), bb, ff, in);
        }
        if (t < nw) r2[t] = pre;
        lds_barrier();
        // each bucket's winner becomes stored policy b of the next stage
        const bool last = st + 1 == P;
        for (int b = t; b < NB; b += kThreads) {
            const unsigned long long key = keys[b];
            if (key == kEmptyKey) {
                nxt.a[b] = make_float4(inf, 0.f, 0.f, 0.f);
                continue;
            }
            if (!last) keys[b] = kEmptyKey;
            const uint32_t from = static_cast<uint32_t>(key);
            const int p = static_cast<int>(from >> 8), f = static_cast<int>(from & 0xffu);
            bp[static_cast<int64_t>(st) * NB + b] = from;
            const float2 te = row[f];
            const float4 a = cur.a[p];
            const double ed = cur.ed[p];
            const float eft = a.y + te.x;
            if (last) {
                tst[b] = fmaxf(a.x, eft + tail);
                continue;
            }
            const uint32_t flags = r0[kRecFlags];
            const int out = static_cast<int>(r0[kRecOut]);
            const float2 *w = reinterpret_cast<const float2 *>(r1 + kRecHdr);
            float m = (flags & kRecSink) ? fmaxf(a.w, eft) : a.w;
            const float eb = a.z + te.y;
            float R = eft + __uint_as_float(r1[kRecEftOutw]);
            float est = fmaxf(__uint_as_float(r1[kRecCst]), eft + __uint_as_float(r1[kRecEftPredw]));
            constexpr int C = L < 16 ? L : 16;   // slots at a time (registers)
#pragma unroll 1
            for (int k0 = 0; k0 < L; k0 += C) {
                float v[C];
#pragma unroll
                for (int k = 0; k < C; ++k) v[k] = cur.live[(k0 + k) * NB + p];
#pragma unroll
                for (int k = 0; k < C; ++k) {
                    nxt.live[(k0 + k) * NB + b] = v[k];
                    R = fmaxf(R, v[k] + w[k0 + k].x);
                    est = fmaxf(est, v[k] + w[k0 + k].y);
                }
            }
            if (out >= 0) nxt.live[out * NB + b] = eft;
            // fixed nodes between this pack and the next one
            if (const int nfix = static_cast<int>(r0[kRecFixCount])) {
                const uint32_t *fx = g.fix + static_cast<int64_t>(r0[kRecFixBegin]) * (kFixHdr + L);
                for (int i = 0; i < nfix; ++i, fx += kFixHdr + L) {
                    float x = __uint_as_float(fx[kFixCst]);
                    for (int k = 0; k < L; ++k) x = fmaxf(x, nxt.live[k * NB + b] + __uint_as_float(fx[kFixHdr + k]));
                    x += __uint_as_float(fx[kFixDur]);
                    if (fx[kFixSink]) m = fmaxf(m, x);
                    const int o = static_cast<int>(fx[kFixOut]);
                    if (o >= 0) nxt.live[o * NB + b] = x;
                }
                R = -inf;
                est = __uint_as_float(r1[kRecCst]);
                for (int k = 0; k < L; ++k) {
                    const float x = nxt.live[k * NB + b];
                    R = fmaxf(R, x + w[k].x);
                    est = fmaxf(est, x + w[k].y);
                }
            }
            const bool closes = flags & kRecCloses;
            nxt.a[b] = make_float4(fmaxf(fmaxf(R, m), __uint_as_float(r1[kRecFloor])), est, closes ? 0.f : eb, m);
            nxt.ed[b] = closes ? ed + static_cast<double>(eb) : ed;
        }
        const State s = cur;
        cur = nxt;
        nxt = s;
        uint32_t *const r = r0;
        r0 = r1;
        r1 = r2;
        r2 = r;
        lds_barrier();
    }

    // the least (energy, bucket) over the stored policies that meet tmax
    __shared__ unsigned long long s_key[kThreads / 64];
    __shared__ int s_cnt[kThreads / 64];
    __shared__ int s_state;
    unsigned long long mine = kEmptyKey;
    int cnt = 0;
    for (int b = t; b < NB; b += kThreads) {
        const unsigned long long key = keys[b];
        if (key == kEmptyKey || !(tst[b] <= tmax)) continue;
        ++cnt;
        const unsigned long long kb = (key & 0xffffffff00000000ull) | static_cast<unsigned long long>(b);
        mine = kb < mine ? kb : mine;
    }
    for (int off = 32; off > 0; off >>= 1) {
        const unsigned long long o = __shfl_xor(mine, off);
        mine = o < mine ? o : mine;
        cnt += __shfl_xor(cnt, off);
    }
    if ((t & 63) == 0) {
        s_key[t >> 6] = mine;
        s_cnt[t >> 6] = cnt;
    }
    __syncthreads();
    if (t == 0) {
        for (int w = 1; w < kThreads / 64; ++w) {
            mine = s_key[w] < mine ? s_key[w] : mine;
            cnt += s_cnt[w];
        }
        const int b = static_cast<int>(mine & 0xffffffffull);
        if (mine == kEmptyKey) {
            res->index = -1;
            res->energy = __builtin_nanf("");
            res->makespan = __builtin_nanf("");
        } else {
            res->index = static_cast<int64_t>(floor(static_cast<double>(tst[b]) / q));
            res->energy = __uint_as_float(static_cast<unsigned int>(mine >> 32));
            res->makespan = tst[b];
        }
        res->num_feasible = cnt;
        s_state = mine == kEmptyKey ? -1 : b;
    }
    __syncthreads();   // (also orders the back pointers' stores before the reads below)
    if (s_state < 0) return;
    // the policy, last pack first: chunks of back pointers through LDS
    uint32_t *chunk = reinterpret_cast<uint32_t *>(lds);
    // bytes per stage of a chunk: its back pointers and its level
    int per = static_cast<int>(l.total / (4u * static_cast<uint32_t>(NB) + 1u));
    per = per > P ? P : per;
    for (int end = P; end > 0;) {
        const int n = end < per ? end : per;
        const int q0 = end - n;
        uint8_t *lev = reinterpret_cast<uint8_t *>(chunk + static_cast<int64_t>(n) * NB);
        for (int64_t i = t; i < static_cast<int64_t>(n) * NB; i += kThreads)
            chunk[i] = bp[static_cast<int64_t>(q0) * NB + i];
        __syncthreads();
        if (t == 0) {
            int s = s_state;
            for (int k = n - 1; k >= 0; --k) {
                const uint32_t v = chunk[k * NB + s];
                lev[k] = static_cast<uint8_t>(v & 0xffu);
                s = static_cast<int>(v >> 8);
            }
            s_state = s;
        }
        __syncthreads();
        for (int k = t; k < n; k += kThreads) best[q0 + k] = lev[k];
        __syncthreads();
        end = q0;
    }
}

uint32_t bits(double x) {
    const float f = static_cast<float>(x);   // exact: a sum along a path
    uint32_t u;
    std::memcpy(&u, &f, 4);
    return u;
}

}  // namespace

SearchHost search_build(const JitGraph &g, const std::vector<float> &ttop, const std::vector<float> &etop,
                        const std::vector<float> &emin, const std::vector<float> &emax,
                        const std::vector<int32_t> &blk_end) {
    SearchHost h;
    // every fp64 sum of block sums is exact when all of them are multiples of one power of two that
    // 2^53 of exceed the largest total: a block's fp32 sum is at least (nearly) the sum of its packs'
    // least energies, so a multiple of that sum's 24th bit; a block that is always zero changes nothing
    {
        int p = 0, low = INT_MAX;
        double total = 0.0;
        for (int32_t e : blk_end) {
            double lo = 0.0, hi = 0.0;
            for (; p <= e; ++p) {
                lo += emin[p];
                hi += emax[p];
            }
            if (hi == 0.0) continue;
            if (lo == 0.0) return h;
            low = std::min(low, std::ilogb(lo * (1.0 - 0x1p-10)) - 23);
            total += hi * (1.0 + 0x1p-10);
        }
        if (low != INT_MAX && !(total < std::ldexp(1.0, 53 + low))) return h;
    }
    const int n = static_cast<int>(g.ops.size());
    // longest path from a step's start (head) and after its end (tail) with packs at the top level
    std::vector<double> head(n, 0.0), tail(n, 0.0), floor_after(n + 1, 0.0);
    std::vector<int32_t> last_use(n, -1);
    for (int i = n - 1; i >= 0; --i) {
        for (int32_t u : g.ops[i].out) tail[i] = std::max(tail[i], head[u]);
        head[i] = tail[i] + (g.ops[i].pack >= 0 ? ttop[g.ops[i].pack] : g.ops[i].dur);
        floor_after[i] = std::max(floor_after[i + 1], static_cast<double>(g.ops[i].cst) + head[i]);
        for (int32_t k : g.ops[i].in) last_use[k] = std::max(last_use[k], i);
    }
    // slots of the live finish times: a slot is free again once its last reader is visited
    std::vector<int32_t> slot(n, -1), owner;   // owner[s]: the step whose value slot s holds, or -1
    auto visit = [&](int i) {
        for (int32_t k : g.ops[i].in)
            if (last_use[k] == i) owner[slot[k]] = -1;
        if (last_use[i] < 0) return;
        size_t s = 0;
        while (s < owner.size() && owner[s] >= 0) ++s;
        if (s == owner.size()) owner.push_back(-1);
        owner[s] = i;
        slot[i] = static_cast<int32_t>(s);
    };
    for (int i = 0; i < n; ++i) {
        visit(i);
        if (owner.size() > static_cast<size_t>(kSearchMaxLive)) return h;
    }
    int L = 4;   // the kernel is compiled for a few slot counts
    while (L < static_cast<int>(owner.size())) L *= 2;
    h.L = L;
    owner.assign(L, -1);   // visited again below: the same slots
    h.rec_words = kRecHdr + 2 * L;
    const uint32_t ninf = 0xff800000u;
    // the blocks' packs at the top level, and each block's sum as the evaluators form it
    const size_t nblk = blk_end.size();
    h.etop.assign((nblk + 2) * kEnergyBlock, 0.f);   // (the kernel asks for one or two rows past the last)
    std::vector<double> later(nblk + 1, 0.0);   // sum of the blocks after block k at the top level
    for (size_t k = 0, p = 0; k < nblk; ++k) {
        float eb = 0.f;
        for (size_t j = 0; p <= static_cast<size_t>(blk_end[k]); ++p, ++j) {
            h.etop[k * kEnergyBlock + j] = etop[p];
            eb += etop[p];
        }
        later[k] = eb;
    }
    for (size_t k = nblk; k-- > 0;) later[k] += later[k + 1];
    int pack = 0;
    for (int i = 0; i < n; ++i) {
        const JitOp &op = g.ops[i];
        if (op.pack < 0) {
            std::vector<uint32_t> fx(kFixHdr + L, ninf);
            fx[kFixCst] = bits(op.cst);
            fx[kFixDur] = bits(op.dur);
            fx[kFixOut] = static_cast<uint32_t>(slot[i]);
            fx[kFixSink] = op.out.empty() ? 1u : 0u;
            for (int32_t k : op.in) fx[kFixHdr + slot[k]] = 0u;
            h.fix.insert(h.fix.end(), fx.begin(), fx.end());
            // (a pack precedes every such node)
            ++h.fixed;
            if (h.recs[h.recs.size() - h.rec_words + kRecFixCount]++ == 0) ++h.fixed_stages;
            visit(i);
            continue;
        }
        std::vector<uint32_t> r(h.rec_words, ninf);
        // the previous stage's pack, when no fixed node lies between
        const bool direct = i > 0 && g.ops[i - 1].pack >= 0;
        r[kRecFixCount] = 0u;
        r[kRecCst] = bits(op.cst);
        r[kRecTail] = bits(tail[i]);
        r[kRecFloor] = bits(floor_after[i + 1]);
        r[kRecOut] = static_cast<uint32_t>(slot[i]);
        const size_t blk = std::lower_bound(blk_end.begin(), blk_end.end(), pack) - blk_end.begin();
        std::memcpy(&r[kRecLater], &later[blk + 1], sizeof(double));
        const int first = blk > 0 ? blk_end[blk - 1] + 1 : 0;
        r[kRecBlkPos] = static_cast<uint32_t>(pack - first);
        r[kRecFlags] = (op.out.empty() ? kRecSink : 0u) | (pack == blk_end[blk] ? kRecCloses : 0u);
        r[kRecFixBegin] = static_cast<uint32_t>(h.fix.size() / (kFixHdr + L));
        for (int s = 0; s < L; ++s) {
            const int k = owner[s];
            double w = -1.0;
            bool pred = false;
            if (k >= 0)
                for (int32_t u : g.ops[k].out) {
                    if (u > i) w = std::max(w, head[u]);
                    if (u == i) pred = true;
                }
            uint32_t *const to = direct && k == i - 1 ? &r[kRecEftOutw] : &r[kRecHdr + 2 * s];
            to[0] = w >= 0.0 ? bits(w) : ninf;
            to[1] = pred ? 0u : ninf;
        }
        h.recs.insert(h.recs.end(), r.begin(), r.end());
        visit(i);
        ++pack;
    }
    return h;
}

// Candidates per stage: a stage's work grows with them on one compute unit, while the launches of a
// search by stages cost the same: 16,032 candidates a stage take 6.5 ms here against 19.8 on 512 packs
// (12,336 on 96 packs 0.99 against 1.90), and past this the lead shrinks.
constexpr int64_t kSearchMaxCandidates = 16384;

bool search_fits(const SearchProg &g, int64_t NB) {
    if (kRecHdr + 2 * (g.F + g.L) + 3 > kThreads || NB * g.F > kSearchMaxCandidates ||
        search_lds(g.F, g.L, static_cast<int>(NB)).total > kSearchLds)
        return false;
    // us a stage here: candidates, the winner's live values, and the fixed nodes after a pack, which one
    // thread per bucket walks one after another with L dependent reads each; fitted to measured stages
    // (L 4: 2.1 with 1,024 candidates and 11.0 with 15,488; L 64: 3.8 with 256, 10.5 with 12,800; a pack's
    // first fixed node 1.9 at L 32 and 2.1 to 3.1 at L 64, further ones as below).  A stage of a search by stages takes its launches at least: 12.4 us, 13.2 to 14.3 with 15,488 candidates
    // (graphs of 12 to 40 packs).  Without this rule 40 packs on 40 chains with 12 fixed nodes a pack took
    // 0.67 ms against 0.48 by stages, with 50 2.2 against 0.50.
    const double cand = static_cast<double>(NB * g.F);
    const double each = g.L == 4 ? 0.10 : g.L == 8 ? 0.14 : g.L == 16 ? 0.43 : g.L == 32 ? 0.69 : 1.2;
    const double here = 1.5 + 0.0006 * cand + g.L / 30.0 + (each * g.fixed + 0.035 * g.L * g.fixed_stages) / g.P;
    return here <= 12.0 + 0.0001 * cand;
}

namespace {
template <int L>
hipError_t launch_search_kernel(const SearchProg &g, const float2 *tab, float tmax, double q, double bmin, int NB,
                                uint32_t *bp, uint8_t *best, emo_selection *res, hipStream_t s) {
    // the dynamic LDS limit is raised once per device (the caller made the graph's device current)
    static std::atomic<uint64_t> done{0};
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    const uint64_t bit = dev < 64 ? uint64_t{1} << dev : 0;
    if (!bit || !(done.load(std::memory_order_acquire) & bit)) {
        e = hipFuncSetAttribute(reinterpret_cast<const void *>(&dp_search_kernel<L>),
                                hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(kSearchLds));
        if (e != hipSuccess) return e;
        done.fetch_or(bit, std::memory_order_acq_rel);
    }
    hipLaunchKernelGGL(dp_search_kernel<L>, dim3(1), dim3(kThreads), search_lds(g.F, L, NB).total, s, g, tab, tmax, q,
                       bmin, NB, bp, best, res);
    return hipGetLastError();
}
}  // namespace

hipError_t launch_search(const SearchProg &g, const float2 *tab, float tmax, double q, int64_t bmin, int64_t NB,
                         void *scratch, uint8_t *best, emo_selection *res, hipStream_t s) {
    auto f = g.L == 4    ? launch_search_kernel<4>
             : g.L == 8  ? launch_search_kernel<8>
             : g.L == 16 ? launch_search_kernel<16>
             : g.L == 32 ? launch_search_kernel<32>
                         : launch_search_kernel<64>;
    return f(g, tab, tmax, q, static_cast<double>(bmin), static_cast<int>(NB), static_cast<uint32_t *>(scratch), best,
             res, s);
}

}  // namespace emo
