// Chain-lane kernels for graphs whose candidate-dependent part is a set of disjoint chains —
// for example kernels in stream order whose other predecessors are candidate-independent host
// launch nodes (folded into constant start-time floors).  Such a graph has little parallelism
// per candidate along a chain but one independent chain per stream, so each candidate gets
// `lanes` lanes (a power of two at least the number of chains, at most 64), one per chain.
//
// Per step of a chain (Eq. 1 and Alg. 1 with at most one candidate-dependent predecessor):
//   EFT = max(EFT of the previous step, cst) + dur
// where cst is the latest finish among the step's candidate-independent predecessors and dur the
// pack's table time at its level (Eq. 3) or the node's fixed duration.  The makespan is the max
// over the chains' last finish times and the candidate-independent makespan (Eq. 2).  Padding
// steps (cst = 0, dur = 0, no pack) leave a chain's finish time unchanged, since finish times
// are >= 0.  Pack energies are summed per chain in fp32 blocks of 64 steps added into fp64, and
// the chains' sums are added in fp64 across the candidate's lanes; this order differs from the
// program order of the other kernel kinds, so energies agree with them to the same 1e-5 bound
// but not bit for bit.  Makespans and slack use the same fp32 operations and are identical.
//
// Slack (backward pass, total float): each chain walks its steps in reverse; a step's latest
// finish is the latest start of the next step on its chain (T after the chain's last step), and
// slack = latest finish - EFT.  Finish times are not stored: the forward pass checkpoints the
// finish time entering each block of kStepBlock steps, and the backward pass recomputes a block's
// finish times from its checkpoint (4 bytes per 16 steps of scratch instead of 4 per step).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <atomic>
#include <type_traits>

#include "emo_internal.h"

namespace emo {
namespace {

constexpr int kChainBlockThreads = 1024;
constexpr int K = kChainStepBlock;
constexpr int kEnergySteps = 64;   // fp32 energy block (steps of one chain)
constexpr int kStageBytes = 32 * 1024;

// Plain variant (the rows of a block do not fit the LDS stage): every lane reads its own table
// entries from device memory.
template <bool SLACK>
__global__ void __launch_bounds__(kChainBlockThreads)
chains_kernel(DevGraph g, DevChains c, const uint8_t *__restrict__ levels, int64_t B,
              float *__restrict__ To, float *__restrict__ Eo, float *__restrict__ S,
              float *__restrict__ ck, int64_t pitch) {
    const int64_t gid = static_cast<int64_t>(blockIdx.x) * kChainBlockThreads + threadIdx.x;
    const int64_t cand0 = gid >> c.lane_log;
    const int j = static_cast<int>(threadIdx.x) & (c.lanes - 1);
    const bool active = cand0 < B;
    const int64_t cand = active ? cand0 : B - 1;
    const uint8_t *__restrict__ row = levels + cand * g.P;
    const ChainStep *__restrict__ st = c.steps + j;
    const int F = g.F;
    const unsigned Fu = static_cast<unsigned>(F);
    const int nblk = c.len / K;
    float f = 0.f, eb = 0.f;
    double ed = 0.0;
    unsigned bad = 0u;
    for (int b = 0; b < nblk; ++b) {
        if (SLACK) ck[static_cast<int64_t>(b) * pitch + gid] = f;
#pragma unroll
        for (int i = 0; i < K; ++i) {
            const ChainStep r = st[static_cast<int64_t>(b * K + i) << c.lane_log];
            const unsigned lv = r.pack >= 0 ? row[r.pack] : 0u;
            bad |= lv >= Fu ? 1u : 0u;
            const unsigned l = lv < Fu ? lv : 0u;
            const float2 te = r.pack >= 0 ? g.tab[static_cast<int64_t>(r.pack) * F + l] : make_float2(r.dur, 0.f);
            f = fmaxf(f, r.cst) + te.x;
            eb += te.y;
        }
        if ((b + 1) % (kEnergySteps / K) == 0) {
            ed += static_cast<double>(eb);
            eb = 0.f;
        }
    }
    ed += static_cast<double>(eb);
    float T = f;
    for (int off = 1; off < c.lanes; off <<= 1) {
        T = fmaxf(T, __shfl_xor(T, off));
        ed += __shfl_xor(ed, off);
        bad |= __shfl_xor(bad, off);
    }
    T = fmaxf(T, c.t_const);
    float E = static_cast<float>(ed + static_cast<double>(g.static_power) * static_cast<double>(T));
    if (bad) {
        T = __builtin_nanf("");
        E = __builtin_nanf("");
    }
    if (active && j == 0) {
        To[cand] = T;
        Eo[cand] = E;
    }
    if (!SLACK) return;
    const float nan = __builtin_nanf("");
    float lft = bad ? 0.f : T;
    for (int b = nblk - 1; b >= 0; --b) {
        float fb = ck[static_cast<int64_t>(b) * pitch + gid];
        int pk[K];
        float ti[K], fi[K];
#pragma unroll
        for (int i = 0; i < K; ++i) {
            const ChainStep r = st[static_cast<int64_t>(b * K + i) << c.lane_log];
            pk[i] = r.pack;
            const unsigned lv = r.pack >= 0 ? row[r.pack] : 0u;
            const unsigned l = lv < Fu ? lv : 0u;
            ti[i] = r.pack >= 0 ? g.tabt[static_cast<int64_t>(r.pack) * F + l] : r.dur;
            fb = fmaxf(fb, r.cst) + ti[i];
            fi[i] = fb;
        }
#pragma unroll
        for (int i = K - 1; i >= 0; --i) {
            if (active && pk[i] >= 0) S[cand * g.P + pk[i]] = bad ? nan : lft - fi[i];
            lft = lft - ti[i];
        }
    }
}

// Staged variant (a block's table rows fit kStageBytes): at step k every candidate of the
// workgroup visits the same packs, so the workgroup copies the rows of a block's K x lanes packs
// into LDS once (about 16x less L2 traffic than every lane reading its entry out of a different
// row), and the loop is software-pipelined so that no memory round trip is exposed:
//   - step records of block b+2 are copied into a 3-deep LDS ring,
//   - table rows of block b+1 are copied into the other half of a double buffer,
//   - level bytes of block b+1 are loaded into registers,
// all while block b is computed from LDS and registers; one barrier per block.  The backward
// pass runs the same pipeline downwards (blocks b-2, b-1), reading times only.
// LDS: rows [2][K * lanes * F] (float2 forward, float backward) | records [3][K * lanes].
constexpr int kRowsPerThread = kStageBytes / 8 / kChainBlockThreads;   // float2 entries

// S here is the chain-ordered slack scratch [B][len * lanes] (row pitch srow); a second kernel
// (gather_slack) writes it out in pack order.
template <bool SLACK>
__global__ void __launch_bounds__(kChainBlockThreads)
chains_staged(DevGraph g, DevChains c, const uint8_t *__restrict__ levels, int64_t B,
              float *__restrict__ To, float *__restrict__ Eo, float *__restrict__ S,
              float *__restrict__ ck, int64_t pitch) {
    const int64_t srow = static_cast<int64_t>(c.len) << c.lane_log;
    extern __shared__ float4 smem[];
    const int t = threadIdx.x;
    const int64_t gid = static_cast<int64_t>(blockIdx.x) * kChainBlockThreads + t;
    const int64_t cand0 = gid >> c.lane_log;
    const int j = t & (c.lanes - 1);
    const bool active = cand0 < B;
    const int64_t cand = active ? cand0 : B - 1;
    const uint8_t *__restrict__ row = levels + cand * g.P;
    const int F = g.F;
    const int nslot = K * c.lanes;
    const int nrow = nslot * F;
    const int nblk = c.len / K;
    float2 *rows2 = reinterpret_cast<float2 *>(smem);                 // forward: [2][nrow]
    float *rows1 = reinterpret_cast<float *>(smem);                   // backward: [2][nrow]
    ChainStep *recs = reinterpret_cast<ChainStep *>(rows2 + 2 * nrow); // [3][nslot]
    const ChainStep *__restrict__ gsteps = c.steps;
    auto rec_slot = [&](int b) { return recs + (b % 3) * nslot; };
    const unsigned Fu = static_cast<unsigned>(F);

    // ------------------------------------------------------------------ forward
    if (t < nslot) rec_slot(0)[t] = gsteps[t];
    if (nblk > 1 && t < nslot) rec_slot(1)[t] = gsteps[nslot + t];
    __syncthreads();
    for (int q = 0; q < kRowsPerThread; ++q) {
        const int e = t + q * kChainBlockThreads;
        if (e < nrow) {
            const int32_t pk = rec_slot(0)[e / F].pack;
            rows2[e] = pk >= 0 ? g.tab[static_cast<int64_t>(pk) * F + e % F] : make_float2(0.f, 0.f);
        }
    }
    unsigned lcur[K];
#pragma unroll
    for (int i = 0; i < K; ++i) {
        const int32_t pk = rec_slot(0)[(i << c.lane_log) + j].pack;
        lcur[i] = pk >= 0 ? row[pk] : 0u;
    }
    __syncthreads();
    float f = 0.f, eb = 0.f;
    double ed = 0.0;
    unsigned bad = 0u;
    for (int b = 0; b < nblk; ++b) {
        if (SLACK) ck[static_cast<int64_t>(b) * pitch + gid] = f;
        const bool more = b + 1 < nblk;
        // prefetch: records of block b+2, rows and level bytes of block b+1
        ChainStep rpre{-1, 0.f, 0.f, 0};
        if (b + 2 < nblk && t < nslot) rpre = gsteps[static_cast<int64_t>(b + 2) * nslot + t];
        float2 rowpre[kRowsPerThread];
        unsigned lnext[K];
        if (more) {
            const ChainStep *rn = rec_slot(b + 1);
#pragma unroll
            for (int q = 0; q < kRowsPerThread; ++q) {
                const int e = t + q * kChainBlockThreads;
                const int32_t pk = e < nrow ? rn[e / F].pack : -1;
                rowpre[q] = pk >= 0 ? g.tab[static_cast<int64_t>(pk) * F + e % F] : make_float2(0.f, 0.f);
            }
#pragma unroll
            for (int i = 0; i < K; ++i) {
                const int32_t pk = rn[(i << c.lane_log) + j].pack;
                lnext[i] = pk >= 0 ? row[pk] : 0u;
            }
        }
        // block b from LDS and registers
        const ChainStep *rb = rec_slot(b);
        const float2 *rowb = rows2 + (b & 1) * nrow;
#pragma unroll
        for (int i = 0; i < K; ++i) {
            const int slot = (i << c.lane_log) + j;
            const ChainStep r = rb[slot];
            bad |= lcur[i] >= Fu ? 1u : 0u;
            const unsigned l = lcur[i] < Fu ? lcur[i] : 0u;
            const float2 tv = rowb[slot * F + l];
            const float2 te = r.pack >= 0 ? tv : make_float2(r.dur, 0.f);
            f = fmaxf(f, r.cst) + te.x;
            eb += te.y;
        }
        if ((b + 1) % (kEnergySteps / K) == 0) {
            ed += static_cast<double>(eb);
            eb = 0.f;
        }
        // commit the prefetched block: its buffers were last read before the previous barrier
        if (more) {
            float2 *dst = rows2 + ((b + 1) & 1) * nrow;
#pragma unroll
            for (int q = 0; q < kRowsPerThread; ++q) {
                const int e = t + q * kChainBlockThreads;
                if (e < nrow) dst[e] = rowpre[q];
            }
        }
        if (b + 2 < nblk && t < nslot) rec_slot(b + 2)[t] = rpre;
        __syncthreads();
        if (more) {
#pragma unroll
            for (int i = 0; i < K; ++i) lcur[i] = lnext[i];
        }
    }
    ed += static_cast<double>(eb);
    float T = f;
    for (int off = 1; off < c.lanes; off <<= 1) {
        T = fmaxf(T, __shfl_xor(T, off));
        ed += __shfl_xor(ed, off);
        bad |= __shfl_xor(bad, off);
    }
    T = fmaxf(T, c.t_const);
    float E = static_cast<float>(ed + static_cast<double>(g.static_power) * static_cast<double>(T));
    if (bad) {
        T = __builtin_nanf("");
        E = __builtin_nanf("");
    }
    if (active && j == 0) {
        To[cand] = T;
        Eo[cand] = E;
    }
    if (!SLACK) return;

    // ------------------------------------------------------------------ backward
    const float nan = __builtin_nanf("");
    float lft = bad ? 0.f : T;
    const int top = nblk - 1;
    __syncthreads();   // the forward pass is done with every buffer
    if (t < nslot) rec_slot(top)[t] = gsteps[static_cast<int64_t>(top) * nslot + t];
    if (top >= 1 && t < nslot) rec_slot(top - 1)[t] = gsteps[static_cast<int64_t>(top - 1) * nslot + t];
    __syncthreads();
    for (int q = 0; q < 2 * kRowsPerThread; ++q) {
        const int e = t + q * kChainBlockThreads;
        if (e < nrow) {
            const int32_t pk = rec_slot(top)[e / F].pack;
            rows1[(top & 1) * nrow + e] = pk >= 0 ? g.tabt[static_cast<int64_t>(pk) * F + e % F] : 0.f;
        }
    }
#pragma unroll
    for (int i = 0; i < K; ++i) {
        const int32_t pk = rec_slot(top)[(i << c.lane_log) + j].pack;
        lcur[i] = pk >= 0 ? row[pk] : 0u;
    }
    float fb = ck[static_cast<int64_t>(top) * pitch + gid];
    __syncthreads();
    for (int b = top; b >= 0; --b) {
        const bool more = b >= 1;
        ChainStep rpre{-1, 0.f, 0.f, 0};
        if (b >= 2 && t < nslot) rpre = gsteps[static_cast<int64_t>(b - 2) * nslot + t];
        float rowpre[2 * kRowsPerThread];
        unsigned lnext[K];
        float fnext = 0.f;
        if (more) {
            const ChainStep *rn = rec_slot(b - 1);
#pragma unroll
            for (int q = 0; q < 2 * kRowsPerThread; ++q) {
                const int e = t + q * kChainBlockThreads;
                const int32_t pk = e < nrow ? rn[e / F].pack : -1;
                rowpre[q] = pk >= 0 ? g.tabt[static_cast<int64_t>(pk) * F + e % F] : 0.f;
            }
#pragma unroll
            for (int i = 0; i < K; ++i) {
                const int32_t pk = rn[(i << c.lane_log) + j].pack;
                lnext[i] = pk >= 0 ? row[pk] : 0u;
            }
            fnext = ck[static_cast<int64_t>(b - 1) * pitch + gid];
        }
        const ChainStep *rb = rec_slot(b);
        const float *rowb = rows1 + (b & 1) * nrow;
        float ti[K], fi[K];
#pragma unroll
        for (int i = 0; i < K; ++i) {
            const int slot = (i << c.lane_log) + j;
            const ChainStep r = rb[slot];
            const unsigned l = lcur[i] < Fu ? lcur[i] : 0u;
            ti[i] = r.pack >= 0 ? rowb[slot * F + l] : r.dur;
            fb = fmaxf(fb, r.cst) + ti[i];
            fi[i] = fb;
        }
        // slack in chain order: the candidate's lanes write 4 * lanes contiguous bytes per step
        float *__restrict__ so = S + cand * srow + (static_cast<int64_t>(b) * K << c.lane_log) + j;
#pragma unroll
        for (int i = K - 1; i >= 0; --i) {
            so[i << c.lane_log] = bad ? nan : lft - fi[i];
            lft = lft - ti[i];
        }
        if (more) {
            float *dst = rows1 + ((b - 1) & 1) * nrow;
#pragma unroll
            for (int q = 0; q < 2 * kRowsPerThread; ++q) {
                const int e = t + q * kChainBlockThreads;
                if (e < nrow) dst[e] = rowpre[q];
            }
        }
        if (b >= 2 && t < nslot) rec_slot(b - 2)[t] = rpre;
        __syncthreads();
        if (more) {
#pragma unroll
            for (int i = 0; i < K; ++i) lcur[i] = lnext[i];
            fb = fnext;
        }
    }
}

// Pack-order slack rows from the chain-ordered scratch: thread (c, q) writes packs 4q..4q+3 of
// candidate c (one 16-byte store; 64 lanes cover 1 KB of a row) from their chain positions,
// which are nearly in order (packs are launched round-robin-like over the streams).
constexpr int kGatherThreads = 256;
__global__ void __launch_bounds__(kGatherThreads)
gather_slack(const float *__restrict__ tmp, const int32_t *__restrict__ pos, int64_t B, int32_t P,
             int64_t srow, float *__restrict__ S) {
    const int64_t q = static_cast<int64_t>(blockIdx.x) * kGatherThreads + threadIdx.x;
    const int64_t per_row = P / 4;
    const int64_t cand = q / per_row;
    if (cand >= B) return;
    const int32_t p = static_cast<int32_t>(q - cand * per_row) * 4;
    const float *__restrict__ src = tmp + cand * srow;
    float4 v;
    v.x = src[pos[p]];
    v.y = src[pos[p + 1]];
    v.z = src[pos[p + 2]];
    v.w = src[pos[p + 3]];
    *reinterpret_cast<float4 *>(S + cand * P + p) = v;
}

// ---------------------------------------------------------------- windowed variant
//
// The lane-per-chain kernels above read each candidate's level bytes at the packs its chains
// are at; when the chains drift thousands of pack ids apart (streams launched in random order),
// every 8-step block of a wave touches up to 64 different cache lines, and slack has to be
// written in chain order and gathered.  The windowed kernel cuts the pack ids into windows of
// W packs instead and turns the layout around: a wave is 64 candidates on ONE chain, and a
// workgroup is G groups of 64 candidates x nc chains.  Per window the workgroup copies into
// LDS, with 16-byte loads issued one or two windows ahead into registers:
//   - the G*64 candidates' level bytes of the window (checked against F on the way),
//   - the window's table rows (time and energy; times only in the second pass),
//   - the window's step block: where each chain's steps start, and the step records.
// Each wave then walks its chain's steps inside the window (the count varies per chain; waves
// meet at the window's barrier).  Slack comes from a second pass over the windows (below), which
// writes each step's slack into an LDS tile [candidate][column] that the workgroup writes out in
// pack order with 16-byte stores.
//
// A wave's steps are read 16 at a time, one per lane of every row of 16 lanes, and handed on by
// broadcast operands.  Column W of every level row is 0 and row W of the table is zero, so a fixed node (column W)
// reads a zero time and energy and adds its own duration; its tile entry is column W's pad.
// Energies are summed per chain in fp32 over each window, added into fp64, and the chains'
// sums are added in chain order.
constexpr size_t kWinLds = 150 * 1024;
constexpr size_t kWinSpare = 1024;                   // 16 spare bytes per lane
constexpr int kWinMaxWaves = 16;

__host__ __device__ inline uint32_t round16u(uint32_t x) { return (x + 15u) & ~15u; }

struct WinLayout {
    uint32_t lvl_pitch;    // bytes per candidate row of a level buffer (W + 4)
    uint32_t lvl_buf;      // bytes of one level buffer
    uint32_t off_bad;      // u32 [NC]: candidate has a level >= F
    uint32_t off_tfin;     // f32 [NC]: makespan (NaN when bad)
    uint32_t off_blk;      // [2] step blocks
    uint32_t off_x;        // phase region: tables (forward, backward), chain sums, slack tile
    uint32_t tab_elems;    // entries of one table buffer ((W + 1) * F)
    uint32_t off_tile;     // f32 [NC][W + 1] (backward)
    uint32_t total;
};

__host__ __device__ inline WinLayout win_layout(int W, int NC, int F, int nwaves, int blk_bytes) {
    WinLayout L;
    L.lvl_pitch = static_cast<uint32_t>(W) + 4u;
    L.lvl_buf = round16u(static_cast<uint32_t>(NC) * L.lvl_pitch);
    L.off_bad = 2u * L.lvl_buf;
    L.off_tfin = L.off_bad + 4u * static_cast<uint32_t>(NC);
    L.off_blk = round16u(L.off_tfin + 4u * static_cast<uint32_t>(NC));
    L.off_x = L.off_blk + 2u * static_cast<uint32_t>(blk_bytes);
    // entries per table buffer, a multiple of 4 so that the second buffer starts 16-byte
    // aligned for its 16-byte stores (with fp32 or float2 entries)
    L.tab_elems = (static_cast<uint32_t>(W + 1) * static_cast<uint32_t>(F) + 3u) & ~3u;
    // (256 spare float2 entries: a lookup with an invalid level byte reads at most 255 entries
    // past a table buffer; the backward tables are followed by the slack tile)
    const uint32_t fwd = (2u * L.tab_elems + 256u) * 8u;
    const uint32_t comb = 64u * 8u * kWinMaxWaves + static_cast<uint32_t>(nwaves) * 64u * 4u;
    L.off_tile = L.off_x + round16u(2u * L.tab_elems * 4u);
    const uint32_t bwd = L.off_tile - L.off_x + static_cast<uint32_t>(NC) * static_cast<uint32_t>(W + 1) * 4u;
    uint32_t m = fwd > comb ? fwd : comb;
    m = m > bwd ? m : bwd;
    L.total = L.off_x + m;
    return L;
}

__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Bit 7 of every byte of a word that holds a level >= F (F <= 128: a byte b < 128 gets bit 7
// from (b + 128 - F) exactly when b >= F, and a byte >= 128 has it already).
__device__ __forceinline__ uint32_t bad_levels(uint32_t x, uint32_t addf) {
    return (((x & 0x7f7f7f7fu) + addf) | x) & 0x80808080u;
}

// max of two non-negative finite floats: their bit patterns order like unsigned integers, and
// the integer max needs none of the NaN-quieting that the compiler adds to fmaxf on operands
// loaded from memory.  Finish times and start floors here are always >= 0 and finite.
__device__ __forceinline__ float fmax_nonneg(float a, float b) {
    const unsigned x = __float_as_uint(a), y = __float_as_uint(b);
    return __uint_as_float(x > y ? x : y);
}


struct WinArgs {
    int W, wlog, nc, NC, F;
    int blk_bytes, hdr_words;
    WinLayout L;
};

// 16-byte pieces a thread of nt copies per window: level rows, the table (forward), the table
// (second pass), the step block.
struct WinSlots {
    int lvl, tab8, tab4, blk;
};
__host__ __device__ inline WinSlots win_slots(int W, int NC, int F, int blk_bytes, int nt) {
    WinSlots s;
    s.lvl = (NC * (W / 16) + nt - 1) / nt;
    s.tab8 = (W * F / 2 + nt - 1) / nt;
    s.tab4 = (W * F / 4 + nt - 1) / nt;
    s.blk = (blk_bytes / 16 + nt - 1) / nt;
    return s;
}

// Buffer resources of the planned copies: raw buffer accesses with a 32-bit per-lane offset and a
// uniform offset, and the hardware's range check (an access at or past `bytes` reads zeros and
// writes nothing).  The fourth word is the CDNA3/CDNA4 raw-buffer configuration.
typedef unsigned int emo_u4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ __amdgpu_buffer_rsrc_t win_rsrc(const void *base, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), static_cast<short>(0),
                                             static_cast<int>(bytes), 0x00020000);
}
// An offset past the tables and the step blocks (they hold less than 2^31 bytes, and a uniform offset
// stays below 2^31 too): loads there read zeros.
constexpr uint32_t kWinNoStore = 0x80000000u;

// The copy of a window, with each thread's pieces at offsets fixed for the whole kernel: win_plan
// computes them once, and a window then costs its loads, its stores and a few scalar operations.
// A thread with no piece in a table or block slot loads past the slot's buffer (the range check
// returns zeros without touching memory) and stores them to its lane's spare 16 bytes at LDS
// offset `spare` (so every load is waited for and every store made on every path, which keeps the
// compiler's count of loads in flight exact).  Level pieces are plain loads (of any alignment: a row
// of P bytes may start anywhere); a thread without one loads row 0's first piece.
template <int NL, int NT, int NB>
struct WinPlan {
    static constexpr int kSlots = NL + NT + NB;
    uint32_t src[kSlots];     // byte offset of the piece in its slot's per-window source
    uint32_t dst0[kSlots];    // LDS byte offset of the piece in buffer 0 (or the spare)
    uint32_t dst1[kSlots];    // in buffer 1
    uint32_t has;             // bit i: the thread has a piece in slot i
};

template <int NL, int NT, int NB>
__device__ __forceinline__ WinPlan<NL, NT, NB> win_plan(const WinArgs &a, int esize, int64_t rows_left, int32_t P,
                                                        uint32_t spare) {
    const int t = threadIdx.x, nt = blockDim.x;
    const int rlog = a.wlog - 4;
    const int n_lvl = a.NC << rlog;
    const int n_tab = (a.W * a.F * esize) >> 4;
    const int n_blk = a.blk_bytes >> 4;
    const uint32_t own = spare + 16u * static_cast<uint32_t>(t & 63);
    WinPlan<NL, NT, NB> p;
    p.has = 0u;
#pragma unroll
    for (int i = 0; i < NL + NT + NB; ++i) {
        bool ok = false;
        uint32_t src = 0u, d0 = 0u, stride = 0u;
        if (i < NL) {
            const int q = t + i * nt;
            const int r = q >> rlog, k = q - (r << rlog);
            const int rr = r < rows_left ? r : static_cast<int>(rows_left - 1);
            ok = q < n_lvl;
            src = static_cast<uint32_t>(rr) * static_cast<uint32_t>(P) + 16u * static_cast<uint32_t>(k);
            d0 = static_cast<uint32_t>(r) * a.L.lvl_pitch + 16u * static_cast<uint32_t>(k);
            stride = a.L.lvl_buf;
        } else if (i < NL + NT) {
            const int q = t + (i - NL) * nt;
            ok = q < n_tab;
            src = 16u * static_cast<uint32_t>(q);
            d0 = a.L.off_x + 16u * static_cast<uint32_t>(q);
            stride = a.L.tab_elems * static_cast<uint32_t>(esize);
        } else {
            const int q = t + (i - NL - NT) * nt;
            ok = q < n_blk;
            src = 16u * static_cast<uint32_t>(q);
            d0 = a.L.off_blk + 16u * static_cast<uint32_t>(q);
            stride = static_cast<uint32_t>(a.blk_bytes);
        }
        // an absent piece reads past its buffer's end (zeros, with no memory traffic)
        p.src[i] = ok ? src : (i < NL ? 0u : kWinNoStore);
        p.dst0[i] = ok ? d0 : own;
        p.dst1[i] = ok ? d0 + stride : own;
        p.has |= ok ? 1u << i : 0u;
    }
    return p;
}

// The per-workgroup buffers of a pass's planned copies: the workgroup's level rows, the pass's
// table (8-byte entries forward, 4-byte in the second pass) and the step blocks.
struct WinBufs {
    const uint8_t *lvl;
    __amdgpu_buffer_rsrc_t tab, blk;
    int32_t tab_win;   // table bytes per window: W * F * esize
};

// One window's copy in flight.
template <int N>
struct WinSet {
    uint4 v[N];
};

// The bytes by which the thread's level piece in slot i reaches past its row's end in the last
// window: the load is moved back by as many, so that it ends with the row (P >= 16), and the store
// drops its first bytes.
__device__ __forceinline__ int win_over(const WinArgs &a, uint32_t has, int i, int w, int32_t P) {
    const int q = (has >> i) & 1u ? static_cast<int>(threadIdx.x) + i * static_cast<int>(blockDim.x) : 0;
    const int end = (w << a.wlog) + 16 * (q & ((1 << (a.wlog - 4)) - 1)) + 16;
    return end > P ? end - P : 0;
}

typedef unsigned int emo_u4a1 __attribute__((ext_vector_type(4), aligned(1)));

// Issues the loads of window w from the plan.  RAG: the last window may reach past the rows.
template <bool RAG, int NL, int NT, int NB>
__device__ __forceinline__ void win_load(const WinArgs &a, const WinPlan<NL, NT, NB> &p, const WinBufs &b, int w,
                                         int nwin, int32_t P, WinSet<NL + NT + NB> &s) {
    // the window offsets are uniform; readfirstlane says so to the compiler (an offset it takes
    // for divergent becomes a loop over the distinct values around each load)
    const int so_lvl = __builtin_amdgcn_readfirstlane(w << a.wlog);
    const int so_tab = __builtin_amdgcn_readfirstlane(w * b.tab_win);
    const int so_blk = __builtin_amdgcn_readfirstlane(w * a.blk_bytes);
    const uint8_t *lbase = b.lvl + so_lvl;
    uint32_t back[NL];
#pragma unroll
    for (int i = 0; i < NL; ++i) back[i] = 0u;
    if (RAG && w == nwin - 1) {
#pragma unroll
        for (int i = 0; i < NL; ++i) back[i] = static_cast<uint32_t>(win_over(a, p.has, i, w, P));
    }
#pragma unroll
    for (int i = 0; i < NL + NT + NB; ++i) {
        emo_u4 v;
        if (i < NL) {
            // (RAG: the base is 256 bytes lower, so that the offset stays non-negative)
            const uint8_t *src = RAG ? lbase - 256 + (p.src[i] + 256u - back[i]) : lbase + p.src[i];
            if (RAG) v = *reinterpret_cast<const emo_u4a1 *>(src);
            else v = *reinterpret_cast<const emo_u4 *>(src);
        } else if (i < NL + NT) {
            v = __builtin_amdgcn_raw_buffer_load_b128(b.tab, p.src[i], so_tab, 0);
        } else {
            v = __builtin_amdgcn_raw_buffer_load_b128(b.blk, p.src[i], so_blk, 0);
        }
        s.v[i] = make_uint4(v.x, v.y, v.z, v.w);
    }
}

// v without its first n bytes, zeros behind (all zeros for n >= 16)
__device__ __forceinline__ uint4 drop_bytes(uint4 v, int n) {
    unsigned long long lo = static_cast<unsigned long long>(v.y) << 32 | v.x;
    unsigned long long hi = static_cast<unsigned long long>(v.w) << 32 | v.z;
    if (n >= 8) {
        lo = n >= 16 ? 0ull : hi;
        hi = 0ull;
        n = n >= 16 ? 0 : n - 8;
    }
    if (n > 0) {
        lo = lo >> (8 * n) | hi << (64 - 8 * n);
        hi >>= 8 * n;
    }
    return make_uint4(static_cast<uint32_t>(lo), static_cast<uint32_t>(lo >> 32), static_cast<uint32_t>(hi),
                      static_cast<uint32_t>(hi >> 32));
}

// Stores window w, loaded by win_load, at the plan's destinations `dst` (its dst0 or dst1), level
// bytes shifted left by SH (the scale of a table entry; 0: as they are).  In the forward pass
// (`badbits` given) a level piece with a byte >= F sets its slot's bit; the caller marks the rows at
// the end of the pass.  hib: the bits of a byte at or above F when F is a power of two (then one
// mask test), else 0.
template <bool RAG, int SH, int NL, int NT, int NB>
__device__ __forceinline__ void win_store(const WinArgs &a, const WinPlan<NL, NT, NB> &p, const uint32_t *dst,
                                          char *lds, int w, int nwin, int32_t P, uint32_t *badbits, uint32_t addf,
                                          uint32_t hib, const WinSet<NL + NT + NB> &s) {
    constexpr uint32_t keep = ((0xffu << SH) & 0xffu) * 0x01010101u;
#pragma unroll
    for (int i = 0; i < NL + NT + NB; ++i) {
        uint4 v = s.v[i];
        if (i < NL) {
            if (RAG && w == nwin - 1) v = drop_bytes(v, win_over(a, p.has, i, w, P));
            if (badbits) {
                const uint32_t b = hib ? (v.x | v.y | v.z | v.w) & hib
                                       : bad_levels(v.x, addf) | bad_levels(v.y, addf) | bad_levels(v.z, addf) |
                                             bad_levels(v.w, addf);
                *badbits |= b && (p.has >> i & 1u) ? 1u << i : 0u;
            }
            // level rows are 4-byte aligned (odd pitch in words)
            uint32_t *d = reinterpret_cast<uint32_t *>(lds + dst[i]);
            d[0] = (v.x << SH) & keep;
            d[1] = (v.y << SH) & keep;
            d[2] = (v.z << SH) & keep;
            d[3] = (v.w << SH) & keep;
        } else {
            *reinterpret_cast<uint4 *>(lds + dst[i]) = v;
        }
    }
}

// Marks the rows of the forward pass's level pieces that held a byte >= F (after the pass; the
// caller's barrier then makes bad[] complete).
template <int NL>
__device__ __forceinline__ void win_mark_bad(const WinArgs &a, uint32_t badbits, uint32_t *bad) {
#pragma unroll
    for (int i = 0; i < NL; ++i)
        if (badbits >> i & 1u)
            bad[(static_cast<int>(threadIdx.x) + i * static_cast<int>(blockDim.x)) >> (a.wlog - 4)] = 1u;
}

// The slack tile's flush, with each thread's (at most NF) 16-byte pieces at LDS and global offsets
// fixed for the whole kernel: a wave covers 4 candidates x 16 pieces when rows are long enough
// (conflict-free LDS reads with the odd row pitch), else whole rows.  Global offsets are bytes from
// the workgroup's first row at the window's first column (32-bit); slack rows are 4-byte aligned.
// Slack rows of a workgroup may span up to 4 GiB (128 levels on one or two chains take workgroups of
// 512 candidates: 4 GiB at 2^21 packs), so a store to drop goes past them: at win_no_slack, from which
// the byte offset of any window (below 4 P) leads neither into the rows nor past 2^32.
__host__ __device__ inline uint32_t win_no_slack(int32_t P) {
    return 0xffffffe0u - 4u * static_cast<uint32_t>(P);
}
template <int NF>
struct FlushPlan {
    uint32_t src[NF];   // LDS byte offset of the piece's first float
    uint32_t dst[NF];   // byte offset in the slack rows
    uint32_t nan;       // bit j: the piece's candidate has an invalid level (its slack row is NaN)
};

// (after the forward pass: tfin holds the makespans, NaN for a candidate with an invalid level)
template <int NF>
__device__ __forceinline__ FlushPlan<NF> flush_plan(const WinArgs &a, int64_t rows_left, int32_t P,
                                                    const float *tfin) {
    const int t = threadIdx.x, nt = blockDim.x;
    const int W = a.W, prlog = a.wlog - 2;
    const int n = a.NC << prlog;
    FlushPlan<NF> f;
    f.nan = 0u;
#pragma unroll
    for (int j = 0; j < NF; ++j) {
        const int q = t + j * nt;
        int r, kk;
        if (prlog >= 4) {
            const int jj = q & 63, blk = q >> 6, kblog = prlog - 4;
            const int rg = blk >> kblog, kb = blk & ((1 << kblog) - 1);
            r = rg * 4 + (jj >> 4);
            kk = kb * 16 + (jj & 15);
        } else {
            r = q >> prlog;
            kk = q & ((1 << prlog) - 1);
        }
        const bool ok = q < n && r < rows_left;
        f.src[j] = ok ? a.L.off_tile + 4u * static_cast<uint32_t>(r * (W + 1) + 4 * kk) : a.L.off_tile;
        f.dst[j] = ok ? 4u * (static_cast<uint32_t>(r) * static_cast<uint32_t>(P) + 4u * static_cast<uint32_t>(kk))
                      : win_no_slack(P);
        const float tr = tfin[ok ? r : 0];
        f.nan |= ok && tr != tr ? 1u << j : 0u;
    }
    return f;
}

// `rows`: the workgroup's slack rows (S from its first row, a range check at the batch's end);
// pieces a thread does not have and rows past the batch store at win_no_slack, which the range
// check drops, so no store needs a lane mask
template <int NF>
__device__ __forceinline__ void flush_window(const FlushPlan<NF> &f, __amdgpu_buffer_rsrc_t rows, const char *lds,
                                             int w, int wlog) {
    // (the window's offset is added to the lanes' offsets: with a scalar offset the compiler lets the
    // next instruction overwrite the third or fourth data register of a 16-byte store, and the store
    // was seen to write the new value; with none it keeps the wait state that such a store needs)
    const uint32_t so = static_cast<uint32_t>(w << wlog) * 4u;
#pragma unroll
    for (int j = 0; j < NF; ++j) {
        const float *src = reinterpret_cast<const float *>(lds + f.src[j]);
        float4 v = make_float4(src[0], src[1], src[2], src[3]);
        if ((f.nan >> j) & 1u) v = make_float4(__builtin_nanf(""), __builtin_nanf(""), __builtin_nanf(""),
                                               __builtin_nanf(""));
        const emo_u4 u = {__float_as_uint(v.x), __float_as_uint(v.y), __float_as_uint(v.z), __float_as_uint(v.w)};
        __builtin_amdgcn_raw_buffer_store_b128(u, rows, f.dst[j] + so, 0, 0);
    }
}

// The last window's flush when it reaches past the rows: a float a lane, consecutive lanes on
// consecutive columns.
__device__ __forceinline__ void flush_last(const WinArgs &a, __amdgpu_buffer_rsrc_t rows, const char *lds,
                                           const float *tfin, int w, int64_t rows_left, int32_t P) {
    const int W = a.W, cols = P - (w << a.wlog);
    const float *tile = reinterpret_cast<const float *>(lds + a.L.off_tile);
    for (int q = threadIdx.x; q < a.NC << a.wlog; q += blockDim.x) {
        const int r = q >> a.wlog, cc = q & (W - 1);
        const float v = tfin[r] != tfin[r] ? __builtin_nanf("") : tile[r * (W + 1) + cc];
        const uint32_t dst = r < rows_left && cc < cols
                                 ? 4u * (static_cast<uint32_t>(r) * static_cast<uint32_t>(P) +
                                         static_cast<uint32_t>((w << a.wlog) + cc))
                                 : win_no_slack(P);
        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), rows, dst, 0, 0);
    }
}

// The wave's step range [k0, k1) in the window's block (scalars).
__device__ __forceinline__ void win_range(const WinArgs &a, const char *lds, int buf, int ch, int &k0, int &k1) {
    const int32_t *hdr = reinterpret_cast<const int32_t *>(lds + a.L.off_blk + buf * a.blk_bytes);
    k0 = __builtin_amdgcn_readfirstlane(hdr[ch]);
    k1 = __builtin_amdgcn_readfirstlane(hdr[ch + 1]);
}

// Keeps the LDS reads issued before it from being moved down to their first use (the compiler
// would otherwise sink the next groups' reads and serialise the round trips again).
__device__ __forceinline__ void win_issue_point() { asm volatile("" ::: "memory"); }

// x of lane J of the lane's row of 16 lanes (every lane active)
template <int J>
__device__ __forceinline__ uint32_t row_bcast(uint32_t x) {
    return static_cast<uint32_t>(
        __builtin_amdgcn_update_dpp(0, static_cast<int>(x), 0x150 + J, 0xf, 0xf, true));
}

// Sixteen consecutive steps of the wave's chain, one per lane of every row of 16 lanes: the LDS
// address of the step's column in the first level row and of its table row, its start floor and its
// fixed duration.  A step's fields reach all lanes as the broadcast operand of the
// instruction that uses them, so a step costs no read of its record.
template <bool FIXED>
struct WinChunk {
    uint32_t col, tab, cst, dur;
};

// ESH: log2 of a table entry's bytes.
template <bool FIXED, int ESH>
__device__ __forceinline__ WinChunk<FIXED> win_chunk(const ChainWinStep *rs, int k, int kmax, uint32_t lvl_base,
                                                     uint32_t tab_base) {
    const int i = k + static_cast<int>(threadIdx.x & 15u);
    const ChainWinStep *r = rs + (i < kmax ? i : kmax);   // (kmax: the block's last no-op step)
    const uint2 v = *reinterpret_cast<const uint2 *>(r);
    WinChunk<FIXED> c;
    c.col = (v.x & 0xffffu) + lvl_base;
    c.tab = ((v.x >> 16) << ESH) + tab_base;
    c.cst = v.y;
    c.dur = FIXED ? __float_as_uint(r->dur) : 0u;
    return c;
}

// LDS by address: the sums above are whole addresses (with a pointer the compiler adds the base last,
// and the broadcast becomes an instruction of its own).
typedef float emo_f2 __attribute__((ext_vector_type(2)));
template <typename T>
__device__ __forceinline__ T lds_at(uint32_t at) {
    return *(const __attribute__((address_space(3))) T *)static_cast<uintptr_t>(at);
}

__device__ __forceinline__ void lds_put(uint32_t at, float x) {
    *(__attribute__((address_space(3))) float *)static_cast<uintptr_t>(at) = x;
}

// The level bytes of steps 4J .. 4J + 3 of a chunk (lrow: the lane's row offset) and their table
// entries.
template <int J, bool FIXED>
__device__ __forceinline__ void chunk_levels(const WinChunk<FIXED> &c, uint32_t lrow, uint32_t *lv) {
    lv[0] = lds_at<uint8_t>(row_bcast<4 * J>(c.col) + lrow);
    lv[1] = lds_at<uint8_t>(row_bcast<4 * J + 1>(c.col) + lrow);
    lv[2] = lds_at<uint8_t>(row_bcast<4 * J + 2>(c.col) + lrow);
    lv[3] = lds_at<uint8_t>(row_bcast<4 * J + 3>(c.col) + lrow);
}

// SH: what is left to scale a level by (0 when the staged bytes are scaled).
template <int J, int SH, typename E, bool FIXED>
__device__ __forceinline__ void chunk_table(const WinChunk<FIXED> &c, const uint32_t *lv, E *te) {
    te[0] = lds_at<E>(row_bcast<4 * J>(c.tab) + (lv[0] << SH));
    te[1] = lds_at<E>(row_bcast<4 * J + 1>(c.tab) + (lv[1] << SH));
    te[2] = lds_at<E>(row_bcast<4 * J + 2>(c.tab) + (lv[2] << SH));
    te[3] = lds_at<E>(row_bcast<4 * J + 3>(c.tab) + (lv[3] << SH));
}

// Walks the chain's steps k0 .. k1 - 1 (whole groups of four, padded with no-op steps) of a window:
// use(integral_constant<int, j>, chunk, entry) for step j of its chunk.  The next group's table
// entries and the level bytes of the group after it are in flight while a group is used; the groups
// past k1 that are read belong to other chains or are no-op steps, and are not used.
// after_chunk(c0): after 16 steps.
template <bool FIXED, int ESH, int SH, typename E, typename Use, typename After>
__device__ __forceinline__ void win_walk(const ChainWinStep *rs, int k0, int k1, int kmax,
                                         uint32_t lvl_base, uint32_t tab_base, uint32_t lrow, Use use, After after) {
    if (k0 >= k1) return;
    WinChunk<FIXED> c = win_chunk<FIXED, ESH>(rs, k0, kmax, lvl_base, tab_base);
    uint32_t l0[4], l1[4];
    E t0[4], t1[4];
    chunk_levels<0>(c, lrow, l0);
    chunk_levels<1>(c, lrow, l1);
    chunk_table<0, SH>(c, l0, t0);
    for (int k = k0;; k += 16) {
        const WinChunk<FIXED> n = win_chunk<FIXED, ESH>(rs, k + 16, kmax, lvl_base, tab_base);
#define EMO_USE4(J, T)                                     \
    win_issue_point();                                     \
    use(std::integral_constant<int, 4 * J>(), c, T[0]);     \
    use(std::integral_constant<int, 4 * J + 1>(), c, T[1]); \
    use(std::integral_constant<int, 4 * J + 2>(), c, T[2]); \
    use(std::integral_constant<int, 4 * J + 3>(), c, T[3])
        chunk_table<1, SH>(c, l1, t1);
        chunk_levels<2>(c, lrow, l0);
        EMO_USE4(0, t0);
        if (k + 4 >= k1) return;
        chunk_table<2, SH>(c, l0, t0);
        chunk_levels<3>(c, lrow, l1);
        EMO_USE4(1, t1);
        if (k + 8 >= k1) return;
        chunk_table<3, SH>(c, l1, t1);
        chunk_levels<0>(n, lrow, l0);
        EMO_USE4(2, t0);
        if (k + 12 >= k1) return;
        chunk_table<0, SH>(n, l0, t0);
        chunk_levels<1>(n, lrow, l1);
        EMO_USE4(3, t1);
        if (k + 16 >= k1) return;
        after(k - k0);
        c = n;
#undef EMO_USE4
    }
}

// Makespan and energy of stream-chain graphs, and with SLACK the slack of every pack.  Slack comes
// from a second forward pass instead of a backward one.  Along a chain with durations
// d_j and start floors cst_j, a step's only successor is the next step, so its latest finish is
// the makespan minus the durations after it; with Pre_i = d_1 + ... + d_i and Tot = Pre_n,
//   slack_i = LFT_i - EFT_i = (T - Tot) - (EFT_i - Pre_i),
// and D_i = EFT_i - Pre_i obeys D_i = max(D_{i-1}, cst_i - Pre_{i-1}), D_0 = 0, because
// EFT_i = max(EFT_{i-1}, cst_i) + d_i.  The forward pass also sums Tot per chain; the second pass
// walks the windows again, sums Pre in the same order, carries D and writes K - D (K = T - Tot)
// through the slack tile.  No finish time is checkpointed or recomputed backwards.  Pre stays
// below the chain's total time, so off the exact-sum grid its rounding is that of sums of that
// size, and every other value takes one rounding: slack agrees with the backward recurrence to
// rounding, and bit for bit when every time sum is exact (every time a multiple of one power of
// two u and every path below 2^24 u, so every sum and difference is exact in fp32 in any order).
//
// RAG: P is not a multiple of W (the last window reaches past the rows, and rows may start at any
// byte).  SCALED (F <= 32): level bytes are staged as byte offsets into a table row.  NL, NT, NB:
// 16-byte pieces of levels, forward table and step block a thread copies per window, DEPTH windows
// ahead.
//
// What bounds it: the second pass its memory pattern (16,384 candidates of 65,536 kernels: 1.07 ms for
// 1.07 GB read and 4.3 GB written in 1 KB pieces of 64 rows), the first pass latency and LDS.  A step used
// to read its 8-byte record from LDS in every lane (four of about ten LDS cycles a step) and to take
// nine instructions; with the records in the lanes of each row of 16 it takes six and no record read:
// first pass 680 -> 532 us (no slack), with slack 1,671 -> 1,600; and pack counts that are no multiple of
// the window, which took dword-wise copies and stores of one float a lane, take the same planned
// 16-byte accesses: 2,043 kernels on 6 streams, 100,003 candidates 979 -> 452 us, 4,097 on 9 streams
// 1,490 -> 670.
template <bool SLACK, bool FIXED, bool RAG, bool SCALED, int NL, int NT, int NB, int DEPTH>
__global__ void __launch_bounds__(kChainBlockThreads, DEPTH == 1 ? 6 : 4)
chains_windowed(DevGraph g, DevChains c, WinArgs a, const uint4 *__restrict__ blocks,
                const uint8_t *__restrict__ levels, int64_t B, float *__restrict__ To,
                float *__restrict__ Eo, float *__restrict__ S) {
    extern __shared__ float4 smem[];
    char *lds = reinterpret_cast<char *>(smem);
    const int t = threadIdx.x, nt = blockDim.x;
    const int wv = __builtin_amdgcn_readfirstlane(t >> 6);
    const int grp = wv / a.nc, ch = wv - grp * a.nc;
    const int lane = t & 63;
    const int cl = grp * 64 + lane;                               // candidate within the workgroup
    const int64_t base = static_cast<int64_t>(blockIdx.x) * a.NC;
    const int64_t gc = base + cl;
    const int W = a.W, F = a.F, nc = a.nc, nwin = c.nwin;
    const int32_t P = g.P;
    const WinLayout &L = a.L;
    const int64_t rows_left = B - base;
    uint8_t *lvl0 = reinterpret_cast<uint8_t *>(lds);             // [2][NC][W + 4] bytes
    uint32_t *bad = reinterpret_cast<uint32_t *>(lds + L.off_bad);
    float *tfin = reinterpret_cast<float *>(lds + L.off_tfin);
    float2 *tab2 = reinterpret_cast<float2 *>(lds + L.off_x);     // forward: [2][W + 1][F]
    float *tabt = reinterpret_cast<float *>(lds + L.off_x);       // second pass: [2][W + 1][F]
    const uint32_t addf = (0x80u - static_cast<uint32_t>(F)) * 0x01010101u;
    // the bits of a byte that is >= F when F is a power of two
    const uint32_t hib = (F & (F - 1)) == 0 ? (0xffu & ~static_cast<uint32_t>(F - 1)) * 0x01010101u : 0u;
    const uint32_t lds0 = static_cast<uint32_t>(
        reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) char *)lds));
    const uint32_t lrow = static_cast<uint32_t>(cl) * L.lvl_pitch;
    const int kmax = (a.blk_bytes >> 4) - (a.hdr_words >> 2) - 1;
    auto recs = [&](int buf) {
        return reinterpret_cast<const ChainWinStep *>(lds + L.off_blk + buf * a.blk_bytes + 4 * a.hdr_words);
    };
    auto window = [&](int w) { return w < nwin ? w : nwin - 1; };

    // ------------------------------------------------------------------ forward
    for (int i = t; i < a.NC; i += nt) {
        bad[i] = 0u;
        *reinterpret_cast<uint32_t *>(lvl0 + i * L.lvl_pitch + W) = 0u;
        *reinterpret_cast<uint32_t *>(lvl0 + L.lvl_buf + i * L.lvl_pitch + W) = 0u;
    }
    for (int i = t; i < F; i += nt) {
        tab2[W * F + i] = make_float2(0.f, 0.f);
        tab2[L.tab_elems + W * F + i] = make_float2(0.f, 0.f);
    }
    const uint32_t spare = L.total;                               // 1 KiB past the layout: spare slots
    uint32_t badbits = 0u;
    float f = 0.f, pre = 0.f;
    double ed = 0.0;
    WinBufs bf;
    bf.lvl = levels + base * P;
    bf.blk = win_rsrc(blocks, static_cast<uint32_t>(static_cast<int64_t>(nwin) * a.blk_bytes));
    {
        const WinPlan<NL, NT, NB> plan = win_plan<NL, NT, NB>(a, 8, rows_left, P, spare);
        // (the spare entries behind the table complete its last 16 bytes)
        bf.tab = win_rsrc(g.tab, static_cast<uint32_t>((static_cast<int64_t>(P) * F * 8 + 15) & ~int64_t{15}));
        bf.tab_win = W * F * 8;
        constexpr int kSh = SCALED ? 3 : 0;
        WinSet<NL + NT + NB> s0, s1;
        win_load<RAG>(a, plan, bf, 0, nwin, P, s0);
        if (DEPTH == 2) win_load<RAG>(a, plan, bf, window(1), nwin, P, s1);
        lds_barrier();
        win_store<RAG, kSh>(a, plan, plan.dst0, lds, 0, nwin, P, &badbits, addf, hib, s0);
        lds_barrier();
        // window w from buffer buf = w & 1; `ld` takes window w + 2, `cm` holds window w + 1
        auto forward_window = [&](int w, int buf, WinSet<NL + NT + NB> &ld, WinSet<NL + NT + NB> &cm) {
            win_load<RAG>(a, plan, bf, window(w + DEPTH), nwin, P, DEPTH == 2 ? ld : cm);
            int k0, k1;
            win_range(a, lds, buf, ch, k0, k1);
            float eb = 0.f;
            win_walk<FIXED, 3, 3 - kSh, emo_f2>(
                recs(buf), k0, k1, kmax, lds0 + buf * L.lvl_buf, lds0 + L.off_x + buf * L.tab_elems * 8u, lrow,
                [&](auto j, const WinChunk<FIXED> &ck, emo_f2 te) {
                    constexpr int J = decltype(j)::value;
                    f = fmax_nonneg(f, __uint_as_float(row_bcast<J>(ck.cst))) + te.x;
                    if (SLACK) pre += te.x;
                    if (FIXED) {
                        const float d = __uint_as_float(row_bcast<J>(ck.dur));
                        f += d;
                        if (SLACK) pre += d;
                    }
                    eb += te.y;
                },
                [&](int done) {   // fp32 energy blocks of at most 64 steps
                    if ((done & 48) == 48) {
                        ed += static_cast<double>(eb);
                        eb = 0.f;
                    }
                });
            ed += static_cast<double>(eb);
            // (after the last window: a copy of it into the idle buffer, which nothing reads)
            win_store<RAG, kSh>(a, plan, buf ? plan.dst0 : plan.dst1, lds, window(w + 1), nwin, P, &badbits, addf,
                                hib, cm);
            lds_barrier();
        };
        for (int w = 0; w < nwin; w += 2) {
            forward_window(w, 0, s0, DEPTH == 2 ? s1 : s0);
            if (w + 1 < nwin) forward_window(w + 1, 1, DEPTH == 2 ? s1 : s0, s0);
        }
    }
    win_mark_bad<NL>(a, badbits, bad);
    // chains' makespans and energies -> the candidate's (chain order)
    double *esum = reinterpret_cast<double *>(lds + L.off_x);
    float *tsum = reinterpret_cast<float *>(lds + L.off_x + 8 * 64 * kWinMaxWaves);
    esum[wv * 64 + lane] = ed;
    tsum[wv * 64 + lane] = f;
    lds_barrier();
    if (ch == 0) {
        float T = c.t_const;
        double e = 0.0;
        for (int j = 0; j < nc; ++j) {
            T = fmaxf(T, tsum[(grp * nc + j) * 64 + lane]);
            e += esum[(grp * nc + j) * 64 + lane];
        }
        float E = static_cast<float>(e + static_cast<double>(g.static_power) * static_cast<double>(T));
        if (bad[cl]) {
            T = __builtin_nanf("");
            E = __builtin_nanf("");
        }
        tfin[cl] = T;
        if (gc < B) {
            To[gc] = T;
            Eo[gc] = E;
        }
    }
    if constexpr (SLACK) {
        lds_barrier();
        // -------------------------------------------------------------- second forward pass
        // a candidate with an invalid level (K = NaN) gets its NaN row from the flush instead
        constexpr int NF = 4 * NL;   // float4 pieces of the tile are four times the level pieces
        const FlushPlan<NF> fp = flush_plan<NF>(a, rows_left, P, tfin);
        const int64_t nrows = rows_left < a.NC ? rows_left : a.NC;
        const __amdgpu_buffer_rsrc_t srows = win_rsrc(S + base * P, static_cast<uint32_t>(nrows * P * 4));
        const WinPlan<NL, 1, NB> plan = win_plan<NL, 1, NB>(a, 4, rows_left, P, spare);
        bf.tab = win_rsrc(g.tabt, static_cast<uint32_t>((static_cast<int64_t>(P) * F * 4 + 15) & ~int64_t{15}));
        bf.tab_win = W * F * 4;
        constexpr int kSh = SCALED ? 2 : 0;
        for (int i = t; i < F; i += nt) {
            tabt[W * F + i] = 0.f;
            tabt[L.tab_elems + W * F + i] = 0.f;
        }
        const float Kc = tfin[cl] - pre;
        const float K = Kc == Kc ? Kc : 0.f;
        float D = 0.f, Pr = 0.f;
        WinSet<NL + 1 + NB> s0, s1;
        win_load<RAG>(a, plan, bf, 0, nwin, P, s0);
        if (DEPTH == 2) win_load<RAG>(a, plan, bf, window(1), nwin, P, s1);
        win_store<RAG, kSh>(a, plan, plan.dst0, lds, 0, nwin, P, nullptr, addf, hib, s0);
        lds_barrier();
        const uint32_t trow = lds0 + L.off_tile + 4u * static_cast<uint32_t>(cl * (W + 1));
        auto scan_window = [&](int w, int buf, WinSet<NL + 1 + NB> &ld, WinSet<NL + 1 + NB> &cm) {
            win_load<RAG>(a, plan, bf, window(w + DEPTH), nwin, P, DEPTH == 2 ? ld : cm);
            int k0, k1;
            win_range(a, lds, buf, ch, k0, k1);
            const uint32_t lvl_base = lds0 + static_cast<uint32_t>(buf) * L.lvl_buf;
            // a chunk's column address times four, plus tr, is its slack's address
            const uint32_t tr = trow - 4u * lvl_base;
            win_walk<FIXED, 2, 2 - kSh, float>(
                recs(buf), k0, k1, kmax, lvl_base, lds0 + L.off_x + buf * L.tab_elems * 4u, lrow,
                [&](auto j, const WinChunk<FIXED> &ck, float tt) {
                    constexpr int J = decltype(j)::value;
                    D = fmaxf(D, __uint_as_float(row_bcast<J>(ck.cst)) - Pr);
                    Pr += tt;
                    if (FIXED) Pr += __uint_as_float(row_bcast<J>(ck.dur));
                    lds_put(row_bcast<J>(4u * ck.col) + tr, K - D);
                },
                [](int) {});
            win_store<RAG, kSh>(a, plan, buf ? plan.dst0 : plan.dst1, lds, window(w + 1), nwin, P, nullptr, addf, hib,
                                cm);
            lds_barrier();
            if (RAG && w == nwin - 1) flush_last(a, srows, lds, tfin, w, rows_left, P);
            else flush_window<NF>(fp, srows, lds, w, a.wlog);
            lds_barrier();
        };
        for (int w = 0; w < nwin; w += 2) {
            scan_window(w, 0, s0, DEPTH == 2 ? s1 : s0);
            if (w + 1 < nwin) scan_window(w + 1, 1, DEPTH == 2 ? s1 : s0, s0);
        }
    }
}

int64_t chain_grid(const DevChains &c, int64_t B) {
    return ((B << c.lane_log) + kChainBlockThreads - 1) / kChainBlockThreads;
}

}  // namespace

namespace {
// Whether the staged kernel applies, and whether slack goes through the chain-ordered scratch
// (staged kernel, P a multiple of 4).
bool staged_ok(const DevGraph &g, const DevChains &c) {
    return static_cast<size_t>(K) * c.lanes * g.F * sizeof(float2) <= static_cast<size_t>(kStageBytes);
}
size_t round256(size_t x) { return (x + 255) & ~static_cast<size_t>(255); }
}  // namespace

namespace {
// The slot counts the kernel is compiled for.
bool slots_compiled(const WinSlots &s) {
    return s.tab4 <= 1 && ((s.lvl == 1 && s.tab8 == 1 && s.blk <= 2) || (s.lvl == 1 && s.tab8 == 2 && s.blk == 1) ||
                           (s.lvl == 2 && s.tab8 == 1 && s.blk == 1));
}
}  // namespace

bool chain_window_fits(int32_t nc, int32_t F, int32_t W, int32_t blk_bytes, int32_t P, int32_t *groups) {
    if (nc < 1 || nc > kWinMaxWaves || F < 1 || F > 128 || W < 16 || W > 256 || blk_bytes % 16 != 0)
        return false;
    // (byte offsets into the table and the step blocks are 32-bit)
    if ((static_cast<int64_t>(P) + W - 1) / W * blk_bytes >= int64_t{1} << 31) return false;
    const int top = kWinMaxWaves / nc;
    const WinLayout L = win_layout(W, 64 * top, F, top * nc, blk_bytes);
    const WinSlots sl = win_slots(W, 64 * top, F, blk_bytes, 64 * top * nc);
    if (L.total > kWinLds || !slots_compiled(sl)) return false;
    // Rows that are not 16-byte aligned take one level piece per thread, so windows half as wide on some
    // chain counts.  Two pieces and the wider window measured both ways: 2,043 kernels on 6 streams 468 us
    // against 447 with one, 9,001 on 3 787 against 810 (273 against 263 without slack), but 8,301 on 7 498
    // against 571; no count of chains or packs separates these, so the narrower window stays.
    if (P % 16 != 0 && sl.lvl > 1) return false;
    // Groups of 64 candidates per workgroup.  Workgroups of one group leave the fewest waves waiting at
    // a barrier and the shortest last round: 2,043 kernels on 6 streams, 100,003 candidates 452 us with one
    // group, 499 with two; 3,001 on 2 streams 650, 684, and 775 with eight; but each copies the window's
    // table, so past 16 levels (a table row larger than two groups' level bytes) two share it: 5,000
    // kernels on 3 streams with 24 levels 796 and 730.  The copy has to fit the threads, and a
    // workgroup's slack rows have 32-bit byte offsets.
    int G = F <= 16 || top == 1 ? 1 : 2;
    while (G <= top && !slots_compiled(win_slots(W, 64 * G, F, blk_bytes, 64 * G * nc))) ++G;
    if (G > top || static_cast<int64_t>(64 * G) * P * 4 > static_cast<int64_t>(win_no_slack(P))) return false;
    *groups = G;
    return true;
}

bool chains_scan_ok(const DevChains &c, const uint8_t *levels, const float *slack) {
    return slack && chains_windowed_ok(c, levels, slack);
}

bool chains_scan_full_ok(const DevChains &c, const uint8_t *levels, const float *slack) {
    return c.full && chains_scan_ok(c, levels, slack);
}

bool chains_windowed_ok(const DevChains &c, const uint8_t *levels, const float *slack) {
    return c.win > 0 && reinterpret_cast<uintptr_t>(levels) % 16 == 0 &&
           reinterpret_cast<uintptr_t>(slack) % 16 == 0;
}

size_t chains_scratch_bytes(const DevGraph &g, const DevChains &c, const uint8_t *levels, int64_t B,
                            const float *slack_ptr) {
    const bool slack = slack_ptr != nullptr;
    // windowed layout: the makespan and energy when the caller does not take them
    if (chains_windowed_ok(c, levels, slack_ptr)) return 2 * round256(static_cast<size_t>(B) * sizeof(float));
    const size_t lanes = static_cast<size_t>(chain_grid(c, B)) * kChainBlockThreads;
    const size_t ck = slack ? round256(static_cast<size_t>(c.len / K) * lanes * sizeof(float)) : 0;
    const size_t tmp = slack && staged_ok(g, c) && g.P % 4 == 0
                           ? round256(static_cast<size_t>(B) * (static_cast<size_t>(c.len) << c.lane_log) * sizeof(float))
                           : 0;
    return ck + tmp + 2 * round256(static_cast<size_t>(B) * sizeof(float));
}

namespace {
struct WinLaunch {
    dim3 grid, block;
    size_t lds;
    hipStream_t stream;
    const uint8_t *levels;
    int64_t B;
    float *T, *E, *S;
};

template <bool SLACK, bool FIXED, bool RAG, bool SCALED, int NL, int NT, int NB, int DEPTH>
hipError_t launch_windowed_kernel(const WinLaunch &l, const DevGraph &g, const DevChains &c, const WinArgs &a) {
    const auto kernel = &chains_windowed<SLACK, FIXED, RAG, SCALED, NL, NT, NB, DEPTH>;
    // the dynamic LDS limit is raised once per device (the caller made the graph's device current)
    static std::atomic<uint64_t> done{0};
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    const uint64_t bit = dev < 64 ? uint64_t{1} << dev : 0;
    if (!bit || !(done.load(std::memory_order_acquire) & bit)) {
        e = hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                                static_cast<int>(kWinLds + kWinSpare));
        if (e != hipSuccess) return e;
        done.fetch_or(bit, std::memory_order_acq_rel);
    }
    hipLaunchKernelGGL(kernel, l.grid, l.block, l.lds, l.stream, g, c, a, c.blocks, l.levels, l.B, l.T, l.E, l.S);
    return hipGetLastError();
}

template <bool SLACK, bool FIXED, bool RAG, bool SCALED, int DEPTH>
hipError_t launch_windowed_slots(const WinSlots &sl, const WinLaunch &l, const DevGraph &g, const DevChains &c,
                                 const WinArgs &a) {
    if (sl.lvl == 2) return launch_windowed_kernel<SLACK, FIXED, RAG, SCALED, 2, 1, 1, DEPTH>(l, g, c, a);
    if (sl.tab8 == 2) return launch_windowed_kernel<SLACK, FIXED, RAG, SCALED, 1, 2, 1, DEPTH>(l, g, c, a);
    if (sl.blk == 2) return launch_windowed_kernel<SLACK, FIXED, RAG, SCALED, 1, 1, 2, DEPTH>(l, g, c, a);
    return launch_windowed_kernel<SLACK, FIXED, RAG, SCALED, 1, 1, 1, DEPTH>(l, g, c, a);
}

// Copies two windows ahead where the waves of one workgroup are all that a compute unit holds (more
// than 12 chains: two workgroups would be more than the 24 waves that 80 registers allow): 65,536
// kernels on 16 streams 1,600 us against 1,618 with one window ahead, 7,000 kernels (24 levels) 498
// against 520.  With fewer chains several workgroups cover for each other, and the registers of the
// second window cost one of them: 8,192 kernels on 12 streams 500 us two ahead, 416 one ahead, 4,097 on 9
// streams 758 and 670.  More than 32 levels and fixed nodes are one ahead everywhere, ahead of what they
// replaced (30,001 candidates with slack: 9,216 kernels of 40 levels on 12 streams 833 -> 686 us, 10,000 of
// 128 on 16 2,226 -> 2,007, 9 chains of 1,000 steps with fixed nodes 1,807 -> 768), 16 chains of 768 steps with
// fixed nodes as before (1,848 and 1,885).
template <bool SLACK, bool RAG>
hipError_t launch_windowed_depth(const WinSlots &sl, const WinLaunch &l, const DevGraph &g, const DevChains &c,
                                 const WinArgs &a) {
    if (g.F <= 32) {
        if (c.fixed) return launch_windowed_slots<SLACK, true, RAG, true, 1>(sl, l, g, c, a);
        return a.nc > 12 ? launch_windowed_slots<SLACK, false, RAG, true, 2>(sl, l, g, c, a)
                         : launch_windowed_slots<SLACK, false, RAG, true, 1>(sl, l, g, c, a);
    }
    return c.fixed ? launch_windowed_slots<SLACK, true, RAG, false, 1>(sl, l, g, c, a)
                   : launch_windowed_slots<SLACK, false, RAG, false, 1>(sl, l, g, c, a);
}

hipError_t launch_windowed(const DevGraph &g, const DevChains &c, const uint8_t *levels, int64_t B,
                           float *T, float *E, float *slack, const SelTargets &tg, void *scratch,
                           hipStream_t s) {
    const int G = c.groups;
    WinArgs a;
    a.W = c.win;
    a.wlog = 0;
    while ((1 << a.wlog) < a.W) ++a.wlog;
    a.nc = c.nc;
    a.NC = 64 * G;
    a.F = g.F;
    a.blk_bytes = c.blk_bytes;
    a.hdr_words = c.hdr_words;
    a.L = win_layout(a.W, a.NC, a.F, G * c.nc, c.blk_bytes);
    const WinSlots sl = win_slots(a.W, a.NC, a.F, a.blk_bytes, a.NC * c.nc);
    char *p = static_cast<char *>(scratch);
    const size_t vec = round256(static_cast<size_t>(B) * sizeof(float));
    WinLaunch l;
    l.T = T ? T : reinterpret_cast<float *>(p);
    l.E = E ? E : reinterpret_cast<float *>(p + vec);
    l.S = slack;
    l.levels = levels;
    l.B = B;
    l.grid = dim3(static_cast<unsigned>((B + a.NC - 1) / a.NC));
    l.block = dim3(static_cast<unsigned>(a.NC * c.nc));
    l.lds = a.L.total + kWinSpare;
    l.stream = s;
    const bool rag = g.P % a.W != 0;
    hipError_t e = slack ? (rag ? launch_windowed_depth<true, true>(sl, l, g, c, a)
                                : launch_windowed_depth<true, false>(sl, l, g, c, a))
                         : (rag ? launch_windowed_depth<false, true>(sl, l, g, c, a)
                                : launch_windowed_depth<false, false>(sl, l, g, c, a));
    if (e == hipSuccess && tg.n) e = launch_select_results(l.T, l.E, B, tg, s);
    return e;
}
}  // namespace

hipError_t launch_chains(const DevGraph &g, const DevChains &c, const uint8_t *levels, int64_t B,
                         float *T, float *E, float *slack, const SelTargets &tg, void *scratch,
                         hipStream_t s) {
    if (chains_windowed_ok(c, levels, slack)) return launch_windowed(g, c, levels, B, T, E, slack, tg, scratch, s);
    const int64_t grid = chain_grid(c, B);
    const int64_t pitch = grid * kChainBlockThreads;
    const bool st = staged_ok(g, c);
    const bool via_tmp = slack && st && g.P % 4 == 0;
    char *p = static_cast<char *>(scratch);
    float *ck = slack ? reinterpret_cast<float *>(p) : nullptr;
    if (slack) p += round256(static_cast<size_t>(c.len / K) * pitch * sizeof(float));
    const int64_t srow = static_cast<int64_t>(c.len) << c.lane_log;
    float *tmp = via_tmp ? reinterpret_cast<float *>(p) : nullptr;
    if (via_tmp) p += round256(static_cast<size_t>(B) * srow * sizeof(float));
    const size_t vec = round256(static_cast<size_t>(B) * sizeof(float));
    float *Ts = T ? T : reinterpret_cast<float *>(p);
    float *Es = E ? E : reinterpret_cast<float *>(p + vec);
    const dim3 gd(static_cast<unsigned>(grid)), bd(kChainBlockThreads);
    const size_t nslot = static_cast<size_t>(K) * c.lanes;
    const size_t dyn = st ? 2 * nslot * g.F * sizeof(float2) + 3 * nslot * sizeof(ChainStep) : 0;
    if (via_tmp) hipLaunchKernelGGL((chains_staged<true>), gd, bd, dyn, s, g, c, levels, B, Ts, Es, tmp, ck, pitch);
    else if (slack) hipLaunchKernelGGL((chains_kernel<true>), gd, bd, 0, s, g, c, levels, B, Ts, Es, slack, ck, pitch);
    else if (st) hipLaunchKernelGGL((chains_staged<false>), gd, bd, dyn, s, g, c, levels, B, Ts, Es, slack, ck, pitch);
    else hipLaunchKernelGGL((chains_kernel<false>), gd, bd, 0, s, g, c, levels, B, Ts, Es, slack, ck, pitch);
    hipError_t e = hipGetLastError();
    if (e == hipSuccess && via_tmp) {
        const int64_t n = B * (g.P / 4);
        hipLaunchKernelGGL(gather_slack, dim3(static_cast<unsigned>((n + kGatherThreads - 1) / kGatherThreads)),
                           dim3(kGatherThreads), 0, s, tmp, c.pos, B, g.P, srow, slack);
        e = hipGetLastError();
    }
    if (e == hipSuccess && tg.n) e = launch_select_results(Ts, Es, B, tg, s);
    return e;
}

}  // namespace emo
