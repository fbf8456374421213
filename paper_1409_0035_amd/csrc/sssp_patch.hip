// Weighted searches on graphs that can be cut into patches (roads, meshes,
// grids): a wave relaxes one patch for one sample in LDS.
//
// k_wsearch (sssp_weighted.hip) runs one workgroup per sample, a global atomic
// per relaxed arc: it is bound by the device's rate of scattered atomics
// (2048 x 2048 grid, 64 samples: 136 ms at 19 G atomics/s) or, on smaller
// graphs, by its chain of rounds (201 x 307 grid: 708 rounds of 6.3 us).  Where
// most arcs stay inside patches of 256 consecutive nodes (the upload grows the
// patches breadth-first and numbers the nodes by them), relaxing inside a patch
// needs neither: its distances are 1 KB of LDS, its inner arcs 32 registers a
// lane, a relaxation is one LDS minimum, and a wave needs no barrier.
//
// Measured (searches alone): 2048 x 2048 grid, 64 samples 136 -> 48 ms; 201 x
// 307 grid, 50 samples 4.44 -> 2.65 ms.  A round is bound by the latency of its
// pairs' chains (distances in, ten or so LDS passes, offers out).
//
// Rounds: a (patch, sample) pair waits with the least distance that a
// neighbouring patch has offered to one of its nodes.  A round has a bound for
// each sample; its waves take the samples of their patch that wait below it in
// turn: they read the distances at the far ends of the arcs into the patch, run
// the patch to its fixed point, write the improved distances (only the owner of
// a patch writes them) and, where one of them beats what a far end outside has,
// let that end's patch wait for the next round.  Every word has one writer a
// round (each neighbouring patch has a slot of its own to leave an offer in),
// so the rounds need no global atomics: offers by atomic minima into inboxes of
// the far ends took 20-80 us a pair, many of them falling into the same few
// lines.  A distance read while its owner writes it is old or new; if old, the
// owner sees that its new one beats ours and lets us wait again.  A sample's
// bound lies `step` past its least wait (16 bucket widths: the distance a front
// covers in about two patches): taking every waiting pair at once instead
// repeats 1.9 times the pairs and 3.5 times the relaxations on a grid.  Label
// correcting: the order of relaxations is free and the distances, once no pair
// waits, are the shortest ones.  A round is a launch, so no fences are needed
// inside; a launch that finds no work returns at once.
#include "internal.h"

#include <algorithm>

namespace ccg {

namespace {

constexpr int kPBlock = 256;
constexpr int kPWaves = kPBlock / 64;
constexpr uint32_t kInf = 0xFFFFFFFFu;
constexpr uint32_t kMaxDist = 0x7FFFFFFEu;
// Samples are dealt to groups, eight or a power of two more, and a group's
// blocks have block indices congruent mod their number: workgroups go to the
// eight XCDs in turn, so a sample's distances, offers and round state stay in
// one XCD's L2.
constexpr int kLgGroups = 3;
constexpr int kLook = 64;           // patches a block looks after
constexpr int64_t kPatchBlocks = 512; // fewer blocks than this leave CUs idle
constexpr int32_t kPatchTurn = 4;     // samples of a group that a block's waves take at once
constexpr int kExt = 4;             // outside arcs a lane has in flight
constexpr int kSelf = kPatchNb - 1; // the slot in which a patch passes on its own wait
constexpr uint32_t kNoWeight = 0xFFFFFFu;  // an empty slot: never improves its own node
constexpr uint32_t kPushLimit = kMaxDist - kNoWeight;  // an inner arc from here on might pass the limit

// One block per patch: the patch of every node.
__global__ void k_patch_of(const int32_t* __restrict__ pstart, int32_t* patch_of) {
    const int32_t a = pstart[blockIdx.x], b = pstart[blockIdx.x + 1];
    for (int32_t v = a + threadIdx.x; v < b; v += blockDim.x) patch_of[v] = blockIdx.x;
}

// One block per patch, a thread per node: the inner arcs into the node's
// slots (weight << 8 | local end), and the number of the others.  With ext set,
// those others in full instead, from eptr[p] on (end, weight, start within the
// patch, end's patch).  icount[q]: arcs of that kind into patch q (a node's
// inner arcs beyond its slots among them, as arcs from the patch to itself;
// *spilled counts those).
__global__ __launch_bounds__(kPatchNodes) void k_patch_arcs(const uint32_t* __restrict__ rp,
                                                            const int2* __restrict__ cw,
                                                            const int32_t* __restrict__ pstart,
                                                            const int32_t* __restrict__ patch_of, uint32_t* ell,
                                                            int32_t* count, int32_t* icount, int32_t* spilled,
                                                            const int32_t* __restrict__ eptr, uint4* ext) {
    __shared__ int32_t s_n, s_spilled;
    const int32_t p = blockIdx.x, j = threadIdx.x, ps = pstart[p], pe = pstart[p + 1], v = ps + j;
    if (j == 0) s_n = s_spilled = 0;
    __syncthreads();
    int slot = 0;
    if (v < pe) {
        for (uint32_t e = rp[v]; e < rp[v + 1]; e++) {
            const int2 x = cw[e];
            if (x.x == v) continue;  // a self-loop improves nothing
            if (x.x >= ps && x.x < pe && slot < kPatchSlots && (uint32_t)x.y < kNoWeight) {
                if (!ext) ell[((int64_t)p * kPatchSlots + slot) * kPatchNodes + j] = (uint32_t)x.y << 8 | (uint32_t)(x.x - ps);
                slot++;
            } else {
                const int32_t at = atomicAdd(&s_n, 1), q = patch_of[x.x];
                if (ext) ext[eptr[p] + at] = make_uint4((uint32_t)x.x, (uint32_t)x.y, (uint32_t)j, (uint32_t)q);
                else {
                    atomicAdd(&icount[q], 1);
                    if (q == p) atomicAdd(&s_spilled, 1);
                }
            }
        }
    }
    if (!ext) {
        for (; slot < kPatchSlots; slot++)
            ell[((int64_t)p * kPatchSlots + slot) * kPatchNodes + j] = kNoWeight << 8 | (uint32_t)j;
        __syncthreads();
        if (j == 0) {
            count[p] = s_n;
            if (s_spilled) atomicAdd(spilled, s_spilled);
        }
    }
}

// The same outside arcs by the patch they lead into: (start, weight, end within
// the patch, start's patch), from iptr[q] on; cursor counts up from zero.
__global__ void k_patch_into(const int32_t* __restrict__ pstart, const int32_t* __restrict__ eptr,
                             const uint4* __restrict__ ext, const int32_t* __restrict__ iptr, int32_t* cursor,
                             uint4* in) {
    const int32_t p = blockIdx.x;
    for (int32_t e = eptr[p] + threadIdx.x; e < eptr[p + 1]; e += blockDim.x) {
        const uint4 x = ext[e];
        const int32_t q = (int32_t)x.w;
        const int32_t at = atomicAdd(&cursor[q], 1);
        in[iptr[q] + at] = make_uint4((uint32_t)pstart[p] + x.z, x.y, x.x - (uint32_t)pstart[q], (uint32_t)p);
    }
}

// The patches that arcs lead from into patch q, kSelf places at most: each has
// a slot of its own in q's waits.  *bad: some patch has more.
__global__ __launch_bounds__(64) void k_patch_from(const int32_t* __restrict__ iptr, const uint4* __restrict__ in,
                                                   int32_t* from, int32_t* bad) {
    __shared__ int32_t s_nb[kPatchNb];
    const int32_t q = blockIdx.x, lane = threadIdx.x;
    if (lane < kPatchNb) s_nb[lane] = -1;
    __syncthreads();
    for (int32_t e = iptr[q] + lane; e < iptr[q + 1]; e += 64) {
        const int32_t p = (int32_t)in[e].w;
        int tries = 0;
        for (int place = p % kSelf; tries < kSelf; tries++, place = (place + 1) % kSelf) {
            const int32_t was = atomicCAS(&s_nb[place], -1, p);
            if (was == -1 || was == p) break;
        }
        if (tries == kSelf) *bad = 1;
    }
    __syncthreads();
    if (lane < kPatchNb) from[(int64_t)q * kPatchNb + lane] = s_nb[lane];
}

// The patches that arcs lead to from patch p (kPatchNb at most), with p's slot
// in each: to (patch << 8 | slot, -1: none); an outside arc keeps the place of
// its end's patch beside its start (start | place << 8).
__global__ __launch_bounds__(64) void k_patch_to(const int32_t* __restrict__ eptr, uint4* ext,
                                                 const int32_t* __restrict__ from, int64_t* to, int32_t* bad) {
    __shared__ int32_t s_nb[kPatchNb];
    const int32_t p = blockIdx.x, lane = threadIdx.x;
    if (lane < kPatchNb) s_nb[lane] = -1;
    __syncthreads();
    for (int32_t e = eptr[p] + lane; e < eptr[p + 1]; e += 64) {
        const int32_t q = (int32_t)ext[e].w;
        int place = q % kPatchNb, tries = 0;
        for (; tries < kPatchNb; tries++, place = (place + 1) % kPatchNb) {
            const int32_t was = atomicCAS(&s_nb[place], -1, q);
            if (was == -1 || was == q) break;
        }
        if (tries == kPatchNb) *bad = 1;
        else ext[e].z |= (uint32_t)place << 8;
    }
    __syncthreads();
    if (lane < kPatchNb) {
        const int32_t q = s_nb[lane];
        int64_t x = -1;
        if (q >= 0)
            for (int slot = 0; slot < kSelf; slot++)
                if (from[(int64_t)q * kPatchNb + slot] == p) x = (int64_t)q << 8 | slot;
        to[(int64_t)p * kPatchNb + lane] = x;
    }
}

// Whether the arcs into every patch are those out of it reversed (undirected
// graphs, unless a node has more inner arcs than slots): sums of a mix of
// (node within the patch, the other end, weight) over both lists.  *differ
// counts up.
__global__ __launch_bounds__(64) void k_patch_same(const int32_t* __restrict__ eptr, const uint4* __restrict__ ext,
                                                   const int32_t* __restrict__ iptr, const uint4* __restrict__ in,
                                                   int32_t* differ) {
    const int32_t p = blockIdx.x, lane = threadIdx.x;
    auto mix = [](const uint4& x) {
        uint64_t z = ((uint64_t)x.x << 32 | x.y) + (uint64_t)(x.z & 0xFF) * 0x9E3779B97F4A7C15ull;
        z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
        z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
        return z ^ (z >> 31);
    };
    uint64_t a = 0, b = 0;
    for (int32_t e = eptr[p] + lane; e < eptr[p + 1]; e += 64) a += mix(ext[e]);
    for (int32_t e = iptr[p] + lane; e < iptr[p + 1]; e += 64) b += mix(in[e]);
    if (wave_sum64((int64_t)(a - b)) != 0 && lane == 0) atomicAdd(differ, 1);
}

__global__ void k_patch_clear(int32_t* p, int64_t count) {
    for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < count; t += (int64_t)gridDim.x * blockDim.x)
        p[t] = 0;
}

struct Bufs {
    uint32_t* W;        // [kg][n] distances, written by the patch's own wave
    int32_t lg;         // log2 of the number of groups
    uint32_t* wait[2];  // [groups][npatch][gs][kPatchNb] offers, by round parity (kInf: none)
    uint8_t* flag[2];   // [groups][npatch] whether some sample of the pair's group waits
    uint32_t* low;      // [kPatchRounds + 1][kg] a sample's least wait, by round (kInf: its search is over)
    uint32_t* ovf;
};

__global__ void k_patch_init(Bufs B, int64_t pairs, int64_t waits, int64_t flags, int32_t kg, int32_t nrounds) {
    const int64_t t0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x, step = (int64_t)gridDim.x * blockDim.x;
    for (int64_t t = t0; t < pairs; t += step) B.W[t] = kInf;
    for (int64_t t = t0; t < waits; t += step) B.wait[0][t] = B.wait[1][t] = kInf;
    for (int64_t t = t0; t < flags; t += step) B.flag[0][t] = B.flag[1][t] = 0;
    for (int64_t t = t0; t < (int64_t)kg * (nrounds + 1); t += step) B.low[t] = t < kg ? 0 : kInf;
    if (t0 == 0) *B.ovf = 0;
}

// A sample's own patch waits at distance 0 in the slot kSelf.
__global__ void k_patch_seed(Bufs B, const int32_t* __restrict__ samples, int32_t kg, int32_t gs, int32_t npatch,
                             const int32_t* __restrict__ patch_of) {
    const int32_t s = (int32_t)(blockIdx.x * blockDim.x + threadIdx.x);
    if (s >= kg) return;
    const int64_t at = (int64_t)(s & ((1 << B.lg) - 1)) * npatch + patch_of[samples[s]];
    B.wait[0][(at * gs + (s >> B.lg)) * kPatchNb + kSelf] = 0;
    B.flag[0][at] = 1;
}

// One round.  A block looks after every nb-th patch (kLook at most) for one
// group of samples: the waiting pairs of the flagged ones are listed, and its
// waves take them in turn (a block per patch and group would be 131,000 blocks
// on the 2048 x 2048 grid, nearly all of which find nothing: 168 us a round
// against 140).
// SAME: the arcs into a patch are those out of it reversed, so one reading of
// their far ends serves both.
template <bool SAME>
__global__ __launch_bounds__(kPBlock) void k_patch_round(Bufs B, const int32_t* __restrict__ pstart, PatchDir A,
                                                         const int32_t* __restrict__ samples, int64_t n, int32_t kg,
                                                         int32_t npatch, int32_t gs, uint32_t step, int32_t r) {
    const int32_t lg = B.lg, b = (int32_t)blockIdx.x >> lg, g = (int32_t)blockIdx.x & ((1 << lg) - 1);
    const int32_t nb = (int32_t)gridDim.x >> lg;
    const int lane = lane_id(), wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    uint8_t* flags = B.flag[r & 1] + (int64_t)g * npatch;
    const int32_t look = b + lane * nb;  // this lane's patch
    const bool set = lane < kLook && look < npatch && flags[look] != 0;
    const uint64_t todo = __ballot(set);
    if (!todo) return;  // the same in every wave
    constexpr int Q = kPatchNodes / 64;
    __shared__ uint32_t s_tile[kPWaves][kPatchNodes], s_old[kPWaves][kPatchNodes];
    __shared__ uint32_t s_near[kPWaves][kPatchNb];  // the least offer to each neighbouring patch
    __shared__ uint16_t s_pair[kLook * 64];         // the pairs to take: place of the patch << 8 | sample of the group
    __shared__ uint8_t s_look[kLook];               // the flagged patches' places
    __shared__ int32_t s_count, s_next;
    uint32_t* nxt = B.wait[(r + 1) & 1];
    uint8_t* nflag = B.flag[(r + 1) & 1];
    // a sample's bound: `step` past its least wait
    const int32_t mine = (lane << lg) + g;  // this lane's sample
    uint32_t* nlow = B.low + (int64_t)(r + 1) * kg;
    uint32_t bound = 0, low_seen = 0;
    if (lane < gs && mine < kg) {
        bound = B.low[(int64_t)r * kg + mine];
        bound = bound > kInf - 1 - step ? kInf : bound + step;
        low_seen = nlow[mine];
    }
    if (threadIdx.x == 0) s_count = s_next = 0;
    if (wave == 0 && set) s_look[__popcll(todo & ((1ull << lane) - 1))] = (uint8_t)lane;
    __syncthreads();  // every wave has read the flags
    if (wave == 0 && set) flags[look] = 0;
    // each pair's least offer, a lane a slot: a wave takes two samples of a
    // flagged patch at a time, kAhead such steps in flight
    constexpr int kAhead = 4, kTwo = 64 / kPatchNb;
    const int32_t per = (gs + kTwo - 1) / kTwo, steps = __popcll(todo) * per;
    for (int32_t t0 = wave; t0 < steps; t0 += kPWaves * kAhead) {
        uint32_t x[kAhead];
        uint32_t* w[kAhead];
#pragma unroll
        for (int u = 0; u < kAhead; u++) {
            const int32_t t = min(t0 + u * kPWaves, steps - 1), l = t % per * kTwo + lane / kPatchNb;
            const int64_t pair0 = (int64_t)g * npatch + b + (int64_t)s_look[t / per] * nb;
            w[u] = B.wait[r & 1] + (pair0 * gs + min(l, gs - 1)) * kPatchNb + lane % kPatchNb;
            x[u] = *w[u];
        }
#pragma unroll
        for (int u = 0; u < kAhead; u++) {
            const int32_t t = t0 + u * kPWaves, l = t % per * kTwo + lane / kPatchNb;
            if (t >= steps) break;
            if (l >= gs) x[u] = kInf;
            if (x[u] != kInf) *w[u] = kInf;
#pragma unroll
            for (int off = 1; off < kPatchNb; off <<= 1) x[u] = min(x[u], (uint32_t)__shfl_xor((int)x[u], off));
            const uint32_t to = (uint32_t)__shfl((int)bound, min(l, 63));
            const uint32_t seen = (uint32_t)__shfl((int)low_seen, min(l, 63));
            if (lane % kPatchNb == 0 && x[u] != kInf) {
                const int32_t i = s_look[t / per];
                if (x[u] < to) {
                    s_pair[atomicAdd(&s_count, 1)] = (uint16_t)(i << 8 | l);
                } else {  // it stays: passed on
                    const int64_t pair0 = (int64_t)g * npatch + b + (int64_t)i * nb;
                    nxt[(pair0 * gs + l) * kPatchNb + kSelf] = x[u];
                    nflag[pair0] = 1;
                    if (x[u] < seen) atomicMin(&nlow[(l << lg) + g], x[u]);
                }
            }
        }
    }
    __syncthreads();
    const int32_t count = s_count;
    uint32_t arc[Q][kPatchSlots];
    uint32_t* tile = s_tile[wave];
    uint32_t* old = s_old[wave];
    uint32_t* near = s_near[wave];
    int32_t at_patch = -1, ps = 0, size = 0, e0 = 0, e1 = 0, i0 = 0, i1 = 0;
    int64_t to = -1;
    bool over = false;
    uint32_t top = 0;  // the largest distance that was pushed along inner arcs
    for (;;) {
        int32_t turn = 0;
        if (lane == 0) turn = atomicAdd(&s_next, 1);
        turn = readlane32(turn, 0);
        if (turn >= count) break;
        const int32_t pair = __builtin_amdgcn_readfirstlane(s_pair[turn]);
        const int32_t p = b + (pair >> 8) * nb, l = pair & 0xFF, s = (l << lg) + g;
        if (p != at_patch) {
            at_patch = p;
            ps = pstart[p];
            size = pstart[p + 1] - ps;
            e0 = A.eptr[p];
            e1 = A.eptr[p + 1];
            i0 = SAME ? e0 : A.iptr[p];
            i1 = SAME ? e1 : A.iptr[p + 1];
            to = lane < kPatchNb ? A.to[(int64_t)p * kPatchNb + lane] : -1;
#pragma unroll
            for (int c = 0; c < kPatchSlots; c++)
#pragma unroll
                for (int q = 0; q < Q; q++)
                    arc[q][c] = A.ell[((int64_t)p * kPatchSlots + c) * kPatchNodes + q * 64 + lane];
        }
        uint32_t* Wr = B.W + (int64_t)s * n;
        uint32_t w0[Q], last[Q];
#pragma unroll
        for (int q = 0; q < Q; q++) {
            const int32_t j = q * 64 + lane;
            w0[q] = j < size ? Wr[ps + j] : kInf;
        }
        // the arcs into the patch; the first 64 kExt of them and their far
        // ends' distances stay in registers for the offers (read again, the
        // 2048 x 2048 grid took 56 ms instead of 48)
        uint4 x[kExt];
        uint32_t far[kExt];
        const uint4* into = SAME ? A.ext : A.in;
#pragma unroll
        for (int u = 0; u < kExt; u++) {
            const int32_t at = i0 + u * 64 + lane;
            x[u] = into[at < i1 ? at : max(i1 - 1, 0)];
        }
#pragma unroll
        for (int u = 0; u < kExt; u++) far[u] = i0 + u * 64 + lane < i1 ? Wr[x[u].x] : kInf;
#pragma unroll
        for (int q = 0; q < Q; q++) {
            tile[q * 64 + lane] = old[q * 64 + lane] = last[q] = w0[q];
        }
        if (samples[s] >= ps && samples[s] < ps + size && lane == 0) tile[samples[s] - ps] = 0;
        __builtin_amdgcn_wave_barrier();
        auto pull = [&](const uint4& y, uint32_t d) {
            const uint64_t c = (uint64_t)d + y.y;
            if (c > kMaxDist) over = true;
            else (void)__hip_atomic_fetch_min(&tile[y.z & 0xFF], (uint32_t)c, __ATOMIC_RELAXED,
                                              __HIP_MEMORY_SCOPE_WORKGROUP);
        };
#pragma unroll
        for (int u = 0; u < kExt; u++)
            if (far[u] != kInf) pull(x[u], far[u]);
        for (int32_t e = i0 + 64 * kExt + lane; e < i1; e += 64) {
            const uint4 y = into[e];
            const uint32_t d = Wr[y.x];
            if (d != kInf) pull(y, d);
        }
        __builtin_amdgcn_wave_barrier();
        // to the fixed point: a node whose distance fell since it last pushed
        // pushes along its inner arcs (the wave's LDS operations are in order)
        for (;;) {
            uint32_t d[Q];
            uint64_t m[Q], all = 0;
#pragma unroll
            for (int q = 0; q < Q; q++)
                d[q] = __hip_atomic_load(&tile[q * 64 + lane], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
#pragma unroll
            for (int q = 0; q < Q; q++) {
                m[q] = __ballot(d[q] < last[q]);
                all |= m[q];
            }
            if (!all) break;
#pragma unroll
            for (int q = 0; q < Q; q++) {
                if (!m[q]) continue;
                if (d[q] < last[q]) {
                    last[q] = d[q];
                    top = max(top, d[q]);
                    const uint32_t from = min(d[q], kPushLimit);  // no sum here wraps
#pragma unroll
                    for (int c = 0; c < kPatchSlots; c++)
                        (void)__hip_atomic_fetch_min(&tile[arc[q][c] & 0xFF], from + (arc[q][c] >> 8),
                                                     __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                }
            }
        }
        bool better = false;
#pragma unroll
        for (int q = 0; q < Q; q++) {
            if (last[q] < w0[q]) {
                better = true;
                Wr[ps + q * 64 + lane] = last[q];
            }
        }
        if (!__ballot(better)) continue;
        if (lane < kPatchNb) near[lane] = kInf;
        __builtin_amdgcn_wave_barrier();
        // the improved nodes' arcs out of the patch that beat their far end
        auto offer = [&](const uint4& y, uint32_t have) {
            const uint32_t j = y.z & 0xFF, d = tile[j];
            if (d >= old[j]) return;
            const uint64_t c = (uint64_t)d + y.y;
            if (c > kMaxDist) over = true;
            else if (c < have) {
                (void)__hip_atomic_fetch_min(&near[y.z >> 8], (uint32_t)c, __ATOMIC_RELAXED,
                                             __HIP_MEMORY_SCOPE_WORKGROUP);
            }
        };
        if constexpr (SAME) {
#pragma unroll
            for (int u = 0; u < kExt; u++)
                if (i0 + u * 64 + lane < i1) offer(x[u], far[u]);
            for (int32_t e = e0 + 64 * kExt + lane; e < e1; e += 64) {
                const uint4 y = A.ext[e];
                offer(y, Wr[y.x]);
            }
        } else {
            for (int32_t e = e0 + lane; e < e1; e += 64) {
                const uint4 y = A.ext[e];
                offer(y, Wr[y.x]);
            }
        }
        __builtin_amdgcn_wave_barrier();
        const uint32_t least = lane < kPatchNb ? near[lane] : kInf;
        const uint32_t seen = (uint32_t)readlane32((int)low_seen, l);
        if (least != kInf) {
            const int64_t q = (int64_t)g * npatch + (to >> 8);
            nxt[(q * gs + l) * kPatchNb + (to & 0xFF)] = least;
            nflag[q] = 1;
            if (least < seen) atomicMin(&nlow[s], least);
        }
        __builtin_amdgcn_wave_barrier();
    }
    if (over || top > kPushLimit) *B.ovf = 1;
}

// The largest distance and whether a node was left unreached.
__global__ void k_patch_max(const uint32_t* __restrict__ W, int64_t count, uint32_t* out, int32_t* unreached) {
    __shared__ uint32_t bm[4];
    uint32_t m = 0;
    bool un = false;
    for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < count; t += (int64_t)gridDim.x * blockDim.x) {
        const uint32_t d = W[t];
        if (d == kInf) un = true;
        else m = max(m, d);
    }
    for (int off = 32; off > 0; off >>= 1) m = max(m, (uint32_t)__shfl_xor((int)m, off));
    if (lane_id() == 0) bm[threadIdx.x >> 6] = m;
    __syncthreads();
    if (threadIdx.x == 0) atomicMax(out, max(max(bm[0], bm[1]), max(bm[2], bm[3])));
    if (un) *unreached = 1;
}

__global__ void k_patch_zero(uint32_t* p) { p[threadIdx.x] = 0; }

// A captured estimate's searches end here: rounds left over mean that this
// search needed more than the captured ones (reported as a distance that no
// captured bound allows), overflow and unreached nodes go to the job's flags.
__global__ void k_patch_fold(const uint32_t* low, int32_t kg, const uint32_t* ovf, const uint32_t* mx, DevFlags* flags,
                             uint32_t* maxd_out) {
    bool more = false;
    for (int32_t t = threadIdx.x; t < kg; t += 64) more = more || low[t] != kInf;
    more = __ballot(more) != 0;
    if (threadIdx.x != 0) return;
    if (mx[1] && !more) flags->disconnected = 1;
    *maxd_out = (more || *ovf) ? kInf : mx[0];
}

inline size_t align256(size_t x) { return (x + 255) & ~size_t(255); }

// log2 of the number of groups: more than eight where that few blocks, one a
// patch and group, would leave the device idle while a block's waves take many
// samples in turn (us, k_wsearch / eight groups / this: 12 x 12 x 12 mesh, 8
// patches, 256 samples 725 / 978 / 601; 23 x 23 grid, 3 patches, 256 samples
// 625 / 632 / 468, 64 samples 510 / 424 / 382; 100 x 100 grid, 40 patches, 256
// samples 1851 / 1893 / 1516).  From 64 patches on more groups lose: 30 x 30 x
// 30 mesh, 107 patches, 64 samples 1362 with eight, 1773 with 16 -- a patch's
// tables are then read by two blocks.
int32_t lg_groups(int32_t npatch, int32_t kg) {
    int32_t lg = kLgGroups;
    while (lg < 6 && ((int64_t)npatch << lg) < kPatchBlocks && (kg >> lg) > kPatchTurn) lg++;
    return lg;
}

// samples of a group: sample s is the (s / groups)-th of group s % groups
int32_t group_size(int32_t kg, int32_t lg) { return (kg + (1 << lg) - 1) >> lg; }

size_t wait_count(int32_t npatch, int32_t kg) {
    const int32_t lg = lg_groups(npatch, kg);
    return ((size_t)npatch << lg) * group_size(kg, lg) * kPatchNb;
}

Bufs carve(void* scratch, int32_t kg, int32_t npatch, uint32_t* Dt, uint32_t** mx) {
    char* p = (char*)scratch;
    Bufs B;
    B.W = Dt;
    B.lg = lg_groups(npatch, kg);
    for (int i = 0; i < 2; i++) {
        B.wait[i] = (uint32_t*)p;
        p += align256(sizeof(uint32_t) * wait_count(npatch, kg));
        B.flag[i] = (uint8_t*)p;
        p += align256((size_t)npatch << B.lg);
    }
    B.low = (uint32_t*)p;
    p += align256(sizeof(uint32_t) * (size_t)kg * (kPatchRounds + 1));
    B.ovf = (uint32_t*)p;
    *mx = (uint32_t*)p + 1;  // the largest distance, whether a node was unreached
    return B;
}

void start(hipStream_t st, const Bufs& B, const PatchGraph& g, int64_t n, const int32_t* samples_dev, int32_t kg,
           int32_t nrounds) {
    const int64_t pairs = n * kg;
    hipLaunchKernelGGL(k_patch_init, dim3((unsigned)std::min<int64_t>((pairs + 255) / 256, 8192)), dim3(256), 0, st, B,
                       pairs, (int64_t)wait_count(g.npatch, kg), (int64_t)g.npatch << B.lg, kg, nrounds);
    hipLaunchKernelGGL(k_patch_seed, dim3((kg + 63) / 64), dim3(64), 0, st, B, samples_dev, kg, group_size(kg, B.lg),
                       g.npatch, g.patch_of);
}

void rounds(hipStream_t st, const Bufs& B, const PatchGraph& g, int dir, int64_t n, const int32_t* samples_dev,
            int32_t kg, uint32_t step, int32_t from, int32_t to) {
    // blocks of a group: 256 (2,048 in all) measured best, a block's waves then
    // passing improvements on within a round; never more than kLook patches a block
    const int32_t nb = std::max(std::min(g.npatch, 256), (g.npatch + kLook - 1) / kLook);
    const dim3 grid((unsigned)(nb << B.lg)), block(kPBlock);
    for (int32_t r = from; r < to; r++) {
        if (g.dir[dir].in)
            hipLaunchKernelGGL((k_patch_round<false>), grid, block, 0, st, B, g.pstart, g.dir[dir], samples_dev, n, kg,
                               g.npatch, group_size(kg, B.lg), step, r);
        else
            hipLaunchKernelGGL((k_patch_round<true>), grid, block, 0, st, B, g.pstart, g.dir[dir], samples_dev, n, kg,
                               g.npatch, group_size(kg, B.lg), step, r);
    }
}

void find_max(hipStream_t st, const Bufs& B, int64_t pairs, uint32_t* mx) {
    hipLaunchKernelGGL(k_patch_zero, dim3(1), dim3(2), 0, st, mx);
    hipLaunchKernelGGL(k_patch_max, dim3((unsigned)std::min<int64_t>((pairs + 255) / 256, 2048)), dim3(256), 0, st,
                       B.W, pairs, mx, (int32_t*)(mx + 1));
}

}  // namespace

size_t patch_scratch(int32_t kg, int32_t npatch) {
    return 2 * (align256(sizeof(uint32_t) * wait_count(npatch, kg)) + align256((size_t)npatch << lg_groups(npatch, kg))) +
           align256(sizeof(uint32_t) * (size_t)kg * (kPatchRounds + 1)) + 512 + 1024;
}

// The patches' arcs of one direction, from its rows: slots, the arcs that do
// not fit them (counted first), those by the patch they lead into, and the
// neighbouring patches.  `mem` gives device memory that the caller keeps (and
// frees, also what was taken when this fails).  False when the patches do not
// serve: too few arcs in slots, or a patch with too many neighbours.
bool build_patch_arcs(hipStream_t st, PatchGraph& g, int d, int64_t arcs, const uint32_t* rp, const int2* cw,
                      const PatchMemory& mem) {
    const size_t np = (size_t)g.npatch;
    const dim3 grid((unsigned)g.npatch);
    PatchDir A;
    uint32_t* ell = (uint32_t*)mem.take(sizeof(uint32_t) * np * kPatchSlots * kPatchNodes);
    int32_t* ptrs = (int32_t*)mem.take(sizeof(int32_t) * (3 * (np + 1) + 2));  // eptr, iptr, spilled, cursor, bad, differ
    int32_t *eptr = ptrs, *iptr = ptrs + np + 1, *spilled = iptr + np + 1, *cursor = spilled + 1;
    hipLaunchKernelGGL(k_patch_clear, dim3(256), dim3(256), 0, st, ptrs, (int64_t)(3 * (np + 1) + 2));
    hipLaunchKernelGGL(k_patch_arcs, grid, dim3(kPatchNodes), 0, st, rp, cw, g.pstart, g.patch_of, ell, eptr, iptr,
                       spilled, (const int32_t*)nullptr, (uint4*)nullptr);
    std::vector<int32_t> h(2 * (np + 1) + 1);
    CCG_HIP(hipMemcpyAsync(h.data(), ptrs, sizeof(int32_t) * h.size(), hipMemcpyDeviceToHost, st));
    CCG_HIP(hipStreamSynchronize(st));
    int64_t at = 0;
    for (int q = 0; q < 2; q++) {
        at = 0;
        for (size_t p = 0; p <= np; p++) {
            int32_t& c = h[(size_t)q * (np + 1) + p];
            const int32_t count = p < np ? c : 0;
            c = (int32_t)at;
            at += count;
        }
    }
    if (!patches_serve(arcs, arcs - at, h.back())) return false;
    CCG_HIP(hipMemcpyAsync(ptrs, h.data(), sizeof(int32_t) * h.size(), hipMemcpyHostToDevice, st));
    const size_t bytes = sizeof(uint4) * (size_t)std::max<int64_t>(at, 1);
    uint4 *ext = (uint4*)mem.take(bytes), *in = (uint4*)mem.take(bytes);
    int32_t* from = (int32_t*)mem.take(sizeof(int32_t) * np * kPatchNb);
    int64_t* to = (int64_t*)mem.take(sizeof(int64_t) * np * kPatchNb);
    hipLaunchKernelGGL(k_patch_arcs, grid, dim3(kPatchNodes), 0, st, rp, cw, g.pstart, g.patch_of, (uint32_t*)nullptr,
                       (int32_t*)nullptr, (int32_t*)nullptr, (int32_t*)nullptr, (const int32_t*)eptr, ext);
    hipLaunchKernelGGL(k_patch_into, grid, dim3(256), 0, st, g.pstart, (const int32_t*)eptr, (const uint4*)ext,
                       (const int32_t*)iptr, cursor, in);
    int32_t* bad = cursor + np;  // two counters, cleared, past the cursors
    hipLaunchKernelGGL(k_patch_from, grid, dim3(64), 0, st, (const int32_t*)iptr, (const uint4*)in, from, bad);
    hipLaunchKernelGGL(k_patch_to, grid, dim3(64), 0, st, (const int32_t*)eptr, ext, (const int32_t*)from, to, bad);
    hipLaunchKernelGGL(k_patch_same, grid, dim3(64), 0, st, (const int32_t*)eptr, (const uint4*)ext,
                       (const int32_t*)iptr, (const uint4*)in, bad + 1);
    CCG_HIP(hipGetLastError());
    int32_t hb[2];
    CCG_HIP(hipMemcpyAsync(hb, bad, sizeof(hb), hipMemcpyDeviceToHost, st));
    CCG_HIP(hipStreamSynchronize(st));
    if (hb[0]) return false;
    mem.drop(from, sizeof(int32_t) * np * kPatchNb);  // read by k_patch_to only
    if (!hb[1]) mem.drop(in, bytes);                  // ext serves both
    A.ell = ell;
    A.eptr = eptr;
    A.ext = ext;
    A.iptr = iptr;
    A.in = hb[1] ? in : nullptr;
    A.to = to;
    g.dir[d] = A;
    return true;
}

void build_patch_of(hipStream_t st, int32_t npatch, const int32_t* pstart, int32_t* patch_of) {
    hipLaunchKernelGGL(k_patch_of, dim3((unsigned)npatch), dim3(kPatchNodes), 0, st, pstart, patch_of);
}

// The searches of kg samples into Dt[j][v].  Returns 0 = done, 2 = unreached
// node, 4 = a distance too near the limit, 6 = more rounds than kPatchRounds
// (the caller then runs the general searches).  *hint: rounds to enqueue
// before the first look, set to the rounds that ran.
int sssp_patch(hipStream_t st, const PatchGraph& g, int dir, int64_t n, const int32_t* samples_dev, int32_t kg,
               uint32_t* Dt, uint32_t step, void* scratch, size_t scratch_size, int32_t* hint, int64_t* maxd,
               TravStats* stats) {
    if (scratch_size < patch_scratch(kg, g.npatch)) throw HipError{hipErrorOutOfMemory, "sssp_patch scratch"};
    uint32_t* mx = nullptr;
    const Bufs B = carve(scratch, kg, g.npatch, Dt, &mx);
    KernelTimer kt;
    start(st, B, g, n, samples_dev, kg, kPatchRounds);
    kt.start(st);
    int32_t done = 0, batch = std::max(*hint, 16);
    std::vector<uint32_t> more((size_t)kg);
    auto left = [&]() { return std::any_of(more.begin(), more.end(), [](uint32_t m) { return m != kInf; }); };
    while (done == 0 || (left() && done < kPatchRounds)) {
        const int32_t to = (int32_t)std::min<int64_t>((int64_t)done + batch, kPatchRounds);
        rounds(st, B, g, dir, n, samples_dev, kg, step, done, to);
        CCG_HIP(hipGetLastError());
        done = to;
        kt.stop(st);
        CCG_HIP(hipMemcpyAsync(more.data(), B.low + (size_t)done * kg, sizeof(uint32_t) * kg, hipMemcpyDeviceToHost, st));
        CCG_HIP(hipStreamSynchronize(st));
        batch = std::min(std::max(done / 2, 16), 512);
    }
    stats->kernel_ms += kt.ms();
    stats->kernel_launches += done;
    stats->launches += done + 4;
    if (left()) return 6;
    find_max(st, B, n * kg, mx);
    std::vector<uint32_t> lows((size_t)kg * (done + 1));
    uint32_t hm[3];  // overflow, largest distance, unreached
    CCG_HIP(hipMemcpyAsync(lows.data(), B.low, sizeof(uint32_t) * lows.size(), hipMemcpyDeviceToHost, st));
    CCG_HIP(hipMemcpyAsync(hm, B.ovf, sizeof(hm), hipMemcpyDeviceToHost, st));
    CCG_HIP(hipStreamSynchronize(st));
    int32_t ran = done;  // the first round that nothing waited for
    while (ran > 0 && std::all_of(lows.begin() + (size_t)(ran - 1) * kg, lows.begin() + (size_t)ran * kg,
                                  [](uint32_t m) { return m == kInf; }))
        ran--;
    *hint = ran;
    stats->levels += ran;
    stats->nodes_visited += n * kg;
    if (hm[0]) return 4;
    *maxd = std::max<int64_t>(*maxd, hm[1]);
    return hm[2] ? 2 : 0;
}

// The same launches without host reads (stream capture), exactly `count`
// rounds; *maxd_out becomes 2^32 - 1 when they were not enough.
void sssp_patch_enqueue(hipStream_t st, const PatchGraph& g, int dir, int64_t n, const int32_t* samples_dev, int32_t kg,
                        uint32_t* Dt, uint32_t step, void* scratch, size_t scratch_size, int32_t count,
                        DevFlags* flags, uint32_t* maxd_out) {
    if (scratch_size < patch_scratch(kg, g.npatch)) throw HipError{hipErrorOutOfMemory, "sssp_patch scratch"};
    uint32_t* mx = nullptr;
    const Bufs B = carve(scratch, kg, g.npatch, Dt, &mx);
    count = std::min<int32_t>(count, kPatchRounds);
    start(st, B, g, n, samples_dev, kg, count);
    rounds(st, B, g, dir, n, samples_dev, kg, step, 0, count);
    find_max(st, B, n * kg, mx);
    hipLaunchKernelGGL(k_patch_fold, dim3(1), dim3(64), 0, st, (const uint32_t*)(B.low + (size_t)count * kg), kg,
                       (const uint32_t*)B.ovf,
                       (const uint32_t*)mx, flags, maxd_out);
    CCG_HIP(hipGetLastError());
}

}  // namespace ccg
