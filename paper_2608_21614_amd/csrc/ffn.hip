// ffn.hip -- grouped SwiGLU expert FFN over the resident and shared experts
// (SAEM Section IV-D.2: resident experts on the matrix cores; Section IV-E.1:
// one batched execution per expert over its contiguous, repacked rows).
//
// Row space of the expert outputs: packed rows [0, T*k) (resident experts
// first, see repack.hip), then the rows of shared expert s at T*k + s*T + t.
//   phase 1: act[p, f] = silu(x[tok(p)] . W1[:,f]) * (x[tok(p)] . W3[:,f])
//   phase 2: y[c][p, h] = sum over K chunk c of act[p, :] . W2[:,h]
//
// Expert weights are in the MFMA tile layout (pack.hip): a 16-row x 32-column
// block is 1 KB of contiguous memory whose 64 16-byte pieces are the 64 lanes'
// MFMA A operands.
//
// Two kernel families:
//  * stream  (T <= 64, decode; bf16 MFMA 16x16x32, fp32 MFMA 16x16x4): the weights
//    are streamed from HBM exactly once.  A workgroup owns 32 features (phase 1: 32 gate + 32 up weight rows) or 64
//    outputs (phase 2: 64 rows of W2) of one expert; the weights are the MFMA
//    M side and the expert's tokens the N side, in tiles of 16.  Its four waves
//    split K interleaved -- wave w takes the 32-wide K steps w, w+4, w+8, ... --
//    so at any moment the workgroup reads 4 KB of contiguous memory per weight
//    tile; each wave double-buffers its loads in registers (the next two K
//    steps are in flight while the MFMAs of the current two run).  In the bf16
//    kernels a group whose rows fill one or two 16-row tiles runs a copy of the
//    K loop built for that many, whatever the kernel's tile count.  The waves'
//    partial tiles are summed through LDS in wave order.  Phase 2 also splits K
//    across workgroups into `ks` chunks whose partial sums the combine adds in
//    fixed order.  SwiGLU is applied in the phase-1 epilogue, so the gate and up
//    projections are never stored.
//    In the fused forward at decode, phase 1 also does the repacking: its
//    workgroups count the top-k ids themselves (the batch is at most 512 pairs)
//    and look their group's tokens up in them, one extra workgroup writes the
//    repack's outputs for phase 2 and the combine, and phase 2's trailing
//    workgroups pack the offloaded rows.  That saves the repack's launch and
//    its chain of dependent memory round trips before the weights start to flow.
//  * tiled   (T > 64, prefill; fp32 has a kernel of its own): output tiles of 128
//    weight rows x up to 256 (fp32: 128) rows of a group (four waves on MFMA 16x16x32), two persistent workgroups per CU that
//    claim items from a queue per XCD, both operands read as 1 KB tile-layout blocks by
//    direct global->LDS loads through a ring of stages; for bf16 a token gather first
//    copies the resident groups' rows into that layout, phase 1 writes the activations
//    in it, and the expert outputs are bf16.
// Both read counts and offsets from device memory: the stream kernel's grid is
// sized for the worst case on the host and surplus workgroups exit at once; the
// tiled kernel runs two workgroups per CU.
#include <algorithm>
#include <type_traits>

#include "block_ops.hpp"
#include "common.hpp"
#include "kernels.hpp"

namespace saem {
namespace {

constexpr int kTClaimPitch = 4;  // int32 words between two claim counters

struct Args {
    int T, H, E, F, k, S, Fs, slots;
    const void* x;
    const int32_t* perm;
    const int32_t* counts;
    const int32_t* seg_start;
    const int32_t* expert_slot;
    const void* w13;
    const void* w2;
    const void* ws13;
    const void* ws2;
    void* act;
    int Fa;
    float* y;
    int ks;
    long long y_ks_stride;
    int max_routed;   // routed groups the grid reserves (>= active resident experts)
    int ipg_r;        // items (workgroups) per routed group
    int ipg_s;        // items per shared group
    // offloaded-row pack done by the workgroups past the FFN items (phase 2 of the fused
    // decode path), or beside the tiled kernels' tables
    const float* topk_w;
    const int32_t* n_res;
    void* off_rows;
    float* off_w;
    void* xg;         // bf16 prefill: gathered token rows in the tile layout
    int32_t* tmeta;   // prefill: tables of the tiled kernels
    int tcap1;        // capacity of the phase-1 table
    int cus;          // prefill: CUs of the device
    int32_t* tclaim;  // prefill: claim counters of the tiled kernels, eight per phase
    uint16_t* y16;    // bf16 prefill: expert outputs [rows][H] in bf16; null: the same values in y
    // decode with the repacking in phase 1 (fused): the ids, and the repack's outputs
    int fused;
    int slot_items;   // fused phase 1: routed item gi is slot gi's expert (every slot can be active)
    const int32_t* topk_idx;
    int32_t* rp_counts;
    int32_t* rp_seg_start;
    int32_t* rp_perm;
    int32_t* rp_inv_perm;
    int32_t* rp_n_res;
};

// off_rows[p - n_res] = x[perm[p] / k] and off_w[p - n_res] = topk_w[perm[p]] for the
// offloaded rows p = n_res + wg, n_res + wg + nwg, ...
__device__ void pack_offloaded(const Args& a, int wg, int nwg, int elt) {
    const int P = a.T * a.k;
    const int nres = *a.n_res;
    const int chunks = a.H * elt / 16;  // 16-byte chunks of a row
    for (int p = nres + wg; p < P; p += nwg) {
        const int q = a.perm[p];
        if (q < 0 || q >= P) continue;
        const int t = q / a.k;
        if (a.off_rows) {
            const u32x4* src = reinterpret_cast<const u32x4*>(static_cast<const uint8_t*>(a.x) + (size_t)t * a.H * elt);
            u32x4* dst = reinterpret_cast<u32x4*>(static_cast<uint8_t*>(a.off_rows) + (size_t)(p - nres) * a.H * elt);
            for (int c = threadIdx.x; c < chunks; c += blockDim.x) dst[c] = src[c];
        }
        if (a.off_w && threadIdx.x == 0) a.off_w[p - nres] = a.topk_w[q];
    }
}

// One group of rows: a resident routed expert or a shared expert.
struct Group {
    int rowbase;   // first row in the row space
    int count;     // rows
    int routed;    // 1: rows are packed pairs (token = perm[p] / k); 0: row n is token n
    int Fg;        // expert width
    const uint8_t* w13;
    const uint8_t* w2;
};

// Active resident routed experts (ascending id) into s_list; returns their number.
// s_info[i]: expert s_list[i]'s (segment start, count, slot), read in the same round trip.
// Must be called by all threads of a 256-thread workgroup.
__device__ int list_active(const Args& a, int* s_list, int* s_wsum, int4* s_info) {
    const int tid = threadIdx.x, wave = tid >> 6, lane = lane_id();
    const int e = tid;
    bool act = false;
    int sl = -1, cnt = 0, seg = 0;
    if (e < a.E) {
        sl = a.expert_slot[e];
        cnt = a.counts[e];
        seg = a.seg_start[e];
        act = is_resident(sl, a.slots) && cnt > 0;
    }
    const unsigned long long b = __ballot(act);
    if (lane == 0) s_wsum[wave] = __popcll(b);
    __syncthreads();
    int base = 0;
    for (int w = 0; w < wave; ++w) base += s_wsum[w];
    if (act) {
        const int pos = base + __popcll(b & ((1ull << lane) - 1ull));
        s_list[pos] = e;
        s_info[pos] = make_int4(seg, cnt, sl, 0);
    }
    const int n = s_wsum[0] + s_wsum[1] + s_wsum[2] + s_wsum[3];
    __syncthreads();
    return n;
}

// list_active for a phase-1 workgroup of the fused decode path, where no repack has
// run yet: the counts come from the top-k ids (P = T k <= 512 pairs, two per thread,
// ids outside [0, E) dropped), and one wave scans them in group order -- resident
// experts by id, then offloaded ones -- into segment starts, as the repack does, and
// compacts the active resident experts in the same pass.  The list, counts and starts
// are the ones list_active reads after a repack.  *id0 / *id1: this thread's ids (pairs
// tid and tid + 256, -1 past P), for group_rows_from_ids.  s_scr: 513 ints of LDS.
// The three loads it needs are PrologueIds, which a caller may issue early.
struct PrologueIds {
    int q0, q1, slot;  // raw top-k ids of pairs tid, tid + 256; expert_slot[tid]
};
__device__ __forceinline__ PrologueIds load_prologue_ids(const Args& a) {
    const int tid = threadIdx.x, P = a.T * a.k;
    PrologueIds p;
    // no branch around the loads, so that a caller's later loads can stay in flight while
    // these are waited for
    const int sl = a.expert_slot[tid < a.E ? tid : 0];
    p.slot = tid < a.E ? sl : -1;
    p.q0 = a.topk_idx[tid < P ? tid : 0];
    p.q1 = a.topk_idx[tid + 256 < P ? tid + 256 : 0];
    return p;
}
__device__ int list_active_from_ids(const Args& a, const PrologueIds& ld, int* s_list, int4* s_info, int* s_scr,
                                    int* id0, int* id1) {
    int* s_cnt = s_scr;         // [256] pairs per expert
    int* s_slot = s_scr + 256;  // [256] slot of each expert (-1 past E)
    int* s_n = s_scr + 512;     // [1] active experts
    const int tid = threadIdx.x, wave = tid >> 6, lane = lane_id();
    const int P = a.T * a.k;
    s_cnt[tid] = 0;
    s_slot[tid] = ld.slot;
    const int q0 = ld.q0, q1 = ld.q1;
    *id0 = (tid < P && q0 >= 0 && q0 < a.E) ? q0 : -1;
    *id1 = (tid + 256 < P && q1 >= 0 && q1 < a.E) ? q1 : -1;
    __syncthreads();
    if (*id0 >= 0) atomicAdd(&s_cnt[*id0], 1);
    if (*id1 >= 0) atomicAdd(&s_cnt[*id1], 1);
    __syncthreads();
    if (wave == 0) {
        int cnt[4], sl[4];
        bool res[4];
        int rs = 0, os = 0, ac = 0;  // lane owns experts 4 lane .. 4 lane + 3
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int e = 4 * lane + i;
            cnt[i] = s_cnt[e];
            sl[i] = s_slot[e];
            res[i] = e < a.E && is_resident(sl[i], a.slots);
            if (res[i]) rs += cnt[i];
            else os += cnt[i];
            if (res[i] && cnt[i] > 0) ++ac;
        }
        int rinc = rs, oinc = os, ainc = ac;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const int x = __shfl_up(rinc, off, 64), y = __shfl_up(oinc, off, 64), z = __shfl_up(ainc, off, 64);
            if (lane >= off) {
                rinc += x;
                oinc += y;
                ainc += z;
            }
        }
        const int rtot = __shfl(rinc, 63, 64);
        int rp = rinc - rs, op = rtot + (oinc - os), pos = ainc - ac;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int e = 4 * lane + i;
            const int start = res[i] ? rp : op;
            if (res[i]) rp += cnt[i];
            else op += cnt[i];
            if (res[i] && cnt[i] > 0) {
                s_list[pos] = e;
                s_info[pos] = make_int4(start, cnt[i], sl[i], 0);
                ++pos;
            }
        }
        if (lane == 63) *s_n = ainc;
    }
    __syncthreads();
    return *s_n;
}

// The tokens of expert e's pairs in index order (its rows in the packed order), from the
// ids list_active_from_ids left in registers: s_tok[n] = token of row n.  s_w8: 8 ints.
__device__ void group_rows_from_ids(int e, int k, int id0, int id1, int* s_tok, int* s_w8) {
    const int tid = threadIdx.x, wave = tid >> 6, lane = lane_id();
    const unsigned long long m0 = __ballot(id0 == e), m1 = __ballot(id1 == e);
    if (lane == 0) {
        s_w8[wave] = __popcll(m0);
        s_w8[4 + wave] = __popcll(m1);
    }
    __syncthreads();
    int b0 = 0, b1 = 0;
    for (int w = 0; w < 4; ++w) {
        b1 += s_w8[w];
        if (w < wave) {
            b0 += s_w8[w];
            b1 += s_w8[4 + w];
        }
    }
    const unsigned long long lt = (1ull << lane) - 1ull;
    // an expert appears at most once per token, so a group holds at most T <= 64 rows
    const int r0 = b0 + __popcll(m0 & lt), r1 = b1 + __popcll(m1 & lt);
    if (id0 == e && r0 < 64) s_tok[r0] = tid / k;
    if (id1 == e && r1 < 64) s_tok[r1] = (tid + 256) / k;
    __syncthreads();
}

// Routed group from its expert's segment start, count and slot.
__device__ Group routed_group_of(const Args& a, int rb, int c, int slot_, size_t elt) {
    Group g;
    const int P = a.T * a.k;
    rb = rb < 0 ? 0 : (rb > P ? P : rb);
    c = c < 0 ? 0 : (c > P - rb ? P - rb : c);
    g.rowbase = rb;
    g.count = c;
    g.routed = 1;
    g.Fg = a.F;
    const size_t slot = (size_t)slot_;
    g.w13 = static_cast<const uint8_t*>(a.w13) + slot * 2 * a.F * a.H * elt;
    g.w2 = static_cast<const uint8_t*>(a.w2) + slot * a.H * a.F * elt;
    return g;
}

__device__ Group shared_group(const Args& a, int s, size_t elt) {
    Group g;
    g.rowbase = a.T * a.k + s * a.T;
    g.count = a.T;
    g.routed = 0;
    g.Fg = a.Fs;
    g.w13 = static_cast<const uint8_t*>(a.ws13) + (size_t)s * 2 * a.Fs * a.H * elt;
    g.w2 = static_cast<const uint8_t*>(a.ws2) + (size_t)s * a.H * a.Fs * elt;
    return g;
}

// Token of row n of a group, or -1 when out of range.
__device__ __forceinline__ int group_token(const Args& a, const Group& g, int n) {
    if (n >= g.count) return -1;
    int t;
    if (g.routed) {
        const int q = a.perm[g.rowbase + n];
        t = (q >= 0) ? q / a.k : -1;
    } else {
        t = n;
    }
    return (t >= 0 && t < a.T) ? t : -1;
}

constexpr int kGMaxGroups = 264;  // 256 routed + 8 shared

// s_out[g] = sum_{g' < g} f(g') for g < n (n <= kGMaxGroups), s_out[n] = the total,
// which is also returned; wave 0 scans, every thread of the workgroup must call.
// *s_tot must not be read by any thread between its previous use and this call.
template <typename Fn>
__device__ int group_prefix(int n, int* s_out, int* s_tot, Fn f) {
    if (threadIdx.x < 64) {
        const int lane = threadIdx.x;
        constexpr int PER = (kGMaxGroups + 63) / 64;
        int v[PER], sum = 0;
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const int gi = PER * lane + i;
            v[i] = gi < n ? f(gi) : 0;
            sum += v[i];
        }
        int inc = sum;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const int o = __shfl_up(inc, off, 64);
            if (lane >= off) inc += o;
        }
        int run = inc - sum;
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const int gi = PER * lane + i;
            if (gi < n) s_out[gi] = run;
            run += v[i];
        }
        if (lane == 63) {
            s_out[n] = inc;
            *s_tot = inc;
        }
    }
    __syncthreads();
    return *s_tot;
}

// ---------------------------------------------------------------------------
// stream kernel (decode)
// ---------------------------------------------------------------------------

// 16-row weight tiles per stream workgroup: two with a single token tile (twice
// the workgroups, for the small grids of the smallest batches), else four.
constexpr int stream_mt(int nt) { return nt == 1 ? 2 : 4; }

// kStreamW: the weights are loaded non-temporally (they do not stay in the
// caches for a later use), which raises the streaming rate when the call's
// weights are far larger than the caches; small weight sets that stay in the
// MALL between calls are read with plain loads.
// The bound of two workgroups per CU keeps every instance at two waves per SIMD: fp32
// operands double the fragment registers, and the one-tile copy of the K loop (below)
// adds registers to the wider bf16 instances; without the bound both would drop to one.
template <typename Elt, int NT, bool kDown, bool kStreamW>
__global__ void __launch_bounds__(256, 2) k_ffn_stream(Args a) {
    using F8 = Frag8<Elt>;
    constexpr int MT = stream_mt(NT);              // 16-row weight tiles per workgroup
    constexpr int MH = MT / 2;                     // phase 1: gate tiles (then as many up tiles)
    constexpr int U = sizeof(Elt) == 2 ? 2 : 1;    // K steps per load batch (two batches in flight)
    __shared__ int s_list[256];
    __shared__ int s_wsum[8];
    __shared__ int4 s_info[256];
    // the epilogue's partial tiles, or the repack's LDS in the fused path's repack
    // workgroup (which never reaches the epilogue).  The fused prologue's scratch has
    // its own arrays: a wave with no K steps of its own writes its partial tiles while
    // the other waves may still read the group's token rows.
    constexpr int kRedBytes = 4 * MT * NT * kWave * 16;
    constexpr int kRepackBytes = repack_lds_ints<256>() * 4;
    __shared__ __attribute__((aligned(16))) uint8_t s_raw[kRedBytes > kRepackBytes ? kRedBytes : kRepackBytes];
    auto& s_red = *reinterpret_cast<f32x4 (*)[4][MT][NT][kWave]>(s_raw);
    __shared__ int s_scr[513];  // fused prologue: pairs and slot per expert, active experts
    __shared__ int s_gtok[64];  // fused prologue: the group's token rows
    __shared__ int s_pos;  // slot-mapped items: the slot's place in the active list

    const int item = blockIdx.x;
    const int n_items = a.max_routed * a.ipg_r + a.S * a.ipg_s;
    if (item >= n_items) {
        if (a.fused && !kDown) {  // the fused path's repack: one workgroup, P <= 512
            if (item == n_items)
                repack_chunks<256>(a.T, a.E, a.k, a.slots, 0, (a.T * a.k + 255) / 256, a.topk_idx, a.expert_slot,
                                   a.rp_counts, a.rp_seg_start, a.rp_perm, a.rp_inv_perm, a.rp_n_res,
                                   reinterpret_cast<int*>(s_raw));
        } else if (a.fused) {  // trailing workgroups of phase 2 pack the offloaded rows
            pack_offloaded(a, item - n_items, gridDim.x - n_items, sizeof(Elt));
        }
        return;
    }
    const int wave = threadIdx.x >> 6, lane = lane_id();
    const int r = lane & 15, kq = (lane >> 4) * 8;

    // A shared expert's item needs no active list (its group is known), so it starts
    // streaming its weights without the prologue's dependent round trips.  So does a routed
    // item of the fused phase 1 when every slot can hold an active expert: item gi then
    // takes slot gi, whose weights are known at once, and issues its first weight batch
    // before the prologue finds the slot's expert, its rows and its tokens.
    const bool shared_item = item < a.S * a.ipg_s;
    const bool by_slot = a.fused && !kDown && a.slot_items && !shared_item;
    Group g;
    int sub = 0;
    int slot = -1;
    if (shared_item) {
        g = shared_group(a, item / a.ipg_s, sizeof(Elt));
        sub = item % a.ipg_s;
    } else if (by_slot) {
        const int i2 = item - a.S * a.ipg_s;
        slot = i2 / a.ipg_r;
        g = routed_group_of(a, 0, 0, slot, sizeof(Elt));  // rows set after the prologue
        sub = i2 % a.ipg_r;
        if (threadIdx.x == 0) s_pos = INT_MAX;  // read after the prologue's barriers
    }

    // weight tiles of this workgroup (16-row tiles in the tile layout) and the K chunk
    const Elt* wp[MT];
    int row0 = 0, kc = 0, c0 = 0, c1 = 0, n_my = 0, sbase = 0, nb = 0;
    auto setup_weights = [&]() {
        if (!kDown) {
            const int f0 = sub * 16 * MH;
            row0 = f0;
            const int nst = a.H / 32;
            const Elt* w = reinterpret_cast<const Elt*>(g.w13);
#pragma unroll
            for (int m = 0; m < MT; ++m) {
                const int rt = (m < MH ? 0 : g.Fg / 16) + f0 / 16 + m % MH;  // gate tiles, then up tiles
                wp[m] = w + (size_t)rt * nst * 512 + lane * 8;
            }
            c0 = 0;
            c1 = nst;
        } else {
            const int h0 = (sub / a.ks) * 16 * MT;
            kc = sub % a.ks;
            row0 = h0;
            const int nst = g.Fg / 32;
            const Elt* w = reinterpret_cast<const Elt*>(g.w2);
#pragma unroll
            for (int m = 0; m < MT; ++m) wp[m] = w + (size_t)(h0 / 16 + m) * nst * 512 + lane * 8;
            c0 = kc * nst / a.ks;
            c1 = (kc + 1) * nst / a.ks;
        }
        // this wave's K steps: c0 + wave + 4 i
        n_my = (c1 - c0 > wave) ? (c1 - c0 - wave + 3) / 4 : 0;
        sbase = c0 + wave;
        nb = n_my / U;
    };
    // batch b holds this wave's steps i = U*b .. U*b+U-1
    auto load_w = [&](F8 (&A)[U][MT], int b) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int s = sbase + 4 * (U * b + u);
#pragma unroll
            for (int m = 0; m < MT; ++m)
                A[u][m] = kStreamW ? load_frag_stream(wp[m] + (size_t)s * 512) : load_frag(wp[m] + (size_t)s * 512);
        }
    };
    F8 A0[U][MT], A1[U][MT];
    const bool early = shared_item || by_slot;  // weights known before the prologue
    int id0 = -1, id1 = -1, nact = 0;
    if (by_slot) {
        // the prologue's loads first, then the weights: loads complete in order, so the ids
        // can be used while the weight batch is still in flight.  No branch around the batch
        // (a K step past the wave's last reads its last one; the batch is used only if nb > 0)
        const PrologueIds ld = load_prologue_ids(a);
        setup_weights();
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int s = min(sbase + 4 * u, c1 - 1);
#pragma unroll
            for (int m = 0; m < MT; ++m)
                A0[u][m] = kStreamW ? load_frag_stream(wp[m] + (size_t)s * 512) : load_frag(wp[m] + (size_t)s * 512);
        }
        nact = list_active_from_ids(a, ld, s_list, s_info, s_scr, &id0, &id1);
    } else if (shared_item) {
        setup_weights();
        if (nb > 0) load_w(A0, 0);
    } else if (a.fused && !kDown) {
        nact = list_active_from_ids(a, load_prologue_ids(a), s_list, s_info, s_scr, &id0, &id1);
    } else {
        nact = list_active(a, s_list, s_wsum, s_info);
    }
    // shared groups first: their items can be longer (Fs > F in phase 2), so they
    // start in the first wave of workgroups instead of forming a tail
    if (by_slot) {
        // the slot's place in the active list (the lowest, should two experts share a slot)
        for (int p = threadIdx.x; p < nact; p += 256)
            if (s_info[p].z == slot) atomicMin(&s_pos, p);
        __syncthreads();
        const int pos = s_pos;
        if (pos == INT_MAX) return;  // no active expert holds the slot
        const int4 info = s_info[pos];
        g = routed_group_of(a, info.x, info.y, info.z, sizeof(Elt));
        group_rows_from_ids(s_list[pos], a.k, id0, id1, s_gtok, s_wsum);
    } else if (!shared_item) {
        const int i2 = item - a.S * a.ipg_s;
        const int gi = i2 / a.ipg_r;
        if (gi >= nact) return;
        const int4 info = s_info[gi];
        g = routed_group_of(a, info.x, info.y, info.z, sizeof(Elt));
        sub = i2 % a.ipg_r;
        // fused path: the group's token rows from the ids (no perm yet)
        if (a.fused && !kDown) group_rows_from_ids(s_list[gi], a.k, id0, id1, s_gtok, s_wsum);
    }
    if (g.count == 0) return;
    if (!early) {
        setup_weights();
        // the first batch's weights go out before the token rows are looked up
        if (nb > 0) load_w(A0, 0);
    }

    // token operand rows (N side)
    const int ntile = min(NT, (g.count + 15) / 16);
    const Elt* bp[NT];
#pragma unroll
    for (int j = 0; j < NT; ++j) {
        bp[j] = nullptr;
        const int n = 16 * j + r;
        if (!kDown) {
            const int t = (a.fused && g.routed) ? (n < g.count ? s_gtok[n] : -1) : group_token(a, g, n);
            if (t >= 0) bp[j] = static_cast<const Elt*>(a.x) + (size_t)t * a.H + kq;
        } else if (n < g.count) {
            bp[j] = static_cast<const Elt*>(a.act) + (size_t)(g.rowbase + n) * a.Fa + kq;
        }
    }

    // the K loop for NL token tiles; in the bf16 kernels a group that fills one or two
    // 16-token tiles runs a copy with that many, without the MFMAs of the tiles past its end
    // (separate copies, not a branch in the loop, so that their accumulators never live at
    // once).  fp32 keeps one loop.
    auto k_loop = [&](auto nl_tag) {
        constexpr int NL = decltype(nl_tag)::value;
        f32x4 acc[MT][NL];
#pragma unroll
        for (int m = 0; m < MT; ++m)
#pragma unroll
            for (int j = 0; j < NL; ++j) acc[m][j] = f32x4{0.f, 0.f, 0.f, 0.f};

        auto load_x = [&](F8 (&B)[U][NL], int b) {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int s = sbase + 4 * (U * b + u);
#pragma unroll
                for (int j = 0; j < NL; ++j) B[u][j] = (j < ntile && bp[j]) ? load_frag(bp[j] + s * 32) : zero_frag<Elt>();
            }
        };
        auto load = [&](F8 (&A)[U][MT], F8 (&B)[U][NL], int b) {
            load_w(A, b);
            load_x(B, b);
        };
        auto mma = [&](const F8 (&A)[U][MT], const F8 (&B)[U][NL]) {
            // tiles past the group's last token see zero operands: no branch, fewer live registers
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int j = 0; j < NL; ++j)
#pragma unroll
                    for (int m = 0; m < MT; ++m) acc[m][j] = mma_frag(A[u][m], B[u][j], acc[m][j]);
        };
        {
            F8 B0[U][NL], B1[U][NL];
            if (nb > 0) load_x(B0, 0);
            // (rolled: unrolling this loop, which the lambda otherwise invites, costs registers)
#pragma unroll 1
            for (int b = 0; b < nb; b += 2) {
                if (b + 1 < nb) load(A1, B1, b + 1);
                mma(A0, B0);
                if (b + 2 < nb) load(A0, B0, b + 2);
                if (b + 1 < nb) mma(A1, B1);
            }
        }
#pragma unroll 1
        for (int i = nb * U; i < n_my; ++i) {
            const int s = sbase + 4 * i;
            F8 A[MT], B[NL];
#pragma unroll
            for (int m = 0; m < MT; ++m)
                A[m] = kStreamW ? load_frag_stream(wp[m] + (size_t)s * 512) : load_frag(wp[m] + (size_t)s * 512);
#pragma unroll
            for (int j = 0; j < NL; ++j) B[j] = (j < ntile && bp[j]) ? load_frag(bp[j] + s * 32) : zero_frag<Elt>();
#pragma unroll
            for (int j = 0; j < NL; ++j)
#pragma unroll
                for (int m = 0; m < MT; ++m) acc[m][j] = mma_frag(A[m], B[j], acc[m][j]);
        }

#pragma unroll
        for (int m = 0; m < MT; ++m)
#pragma unroll
            for (int j = 0; j < NL; ++j) s_red[wave][m][j][lane] = acc[m][j];
    };
    if constexpr (sizeof(Elt) == 2 && NT > 1) {
        if (ntile == 1) k_loop(std::integral_constant<int, 1>{});
        else if (NT > 2 && ntile == 2) k_loop(std::integral_constant<int, 2>{});
        else k_loop(std::integral_constant<int, NT>{});
    } else {
        k_loop(std::integral_constant<int, NT>{});
    }
    __syncthreads();

    if (!kDown) {
        // pair gate tile m with up tile m + MH; lane l holds features 4*(l/16)..+3 of token l%16
        for (int task = threadIdx.x; task < MH * NT * kWave; task += 256) {
            const int m = task / (NT * kWave);
            const int j = (task / kWave) % NT;
            const int l = task % kWave;
            const int n = 16 * j + (l & 15);
            if (j >= ntile || n >= g.count) continue;
            f32x4 gv = s_red[0][m][j][l], uv = s_red[0][m + MH][j][l];
#pragma unroll
            for (int w = 1; w < 4; ++w) {
                gv += s_red[w][m][j][l];
                uv += s_red[w][m + MH][j][l];
            }
            const int f = row0 + 16 * m + 4 * (l >> 4);
            const f32x4 av = {silu(gv.x) * uv.x, silu(gv.y) * uv.y, silu(gv.z) * uv.z, silu(gv.w) * uv.w};
            Elt* dst = static_cast<Elt*>(a.act) + (size_t)(g.rowbase + n) * a.Fa + f;
            if constexpr (sizeof(Elt) == 2) {
                u32x2 packed;
                packed.x = pack_bf16x2(av.x, av.y);
                packed.y = pack_bf16x2(av.z, av.w);
                *reinterpret_cast<u32x2*>(dst) = packed;
            } else {
                *reinterpret_cast<f32x4*>(dst) = av;
            }
        }
    } else {
        for (int task = threadIdx.x; task < MT * NT * kWave; task += 256) {
            const int m = task / (NT * kWave);
            const int j = (task / kWave) % NT;
            const int l = task % kWave;
            const int n = 16 * j + (l & 15);
            if (j >= ntile || n >= g.count) continue;
            f32x4 v = s_red[0][m][j][l];
#pragma unroll
            for (int w = 1; w < 4; ++w) v += s_red[w][m][j][l];
            const int h = row0 + 16 * m + 4 * (l >> 4);
            float* dst = a.y + (long long)kc * a.y_ks_stride + (size_t)(g.rowbase + n) * a.H + h;
            *reinterpret_cast<f32x4*>(dst) = v;
        }
    }
}

// ---------------------------------------------------------------------------
// tiled kernel (prefill)
// ---------------------------------------------------------------------------
//
// One item = 128 weight rows (phase 1: 64 features, their gate and up rows; phase 2: 128
// rows of W2) x up to 256 of a group's rows.  Four waves in 2 (weight rows) x 2 (tokens);
// a wave holds 64 weight rows x every second 16-token block, so that a short item keeps
// all of them busy; a phase-1 wave holds the gate and the up rows of the same 32
// features, so SwiGLU runs in registers.  The tile runs at the number of token blocks
// that the item has, rounded up to a multiple of four (four copies of the K loop): loads,
// LDS reads and MFMAs for the rows past a group's end are left out.
//
// Operands: both are read as 1 KB blocks of the MFMA tile layout (16 rows x 32
// columns; lane l's 16 bytes are row l % 16, columns 8 (l / 16) .. + 7): the
// weights as they are stored, the tokens from a copy that the token gather
// (k_gather_tokens) makes of the resident groups' rows, and phase 2's from the
// activations, which phase 1 writes in that layout.  Gathered 64-byte pieces of
// row-major rows in their place filled the LDS at 14 TB/s against 19.
//
// K runs in 32-wide slabs through a ring of LDS stages filled by direct global->LDS
// loads: one wave instruction moves one 1 KB block, lane l's 16 bytes landing at byte
// 16 l, so every MFMA operand is one conflict-free 16-byte LDS read per lane.  The loads
// are inline assembly and waited for by count: a wave issues L per slab and no other
// vector-memory instruction in the K loop.  Fragments are double-buffered in registers:
// while slab kt's MFMAs issue, slab kt + 1's fragments are read and slab kt + S goes out
// over slab kt's stage, so a slab needs one barrier.
//
// What bounds it: on groups of many rows, the power limit -- the chip runs the K loop at
// 1.4 to 1.8 GHz -- and the L2; hence the 16x16x32 MFMA, which on random operands alone
// sustains 1.90 PFLOP/s against 1.65 for 32x32x16, and LDS reads and loads kept few.  On
// groups of few rows, the weight stream from HBM and the last round of items.  Two
// workgroups per CU let one's prologue and epilogue overlap the other's K loop; half the
// weight rows of a 256 x 256 tile halve the last round.  Before (256 x 256 tiles, eight
// waves on 32x32x16, one workgroup per CU) and now, phase 1 / phase 2 in us, bf16:
//   64 experts x 1024 rows, H 2048, F 1408:   680 / 384 -> 618 / 363
//   48 experts x  256 rows, H 2048, F 1408:   184 /  95 -> 161 /  91
//   48 experts x  100 rows, H 2048, F 1408:   158 /  82 -> 126 /  69
//   48 experts x   40 rows, H 2048, F 1408:   140 /  72 -> 106 /  66
//    8 experts x   83 rows, H 4096, F 14336:  386 / 284 -> 347 / 169
//   64 experts x   16 rows, H 2048, F 768:     93 /  50 ->  70 /  42
// (phase 2 storing bf16 rows).  A copy without the MFMAs takes 572 instead of 625 us in the first
// line and the same 107 in the fourth: the loads bound the kernel throughout.
// The weights of an item of up to 64 rows are loaded non-temporally (118 -> 108 us for
// phase 1 at 40 rows a group, 79 -> 72 at 16; phase 2 63 -> 66 and 51 -> 42): a group of so few
// rows reads them once.  (So does the short last tile of a longer group, whose other items read
// the same panel; it is one item in two at most.)  With more rows it gained nothing (128 -> 122
// and 69 -> 80 us at 100 rows).
//
// Registers: the widest copies fill the 256 of two waves per SIMD.  The compiler spills 4 (phase
// 1) and 7 (phase 2) vector registers to scratch, all outside the K loop, and 41 and 20 scalars to
// lanes of a vector register, of which the K loop reads back two to six per two slabs.
//
// The gathered rows, the activations and the expert outputs are stored non-temporally: the next
// launch reads them, from other XCDs, and here they would push the panels out of the L2
// (layer calls: 333 tokens x 8 wide experts 549 -> 540 us, 8192 tokens 1243 -> 1227).
//
// Items come from tables that the token gather writes.  Workgroups start on items
// 0, 1, ... and claim further ones from a counter per XCD (the hardware deals workgroups
// to the 8 XCDs round-robin), then from the other XCDs' once theirs is used up, so that
// items of unequal length even out.  An XCD takes chunks of kTChunk neighbouring items,
// which share weight and token panels in its L2.  Which workgroup runs an item does not
// change its result.  Up to one item per CU are dealt out evenly and without claims: in chunks
// of 32, 192 items left two XCDs idle and others with items to be claimed late (phase 1 /
// phase 2 in us; 4000 tokens, 16 experts, k 4, H 192, F 192: 23.6 / 26.5 -> 15.6 / 16.1; 5774
// tokens, 4 experts + 2 shared, H 128, F 64: 23.2 / 23.4 -> 14.6 / 15.0).  An XCD's run is
// then its share of neighbouring items; for fp32 eight items in turn, since a run that is one
// whole expert was slower there (16 experts of H 3072, F 1024, 43 rows each: 75 against 55 us).

constexpr int kTR = 128;           // weight rows per item
constexpr int kTF = kTR / 2;       // features per item in phase 1
constexpr int kTN = 256;           // group rows (tokens) per item
constexpr int kTB = 4;             // token tiles that consecutive items sweep together
constexpr int kTChunk = 32;        // consecutive items an XCD takes together
constexpr int kTLds = 80 * 1024;   // LDS of a workgroup: two workgroups per CU
constexpr int kTabWgs = 16;        // workgroups of the token gather that write the item tables

// Tables of the tiled kernels, written by the token gather into tmeta: int32 header[8]
// (items of phase 1, of phase 2), TileGroup[groups], then one TileItem per item of
// phase 1 and of phase 2.  All are read with scalar loads.
struct __attribute__((aligned(16))) TileGroup {
    int32_t wsel;     // slot of the routed expert (>= 0), or -(s + 1) for shared expert s
    int32_t count;    // rows of the group
    int32_t rowbase;  // first row of the group in the packed row space (y)
    int32_t blk;      // first row block of the group's activations
};
struct __attribute__((aligned(8))) TileItem {
    uint32_t wt;      // weight tile
    uint32_t gt;      // group | token tile << 9
};
constexpr int kTHeader = 8;
constexpr int kTPitch = 136;       // phase 2's staged token rows, in elements

typedef __attribute__((address_space(3))) uint8_t lds_u8;

// One direct global -> LDS load of 16 bytes per lane: lane l's bytes from base + voff land
// at LDS byte address lds + 16 l (lds and base are wave-uniform, lds passed through M0).
template <bool kNt>
__device__ __forceinline__ void lds_load_1k(uint32_t lds, const void* base, uint32_t voff) {
    if constexpr (kNt)
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 nt"
                     :
                     : "s"(lds), "v"(voff), "s"(base)
                     : "memory", "m0");
    else
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                     :
                     : "s"(lds), "v"(voff), "s"(base)
                     : "memory", "m0");
}

// Wait until at most N of this wave's vector-memory operations are outstanding and its LDS
// accesses are done, then a workgroup barrier.  The wait is the builtin, so that the
// compiler knows the LDS reads before it have landed and adds no waits of its own.
template <int N>
__device__ __forceinline__ void wait_then_barrier() {
    static_assert(N >= 0 && N < 64, "vmcnt is six bits");
    __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | ((N >> 4) << 14));
    asm volatile("s_barrier" : : : "memory");
}

// acc += A B (16 x 16 x 32), the accumulator tied in place.  Written out because the
// compiler, given the builtin, picks another register for the result than for the addend
// and fills the K loop with copies.  The caller keeps the waits that the compiler would
// add between an MFMA and other uses of its accumulator.
__device__ __forceinline__ void mfma_tied(f32x4& acc, bf16x8 a, bf16x8 b) {
    asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(acc) : "v"(a), "v"(b));
}

// Weight tiles of a group of width Fg: rows of W2 in phase 2, in phase 1 half as many features
// (their gate and up rows).
__host__ __device__ constexpr int weight_tiles(int H, int Fg, bool down, int rows = kTR) {
    return down ? (H + rows - 1) / rows : (Fg + rows / 2 - 1) / (rows / 2);
}

// Groups of the active list that the tables, the gathered rows and the activations have room
// for.  Only experts that share a slot, which the interface forbids but promises to survive,
// make the list longer; the ones past it are not run.
__device__ __forceinline__ int runnable(const Args& a, int nact) { return min(nact, a.max_routed); }

// The groups of the tiled kernels -- the S shared experts and the active resident routed
// ones, with their (segment start, count, slot) in s_info -- in order of falling row count,
// so that the long items start first: s_ord[o] = group, s_rows[group] = its rows (group gi:
// shared expert gi for gi < S, else entry gi - S of the active list).
__device__ void order_groups(const Args& a, int nact, const int4* s_info, int* s_rows, int16_t* s_ord) {
    const int ng = nact + a.S;
    const int P = a.T * a.k;
    for (int gi = threadIdx.x; gi < ng; gi += 256) {
        int rows = a.T;
        if (gi >= a.S) {
            const int4 inf = s_info[gi - a.S];
            rows = min(max(inf.y, 0), P - min(max(inf.x, 0), P));
        }
        s_rows[gi] = rows;
    }
    __syncthreads();
    for (int gi = threadIdx.x; gi < ng; gi += 256) {
        const int rows = s_rows[gi];
        int rank = 0;
        for (int o = 0; o < ng; ++o) {
            const int r = s_rows[o];
            rank += (r > rows || (r == rows && o < gi)) ? 1 : 0;
        }
        s_ord[rank] = (int16_t)gi;
    }
    __syncthreads();
}

// Writes the ordered groups' table and clears the claim counters.  s_bpre: the routed
// groups' row-block prefix (rb_routed blocks in all); without it (fp32) a group's
// activations are its rows in the row space.
__device__ void write_tile_groups(const Args& a, int ng, const int4* s_info, const int* s_rows, const int16_t* s_ord,
                                  const int* s_bpre, int rb_routed, TileGroup* groups) {
    const int P = a.T * a.k;
    if (threadIdx.x < 2 * 8) a.tclaim[threadIdx.x * kTClaimPitch] = 0;
    for (int o = threadIdx.x; o < ng; o += 256) {
        const int gi = s_ord[o];
        TileGroup g;
        g.count = s_rows[gi];
        if (gi < a.S) {
            g.wsel = -(gi + 1);
            g.rowbase = P + gi * a.T;
            g.blk = rb_routed + gi * ((a.T + 15) / 16);
        } else {
            const int4 inf = s_info[gi - a.S];
            g.wsel = inf.z;
            g.rowbase = min(max(inf.x, 0), P);
            g.blk = s_bpre ? s_bpre[gi - a.S] : 0;
        }
        groups[o] = g;
    }
}

// Item `local` of a group with nwt weight tiles and ntt token tiles: the items go through
// blocks of kTB token tiles, weight tile by weight tile, so that consecutive items share
// their weight and token panels.
__device__ __forceinline__ void item_tiles(int local, int nwt, int ntt, int* wt, int* tt) {
    const int tb = local / (nwt * kTB), rest = local - tb * nwt * kTB;
    const int width = min(kTB, ntt - tb * kTB);
    *wt = rest / width;
    *tt = tb * kTB + rest % width;
}

// Writes the item tables of both bf16 phases (workgroups part = 0 .. parts - 1 share the
// entries; part 0 also writes the groups and the item counts).
__device__ void write_tile_items(const Args& a, int nact, const int4* s_info, const int* s_bpre, int rb_routed,
                                 int* s_ipre, int* s_tot, int* s_rows, int16_t* s_ord, int part, int parts) {
    const int ng = nact + a.S;
    order_groups(a, nact, s_info, s_rows, s_ord);
    TileGroup* groups = reinterpret_cast<TileGroup*>(a.tmeta + kTHeader);
    if (part == 0) write_tile_groups(a, ng, s_info, s_rows, s_ord, s_bpre, rb_routed, groups);
    TileItem* tab = reinterpret_cast<TileItem*>(groups + a.max_routed + a.S);
    for (int ph = 0; ph < 2; ++ph) {
        const bool down = ph == 1;
        const int total = group_prefix(ng, s_ipre, s_tot + ph, [&](int o) {
            const int gi = s_ord[o];
            return weight_tiles(a.H, gi < a.S ? a.Fs : a.F, down) * ((s_rows[gi] + kTN - 1) / kTN);
        });
        TileItem* out = tab + (down ? a.tcap1 : 0);
        for (int i = part * 256 + threadIdx.x; i < total; i += parts * 256) {
            int lo = 0, hi = ng - 1;  // last group with s_ipre[g] <= i
            while (lo < hi) {
                const int mid = (lo + hi + 1) >> 1;
                if (s_ipre[mid] <= i) lo = mid;
                else hi = mid - 1;
            }
            const int gi = s_ord[lo];
            const int nwt = weight_tiles(a.H, gi < a.S ? a.Fs : a.F, down);
            const int ntt = (s_rows[gi] + kTN - 1) / kTN;
            const int local = i - s_ipre[lo];
            int wt, tt;
            item_tiles(local, nwt, ntt, &wt, &tt);
            TileItem it;
            it.wt = wt;
            it.gt = (uint32_t)lo | (uint32_t)tt << 9;
            out[i] = it;
        }
        if (part == 0 && threadIdx.x == 0) a.tmeta[ph] = total;
        __syncthreads();  // s_ipre is rewritten for the next phase
    }
}

// The bf16 prefill operands in the MFMA tile layout (16-row x 32-column blocks of
// 1 KB), so that every operand load of the tiled kernel is one contiguous 1 KB
// block.  Row-block space (16 rows per block):
//   xg: routed group gi (active list order) at blocks [bpre[gi], bpre[gi + 1]),
//       its rows in packed order, the rows past the group zero; then, when there
//       are shared experts, the batch's tokens in order at [RB, RB + ceil(T / 16)),
//       RB = bpre[nact];
//   act: the same for the routed groups; shared expert s at RB + s ceil(T / 16).
// Block (rb, c) of a buffer with K columns starts at element (rb K / 32 + c) 512.
// The first `parts` workgroups write the tiled kernels' item tables instead (a chain of its
// own, beside the copies); the workgroups past the row blocks pack the offloaded rows.
// A row block's columns are split over `split` workgroups, so that a short batch fills the
// CUs too.  A chain of memory round trips bounds short batches (150 tokens, 64 of 128
// experts: 13.8 us when the first copying workgroups wrote the tables, 9.2 now; 333
// tokens x 8 experts, H 4096: 17.5, 8.4), the copy's traffic long ones (8192 tokens: 268 MB
// written and as much read, 74 us).
__global__ void __launch_bounds__(256) k_gather_tokens(Args a, int parts, int blocks_max, int split) {
    __shared__ int s_list[256];
    __shared__ int4 s_info[256];
    __shared__ int s_wsum[8];
    __shared__ int s_bpre[257];
    __shared__ int s_ipre[kGMaxGroups + 1];
    __shared__ int s_rows[kGMaxGroups];
    __shared__ int16_t s_ord[kGMaxGroups];
    __shared__ int s_tok[16];
    const int wg = (int)blockIdx.x - parts;
    if (wg >= blocks_max * split) {
        pack_offloaded(a, wg - blocks_max * split, gridDim.x - parts - blocks_max * split, 2);
        return;
    }
    const int nact = runnable(a, list_active(a, s_list, s_wsum, s_info));
    const int rb_routed =
        group_prefix(nact, s_bpre, s_wsum + 4, [&](int gi) { return (max(s_info[gi].y, 0) + 15) / 16; });
    if (wg < 0) {
        write_tile_items(a, nact, s_info, s_bpre, rb_routed, s_ipre, s_wsum + 5, s_rows, s_ord, blockIdx.x, parts);
        return;
    }
    const int pid = wg / split, cs = wg % split;  // row block, column part
    if (threadIdx.x < 16) {
        const int r = threadIdx.x;
        int t = -1;
        if (pid < rb_routed) {
            int lo = 0, hi = nact - 1;
            while (lo < hi) {
                const int mid = (lo + hi + 1) >> 1;
                if (s_bpre[mid] <= pid) lo = mid;
                else hi = mid - 1;
            }
            const int4 inf = s_info[lo];
            const Group g = routed_group_of(a, inf.x, inf.y, inf.z, 2);
            t = group_token(a, g, 16 * (pid - s_bpre[lo]) + r);
        } else {
            const int n = 16 * (pid - rb_routed) + r;
            t = (a.S > 0 && n < a.T) ? n : -1;
        }
        s_tok[r] = t;
    }
    __syncthreads();
    if (pid >= rb_routed && (a.S == 0 || pid - rb_routed >= (a.T + 15) / 16)) return;
    // 16-byte piece j of block c: row j % 16, columns 32 c + 8 (j / 16) .. + 7; a batch's
    // loads all go out before its stores (one memory round trip per batch, not per piece)
    const int nc = a.H / 32;
    const int i0 = 64 * (int)((long long)nc * cs / split), i1 = 64 * (int)((long long)nc * (cs + 1) / split);
    const uint16_t* x = static_cast<const uint16_t*>(a.x);
    u32x4* dst = reinterpret_cast<u32x4*>(static_cast<uint16_t*>(a.xg) + (size_t)pid * nc * 512);
    constexpr int kBatch = 16;
    for (int base = i0; base < i1; base += 256 * kBatch) {
        u32x4 v[kBatch];
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
            const int idx = base + 256 * u + threadIdx.x;
            const int c = idx >> 6, j = idx & 63;
            const int t = idx < i1 ? s_tok[j & 15] : -1;
            v[u] = u32x4{0u, 0u, 0u, 0u};
            if (t >= 0) v[u] = *reinterpret_cast<const u32x4*>(x + (size_t)t * a.H + 32 * c + 8 * (j >> 4));
        }
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
            const int idx = base + 256 * u + threadIdx.x;
            if (idx < i1) __builtin_nontemporal_store(v[u], dst + idx);
        }
    }
}

// Item of the q-th claim on XCD x's queue: the XCDs take chunks of kTChunk items in turn.
__device__ __forceinline__ int claimed_item(int q, int x) {
    return ((q / kTChunk) * 8 + x) * kTChunk + q % kTChunk;
}

// At most one item per CU: no claims.  The q-th workgroup of XCD x takes this item; the XCDs get
// equal runs of neighbouring items (run: their length), or with run 0 eight items in turn.
__device__ __forceinline__ int few_item(int q, int x, int run) {
    return run == 0 ? ((q / 8) * 8 + x) * 8 + q % 8 : (q < run ? x * run + q : INT_MAX);
}

// The next item of XCD queue *xcd, or of another queue (then *xcd) once that one is empty;
// -1 when all are.  By one wave; the counters only grow, so the loop ends.
__device__ int next_item(int32_t* claim, int q0, int n_items, int* xcd) {
    const int lane = lane_id();
    for (;;) {
        const int x = (*xcd + (lane & 7)) & 7;
        const int q = __hip_atomic_load(claim + x * kTClaimPitch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const unsigned long long some = __ballot(lane < 8 && claimed_item(q0 + q, x) < n_items);
        if (!some) return -1;
        *xcd = (*xcd + __ffsll((long long)some) - 1) & 7;
        int got = 0;
        if (lane == 0)
            got = __hip_atomic_fetch_add(claim + *xcd * kTClaimPitch, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const int it = claimed_item(q0 + __builtin_amdgcn_readfirstlane(got), *xcd);
        if (it < n_items) return it;
    }
}

// A persistent kernel, two workgroups per CU.  tab, groups: this phase's tables, passed on
// their own and restrict-qualified, so that the compiler knows the kernel's stores leave
// them alone and reads them through scalar loads.  claim: eight counters, one per XCD.
template <bool kDown>
__global__ void __launch_bounds__(256, 2)
    k_ffn_tiled(Args a, const TileItem* __restrict__ tab, const TileGroup* __restrict__ groups, int32_t* claim) {
    __shared__ __attribute__((aligned(1024))) uint8_t sbuf[kTLds];
    int32_t* s_next = reinterpret_cast<int32_t*>(sbuf + kTLds - 16);  // free once the K loop is done

    const int tid = threadIdx.x, lane = lane_id();
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave & 1, wn = wave >> 1;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_u8*)sbuf;
    const uint32_t off0 = 16 * lane;  // this lane's 16 bytes of a 1 KB block
    const int n_items = a.tmeta[kDown ? 1 : 0];
    const int q0 = gridDim.x / 8;  // claims up to here are the workgroups' first items
    int xcd = blockIdx.x % 8;
    const bool few = n_items <= a.cus;
    int item = few ? few_item(blockIdx.x / 8, xcd, (n_items + 7) / 8) : claimed_item(blockIdx.x / 8, xcd);
    if (few && item >= n_items) return;

    if (item >= n_items) {
        if (wave == 0) {
            const int it = next_item(claim, q0, n_items, &xcd);
            if (lane == 0) *s_next = it;
        }
        __syncthreads();
        item = __builtin_amdgcn_readfirstlane(*s_next);
        __syncthreads();
    }

    while (item >= 0) {
        const TileItem ti = tab[item];
        const TileGroup tg = groups[ti.gt & 511];
        const int n0 = (int)(ti.gt >> 9) * kTN;  // first group row of the item
        const bool shared = tg.wsel < 0;
        const int Fg = shared ? a.Fs : a.F;
        const int K = kDown ? Fg : a.H;
        const int nk = K / 32;  // slabs (even: H and the widths are multiples of 64)
        // phase 1: features r0 .. r0 + 63 (gate rows in LDS blocks 0..3, up rows in 4..7);
        // phase 2: rows r0 .. r0 + 127 of W2
        const int r0 = (int)ti.wt * (kDown ? kTR : kTF);
        const size_t wsize = (size_t)(kDown ? 1 : 2) * Fg * a.H;  // elements of one expert's matrix
        const uint16_t* wbase = shared ? static_cast<const uint16_t*>(kDown ? a.ws2 : a.ws13) + (size_t)(-tg.wsel - 1) * wsize
                                       : static_cast<const uint16_t*>(kDown ? a.w2 : a.w13) + (size_t)tg.wsel * wsize;
        // this wave's weight blocks: wave and 4 + wave.  A row tile past the matrix (H not a
        // multiple of 128) reads tile 0 instead: its rows are never stored
        const uint16_t* gw[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            int rt;
            if (kDown) {
                rt = r0 / 16 + 4 * i + wave;
                if (16 * rt >= a.H) rt = 0;
            } else {
                rt = i * (Fg / 16) + r0 / 16 + wave;
            }
            gw[i] = wbase + (size_t)rt * nk * 512;
        }
        // first block of the group's token operand, and the elements of one row block
        const int kx = kDown ? a.Fa : a.H;
        const int xblk = (!kDown && shared) ? tg.blk - (-tg.wsel - 1) * ((a.T + 15) / 16) : tg.blk;
        const uint16_t* xbase = static_cast<const uint16_t*>(kDown ? a.act : a.xg) + (size_t)xblk * (kx / 32) * 512;
        const int nblk = min(kTN / 16, (tg.count - n0 + 15) / 16);  // token blocks of the item

        // the item with its tokens in NB blocks (4, 8, 12 or 16)
        auto run = [&](auto nb_tag) {
            constexpr int NB = decltype(nb_tag)::value;
            constexpr int NF = NB / 2;            // token fragments of a wave: blocks 2 n + wn
            constexpr int L = (8 + NB) / 4;       // loads of a wave per slab
            constexpr int kSlab = (8 + NB) * 1024;
            constexpr int S = NB == 4 ? 6 : kTLds / kSlab;  // stages of the ring
            static_assert(S * kSlab <= kTLds && (S - 1) * L < 64, "ring");
            constexpr bool kNtW = NB == 4;        // weights loaded non-temporally
            uint32_t off = off0;  // opaque: its uses' sums are made here, not kept across the items
            asm volatile("" : "+v"(off));
            // a token block past the group reads the group's first block instead (never stored)
            const uint16_t* gx[NB / 4];
#pragma unroll
            for (int i = 0; i < NB / 4; ++i) {
                const int tb = 4 * i + wave;
                gx[i] = xbase + (size_t)(tb < nblk ? n0 / 16 + tb : 0) * (kx / 32) * 512;
            }
            auto load = [&](int i, int kt, int stage) {
                const uint32_t to = lds0 + stage * kSlab + (4 * i + wave) * 1024;
                if (i < 2) lds_load_1k<kNtW>(to, gw[i < 2 ? i : 0] + (size_t)kt * 512, off);
                else lds_load_1k<false>(to, gx[i < 2 ? 0 : i - 2] + (size_t)kt * 512, off);
            };
            auto rd = [&](int stage, int b) {
                return __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(sbuf + stage * kSlab + b * 1024 + off));
            };
            // weight fragment m: phase 1: m = 0, 1 gate rows, m = 2, 3 the up rows of the same features
            auto ablk = [&](int m) { return kDown ? 4 * wm + m : (m < 2 ? 2 * wm + m : 4 + 2 * wm + m - 2); };

            f32x4 acc[NF][4];
#pragma unroll
            for (int n = 0; n < NF; ++n)
#pragma unroll
                for (int m = 0; m < 4; ++m) acc[n][m] = f32x4{0.f, 0.f, 0.f, 0.f};
            bf16x8 A[2][4], B[2][NF];

#pragma unroll
            for (int st = 0; st < S; ++st)
                if (st < nk) {
#pragma unroll
                    for (int i = 0; i < L; ++i) load(i, st, st);
                }
            if (nk >= S) wait_then_barrier<(S - 1) * L>();
            else wait_then_barrier<0>();
#pragma unroll
            for (int m = 0; m < 4; ++m) A[0][m] = rd(0, ablk(m));
#pragma unroll
            for (int n = 0; n < NF; ++n) B[0][n] = rd(0, 8 + 2 * n + wn);
            asm volatile("s_nop 7" ::: "memory");

            // Slab kt: its fragments are in registers (set P).  Once slab kt + 1 has landed
            // everywhere, read its fragments and load slab kt + S over slab kt, spread
            // between the MFMAs.  Past the last slab the read returns stale LDS, unused.
            int stage = 0;
            auto slab = [&](auto p_tag, auto tail_tag, int kt) {
                constexpr int P = decltype(p_tag)::value;
                constexpr bool kTail = decltype(tail_tag)::value;
                const int nst = stage == S - 1 ? 0 : stage + 1;
                __builtin_amdgcn_sched_barrier(0);
                wait_then_barrier<kTail ? 0 : (S - 2) * L>();
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int n = 0; n < NF; ++n) {
                    constexpr int kA = NF == 2 ? 2 : 1;  // weight fragments read per step
#pragma unroll
                    for (int i = 0; i < kA; ++i)
                        if (kA * n + i < 4) A[P ^ 1][kA * n + i] = rd(nst, ablk(kA * n + i));
                    B[P ^ 1][n] = rd(nst, 8 + 2 * n + wn);
#pragma unroll
                    for (int i = n * L / NF; i < (n + 1) * L / NF; ++i)
                        if (!kTail || kt + S < nk) load(i, kt + S, stage);
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const int m = (n & 1) ? 3 - q : q;  // neighbouring MFMAs share an operand
                        mfma_tied(acc[n][m], A[P][m], B[P][n]);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
                stage = nst;
            };
            using P0 = std::integral_constant<int, 0>;
            using P1 = std::integral_constant<int, 1>;
            int kt = 0;
#pragma unroll 1
            for (; kt + 1 + S < nk; kt += 2) {
                slab(P0{}, std::false_type{}, kt);
                slab(P1{}, std::false_type{}, kt + 1);
            }
            // claim the next item while the last slabs run (their waits cover the atomic)
            int got = 0;
            if (!few && wave == 0 && lane == 0)
                got = __hip_atomic_fetch_add(claim + xcd * kTClaimPitch, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll 1
            for (; kt < nk; kt += 2) {
                slab(P0{}, std::true_type{}, kt);
                slab(P1{}, std::true_type{}, kt + 1);
            }
            // MFMA results are read below: cover the longest wait they need
            asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int n = 0; n < NF; ++n)
#pragma unroll
                for (int m = 0; m < 4; ++m) asm volatile("" : "+a"(acc[n][m]));

            // Epilogue through the idle ring, so that the global stores are whole tile-layout
            // blocks or 256-byte runs of rows.  Lane holds column (token) lane % 16 of each
            // 16 x 16 tile, rows 4 (lane / 16) .. + 3.
            __syncthreads();  // every wave is done with the last stage
            if (wave == 0) {
                int it = claimed_item(q0 + __builtin_amdgcn_readfirstlane(got), xcd);
                if (few) it = -1;
                else if (it >= n_items) it = next_item(claim, q0, n_items, &xcd);
                if (lane == 0) *s_next = it;
            }
            int elane = lane;  // opaque: the addresses below are not worth registers in the K loop
            asm volatile("" : "+v"(elane));
            if (!kDown) {
                // act = silu(gate) * up in bf16, in the tile layout: token block tb, feature
                // block fb at LDS block 2 tb + fb (this wave: tb = 2 n + wn, fb = wm)
                uint8_t* ep = sbuf + (2 * wn + wm) * 1024 + 16 * ((elane & 15) + 16 * (elane >> 5)) + 8 * ((elane >> 4) & 1);
#pragma unroll
                for (int n = 0; n < NF; ++n)
#pragma unroll
                    for (int m = 0; m < 2; ++m) {
                        const f32x4 gv = acc[n][m], uv = acc[n][m + 2];
                        u32x2 packed;
                        packed.x = pack_bf16x2(silu(gv.x) * uv.x, silu(gv.y) * uv.y);
                        packed.y = pack_bf16x2(silu(gv.z) * uv.z, silu(gv.w) * uv.w);
                        *reinterpret_cast<u32x2*>(ep + n * 4096 + m * 512) = packed;
                    }
            } else {
                // expert outputs in bf16, rounded once (the combine sums them in fp32), as
                // token rows of 128 outputs
                uint8_t* ep = sbuf + ((16 * wn + (elane & 15)) * kTPitch + 64 * wm + 4 * (elane >> 4)) * 2;
#pragma unroll
                for (int n = 0; n < NF; ++n)
#pragma unroll
                    for (int m = 0; m < 4; ++m) {
                        const f32x4 v = acc[n][m];
                        u32x2 packed;
                        packed.x = pack_bf16x2(v.x, v.y);
                        packed.y = pack_bf16x2(v.z, v.w);
                        *reinterpret_cast<u32x2*>(ep + n * (32 * kTPitch * 2) + m * 32) = packed;
                    }
            }
        };
        if (nblk <= 4) run(std::integral_constant<int, 4>{});
        else if (nblk <= 8) run(std::integral_constant<int, 8>{});
        else if (nblk <= 12) run(std::integral_constant<int, 12>{});
        else run(std::integral_constant<int, 16>{});
        __syncthreads();
        const int next = __builtin_amdgcn_readfirstlane(*s_next);
        if (!kDown) {
            // nblk x 2 blocks of 1 KB
            uint16_t* act = static_cast<uint16_t*>(a.act) +
                            ((size_t)(tg.blk + n0 / 16) * (a.Fa / 32) + r0 / 32) * 512;
            for (int c = tid; c < nblk * 2 * 64; c += 256) {
                const int blk = c >> 6, piece = c & 63;
                const u32x4 v = *reinterpret_cast<const u32x4*>(sbuf + blk * 1024 + 16 * piece);
                __builtin_nontemporal_store(
                    v, reinterpret_cast<u32x4*>(act + ((size_t)(blk >> 1) * (a.Fa / 32) + (blk & 1)) * 512 + 8 * piece));
            }
        } else {
            // the group's rows x 16 pieces of 8 outputs, those that exist: bf16 rows for the
            // combine, or (moe_grouped_ffn on its own) the same values widened into y, where a
            // pass of its own that widened bf16 rows moved half the bytes again
            const int rows = min(kTN, tg.count - n0);
            const size_t at = (size_t)(tg.rowbase + n0) * a.H + r0;
            for (int c = tid; c < rows * 16; c += 256) {
                const int nl = c >> 4, piece = c & 15;
                if (r0 + 8 * piece >= a.H) continue;
                const u32x4 v = *reinterpret_cast<const u32x4*>(sbuf + (nl * kTPitch + 8 * piece) * 2);
                const size_t to = at + (size_t)nl * a.H + 8 * piece;
                if (a.y16) {
                    __builtin_nontemporal_store(v, reinterpret_cast<u32x4*>(a.y16 + to));
                } else {
                    *reinterpret_cast<f32x4*>(a.y + to) = bf16x4_to_f32(u32x2{v.x, v.y});
                    *reinterpret_cast<f32x4*>(a.y + to + 4) = bf16x4_to_f32(u32x2{v.z, v.w});
                }
            }
        }
        __syncthreads();  // the epilogue is done with the LDS
        item = next;
    }
}

// ---------------------------------------------------------------------------
// tiled kernel, fp32 prefill
// ---------------------------------------------------------------------------
//
// The same kind of items (128 weight rows x up to 128 of a group's rows, or smaller) and claim
// queues on v_mfma_f32_16x16x4_f32.  fp32 has a sixteenth of the bf16 MFMA rate, so the MFMAs bound
// it and its operands need no gathered copy: a 32-wide K slab of a row-major token row is a
// whole 128-byte line, loaded straight into the LDS (eight lanes a row).  LDS images, both
// read without bank conflicts:
//   weight block (2 KB): two 1 KB chunks of 32 lanes' values, in each the lanes' first 16
//     bytes and then their second ones;
//   token block (16 rows x 128 bytes): row r's 16-byte piece p at slot p ^ (r % 8).
// Two stages or more per ring; a slab's fragments are read behind its barrier, while the
// CU's other workgroup multiplies.  The accumulators are added into a second set every
// kFFlush slabs, so that no fp32 sum chain is longer than 256 products (the interleaved K
// split of the stream kernel, which ran these batches before, had chains of K / 4).
//
// Before (the decode stream kernel over 64-row chunks: 64 x 64 tiles, both operands from L2
// into registers, which asks 16 bytes per clock of every CU's load path) and now, phase 1 /
// phase 2 in us:
//   64 experts x 256 rows, H 2048, F 1408:  1907 / 1014 -> 1567 / 787 (121 TFLOP/s)
//   48 experts x 100 rows, H 2048, F 1408:   713 /  388 ->  647 / 283
//   48 experts x  40 rows, H 2048, F 1408:   395 /  218 ->  350 / 157
//    8 experts x  83 rows, H 4096, F 4096:   801 /  412 ->  402 / 222
// Token tiles of 64 or 96 rows instead of 128: 1693 / 871 and 1674 / 857 at 256 rows.  What is
// left: the last round of items (2816 for 512 workgroups in the first line) and the fragment
// reads behind each barrier.
//
// Item shapes.  A CU multiplies a slab of 128 x 128 for 2 us, so a phase of few such items takes as
// long as one of them, with most CUs idle; smaller items share it out.  The sums are the same in
// every shape.  64 x 32 takes two slabs per stage, since a slab's MFMAs (0.2 us) are short against
// a barrier.  Phase 1 / phase 2 in us, the stream kernel, 128 x 128 alone, and as chosen now:
//    1 expert  x 257 rows, H 2048, F 1024:    45 / 27,   145 /  77,   45 / 26
//    8 experts x  12 rows, H 2048, F 1024:    46 / 28,    54 /  32,   34 / 21
//    4 experts x  75 rows, H 1024, F 4096:   113 / 79,    65 / 215,   63 / 54
//    2 experts x  18 rows, H 4096, F 4096:    88 / 83,   102 /  97,   62 / 56
//   64 experts x  64 rows, H  512, F  256:    62 / 38,    38 /  24,   39 / 24

constexpr int kFN = 128;    // largest number of group rows per item
constexpr int kFLds = 72 * 1024;  // the ring of a workgroup: two workgroups per CU
// Item shapes: 128 weight rows x 128 or 32 group rows, and 64 x 32.
constexpr int kFShapes = 3;
__host__ __device__ constexpr int shape_rows(int shape) { return shape == 0 ? kFN : 32; }
__host__ __device__ constexpr int shape_weights(int shape) { return shape < 2 ? kTR : kTR / 2; }
static_assert(kFN == 128 && kTR == 128, "k_ffn_tiled_f32 shifts by these");
constexpr int kFFlush = 8;  // slabs between two additions into the second accumulators

__device__ __forceinline__ void mfma_tied_f32(f32x4& acc, float a, float b) {
    asm volatile("v_mfma_f32_16x16x4_f32 %0, %1, %2, %0" : "+v"(acc) : "v"(a), "v"(b));
}

// 16 bytes per lane from a per-lane address (see the uniform-base form above).
__device__ __forceinline__ void lds_load_1k_lanes(uint32_t lds, const void* p) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off"
                 :
                 : "s"(lds), "v"(p)
                 : "memory", "m0");
}

// The item shape of a phase: the first whose longest item is at most so many times a CU's share of
// the phase's work, else the last.  Full 128 x 128 tiles take half the LDS reads of 128 x 32 ones
// and win where a CU has several in turn; with one or two per CU, unequal ones leave CUs idle, which
// counts for less where an item's fixed costs (some 8 us) weigh more, at small K.  Times at a longest
// item of so many shares, 128 x 128 and 128 x 32 in us:
//   K above 512: 0.4: 445, 490 (8 x 83 rows, H 4096, F 4096);   0.6: 599, 512 (64 x 86, H 4096, F 512);
//     1.0 to 1.3: 509, 370 (8 x 128, H 4096, F 2048); 751, 345 (2 x 143, H 6144, F 4096); 137, 105 (64 x
//     8 + 2 shared x 1014, H 1536); 245, 263 (8 x 83, phase 2);   1.4: 569, 592 (4 x 173, H 8192)
//   K to 512: 1.1: 109, 85;   1.4: 21, 25;   1.6: 40, 47 (64 x 64, H 512);   1.9: 79, 69;   2.2: 116, 68
// and of the second shape's longest item, 128 x 32 and 64 x 32:
//   0.8: 20, 21;   1.0: 25, 31 and 78, 73;   1.1: 21, 22;   1.3: 52, 51 and 38, 35;   1.6: 36, 24.
// By every thread of the workgroup; s_red: 4 kFShapes floats.
__device__ int item_shape(const Args& a, int ng, const int* s_rows, bool down, float* s_red) {
    const float limit[kFShapes - 1] = {(down ? a.Fa : a.H) <= 512 ? 1.6f : 0.8f, 1.5f};
    constexpr int N = kFShapes;
    float v[N] = {};  // work, and each shape's longest item per weight row
    for (int gi = threadIdx.x; gi < ng; gi += 256) {
        const int Fg = gi < a.S ? a.Fs : a.F;
        const float K = down ? Fg : a.H, w = down ? a.H : 2 * Fg;
        const int rows = (s_rows[gi] + 31) / 32 * 32;
        v[0] += K * w * rows;
#pragma unroll
        for (int i = 0; i < kFShapes - 1; ++i) v[1 + i] = fmaxf(v[1 + i], K * min(rows, shape_rows(i)));
    }
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1)
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const float o = __shfl_xor(v[i], off, kWave);
            v[i] = i == 0 ? v[i] + o : fmaxf(v[i], o);
        }
    if (lane_id() == 0)
#pragma unroll
        for (int i = 0; i < N; ++i) s_red[N * (threadIdx.x >> 6) + i] = v[i];
    __syncthreads();
    const float share = (s_red[0] + s_red[N] + s_red[2 * N] + s_red[3 * N]) / a.cus;
    int shape = 0;
    for (; shape < kFShapes - 1; ++shape) {
        const int i = 1 + shape;
        const float longest = fmaxf(fmaxf(s_red[i], s_red[N + i]), fmaxf(s_red[2 * N + i], s_red[3 * N + i]));
        if (longest * shape_weights(shape) <= limit[shape] * share) break;
    }
    return shape;
}

// fp32 prefill: the groups in order and the prefix of their items, in tmeta: int32 header[8]
// (items of phase 1, of phase 2, groups, item shape of phase 1, of phase 2), TileGroup[groups],
// first item[groups] of phase 1 and of phase 2.  A workgroup for each phase (a chain of round
// trips and scans); the others pack the offloaded rows.
__global__ void __launch_bounds__(256) k_tile_groups(Args a) {
    __shared__ int s_list[256];
    __shared__ int4 s_info[256];
    __shared__ int s_wsum[8];
    __shared__ int s_ipre[kGMaxGroups + 1];
    __shared__ int s_rows[kGMaxGroups];
    __shared__ int16_t s_ord[kGMaxGroups];
    __shared__ float s_red[4 * kFShapes];
    if (blockIdx.x > 1) {
        pack_offloaded(a, blockIdx.x - 2, gridDim.x - 2, 4);
        return;
    }
    const int ph = blockIdx.x;
    const int nact = runnable(a, list_active(a, s_list, s_wsum, s_info));
    const int ng = nact + a.S;
    order_groups(a, nact, s_info, s_rows, s_ord);
    TileGroup* groups = reinterpret_cast<TileGroup*>(a.tmeta + kTHeader);
    if (ph == 0) write_tile_groups(a, ng, s_info, s_rows, s_ord, nullptr, 0, groups);
    const int shape = item_shape(a, ng, s_rows, ph == 1, s_red), tn = shape_rows(shape), wr = shape_weights(shape);
    const int total = group_prefix(ng, s_ipre, s_wsum + 5, [&](int o) {
        const int gi = s_ord[o];
        return weight_tiles(a.H, gi < a.S ? a.Fs : a.F, ph == 1, wr) * ((s_rows[gi] + tn - 1) / tn);
    });
    int32_t* pre = reinterpret_cast<int32_t*>(groups + a.max_routed + a.S) + ph * (a.max_routed + a.S);
    for (int o = threadIdx.x; o < ng; o += 256) pre[o] = s_ipre[o];
    if (threadIdx.x == 0) {
        a.tmeta[ph] = total;
        a.tmeta[3 + ph] = shape;
        if (ph == 0) a.tmeta[2] = ng;
    }
}

template <bool kDown>
__global__ void __launch_bounds__(256, 2)
    k_ffn_tiled_f32(Args a, const TileGroup* __restrict__ groups, const int32_t* __restrict__ pre, int32_t* claim) {
    __shared__ __attribute__((aligned(1024))) uint8_t sbuf[kFLds];
    __shared__ int32_t s_next;
    __shared__ uint8_t s_live[kFN];  // phase 1: the item's row names a token of the batch
    const int tid = threadIdx.x, lane = lane_id();
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave & 1, wn = wave >> 1;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_u8*)sbuf;
    const uint32_t woff = 16 * (2 * (lane & 31) + (lane >> 5));  // a lane's bytes of a 1 KB weight chunk
    const int n_items = a.tmeta[kDown ? 1 : 0], ng = a.tmeta[2];
    const int shape = a.tmeta[kDown ? 4 : 3], tn = shape_rows(shape), wr = shape_weights(shape);
    const int ltn = shape == 0 ? 7 : 5, lwt = (shape < 2 ? 7 : 6) - (kDown ? 0 : 1);  // log2 of a token and a weight tile
    const int q0 = gridDim.x / 8;
    int xcd = blockIdx.x % 8;
    const bool few = n_items <= a.cus;
    int item = few ? few_item(blockIdx.x / 8, xcd, 0) : claimed_item(blockIdx.x / 8, xcd);
    if (few && item >= n_items) return;
    if (item >= n_items) {
        if (wave == 0) {
            const int it = next_item(claim, q0, n_items, &xcd);
            if (lane == 0) s_next = it;
        }
        __syncthreads();
        item = __builtin_amdgcn_readfirstlane(s_next);
    }

    while (item >= 0) {
        // last group whose first item is <= item: the groups at or below it, counted
        int below = 0;
        for (int o = 0; o < ng; o += kWave) below += __popcll(__ballot(o + lane < ng && pre[min(o + lane, ng - 1)] <= item));
        const int go = __builtin_amdgcn_readfirstlane(below - 1);
        const TileGroup tg = groups[go];
        const bool shared = tg.wsel < 0;
        const int Fg = shared ? a.Fs : a.F;
        int wt, tt;
        item_tiles(item - pre[go], ((kDown ? a.H : Fg) + (1 << lwt) - 1) >> lwt, (tg.count + tn - 1) >> ltn, &wt, &tt);
        const int n0 = __builtin_amdgcn_readfirstlane(tt) << ltn;
        const int r0 = __builtin_amdgcn_readfirstlane(wt) << lwt;
        const int K = kDown ? Fg : a.H;
        const int nk = K / 32;
        const size_t wsize = (size_t)(kDown ? 1 : 2) * Fg * a.H;
        const float* wbase = shared ? static_cast<const float*>(kDown ? a.ws2 : a.ws13) + (size_t)(-tg.wsel - 1) * wsize
                                    : static_cast<const float*>(kDown ? a.w2 : a.w13) + (size_t)tg.wsel * wsize;
        // this wave's weight blocks (one if the item has four); phase 1: gate rows in the first half of
        // the blocks, the same features' up rows in the second; a row tile past the matrix reads
        // tile 0 (never stored)
        const float* gw[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int b = wr < kTR ? wave : 2 * wave + i;
            int rt;
            if (kDown) {
                rt = r0 / 16 + b;
                if (16 * rt >= a.H) rt = 0;
            } else {
                const int half = wr / 32;
                rt = (b >= half ? Fg / 16 + b - half : b) + r0 / 16;
            }
            gw[i] = wbase + (size_t)rt * nk * 512;
        }
        const int rows = min(tn, tg.count - n0);

        // the item with its weight rows in WB blocks (4 or 8), its tokens in NB (2, 4, 6 or 8)
        auto run = [&](auto wb_tag, auto nb_tag) {
            constexpr int WB = decltype(wb_tag)::value, NB = decltype(nb_tag)::value;
            constexpr int NW = WB / 2, NF = NB / 2;  // a wave's weight fragments, and its tokens': blocks 2 n + wn
            constexpr int U = WB == 4 ? 2 : 1;              // slabs per stage and barrier (nk is even)
            constexpr int LW = WB / 2, LX = NB / 2, L = U * (LW + LX);  // loads of a wave per slab, per stage
            constexpr int kSlab = (WB + NB) * 2048, kTok = WB * 2048;
            constexpr int S = NB <= 4 ? 3 : 2;              // stages of the ring
            static_assert(S * U * kSlab <= kFLds && (S - 1) * L < 64, "ring");
            const int ns = nk / U;
            // this wave's first weight and token chunk of stage 0; opaque, so that the sums with them are
            // made where they are used and not kept in registers across the items
            uint32_t wring = lds0 + wave * LW * 1024, xring = lds0 + kTok + wave * LX * 1024;
            asm volatile("" : "+s"(wring), "+s"(xring));
            // token row of this lane in load i: row 8 (j % 2) + lane / 8 of token block j / 2,
            // j = wave LX + i; rows past the group read the item's first row (never stored), and
            // rows that name no token read the batch's first (zeros are stored in their place)
            const float* gx[LX];
            int tok[LX];  // the loads' rows, then their tokens
#pragma unroll
            for (int i = 0; i < LX; ++i) {
                const int n = 8 * (wave * LX + i) + (lane >> 3);
                tok[i] = n0 + (n < rows ? n : 0);
            }
            if (!kDown) {
                if (!shared) {
                    // all of the loads before the first use
#pragma unroll
                    for (int i = 0; i < LX; ++i) tok[i] = a.perm[tg.rowbase + tok[i]];
#pragma unroll
                    for (int i = 0; i < LX; ++i) {
                        const int q = tok[i], t = max(q, 0) / a.k;
                        tok[i] = q < 0 || t >= a.T ? -1 : t;
                    }
                }
            }
#pragma unroll
            for (int i = 0; i < LX; ++i)
                gx[i] = static_cast<const float*>(kDown ? a.act : a.x) + 4 * ((lane & 7) ^ (lane >> 3)) +
                        (kDown ? (size_t)(tg.rowbase + tok[i]) * a.Fa : (size_t)max(tok[i], 0) * a.H);
            auto issue = [&](int st, int stage) {
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const uint32_t to = (stage * U + u) * kSlab;
                    const int kt = st * U + u;
#pragma unroll
                    for (int i = 0; i < LW; ++i)
                        lds_load_1k<false>(wring + to + i * 1024, gw[i / 2] + (size_t)kt * 512 + (i % 2) * 256, woff);
#pragma unroll
                    for (int i = 0; i < LX; ++i) lds_load_1k_lanes(xring + to + i * 1024, gx[i] + (size_t)kt * 32);
                }
            };
            f32x4 acc[NF][NW], tot[NF][NW];
#pragma unroll
            for (int n = 0; n < NF; ++n)
#pragma unroll
                for (int m = 0; m < NW; ++m) acc[n][m] = tot[n][m] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int st = 0; st < S - 1; ++st)
                if (st < ns) issue(st, st);
            if (!kDown && (lane & 7) == 0)
#pragma unroll
                for (int i = 0; i < LX; ++i) s_live[8 * (wave * LX + i) + (lane >> 3)] = tok[i] >= 0;
            // this lane's first piece of a weight block, and of a token block's row lane % 16
            const uint8_t* aw = sbuf + (lane >> 5) * 1024 + (lane & 31) * 16;
            const uint8_t* bx = sbuf + kTok + (lane & 15) * 128;
            const int p0 = 2 * (lane >> 4), sw = lane & 7;
            const int b_lo = ((p0 ^ sw) * 16), b_hi = (((p0 + 1) ^ sw) * 16);
            int stage = 0, got = 0;
#pragma unroll 1
            for (int st = 0; st < ns; ++st) {
                __builtin_amdgcn_sched_barrier(0);
                if (S > 2 && ns - 1 - st >= S - 2) wait_then_barrier<(S - 2) * L>();
                else wait_then_barrier<0>();
                __builtin_amdgcn_sched_barrier(0);
                if (st + S - 1 < ns) issue(st + S - 1, stage == 0 ? S - 1 : stage - 1);
                // claim the next item while the last slabs run
                if (!few && st == (U == 1 ? ns - 2 : ns - 1) && wave == 0 && lane == 0)
                    got = __hip_atomic_fetch_add(claim + xcd * kTClaimPitch, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int so = (stage * U + u) * kSlab, kt = st * U + u;
                    f32x4 A[2][NW], B[2][NF];
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
#pragma unroll
                        for (int m = 0; m < NW; ++m) {
                            constexpr int kHalf = NW / 2;  // phase 1: as many gate as up fragments
                            const int blk = kDown ? NW * wm + m : m / kHalf * (WB / 2) + kHalf * wm + m % kHalf;
                            A[h][m] = *reinterpret_cast<const f32x4*>(aw + so + blk * 2048 + h * 512);
                        }
#pragma unroll
                        for (int n = 0; n < NF; ++n)
                            B[h][n] = *reinterpret_cast<const f32x4*>(bx + so + (2 * n + wn) * 2048 + (h ? b_hi : b_lo));
                    }
                    // K 8 (lane / 16) + 4 h + i of the slab, over all tiles before the next i
#pragma unroll
                    for (int h = 0; h < 2; ++h)
#pragma unroll
                        for (int i = 0; i < 4; ++i)
#pragma unroll
                            for (int n = 0; n < NF; ++n)
#pragma unroll
                                for (int m = 0; m < NW; ++m) mfma_tied_f32(acc[n][m], A[h][m][i], B[h][n][i]);
                    if (u == U - 1 && (kt % kFFlush == kFFlush - 1 || kt == nk - 1)) {
                        // the MFMAs' results are read as ordinary registers: cover their latency
                        asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");
                        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                        for (int n = 0; n < NF; ++n)
#pragma unroll
                            for (int m = 0; m < NW; ++m) {
                                asm volatile("" : "+v"(acc[n][m]));
                                tot[n][m] += acc[n][m];
                                acc[n][m] = f32x4{0.f, 0.f, 0.f, 0.f};
                            }
                        asm volatile("s_nop 7" ::: "memory");
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
                stage = stage == S - 1 ? 0 : stage + 1;
            }
            if (wave == 0) {
                int it = claimed_item(q0 + __builtin_amdgcn_readfirstlane(got), xcd);
                if (few) it = -1;
                else if (it >= n_items) it = next_item(claim, q0, n_items, &xcd);
                if (lane == 0) s_next = it;
            }
            // lane holds token lane % 16 of each 16 x 16 tile, weight rows 4 (lane / 16) .. + 3
#pragma unroll
            for (int n = 0; n < NF; ++n) {
                const int nl = 16 * (2 * n + wn) + (lane & 15);
                if (nl >= rows) continue;
                if (!kDown) {
                    float* dst = static_cast<float*>(a.act) + (size_t)(tg.rowbase + n0 + nl) * a.Fa + r0 + 8 * NW * wm +
                                 4 * (lane >> 4);
                    const bool live = s_live[nl];
#pragma unroll
                    for (int m = 0; m < NW / 2; ++m) {
                        const f32x4 gv = tot[n][m], uv = tot[n][m + NW / 2];
                        const f32x4 v = {silu(gv.x) * uv.x, silu(gv.y) * uv.y, silu(gv.z) * uv.z, silu(gv.w) * uv.w};
                        *reinterpret_cast<f32x4*>(dst + 16 * m) = live ? v : f32x4{0.f, 0.f, 0.f, 0.f};
                    }
                } else {
                    const int h = r0 + 16 * NW * wm + 4 * (lane >> 4);
                    float* dst = a.y + (size_t)(tg.rowbase + n0 + nl) * a.H + h;
#pragma unroll
                    for (int m = 0; m < NW; ++m)
                        if (h + 16 * m < a.H) *reinterpret_cast<f32x4*>(dst + 16 * m) = tot[n][m];
                }
            }
        };
        const int nb = (rows + 31) / 32;
        using W4 = std::integral_constant<int, 4>;
        using W8 = std::integral_constant<int, 8>;
        if (wr < kTR) run(W4{}, std::integral_constant<int, 2>{});
        else if (nb <= 1) run(W8{}, std::integral_constant<int, 2>{});
        else if (nb == 2) run(W8{}, std::integral_constant<int, 4>{});
        else if (nb == 3) run(W8{}, std::integral_constant<int, 6>{});
        else run(W8{}, std::integral_constant<int, 8>{});
        __syncthreads();  // every wave is done with the ring
        item = __builtin_amdgcn_readfirstlane(s_next);
    }
}

// y_out[p] = sum_c y[c][p] for resident packed rows p < n_res and all shared rows.
__global__ void __launch_bounds__(256) k_reduce_splits(int T, int H, int E, int k, int S, int slots,
                                                       const int32_t* __restrict__ counts,
                                                       const int32_t* __restrict__ expert_slot,
                                                       const float* __restrict__ y, int ks, long long stride,
                                                       float* __restrict__ y_out) {
    // every row's workgroup adds up n_res itself, one expert per thread
    __shared__ int s_sum[4];
    int n = 0;
    if ((int)threadIdx.x < E && is_resident(expert_slot[threadIdx.x], slots)) n = max(counts[threadIdx.x], 0);
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) n += __shfl_xor(n, off, kWave);
    if (lane_id() == 0) s_sum[threadIdx.x >> 6] = n;
    __syncthreads();
    const int nres = s_sum[0] + s_sum[1] + s_sum[2] + s_sum[3];
    const int P = T * k;
    const int row = blockIdx.x;
    if (row < P && row >= nres) return;
    for (int h = threadIdx.x * 4; h < H; h += 1024) {
        constexpr int kMax = 16;  // same order as the combine: chunk 0, then 1, ...
        f32x4 p[kMax];
#pragma unroll
        for (int c = 0; c < kMax; ++c)
            if (c < ks) p[c] = *reinterpret_cast<const f32x4*>(y + c * stride + (size_t)row * H + h);
        f32x4 v = p[0];
#pragma unroll
        for (int c = 1; c < kMax; ++c)
            if (c < ks) v += p[c];
        *reinterpret_cast<f32x4*>(y_out + (size_t)row * H + h) = v;
    }
}

int max_routed_groups(const Shape& s) {
    int m = s.E < s.slots ? s.E : s.slots;
    const int pairs = s.T * s.k;
    return m < pairs ? m : pairs;
}

bool use_stream(const Shape& s) { return s.T <= 64; }

template <typename Elt, bool kDown, bool kStreamW>
void launch_stream_w(int nt, int grid, const Args& a, hipStream_t st) {
    switch (nt) {
        case 1: hipLaunchKernelGGL((k_ffn_stream<Elt, 1, kDown, kStreamW>), dim3(grid), dim3(256), 0, st, a); break;
        case 2: hipLaunchKernelGGL((k_ffn_stream<Elt, 2, kDown, kStreamW>), dim3(grid), dim3(256), 0, st, a); break;
        case 3: hipLaunchKernelGGL((k_ffn_stream<Elt, 3, kDown, kStreamW>), dim3(grid), dim3(256), 0, st, a); break;
        default: hipLaunchKernelGGL((k_ffn_stream<Elt, 4, kDown, kStreamW>), dim3(grid), dim3(256), 0, st, a); break;
    }
}

template <typename Elt, bool kDown>
void launch_stream(int nt, bool stream_w, int grid, const Args& a, hipStream_t st) {
    if (stream_w) launch_stream_w<Elt, kDown, true>(nt, grid, a, st);
    else launch_stream_w<Elt, kDown, false>(nt, grid, a, st);
}

// Non-temporal weight loads when the weights one call can touch (every slot and
// shared expert) exceed a quarter of the 256 MB MALL: then they cannot stay in
// the caches from one call to the next anyway.
bool stream_weights(const Shape& s) {
    const long long b = s.bf16 ? 2 : 4;
    const long long bytes = 3ll * s.H * ((long long)s.slots * s.F + (long long)s.S * s.Fs) * b;
    return bytes > (64ll << 20);
}

}  // namespace

bool ffn_fuses_repack(const Shape& s) { return use_stream(s) && s.T > 0; }

namespace {
// bf16 prefill: row blocks of the routed groups padded to 16 rows (at most 15 pad
// rows per group) and of the batch in order
long long tiled_routed_rows(const Shape& s) {
    return (long long)s.T * s.k + 15ll * max_routed_groups(s);
}
long long tiled_t16(const Shape& s) { return (s.T + 15) / 16 * 16ll; }
bool use_tiled(const Shape& s) { return !use_stream(s); }
bool tiled_bf16(const Shape& s) { return s.bf16 && use_tiled(s); }

// Worst-case items of a tiled phase for items of `rows` weight rows (phase 1: half as many
// features) x tn group rows: the routed groups have at most ceil(P / tn) full token tiles plus
// one partial tile each
long long tiled_items_of(const Shape& s, bool down, int rows, int tn) {
    const long long P = (long long)s.T * s.k;
    const long long G = max_routed_groups(s);
    const long long rt = G == 0 ? 0 : (P + tn - 1) / tn + G;
    const long long tps = (s.T + tn - 1) / tn;
    if (down) return (rt + (long long)s.S * tps) * ((s.H + rows - 1) / rows);
    const int f = rows / 2;
    const long long wt_r = (s.F + f - 1) / f, wt_s = s.S > 0 ? (s.Fs + f - 1) / f : 0;
    return rt * wt_r + (long long)s.S * tps * wt_s;
}
// Entries of a phase's table (bf16).
long long tiled_items(const Shape& s, bool down) { return tiled_items_of(s, down, kTR, kTN); }

Args make_args(const Shape& s, const FfnArgs& fa) {
    Args a;
    a.T = s.T; a.H = s.H; a.E = s.E; a.F = s.F; a.k = s.k; a.S = s.S; a.Fs = s.Fs; a.slots = s.slots;
    a.x = fa.x; a.perm = fa.perm; a.counts = fa.counts; a.seg_start = fa.seg_start; a.expert_slot = fa.expert_slot;
    a.w13 = fa.w13; a.w2 = fa.w2; a.ws13 = fa.ws13; a.ws2 = fa.ws2;
    a.act = fa.act; a.Fa = fa.Fa; a.y = fa.y; a.ks = fa.ks; a.y_ks_stride = fa.y_ks_stride;
    a.max_routed = max_routed_groups(s);
    a.ipg_r = a.ipg_s = 0;
    a.topk_w = fa.topk_w;
    a.n_res = fa.n_res;
    a.off_rows = fa.off_rows;
    a.off_w = fa.off_w;
    a.xg = fa.xg;
    a.tmeta = fa.tmeta;
    a.cus = 0;
    a.tclaim = fa.tclaim;
    a.tcap1 = tiled_bf16(s) ? (int)tiled_items(s, false) : 0;
    a.y16 = static_cast<uint16_t*>(fa.y16);
    a.fused = fa.topk_idx != nullptr;
    // every slot can hold an active expert: the fused phase 1 maps routed items to slots
    a.slot_items = (s.T * s.k >= s.slots && s.E >= s.slots) ? 1 : 0;
    a.topk_idx = fa.topk_idx;
    a.rp_counts = fa.rp_counts;
    a.rp_seg_start = fa.rp_seg_start;
    a.rp_perm = fa.rp_perm;
    a.rp_inv_perm = fa.rp_inv_perm;
    a.rp_n_res = fa.rp_n_res;
    return a;
}
}  // namespace

long long ffn_act_rows(const Shape& s) {
    if (tiled_bf16(s)) return tiled_routed_rows(s) + (long long)s.S * tiled_t16(s);
    return (long long)s.T * s.k + (long long)s.S * s.T;
}

long long ffn_gather_rows(const Shape& s) {
    if (!tiled_bf16(s)) return 0;
    return tiled_routed_rows(s) + (s.S > 0 ? tiled_t16(s) : 0);
}

size_t ffn_tile_meta_bytes(const Shape& s) {
    if (!use_tiled(s)) return 0;
    if (!s.bf16) return kTHeader * 4 + (sizeof(TileGroup) + 2 * 4) * (size_t)(max_routed_groups(s) + s.S);
    const size_t need = kTHeader * 4 + sizeof(TileGroup) * (size_t)(max_routed_groups(s) + s.S) +
                        sizeof(TileItem) * (size_t)(tiled_items(s, false) + tiled_items(s, true));
    // the workspace of a shape is part of the interface (the fixed scratch array accepts or
    // refuses a layer by it): the tables keep the room that 32 bytes per 256-row tile take,
    // which is always enough
    const size_t room = 32 + 32 * (size_t)(tiled_items_of(s, false, 256, kTN) + tiled_items_of(s, true, 256, kTN));
    return need > room ? need : room;
}

size_t ffn_tile_claim_bytes(const Shape& s) { return use_tiled(s) ? 2 * 8 * kTClaimPitch * sizeof(int32_t) : 0; }

hipError_t launch_ffn_prepare(const Shape& s, const FfnArgs& fa, hipStream_t st) {
    if (s.T == 0 || !use_tiled(s)) return hipSuccess;
    Args a = make_args(s, fa);
    if (hipError_t e = device_cus(&a.cus); e != hipSuccess) return e;
    const int P = s.T * s.k;
    // pack workgroups: beside the one chain of the fp32 tables, enough to fill the chip with row
    // copies (24000 rows of 8 KB: 105 us with 256, 61 with 1024)
    const int pack_max = s.bf16 ? 256 : 1024;
    const int n_pack = (fa.off_rows || fa.off_w) ? (P < pack_max ? P : pack_max) : 0;
    if (!s.bf16) {
        hipLaunchKernelGGL(k_tile_groups, dim3((unsigned)(2 + n_pack)), dim3(256), 0, st, a);
        return hipGetLastError();
    }
    const long long blocks = ffn_gather_rows(s) / 16;
    // about two workgroups per CU over the blocks that the batch needs at least, of eight
    // 32-column blocks or more each
    const long long least = ((long long)P * (a.max_routed > 0) + (s.S > 0 ? s.T : 0) + 15) / 16;
    long long split = least > 0 ? 2 * a.cus / least : 1;
    if (split > s.H / 256) split = s.H / 256;
    if (split < 1) split = 1;
    hipLaunchKernelGGL(k_gather_tokens, dim3((unsigned)(kTabWgs + blocks * split + n_pack)), dim3(256), 0, st, a, kTabWgs,
                       (int)blocks, (int)split);
    return hipGetLastError();
}

int ffn_down_splits(const Shape& s) {
    if (!use_stream(s)) return 1;
    // Phase-2 work items: (groups) x (H / rows) x ks, each streaming `rows` rows
    // (16 per weight tile) of one K chunk.  Smallest ks (a power of two <= 16) such that
    //  * there are >= 512 workgroups (two per CU), and
    //  * the longest workgroup streams at most 1/400 of the phase's weights: one
    //    workgroup streams at about 1/200 of the chip's HBM rate, so with a 2x
    //    margin it then ends before the phase does, instead of forming its tail
    //    (a shared expert wider than the routed ones, or few wide experts);
    // while every wave keeps >= 8 K steps of 32.
    const long long groups_r = max_routed_groups(s);
    const long long groups = groups_r + s.S;
    if (groups == 0) return 1;
    int steps = s.F / 32;
    if (s.S > 0 && s.Fs / 32 < steps) steps = s.Fs / 32;
    const long long kmax = (s.S > 0 && s.Fs > s.F) ? s.Fs : s.F;
    const long long weights = (groups_r * s.F + (long long)s.S * s.Fs) * s.H;  // elements, worst case
    const long long rows = 16 * stream_mt((s.T + 15) / 16);
    auto balanced = [&](int ks) { return groups * (s.H / rows) * ks >= 512 && rows * kmax / ks * 400 <= weights; };
    int ks = 1;
    while (ks < 16 && !balanced(ks) && steps / (ks * 2) >= 16) ks *= 2;
    return ks;
}

hipError_t launch_grouped_ffn(const Shape& s, const FfnArgs& fa, hipStream_t st, hipEvent_t between) {
    if (s.T == 0) return hipSuccess;
    auto mark = [&]() -> hipError_t {
        hipError_t e = hipGetLastError();
        if (e == hipSuccess && between) e = hipEventRecord(between, st);
        return e;
    };
    Args a = make_args(s, fa);
    if (use_stream(s)) {
        const int nt = (s.T + 15) / 16;
        const bool sw = stream_weights(s);
        // phase 1: 32 features per workgroup
        const int mt = stream_mt(nt);
        a.ipg_r = s.F / (8 * mt);
        a.ipg_s = s.S > 0 ? s.Fs / (8 * mt) : 1;
        const int P = s.T * s.k;
        const int n_pack = (a.fused && (fa.off_rows || fa.off_w)) ? (P < 64 ? P : 64) : 0;  // pack workgroups (P >= 1)
        // phase 1, then (fused) the repack workgroup
        int grid = a.max_routed * a.ipg_r + s.S * a.ipg_s + (a.fused ? 1 : 0);
        if (grid > 0) {
            if (s.bf16) launch_stream<uint16_t, false>(nt, sw, grid, a, st);
            else launch_stream<float, false>(nt, sw, grid, a, st);
        }
        if (hipError_t e = mark(); e != hipSuccess) return e;
        // phase 2: 64 output rows x one K chunk per workgroup; (fused) then the pack
        // workgroups, which read the perm and n_res that phase 1 wrote
        a.ipg_r = (s.H / (16 * mt)) * a.ks;
        a.ipg_s = (s.H / (16 * mt)) * a.ks;
        grid = a.max_routed * a.ipg_r + s.S * a.ipg_s + n_pack;
        if (grid > 0) {
            if (s.bf16) launch_stream<uint16_t, true>(nt, sw, grid, a, st);
            else launch_stream<float, true>(nt, sw, grid, a, st);
        }
        return hipGetLastError();
    }
    // tiled: two workgroups per CU, each claiming items from the tables written before; the
    // offloaded rows were packed there
    if (hipError_t e = device_cus(&a.cus); e != hipSuccess) return e;
    const long long wgs = 2 * a.cus;
    const TileGroup* groups = reinterpret_cast<const TileGroup*>(a.tmeta + kTHeader);
    const long long n_groups = a.max_routed + a.S;
    for (int down = 0; down < 2; ++down) {
        // a workgroup per CU at least, so that as many items all start at once
        const long long items = s.bf16 ? tiled_items(s, down == 1)
                                       : tiled_items_of(s, down == 1, shape_weights(kFShapes - 1), shape_rows(kFShapes - 1));
        const unsigned grid = items == 0 ? 0 : (unsigned)std::min(wgs, std::max<long long>(a.cus, (items + 7) / 8 * 8));
        int32_t* claim = a.tclaim + down * 8 * kTClaimPitch;
        if (grid > 0 && s.bf16) {
            const TileItem* tab = reinterpret_cast<const TileItem*>(groups + n_groups) + (down ? a.tcap1 : 0);
            if (down) hipLaunchKernelGGL((k_ffn_tiled<true>), dim3(grid), dim3(256), 0, st, a, tab, groups, claim);
            else hipLaunchKernelGGL((k_ffn_tiled<false>), dim3(grid), dim3(256), 0, st, a, tab, groups, claim);
        } else if (grid > 0) {
            const int32_t* pre = reinterpret_cast<const int32_t*>(groups + n_groups) + down * n_groups;
            if (down) hipLaunchKernelGGL((k_ffn_tiled_f32<true>), dim3(grid), dim3(256), 0, st, a, groups, pre, claim);
            else hipLaunchKernelGGL((k_ffn_tiled_f32<false>), dim3(grid), dim3(256), 0, st, a, groups, pre, claim);
        }
        if (!down) {
            if (hipError_t e = mark(); e != hipSuccess) return e;
        }
    }
    return hipGetLastError();
}

hipError_t launch_reduce_splits(const Shape& s, const int32_t* counts, const int32_t* expert_slot, const float* y,
                                int ks, long long y_ks_stride, float* y_out, hipStream_t st) {
    const int rows = s.T * s.k + s.S * s.T;
    if (rows == 0) return hipSuccess;
    hipLaunchKernelGGL(k_reduce_splits, dim3(rows), dim3(256), 0, st, s.T, s.H, s.E, s.k, s.S, s.slots, counts,
                       expert_slot, y, ks, y_ks_stride, y_out);
    return hipGetLastError();
}

bool ffn_y_bf16(const Shape& s) { return tiled_bf16(s); }

size_t ffn_y_bytes(const Shape& s) {
    const long long rows = (long long)s.T * s.k + (long long)s.S * s.T;
    if (ffn_y_bf16(s)) return (size_t)rows * s.H * 2;
    return (size_t)ffn_down_splits(s) * rows * s.H * 4;
}

}  // namespace saem
