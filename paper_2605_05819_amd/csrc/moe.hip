// Expert-gathered compensated linear for a MoE layer (decode):
//
//     y[t][j] = deq(Q_e) x + B_e[:, :r_e] (A_e[:r_e] x),   e = ids[t][j]
//
// with x = x[t] (shared by a token's slots, e.g. gate/up) or x[t][j] (the
// slot's own input, e.g. down).  The paper regroups the same projection of
// all activated experts into one step (Section 4.2.2, Cross-Expert Pipeline
// Reorganization; Appendix A.1, MoE Layer); here that is one pair of launches
// over every routed expert, and only routed experts' codes, scales, zeros and
// factors are read.
//
// A call covers a window of up to 4 linears over the same routing and input
// (e.g. a layer's gate and up); a single linear is the window of one.
//
//  * moe_prep_kernel: workgroup (linear, j, q), j < min(E, T*k), reads the
//    routing table -- so no workgroup ever waits for another -- counts slots
//    per expert, scans the counts and takes e = the j-th routed expert in
//    ascending id order (none: it exits).  It computes t[slot][i] =
//    A_e[i] . x_slot for the rank rows i = 16q .. 16q + 15 (8 or 4 rows where
//    16 would leave CUs without a workgroup) of its linear over
//    all of e's slots on MFMA, 16 slots per pass, its four waves splitting K.
//    Bound by its chain (routing tables, then two rounds of loads): fewer,
//    larger workgroups (one rank row per wave before) take 17.0 -> 12.9 us at
//    512 slots over 128 experts of 2048 x 768, two linears of rank <= 32.  A
//    gated call forms SiLU(g) u as it reads the activations.  Workgroup
//    (0, j, 0) also writes e's entry of the active-expert table (for the
//    streamed kernel one for every 16 of its slots) and e's slots, in slot
//    order, into the sorted slot list, and (linear, j, 0) that
//    linear's rank of e; workgroups (linear, 0, 0) write the number of
//    routed experts and zero rows for slots whose id is out of range.  The
//    remaining workgroups prepare the activations (fp16, pair-permuted,
//    per-chunk sums) exactly as the dense decode does.
//  * moe_kernel: one workgroup per (linear, active expert, row batch); the
//    grid is sized for the most experts T*k slots can reach and surplus
//    workgroups exit on the device-side count.  Each wave loads its slice
//    (4 rows for 4-bit codes, 2 for 2-bit, per row set of LG lanes; one
//    16-byte chunk per lane) of the expert's backbone and factor entries
//    once and applies it to every slot routed to that expert.  Same
//    arithmetic as the dense decode kernel: mask-only unpack into subnormal
//    fp16 lanes, v_dot2, per-chunk scale and zero in fp32, B t in the same
//    partial sums, transposing butterfly, fixed-order K-slice reduction.
//  * moe_stream_kernel: 4-bit codes of many experts, the tiles of all of them
//    shared evenly by the resident workgroups and streamed through MFMA.
//  * moe_mfma_kernel: with several slots per expert (4-bit codes) where the
//    streamed kernel does not apply, the expert's rows against its slots on
//    MFMA (slots as the columns).

#include "cl_device.h"
#include "cl_internal.h"
#include "gemv_common.h"
#include "mfma_common.h"

namespace cl {

// Routing-error record of this device: zero, or bit 63 set with the slot
// (bits 32..62) and the id (bits 0..31) of an out-of-range routing entry seen
// by a MoE call since the record was last read.  Each device holds its own
// copy for the life of the process.
__device__ unsigned long long moe_routing_error;

namespace {

// rows per wave batch: 4 for 4-bit codes, 2 for 2-bit (twice the
// activation registers per chunk)
constexpr int rows_per_wave(int bits) { return bits == 4 ? 4 : 2; }
constexpr int kMaxSlots = 1024;      // T * k
constexpr int kMaxExperts = 1024;
constexpr int kTab = 24;             // ints per active-expert table entry
constexpr int kMaxMoeWin = 4;        // linears per window
// Direct path (moe_direct_kernel): at most this many slots; row batches per
// wave counted for 4 waves of 4 rows per row set of LG lanes (64 rows per
// workgroup, 32 with two chunks per lane; the launch splits them over 8
// waves)
constexpr int kDirectMaxSlots = 8;
constexpr int direct_batches(int lg, int cpl) { return cpl == 2 ? 2 : (lg == 64 ? 4 : 2); }
// Streamed path: workgroups of 4 waves that share the tiles (two per CU), and
// the tiles in flight per wave.
constexpr int kStreamBlocks = 512;
constexpr int kStreamDepth = 2;
constexpr int kStreamMaxRows = (1 << 29) / kMaxSlots - 1;   // 31-bit byte offsets of fp32 outputs
// Gated calls off the one-launch path form SiLU(g) u in the preparation, once
// per workgroup that reads the slot, up to this width (128 experts of 768: a
// kernel of its own took 4.7 us of a layer); on wider rows the repeated
// exponentials cost as much as that launch (16 experts of 1536: 10.8 against
// 5.9 + 4.5 us).
constexpr int kGateFuseMaxWidth = 1024;
// MFMA path: 16-row tiles per workgroup and K blocks in flight per wave.
// Measured on the 48-layer T = 64 step with the workgroup's loads issued in
// need order (scales and zeros, slot ids, code blocks): 8 x 1 166 us per
// layer, 4 x 2 191, 8 x 2 229, 12 x 1 230, 16 x 1 227 (with the code loads
// issued after the scale/zero copy: 4 x 2 213 us; one tile of 16 rows had
// taken 389, every workgroup re-reading its slots' activations).  Once the
// pipeline's tail stopped re-reading code blocks: 4 x 1 143.7 us, 8 x 1
// 150.5, 2 x 1 153.0, 6 x 1 161.7, 4 x 2 ~160 (165 VGPRs at 4 x 1: three
// waves per SIMD against two).
constexpr int kMoeTpw = 4;
constexpr int kMoeNbuf = 1;

// One linear of a window: its stacked experts and its share of the grids.
struct MoeLin {
    const uint32_t* q;
    const uint16_t* s;
    const uint16_t* z;
    const uint16_t* A;
    const uint16_t* B;
    const int32_t* ranks;
    const int32_t* slot_rank;  // [T*k] per-slot ranks (clamped to 0..r_max), or null: ranks[e]
    void* y;
    float* t;                // [T*k][r_max] (workspace)
    size_t q_stride, sz_stride, a_stride, b_stride;   // elements per expert
    int d_out, r_max;
    int rq;                  // preparation workgroups per expert (rr rank rows each)
    int bpe;                 // backbone batches per expert
    int prep_end;            // rank workgroups of linears 0 .. this one (prefix sum)
    int blk_end;             // backbone workgroups of linears 0 .. this one (prefix sum)
    int nrb;                 // direct path: row blocks per slot
};

// A window of n linears over the same routing and activations (one linear
// is the window n = 1).
struct MoeArgs {
    MoeLin lin[kMaxMoeWin];
    int n;
    const int32_t* ids;
    const uint16_t* x;
    const uint16_t* u;       // gated input: the activations are SiLU(x) u elementwise (null: x)
    int E, T, k, d_in, G, act, out, x_per_slot;
    // workspace
    int* n_active;
    int* table;              // [max_active + S / 16][kTab]: expert, first sorted index, slot count, first slot,
                             // then each linear's rank, then its first 16 slots (padded with the first)
    int split;               // an entry for every 16 slots of an expert (n_active counts those)
    int* sorted;             // [T*k] slot ids grouped by expert, slot order within
    f16x2* xp;               // [rows][d_in/2]
    float* sx;               // [rows][chunks]
    int ks, cps;             // K slices, chunks per slice
    int rr;                  // rank rows per preparation workgroup: 16 or 4
    int rb;                  // direct path: rows per workgroup
    int nrbm;                // direct path: row blocks per (linear, slot) unit (the largest linear's)
};

template <int BITS, bool GATED>
__global__ __launch_bounds__(256) void moe_prep_kernel(MoeArgs a) {
    constexpr int CPW = 32 / BITS, HPW = CPW / 2, PPC = 4 * HPW;
    // sids[S], mys[S] (this expert's slots, in slot order), hist[E] (slots
    // per expert), rk[E] (the experts' ranks): sized by the call, so more
    // workgroups fit a CU
    extern __shared__ int prep_lds[];
    __shared__ int wsum[4][2];
    __shared__ int wcnt[4];
    __shared__ int sel, sel_lt, sel_n, sel_at, srank;
    __shared__ f32x4 tred[4][64];          // the waves' K parts of a 16 x 16 tile of t
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = tid >> 6;
    const int S = a.T * a.k;
    const int blk = blockIdx.x;
    int* const sids = prep_lds;
    int* const mys = sids + S;
    int* const hist = mys + S;
    int* const rk = hist + a.E;

    if (blk < a.lin[a.n - 1].prep_end) {
        // workgroup (linear li, j, quad): the j-th routed expert (ascending
        // id), its a.rr rank rows from a.rr quad of linear li; every workgroup
        // derives the routing itself
        int li = 0;
        while (blk >= a.lin[li].prep_end) ++li;
        const MoeLin& L = a.lin[li];
        const int local = blk - (li ? a.lin[li - 1].prep_end : 0);
        const int j = local / L.rq;
        const int quad = local - j * L.rq;
        // The experts' ranks, the routing ids and the per-slot ranks are
        // loaded in one round trip: every load is unconditional (clamped
        // index, out-of-range values replaced afterwards), so none waits at
        // a branch for the ones before it.  The histogram is cleared
        // meanwhile.
        for (int i = tid; i < a.E; i += 256) hist[i] = 0;
        if (tid == 0) sel = -1;
        constexpr int kPer = kMaxExperts / 256;       // experts and slots per thread, at most
        const bool dyn = L.slot_rank != nullptr;
        const int32_t* rsrc = L.r_max > 0 ? L.ranks : a.ids;    // ranks may be null when r_max is 0
        const int32_t* ssrc = dyn ? L.slot_rank : a.ids;
        int rkv[kPer], idv[kPer], srv[kPer];
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
            const int i = tid + 256 * u;
            rkv[u] = rsrc[min(i, a.E - 1)];
            idv[u] = a.ids[min(i, S - 1)];
            srv[u] = ssrc[min(i, S - 1)];
        }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
            const int i = tid + 256 * u;
            if (i < a.E) rk[i] = L.r_max > 0 ? rkv[u] : 0;
            if (i < S) {
                sids[i] = idv[u];
                if (idv[u] >= 0 && idv[u] < a.E) atomicAdd(&hist[idv[u]], 1);
            }
        }
        __syncthreads();
        // block scan over the experts (thread t owns experts 4 t .. 4 t + 3):
        // the first sorted slot of each expert and its index among the
        // routed experts; expert e with index j is this workgroup's
        int c[4], cs = 0, fs = 0;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int ex = 4 * tid + q;
            c[q] = ex < a.E ? hist[ex] : 0;
            cs += c[q];
            // routed experts, and table entries in the upper half
            fs += c[q] > 0 ? 1 + ((a.split ? (c[q] + 15) / 16 : 1) << 16) : 0;
        }
        int ic = cs, ifl = fs;                   // inclusive scan within the wave
        for (int off = 1; off < 64; off <<= 1) {
            const int tc = __shfl_up(ic, off, 64), tf = __shfl_up(ifl, off, 64);
            if (lane >= off) { ic += tc; ifl += tf; }
        }
        if (lane == 63) { wsum[wave][0] = ic; wsum[wave][1] = ifl; }
        __syncthreads();
        int pc = ic - cs, pf = ifl - fs;
        for (int w2 = 0; w2 < wave; ++w2) { pc += wsum[w2][0]; pf += wsum[w2][1]; }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            if (c[q] > 0) {
                if ((pf & 0xffff) == j) { sel = 4 * tid + q; sel_lt = pc; sel_n = c[q]; sel_at = pf >> 16; }
                pc += c[q];
                pf += 1 + ((a.split ? (c[q] + 15) / 16 : 1) << 16);
            }
        }
        if (li == 0 && j == 0 && quad == 0 && tid == 0)
            *a.n_active = (wsum[0][1] + wsum[1][1] + wsum[2][1] + wsum[3][1]) >> 16;
        __syncthreads();
        if (j == 0 && quad == 0) {
            // out-of-range ids: their output rows are zero.  One parallel
            // check first (valid routing skips the rest), then each wave
            // zeroes the rows of its share of the slots.
            int bad = 0;
            for (int sl = tid; sl < S; sl += 256) bad |= !(sids[sl] >= 0 && sids[sl] < a.E);
            if (__syncthreads_or(bad)) {
                for (int sl = wave; sl < S; sl += 4) {
                    const int id = sids[sl];
                    if (id >= 0 && id < a.E) continue;
                    // the device's routing-error record (reported by
                    // cl_moe_status): a flag bit, the slot and the id
                    if (li == 0 && lane == 0)
                        __hip_atomic_store(&moe_routing_error,
                                           (1ull << 63) | (static_cast<unsigned long long>(sl) << 32) |
                                               static_cast<uint32_t>(id),
                                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    for (int o = lane; o < L.d_out; o += 64)
                        store_out(L.y, static_cast<size_t>(sl) * L.d_out + o, 0.f, a.out);
                }
            }
        }
        const int e = sel;
        if (e < 0) return;                      // fewer than j + 1 routed experts
        const int ne = sel_n, cnt_lt = sel_lt;
        int* const ent = a.table + kTab * sel_at;
        int rank = rk[e];
        rank = rank < 0 ? 0 : (rank > L.r_max ? L.r_max : rank);
        // per-slot ranks: the expert's rank here is the largest of its slots'
        // (A_e x is computed that far; each slot reads its own prefix)
        if (dyn && tid == 0) srank = 0;
        // this expert's slots in slot order (ballots, 256 slots per pass)
        int base_pos = 0;
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
            if (256 * u >= S) break;
            const int sl = 256 * u + tid;
            const bool mine = sl < S && sids[sl] == e;
            const unsigned long long m = __ballot(mine);
            if (lane == 0) wcnt[wave] = __popcll(m);
            __syncthreads();
            int off = base_pos;
            for (int w2 = 0; w2 < wave; ++w2) off += wcnt[w2];
            if (mine) {
                const int pos = off + __popcll(m & ((1ull << lane) - 1ull));
                if (li == 0 && quad == 0) {
                    a.sorted[cnt_lt + pos] = sl;
                    // entries 8 + pos, and past the last slot the first again
                    const int part = a.split ? pos >> 4 : 0, at = pos - 16 * part;
                    int* const pe = ent + kTab * part;
                    if (at < 16) pe[8 + at] = sl;
                    if (at == 0) {
                        pe[3] = sl;
                        for (int u = ne - 16 * part; u < 16; ++u) pe[8 + u] = sl;
                    }
                }
                mys[pos] = sl;
                if (dyn) {
                    const int rs = srv[u];
                    atomicMax(&srank, rs < 0 ? 0 : (rs > L.r_max ? L.r_max : rs));
                }
            }
            base_pos += wcnt[0] + wcnt[1] + wcnt[2] + wcnt[3];
            __syncthreads();
        }
        if (dyn) rank = srank;
        if (quad == 0 && tid == 0) {
            for (int first = 0; first < (a.split ? ne : 1); first += 16) {
                int* const pe = ent + kTab * (first / 16);
                if (li == 0) {
                    pe[0] = e;
                    pe[1] = cnt_lt + first;
                    pe[2] = a.split ? min(16, ne - first) : ne;
                }
                pe[4 + li] = rank;
            }
        }
        // t[slot][i] = A_e[i] . x_slot for 16 slots and 16 rank rows at a
        // time on v_mfma_f32_16x16x32_f16 (slots the A operand, rows of A_e
        // the B operand, both in natural k order); the four waves split K,
        // UN 32-column steps of loads in flight each.  Four accumulators: the
        // shorter chains leave t's error at the level of pairwise fp32 sums
        // (where the factor term dominates the output, 1.2e-7 of it against
        // 1.6e-7 with one).  Rows past the rank and absent slots repeat
        // present ones and are not stored.
        constexpr int UN = 8;
        if (a.rr * quad >= rank) return;
        const int g = lane >> 4, r = lane & 15;
        const int i = a.rr * quad + r;
        const uint16_t* ar = L.A + static_cast<size_t>(e) * L.a_stride +
                             static_cast<size_t>(min(a.rr * quad + min(r, a.rr - 1), rank - 1)) * a.d_in + 8 * g;
        const int nsteps = a.d_in / 32, spw = (nsteps + 3) / 4;
        const int s0 = wave * spw, s1 = min(s0 + spw, nsteps);
        for (int j0 = 0; j0 < ne; j0 += 16) {
            const int sl = mys[min(j0 + r, ne - 1)];
            const int xrow = a.x_per_slot ? sl : sl / a.k;
            const uint16_t* xr = a.x + static_cast<size_t>(xrow) * a.d_in + 8 * g;
            const uint16_t* ur = GATED ? a.u + static_cast<size_t>(xrow) * a.d_in + 8 * g : xr;
            f32x4 acc[4] = {};
            for (int sb = s0; sb < s1; sb += UN) {
                u32x4 av[UN], xv[UN], uv[GATED ? UN : 1];
#pragma unroll
                for (int v = 0; v < UN; ++v) {
                    const int k = 32 * (sb + v < s1 ? sb + v : s0);
                    av[v] = *reinterpret_cast<const u32x4*>(ar + k);
                    xv[v] = *reinterpret_cast<const u32x4*>(xr + k);
                    if constexpr (GATED) uv[v] = *reinterpret_cast<const u32x4*>(ur + k);
                }
                __builtin_amdgcn_sched_barrier(0);   // all loads out before any is converted
                auto products = [&](auto x8) {
#pragma unroll
                    for (int v = 0; v < UN; ++v)
                        if (sb + v < s1) acc[v & 3] = mfma(x8(v), av[v], acc[v & 3]);
                };
                if constexpr (GATED) products([&](int v) { return gated8_to_f16(xv[v], uv[v], a.act); });
                else if (a.act == DT_FP16) products([&](int v) { return xv[v]; });
                else products([&](int v) { return act8_to_f16(xv[v], DT_BF16); });
            }
            tred[wave][lane] = (acc[0] + acc[1]) + (acc[2] + acc[3]);
            __syncthreads();
            // lane (g, r) of wave w: slot 4 g + w of the pass, rank row r
            {
                float tot = 0.f;
#pragma unroll
                for (int v = 0; v < 4; ++v) tot += tred[v][lane][wave];
                const int u = j0 + 4 * g + wave;
                if (u < ne && r < a.rr && i < rank) L.t[static_cast<size_t>(mys[u]) * L.r_max + i] = tot;
            }
            __syncthreads();                     // tred is reused by the next pass
        }
        return;
    }
    // activation preparation, one thread per (row, chunk)
    const int rows = a.x_per_slot ? S : a.T;
    const int chunks = a.d_in / CPW / 4;
    const long long item = static_cast<long long>(blk - a.lin[a.n - 1].prep_end) * 256 + tid;
    if (item >= static_cast<long long>(rows) * chunks) return;
    const int row = static_cast<int>(item / chunks);
    const int c = static_cast<int>(item % chunks);
    f16x2 v[PPC];
    if constexpr (GATED) {
        const uint16_t *gr = a.x + static_cast<size_t>(row) * a.d_in, *ur = a.u + static_cast<size_t>(row) * a.d_in;
        load_chunk_pairs<BITS>(c, v, [&](int at, uint32_t out[4]) {
            const u32x4 h = gated8_to_f16(*reinterpret_cast<const u32x4*>(gr + at),
                                          *reinterpret_cast<const u32x4*>(ur + at), a.act);
#pragma unroll
            for (int q = 0; q < 4; ++q) { const uint32_t hq = h[q]; out[q] = hq; }
        });
    } else {
        load_chunk_x<BITS>(a.x + static_cast<size_t>(row) * a.d_in, c, a.act, v);
    }
    const f16x2 one = {static_cast<f16>(1.0f), static_cast<f16>(1.0f)};
    float sum = 0.f;
    f16x2* dst = a.xp + static_cast<size_t>(row) * (a.d_in / 2) + static_cast<size_t>(c) * PPC;
#pragma unroll
    for (int p = 0; p < PPC; ++p) {
        sum = dot2(v[p], one, sum);
        dst[p] = v[p];
    }
    a.sx[static_cast<size_t>(row) * chunks + c] = sum;
}

// NB: factor columns per lane (r_max <= NB * 64 * ks); 0 when r_max is 0.
// HOIST: unpack the codes once into fp16 lanes held in registers (for
// experts that meet several slots); otherwise unpack per slot.
// Sum R values over each group of LG consecutive lanes (LG = 16, 32 or 64,
// a power of two >= R, R <= 16) with a transposing butterfly; on return lane
// l holds the total of value index (l % LG) / (LG / R) of its group.
template <int R, int LG>
__device__ __forceinline__ float group_sum_multi(float (&v)[R]) {
    const int lane = threadIdx.x & 63;
    float a[R];
#pragma unroll
    for (int i = 0; i < R; ++i) a[i] = v[i];
    int n = R;
    int bit = LG / 2;
#pragma unroll
    for (int step = 0; step < 4; ++step) {
        if (n > 1) {
            const bool up = (lane & bit) != 0;
            const int h = n / 2;
#pragma unroll
            for (int i = 0; i < R / 2; ++i) {
                if (i < h) {
                    const float mine = up ? a[i + h] : a[i];
                    const float other = up ? a[i] : a[i + h];
                    a[i] = mine + __shfl_xor(other, bit, 64);
                }
            }
            n = h;
            bit >>= 1;
        }
    }
    float r = a[0];
    for (; bit > 0; bit >>= 1) r += __shfl_xor(r, bit, 64);
    return r;
}

// Without the hoisted unpack the kernel keeps no next-slot prefetch (it
// cost 19 VGPRs) and the 4-bit, one-factor-column instance is held to 128
// VGPRs (4 waves per SIMD): measured on MI355X, the 48-layer T = 1 and
// T = 8 steps went from 39.3 and 102.9 us to 37.3 and 94.1 us.  The
// 64-lane instance then keeps one register in scratch (one store and one
// load per wave); held to 168 VGPRs instead (3 waves per SIMD) it has none,
// but the T = 8 step takes 79.7 us against 75.1.
//
// LG: lanes per row set.  Rows of at least 64 chunks use the whole wave
// (LG = 64); shorter rows (the 768-wide down projection: 24 chunks) give
// each group of LG = 32 or 16 lanes its own R rows, so a wave covers
// 64 / LG row sets and fewer lanes idle (24 of 64 lanes were busy).
template <int BITS, int CPL, int NB, bool HOIST, int LG>
__global__ __launch_bounds__(512)
__attribute__((amdgpu_waves_per_eu(!HOIST && BITS == 4 && NB <= 1 ? 4 : 1)))
void moe_kernel(MoeArgs a) {
    constexpr int R = rows_per_wave(BITS);
    constexpr int CPW = 32 / BITS;
    constexpr int HPW = CPW / 2;
    constexpr int CPC = 4 * CPW;
    constexpr int PPC = 4 * HPW;
    constexpr int NACC = BITS == 4 ? 2 : 4;
    constexpr int NBA = NB > 0 ? NB : 1;
    __shared__ float red[8][R];

    // the active-expert count and this entry are read together (the entry
    // exists for every ae below min(E, T k); it is used only if ae is active)
    // workgroup -> (linear li, active expert ae, row batch)
    const int blk = blockIdx.x;
    int li = 0;
    while (blk >= a.lin[li].blk_end) ++li;
    const MoeLin& L = a.lin[li];
    const int local = blk - (li ? a.lin[li - 1].blk_end : 0);
    const int ae = local / L.bpe;
    const int n_active = *a.n_active;
    const int* ent = a.table + kTab * ae;
    const int e = ent[0], sbeg = ent[1], scnt = ent[2], slot0 = ent[3], rank = ent[4 + li];
    if (ae >= n_active) return;                     // whole workgroup: no routed expert here
    const int batch = local - ae * L.bpe;

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int waves = blockDim.x >> 6;
    const int ks = a.ks;
    const int rg_per_block = waves / ks;
    const int slice = wave % ks;
    const int rgw = wave / ks;
    const int words = a.d_in / CPW;
    const int chunks = words / 4;
    const int groups = a.d_in / a.G;
    const int c_begin = slice * a.cps;
    const int c_end = min(chunks, c_begin + a.cps);
    constexpr int SETS = 64 / LG;                  // row sets per wave
    const int lg = lane % LG;                      // lane within its row set
    const int row0 = ((batch * rg_per_block + rgw) * SETS + lane / LG) * R;
    const bool active = row0 < L.d_out;
    const int base = active ? row0 : 0;
    const int nrows = active ? min(R, L.d_out - row0) : 1;

    int cidx[CPL];
    float cmask[CPL];
#pragma unroll
    for (int j = 0; j < CPL; ++j) {
        cidx[j] = c_begin + lg + LG * j;
        const bool valid = cidx[j] < c_end;
        cmask[j] = valid ? 1.f : 0.f;
        if (!valid) cidx[j] = c_begin;
    }

    // this expert's rows: codes, scales, zeros, factor entries (loaded once)
    const uint32_t* qe = L.q + static_cast<size_t>(e) * L.q_stride;
    const uint16_t* se = L.s + static_cast<size_t>(e) * L.sz_stride;
    const uint16_t* ze = L.z + static_cast<size_t>(e) * L.sz_stride;
    u32x4 qv[R][CPL];
    float sc[R][CPL], zc[R][CPL];
    float bv[R][NBA];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int row = base + (r < nrows ? r : 0);
        const u32x4* qr = reinterpret_cast<const u32x4*>(qe + static_cast<size_t>(row) * words);
#pragma unroll
        for (int j = 0; j < CPL; ++j) {
            qv[r][j] = __builtin_nontemporal_load(qr + cidx[j]);
            const size_t gi = static_cast<size_t>(row) * groups + (cidx[j] * CPC) / a.G;
            sc[r][j] = f16_bits_to_f32(se[gi]) * cmask[j];
            zc[r][j] = f16_bits_to_f32(ze[gi]);
        }
#pragma unroll
        for (int m = 0; m < NB; ++m) {
            const int i = lg + LG * (slice + ks * m);
            const uint16_t* Be = L.B + static_cast<size_t>(e) * L.b_stride;
            bv[r][m] = i < rank ? f16_bits_to_f32(Be[static_cast<size_t>(row) * L.r_max + i]) : 0.f;
        }
    }

    // The expert's slot ids, 64 at a time in the lanes (read back with a
    // shuffle); with the hoisted unpack each slot's activations are loaded
    // one slot ahead, otherwise at the slot itself.
    auto load_x = [&](int sl, f16x2 (&xv)[PPC], float& sxv, float (&tv)[NBA]) {
        const int xrow = a.x_per_slot ? sl : sl / a.k;
        // this slot's rank: its own (per-slot ranks) or the expert's
        int rs = rank;
        if (L.slot_rank) {
            const int v = L.slot_rank[sl];
            rs = v < 0 ? 0 : (v > L.r_max ? L.r_max : v);
        }
        const u32x4* src = reinterpret_cast<const u32x4*>(a.xp + static_cast<size_t>(xrow) * (a.d_in / 2) +
                                                          static_cast<size_t>(cidx[0]) * PPC);
#pragma unroll
        for (int p4 = 0; p4 < PPC / 4; ++p4) {
            const u32x4 u = src[p4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const uint32_t uq = u[q];
                xv[4 * p4 + q] = __builtin_bit_cast(f16x2, uq);
            }
        }
        sxv = a.sx[static_cast<size_t>(xrow) * chunks + cidx[0]];
#pragma unroll
        for (int m = 0; m < NB; ++m) {
            const int i = lg + LG * (slice + ks * m);
            tv[m] = i < rs ? L.t[static_cast<size_t>(sl) * L.r_max + i] : 0.f;
        }
    };
    // the unpacked codes (HOIST), from the raw loads above
    constexpr int UPW = BITS == 4 ? 4 : 8;       // fp16 pairs per word
    f16x2 un[HOIST ? R : 1][HOIST ? 4 * UPW : 1];
    if constexpr (HOIST) {
#pragma unroll
        for (int rr0 = 0; rr0 < R; ++rr0)
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                const uint32_t qw = qv[rr0][0][w];
                unpack_word<BITS>(qw, &un[rr0][w * UPW]);
            }
    }
    // the first slot comes with the table entry, so its activations load
    // together with the codes; the rest of the slot ids are read meanwhile
    int lane_slot = lane < scnt ? a.sorted[sbeg + lane] : 0;
    f16x2 xn[HOIST ? PPC : 1];
    float sxn = 0.f, tn[HOIST ? NBA : 1];
    if constexpr (HOIST) load_x(slot0, xn, sxn, tn);
    for (int jslot = 0; jslot < scnt; ++jslot) {
        if constexpr (!HOIST) {
            if (jslot > 0 && (jslot & 63) == 0) {
                const int j = jslot + lane;
                lane_slot = j < scnt ? a.sorted[sbeg + j] : 0;
            }
        }
        const int sl = __shfl(lane_slot, jslot & 63, 64);
        f16x2 xv[PPC];
        float tv[NBA];
        float sxv;
        if constexpr (HOIST) {
#pragma unroll
            for (int p = 0; p < PPC; ++p) xv[p] = xn[p];
            sxv = sxn;
#pragma unroll
            for (int m = 0; m < NBA; ++m) tv[m] = tn[m];
            if (jslot + 1 < scnt) {
                if (((jslot + 1) & 63) == 0) {
                    const int j = jslot + 1 + lane;
                    lane_slot = j < scnt ? a.sorted[sbeg + j] : 0;
                }
                load_x(__shfl(lane_slot, (jslot + 1) & 63, 64), xn, sxn, tn);
            }
        } else {
            load_x(jslot == 0 ? slot0 : sl, xv, sxv, tv);
        }
        float acc[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            float d[NACC];
#pragma unroll
            for (int q = 0; q < NACC; ++q) d[q] = 0.f;
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                if constexpr (HOIST) dot_unpacked<BITS>(&un[r][w * UPW], xv + w * HPW, d);
                else dot_word<BITS>(qv[r][0][w], xv + w * HPW, d);
            }
            const float v = fmaf(combine<BITS>(d), 16777216.0f, -zc[r][0] * sxv);
            acc[r] = sc[r][0] * v;
        }
#pragma unroll
        for (int m = 0; m < NB; ++m)
#pragma unroll
            for (int r = 0; r < R; ++r) acc[r] = fmaf(bv[r][m], tv[m], acc[r]);
        const float tot = group_sum_multi<R, LG>(acc);
        constexpr int SPAN = LG / R;
        const int rr = (lg / SPAN) & (R - 1);
        if (ks == 1 || LG < 64) {               // short rows always have one K slice
            if ((lane & (SPAN - 1)) == 0 && active && row0 + rr < L.d_out)
                store_out(L.y, static_cast<size_t>(sl) * L.d_out + row0 + rr, tot, a.out);
        } else {
            if ((lane & (SPAN - 1)) == 0) red[wave][rr] = tot;
            __syncthreads();
            if (slice == 0 && lane < R && active && row0 + lane < L.d_out) {
                float v = 0.f;
                for (int kk = 0; kk < ks; ++kk) v += red[wave + kk][lane];
                store_out(L.y, static_cast<size_t>(sl) * L.d_out + row0 + lane, v, a.out);
            }
            __syncthreads();
        }
    }
}

// Few slots, 4-bit codes: one launch and no preparation.  Workgroup =
// (linear, slot, block of a.rb rows), the row blocks of one (linear, slot)
// unit on one XCD (48-layer T = 1 step 18.8 -> 18.5 us).  It reads the slot's expert id, forms
// the slot's activations in registers (the same fp16 pairs and chunk sums the
// preparation writes), computes t = A_e[:r] x itself (each of its NWV waves
// takes rows i = wave + NWV p below the rank, UR rows with all their loads in flight,
// one butterfly sum per row; the slot's other workgroups repeat this small
// product, r x d_in multiply-adds over A_e rows that L2 serves after the
// first), and then applies its rows' codes with the arithmetic of
// moe_kernel: row batches of 4 rows per row set of LG lanes, CPL chunks per
// lane.  Every load of the workgroup's NBW batches per wave is issued right
// after the id arrives, before the A_e x product: with one batch in flight
// per wave the layer waited one memory round trip per batch.  At one
// token with 8 routed experts this replaces the preparation launch and its
// dependent memory round trips (ids, A_e rows, then the backbone's reads of
// t and the activations).
// The gated activations h = SiLU(g) u of every slot, 8 per thread, as fp16.
__global__ __launch_bounds__(256) void moe_gate_kernel(const uint16_t* g, const uint16_t* u, uint16_t* h, size_t n8,
                                                       int act) {
    const size_t i = static_cast<size_t>(blockIdx.x) * 256 + threadIdx.x;
    if (i >= n8) return;
    reinterpret_cast<u32x4*>(h)[i] =
        gated8_to_f16(reinterpret_cast<const u32x4*>(g)[i], reinterpret_cast<const u32x4*>(u)[i], act);
}

template <int LG, int CPL, int NB, int QX, int NBW, bool GATED, int NWV>
__global__ __launch_bounds__(64 * NWV) void moe_direct_kernel(MoeArgs a) {
    constexpr int R = 4, CPC = 32, PPC = 16, HPW = 4, NACC = 2;
    constexpr int SETS = 64 / LG;
    constexpr int NBA = NB > 0 ? NB : 1;
    constexpr int UR = (QX > 4 || NWV > 4) ? 4 : 8;   // rank rows per wave in flight
    __shared__ float tsh[NBA * LG];                // t of the slot, zero past its rank
    __shared__ int rks[256];                       // the experts' ranks (E <= 256)
    // unit u = (linear u / S, slot u % S); workgroup i runs on XCD i % 8, so
    // the row blocks of unit u go to XCD u % 8: its A_e rows and activations
    // stay in one L2
    const int blk = blockIdx.x;
    const int S = a.T * a.k;
    const int nrbm = a.nrbm;
    const int j = blk / 8;
    const int u = blk % 8 + 8 * (j / nrbm);
    const int rbi = j % nrbm;
    if (u >= a.n * S) return;
    const int li = u / S;
    const int sl = u - li * S;
    const MoeLin& L = a.lin[li];
    if (rbi >= L.nrb) return;
    const int rfirst = rbi * a.rb;
    const int rend = min(L.d_out, rfirst + a.rb);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lg = lane % LG;
    const int chunks = a.d_in / CPC;
    const int words = a.d_in / 8;
    const int groups = a.d_in / a.G;

    const int e = a.ids[sl];
    const int xrow = a.x_per_slot ? sl : sl / a.k;
    const uint16_t* xr = a.x + static_cast<size_t>(xrow) * a.d_in;
    // activations of this lane's chunks (unpack pair order) and their sums
    int cidx[CPL];
    float cmask[CPL];
#pragma unroll
    for (int j = 0; j < CPL; ++j) {
        cidx[j] = lg + LG * j;
        cmask[j] = cidx[j] < chunks ? 1.f : 0.f;
        if (cidx[j] >= chunks) cidx[j] = 0;
    }
    // raw loads here; the conversion (load_chunk_x's pairs and the chunk
    // sums) waits until the other loads are out
    u32x4 xraw[CPL][4];
#pragma unroll
    for (int j = 0; j < CPL; ++j)
#pragma unroll
        for (int w = 0; w < 4; ++w) xraw[j][w] = *reinterpret_cast<const u32x4*>(xr + (cidx[j] * 4 + w) * 8);
    // gated input: the up rows beside the gate rows, SiLU(g) u formed at
    // the conversions below
    const uint16_t* ur = GATED ? a.u + static_cast<size_t>(xrow) * a.d_in : xr;
    u32x4 uraw[GATED ? CPL : 1][4];
    if constexpr (GATED) {
#pragma unroll
        for (int j = 0; j < CPL; ++j)
#pragma unroll
            for (int w = 0; w < 4; ++w) uraw[j][w] = *reinterpret_cast<const u32x4*>(ur + (cidx[j] * 4 + w) * 8);
    }
    // the rank comes with the id: per-slot ranks one word, static ranks the
    // whole table (thread i its expert i, E <= 256) for an LDS lookup once e
    // is known; both loads unconditional from selected pointers (a load
    // under a branch is waited for where the branches meet)
    const bool rtab = L.r_max > 0 && !L.slot_rank && a.E <= 256;
    const int rk_tab = (rtab ? L.ranks : a.ids)[rtab ? min(tid, a.E - 1) : 0];
    const int rk_slot = (L.slot_rank ? L.slot_rank : a.ids)[sl];
    if (e < 0 || e >= a.E) {
        // out-of-range id: this slot's rows are zero, and the device's
        // routing-error record notes it (as the preparation does)
        if (li == 0 && rbi == 0 && tid == 0)
            __hip_atomic_store(&moe_routing_error,
                               (1ull << 63) | (static_cast<unsigned long long>(sl) << 32) | static_cast<uint32_t>(e),
                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        for (int o = rfirst + tid; o < rend; o += 64 * NWV)
            store_out(L.y, static_cast<size_t>(sl) * L.d_out + o, 0.f, a.out);
        return;
    }

    // row batches: batch b covers rows rfirst + b R SETS .. + R SETS - 1, a
    // row set of LG lanes R consecutive rows; wave w takes b = w, w + NWV, ...
    const uint32_t* qe = L.q + static_cast<size_t>(e) * L.q_stride;
    const uint16_t* se = L.s + static_cast<size_t>(e) * L.sz_stride;
    const uint16_t* ze = L.z + static_cast<size_t>(e) * L.sz_stride;
    const uint16_t* Be = L.B + static_cast<size_t>(e) * L.b_stride;
    const int nbatch = (rend - rfirst + R * SETS - 1) / (R * SETS);
    // scales, zeros and factor entries one per register: 16-bit loads into
    // register halves make each load wait for the one before
    struct Bt {
        u32x4 q[R][CPL];
        uint32_t s[R][CPL], z[R][CPL], b[R][NBA];
    };
    auto row_of = [&](int b, int& row0, int& nrows) {
        row0 = rfirst + b * R * SETS + (lane / LG) * R;
        nrows = row0 < rend ? min(R, rend - row0) : 0;
    };
    auto load_batch = [&](int b, Bt& bt) {
        int row0, nrows;
        row_of(b, row0, nrows);
        const int base = nrows > 0 ? row0 : rfirst;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int row = base + (r < nrows ? r : 0);
#pragma unroll
            for (int j = 0; j < CPL; ++j) {
                bt.q[r][j] = __builtin_nontemporal_load(
                    reinterpret_cast<const u32x4*>(qe + static_cast<size_t>(row) * words) + cidx[j]);
                const size_t gi = static_cast<size_t>(row) * groups + (cidx[j] * CPC) / a.G;
                bt.s[r][j] = se[gi];
                bt.z[r][j] = ze[gi];
            }
#pragma unroll
            for (int m = 0; m < NB; ++m) {
                const int i = lg + LG * m;
                bt.b[r][m] = Be[static_cast<size_t>(row) * L.r_max + (i < L.r_max ? i : 0)];
            }
        }
    };
    // all of this wave's batches (b = wave + NWV u) load before the t product,
    // unconditionally (a batch past the last reads the last one's rows): a
    // load under a branch is waited for where the branches meet
    Bt bts[NBW];
#pragma unroll
    for (int u = 0; u < NBW; ++u) load_batch(min(wave + NWV * u, nbatch - 1), bts[u]);

    // t = A_e[:rank] x: x as fp16 runs, lane l and pass q holding columns
    // 512 q + 8 l .. + 7
    // raw loads now, the conversion after the A loads are out
    u32x4 xw[QX], uw[GATED ? QX : 1];
#pragma unroll
    for (int q = 0; q < QX; ++q) {
        const int c = 512 * q + 8 * lane;
        xw[q] = *reinterpret_cast<const u32x4*>(xr + (c < a.d_in ? c : 0));
        if constexpr (GATED) uw[q] = *reinterpret_cast<const u32x4*>(ur + (c < a.d_in ? c : 0));
    }
    bool xconv = false;
    // the slot's rank (the batches' loads are out; the A rows wait for it)
    if (tid < 256) rks[tid] = rk_tab;
    __syncthreads();
    int rank = L.slot_rank ? rk_slot : (rtab ? rks[e] : (L.r_max > 0 ? L.ranks[e] : 0));
    rank = L.r_max == 0 ? 0 : (rank < 0 ? 0 : (rank > L.r_max ? L.r_max : rank));
    const uint16_t* Ae = L.A + static_cast<size_t>(e) * L.a_stride;
    // rows below the rank only
    for (int p0 = 0; wave + NWV * p0 < rank; p0 += UR) {
        // clamped addresses and selects: the loads carry no branches
        u32x4 av[UR][QX];
#pragma unroll
        for (int u = 0; u < UR; ++u) {
            const int i = wave + NWV * (p0 + u);
            const int ic = i < rank ? i : wave;
#pragma unroll
            for (int q = 0; q < QX; ++q) {
                const int c = 512 * q + 8 * lane;
                av[u][q] = *reinterpret_cast<const u32x4*>(Ae + static_cast<size_t>(ic) * a.d_in + (c < a.d_in ? c : 0));
            }
        }
        // keep the value work below the loads above (hoisted, it waited for
        // earlier loads before these were issued)
        __builtin_amdgcn_sched_barrier(0);
        if (!xconv) {
#pragma unroll
            for (int q = 0; q < QX; ++q) {
                u32x4 v;
                if constexpr (GATED) v = gated8_to_f16(xw[q], uw[q], a.act);
                else v = act8_to_f16(xw[q], a.act);
                xw[q] = 512 * q + 8 * lane < a.d_in ? v : u32x4{0u, 0u, 0u, 0u};
            }
            xconv = true;
        }
        float d[UR];
#pragma unroll
        for (int u = 0; u < UR; ++u) {
            d[u] = 0.f;
#pragma unroll
            for (int q = 0; q < QX; ++q)
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    // copy the vector elements to scalars first: a bit_cast
                    // of a subscripted ext_vector reads element 0
                    const uint32_t ak = av[u][q][k], xk = xw[q][k];
                    d[u] = dot2(__builtin_bit_cast(f16x2, ak), __builtin_bit_cast(f16x2, xk), d[u]);
                }
        }
        // lane l holds the total of row p0 + l / (64 / UR)
        const float tot = wave_sum_multi<UR>(d);
        const int u = lane / (64 / UR);
        const int i = wave + NWV * (p0 + u);
        if (lane % (64 / UR) == 0 && i < rank) tsh[i] = tot;
    }
    for (int i = rank + tid; i < NBA * LG; i += 64 * NWV) tsh[i] = 0.f;
    __syncthreads();
    // the activations of this lane's chunks in the unpack's pair order,
    // (x[w 8 + p], x[w 8 + p + 4]) for word w and pair p, and their sums
    f16x2 xv[CPL][PPC];
    float sxv[CPL];
    const f16x2 one = {static_cast<f16>(1.0f), static_cast<f16>(1.0f)};
#pragma unroll
    for (int j = 0; j < CPL; ++j) {
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            u32x4 u;
            if constexpr (GATED) u = gated8_to_f16(xraw[j][w], uraw[j][w], a.act);
            else u = act8_to_f16(xraw[j][w], a.act);
#pragma unroll
            for (int pp = 0; pp < 4; ++pp) {
                const uint32_t lo = u[pp / 2], hi = u[(pp + 4) / 2];
                const uint32_t va = (pp & 1) ? (lo >> 16) : (lo & 0xffff);
                const uint32_t vb = (pp & 1) ? (hi & 0xffff0000u) : (hi << 16);
                xv[j][w * HPW + pp] = __builtin_bit_cast(f16x2, va | vb);
            }
        }
        float sum = 0.f;
#pragma unroll
        for (int p = 0; p < PPC; ++p) sum = dot2(xv[j][p], one, sum);
        sxv[j] = sum;
    }
    float tv[NBA];
#pragma unroll
    for (int m = 0; m < NBA; ++m) tv[m] = NB > 0 ? tsh[lg + LG * m] : 0.f;

#pragma unroll
    for (int u = 0; u < NBW; ++u) {
        const int b = wave + NWV * u;
        if (b >= nbatch) break;
        const Bt& cur = bts[u];
        int row0, nrows;
        row_of(b, row0, nrows);
        float acc[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            acc[r] = 0.f;
#pragma unroll
            for (int j = 0; j < CPL; ++j) {
                float d[NACC];
#pragma unroll
                for (int q = 0; q < NACC; ++q) d[q] = 0.f;
#pragma unroll
                for (int w = 0; w < 4; ++w) dot_word<4>(cur.q[r][j][w], xv[j] + w * HPW, d);
                const float v = fmaf(combine<4>(d), 16777216.0f, -f16_bits_to_f32(cur.z[r][j]) * sxv[j]);
                acc[r] = fmaf(f16_bits_to_f32(cur.s[r][j]) * cmask[j], v, acc[r]);
            }
#pragma unroll
            for (int m = 0; m < NB; ++m) {
                const float bvm = lg + LG * m < rank ? f16_bits_to_f32(cur.b[r][m]) : 0.f;
                acc[r] = fmaf(bvm, tv[m], acc[r]);
            }
        }
        const float tot = group_sum_multi<R, LG>(acc);
        constexpr int SPAN = LG / R;
        const int rr = (lg / SPAN) & (R - 1);
        if ((lane & (SPAN - 1)) == 0 && rr < nrows)
            store_out(L.y, static_cast<size_t>(sl) * L.d_out + row0 + rr, tot, a.out);
    }
}

// One value to element idx of an array of n; idx < 0: dropped by the bounds
// check.  n * 4 bytes must stay below 2^31.
__device__ __forceinline__ void buffer_store_out(void* y, uint32_t n, int idx, float v, int out) {
    const uint32_t es = out == DT_FP32 ? 4 : 2;
    const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(y, 0, n * es, 0x00027000);
    const uint32_t off = static_cast<uint32_t>(idx) * es;
    if (out == DT_FP32)
        __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, v), rsrc, idx < 0 ? 0xFFFFFFF0u : off, 0, 0);
    else
        __builtin_amdgcn_raw_buffer_store_b16(out == DT_FP16 ? f32_to_f16_bits(v) : f32_to_bf16_bits(v), rsrc,
                                              idx < 0 ? 0xFFFFFFF0u : off, 0, 0);
}

// The 4-bit backbone off the one-launch path, rows of at most 4096 codes: the
// expert's rows against its slots on v_mfma_f32_16x16x32_f16, streamed.
// Bound by HBM (the routed experts' codes).  The tiles of 16 rows of every
// routed expert and linear form one list (expert, linear, tile), once for every
// 16 slots of the expert, that the resident workgroups share evenly: a
// workgroup's start (table entries, slot ids, activations: three dependent round
// trips) is paid once or twice per call instead of once per 64 rows, no last
// wave of workgroups is nearly empty, and an expert of many slots is no one's
// double share (with a loop over its slots in the workgroups that held it, 64
// experts of 3072 x 2048 at 512 slots took 116 us where one had 17 of them and
// 175 on skewed routing; now 88 and 85, against 105 on moe_mfma_kernel).
// A workgroup's waves split K into KW = a.ks parts of NBK 128-code
// blocks and the tiles into blockDim / 64 / KW sets; D tiles per wave are in
// flight ahead of the one computed, across the borders of experts.  The slots
// of a table entry keep their activations (MFMA A operand, NBK x 64 bytes per
// lane) and their t operand in registers, so a tile costs its codes, scales,
// zeros (lane group g loads those of every fourth part; a shuffle hands them on)
// and factor row only.  Absent slots repeat a present one; their rows of
// the product are not stored.  Codes become the exact integers q - z, each
// quantization group's partial is scaled in fp32, the rank term is MFMA steps
// over [t | B_e] with t 2^-e as three fp16 parts that hold all of its 24 bits
// (e the exponent of the step's largest |t| of the slot, restored in fp32:
// neither overflow nor fp16's subnormal range is met); the K parts meet in LDS
// in a fixed order; one rounding.  Two tiles in flight (four layers of 128
// experts, 2048 x 768, at 512 slots: 502 us; three 510, one 527) and two
// workgroups per CU (one: 1.6 times the time; 256 registers do not fit three).
// Where the line lies: see stream_pays (NBK <= 4 blocks on KW <= 8 waves keep the
// activations within 64 registers; groups of 32 codes, four scales per block,
// were 2 % slower than on the kernels below).  gate,up / down of the layer above,
// traced: 65 / 50 -> 59 / 39 us at 512 slots, 36 / 23 -> 31 / 21 us at 64 (against
// moe_mfma_kernel and moe_kernel).
template <int NBK, int GPB, int KW, int D>
__global__ __launch_bounds__(KW > 4 ? 64 * KW : 256) __attribute__((amdgpu_waves_per_eu(2))) void moe_stream_kernel(MoeArgs a) {
    extern __shared__ float red[];                // [2][waves][4][64]
    constexpr int SPG = 4 / GPB, NP = NBK * GPB, NU = (NP + 3) / 4;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    constexpr int waves = KW > 4 ? KW : 4, RW = waves / KW;
    const int kw = wave % KW, rw = wave / KW;
    const int g = lane >> 4, r = lane & 15;
    // this workgroup's share [beg, end) of the list
    const int per = a.lin[a.n - 1].blk_end;       // tiles per expert, all linears
    const long long total = static_cast<long long>(*a.n_active) * per;
    const int beg = static_cast<int>(total * blockIdx.x / gridDim.x);
    const int end = static_cast<int>(total * (blockIdx.x + 1) / gridDim.x);
    if (beg >= end) return;
    const int ae0 = beg / per;
    // lane i: the table entry of active expert ae0 + i (a share spans few)
    const int elast = (end - 1) / per;
    const int* ent = a.table + kTab * min(ae0 + lane, elast);
    const int v_e = ent[0], v_scnt = ent[2];
    int v_rank[kMaxMoeWin];
#pragma unroll
    for (int i = 0; i < kMaxMoeWin; ++i) v_rank[i] = ent[4 + i];
    auto of = [&](int v, int ae) { return __builtin_amdgcn_readlane(v, ae - ae0); };
    auto rank_of = [&](int ae, int li) {
        return of(li == 0 ? v_rank[0] : li == 1 ? v_rank[1] : li == 2 ? v_rank[2] : v_rank[3], ae);
    };

    const int K = a.d_in;
    const int nkb = (K + 127) / 128, kb0 = kw * NBK;
    const int words_row = K / 8;
    const int groups = K / a.G;
    const uint32_t mlo = __builtin_amdgcn_readfirstlane(0x000F000Fu);
    const uint32_t mhi = __builtin_amdgcn_readfirstlane(0x00F000F0u);
    const uint32_t bias = 0x64006400u;
    const u32x4 zero = {0u, 0u, 0u, 0u};
    const f32x4 fzero = {0.f, 0.f, 0.f, 0.f};
    // this lane's word of each block, and the quantization group of its parts
    // (part p = GPB b + q: codes 32 SPG q .. of block b)
    int wo[NBK], go[NU];
#pragma unroll
    for (int b = 0; b < NBK; ++b) wo[b] = min((kb0 + b) * 16 + 4 * g, words_row - 4);
#pragma unroll
    for (int u = 0; u < NU; ++u) {
        const int p = min(g + 4 * u, NP - 1);
        go[u] = min(kb0 * 128 + 32 * SPG * p, K - 1) / a.G;
    }
    const int from = 4 * r;                       // shuffle source (bytes) of part p: from + 64 (p % 4)

    // position in the list; the loads run D steps ahead of the arithmetic
    struct Pos {
        int ae, li, lo, hi, t;
    };
    auto enter = [&](Pos& c) {                    // the share's tiles of (ae, li)
        const int base = c.ae * per + (c.li ? a.lin[c.li - 1].blk_end : 0);
        c.lo = max(beg - base, 0);
        c.hi = min(end - base, a.lin[c.li].blk_end - (c.li ? a.lin[c.li - 1].blk_end : 0));
        c.t = c.lo;
    };
    auto over = [&](const Pos& c) { return c.ae > elast; };
    auto advance = [&](Pos& c) {                  // true: another (ae, li)
        c.t += RW;
        if (c.t < c.hi) return false;
        c.t = c.lo;
        Pos nx = c;
        do {
            if (++nx.li == a.n) { nx.li = 0; ++nx.ae; }
            if (over(nx)) {                       // tiles of the last segment stay addressable
                c.ae = nx.ae;
                return true;
            }
            enter(nx);
        } while (nx.lo >= nx.hi);
        c = nx;
        return true;
    };

    struct Tile {
        u32x4 w[NBK];
        u32x4 b;
        uint32_t s[NU], z[NU];
    };
    // what the loads need of the segment (ae, li)
    const uint32_t* q_seg = nullptr;
    const uint16_t *s_seg = nullptr, *z_seg = nullptr, *b_seg = nullptr;
    int d_out_seg = 0, r_max_seg = 0, ko_seg = 0;
    bool pre_seg = false;
    auto rank_rows_aligned = [&](const MoeLin& L) {
        return L.r_max > 0 && (L.r_max & 7) == 0 && (reinterpret_cast<uintptr_t>(L.B) & 15) == 0;
    };
    auto load_segment = [&](const Pos& c) {
        const MoeLin& L = a.lin[c.li];
        const size_t e = of(v_e, c.ae);
        q_seg = L.q + e * L.q_stride;
        s_seg = L.s + e * L.sz_stride;
        z_seg = L.z + e * L.sz_stride;
        b_seg = L.B + e * L.b_stride;
        d_out_seg = L.d_out;
        r_max_seg = L.r_max;
        pre_seg = rank_rows_aligned(L) && 32 * kw < rank_of(c.ae, c.li);
        ko_seg = 32 * kw + 8 * g + 8 <= L.r_max ? 32 * kw + 8 * g : 0;
    };
    auto load_tile = [&](const Pos& c, Tile& t) {
        // a tile past the segment, or past the list, repeats one row of the last
        const bool live = c.t + rw < c.hi && !over(c);
        const int row0 = 16 * min(c.t + rw, c.hi - 1);
        const int rr = live ? min(r, d_out_seg - 1 - row0) : 0;
        const uint32_t* qt = q_seg + static_cast<size_t>(row0) * words_row;
        const uint16_t* st = s_seg + static_cast<size_t>(row0) * groups;
        const uint16_t* zt = z_seg + static_cast<size_t>(row0) * groups;
#pragma unroll
        for (int u = 0; u < NU; ++u) {
            t.s[u] = st[static_cast<uint32_t>(rr * groups + go[u])];
            t.z[u] = zt[static_cast<uint32_t>(rr * groups + go[u])];
        }
        // without a prefetched factor row: a line of the codes
        const char* bt = pre_seg ? reinterpret_cast<const char*>(b_seg + static_cast<size_t>(row0) * r_max_seg)
                                 : reinterpret_cast<const char*>(qt);
        t.b = *reinterpret_cast<const u32x4*>(bt + static_cast<uint32_t>(pre_seg ? 2 * (rr * r_max_seg + ko_seg) : 0));
#pragma unroll
        for (int b = 0; b < NBK; ++b)
            t.w[b] = __builtin_nontemporal_load(
                reinterpret_cast<const u32x4*>(qt + static_cast<uint32_t>(rr * words_row + wo[b])));
    };

    // the entry's slots and activations
    int sl = 0, osl[4], osl_k = 0;
    u32x4 x[NBK][4];
    auto load_x = [&](const Pos& c) {
        sl = a.table[kTab * c.ae + 8 + r];
        const int xrow = a.x_per_slot ? sl : sl / a.k;
        const u32x4* xr = reinterpret_cast<const u32x4*>(a.xp + static_cast<size_t>(xrow) * (K / 2));
#pragma unroll
        for (int b = 0; b < NBK; ++b) {
            const int kb = min(kb0 + b, nkb - 1);
#pragma unroll
            for (int t = 0; t < 4; ++t)
                x[b][t] = xr[GPB == 1 ? wo[b] + t : (kb * 128 + 32 * t < K ? kb * 16 + 4 * t + g : g)];
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) osl[q] = __shfl(sl, 4 * g + q, 64);
        osl_k = __shfl(sl, 4 * g + (kw & 3), 64);
    };
    // t operand of the rank step at factor column kr, and the factors that
    // restore it for this lane's accumulators (slots 4 g .. 4 g + 3)
    struct TOp {
        u32x4 hi, mid, lo;
        f32x4 up;
    };
    auto t_operand = [&](const MoeLin& L, int rank, int kr) {
        int rs = rank;
        if (L.slot_rank) {
            const int v = L.slot_rank[sl];
            rs = v < 0 ? 0 : (v > L.r_max ? L.r_max : v);
        }
        const float* trow = L.t + static_cast<size_t>(sl) * L.r_max;
        const int k = kr + 8 * g;
        float v[8], top = 0.f;
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const float tv = trow[k + q < L.r_max ? k + q : 0];
            v[q] = k + q < rs ? tv : 0.f;
            top = fmaxf(top, fabsf(v[q]));
        }
        top = fmaxf(top, __shfl_xor(top, 16, 64));
        top = fmaxf(top, __shfl_xor(top, 32, 64));
        const uint32_t ex = min(max(__builtin_bit_cast(uint32_t, top) >> 23, 1u), 253u);
        const float down = __builtin_bit_cast(float, (254u - ex) << 23);
        const float up = __builtin_bit_cast(float, ex << 23);
        TOp o;
        uint32_t h[4], m[4], l[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) split3_f16x2(v[2 * q] * down, v[2 * q + 1] * down, h[q], m[q], l[q]);
        o.hi = u32x4{h[0], h[1], h[2], h[3]};
        o.mid = u32x4{m[0], m[1], m[2], m[3]};
        o.lo = u32x4{l[0], l[1], l[2], l[3]};
#pragma unroll
        for (int q = 0; q < 4; ++q) o.up[q] = __shfl(up, 4 * g + q, 64);
        return o;
    };
    // B's columns at and past the rank count as zero (t's are, but 0 x inf)
    auto rank_step = [&](const TOp& o, u32x4 bw, int kr, int rank, f32x4& acc) {
        const int k = kr + 8 * g;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const uint32_t v = bw[q];
            const uint32_t lo = k + 2 * q < rank ? v & 0xffffu : 0u;
            const uint32_t hi = k + 2 * q + 1 < rank ? v & 0xffff0000u : 0u;
            bw[q] = lo | hi;
        }
        const f32x4 ph = mfma(o.hi, bw, fzero), pm = mfma(o.mid, bw, fzero), pl = mfma(o.lo, bw, fzero);
#pragma unroll
        for (int q = 0; q < 4; ++q)
            acc[q] = fmaf(o.up[q], fmaf(0x1p-11f, fmaf(0x1p-11f, pl[q], pm[q]), ph[q]), acc[q]);
    };

    Pos lp, cp;
    lp.ae = ae0;
    lp.li = 0;
    while (true) {                                // the segment of `beg`
        enter(lp);
        if (lp.lo < lp.hi) break;
        ++lp.li;
    }
    cp = lp;
    load_x(cp);
    load_segment(lp);
    Tile ring[D];
#pragma unroll
    for (int d = 0; d < D; ++d) {
        load_tile(lp, ring[d]);
        if (!over(lp) && advance(lp) && !over(lp)) load_segment(lp);
    }
    int rank = rank_of(cp.ae, cp.li);
    TOp t0{zero, zero, zero, fzero};
    if (32 * kw < rank) t0 = t_operand(a.lin[cp.li], rank, 32 * kw);
    int par = 0;
    // Past the end of the list a step only keeps the pipeline's shape: a way
    // out of the middle of the unrolled loop would join its head in the
    // structured control flow, with this tile's loads the youngest, and every
    // round would drain all loads in flight.
    auto do_step = [&](Tile& t) {
        const bool live = !over(cp);
        const MoeLin& L = a.lin[cp.li];
        const bool pre = rank_rows_aligned(L) && 32 * kw < rank;
        f32x4 acc = fzero;
        if (live) {
#pragma unroll
            for (int b = 0; b < NBK; ++b) {
                uint32_t w[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) { const uint32_t v = t.w[b][q]; w[q] = v; }
                if constexpr (GPB > 1) transpose_words(w);
#pragma unroll
                for (int q = 0; q < GPB; ++q) {
                    constexpr int four = 4;
                    const int p = GPB * b + q;
                    const uint32_t sz = __builtin_amdgcn_ds_bpermute(from + 64 * (p % four),
                                                                     t.s[p / four] | (t.z[p / four] << 16));
                    const Zq zq = make_zq(sz >> 16);
                    f32x4 pp = mfma(x[b][SPG * q], codes_minus_zero(w[SPG * q], zq, mlo, mhi, bias), fzero);
#pragma unroll
                    for (int u = SPG * q + 1; u < SPG * q + SPG; ++u)
                        pp = mfma(x[b][u], codes_minus_zero(w[u], zq, mlo, mhi, bias), pp);
                    const bool on = (kb0 + b) * 128 + 32 * SPG * q < K;
                    acc = fma4(on ? f16_bits_to_f32(static_cast<uint16_t>(sz)) : 0.f, pp, acc);
                }
            }
            if (pre) rank_step(t0, t.b, 32 * kw, rank, acc);
        }
        load_tile(lp, t);
        if (!over(lp) && advance(lp) && !over(lp)) load_segment(lp);
        const int tile = cp.t + rw;
        const int row = 16 * tile + r;
        const bool rowv = live && tile < cp.hi && row < L.d_out;
        // rank steps that were not prefetched: past 32 KW columns, or rows of
        // B that are not 16-byte aligned
        for (int kr = 32 * (pre ? kw + KW : kw); kr < (live ? rank : 0); kr += 32 * KW) {
            const TOp o = kr == 32 * kw ? t0 : t_operand(L, rank, kr);
            const uint16_t* brow = L.B + static_cast<size_t>(of(v_e, cp.ae)) * L.b_stride +
                                   static_cast<size_t>(min(row, L.d_out - 1)) * L.r_max;
            u32x4 bw;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int k = kr + 8 * g + 2 * q;
                const uint32_t lo = brow[k < L.r_max ? k : 0], hi = brow[k + 1 < L.r_max ? k + 1 : 0];
                bw[q] = lo | (hi << 16);
            }
            rank_step(o, bw, kr, rank, acc);
        }
        // the K parts summed in order: wave kw takes the slots 4 g + QN kw ..
        // of the tile.  Buffer stores, whose bounds check drops the absent
        // slots and rows: with a branch around them the compiler would have
        // to count them as not issued and wait for younger loads instead.
        constexpr int QN = KW >= 4 ? 1 : 4 / KW;
        const int q0 = KW > 1 ? QN * kw : 0;
        float v[QN];
        if constexpr (KW > 1) {
            float* const rb = red + (par * waves + rw * KW) * 256;
#pragma unroll
            for (int q = 0; q < 4; ++q) rb[kw * 256 + q * 64 + lane] = acc[q];
            __syncthreads();
#pragma unroll
            for (int q = 0; q < QN; ++q) {
                v[q] = rb[((q0 + q) & 3) * 64 + lane];
#pragma unroll
                for (int u = 1; u < KW; ++u) v[q] += rb[u * 256 + ((q0 + q) & 3) * 64 + lane];
            }
            par ^= 1;
        } else {
#pragma unroll
            for (int q = 0; q < 4; ++q) v[q] = acc[q];
        }
        const int scnt = of(v_scnt, min(cp.ae, elast));
#pragma unroll
        for (int q = 0; q < QN; ++q) {
            const bool on = rowv && q0 + q < 4 && 4 * g + q0 + q < scnt;
            const int os = KW == 1 ? osl[q] : KW == 2 ? (kw ? osl[2 + q] : osl[q]) : osl_k;
            if (L.d_out <= kStreamMaxRows)
                buffer_store_out(L.y, static_cast<uint32_t>(a.T * a.k) * L.d_out, on ? os * L.d_out + row : -1, v[q],
                                 a.out);
            else if (on)
                store_out(L.y, static_cast<size_t>(os) * L.d_out + row, v[q], a.out);
        }
        const int ae = cp.ae;
        if (live && advance(cp) && !over(cp)) {
            if (cp.ae != ae) load_x(cp);
            rank = rank_of(cp.ae, cp.li);
            if (32 * kw < rank) t0 = t_operand(a.lin[cp.li], rank, 32 * kw);
            // wait here, once per segment: x pending where the paths meet
            // would make every step wait for all loads in flight
            __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0)
        }
    };
    while (!over(cp)) {
#pragma unroll
        for (int d = 0; d < D; ++d) do_step(ring[d]);
    }
}

// Many slots per expert, 4-bit codes: the expert's rows against its slots on
// MFMA (v_mfma_f32_16x16x32_f16), so the per-slot VALU work of the kernel
// above (every slot's dot products on every lane) becomes MFMA rows.
// Workgroup = (linear, active expert, TPW tiles of 16 rows); its four waves
// split the 128-code blocks of K (wave w takes blocks w, w + 4, ..., NBUF in
// flight); the expert's slots go in passes of 16.  Per block a lane loads,
// for each tile, 16 bytes of codes of row r = lane % 16, and once for all
// tiles the matching four 16-byte words of prepared activations of its
// pass's slot r.  The activations are the MFMA's A operand and the codes its
// B operand, so lane (g, r) accumulates slots 4 g .. 4 g + 3 of the pass for
// weight row r.  As in the many-token dense decode the codes become the
// exact fp16 integers q - z and each quantization group's steps run into a
// fresh fp32 partial that the group's scale multiplies in fp32 (GPB groups
// per 128-code block; with more than one the code words are transposed
// across the lane groups first).  The rank term is extra MFMA steps over
// [t | B_e] (t split into fp16 hi and lo parts, one step each); the waves'
// tiles are summed through LDS in a fixed order; one rounding to the output
// dtype.
template <int TPW, int NBUF, int GPB>
__global__ __launch_bounds__(256) void moe_mfma_kernel(MoeArgs a) {
    __shared__ f32x4 red[4][TPW][64];
    extern __shared__ uint16_t szl[];             // [2][16 TPW][szl_stride(groups)]: the rows' scales, then zeros
    const int blk = blockIdx.x;
    int li = 0;
    while (blk >= a.lin[li].blk_end) ++li;
    const MoeLin& L = a.lin[li];
    const int local = blk - (li ? a.lin[li - 1].blk_end : 0);
    const int ae = local / L.bpe;                 // bpe: workgroups (16 TPW rows) per expert
    const int n_active = *a.n_active;
    const int* ent = a.table + kTab * ae;
    const int e = ent[0], sbeg = ent[1], scnt = ent[2], rank = ent[4 + li];
    if (ae >= n_active) return;                   // whole workgroup: no routed expert here
    const int row0 = (local - ae * L.bpe) * 16 * TPW;
    const int lane = threadIdx.x & 63;
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int g = lane >> 4, r = lane & 15;
    int row[TPW];
    bool rowv[TPW];
#pragma unroll
    for (int j = 0; j < TPW; ++j) {
        rowv[j] = row0 + 16 * j + r < L.d_out;
        row[j] = rowv[j] ? row0 + 16 * j + r : L.d_out - 1;
    }
    const int K = a.d_in;
    const int nkb = (K + 127) / 128;
    const int words_row = K / 8;
    const int groups = K / a.G;
    const uint32_t* qe = L.q + static_cast<size_t>(e) * L.q_stride;
    const uint16_t* se = L.s + static_cast<size_t>(e) * L.sz_stride;
    const uint16_t* ze = L.z + static_cast<size_t>(e) * L.sz_stride;
    const uint16_t* Be = L.B + static_cast<size_t>(e) * L.b_stride;
    const uint32_t mlo = __builtin_amdgcn_readfirstlane(0x000F000Fu);
    const uint32_t mhi = __builtin_amdgcn_readfirstlane(0x00F000F0u);
    const uint32_t bias = 0x64006400u;
    const u32x4 zero = {0u, 0u, 0u, 0u};

    struct Blk {
        u32x4 w[TPW];
        u32x4 x[4];
    };
    // codes of block kb for this lane's tiles, and the activations of the
    // words it feeds to MFMA step t: 4 g + t of the block, or 4 t + g once
    // the codes are transposed (a word past K reads word g, met by a zero
    // scale).  Loads are unconditional (clamped addresses) and nothing
    // consumes a loaded value before compute.  A block past the last one
    // (the pipeline's tail) reads one line, the expert's first 16 bytes, on
    // every lane: reloading a block already computed fetched its lines from
    // HBM a second time (the streamed code lines have left L2 by then; the
    // down linear's 6 blocks on 4 waves had fetched 2.25 times its bytes).
    auto load_w = [&](int kb, Blk& b) {
        const bool live = kb < nkb;
        const int wi = min(kb * 16 + 4 * g, words_row - 4);
#pragma unroll
        for (int j = 0; j < TPW; ++j)
            b.w[j] = __builtin_nontemporal_load(
                live ? reinterpret_cast<const u32x4*>(qe + static_cast<size_t>(row[j]) * words_row + wi)
                     : reinterpret_cast<const u32x4*>(qe));
    };
    auto load_x = [&](int kb, Blk& b, const u32x4* xr) {
        const int wi = min(kb * 16 + 4 * g, words_row - 4);
#pragma unroll
        for (int t = 0; t < 4; ++t)
            b.x[t] = xr[GPB == 1 ? wi + t : (kb * 128 + 32 * t < K ? kb * 16 + 4 * t + g : g)];
    };
    // rank-term operands of the step at factor column kr: this lane's slot's
    // t (8 floats, zero past its rank) and the tiles' B entries
    struct RankOp {
        float t[8];
        uint32_t bw[TPW][4];
    };
    // 16-byte loads when every row of t and B starts 16-byte aligned (r_max a
    // multiple of 8: t rows of r_max floats in the 256-byte aligned
    // workspace, B rows of r_max halves); a step past r_max reads column 0
    const bool rvec = (L.r_max & 7) == 0 && (reinterpret_cast<uintptr_t>(L.B) & 15) == 0;
    auto rank_load = [&](int kr, int sl, RankOp& o) {
        const int k = kr + 8 * g;
        const float* trow = L.t + static_cast<size_t>(sl) * L.r_max;
        if (rvec) {
            const int kk = k + 8 <= L.r_max ? k : 0;
            const f32x4 t0 = *reinterpret_cast<const f32x4*>(trow + kk);
            const f32x4 t1 = *reinterpret_cast<const f32x4*>(trow + kk + 4);
#pragma unroll
            for (int q = 0; q < 4; ++q) { o.t[q] = t0[q]; o.t[4 + q] = t1[q]; }
#pragma unroll
            for (int j = 0; j < TPW; ++j) {
                const u32x4 v = *reinterpret_cast<const u32x4*>(Be + static_cast<size_t>(row[j]) * L.r_max + kk);
#pragma unroll
                for (int q = 0; q < 4; ++q) { const uint32_t vq = v[q]; o.bw[j][q] = vq; }
            }
            return;
        }
#pragma unroll
        for (int q = 0; q < 8; ++q) o.t[q] = trow[k + q < L.r_max ? k + q : 0];
#pragma unroll
        for (int j = 0; j < TPW; ++j) {
            const uint16_t* brow = Be + static_cast<size_t>(row[j]) * L.r_max;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int k0 = k + 2 * q, k1 = k0 + 1;
                const uint32_t lo = brow[k0 < L.r_max ? k0 : 0];
                const uint32_t hi = brow[k1 < L.r_max ? k1 : 0];
                o.bw[j][q] = lo | (hi << 16);
            }
        }
    };

    // What is needed first is issued first (vector loads complete in issue
    // order): the scales and zeros of the workgroup's rows, then this lane's
    // slot of the first pass, then the first round of code blocks; the LDS
    // copy of the scales and zeros then waits only for them, and the code
    // loads stay in flight across the barrier.  (Issued after the copy, the
    // code loads had one more dependent round trip per workgroup.)
    const int nval = min(16 * TPW, L.d_out - row0) * groups;
    const uint16_t* ssrc = se + static_cast<size_t>(row0) * groups;
    const uint16_t* zsrc = ze + static_cast<size_t>(row0) * groups;
    const int RS = szl_stride(groups);            // padded row stride of the tables
    uint16_t* zl = szl + 16 * TPW * RS;
    const bool al = ((reinterpret_cast<uintptr_t>(ssrc) | reinterpret_cast<uintptr_t>(zsrc)) & 15) == 0;
    const int n16 = al ? nval / 8 : 0;
    // table entry of the run's value i (row i / groups, column i % groups;
    // the identity on an unpadded table, where pieces may span rows)
    auto tix = [&](int i) { return RS == groups ? i : i / groups * RS + i % groups; };
    // first 16-byte piece of each array per thread (a valid aligned address
    // when this thread has none)
    const u32x4* s16p = n16 ? reinterpret_cast<const u32x4*>(ssrc) + min(tid, n16 - 1)
                            : reinterpret_cast<const u32x4*>(a.table);
    const u32x4* z16p = n16 ? reinterpret_cast<const u32x4*>(zsrc) + min(tid, n16 - 1)
                            : reinterpret_cast<const u32x4*>(a.table);
    const u32x4 s_first = *s16p, z_first = *z16p;
    int sl = a.sorted[sbeg + (r < scnt ? r : 0)];
    constexpr int SPAN = 4 * NBUF;
    const int rounds = (nkb + SPAN - 1) / SPAN;
    Blk b[NBUF];
#pragma unroll
    for (int j = 0; j < NBUF; ++j) load_w(wave + 4 * j, b[j]);
    if (tid < n16) {
        *reinterpret_cast<u32x4*>(szl + tix(8 * tid)) = s_first;
        *reinterpret_cast<u32x4*>(zl + tix(8 * tid)) = z_first;
    }
    for (int i = tid + 256; i < n16; i += 256) {           // rows with more than 32 groups
        *reinterpret_cast<u32x4*>(szl + tix(8 * i)) = reinterpret_cast<const u32x4*>(ssrc)[i];
        *reinterpret_cast<u32x4*>(zl + tix(8 * i)) = reinterpret_cast<const u32x4*>(zsrc)[i];
    }
    for (int i = 8 * n16 + tid; i < nval; i += 256) {      // misaligned runs, the last few values
        szl[tix(i)] = ssrc[i];
        zl[tix(i)] = zsrc[i];
    }
    __syncthreads();

    for (int p0 = 0; p0 < scnt; p0 += 16) {
        if (p0 > 0) {
            // a later pass of 16 slots: its slots and its first code round
            sl = a.sorted[sbeg + (p0 + r < scnt ? p0 + r : 0)];
#pragma unroll
            for (int j = 0; j < NBUF; ++j) load_w(wave + 4 * j, b[j]);
        }
        // this lane's slot (MFMA row r of the activations); absent slots read
        // a present one and are masked to zero
        const bool sv = p0 + r < scnt;
        const int xrow = a.x_per_slot ? sl : sl / a.k;
        const u32x4* xr = reinterpret_cast<const u32x4*>(a.xp + static_cast<size_t>(xrow) * (K / 2));
#pragma unroll
        for (int j = 0; j < NBUF; ++j) load_x(wave + 4 * j < nkb ? wave + 4 * j : 0, b[j], xr);
        // this lane's slot's rank: its own (per-slot ranks) or the expert's
        int rs = rank;
        if (L.slot_rank) {
            const int v = L.slot_rank[sl];
            rs = v < 0 ? 0 : (v > L.r_max ? L.r_max : v);
        }
        f32x4 acc[TPW];
#pragma unroll
        for (int j = 0; j < TPW; ++j) acc[j] = f32x4{0.f, 0.f, 0.f, 0.f};
        auto compute = [&](int kb, const Blk& bk) {
            // per group: MFMA steps into a fresh partial of sum (q - z) x,
            // then acc += s * partial in fp32; past K, past the matrix or a
            // padding block the scale is 0
            constexpr int SPG = 4 / GPB;
            u32x4 xv[4];
#pragma unroll
            for (int t = 0; t < 4; ++t) xv[t] = sv ? bk.x[t] : zero;
#pragma unroll
            for (int j = 0; j < TPW; ++j) {
                uint32_t w[4];
#pragma unroll
                for (int t = 0; t < 4; ++t) { const uint32_t v = bk.w[j][t]; w[t] = v; }
                if constexpr (GPB > 1) transpose_words(w);
#pragma unroll
                for (int q = 0; q < GPB; ++q) {
                    const int kc = kb * 128 + 32 * SPG * q;
                    const bool on = kb < nkb && kc < K && rowv[j];
                    const int lr = (16 * j + r) * RS + (on ? kc / a.G : 0);
                    const Zq zq = make_zq(szl[16 * TPW * RS + lr]);
                    f32x4 pp = mfma(xv[SPG * q], codes_minus_zero(w[SPG * q], zq, mlo, mhi, bias),
                                    f32x4{0.f, 0.f, 0.f, 0.f});
#pragma unroll
                    for (int t = SPG * q + 1; t < SPG * q + SPG; ++t)
                        pp = mfma(xv[t], codes_minus_zero(w[t], zq, mlo, mhi, bias), pp);
                    acc[j] = fma4(on ? f16_bits_to_f32(szl[lr]) : 0.f, pp, acc[j]);
                }
            }
        };
        for (int rd = 0; rd < rounds; ++rd) {
#pragma unroll
            for (int j = 0; j < NBUF; ++j) {
                const int kb = wave + SPAN * rd + 4 * j;
                compute(kb, b[j]);
                const int kn = kb + SPAN;
                load_w(kn, b[j]);
                load_x(kn < nkb ? kn : 0, b[j], xr);
            }
        }
        // rank-r term: 32 factor columns per step, wave w taking steps w, w + 4
        // (t as fp16 hi + lo parts, two MFMA steps; entries past the slot's
        // rank, past the expert's rank or of absent slots and rows are zero)
        auto rank_mma = [&](int kr, const RankOp& o) {
            const int k = kr + 8 * g;
            uint32_t tw[4], tlo[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int k0 = k + 2 * q, k1 = k0 + 1;
                split_f16x2((sv && k0 < rs) ? o.t[2 * q] : 0.f, (sv && k1 < rs) ? o.t[2 * q + 1] : 0.f, tw[q],
                            tlo[q]);
            }
#pragma unroll
            for (int j = 0; j < TPW; ++j) {
                uint32_t aw[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int k0 = k + 2 * q, k1 = k0 + 1;
                    const uint32_t lo = (rowv[j] && k0 < rank) ? (o.bw[j][q] & 0xffffu) : 0u;
                    const uint32_t hi = (rowv[j] && k1 < rank) ? (o.bw[j][q] >> 16) : 0u;
                    aw[q] = lo | (hi << 16);
                }
                const u32x4 bop = {aw[0], aw[1], aw[2], aw[3]};
                acc[j] = mfma(u32x4{tw[0], tw[1], tw[2], tw[3]}, bop, acc[j]);
                acc[j] = mfma(u32x4{tlo[0], tlo[1], tlo[2], tlo[3]}, bop, acc[j]);
            }
        };
        // (prefetching the first step's operands ahead of the K loop kept
        // them live through it: 256 VGPRs plus 72 AGPRs, one wave per SIMD)
        for (int kr = 32 * wave; kr < rank; kr += 128) {
            RankOp o2;
            rank_load(kr, sl, o2);
            rank_mma(kr, o2);
        }
#pragma unroll
        for (int j = 0; j < TPW; ++j) red[wave][j][lane] = acc[j];
        __syncthreads();
        // wave w sums and stores tiles w, w + 4, ... in a fixed order;
        // v[e] = y[slot of pass row 4 g + e][row0 + 16 j + r]
        int osl[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) osl[q] = __shfl(sl, 4 * g + q, 64);
#pragma unroll
        for (int j = 0; j < TPW; ++j) {
            if (j % 4 != wave || !rowv[j]) continue;
            const f32x4 v = red[0][j][lane] + red[1][j][lane] + red[2][j][lane] + red[3][j][lane];
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (p0 + 4 * g + q < scnt) store_out(L.y, static_cast<size_t>(osl[q]) * L.d_out + row[j], v[q], a.out);
        }
        __syncthreads();                           // red is reused by the next pass
    }
}

size_t up256(size_t n) { return (n + 255) / 256 * 256; }

struct MoeLayout {
    size_t n_active, table, sorted, t[kMaxMoeWin], xp, sx, h, total;
};

MoeLayout moe_layout(int n, const QW* w, const int* r_max, int E, int T, int k, int x_per_slot) {
    const int S = T * k;
    const int max_active = S < E ? S : E;
    const int rows = x_per_slot ? S : T;
    const size_t chunks = static_cast<size_t>(w[0].d_in) / (32 / w[0].bits) / 4;
    MoeLayout l;
    l.n_active = 0;
    l.table = 256;
    l.sorted = l.table + up256(static_cast<size_t>(max_active + S / 16) * kTab * sizeof(int));
    size_t off = l.sorted + up256(static_cast<size_t>(S) * sizeof(int));
    for (int i = 0; i < n; ++i) {
        l.t[i] = off;
        off += up256(static_cast<size_t>(S) * r_max[i] * sizeof(float));
    }
    l.xp = off;
    l.sx = l.xp + up256(static_cast<size_t>(rows) * w[0].d_in * 2);
    l.h = l.sx + up256(static_cast<size_t>(rows) * chunks * sizeof(float));
    // gated per-slot input (x_per_slot 2): SiLU(g) u of every slot in fp16
    l.total = l.h + (x_per_slot == 2 ? up256(static_cast<size_t>(S) * w[0].d_in * 2) : 0);
    return l;
}

template <int BITS, int CPL, int NB, int LG>
hipError_t launch_moe4(const MoeArgs& a, bool hoist, int blocks, int threads, hipStream_t st) {
    if (hoist)
        hipLaunchKernelGGL((moe_kernel<BITS, CPL, NB, true, LG>), dim3(blocks), dim3(threads), 0, st, a);
    else
        hipLaunchKernelGGL((moe_kernel<BITS, CPL, NB, false, LG>), dim3(blocks), dim3(threads), 0, st, a);
    return hipGetLastError();
}

template <int BITS, int LG>
hipError_t launch_moe3(const MoeArgs& a, int nb, bool hoist, int blocks, int threads, hipStream_t st) {
    switch (nb) {
        case 0: return launch_moe4<BITS, 1, 0, LG>(a, hoist, blocks, threads, st);
        case 1: return launch_moe4<BITS, 1, 1, LG>(a, hoist, blocks, threads, st);
        case 2: return launch_moe4<BITS, 1, 2, LG>(a, hoist, blocks, threads, st);
        default: return launch_moe4<BITS, 1, 4, LG>(a, hoist, blocks, threads, st);
    }
}

template <int BITS>
hipError_t launch_moe2(const MoeArgs& a, int lg, int nb, bool hoist, int blocks, int threads, hipStream_t st) {
    if (lg == 16) return launch_moe3<BITS, 16>(a, nb, hoist, blocks, threads, st);
    if (lg == 32) return launch_moe3<BITS, 32>(a, nb, hoist, blocks, threads, st);
    return launch_moe3<BITS, 64>(a, nb, hoist, blocks, threads, st);
}

// Eight waves per workgroup, each with half the row batches of four (the
// rows per workgroup unchanged): two waves per SIMD where four held one,
// and the t product's rank rows spread over twice the waves (48-layer
// T = 1 step 18.9 -> 16.7 us).  The gated instance keeps four: every wave
// forms SiLU(g) u for the whole activation row it converts, so eight
// waves doubled that work (down 9.4 -> 11.2 us).
template <int LG, int CPL, int QX, bool G>
hipError_t launch_direct4(const MoeArgs& a, int nb, int blocks, hipStream_t st) {
    constexpr int NWV = G ? 4 : 8;
    constexpr int NBW = direct_batches(LG, CPL) * 4 / NWV;
    const dim3 th(64 * NWV);
    if (nb == 0) hipLaunchKernelGGL((moe_direct_kernel<LG, CPL, 0, QX, NBW, G, NWV>), dim3(blocks), th, 0, st, a);
    else if (nb == 1) hipLaunchKernelGGL((moe_direct_kernel<LG, CPL, 1, QX, NBW, G, NWV>), dim3(blocks), th, 0, st, a);
    else hipLaunchKernelGGL((moe_direct_kernel<LG, CPL, 2, QX, NBW, G, NWV>), dim3(blocks), th, 0, st, a);
    return hipGetLastError();
}

template <int LG, int CPL, int QX>
hipError_t launch_direct3(const MoeArgs& a, int nb, int blocks, hipStream_t st) {
    return a.u ? launch_direct4<LG, CPL, QX, true>(a, nb, blocks, st)
               : launch_direct4<LG, CPL, QX, false>(a, nb, blocks, st);
}

// (LG, CPL, QX) instances: 24-32 chunk rows (d_in <= 1024), 64-chunk rows
// (d_in <= 2048), 128-chunk rows (d_in <= 4096)
hipError_t launch_direct(const MoeArgs& a, int lg, int cpl, int nb, int qx, int blocks, hipStream_t st) {
    if (lg == 32) return launch_direct3<32, 1, 2>(a, nb, blocks, st);
    if (cpl == 1 && qx <= 4) return launch_direct3<64, 1, 4>(a, nb, blocks, st);
    return launch_direct3<64, 2, 8>(a, nb, blocks, st);
}

template <int NBK, int KW>
hipError_t launch_stream2(const MoeArgs& a, int blocks, hipStream_t st) {
    constexpr int waves = KW > 4 ? KW : 4;
    const dim3 grid(blocks), block(64 * waves);
    const size_t lds = static_cast<size_t>(2) * waves * 256 * sizeof(float);
    if (a.G % 128 == 0)
        hipLaunchKernelGGL((moe_stream_kernel<NBK, 1, KW, kStreamDepth>), grid, block, lds, st, a);
    else
        hipLaunchKernelGGL((moe_stream_kernel<NBK, 2, KW, kStreamDepth>), grid, block, lds, st, a);
    return hipGetLastError();
}

// Whether a linear takes the streamed kernel.  It can where a workgroup's share of
// K fits (rows of at most 4096 codes in groups of a multiple of 64); it pays
// where a workgroup's start is spread over enough codes.  Times of captured
// calls (gate,up windows, single linears and gated calls; 16 to 160 experts, 9 to
// 512 slots, 512 to 4096 columns, even and skewed routing) against
// moe_mfma_kernel / moe_kernel:
//   experts in reach x columns >= 72 K: 0.60 to 1.05 of their time (96 experts
//   of 768 at 256 slots 0.84 to 0.95, 48 of 1536 0.93 to 0.95, 24 of 4096 0.77 to
//   0.90; but 24 of 4096 at 64 slots, 1.05 to 1.07).
//   below it the rows count as well: from 72 M codes in reach 0.80 to 1.02 (64
//   experts of 768 x 2048, 48 of 768 x 2048), with fewer up to 1.23 (64 of
//   1024 x 384) and 1.67 (40 of 512 x 192).
//   fewer than two slots an expert, rows of 1536 and more: 0.59 to 1.0 from 32
//   experts, 24 on long rows (the other kernel is the VALU's).  Groups of 64,
//   whose blocks carry two scales: 1.09 at 32 of 2048; on rows of 1024 1.05 to
//   1.14 with up to 128 experts of 1024 x 2048, 0.80 with 160.
// It reads one linear at a time, so that a window's outputs equal the single
// calls' (a window of both kinds goes in two parts).
bool stream_pays(const QW& w, int S, int experts) {
    if (w.bits != 4 || w.d_in > 4096 || w.G % 64 || experts < 24) return false;
    const bool half = w.G % 128 != 0, few = S < 2 * experts;
    const long long codes = static_cast<long long>(experts) * w.d_in * w.d_out;
    if (half && few && w.d_in > 768 && w.d_in < 1536) return codes >= 240 << 20;
    if (experts < 32 && !few && S < 5 * experts) return false;
    if (experts * w.d_in >= 72 << 10) return true;
    if (few && w.d_in >= 1536 && experts >= (half ? 40 : w.d_in >= 3072 ? 24 : 32)) return true;
    return experts >= 32 && codes >= 72 << 20;
}

// Rows of nkb 128-code blocks: the fewest waves that leave each at most four.
hipError_t launch_stream(const MoeArgs& a, int nkb, int blocks, hipStream_t st) {
    if (nkb > 16) return nkb <= 24 ? launch_stream2<3, 8>(a, blocks, st) : launch_stream2<4, 8>(a, blocks, st);
    if (nkb > 8) return nkb <= 12 ? launch_stream2<3, 4>(a, blocks, st) : launch_stream2<4, 4>(a, blocks, st);
    if (nkb > 4) return nkb <= 6 ? launch_stream2<3, 2>(a, blocks, st) : launch_stream2<4, 2>(a, blocks, st);
    return nkb <= 2 ? launch_stream2<2, 1>(a, blocks, st) : launch_stream2<4, 1>(a, blocks, st);
}

}  // namespace

bool moe_fits(const QW& w, int E, int T, int k) {
    // one chunk per lane over at most 8 K slices: d_in <= 16384 (4-bit), 32768 (2-bit)
    const int chunks = w.d_in / (32 / w.bits) / 4;
    return chunks <= 8 * 64 && E <= kMaxExperts && T * k <= kMaxSlots;
}

size_t moe_workspace_bytes(int n, const QW* w, const int* r_max, int E, int T, int k, int x_per_slot) {
    return moe_layout(n, w, r_max, E, T, k, x_per_slot).total;
}

hipError_t launch_moe_decode(int n, const QW* w, const uint16_t* const* A, const uint16_t* const* B,
                             const int* r_max, const int32_t* const* ranks, const int32_t* const* slot_ranks,
                             int E, const void* x, const void* u, int x_per_slot,
                             const int32_t* ids, int T, int k, int act, void* const* y, int out, void* ws,
                             hipStream_t st) {
    if (n < 1 || n > kMaxMoeWin) return hipErrorInvalidConfiguration;
    const int S = T * k;
    const int max_active = S < E ? S : E;
    // on or off the streamed kernel: a window of both kinds goes in two parts,
    // one after the other in the same workspace
    const bool stream = stream_pays(w[0], S, max_active);
    for (int other = 1; other < n; ++other) {
        if (stream_pays(w[other], S, max_active) == stream) continue;
        for (const bool part : {stream, !stream}) {
            QW pw[kMaxMoeWin];
            const uint16_t *pA[kMaxMoeWin], *pB[kMaxMoeWin];
            const int32_t *pr[kMaxMoeWin], *ps[kMaxMoeWin];
            int pm[kMaxMoeWin], m = 0;
            void* py[kMaxMoeWin];
            for (int i = 0; i < n; ++i) {
                if (stream_pays(w[i], S, max_active) != part) continue;
                pw[m] = w[i]; pA[m] = A[i]; pB[m] = B[i]; pm[m] = r_max[i]; pr[m] = ranks[i];
                ps[m] = slot_ranks ? slot_ranks[i] : nullptr;
                py[m++] = y[i];
            }
            const hipError_t e = launch_moe_decode(m, pw, pA, pB, pm, pr, slot_ranks ? ps : nullptr, E, x, u,
                                                   x_per_slot, ids, T, k, act, py, out, ws, st);
            if (e != hipSuccess) return e;
        }
        return hipSuccess;
    }
    const MoeLayout l = moe_layout(n, w, r_max, E, T, k, x_per_slot);
    char* wsb = static_cast<char*>(ws);
    const int d_in = w[0].d_in, bits = w[0].bits;
    MoeArgs a{};
    a.n = n;
    a.ids = ids;
    a.x = static_cast<const uint16_t*>(x);
    a.u = static_cast<const uint16_t*>(u);
    a.E = E; a.T = T; a.k = k; a.d_in = d_in; a.G = w[0].G;
    a.act = act; a.out = out; a.x_per_slot = x_per_slot ? 1 : 0;
    a.n_active = reinterpret_cast<int*>(wsb + l.n_active);
    a.table = reinterpret_cast<int*>(wsb + l.table);
    a.sorted = reinterpret_cast<int*>(wsb + l.sorted);
    a.xp = reinterpret_cast<f16x2*>(wsb + l.xp);
    a.sx = reinterpret_cast<float*>(wsb + l.sx);
    // K split as in the dense decode: one chunk per lane, a power-of-two
    // number of slices (at most 8, which moe_fits guarantees)
    const int chunks = d_in / (32 / bits) / 4;
    int ks = (chunks + 63) / 64;
    while (ks & (ks - 1)) ++ks;
    a.ks = ks;
    a.cps = (chunks + a.ks - 1) / a.ks;
    // lanes per row set: rows shorter than 64 chunks share a wave between
    // 2 or 4 row sets (one K slice)
    int rmax = 0;
    for (int i = 0; i < n; ++i) rmax = max(rmax, r_max[i]);
    int lg = chunks <= 16 ? 16 : (chunks <= 32 ? 32 : 64);
    if (rmax > 4 * lg) lg = 64;                    // at most 4 factor columns per lane
    const int sets = 64 / lg;
    const int threads = 64 * (a.ks > 4 ? a.ks : 4);
    if (a.ks > 8 || threads > 512 || threads % (64 * a.ks)) return hipErrorInvalidConfiguration;
    if (lg < 64 && a.ks != 1) return hipErrorInvalidConfiguration;
    const int rg_per_block = threads / 64 / a.ks * sets;
    // experts meeting two or more slots on average: 4-bit codes go to MFMA
    // (tiles of 16 rows), 2-bit codes are unpacked once per batch
    const bool many = S >= 2 * max_active;
    const bool on_mfma = many && bits == 4;
    const int nkb = (d_in + 127) / 128;
    a.split = stream;
    // Rank rows per preparation workgroup: 16 where that gives most CUs one,
    // fewer where it would leave them idle (a workgroup streams its rows of
    // A_e at one CU's share of the memory rate): 16 experts, 2048 x 768, rank 32:
    // a layer 39.8 us with 16 rows, 38.7 with 4; 128 experts, 64 slots: 64.3 with
    // 16, 67.1 with 4.  Gated calls repeat SiLU(g) u per workgroup, so they go
    // to fewer rows later.
    int wide = 0;
    for (int i = 0; i < n; ++i) wide += max_active * ((r_max[i] + 15) / 16);
    a.rr = a.u && d_in <= kGateFuseMaxWidth ? (wide > 32 ? 16 : 4) : (wide >= 192 ? 16 : wide >= 96 && d_in <= 2048 ? 8 : 4);
    int prep_end = 0, blk_end = 0;
    for (int i = 0; i < n; ++i) {
        MoeLin& L = a.lin[i];
        L.q = w[i].q; L.s = w[i].s; L.z = w[i].z; L.A = A[i]; L.B = B[i]; L.ranks = ranks[i];
        L.slot_rank = slot_ranks ? slot_ranks[i] : nullptr;
        L.y = y[i];
        L.t = reinterpret_cast<float*>(wsb + l.t[i]);
        L.q_stride = static_cast<size_t>(w[i].d_out) * (d_in / (32 / bits));
        L.sz_stride = static_cast<size_t>(w[i].d_out) * (d_in / w[i].G);
        L.a_stride = static_cast<size_t>(r_max[i]) * d_in;
        L.b_stride = static_cast<size_t>(w[i].d_out) * r_max[i];
        L.d_out = w[i].d_out;
        L.r_max = r_max[i];
        L.rq = r_max[i] > 0 ? (r_max[i] + a.rr - 1) / a.rr : 1;
        const int rgroups = (w[i].d_out + rows_per_wave(bits) - 1) / rows_per_wave(bits);
        L.bpe = stream ? (w[i].d_out + 15) / 16
                       : on_mfma ? (w[i].d_out + 16 * kMoeTpw - 1) / (16 * kMoeTpw)
                                 : (rgroups + rg_per_block - 1) / rg_per_block;
        prep_end += max_active * L.rq;
        blk_end += stream ? L.bpe : max_active * L.bpe;       // streamed: tiles per expert
        L.prep_end = prep_end;
        L.blk_end = blk_end;
    }
    // few slots, 4-bit codes, rows of at most 4096 codes: the direct path
    // (one launch, no preparation, no workspace)
    const int dlg = chunks <= 32 ? 32 : 64;
    const int dcpl = (chunks + dlg - 1) / dlg;
    if (bits == 4 && S <= kDirectMaxSlots && dcpl <= 2 && rmax <= 2 * dlg) {
        a.rb = 16 * (64 / dlg) * direct_batches(dlg, dcpl);
        int nrbm = 0;
        for (int i = 0; i < n; ++i) {
            MoeLin& L = a.lin[i];
            L.nrb = (w[i].d_out + a.rb - 1) / a.rb;
            nrbm = max(nrbm, L.nrb);
        }
        a.nrbm = nrbm;
        const int dblk = 8 * ((n * S + 7) / 8) * nrbm;
        const int dnb = rmax == 0 ? 0 : (rmax <= dlg ? 1 : 2);
        const int qx = d_in <= 1024 ? 2 : (d_in <= 2048 ? 4 : 8);
        return launch_direct(a, dlg, dcpl, dnb, qx, dblk, st);
    }
    const int per = lg * a.ks;                     // factor columns per lane pass
    const int nb = rmax == 0 ? 0 : (rmax <= per ? 1 : (rmax <= 2 * per ? 2 : 4));
    if (rmax > 4 * per) return hipErrorInvalidConfiguration;

    if (a.u && d_in > kGateFuseMaxWidth) {
        uint16_t* h = reinterpret_cast<uint16_t*>(wsb + l.h);
        const size_t n8 = static_cast<size_t>(S) * d_in / 8;
        hipLaunchKernelGGL(moe_gate_kernel, dim3(static_cast<unsigned>((n8 + 255) / 256)), dim3(256), 0, st, a.x, a.u,
                           h, n8, a.act);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        a.x = h;
        a.u = nullptr;
        a.act = DT_FP16;
    }
    const int rows = x_per_slot ? S : T;
    const long long items = static_cast<long long>(rows) * chunks;
    const unsigned pgrid = static_cast<unsigned>(prep_end + (items + 255) / 256);
    const size_t plds = static_cast<size_t>(2 * S + 2 * E) * sizeof(int);
    auto prep = bits == 4 ? (a.u ? moe_prep_kernel<4, true> : moe_prep_kernel<4, false>)
                          : (a.u ? moe_prep_kernel<2, true> : moe_prep_kernel<2, false>);
    hipLaunchKernelGGL(prep, dim3(pgrid), dim3(256), plds, st, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (stream) {
        const int blocks = static_cast<int>(min(static_cast<long long>(nkb > 16 ? kStreamBlocks / 2 : kStreamBlocks),
                                                static_cast<long long>(max_active) * blk_end));
        return launch_stream(a, nkb, blocks, st);
    }
    if (on_mfma) {
        const size_t lds = static_cast<size_t>(2) * 16 * kMoeTpw * szl_stride(d_in / w[0].G) * 2;
        // quantization groups a 128-code block can meet (see the kernel)
        const int G = w[0].G;
        if (G % 128 == 0)
            hipLaunchKernelGGL((moe_mfma_kernel<kMoeTpw, kMoeNbuf, 1>), dim3(blk_end), dim3(256), lds, st, a);
        else if (G % 64 == 0)
            hipLaunchKernelGGL((moe_mfma_kernel<kMoeTpw, 1, 2>), dim3(blk_end), dim3(256), lds, st, a);
        else
            hipLaunchKernelGGL((moe_mfma_kernel<kMoeTpw, 1, 4>), dim3(blk_end), dim3(256), lds, st, a);
        return hipGetLastError();
    }
    return bits == 4 ? launch_moe2<4>(a, lg, nb, many, blk_end, threads, st)
                     : launch_moe2<2>(a, lg, nb, many, blk_end, threads, st);
}

hipError_t moe_take_routing_error(hipStream_t st, unsigned long long* word) {
    unsigned long long v = 0;
    hipError_t e = hipMemcpyFromSymbolAsync(&v, HIP_SYMBOL(moe_routing_error), sizeof(v), 0,
                                            hipMemcpyDeviceToHost, st);
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    if (e == hipSuccess && v) {
        const unsigned long long zero = 0;
        e = hipMemcpyToSymbolAsync(HIP_SYMBOL(moe_routing_error), &zero, sizeof(zero), 0, hipMemcpyHostToDevice,
                                   st);
        if (e == hipSuccess) e = hipStreamSynchronize(st);
    }
    *word = v;
    return e;
}

}  // namespace cl
