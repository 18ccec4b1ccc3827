// The un-predicted projection of plans whose rows can wait for their selection on the chip (FILTER and unconstrained
// layers): a workgroup keeps its rows' candidate and kept-form dual in registers, publishes their keys, and writes every
// row once, in its final form and with its packed copy, when the layer's selection is known.  The workgroup that finds all
// of a layer's keys published makes the selection (Eq. (10)); nothing is read or written twice.
// Part of the single translation unit built from hsadmm.hip (included there, in order).
#ifndef KERNELS_HELD_HPP
#define KERNELS_HELD_HPP
#include "hsadmm_device.hpp"
#include "kernels_project.hpp"
#include "kernels_select.hpp"
#include "kernels_hinted.hpp"
#include "kernels_weighted.hpp"

namespace {

// What bounds it: HBM traffic (R + 3 arenas and the packed rows, the bytes the step cannot do without), and below that
// the time rows spend on the chip: a layer's first rows wait for its last, then about 7 us for keys to arrive, tags to be
// looked at, the selection (3 to 5 us) and the ranks to come back.  Meanwhile other workgroups load, so the more elements
// the chip holds the better: four workgroups a compute unit, each ten slots of 1024 elements, the candidate in 40 registers a
// thread, the dual in 32 KB of LDS and 8 registers (10 M elements on 256 units).  ResNet-50, 4 replicas, a step: eight slots all
// in registers 178 us, ten of them on three workgroups 178, twelve on three 198, twenty on two 198; with LDS ten on four
// 162, twelve 168 to 173, sixteen on three 206, twenty-four on two 179.  Before (pass 1, selection, fix-up and packing) / now:
// ResNet-50, 4 replicas 183 / 159; ResNet-18, 1 replica 77.7 / 61.2; of width 45, 3 replicas 60.8 / 47; a plain network
// of width 16 21.0 / 15.4.
constexpr int kHeldSlots = 10;           // 128-bit chunks a thread holds
constexpr int kHeldLdsSlots = 8;         // ... the duals of the first ones in LDS, the others' in registers
constexpr int kHeldPerUnit = 4;          // workgroups on a compute unit at once (as many waves on each of its SIMDs)
// Slots whose loads are in flight together.  Four with a run-time replica count (a plain network of width 200, 6 replicas: 56
// us with two, 53 with four); eight replicas one, as two spill (ResNet-152: 396 / 418 us).
constexpr int held_batch(int R) { return R <= 2 ? 4 : R == 8 ? 1 : 2; }
constexpr int kHeldRows = kBlock;        // rows of an item, at most
constexpr int kNotSelected = INT32_MIN;  // a group's rank before its layer's selection
// How long a workgroup waits for its layer's selection, in ticks of the 100 MHz clock: 300 us, six times what was seen.  The
// wait ends by itself once every workgroup of the layer has found a place on the chip; other streams' work may hold the
// places, and such work may be waiting in the same way, so after this long the rows are written as they stand (either outcome
// can be finished from that form) and the place is given up.
constexpr long long kHeldPatience = 30000;

// WorkItem fields of a held row item: aux = index of the layer's first held item | items of the layer << 32; khw = chunks
// (slots) of a thread per row.
struct HeldArgs {
    unsigned long long* tag;        // per held item: gen once the item's keys are published
    unsigned long long* state;      // per held item: who finishes its rows if they were written too early (held_finish_early)
    unsigned long long gen;         // this call's number; neither it nor the three after it are any other call's, or a value
                                    // that anything else writes there
    long long patience;             // ticks
    const DevLayer* layers;
    uint8_t* mask;
    IndexMaps im;
    CopyOut co;                     // the caller's layer_off / kept_idx (nulls: no compaction)
    float* packed;                  // null: no compaction
    int n_layers, pack_align;
};

// What the threads of a workgroup tell each other about rows written too early.
struct HeldTurn {
    unsigned long long early[kWaves];
    unsigned long long was;
};

// LDS: slots whose dual waits here.
template <int LDS>
struct HeldShared {
    v4f dual[LDS][kBlock];
    TopkShared topk;
    double wsum[kHeldSlots][kWaves];
    int rank[kHeldRows];
    HeldTurn turn;
};

// Called by the whole workgroup when all keys of the item's rows have been stored by put_agent.  Publishes the item and
// returns whether all items of its layer are published now (two workgroups that finish together may both be told so).
// A store has arrived before the tags are looked at, so the one whose store arrives last sees all the others'.
__device__ __forceinline__ bool held_publish(const WorkItem& it, const HeldArgs& h)
{
    if (threadIdx.x == 0) put_agent(&h.state[blockIdx.x], h.gen);
    stores_arrived();
    __syncthreads();
    if (threadIdx.x == 0) {
        put_agent(&h.tag[blockIdx.x], h.gen);
        stores_arrived();
    }
    __syncthreads();
    const int first = (int)(it.aux & 0xffffffffll), n = (int)(it.aux >> 32);
    bool ok = true;
    for (int k = threadIdx.x; k < n; k += kBlock) ok = ok && get_agent(&h.tag[first + k]) == h.gen;
    return __syncthreads_and(ok) != 0;
}

// The selection of the item's layer by this workgroup, with everything a later kernel or the caller reads of it.
__device__ __forceinline__ void held_select(const WorkItem& it, const HeldArgs& h, const double* key, TopkShared& topk)
{
    const DevLayer& L = h.layers[it.layer];
    const int G = L.G, first = L.group_base, kk = L.k;
    int32_t* pos_l = h.im.pos + first;
    int32_t* sel_l = h.im.sel ? h.im.sel + first : nullptr;
    int32_t* kidx_l = h.im.kept_idx + L.kept_start;
    int32_t* ck_l = h.co.kept_idx ? h.co.kept_idx + L.kept_start : nullptr;
    uint8_t* ml = h.mask + first;
    const unsigned long long* kb = reinterpret_cast<const unsigned long long*>(key + first);
    if (kk >= G) {
        for (int g = threadIdx.x; g < G; g += kBlock) {
            ml[g] = 1; kidx_l[g] = g;
            put_agent(&pos_l[g], g);
            if (sel_l) sel_l[g] = g;
            if (ck_l) ck_l[g] = g;
        }
    } else if (G <= kTopkRegs * kBlock) {
        topk_layer<true, kBlock, true>(G, kb, ml, kk, topk, pos_l, kidx_l, sel_l, ck_l);
    } else {
        topk_layer<false, kBlock, true>(G, kb, ml, kk, topk, pos_l, kidx_l, sel_l, ck_l);
    }
}

// The layer's entries of the index mappings that the plan alone decides.
__device__ __forceinline__ void held_layer_entries(const WorkItem& it, const HeldArgs& h)
{
    const int l = it.layer;
    const DevLayer& L = h.layers[l];
    const int c0 = (L.mode == HSADMM_MODE_NONE) ? L.G : L.k;
    h.im.cnt[l] = c0;
    h.im.cnt[h.n_layers + l] = L.kept_start;
    h.im.cnt[2 * h.n_layers + l] = 0;
    h.im.layer_off[l] = L.packed_off;
    if (h.co.layer_off) h.co.layer_off[l] = L.packed_off;
    if (l == h.n_layers - 1) {
        const int64_t end = L.packed_off + packed_size(L.mode, L.unit, c0, 0, h.pack_align);
        h.im.layer_off[h.n_layers] = end;
        if (h.co.layer_off) h.co.layer_off[h.n_layers] = end;
    }
}

// Waits for the ranks of n groups (a thread each) from group g0 on -> rank (-1: pruned); false if the patience ran out first.
// Behind it the ranks that this workgroup has stored have arrived, if it has selected.
__device__ __forceinline__ bool held_wait_groups(int g0, int n, const HeldArgs& h, int* rank)
{
    const int t = threadIdx.x;
    int r = -1;
    if (t < n) {
        const long long until = (long long)__builtin_amdgcn_s_memrealtime() + h.patience;
        for (;;) {
            r = get_agent(&h.im.pos[g0 + t]);
            if (r != kNotSelected || (long long)__builtin_amdgcn_s_memrealtime() > until) break;
            __builtin_amdgcn_s_sleep(8);
        }
        rank[t] = r;
    }
    stores_arrived();
    return __syncthreads_or(t < n && r == kNotSelected) == 0;
}

// Rows that were written before their selection was known.
//
// An item's state word says who finishes them.  It is gen before the item's keys are published and then only gains bits: the
// item's workgroup adds 2 once its rows lie in memory in their early form, a workgroup that has made the layer's selection adds
// 1 once the ranks lie there.  The item's workgroup finishes what has a 1 before its 2, the first to add a 1 what has a 2.
// Nobody waits for anybody, so there is nothing to give up, however long other work keeps a layer's last workgroups off the
// chip.  (Two workgroups may both have selected: the second finds the first's 1.)
__device__ __forceinline__ unsigned long long gain_agent(unsigned long long* p, unsigned long long bit)
{
    return __hip_atomic_fetch_or(p, bit, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Called by the whole workgroup behind its own rows.  early: it has stored them in their early form; n: items of its layer, from the
// first one on, if it has made their selection, else 0.  What is to be finished by it goes to finish.  (Told that this
// is rare, the compiler spills for this code and not for the loads.  Plain network of width 24, channel groups, 1, 4, 8 replicas,
// us, not told / told: 26.6 / 26.3, 31.3 / 29.6, 37.0 / 33.2.)
template <typename F>
__device__ __forceinline__ void held_finish_early(const WorkItem* __restrict__ items, const HeldArgs& h, bool early, int first, int n,
                                                  HeldTurn& turn, F finish)
{
    if (__builtin_expect(!early && n == 0, 1)) return;
    for (int k0 = early ? -kBlock : 0; k0 < n; k0 += kBlock) {
        const bool own = k0 < 0;
        if (own) {
            __threadfence();
            __syncthreads();
            if (threadIdx.x == 0) turn.was = gain_agent(&h.state[blockIdx.x], 2ull);
            __syncthreads();
        }
        const int k = k0 + (int)threadIdx.x;
        const bool mine = own ? threadIdx.x == 0 && (turn.was & 1ull) != 0ull
                              : k < n && gain_agent(&h.state[first + k], 1ull) == h.gen + 2ull;
        const unsigned long long b = __ballot(mine);
        if ((threadIdx.x & (kWave - 1)) == 0) turn.early[threadIdx.x / kWave] = b;
        if (__builtin_expect(__syncthreads_or(mine) == 0, 1)) continue;
        __threadfence();                                         // the rows as their workgroups left them
        for (int w = 0; w < kWaves; ++w) {
            unsigned long long m = turn.early[w];
            unsigned int lo = __builtin_amdgcn_readfirstlane((unsigned int)m), hi = __builtin_amdgcn_readfirstlane((unsigned int)(m >> 32));
            for (m = ((unsigned long long)hi << 32) | lo; m != 0ull; m &= m - 1ull)
                finish(items[own ? (int)blockIdx.x : first + k0 + w * kWave + __builtin_ctzll(m)]);
        }
        __syncthreads();                                         // (the masks may be written again)
    }
}

// Where the slots of a thread lie in a row item; the last floats of a ragged row lie in the slot behind its words, one to a
// lane.  WHOLE: no row has a tail (a choice made per slot would have loads wait for each other).
template <bool WHOLE>
struct HeldPlaces {
    int64_t base;
    int nr, row_len, nchunk, lpr, rows_at_once, sub, j, cpr, tail_slot, nslot;
    bool wide;
    __device__ __forceinline__ explicit HeldPlaces(const WorkItem& it)
    {
        base = it.base;
        nr = it.nr;
        row_len = it.row_len;
        nchunk = row_len >> 2;
        wide = it.lpr > kWave;
        lpr = wide ? kBlock : it.lpr;
        rows_at_once = kBlock / lpr;
        sub = threadIdx.x / lpr;
        j = threadIdx.x - sub * lpr;
        cpr = it.khw;                                            // slots per row
        tail_slot = WHOLE ? cpr : cpr - 1;
        nslot = cpr * ((nr + rows_at_once - 1) / rows_at_once);
    }
    __device__ __forceinline__ int row(int rd) const { return rd * rows_at_once + sub; }
    __device__ __forceinline__ v4f fetch(const float* p, int q, int rd) const
    {
        v4f x = {0.f, 0.f, 0.f, 0.f};
        if (row(rd) < nr) {
            const float* r = p + base + (int64_t)row(rd) * row_len;
            if (WHOLE || q != tail_slot) {
                const int c = j + q * lpr;
                if (c < nchunk) x = ld4(r + 4 * c);
            } else if (j < (row_len & 3)) {
                x.x = ld1(r + 4 * nchunk + j);
            }
        }
        return x;
    }
    __device__ __forceinline__ void put(float* p, int q, int rd, const v4f& x) const
    {
        if (row(rd) >= nr) return;
        float* r = p + base + (int64_t)row(rd) * row_len;
        if (WHOLE || q != tail_slot) {
            const int c = j + q * lpr;
            if (c < nchunk) st4(r + 4 * c, x);
        } else if (j < (row_len & 3)) {
            st1(r + 4 * nchunk + j, x.x);
        }
    }
    // the same into a packed row, which may begin at any float
    __device__ __forceinline__ void put_packed(float* r, int q, const v4f& x) const
    {
        if (WHOLE || q != tail_slot) {
            const int c = j + q * lpr;
            if (c < nchunk) st4u(r + 4 * c, x);
        } else if (j < (row_len & 3)) {
            r[4 * nchunk + j] = x.x;
        }
    }
};

// The early form of a row: the kept one where most of the layer is kept, else the pruned one with the kept form's dual in Z.
__device__ __forceinline__ bool held_early_kept(const DevLayer& L) { return 2 * L.k >= L.G; }

// From its early to its final form.
template <bool WHOLE>
__device__ __forceinline__ void held_rows_finish(const WorkItem& it, const ProjectArgs& a, const HeldArgs& h)
{
    constexpr int B = 5;                                         // slots whose loads are in flight together
    const HeldPlaces<WHOLE> at(it);
    const v4f zero4 = {0.f, 0.f, 0.f, 0.f};
    const bool kept_form = held_early_kept(h.layers[it.layer]);
    float* const pk_layer = h.packed ? h.packed + it.packed_off : nullptr;
    int q = 0, rd = 0;
    for (int s0 = 0; s0 < at.nslot; s0 += B) {
        v4f z[B], u[B];
        int qb[B], rb[B], rank[B];
#pragma unroll
        for (int i = 0; i < B; ++i) {
            qb[i] = q; rb[i] = s0 + i < at.nslot ? rd : it.nr;   // (no such row)
            if (++q == at.cpr) { q = 0; ++rd; }
            const int row = at.row(rb[i]);
            rank[i] = row < it.nr ? get_agent(&h.im.pos[it.g0 + row]) : -1;
            z[i] = at.fetch(a.Z, qb[i], rb[i]);
            u[i] = kept_form ? zero4 : at.fetch(a.U, qb[i], rb[i]);
        }
#pragma unroll
        for (int i = 0; i < B; ++i) {
            const bool kept = rank[i] >= 0;
            const v4f v = kept_form ? z[i] : u[i];               // the candidate
            if (!kept) at.put(a.Z, qb[i], rb[i], zero4);
            else if (!kept_form) at.put(a.Z, qb[i], rb[i], v);
            if (kept != kept_form) at.put(a.U, qb[i], rb[i], z[i]);
            if (kept && pk_layer) at.put_packed(pk_layer + (int64_t)rank[i] * it.row_len, qb[i], v);
        }
    }
}

// One FILTER row item.
template <int R, bool WHOLE, typename SHARED>
__device__ __forceinline__ void held_rows(const WorkItem* __restrict__ items, const WorkItem& it, const ProjectArgs& a, int Rrt, const HeldArgs& h, SHARED& sh)
{
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = threadIdx.x / kWave;
    const HeldPlaces<WHOLE> at(it);
    const v4f zero4 = {0.f, 0.f, 0.f, 0.f};
    if (threadIdx.x < it.nr) put_agent(&h.im.pos[it.g0 + threadIdx.x], (int32_t)kNotSelected);
    v4f V[kHeldSlots];                                           // the candidate
    v4f D[kHeldSlots > kHeldLdsSlots ? kHeldSlots - kHeldLdsSlots : 1];   // the dual of a kept group (the first slots': in LDS)
    {
        constexpr int B = held_batch(R);
        int q = 0, rd = 0;
        double acc = 0.0;
#pragma unroll
        for (int s0 = 0; s0 < kHeldSlots; s0 += B)
            if (s0 < at.nslot) {
                v4f w[B], u[B];
                int qb[B], rb[B];
#pragma unroll
                for (int i = 0; i < B; ++i) {
                    qb[i] = q; rb[i] = s0 + i < at.nslot ? rd : it.nr;   // (no such row)
                    if (++q == at.cpr) { q = 0; ++rd; }
                }
#pragma unroll
                for (int i = 0; i < B; ++i) {
                    w[i] = at.fetch(a.W[0], qb[i], rb[i]);
                    u[i] = at.fetch(a.Ur, qb[i], rb[i]);
                }
                if (R > 1) {
                    v4f x[B][R > 1 ? R - 1 : 1];
#pragma unroll
                    for (int i = 0; i < B; ++i)
#pragma unroll
                        for (int r = 1; r < R; ++r) x[i][r - 1] = at.fetch(a.W[r], qb[i], rb[i]);
#pragma unroll
                    for (int i = 0; i < B; ++i)
#pragma unroll
                        for (int r = 1; r < R; ++r) w[i] = w[i] + x[i][r - 1];
                } else if (R == 0) {
                    for (int r = 1; r < Rrt; ++r) {
                        v4f x[B];
#pragma unroll
                        for (int i = 0; i < B; ++i) x[i] = at.fetch(a.W[r], qb[i], rb[i]);
#pragma unroll
                        for (int i = 0; i < B; ++i) w[i] = w[i] + x[i];
                    }
                }
#pragma unroll
                for (int i = 0; i < B; ++i) {
                    const int s = s0 + i;
                    if (s >= kHeldSlots) continue;               // (no such slot: nothing was fetched for it either)
                    const v4f wb = w[i] * a.inv_R;
                    const v4f v = wb + u[i];
                    const v4f d = u[i] + (wb - v);
                    V[s] = v;
                    if (s < kHeldLdsSlots) sh.dual[s][threadIdx.x] = d;
                    else D[s - kHeldLdsSlots] = d;
                    if (a.Wbar) at.put(a.Wbar, qb[i], rb[i], wb);
                    acc = sq4(acc, v);                           // (lanes without an element add zeros)
                    if (s < at.nslot && qb[i] == at.cpr - 1) {   // the row is complete
                        if (!at.wide) {
                            acc = wave_xor_sum(acc, at.lpr);
                            const int row = at.row(rb[i]);
                            if (at.j == 0 && row < it.nr) put_agent(&a.key[it.g0 + row], acc);
                        } else {
                            acc = wave_xor_sum(acc, kWave);
                            if (lane == 0) sh.wsum[rb[i]][wave] = acc;
                        }
                        acc = 0.0;
                    }
                }
            }
    }
    if (at.wide) {
        __syncthreads();
        if (threadIdx.x < it.nr) {
            double s = sh.wsum[threadIdx.x][0];
            for (int w = 1; w < kWaves; ++w) s += sh.wsum[threadIdx.x][w];
            put_agent(&a.key[it.g0 + threadIdx.x], s);
        }
    }
    const bool selects = held_publish(it, h);
    if (selects) held_select(it, h, a.key, sh.topk);
    const bool known = held_wait_groups(it.g0, it.nr, h, sh.rank);
    const bool kept_default = held_early_kept(h.layers[it.layer]);
    float* const pk_layer = (h.packed && known) ? h.packed + it.packed_off : nullptr;
    int q = 0, rd = 0;
#pragma unroll
    for (int s = 0; s < kHeldSlots; ++s) {
        if (s < at.nslot) {
            const int row = at.row(rd);
            if (row < it.nr) {
                const int rank = known ? sh.rank[row] : (kept_default ? 0 : -1);
                const bool kept = rank >= 0;
                const v4f d = s < kHeldLdsSlots ? sh.dual[s][threadIdx.x] : D[s < kHeldLdsSlots ? 0 : s - kHeldLdsSlots];
                const v4f z = kept ? V[s] : (known ? zero4 : d);
                at.put(a.Z, q, rd, z);
                at.put(a.U, q, rd, kept ? d : V[s]);
                if (pk_layer && kept) at.put_packed(pk_layer + (int64_t)rank * it.row_len, q, z);
            }
            if (++q == at.cpr) { q = 0; ++rd; }
        }
    }
    held_finish_early(items, h, !known, (int)(it.aux & 0xffffffffll), selects ? (int)(it.aux >> 32) : 0, sh.turn,
                      [&](const WorkItem& x) { held_rows_finish<WHOLE>(x, a, h); });   // (a layer's rows are of one length)
}

// The mappings of an unconstrained layer's rows: always kept, packed at their own index.
__device__ __forceinline__ void held_none_entries(const WorkItem& it, const HeldArgs& h)
{
    for (int rr = threadIdx.x; rr < it.nr; rr += kBlock) {
        const int g = it.g0 + rr, row = it.row0 + rr;
        const int k = h.layers[it.layer].kept_start + row;
        h.mask[g] = 1;
        h.im.pos[g] = row;
        h.im.kept_idx[k] = row;
        if (h.im.sel) h.im.sel[g] = row;
        if (h.co.kept_idx) h.co.kept_idx[k] = row;
    }
}

template <int R>
__global__ __launch_bounds__(kBlock, kHeldPerUnit) void project_held(const WorkItem* __restrict__ items, ProjectArgs a, int Rrt,
                                                          HeldArgs h)
{
    __shared__ HeldShared<kHeldLdsSlots> sh;
    const WorkItem it = items[blockIdx.x];
    if (it.row0 == 0 && threadIdx.x == 0) held_layer_entries(it, h);
    if (item_mode(it) == HSADMM_MODE_NONE) {                     // final at once
        const HintArgs hint{nullptr, h.packed, 0, nullptr, h.layers};
        held_none_entries(it, h);
        project_rows_hinted<R, R != 8>(it, a, Rrt, hint);        // (one chunk at a time with eight replicas: no registers to spare)
    } else {
        if (item_vec(it)) held_rows<R, true>(items, it, a, Rrt, h, sh);
        else held_rows<R, false>(items, it, a, Rrt, h, sh);
    }
}

// ------------------------------------------------------------------ the full candidate of Eq. (9)

// What the weighted forms need beside HeldArgs.
struct HeldWeighted {
    const float* Zg;
    const float* Vd;
    const float* coef;
};

// Three values a slot wait, two of them in registers, so three workgroups share a unit.  Weighted steps of ResNet-50, us, in two
// launches that touch Z, U and the kept rows' z and v twice / in this one: 303 / 271 with 4 replicas; ResNet-152 with 8
// 641 / 587; a plain network of width 100 with 1, 4, 8 replicas 34.2 / 31.4, 36.8 / 35.2, 53.8 / 43.0.  (The residual norms
// on the way need the replicas' values until z~ is known: ResNet-50 350 / 341 us, but ResNet-18 of width 45 with 3 replicas
// 130 / 137 and a plain network of width 128 with 8 57 / 66.  They keep the other path.)
constexpr int kHeldWeightedPerUnit = 3;
constexpr int kHeldWeightedLds = kHeldSlots;
constexpr int held_weighted_batch(int R) { return R == 8 ? 1 : 2; }

// From the early form, t in Z and the dual of a kept row in U, to the final one.
template <bool WHOLE>
__device__ __forceinline__ void held_weighted_finish(const WorkItem& it, const ProjectArgs& a, const HeldArgs& h,
                                                     const HeldWeighted& x)
{
    constexpr int B = 5;                                         // slots whose loads are in flight together
    const HeldPlaces<WHOLE> at(it);
    const float al = x.coef[2 * it.layer], bl = x.coef[2 * it.layer + 1];
    const v4f zero4 = {0.f, 0.f, 0.f, 0.f};
    float* const pk_layer = h.packed ? h.packed + it.packed_off : nullptr;
    int q = 0, rd = 0;
    for (int s0 = 0; s0 < at.nslot; s0 += B) {
        v4f t[B], zg[B], vd[B];
        int qb[B], rb[B], rank[B];
#pragma unroll
        for (int i = 0; i < B; ++i) {
            qb[i] = q; rb[i] = s0 + i < at.nslot ? rd : it.nr;   // (no such row)
            if (++q == at.cpr) { q = 0; ++rd; }
            const int row = at.row(rb[i]);
            rank[i] = row < it.nr ? get_agent(&h.im.pos[it.g0 + row]) : -1;
            t[i] = at.fetch(a.Z, qb[i], rb[i]);
            zg[i] = at.fetch(x.Zg, qb[i], rb[i]);
            vd[i] = at.fetch(x.Vd, qb[i], rb[i]);
        }
#pragma unroll
        for (int i = 0; i < B; ++i) {
            const bool kept = rank[i] >= 0;
            const v4f qd = zg[i] - vd[i];
            const v4f att = t[i] * al;
            const v4f bq = qd * bl;
            const v4f zt = att + bq;
            at.put(a.Z, qb[i], rb[i], kept ? zt : zero4);
            if (!kept) at.put(a.U, qb[i], rb[i], t[i]);
            else if (pk_layer) at.put_packed(pk_layer + (int64_t)rank[i] * it.row_len, qb[i], zt + vd[i]);
        }
    }
}

// One FILTER row item: held_rows with the candidate z~ = fl(fl(a t) + fl(b (z - v))), t = Wbar + U.  z~ and t wait in
// registers, the dual of a kept row in LDS; what is packed is z~ + v, v read again.
template <int R, bool WHOLE, typename SHARED>
__device__ __forceinline__ void held_weighted_rows(const WorkItem* __restrict__ items, const WorkItem& it, const ProjectArgs& a, int Rrt, const HeldArgs& h,
                                                   const HeldWeighted& x, SHARED& sh)
{
    const int RR = R > 0 ? R : Rrt;
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = threadIdx.x / kWave;
    const HeldPlaces<WHOLE> at(it);
    const v4f zero4 = {0.f, 0.f, 0.f, 0.f};
    const float al = x.coef[2 * it.layer], bl = x.coef[2 * it.layer + 1];
    if (threadIdx.x < it.nr) put_agent(&h.im.pos[it.g0 + threadIdx.x], (int32_t)kNotSelected);
    v4f Zt[kHeldSlots], T[kHeldSlots];
    {
        constexpr int B = held_weighted_batch(R);
        constexpr int kIn = R > 0 ? R : 1;
        int q = 0, rd = 0;
        double acc = 0.0;
#pragma unroll
        for (int s0 = 0; s0 < kHeldSlots; s0 += B)
            if (s0 < at.nslot) {
                v4f in[B][kIn], u[B], zg[B], vd[B];
                int qb[B], rb[B];
#pragma unroll
                for (int i = 0; i < B; ++i) {
                    qb[i] = q; rb[i] = s0 + i < at.nslot ? rd : it.nr;   // (no such row)
                    if (++q == at.cpr) { q = 0; ++rd; }
                }
#pragma unroll
                for (int i = 0; i < B; ++i) {
#pragma unroll
                    for (int r = 0; r < kIn; ++r) in[i][r] = at.fetch(a.W[r], qb[i], rb[i]);
                    u[i] = at.fetch(a.Ur, qb[i], rb[i]);
                    zg[i] = at.fetch(x.Zg, qb[i], rb[i]);
                    vd[i] = at.fetch(x.Vd, qb[i], rb[i]);
                }
                v4f sum[B];
#pragma unroll
                for (int i = 0; i < B; ++i) {
                    sum[i] = in[i][0];
#pragma unroll
                    for (int r = 1; r < kIn; ++r) sum[i] = sum[i] + in[i][r];
                }
                if (R == 0)
                    for (int r = 1; r < RR; ++r) {
                        v4f y[B];
#pragma unroll
                        for (int i = 0; i < B; ++i) y[i] = at.fetch(a.W[r], qb[i], rb[i]);
#pragma unroll
                        for (int i = 0; i < B; ++i) sum[i] = sum[i] + y[i];
                    }
#pragma unroll
                for (int i = 0; i < B; ++i) {
                    const int s = s0 + i;
                    const v4f wb = sum[i] * a.inv_R;
                    const v4f t = wb + u[i];
                    const v4f qd = zg[i] - vd[i];
                    const v4f att = t * al;
                    const v4f bq = qd * bl;
                    const v4f zt = att + bq;
                    Zt[s] = zt;
                    T[s] = t;
                    sh.dual[s][threadIdx.x] = u[i] + (wb - zt);
                    if (a.Wbar) at.put(a.Wbar, qb[i], rb[i], wb);
                    acc = sq4(acc, zt);                          // (lanes without an element add zeros)
                    if (s < at.nslot && qb[i] == at.cpr - 1) {   // the row is complete
                        if (!at.wide) {
                            acc = wave_xor_sum(acc, at.lpr);
                            const int row = at.row(rb[i]);
                            if (at.j == 0 && row < it.nr) put_agent(&a.key[it.g0 + row], acc);
                        } else {
                            acc = wave_xor_sum(acc, kWave);
                            if (lane == 0) sh.wsum[rb[i]][wave] = acc;
                        }
                        acc = 0.0;
                    }
                }
            }
    }
    if (at.wide) {
        __syncthreads();
        if (threadIdx.x < it.nr) {
            double s = sh.wsum[threadIdx.x][0];
            for (int w = 1; w < kWaves; ++w) s += sh.wsum[threadIdx.x][w];
            put_agent(&a.key[it.g0 + threadIdx.x], s);
        }
    }
    const bool selects = held_publish(it, h);
    if (selects) held_select(it, h, a.key, sh.topk);
    const bool known = held_wait_groups(it.g0, it.nr, h, sh.rank);
    float* const pk_layer = (h.packed && known) ? h.packed + it.packed_off : nullptr;
    {
        constexpr int B = 5;
        int q = 0, rd = 0;
#pragma unroll
        for (int s0 = 0; s0 < kHeldSlots; s0 += B) {
            if (s0 < at.nslot) {
                v4f vd[B];
                int qb[B], rb[B], rank[B];
#pragma unroll
                for (int i = 0; i < B; ++i) {
                    qb[i] = q; rb[i] = s0 + i < at.nslot ? rd : it.nr;
                    if (++q == at.cpr) { q = 0; ++rd; }
                    const int row = at.row(rb[i]);
                    rank[i] = row < it.nr ? (known ? sh.rank[row] : 0) : -1;
                    vd[i] = zero4;
                    if (pk_layer && rank[i] >= 0) vd[i] = at.fetch(x.Vd, qb[i], rb[i]);
                }
#pragma unroll
                for (int i = 0; i < B; ++i) {
                    const int s = s0 + i;
                    const bool kept = rank[i] >= 0;
                    const v4f d = sh.dual[s][threadIdx.x];
                    // (written too early: t and the dual of a kept row, from which either outcome can be formed)
                    at.put(a.Z, qb[i], rb[i], known ? (kept ? Zt[s] : zero4) : T[s]);
                    at.put(a.U, qb[i], rb[i], kept ? d : T[s]);
                    if (pk_layer && kept) at.put_packed(pk_layer + (int64_t)rank[i] * it.row_len, qb[i], Zt[s] + vd[i]);
                }
            }
        }
    }
    held_finish_early(items, h, !known, (int)(it.aux & 0xffffffffll), selects ? (int)(it.aux >> 32) : 0, sh.turn,
                      [&](const WorkItem& y) { held_weighted_finish<WHOLE>(y, a, h, x); });
}

template <int R>
__global__ __launch_bounds__(kBlock, kHeldWeightedPerUnit) void weighted_held(const WorkItem* __restrict__ items, WeightedArgs w,
                                                                              int Rrt, HeldArgs h, HeldWeighted x)
{
    __shared__ HeldShared<kHeldWeightedLds> sh;
    const WorkItem it = items[blockIdx.x];
    if (it.row0 == 0 && threadIdx.x == 0) held_layer_entries(it, h);
    if (item_mode(it) == HSADMM_MODE_NONE) {
        const WeightedHint hint{nullptr, h.packed, nullptr, h.layers};
        held_none_entries(it, h);
        weighted_rows_hinted<R, false>(it, w, Rrt, hint);
    } else {
        if (item_vec(it)) held_weighted_rows<R, true>(items, it, w.p, Rrt, h, x, sh);
        else held_weighted_rows<R, false>(items, it, w.p, Rrt, h, x, sh);
    }
}

// ------------------------------------------------------------------ input-channel groups

// A tile of a CHANNEL layer (kChanRows rows by one column strip, project_tile's) waits in the same way: a wave has its
// sixteen rows in as many slots, the candidate in registers, the dual of a kept element in LDS and registers.  The tile that
// finds its strip complete adds up the strip's column sums, the one that finds the layer's strips complete finishes the
// channel keys and selects; additions in the order of the other forms.  Bounded by HBM traffic, R + 3 arenas and the packed
// rows; before, pass 1 parked the mean (or the replicas were read twice) and a final pass read it and the dual again, R + 6.
// Three workgroups a compute unit hold 12.6 M elements, two (weighted: three values an element; eight replicas) 8.4 M.
// Before / with it, us: ResNet-152, 4 replicas, a step 525 / 441, weighted 808 / 688; ResNet-50, keep 0.5, 1, 2, 4, 8
// replicas 164 / 141, 193 / 158, 243 / 193, 322 / 255, weighted 280 / 250, 313 / 266, 368 / 299, 449 / 374; plain network of
// width 64, 4 replicas 38.5 / 33.1.
constexpr int kHeldTileSlots = kChanRows / kWaves;
constexpr int kHeldTileLds = 10;         // ... the duals of the first ones in LDS
constexpr int held_tile_per_unit(int R, bool weighted) { return weighted || R == 8 ? 2 : 3; }
// slots whose loads are in flight together, as many as spill nothing
constexpr int held_tile_batch(int R, bool weighted) { return weighted ? (R == 1 ? 4 : R == 8 ? 1 : 2) : (R <= 2 ? 4 : 2); }

// WorkItem fields of a held tile: lpr = index of the layer's first tile.
struct HeldTiles {
    unsigned long long* strip_tag;      // per strip (at the layer's first tile + strip): gen once its column sums are complete
    unsigned long long* strip_claim;    // ... gen once a tile has begun to add them up
    double* colpart;
};

// The waves' column sums are through before the selection begins, so they share its place: LDS is given out in pieces of 1280
// bytes, and a workgroup with both took 43 of the 128 pieces a unit has.
struct HeldTileShared {
    v4f dual[kHeldTileLds][kBlock];
    union {
        double part[kWaves][kWave * 4];
        struct {
            TopkShared topk;
            int rank[kBlock];
        } sel;
    };
    int claimed;
    HeldTurn turn;
};

__device__ __forceinline__ int tile_strip_cols(const WorkItem& it) { return kWave * (item_vec(it) ? 4 : 1); }
__device__ __forceinline__ int tile_strips(const WorkItem& it) { return (it.row_len + tile_strip_cols(it) - 1) / tile_strip_cols(it); }

// Called by the whole workgroup when its column sums have been stored by put_agent.  True: all column sums of the layer are
// complete, in the first row block's place.
__device__ __forceinline__ bool held_tile_publish(const WorkItem& it, const HeldArgs& h, const HeldTiles& x, HeldTileShared& sh)
{
    const int cols = tile_strip_cols(it);
    const int n_strips = tile_strips(it);
    const int n_rb = h.layers[it.layer].n_rowblocks;
    const int strip = it.col0 / cols;
    const int first = it.lpr;
    if (threadIdx.x == 0) put_agent(&h.state[blockIdx.x], h.gen);
    stores_arrived();
    __syncthreads();
    if (threadIdx.x == 0) {
        put_agent(&h.tag[blockIdx.x], h.gen);
        stores_arrived();
    }
    __syncthreads();
    bool ok = true;
    for (int rb = threadIdx.x; rb < n_rb; rb += kBlock) ok = ok && get_agent(&h.tag[first + rb * n_strips + strip]) == h.gen;
    if (__syncthreads_and(ok) == 0) return false;
    // one tile alone adds the strip up, as the sums take the place of the first row block's
    if (threadIdx.x == 0)
        sh.claimed = __hip_atomic_exchange(&x.strip_claim[first + strip], h.gen, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == h.gen;
    __syncthreads();
    if (sh.claimed) return false;
    double* const sums = x.colpart + h.layers[it.layer].colpart_off;
    const int col = it.col0 + (int)threadIdx.x;
    if ((int)threadIdx.x < cols && col < it.row_len) {
        double acc = 0.0;
        int rb = 0;
        for (; rb + 8 <= n_rb; rb += 8) {
            double p[8];
#pragma unroll
            for (int b = 0; b < 8; ++b) p[b] = get_agent(&sums[(int64_t)(rb + b) * it.row_len + col]);
#pragma unroll
            for (int b = 0; b < 8; ++b) acc += p[b];
        }
        for (; rb < n_rb; ++rb) acc += get_agent(&sums[(int64_t)rb * it.row_len + col]);
        put_agent(&sums[col], acc);
    }
    stores_arrived();
    __syncthreads();
    if (threadIdx.x == 0) {
        put_agent(&x.strip_tag[first + strip], h.gen);
        stores_arrived();
    }
    __syncthreads();
    ok = true;
    for (int s = threadIdx.x; s < n_strips; s += kBlock) ok = ok && get_agent(&x.strip_tag[first + s]) == h.gen;
    return __syncthreads_and(ok) != 0;
}

// The channel keys from the column sums, then the selection.
__device__ __forceinline__ void held_tile_select(const WorkItem& it, const HeldArgs& h, const HeldTiles& x, double* key,
                                                 HeldTileShared& sh)
{
    const DevLayer& L = h.layers[it.layer];
    const double* const sums = x.colpart + L.colpart_off;
    if (L.khw == 1) {
        constexpr int B = kTopkInFlight;
        for (int g0 = (int)threadIdx.x; g0 < L.G; g0 += B * kBlock) {
            double y[B];
#pragma unroll
            for (int i = 0; i < B; ++i) y[i] = g0 + i * kBlock < L.G ? get_agent(&sums[g0 + i * kBlock]) : 0.0;
#pragma unroll
            for (int i = 0; i < B; ++i)
                if (g0 + i * kBlock < L.G) put_agent(&key[L.group_base + g0 + i * kBlock], y[i]);
        }
    } else {
        for (int g = threadIdx.x; g < L.G; g += kBlock) {
            const double* const c = sums + (int64_t)g * L.khw;
            double acc = 0.0;
            for (int t = 0; t < L.khw; t += 9) {                 // (a 3 x 3 kernel's in one go; a zero added to a sum of squares leaves it)
                double y[9];
#pragma unroll
                for (int i = 0; i < 9; ++i) y[i] = t + i < L.khw ? get_agent(&c[t + i]) : 0.0;
#pragma unroll
                for (int i = 0; i < 9; ++i) acc += y[i];
            }
            put_agent(&key[L.group_base + g], acc);
        }
    }
    stores_arrived();
    __syncthreads();
    held_select(it, h, key, sh.sel.topk);
}

// A tile that was written before its selection was known, from that form to its final one: the lanes and rows of held_tile, four
// of a wave's rows in flight.
template <bool WEIGHTED, bool VEC>
__device__ __forceinline__ void held_tile_finish(const WorkItem& it, const ProjectArgs& a, const HeldArgs& h)
{
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = threadIdx.x / kWave;
    const int row_len = it.row_len;
    constexpr int vw = VEC ? 4 : 1, B = 4;
    const int col = it.col0 + lane * vw;
    if (col >= row_len) return;
    const DivKhw div(it.khw);
    const float al = WEIGHTED ? a.coef[2 * it.layer] : 1.f, bl = WEIGHTED ? a.coef[2 * it.layer + 1] : 0.f;
    const v4f zero4 = {0.f, 0.f, 0.f, 0.f};
    bool kept[4] = {true, true, true, true};
    int pc[4] = {-1, -1, -1, -1};                // packed column, -1: not packed
#pragma unroll
    for (int i = 0; i < vw; ++i) {
        const int ch = div(col + i);
        const int r = get_agent(&h.im.pos[it.g0 + ch]);
        kept[i] = r >= 0;
        if (h.packed && r >= 0) pc[i] = r * it.khw + (col + i - ch * it.khw);
    }
    auto fetch = [&](const float* p, int rr) -> v4f {
        v4f v = zero4;
        if (rr < it.nr) {
            if (VEC) v = ld4(p + it.base + (int64_t)rr * row_len + col);
            else v.x = ld1(p + it.base + (int64_t)rr * row_len + col);
        }
        return v;
    };
    auto put = [&](float* p, int rr, const v4f& v) {
        if (rr >= it.nr) return;
        if (VEC) st4(p + it.base + (int64_t)rr * row_len + col, v);
        else st1(p + it.base + (int64_t)rr * row_len + col, v.x);
    };
    const int64_t packed_row_len = (int64_t)it.k * it.khw;
    for (int r0 = wave; r0 < it.nr; r0 += B * kWaves) {
        v4f p[B], d[B], zg[B], vd[B];
#pragma unroll
        for (int i = 0; i < B; ++i) {
            p[i] = fetch(a.Z, r0 + i * kWaves);                  // the dual of a pruned element
            d[i] = fetch(a.U, r0 + i * kWaves);                  // ... of a kept one
            if (WEIGHTED) {
                zg[i] = fetch(a.Zg, r0 + i * kWaves);
                vd[i] = fetch(a.Vd, r0 + i * kWaves);
            }
        }
#pragma unroll
        for (int i = 0; i < B; ++i) {
            const int rr = r0 + i * kWaves;
            v4f c = p[i];
            if (WEIGHTED) {
                const v4f q = zg[i] - vd[i];
                const v4f at = p[i] * al;
                const v4f bq = q * bl;
                c = at + bq;
            }
            v4f z, u;
            z.x = kept[0] ? c.x : 0.f; z.y = kept[1] ? c.y : 0.f; z.z = kept[2] ? c.z : 0.f; z.w = kept[3] ? c.w : 0.f;
            u.x = kept[0] ? d[i].x : p[i].x; u.y = kept[1] ? d[i].y : p[i].y;
            u.z = kept[2] ? d[i].z : p[i].z; u.w = kept[3] ? d[i].w : p[i].w;
            put(a.Z, rr, z);
            put(a.U, rr, u);
            if (h.packed && rr < it.nr) {
                float* row = h.packed + it.packed_off + (it.row0 + rr) * packed_row_len;
                const v4f y = WEIGHTED ? z + vd[i] : z;
                if (pc[0] >= 0) row[pc[0]] = y.x;
                if (pc[1] >= 0) row[pc[1]] = y.y;
                if (pc[2] >= 0) row[pc[2]] = y.z;
                if (pc[3] >= 0) row[pc[3]] = y.w;
            }
        }
    }
}

// VEC: rows of whole words (four columns a lane, else one); a choice within the loop would make loads wait for each other.
template <int R, bool WEIGHTED, bool VEC>
__device__ __forceinline__ void held_tile(const WorkItem* __restrict__ items, const WorkItem& it, const ProjectArgs& a, int Rrt, const HeldArgs& h,
                                          const HeldTiles& x, HeldTileShared& sh)
{
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = threadIdx.x / kWave;
    const int row_len = it.row_len;
    constexpr int vw = VEC ? 4 : 1;
    const int col = it.col0 + lane * vw;
    const bool in = col < row_len;
    const int khw = it.khw;
    const DivKhw div(khw);
    const int last_col = min(row_len, it.col0 + kWave * vw) - 1;
    const int ch0 = div(it.col0), n_ch = div(last_col) - ch0 + 1;        // the strip's channels, at most a thread each
    const float al = WEIGHTED ? a.coef[2 * it.layer] : 1.f, bl = WEIGHTED ? a.coef[2 * it.layer + 1] : 0.f;
    const v4f zero4 = {0.f, 0.f, 0.f, 0.f};
    if ((int)threadIdx.x < n_ch) put_agent(&h.im.pos[it.g0 + ch0 + threadIdx.x], (int32_t)kNotSelected);
    auto fetch = [&](const float* p, int s) -> v4f {
        v4f v = zero4;
        const int rr = wave + s * kWaves;
        if (in && rr < it.nr) {
            if (VEC) v = ld4(p + it.base + (int64_t)rr * row_len + col);
            else v.x = ld1(p + it.base + (int64_t)rr * row_len + col);
        }
        return v;
    };
    auto put = [&](float* p, int s, const v4f& v) {
        const int rr = wave + s * kWaves;
        if (!in || rr >= it.nr) return;
        if (VEC) st4(p + it.base + (int64_t)rr * row_len + col, v);
        else st1(p + it.base + (int64_t)rr * row_len + col, v.x);
    };
    v4f V[kHeldTileSlots], D[kHeldTileSlots - kHeldTileLds], T[WEIGHTED ? kHeldTileSlots : 1];
    {
        constexpr int B = held_tile_batch(R, WEIGHTED);
        constexpr int kIn = R > 0 ? R : 1;
        double acc0 = 0.0, acc1 = 0.0, acc2 = 0.0, acc3 = 0.0;
#pragma unroll
        for (int s0 = 0; s0 < kHeldTileSlots; s0 += B)
            if (s0 * kWaves < it.nr) {
                v4f w[B][kIn], u[B], zg[B], vd[B], sum[B];
#pragma unroll
                for (int i = 0; i < B; ++i) {
#pragma unroll
                    for (int r = 0; r < kIn; ++r) w[i][r] = fetch(a.W[r], s0 + i);
                    u[i] = fetch(a.Ur, s0 + i);
                    if (WEIGHTED) {
                        zg[i] = fetch(a.Zg, s0 + i);
                        vd[i] = fetch(a.Vd, s0 + i);
                    }
                }
#pragma unroll
                for (int i = 0; i < B; ++i) {
                    sum[i] = w[i][0];
#pragma unroll
                    for (int r = 1; r < kIn; ++r) sum[i] = sum[i] + w[i][r];
                }
                if (R == 0)
                    for (int r = 1; r < Rrt; ++r) {
                        v4f y[B];
#pragma unroll
                        for (int i = 0; i < B; ++i) y[i] = fetch(a.W[r], s0 + i);
#pragma unroll
                        for (int i = 0; i < B; ++i) sum[i] = sum[i] + y[i];
                    }
#pragma unroll
                for (int i = 0; i < B; ++i) {
                    const int s = s0 + i;
                    const v4f wb = sum[i] * a.inv_R;
                    v4f v = wb + u[i];
                    if (WEIGHTED) {
                        T[WEIGHTED ? s : 0] = v;
                        const v4f q = zg[i] - vd[i];
                        const v4f at = v * al;
                        const v4f bq = q * bl;
                        v = at + bq;
                    }
                    V[s] = v;
                    const v4f d = u[i] + (wb - v);
                    if (s < kHeldTileLds) sh.dual[s][threadIdx.x] = d;
                    else D[s - kHeldTileLds] = d;
                    if (a.Wbar) put(a.Wbar, s, wb);
                    acc0 = fma((double)v.x, (double)v.x, acc0);  // (rows that are not there add zeros)
                    acc1 = fma((double)v.y, (double)v.y, acc1);
                    acc2 = fma((double)v.z, (double)v.z, acc2);
                    acc3 = fma((double)v.w, (double)v.w, acc3);
                }
            }
        sh.part[wave][lane * 4 + 0] = acc0;
        sh.part[wave][lane * 4 + 1] = acc1;
        sh.part[wave][lane * 4 + 2] = acc2;
        sh.part[wave][lane * 4 + 3] = acc3;
    }
    __syncthreads();
    if ((int)threadIdx.x < kWave * vw && it.col0 + (int)threadIdx.x < row_len) {
        const int k = VEC ? (int)threadIdx.x : 4 * (int)threadIdx.x;
        double s = sh.part[0][k];
        for (int w = 1; w < kWaves; ++w) s += sh.part[w][k];
        put_agent(&x.colpart[it.aux + it.col0 + threadIdx.x], s);
    }
    const bool selects = held_tile_publish(it, h, x, sh);
    if (selects) held_tile_select(it, h, x, a.key, sh);
    const bool known = held_wait_groups(it.g0 + ch0, n_ch, h, sh.sel.rank);
    bool kept[4] = {true, true, true, true};
    int pc[4] = {-1, -1, -1, -1};                // packed column, -1: not packed
    if (known && in) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (i < vw) {
                const int ch = div(col + i);
                const int r = sh.sel.rank[ch - ch0];
                kept[i] = r >= 0;
                if (h.packed && r >= 0) pc[i] = r * khw + (col + i - ch * khw);
            }
    }
    const int64_t packed_row_len = (int64_t)it.k * khw;
    float* const pk = h.packed ? h.packed + it.packed_off + it.row0 * packed_row_len : nullptr;
#pragma unroll
    for (int s0 = 0; s0 < kHeldTileSlots; s0 += 4)
        if (s0 * kWaves < it.nr) {
            v4f vd[4];
            if (WEIGHTED) {
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    vd[i] = zero4;
                    if (pc[0] >= 0 || pc[1] >= 0 || pc[2] >= 0 || pc[3] >= 0) vd[i] = fetch(a.Vd, s0 + i);
                }
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int s = s0 + i;
                const v4f d = s < kHeldTileLds ? sh.dual[s][threadIdx.x] : D[s < kHeldTileLds ? 0 : s - kHeldTileLds];
                const v4f p = WEIGHTED ? T[WEIGHTED ? s : 0] : V[s];             // the dual of a pruned element
                v4f z, u;
                z.x = kept[0] ? V[s].x : 0.f; z.y = kept[1] ? V[s].y : 0.f; z.z = kept[2] ? V[s].z : 0.f; z.w = kept[3] ? V[s].w : 0.f;
                u.x = kept[0] ? d.x : p.x; u.y = kept[1] ? d.y : p.y; u.z = kept[2] ? d.z : p.z; u.w = kept[3] ? d.w : p.w;
                // (written too early: the candidate, or what it is made of, and the dual of a kept element)
                put(a.Z, s, known ? z : p);
                put(a.U, s, u);
                const int rr = wave + s * kWaves;
                if (pk && in && rr < it.nr) {
                    float* row = pk + rr * packed_row_len;
                    const v4f c = WEIGHTED ? z + vd[i] : z;
                    if (pc[0] >= 0) row[pc[0]] = c.x;
                    if (pc[1] >= 0) row[pc[1]] = c.y;
                    if (pc[2] >= 0) row[pc[2]] = c.z;
                    if (pc[3] >= 0) row[pc[3]] = c.w;
                }
            }
        }
    held_finish_early(items, h, !known, it.lpr, selects ? tile_strips(it) * h.layers[it.layer].n_rowblocks : 0, sh.turn,
                      [&](const WorkItem& y) { held_tile_finish<WEIGHTED, VEC>(y, a, h); });
}

template <int R, bool WEIGHTED>
__global__ __launch_bounds__(kBlock, held_tile_per_unit(R, WEIGHTED)) void tiles_held(const WorkItem* __restrict__ items, WeightedArgs w,
                                                                                   int Rrt, HeldArgs h, HeldTiles x)
{
    __shared__ HeldTileShared sh;
    const WorkItem it = items[blockIdx.x];
    if (it.row0 == 0 && it.col0 == 0 && threadIdx.x == 0) held_layer_entries(it, h);
    if (item_mode(it) == HSADMM_MODE_NONE) {                     // final at once
        held_none_entries(it, h);
        if constexpr (WEIGHTED) {
            const WeightedHint hint{nullptr, h.packed, nullptr, h.layers};
            weighted_rows_hinted<R, false>(it, w, Rrt, hint);
        } else {
            const HintArgs hint{nullptr, h.packed, 0, nullptr, h.layers};
            project_rows_hinted<R>(it, w.p, Rrt, hint);
        }
    } else {
        if (item_vec(it)) held_tile<R, WEIGHTED, true>(items, it, w.p, Rrt, h, x, sh);
        else held_tile<R, WEIGHTED, false>(items, it, w.p, Rrt, h, x, sh);
    }
}

// Inside a captured graph a call's number is the same in every replay: the tags are cleared first.
__global__ __launch_bounds__(kBlock) void held_clear(unsigned long long* tags, int n)
{
    const int i = (int)(blockIdx.x * kBlock + threadIdx.x);
    if (i < n) tags[i] = 0ull;
}

}  // namespace
#endif
