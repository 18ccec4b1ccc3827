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
// ResNet-50, 4 replicas 183 / 162; ResNet-18, 1 replica 77.7 / 62.0; of width 45, 3 replicas 60.8 / 46.2; a plain network
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
constexpr int kHeldCleaners = 16;        // workgroups at the end of the grid that finish what was written too early
constexpr long long kHeldCleanLimit = 400000000;   // ... give up themselves after four seconds: every wave comes to an end

// WorkItem fields of a held row item: aux = index of the layer's first held item | items of the layer << 32; khw = chunks
// (slots) of a thread per row.
struct HeldArgs {
    unsigned long long* tag;        // per held item: gen once the item's keys are published
    unsigned long long* state;      // per held item: gen + 1 when it is done, gen + 2 when it was written too early
    unsigned long long gen;         // this call's number; neither it nor the two after it are any other call's, or a value
                                    // that anything else writes there
    int32_t* pred;                  // groups_total: the form of a row written too early (kKeptNoRank or -1)
    long long patience;             // ticks
    const DevLayer* layers;
    uint8_t* mask;
    IndexMaps im;
    CopyOut co;                     // the caller's layer_off / kept_idx (nulls: no compaction)
    float* packed;                  // null: no compaction
    int n_layers, pack_align;
    int n_items, n_held;            // items of the launch, and how many of them are held (the first ones)
};

// LDS: slots whose dual waits here.
template <int LDS>
struct HeldShared {
    v4f dual[LDS][kBlock];
    TopkShared topk;
    double wsum[kHeldSlots][kWaves];
    int rank[kHeldRows];
};

// Called by the whole workgroup when all keys of the item's rows have been stored by put_agent.  Publishes the item and
// returns whether all items of its layer are published now (two workgroups that finish together may both be told so).
// A store has arrived before the tags are looked at, so the one whose store arrives last sees all the others'.
__device__ __forceinline__ bool held_publish(const WorkItem& it, const HeldArgs& h)
{
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

// Waits for the ranks of the item's rows -> rank (-1: pruned); false if the patience ran out first.
__device__ __forceinline__ bool held_wait(const WorkItem& it, const HeldArgs& h, int* rank)
{
    const int t = threadIdx.x;
    int r = -1;
    if (t < it.nr) {
        const long long until = (long long)__builtin_amdgcn_s_memrealtime() + h.patience;
        for (;;) {
            r = get_agent(&h.im.pos[it.g0 + t]);
            if (r != kNotSelected || (long long)__builtin_amdgcn_s_memrealtime() > until) break;
            __builtin_amdgcn_s_sleep(8);
        }
        rank[t] = r;
    }
    return __syncthreads_or(t < it.nr && r == kNotSelected) == 0;
}

// Where the slots of a thread lie in a row item.  The choice between a row's words and a ragged row's last floats (in the
// slot behind them, one to a lane) is one that the whole workgroup makes, so that no load waits for another's register.
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
        tail_slot = (row_len & 3) ? cpr - 1 : cpr;
        nslot = cpr * ((nr + rows_at_once - 1) / rows_at_once);
    }
    __device__ __forceinline__ int row(int rd) const { return rd * rows_at_once + sub; }
    __device__ __forceinline__ v4f fetch(const float* p, int q, int rd) const
    {
        v4f x = {0.f, 0.f, 0.f, 0.f};
        if (row(rd) < nr) {
            const float* r = p + base + (int64_t)row(rd) * row_len;
            if (q != tail_slot) {
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
        if (q != tail_slot) {
            const int c = j + q * lpr;
            if (c < nchunk) st4(r + 4 * c, x);
        } else if (j < (row_len & 3)) {
            st1(r + 4 * nchunk + j, x.x);
        }
    }
    // the same into a packed row, which may begin at any float
    __device__ __forceinline__ void put_packed(float* r, int q, const v4f& x) const
    {
        if (q != tail_slot) {
            const int c = j + q * lpr;
            if (c < nchunk) st4u(r + 4 * c, x);
        } else if (j < (row_len & 3)) {
            r[4 * nchunk + j] = x.x;
        }
    }
};

// One FILTER row item.
template <int R, typename SHARED>
__device__ __forceinline__ void held_rows(const WorkItem& it, const ProjectArgs& a, int Rrt, const HeldArgs& h, SHARED& sh)
{
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = threadIdx.x / kWave;
    const HeldPlaces at(it);
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
    if (held_publish(it, h)) held_select(it, h, a.key, sh.topk);
    const bool known = held_wait(it, h, sh.rank);
    if (known && threadIdx.x == 0) put_agent(&h.state[blockIdx.x], h.gen + 1);   // (no one reads the rows in this launch)
    const DevLayer& L = h.layers[it.layer];
    const bool kept_default = 2 * L.k >= L.G;                    // written too early: in the likelier form
    if (!known) {
        if (threadIdx.x < it.nr) h.pred[it.g0 + threadIdx.x] = kept_default ? 0x7fffffff : -1;
    }
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
    if (!known) {                                                // a cleaner reads the rows on another compute unit
        __threadfence();
        __syncthreads();
        if (threadIdx.x == 0) put_agent(&h.state[blockIdx.x], h.gen + 2);
    }
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

// A workgroup behind all the items: waits until every item of its share is done, and takes those that were written before
// their selection was known (none, unless other work held places that a layer's workgroups needed) from that form to their
// final one (finish).  Its waits end because no workgroup that it waits for waits without end.
template <typename F>
__device__ __forceinline__ void held_clean(const WorkItem* __restrict__ items, const HeldArgs& h, F finish)
{
    const int n_held = h.n_held;
    const int c = (int)blockIdx.x - h.n_items;
    const long long until = (long long)__builtin_amdgcn_s_memrealtime() + kHeldCleanLimit;
    for (int i0 = c; i0 < n_held; i0 += kHeldCleaners * kBlock) {
        const int i = i0 + (int)threadIdx.x * kHeldCleaners;
        unsigned long long st = h.gen + 1;
        while (i < n_held) {
            st = get_agent(&h.state[i]);
            if (st == h.gen + 1 || st == h.gen + 2 || (long long)__builtin_amdgcn_s_memrealtime() > until) break;
            __builtin_amdgcn_s_sleep(16);
        }
        if (__syncthreads_or(st == h.gen + 2) == 0) continue;
        for (int t = 0; t < kBlock; ++t) {
            const int k = i0 + t * kHeldCleaners;
            if (k >= n_held) break;
            if (get_agent(&h.state[k]) != h.gen + 2) continue;
            const WorkItem it = items[k];
            if ((int)threadIdx.x < it.nr)
                while (get_agent(&h.im.pos[it.g0 + threadIdx.x]) == kNotSelected &&
                       (long long)__builtin_amdgcn_s_memrealtime() <= until) __builtin_amdgcn_s_sleep(16);
            __syncthreads();
            __threadfence();                                     // the item's rows as its workgroup left them
            finish(it);
        }
    }
}

template <int R>
__global__ __launch_bounds__(kBlock, kHeldPerUnit) void project_held(const WorkItem* __restrict__ items, ProjectArgs a, int Rrt,
                                                          HeldArgs h)
{
    __shared__ HeldShared<kHeldLdsSlots> sh;
    if ((int)blockIdx.x >= h.n_items) {
        held_clean(items, h, [&](const WorkItem& it) {
            hinted_repair_rows<1>(it, a, 1, h.pred, h.im.pos, true, h.packed ? h.packed + it.packed_off : nullptr);
        });
        return;
    }
    const WorkItem it = items[blockIdx.x];
    if (it.row0 == 0 && threadIdx.x == 0) held_layer_entries(it, h);
    if (item_mode(it) == HSADMM_MODE_NONE) {                     // final at once
        const HintArgs hint{nullptr, h.packed, 0, nullptr, h.layers};
        held_none_entries(it, h);
        project_rows_hinted<R, R != 8>(it, a, Rrt, hint);        // (one chunk at a time with eight replicas: no registers to spare)
    } else {
        held_rows<R>(it, a, Rrt, h, sh);
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
// launches that touch Z, U and the kept rows' z and v twice / in this one: 250 / 231, 300 / 277, 338 / 320, 374 / 347 with 1, 4, 6,
// 8 replicas.  (The residual norms on the way need the replicas' values until z~ is known; with them the launch gained nothing:
// 345 / 347 us with 4 replicas, small networks 3 to 15 % slower.  They keep the other path.)
constexpr int kHeldWeightedPerUnit = 3;
constexpr int kHeldWeightedLds = kHeldSlots;
constexpr int held_weighted_batch(int R) { return R == 8 ? 1 : 2; }

// One FILTER row item: held_rows with the candidate z~ = fl(fl(a t) + fl(b (z - v))), t = Wbar + U.  z~ and t wait in
// registers, the dual of a kept row in LDS; what is packed is z~ + v, v read again.
template <int R, typename SHARED>
__device__ __forceinline__ void held_weighted_rows(const WorkItem& it, const ProjectArgs& a, int Rrt, const HeldArgs& h,
                                                   const HeldWeighted& x, SHARED& sh)
{
    const int RR = R > 0 ? R : Rrt;
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = threadIdx.x / kWave;
    const HeldPlaces at(it);
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
    if (held_publish(it, h)) held_select(it, h, a.key, sh.topk);
    const bool known = held_wait(it, h, sh.rank);
    if (known && threadIdx.x == 0) put_agent(&h.state[blockIdx.x], h.gen + 1);   // (no one reads the rows in this launch)
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
    if (!known) {                                                // a cleaner reads the rows on another compute unit
        __threadfence();
        __syncthreads();
        if (threadIdx.x == 0) put_agent(&h.state[blockIdx.x], h.gen + 2);
    }
}

// weighted_fixup_rows by a cleaner: the item's ranks and rows as other workgroups of this launch left them.
__device__ __forceinline__ void held_weighted_finish(const WorkItem& it, const ProjectArgs& a, const HeldArgs& h,
                                                     const HeldWeighted& x)
{
    const HeldPlaces at(it);
    const float al = x.coef[2 * it.layer], bl = x.coef[2 * it.layer + 1];
    const v4f zero4 = {0.f, 0.f, 0.f, 0.f};
    int q = 0, rd = 0;
    for (int s = 0; s < at.nslot; ++s) {
        const int row = at.row(rd);
        if (row < it.nr) {
            const int rank = get_agent(&h.im.pos[it.g0 + row]);
            const v4f t = at.fetch(a.Z, q, rd);
            if (rank >= 0) {
                const v4f vd = at.fetch(x.Vd, q, rd);
                const v4f qd = at.fetch(x.Zg, q, rd) - vd;
                const v4f att = t * al;
                const v4f bq = qd * bl;
                const v4f zt = att + bq;
                at.put(a.Z, q, rd, zt);
                if (h.packed) at.put_packed(h.packed + it.packed_off + (int64_t)rank * it.row_len, q, zt + vd);
            } else {
                at.put(a.U, q, rd, t);
                at.put(a.Z, q, rd, zero4);
            }
        }
        if (++q == at.cpr) { q = 0; ++rd; }
    }
}

template <int R>
__global__ __launch_bounds__(kBlock, kHeldWeightedPerUnit) void weighted_held(const WorkItem* __restrict__ items, WeightedArgs w,
                                                                              int Rrt, HeldArgs h, HeldWeighted x)
{
    __shared__ HeldShared<kHeldWeightedLds> sh;
    if ((int)blockIdx.x >= h.n_items) {
        held_clean(items, h, [&](const WorkItem& it) { held_weighted_finish(it, w.p, h, x); });
        return;
    }
    const WorkItem it = items[blockIdx.x];
    if (it.row0 == 0 && threadIdx.x == 0) held_layer_entries(it, h);
    if (item_mode(it) == HSADMM_MODE_NONE) {
        const WeightedHint hint{nullptr, h.packed, nullptr, h.layers};
        held_none_entries(it, h);
        weighted_rows_hinted<R, false>(it, w, Rrt, hint);
    } else {
        held_weighted_rows<R>(it, w.p, Rrt, h, x, sh);
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
