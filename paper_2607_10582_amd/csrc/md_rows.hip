// gfx950 session kernel: one decode step's append and observation for
// batches of short sessions, in one launch.
//
// A workgroup takes one session and one range of its (layer, KV head) rows,
// and every row whole: all of the session's tokens, so that a row's softmax
// needs nothing from other workgroups (the fused kernel's units of 256 tokens
// exchange every row's statistics; the multi-kernel path writes the logits to
// HBM).  Its eight waves take the session's 16-token tiles in turn and hold a
// row's 2^(logit - max) in LDS until the waves' statistics meet at the row's
// one barrier; then each wave adds its tokens' softmax weights to their mass.
// The mass of a token sums over rows (Sec. III-C), so the row ranges' partial
// masses go to scratch, and the workgroup that finishes a session last adds
// them in range order and runs the epilogue (Eq. 2 - 5) for its tokens.
// No workgroup waits for another one, so the grid needs no residency.
//
// The append (Fig. 1) runs in the same launch: every workgroup works out its
// session's new token from the counters as they stand before the step, reads
// its key from new_k in place of the pool, and writes its own rows of it to
// the pool; the workgroup that finishes the session writes the token's state.
// The counters, page tables and the free list are committed by whichever
// workgroup is the last to have read them, as a count of arrivals tells
// (md_arrive.h).  One more workgroup, dispatched last, has no rows: it works
// the commit out while the others read, and as a rule arrives last and
// commits under their rows; if it does not, the last of the others commits
// when it is done.
//
// What bounds it: for a single session of a few hundred tokens the chain of
// dependent memory round trips (counters and page table, keys, partial
// masses, token state); for a batch the key stream.

#include <algorithm>

#include "md_arrive.h"
#include "md_device.h"

namespace md {

namespace {

constexpr int kRW = kRowsWaves;            // waves per workgroup
constexpr int kRT = 64 * kRW;              // threads
constexpr int kMaxNc = 8;                  // 64-token chunks per wave
constexpr int kMaxTiles = 4 * kMaxNc;      // tiles per wave

struct RowsLds {
    uint32_t* qs;     // [2][3][G][64] hi, mid, lo bf16 query terms of two rows
    float2* wstat;    // [2][kRW][16] per-wave row statistics
    float* wmax;      // [kRW][kMaxNc][16] maximum of each held chunk per head
    float* mass;      // [kRW][64 nc] the waves' tokens' masses so far
    uint32_t* unseen; // [kRW][nc][64] window: tokens a lane's column does not see
    float* red;       // [kRW][8][64] sums of partial masses (rowbuf's place, after the rows)
    float* rowbuf;    // [kRW][G][64 nc + 4] 2^(logit - chunk max) of the row
};

__host__ __device__ constexpr int rows_stride(int nc) { return 64 * nc + 4; }

__device__ __forceinline__ RowsLds rows_carve(unsigned char* p, int G, int nc, bool window) {
    RowsLds l;
    l.qs = reinterpret_cast<uint32_t*>(p);
    p += (size_t)2 * 3 * G * 64 * sizeof(uint32_t);
    l.wstat = reinterpret_cast<float2*>(p);
    p += (size_t)2 * kRW * 16 * sizeof(float2);
    l.wmax = reinterpret_cast<float*>(p);
    p += (size_t)kRW * kMaxNc * 16 * sizeof(float);
    l.mass = reinterpret_cast<float*>(p);
    p += (size_t)kRW * 64 * nc * sizeof(float);
    l.unseen = reinterpret_cast<uint32_t*>(p);
    if (window) p += (size_t)kRW * 64 * nc * sizeof(uint32_t);
    l.red = l.rowbuf = reinterpret_cast<float*>(p);
    return l;
}

// What the append does to one session, from the counters before it and the
// session's place among those that take a page (rank).
struct Append {
    bool ok;          // the counters are consistent
    bool app;         // the step's token joins the session
    bool opened;      // in a page off the free list
    bool closed;      // region-aligned: the last page's unused slots become holes
    int n;            // slots in use after the append
    int phys, slot;   // the token's page and place (app)
    int status;       // device status bits
};

__device__ __forceinline__ Append append_of(const Dims& dm, const View& v, int s, int np, int nt, int fc, int rank,
                                            bool any, uint8_t reg) {
    Append a{counters_ok(np, nt, dm), false, false, false, nt, -1, 0, 0};
    if (!a.ok) {
        a.n = 0;
        a.status = kDevCorrupt;
        return a;
    }
    if (!any) return a;
    bool open = !(np > 0 && nt < np * dm.P);
    if (!open) {
        const int p = v.page_table[(size_t)s * dm.MP + np - 1];
        if ((unsigned)p < (unsigned)dm.NP) {
            a.phys = p;
            a.slot = nt - (np - 1) * dm.P;
            if (dm.aligned && a.slot > 0 && v.region[(size_t)p * dm.P + a.slot - 1] != reg) {
                a.closed = open = true;
                a.phys = -1;
                a.n = np * dm.P;
            }
        } else {
            a.status = kDevCorrupt;
        }
    }
    if (open) {
        const int idx = np < dm.MP ? min(fc, dm.NP) - 1 - rank : -1;
        if (idx >= 0) {
            const int p = v.free_list[idx];
            if ((unsigned)p < (unsigned)dm.NP) {
                a.phys = p;
                a.slot = 0;
                a.opened = true;
            } else {
                a.status = kDevCorrupt;
            }
        } else {
            a.status = MD_DEV_CAPACITY;
        }
    }
    a.app = a.phys >= 0;
    a.n += a.app ? 1 : 0;
    return a;
}

// The commit: the counters, page tables and the free list after the append,
// and the scoring kernel's work list.  Whole workgroup.  The workgroup without
// rows (early) arrives once it has worked them out, and leaves them to a
// later one if it is not the last; any other comes here as the last.
__device__ __forceinline__ void rows_commit(const Dims& dm, const View& v, const Scratch& sc, const uint16_t* new_k,
                                            const uint8_t* new_region, bool early) {
    __shared__ int lds[3 * 17];
    __shared__ int sh_mine;
    const int tid = threadIdx.x;
    constexpr int kPer = kMaxSessions / kRT;
    const int fc = v.free_count[0];
    int np[kPer], nt[kPer], op[kPer], clk[kPer], ser[kPer], live[kPer];
    uint8_t reg[kPer];
    int opens = 0;
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
        const int s = tid * kPer + k;
        np[k] = nt[k] = op[k] = clk[k] = ser[k] = live[k] = 0;
        reg[k] = 0;
        if (s < dm.S) {
            np[k] = v.n_pages[s];
            nt[k] = v.n_tokens[s];
            clk[k] = v.clock[s];
            ser[k] = v.next_serial[s];
            live[k] = v.n_live[s];
            if (new_k != nullptr) {
                reg[k] = new_region[s];
                op[k] = opens_page(dm, v, s, new_region) ? 1 : 0;
            }
        }
        opens += op[k];
    }
    int taken;
    int rank = block_exclusive_scan(opens, lds, &taken);
    Append ap[kPer];
    int tiles = 0, tokens = 0;
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
        const int s = tid * kPer + k;
        ap[k] = Append{false, false, false, false, 0, -1, 0, 0};
        if (s < dm.S) {
            ap[k] = append_of(dm, v, s, np[k], nt[k], fc, rank, new_k != nullptr, reg[k]);
            live[k] = dm.aligned ? live[k] + (ap[k].app ? 1 : 0) : ap[k].n;
            tiles += (ap[k].n + kTile - 1) / kTile;
            tokens += ap[k].ok && ap[k].n > 0 ? live[k] : 0;
        }
        rank += op[k];
    }
    const int m[2] = {tiles, tokens};
    int ex[2], tot[2];
    block_exclusive_scan_n<2>(m, lds, ex, tot);
    if (early) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the old counters are in registers
        lds_sync();
        if (tid == 0) sh_mine = arrive_last(sc.rows_read, arrive(sc.rows_read), (int)gridDim.x);
        lds_sync();
        if (!sh_mine) return;
    }
    int st = 0;
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
        const int s = tid * kPer + k;
        if (s >= dm.S) continue;
        const Append& a = ap[k];
        st |= a.status;
        v.clock[s] = clk[k] + 1;
        sc.score_prefix[s] = ex[0];
        sc.chunks[s] = a.n > 0 ? 1 : 0;   // the rows' normalisers are in rstats
        ex[0] += (a.n + kTile - 1) / kTile;
        if (!a.ok) continue;
        if (a.opened) {
            v.page_table[(size_t)s * dm.MP + np[k]] = a.phys;
            v.page_serial[(size_t)s * dm.MP + np[k]] = ser[k];
            if (dm.quant) v.page_format[a.phys] = 0;   // a reused page holds bf16 keys again
            v.next_serial[s] = ser[k] + 1;
            v.n_pages[s] = np[k] + 1;
        }
        v.n_tokens[s] = a.n;
        if (dm.aligned) v.n_live[s] = live[k];
    }
    if (st != 0) atomicOr(sc.status, st);
    if (tid == 0) {
        sc.score_prefix[dm.S] = tot[0];
        v.free_count[0] = max(min(fc, dm.NP) - taken, 0);
        atomicAdd(&sc.counters[0], (unsigned long long)tot[1]);
        atomicAdd(&sc.counters[1], 1ull);
    }
}

// One workgroup's rows of its session, and the session's tokens if it
// finishes them last.  Returns whether the commit is this workgroup's.
template <int GS, bool QT, bool WN>
__device__ __forceinline__ bool rows_work(const Dims& dm, const View& v, const Scratch& sc,
                                          const float* __restrict__ q, const uint16_t* __restrict__ new_k,
                                          const uint8_t* __restrict__ new_region, float* abar_out, int rg,
                                          int nc_cap) {
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ int sh_rank, sh_bad, sh_old, sh_commit;
    const int tid = threadIdx.x, lane = lane_id();
    const int wv = uni(tid >> 6);
    const int s = (int)blockIdx.x / rg, grp = (int)blockIdx.x - s * rg;
    const int r0 = grp * dm.LHkv / rg, r1 = (grp + 1) * dm.LHkv / rg;
    const int G = dm.G * dm.W;
    const RowsLds sm = rows_carve(smem, G, nc_cap, WN);
    const int stride = rows_stride(nc_cap);
    const int h = lane & 15, g = lane >> 4, hh = min(h, G - 1);

    // ---- queries: float4 f = tid of a row (G * 32 <= kRT of them)
    f32x4 qv = f32x4{0.f, 0.f, 0.f, 0.f};
    const bool q_on = tid < G * 32;
    auto load_q = [&](int r) {
        const int f = min(tid, G * 32 - 1), c = f >> 5;
        const int l = r / dm.Hkv, kv = r - l * dm.Hkv, w = c / dm.G, hd = c - w * dm.G;
        qv = reinterpret_cast<const f32x4*>(
            q + ((((size_t)s * dm.W + w) * dm.L + l) * dm.Hq + kv * dm.G + hd) * kHeadDim)[f & 31];
    };
    if (r0 < r1) load_q(r0);

    // ---- the counters before the append; the pages of this wave's tiles
    // (its chunk k is the session's chunk wv + kRW k of 64 tokens, whatever
    // the session's length; lane 4k + u holds tile u of chunk k)
    const int32_t* ptab = v.page_table + (size_t)s * dm.MP;
    const int tile = 4 * (wv + kRW * (lane >> 2)) + (lane & 3);   // lane < kMaxTiles
    const int pg = (tile * 16) >> dm.Pshift;
    int p = -1;
    if (lane < kMaxTiles && pg < dm.MP) p = ptab[pg];
    const int np0 = v.n_pages[s], nt0 = v.n_tokens[s], t_now = v.clock[s] + 1, fc = v.free_count[0];
    const int live0 = v.n_live[s];
    const uint8_t reg_new = new_k != nullptr ? new_region[s] : 0;
    if (tid == 0) sh_rank = sh_bad = 0;
    int rank_mine = 0;
    if (new_k != nullptr)
        for (int s2 = tid; s2 < s; s2 += kRT) rank_mine += opens_page(dm, v, s2, new_region) ? 1 : 0;
    lds_sync();
    if (new_k != nullptr && s > 0) {
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) rank_mine += __shfl_xor(rank_mine, o);
        if (lane == 0 && rank_mine > 0) atomicAdd(&sh_rank, rank_mine);
        lds_sync();
    }
    const Append ap = append_of(dm, v, s, np0, nt0, fc, sh_rank, new_k != nullptr, reg_new);
    const int n = ap.n;
    const int n_old = ap.ok ? nt0 : 0;         // tokens (and holes) before the append
    const int tok_new = ap.app ? n - 1 : -1;

    // every counter this workgroup needs is in registers: say so (the count
    // before it is looked at when the rows are done, so nothing waits for it)
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    lds_sync();
    int arrived = 0;
    if (tid == 0) arrived = arrive(sc.rows_read);

    // ---- tiles
    int myslot = 0;
    bool myok = false, mynew = false;
    if (lane < kMaxTiles && tile * 16 < n) {
        mynew = tok_new >= 0 && (tok_new >> 4) == tile;
        if (ap.opened && pg == np0) p = ap.phys;
        if ((unsigned)p < (unsigned)dm.NP) {
            myslot = (p << dm.Pshift) + ((tile * 16) & (dm.P - 1));
            myok = true;
        } else {
            atomicOr(sc.status, kDevCorrupt);
        }
    }
    const uint32_t vmask = (uint32_t)__ballot(myok);
    const uint32_t nmask = (uint32_t)__ballot(mynew && myok);
    const int i_new = nmask ? __ffs(nmask) - 1 : -1;   // the tile that takes the new token, if this wave's
    const int h_new = tok_new & 15;
    uint32_t qmask = 0;
    if constexpr (QT) qmask = (uint32_t)__ballot(myok && !mynew && v.page_format[myslot >> dm.Pshift] != 0);
    // region-aligned pages: a tile's slots before its first hole (lane i's
    // tile); the slots a closing page leaves unused are holes too
    int mylim = 16;
    if (dm.aligned && myok) {
        const u32x4 rb = *reinterpret_cast<const u32x4*>(v.region + myslot);
        const int used = min(16, max(0, n_old - tile * 16));
        for (int k = 15; k >= 0; --k)
            if (k < used && ((rb[k >> 2] >> (8 * (k & 3))) & 0xffu) == (uint32_t)kHole) mylim = k;
        mylim = min(mylim, used);
    }
    // this wave's chunks: no wave loads tiles that hold no token, but for the
    // last chunk's (what a row loads sets its time)
    const int n_chunks = (n + 63) >> 6;
    const int nc = n_chunks > wv ? min(nc_cap, (n_chunks - wv + kRW - 1) / kRW) : 0;
    // window: bit 4u + i of a chunk's word marks this lane's column as blind
    // to token 4g + i of tile u (inserted after its query's step)
    uint32_t* const blind = sm.unseen + (size_t)wv * nc_cap * 64 + lane;
    if constexpr (WN) {
        const int t_lim = t_now - (dm.W - 1 - min(h / dm.G, dm.W - 1));
        for (int c = 0; c < nc; ++c) {
            uint32_t m = 0;
            for (int u = 0; u < 4; ++u) {
                const int slot = __builtin_amdgcn_readlane(myslot, 4 * c + u);
                const int tok0 = (wv + kRW * c) * 64 + 16 * u + 4 * g;
                if ((vmask >> (4 * c + u)) & 1u) {
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const int ti = tok0 + i == tok_new ? t_now : v.t_ins[slot + 4 * g + i];
                        m |= ti > t_lim ? 1u << (4 * u + i) : 0u;
                    }
                }
            }
            blind[c * 64] = m;
        }
    }

    // ---- this workgroup's rows of the new key, into the pool
    if (ap.app) {
        const u32x4* src = reinterpret_cast<const u32x4*>(new_k) + ((size_t)s * dm.LHkv + r0) * 16;
        for (int i = tid; i < (r1 - r0) * 16; i += kRT) {
            u32x4* blk = reinterpret_cast<u32x4*>(
                v.k_pool + (((size_t)ap.phys * dm.LHkv + r0 + (i >> 4)) * dm.P + (ap.slot & ~15)) * kHeadDim);
            blk[(i & 15) * 16 + (ap.slot & 15)] = src[i];
        }
    }

    // K tile 4c + u of row r in the MFMA A layout (see k_attend); a tile
    // without cached tokens, or past the last row, reads the pool's first
    // tile.  The new token's lanes of its tile read new_k.  No branches: a
    // load under one is copied where the branches meet, and the copy waits
    // for every load in flight.
    auto load_chunk = [&](u32x4 (&ring)[4][4], int r, int c) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int i = 4 * c + u;
            const int slot = __builtin_amdgcn_readlane(myslot, i & 31);
            const bool ok = r < r1 && ((vmask >> (i & 31)) & 1u);
            const size_t e = ok ? ((size_t)(slot >> dm.Pshift) * dm.LHkv + r) * dm.P + (slot & (dm.P - 1)) : 0;
            const uint64_t base = reinterpret_cast<uint64_t>(v.k_pool + e * kHeadDim);
            const uint64_t row = reinterpret_cast<uint64_t>(new_k) + ((size_t)s * dm.LHkv + r) * (kHeadDim * 2);
            const bool fresh = ok && i == i_new && h == h_new;
            const uint64_t from = fresh ? row + 16u * g : base + 16u * lane;
            const uint32_t step = fresh ? 64u : 1024u;
            const bool qt = QT && ok && ((qmask >> (i & 31)) & 1u);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                uint64_t at = from + step * j;
                if (QT && j >= 2) at = qt ? base + 2048u + 16u * (j - 2) : at;
                ring[u][j] = __builtin_nontemporal_load((gvec)at);
            }
        }
    };

    auto store_q = [&](int r) {
        if (!q_on) return;
        uint32_t* qb = sm.qs + (size_t)(r & 1) * 3 * G * 64;
        const int hd = tid >> 5, d2 = 2 * (tid & 31);
        uint32_t t[3][4];
        bool bad = false;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            bad |= !isfinite(qv[e]);
            split3(qv[e], t[0][e], t[1][e], t[2][e]);
        }
#pragma unroll
        for (int k = 0; k < 3; ++k)
            *reinterpret_cast<uint2*>(qb + (k * G + hd) * 64 + d2) =
                make_uint2(t[k][0] | (t[k][1] << 16), t[k][2] | (t[k][3] << 16));
        if (bad) sh_bad = 1;   // the step of the session is void
    };

    // attention mass of the wave's tokens, summed over the rows
    float* const mass = sm.mass + (size_t)wv * 64 * nc_cap + lane;
    for (int c = 0; c < nc; ++c) mass[64 * c] = 0.0f;
    float* const rb = sm.rowbuf + (size_t)wv * G * stride;
    float* const wm = sm.wmax + wv * kMaxNc * 16;
    float run_m = -INFINITY, run_l = 0.0f;   // the row so far, per column

    auto do_chunk = [&](u32x4 (&ring)[4][4], int r, int c, int r_next, int c_next) {
        const uint32_t* qb = sm.qs + (size_t)(r & 1) * 3 * G * 64 + hh * 64 + 4 * g;
        float qsc[4];
        if constexpr (QT) {
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                qsc[u] = 1.0f;
                if ((qmask >> (4 * c + u)) & 1u) {
                    qsc[u] = __uint_as_float(__builtin_amdgcn_readfirstlane(ring[u][2][0]));
                    ring[u][3] = codes_to_bf16<1>(ring[u][1]);
                    ring[u][2] = codes_to_bf16<0>(ring[u][1]);
                    ring[u][1] = codes_to_bf16<1>(ring[u][0]);
                    ring[u][0] = codes_to_bf16<0>(ring[u][0]);
                }
            }
        }
        f32x4 x[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) x[u] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            u32x4 bq[3];
#pragma unroll
            for (int k = 0; k < 3; ++k) bq[k] = *reinterpret_cast<const u32x4*>(qb + k * G * 64 + 16 * j);
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int k = 0; k < 3; ++k)
                    x[u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                        __builtin_bit_cast(bf16x8, ring[u][j]), __builtin_bit_cast(bf16x8, bq[k]), x[u], 0, 0, 0);
        }
        if constexpr (QT) {
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if ((qmask >> (4 * c + u)) & 1u) x[u] *= qsc[u];
        }
        if (c == 0) {   // the next row's query, the one after it requested
            if (r + 1 < r1) store_q(r + 1);
            load_q(min(r + 2, r1 - 1));
        }
        load_chunk(ring, r_next, c_next);
        float mx = -INFINITY;
        uint32_t hide = 0;
        if constexpr (WN) hide = blind[c * 64];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int t0 = (wv + kRW * c) * 64 + 16 * u + 4 * g;
            const bool tv = (vmask >> (4 * c + u)) & 1u;
            const int lim = dm.aligned ? __builtin_amdgcn_readlane(mylim, 4 * c + u) : 16;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const bool live = tv && ((t0 + i < n_old && 4 * g + i < lim) || t0 + i == tok_new) &&
                                  !(WN && ((hide >> (4 * u + i)) & 1u));
                x[u][i] = live ? x[u][i] * kLogitScale : -INFINITY;
                mx = fmaxf(mx, x[u][i]);
            }
        }
        mx = fmaxf(mx, __shfl_xor(mx, 16));
        mx = fmaxf(mx, __shfl_xor(mx, 32));
        const float ms = mx == -INFINITY ? 0.0f : mx;
        float ls = 0.0f;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            f32x4 pv;
#pragma unroll
            for (int i = 0; i < 4; ++i) pv[i] = hw_exp2(x[u][i] - ms);
            ls += (pv[0] + pv[1]) + (pv[2] + pv[3]);
            if (h < G) *reinterpret_cast<f32x4*>(rb + (size_t)h * stride + 64 * c + 16 * u + 4 * g) = pv;
        }
        ls += __shfl_xor(ls, 16);
        ls += __shfl_xor(ls, 32);
        merge_stat(run_m, run_l, mx, ls);
        // (the maximum itself: a chunk that this column does not see weighs
        // 2^-inf = 0 in its row, not 2^(0 - M), which is infinite for M below -128)
        if (g == 0) wm[c * 16 + h] = mx;
        if (c != nc - 1) return;
        // ---- the row is complete: the waves' statistics meet, every wave
        // turns its held values into softmax weights
        if (g == 0) sm.wstat[((r & 1) * kRW + wv) * 16 + h] = make_float2(run_m, run_l);
        run_m = -INFINITY;
        run_l = 0.0f;
        lds_sync();
        float M = -INFINITY, La = 0.0f;
        float2 st[kRW];
#pragma unroll
        for (int k = 0; k < kRW; ++k) {
            st[k] = sm.wstat[((r & 1) * kRW + k) * 16 + h];
            M = fmaxf(M, st[k].x);
        }
        const float Ms = M == -INFINITY ? 0.0f : M;   // a row with no live token gives zero weights
#pragma unroll
        for (int k = 0; k < kRW; ++k) La += st[k].y * hw_exp2(st[k].x - Ms);
        const float inv = La > 0.0f ? 1.0f / La : 0.0f;
        if (dm.H > 0 && wv == 0 && g == 0 && h < G)
            sc.rstats[(size_t)s * dm.R + (size_t)r * G + h] = make_float2(Ms, inv);
        for (int k = 0; k < nc; ++k) {
            const float f = h < G ? hw_exp2(wm[k * 16 + h] - Ms) * inv : 0.0f;
            float a = mass[64 * k];
#pragma unroll
            for (int hd = 0; hd < GS; ++hd) {   // heads past the group read a valid row and weigh zero
                const float fh = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(f), hd));
                a = fmaf(rb[(size_t)min(hd, G - 1) * stride + 64 * k + lane], fh, a);
            }
            mass[64 * k] = a;
        }
    };

    const bool work = n > 0 && r0 < r1;
    if (work && nc == 0) {   // a wave without tokens stages its share of the queries
        store_q(r0);
        load_q(min(r0 + 1, r1 - 1));
        lds_sync();
        for (int r = r0; r < r1; ++r) {
            if (r + 1 < r1) store_q(r + 1);
            load_q(min(r + 2, r1 - 1));
            if (lane < 16) sm.wstat[((r & 1) * kRW + wv) * 16 + lane] = make_float2(-INFINITY, 0.0f);
            lds_sync();
        }
    } else if (work) {
        // Two rings: item k (row, chunk) sits in ring k & 1; item k + 2's
        // loads go out as soon as item k has been through MFMA.
        u32x4 ringA[4][4], ringB[4][4];
        auto step = [&](int& r, int& c) {
            if (++c == nc) {
                c = 0;
                ++r;
            }
        };
        // loads in the order every item issues them, so that no wait for a
        // query is a wait for a whole ring
        int ra = r0, ca = 0;
        store_q(r0);
        load_chunk(ringA, ra, ca);
        load_q(min(r0 + 1, r1 - 1));
        int rb2 = ra, cb = ca;
        step(rb2, cb);
        load_chunk(ringB, rb2, cb);
        lds_sync();
        const int items = (r1 - r0) * nc;
        int rn = rb2, cn = cb, it = 0;
        for (; it + 1 < items; it += 2) {
            step(rn, cn);
            const int r2 = rn, c2 = cn;
            do_chunk(ringA, ra, ca, r2, c2);
            step(rn, cn);
            do_chunk(ringB, rb2, cb, rn, cn);
            ra = r2;
            ca = c2;
            rb2 = rn;
            cb = cn;
        }
        if (it < items) do_chunk(ringA, ra, ca, r1, 0);
    }

    // ---- partial masses, and who finishes the session
    const int cap = nc_cap * 64 * kRW;
    float* part = sc.rows_part + (size_t)s * rg * cap;
    if (work) {
        for (int k = 0; k < nc; ++k) {
            const int tok = (wv + kRW * k) * 64 + lane;
            __hip_atomic_store(part + (size_t)grp * cap + tok, mass[64 * k], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
    // the partial masses are at the coherence point before the session's
    // count says so
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    lds_sync();
    if (tid == 0) {
        if (sh_bad) atomicOr(sc.status, MD_DEV_NONFINITE);
        sh_old = __hip_atomic_fetch_add(sc.rows_done + s, 1 + (sh_bad ? 1 << 16 : 0), __ATOMIC_RELAXED,
                                        __HIP_MEMORY_SCOPE_AGENT);
        sh_commit = arrive_last(sc.rows_read, arrived, (int)gridDim.x);
    }
    lds_sync();
    const bool commit = sh_commit != 0;
    if ((sh_old & 0xffff) != rg - 1) return commit;
    const bool is_void = (sh_old >> 16) != 0 || sh_bad != 0;
    if (tid == 0) {
        sc.rows_done[s] = 0;
        sc.valid[s] = ap.ok && !is_void ? 1 : 0;
    }
    // ---- the session's masses: the ranges' partial masses in a fixed order
    // (wave w adds ranges w, w + kRW, ..., then the waves' sums are added).
    // Eight blocks of 64 tokens at a time, all loads of a wave in flight
    // together: one load after the other cost 25 us of a 41 us launch (56
    // ranges, 671 tokens).
    float* const total = sm.mass;
    for (int b0 = 0; b0 < n_chunks; b0 += 8) {
        float sum[8];
#pragma unroll
        for (int b = 0; b < 8; ++b) sum[b] = 0.0f;
        for (int k0 = wv; k0 < rg; k0 += 4 * kRW) {
            float x[4][8];
#pragma unroll
            for (int k = 0; k < 4; ++k)
#pragma unroll
                for (int b = 0; b < 8; ++b) {
                    const bool on = k0 + k * kRW < rg && b0 + b < n_chunks;
                    const float* at = part + (on ? (size_t)(k0 + k * kRW) * cap + (b0 + b) * 64 + lane : lane);
                    x[k][b] = __hip_atomic_load(at, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
#pragma unroll
            for (int k = 0; k < 4; ++k)
#pragma unroll
                for (int b = 0; b < 8; ++b) sum[b] += k0 + k * kRW < rg ? x[k][b] : 0.0f;
        }
#pragma unroll
        for (int b = 0; b < 8; ++b) sm.red[(wv * 8 + b) * 64 + lane] = sum[b];
        lds_sync();
        float t = 0.0f;
#pragma unroll
        for (int k = 0; k < kRW; ++k) t += sm.red[(k * 8 + wv) * 64 + lane];
        if (b0 + wv < n_chunks) total[(b0 + wv) * 64 + lane] = t;
        lds_sync();
    }
    // ---- the session's tokens: Eq. 2 - 5.  Each page's P tokens are P
    // consecutive lanes.
    const int n_live = dm.aligned ? live0 + (ap.app ? 1 : 0) : n;
    const float aw = attention_weight(dm.alpha, dm.norm_attn, n_live);
    const size_t rbase = (size_t)s * dm.n_regions;
    const float b_l = lane < dm.n_regions ? v.b[rbase + lane] : 0.0f;
    const float lam_l = lane < dm.n_regions ? v.lam[rbase + lane] : 0.0f;
    for (int t0 = wv * 64; t0 < n; t0 += kRT) {
        const int tok = t0 + lane;
        const int tp = tok >> dm.Pshift;
        int phys = -1;
        if (tok < n) phys = (ap.opened && tp == np0) ? ap.phys : ptab[tp];
        const bool in = (unsigned)phys < (unsigned)dm.NP;
        const size_t si = in ? ((size_t)phys << dm.Pshift) + (tok & (dm.P - 1)) : 0;
        const bool fresh = in && tok == tok_new;
        const bool old = in && tok < n_old;
        float a = 0.0f;
        int tr = t_now, r = reg_new;
        if (old) {
            a = v.imp[si];
            tr = v.t_ref[si];
            r = v.region[si];
        }
        const bool live = fresh || (old && !(dm.aligned && r == kHole));
        if (live && r >= dm.n_regions) {
            atomicOr(sc.status, kDevCorrupt);
            r = dm.n_regions - 1;
        }
        const float br = __shfl(b_l, r & 63), lamr = __shfl(lam_l, r & 63);
        float sci = 0.0f;
        bool pin = false;
        if (live && !is_void) {
            const float abar = total[tok] / (float)dm.R;
            a = fmaf(dm.rho, a, (1.0f - dm.rho) * abar);
            v.imp[si] = a;
            const bool hot = abar >= dm.tau_scale / (float)n_live;
            if (hot) tr = t_now;
            if (hot || fresh) v.t_ref[si] = tr;
            if (abar_out != nullptr) abar_out[si] = abar;
            pin = (dm.pin_mask >> r) & 1u;
            sci = pin ? INFINITY : retention_score(br, lamr, t_now, tr, aw, a);
        }
        if (fresh) {
            v.region[si] = reg_new;
            v.t_ins[si] = t_now;
            if (is_void) {
                v.imp[si] = 0.0f;
                v.t_ref[si] = t_now;
            }
        }
        if (ap.closed && in && tok >= n_old && !fresh) {   // the closed page's unused slots
            v.region[si] = (uint8_t)kHole;
            v.t_ins[si] = 0;
            v.t_ref[si] = 0;
            v.imp[si] = 0.0f;
        }
        float ps;
        const bool has = page_score_of(sci, live, pin, dm.P, &ps);
        if ((lane & (dm.P - 1)) == 0 && has && !is_void) sc.pscore[(size_t)s * dm.MP + tp] = ps;
    }
    return commit;
}

// GS: head slots (4, 8 or 16 >= G, the MFMA columns: query heads per KV head
// times window queries); QT: quantised tier; WN: window of several queries.
template <int GS, bool QT, bool WN>
__global__ void __launch_bounds__(kRT) __attribute__((amdgpu_waves_per_eu(2, 2)))
k_rows(Dims dm, View v, Scratch sc, const float* __restrict__ q, const uint16_t* __restrict__ new_k,
       const uint8_t* __restrict__ new_region, float* abar_out, int rg, int nc_cap) {
    const bool rowless = blockIdx.x == gridDim.x - 1;
    if (!rowless && !rows_work<GS, QT, WN>(dm, v, sc, q, new_k, new_region, abar_out, rg, nc_cap)) return;
    rows_commit(dm, v, sc, new_k, new_region, rowless);
}

template <bool QT, bool WN>
const void* rows_for(int G) {
    if (G <= 4) return reinterpret_cast<const void*>(&k_rows<4, QT, WN>);
    if (G <= 8) return reinterpret_cast<const void*>(&k_rows<8, QT, WN>);
    return reinterpret_cast<const void*>(&k_rows<16, QT, WN>);
}

}  // namespace

size_t rows_lds_bytes(int G, int nc, int window) {
    return (size_t)2 * 3 * G * 64 * sizeof(uint32_t) + (size_t)2 * kRW * 16 * sizeof(float2) +
           (size_t)kRW * kMaxNc * 16 * sizeof(float) + (size_t)kRW * 64 * nc * sizeof(float) * (window > 1 ? 2 : 1) +
           std::max((size_t)kRW * 8 * 64, (size_t)kRW * G * rows_stride(nc)) * sizeof(float);
}

const void* rows_kernel(int G, int quant, int window) {
    if (window > 1) return quant ? rows_for<true, true>(G) : rows_for<false, true>(G);
    return quant ? rows_for<true, false>(G) : rows_for<false, false>(G);
}

// 64-token chunks per wave for sessions of up to `tokens` slots; 0 when the
// kernel cannot hold a row of them.
int rows_chunks(int G, int window, int64_t tokens) {
    const int64_t nc = (tokens + 64 * kRW - 1) / (64 * kRW);
    if (nc > kMaxNc || rows_lds_bytes(G, (int)nc, window) > kRowsLds) return 0;
    return (int)std::max<int64_t>(nc, 1);
}

hipError_t launch_rows(const Dims& dm, const View& v, const Scratch& sc, const float* q, const uint16_t* new_k,
                       const uint8_t* new_region, float* abar_out, int rg, hipStream_t st, hipEvent_t t0,
                       hipEvent_t t1) {
    Dims d = dm;
    View vv = v;
    Scratch ss = sc;
    int nc = dm.rows_nc;
    void* args[] = {&d, &vv, &ss, &q, &new_k, &new_region, &abar_out, &rg, &nc};
    const int G = dm.G * dm.W;
    const void* fn = rows_kernel(G, dm.quant, dm.W);
    const dim3 grid(dm.S * rg + 1), block(kRT);
    const unsigned lds = (unsigned)rows_lds_bytes(G, nc, dm.W);
    if (t0 != nullptr && t1 != nullptr) return hipExtLaunchKernel(fn, grid, block, args, lds, st, t0, t1, 0);
    return hipLaunchKernel(fn, grid, block, args, lds, st);
}

}  // namespace md
