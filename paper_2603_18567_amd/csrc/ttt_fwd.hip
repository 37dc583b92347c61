// Forward TTT attention kernel (gfx950): streams K_0/V_0 tiles through LDS with an online softmax
// (Sec. 4.2.1: nothing of size T x T is stored), then folds in the <= j diagonal keys of the later
// cache blocks (suffix part of Alg. 2) row by row on the vector ALU.
//
// Work split: one workgroup = one tile of QT consecutive packed tokens x one query head x one step.
// With two key groups (KS = 2, for launches that would end with a few long workgroups) the halves of a
// workgroup take every second key tile of the same rows and meet at the end, in LDS.
// Each wave owns QB blocks of 32 query rows and keeps, per lane, everything that belongs to ONE
// query row: scores are computed transposed (S^T = K Q^T) so that the accumulator's column index --
// the lane -- is the query row; running max / sum / rescale are then per-lane scalars and the only
// cross-lane traffic of the softmax is one exchange between the two lane halves.  The same layout
// lets exp(S^T) be fed straight back as the B operand of O^T = V^T P^T.
//
// Tiles are cut over the packed token axis, not per document: a row's visible prefix is
// [tok_start[i], i], so a wave visits the kv tiles that intersect [tok_start[first row], last row]
// and nothing else; tiles strictly inside that range for every row skip the mask code.
#include <float.h>

#include <algorithm>
#include <type_traits>

#include "ttt_args.hpp"

namespace ttt {

template <typename T, int D, int QB, int NW, int KS, int WPE, int N>
__global__ __launch_bounds__(NW * 64) __attribute__((amdgpu_waves_per_eu(WPE))) void ttt_fwd_kernel(const FwdArgs<N> a) {
    using E = Elem<T>;
    using frag = typename E::frag;
    constexpr int KT = 64;                // kv rows per LDS tile
    constexpr int KB = KT / 32;
    constexpr int NWG = NW / KS;          // waves of a key group
    constexpr int QT = NWG * QB * 32;
    constexpr int DC = D / 16;            // contraction chunks over head_dim
    constexpr int DB = D / 32;            // 32-wide blocks of head_dim
    constexpr int NT = NW * 64;
    constexpr int TILE_BYTES = KT * D * E::kBytes;
    constexpr float kLazy = 8.f;          // log2 of the largest p tolerated before the reference max moves
    constexpr bool kDiagLds = sizeof(T) == 2;   // diagonal rows may go through LDS

    extern __shared__ __align__(16) char smem[];
    // LDS of a key group: K stage 0, K stage 1, V stage 0, V stage 1
    constexpr int GROUP_BYTES = 4 * TILE_BYTES;
    auto sK = [&](int s) -> char* { return smem + s * TILE_BYTES; };
    auto sV = [&](int s) -> char* { return smem + (2 + s) * TILE_BYTES; };

    const Geometry& geo = a.geo;
    const FwdSlice& sl = slice_of(a, &FwdSlice::first, blockIdx.x);
    int g, rest;
    if (!decode_block(a.map, sl.rest_count, blockIdx.x - sl.first, g, rest)) return;
    // The waves of a workgroup are 2^pack_log2 query heads of the kv group x NW >> pack_log2 blocks of
    // rows: heads that share K_0 / V_0 also share the key range, so all waves of a workgroup see
    // (almost) the same number of key tiles and none idles while the tile on the diagonal is finished.
    const int pk = a.pack_log2;
    const int n_hgrp = geo.G >> pk;
    const int hgrp = rest % n_hgrp;
    rest /= n_hgrp;
    const int j = geo.step_begin + rest % sl.n_steps;
    const int tile = sl.n_tiles - 1 - rest / sl.n_steps;   // long-prefix tiles first

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int kg = KS == 1 ? 0 : wave / NWG, gwave = wave % NWG;   // key group, wave within it
    const int h = g * geo.G + (hgrp << pk) + (gwave & ((1 << pk) - 1));
    const int n = lane & 31, hh = lane >> 5;
    const int t0 = sl.t0, Tn = sl.t1;   // first token of the slice, one past its last
    const int qt_rows = QT >> pk;   // rows of a workgroup
    const int q_tile0 = t0 + tile * qt_rows;
    const int wq0 = q_tile0 + (gwave >> pk) * (QB * 32);
    const bool active = wq0 < Tn;

    const T* Qj = static_cast<const T*>(a.q[j]) + (int64_t)h * geo.q_sh;
    const T* K0 = static_cast<const T*>(a.k[0]) + (int64_t)g * geo.kv_sh;
    const T* V0 = static_cast<const T*>(a.v[0]) + (int64_t)g * geo.kv_sh;

    // rows of this lane, their clamped copies and document starts; the starts of the wave's first and last row
    int qi[QB], qc[QB], st[QB];
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
        qi[qb] = wq0 + 32 * qb + n;
        qc[qb] = qi[qb] < Tn ? qi[qb] : Tn - 1;
    }
    const int hi_w = min(wq0 + QB * 32 - 1, Tn - 1);
    const int hi = min(q_tile0 + qt_rows - 1, Tn - 1);
    int lo, lo_w, st_hi;
    if (a.tok_start) {
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) st[qb] = a.tok_start[qc[qb]];
        lo_w = active ? __builtin_amdgcn_readfirstlane(a.tok_start[min(wq0, Tn - 1)]) : 0;
        st_hi = active ? __builtin_amdgcn_readfirstlane(a.tok_start[hi_w]) : 0;
        lo = __builtin_amdgcn_readfirstlane(a.tok_start[q_tile0]);
    } else {
        // one document start per lane: the last one at or before the workgroup's first row, then those inside its rows
        const int starts = a.cu[sl.doc0 + min(lane, sl.n_docs - 1)];
        int r = __popcll(__ballot(lane < sl.n_docs && starts <= q_tile0)) - 1;
        lo = lo_w = st_hi = __builtin_amdgcn_readlane(starts, r);
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) st[qb] = lo;
        for (++r; r < sl.n_docs; ++r) {
            const int s = __builtin_amdgcn_readlane(starts, r);
            if (s > hi) break;
#pragma unroll
            for (int qb = 0; qb < QB; ++qb) st[qb] = s <= qc[qb] ? s : st[qb];
            lo_w = s <= min(wq0, Tn - 1) ? s : lo_w;
            st_hi = s <= hi_w ? s : st_hi;
        }
    }
    const int u_lo = (lo - t0) / KT, u_hi = (hi - t0) / KT;   // key tiles, counted from t0

    // Q as the stationary B operand: lane (n,hh) holds Q[row n][16t + 8hh .. +8]
    frag qf[QB][DC];
#pragma unroll
    for (int qb = 0; qb < QB; ++qb)
#pragma unroll
        for (int t = 0; t < DC; ++t)
            qf[qb][t] = gload_frag<T>(Qj + (int64_t)qc[qb] * geo.q_st + t * 16 + hh * 8);

    f32x16 oacc[QB][DB];
    float m[QB], l[QB];
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
        m[qb] = -INFINITY;
        l[qb] = 0.f;
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int i = 0; i < 16; ++i) oacc[qb][db][i] = 0.f;
    }
    const float c = geo.scale_log2;

    LaneFrags<T, D> lf;
    // Operand reads at byte offsets from this key group's LDS.  With one key group at head_dim 128 the 64 address
    // registers that sums of pointers take are to be had, and the schedule around them is the better one (seven
    // steps, 64/4 heads, 8192 tokens: 7130 us, 7180 with 32-bit sums; head_dim 64: 4500 against 4070).
    constexpr bool kPointerSums = sizeof(T) == 2 && D == 128 && KS == 1;
    if constexpr (kPointerSums) lf.init(lane);
    else lf.init_at(smem + kg * GROUP_BYTES, lane);
    auto row_frag = [&](uint32_t tile, int rb, int t) -> frag {
        if constexpr (kPointerSums) return lf.rowwise(smem + tile, rb, t);
        else return lf.rowwise_at(tile, rb, t);
    };
    auto col_frag = [&](uint32_t tile, int c16, int db) -> frag {
        if constexpr (kPointerSums) return lf.transposed(smem + tile, c16, db);
        else return lf.transposed_at(tile, c16, db);
    };

    // K_0 / V_0 rows of tile u -> stage s.  Tiles that lie inside the tensor (all but the last one)
    // take the copy with precomputed lane offsets.
    constexpr bool kFastCopy = sizeof(T) == 2;
    struct NoCopy { TTT_DEV void init(int64_t, int) {} };
    typename std::conditional<kFastCopy, TileCopy<T, D, KT, NT>, NoCopy>::type tile_copy;
    tile_copy.init(geo.kv_st, tid);
    auto load_tile = [&](int s, int u0) {
#pragma unroll
        for (int x = 0; x < KS; ++x) {
            const int u = u0 + x;
            if (KS > 1 && u > u_hi) break;
            char* const tk = sK(s) + x * GROUP_BYTES;
            char* const tv = sV(s) + x * GROUP_BYTES;
            if constexpr (kFastCopy) {
                if (t0 + (u + 1) * KT <= Tn) {
                    const int64_t first = (int64_t)(t0 + u * KT) * geo.kv_st;
                    tile_copy.copy(lds_addr(tk), K0 + first);
                    tile_copy.copy(lds_addr(tv), V0 + first);
                    continue;
                }
            }
            int tid_here = tid;
            if constexpr (KS > 1) asm volatile("" : "+v"(tid_here));   // computed here, not carried through the main loop
            tile_load_async<T, D, KT, NT>(tk, K0, geo.kv_st, t0 + u * KT, Tn - 1, tid_here);
            tile_load_async<T, D, KT, NT>(tv, V0, geo.kv_st, t0 + u * KT, Tn - 1, tid_here);
        }
    };

    // Diagonal keys whose rows go through LDS (the waves of a row block want the same K_l / V_l rows): a slot holds the
    // workgroup's rows of one block; a.diag_slots of them lie behind the tile stages.
    const int diag_bytes = a.diag_rows * (D * E::kBytes), slot_bytes = 2 * diag_bytes;
    auto request_diag = [&](int lb, int n, int at) {   // blocks lb .. lb + n - 1 to the slots from byte `at` on
        if constexpr (kDiagLds) {
            for (int i = 0; i < n; ++i, at += slot_bytes) {
                const T* Kl = static_cast<const T*>(a.k[lb + i]) + (int64_t)g * geo.kv_sh;
                const T* Vl = static_cast<const T*>(a.v[lb + i]) + (int64_t)g * geo.kv_sh;
                if (q_tile0 + a.diag_rows <= Tn) {
                    const int64_t first = (int64_t)q_tile0 * geo.kv_st;
                    tile_copy.copy_rows(lds_addr(smem) + at, Kl + first, a.diag_rows);
                    tile_copy.copy_rows(lds_addr(smem) + at + diag_bytes, Vl + first, a.diag_rows);
                } else {
                    int tid_here = tid;
                    asm volatile("" : "+v"(tid_here));   // computed here, not carried through the main loop
                    for (int r = 0; r < a.diag_rows; r += tile_copy.kRowsPerIter) {
                        tile_load_async<T, D, tile_copy.kRowsPerIter, NT>(smem + at + r * (D * E::kBytes), Kl, geo.kv_st, q_tile0 + r, Tn - 1, tid_here);
                        tile_load_async<T, D, tile_copy.kRowsPerIter, NT>(smem + at + diag_bytes + r * (D * E::kBytes), Vl, geo.kv_st, q_tile0 + r, Tn - 1, tid_here);
                    }
                }
            }
        }
    };

    // scores, softmax and O of this wave's rows and the tile in stage ST
    auto tile_work = [&](auto stage_c, const int kv0) {
        constexpr int ST = decltype(stage_c)::value;
        constexpr uint32_t tk = ST * TILE_BYTES, tv = (2 + ST) * TILE_BYTES;
        // S^T[kv, q] = K Q^T
        f32x16 sacc[KB][QB];
#pragma unroll
        for (int kb = 0; kb < KB; ++kb)
#pragma unroll
            for (int qb = 0; qb < QB; ++qb)
#pragma unroll
                for (int i = 0; i < 16; ++i) sacc[kb][qb][i] = 0.f;
#pragma unroll
        for (int t = 0; t < DC; ++t) {
            frag kf[KB];
#pragma unroll
            for (int kb = 0; kb < KB; ++kb) kf[kb] = row_frag(tk, kb, t);
#pragma unroll
            for (int kb = 0; kb < KB; ++kb)
#pragma unroll
                for (int qb = 0; qb < QB; ++qb) sacc[kb][qb] = mma(kf[kb], qf[qb][t], sacc[kb][qb]);
        }
        // mask (only tiles that touch the diagonal or a document start of this wave's rows)
        if (kv0 + KT - 1 > wq0 || kv0 < st_hi) {
#pragma unroll
            for (int kb = 0; kb < KB; ++kb)
#pragma unroll
                for (int qb = 0; qb < QB; ++qb)
#pragma unroll
                    for (int i = 0; i < 16; ++i) {
                        const int kv = kv0 + kb * 32 + acc_row(i, hh);
                        const bool ok = kv <= qi[qb] && kv >= st[qb];
                        sacc[kb][qb][i] = ok ? sacc[kb][qb][i] : -INFINITY;
                    }
        }
        // online softmax, one query row per lane.  The reference maximum m[] is only moved (and O, l
        // rescaled) when a row's tile maximum exceeds it by more than 2^kLazy, so the accumulator
        // rescale is a rare, wave-uniform branch; p stays below 2^kLazy otherwise.
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) {
            float mx = sacc[0][qb][0];
#pragma unroll
            for (int kb = 0; kb < KB; ++kb)
#pragma unroll
                for (int i = 0; i < 16; ++i) mx = fmaxf(mx, sacc[kb][qb][i]);
            mx = half_max(mx);
            const bool grow = (mx - m[qb]) * c > kLazy;   // false while everything is masked (-inf)
            if (__any(grow)) {
                const float m_new = grow ? mx : m[qb];
                const float alpha = grow ? fast_exp2((m[qb] - m_new) * c) : 1.f;   // m = -inf -> 0
                m[qb] = m_new;
                l[qb] *= alpha;
#pragma unroll
                for (int db = 0; db < DB; ++db)
#pragma unroll
                    for (int i = 0; i < 16; ++i) oacc[qb][db][i] *= alpha;
            }
            const float mc = m[qb] == -INFINITY ? 0.f : m[qb] * c;
            float sum = 0.f;
#pragma unroll
            for (int kb = 0; kb < KB; ++kb)
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    const float p = fast_exp2(fmaf(sacc[kb][qb][i], c, -mc));
                    sacc[kb][qb][i] = p;
                    sum += p;
                }
            l[qb] += sum;
        }
        // O^T[d, q] += V^T P^T
#pragma unroll
        for (int c4 = 0; c4 < KT / 16; ++c4) {
            frag pf[QB];
#pragma unroll
            for (int qb = 0; qb < QB; ++qb) pf[qb] = acc_chunk<T>(sacc[c4 / 2][qb], c4 % 2);
#pragma unroll
            for (int db = 0; db < DB; ++db) {
                const frag vf = col_frag(tv, c4, db);
#pragma unroll
                for (int qb = 0; qb < QB; ++qb) oacc[qb][db] = mma(vf, pf[qb], oacc[qb][db]);
            }
        }
    };
    // one kv tile (of each key group), which is in LDS: start the copy of the next one into the other stage, compute from
    // this one, wait for the copy
    auto step = [&](auto stage_c, int u) {
        constexpr int ST = decltype(stage_c)::value;
        if (u + KS <= u_hi) load_tile(ST ^ 1, u + KS);
        const int kv0 = t0 + (u + kg) * KT;
        if (active && kv0 <= hi_w && kv0 + KT - 1 >= lo_w) tile_work(stage_c, kv0);
        wait_async_copies();
        __syncthreads();   // the next tile is in LDS for everyone; everyone is done with this stage
    };

    load_tile(0, u_lo);

    // Diagonal keys of blocks 1..j (suffix part of the mask): one key per block and row.  Row-wise dot products on
    // the vector ALU; straight from global memory they are taken first, so that their latency overlaps the first
    // tile copy.
    // (no_score: the row may have no maximum yet.  A key of score -inf then has weight 0, a NaN stays NaN.)
    auto diag_key = [&](const frag (&dk)[QB][DC], const frag (&dv)[QB][DC], auto no_score) {
        float s[QB];
        float vv[QB][DB][16];   // the key's value row in accumulator order
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) {
            s[qb] = 0.f;
#pragma unroll
            for (int t = 0; t < DC; ++t) s[qb] = dot8(qf[qb][t], dk[qb][t], s[qb]);
            frags_to_acc_order<T, DC>(dv[qb], vv[qb]);
        }
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) {
            const float sc = half_sum(s[qb]);
            const bool grow = (sc - m[qb]) * c > kLazy;   // always for the first key (m = -inf)
            if (__any(grow)) {
                const float m_new = grow ? sc : m[qb];
                const float alpha = grow ? fast_exp2((m[qb] - m_new) * c) : 1.f;
                m[qb] = m_new;
                l[qb] *= alpha;
#pragma unroll
                for (int db = 0; db < DB; ++db)
#pragma unroll
                    for (int i = 0; i < 16; ++i) oacc[qb][db][i] *= alpha;
            }
            const float p = fast_exp2((sc - (decltype(no_score)::value ? fmaxf(m[qb], -FLT_MAX) : m[qb])) * c);
            l[qb] += 0.5f * p;   // the two lane halves are added at the end
#pragma unroll
            for (int db = 0; db < DB; ++db)
#pragma unroll
                for (int i = 0; i < 16; ++i) oacc[qb][db][i] = fmaf(p, vv[qb][db][i], oacc[qb][db][i]);
        }
    };
    if (!(kDiagLds && a.diag_rows > 0) && active && j >= 1 + kg) {
        // the fragments of block lb + 1 are requested from global memory before block lb is consumed
        frag dk[QB][DC], dv[QB][DC], nk[QB][DC], nv[QB][DC];
        auto request = [&](int lb, frag (&rk)[QB][DC], frag (&rv)[QB][DC]) {
            const T* Kl = static_cast<const T*>(a.k[lb]) + (int64_t)g * geo.kv_sh;
            const T* Vl = static_cast<const T*>(a.v[lb]) + (int64_t)g * geo.kv_sh;
#pragma unroll
            for (int qb = 0; qb < QB; ++qb) {
                const T* krow = Kl + (int64_t)qc[qb] * geo.kv_st;
                const T* vrow = Vl + (int64_t)qc[qb] * geo.kv_st;
#pragma unroll
                for (int t = 0; t < DC; ++t) {
                    rk[qb][t] = gload_frag<T>(krow + t * 16 + hh * 8);
                    rv[qb][t] = gload_frag<T>(vrow + t * 16 + hh * 8);
                }
            }
        };
        request(1 + kg, dk, dv);
        for (int lb = 1 + kg; lb <= j; lb += KS) {
            if (lb + KS <= j) request(lb + KS, nk, nv);
            diag_key(dk, dv, IntC<1>{});
#pragma unroll
            for (int qb = 0; qb < QB; ++qb)
#pragma unroll
                for (int t = 0; t < DC; ++t) {
                    dk[qb][t] = nk[qb][t];
                    dv[qb][t] = nv[qb][t];
                }
        }
    }

    wait_async_copies();
    __syncthreads();   // the first tile is in LDS for everyone
    // the diagonal rows of the first blocks are requested behind it and wait in LDS until the tiles are done
    const int diag_first = kDiagLds && a.diag_rows > 0 ? min(j, a.diag_slots) : 0;
    request_diag(1, diag_first, KS * GROUP_BYTES);

    for (int u = u_lo; u <= u_hi; u += 2 * KS) {
        step(IntC<0>{}, u);
        if (u + KS <= u_hi) step(IntC<1>{}, u + KS);
    }

    if constexpr (kDiagLds) {
        // The diagonal keys that wait in LDS; further blocks are requested into the free half -- the tile stages and
        // the blocks' own slots in turn -- before those of the other half are worked on.  (Taken before the tiles,
        // three blocks at a time, every group's copies were waited for: at 4096 tokens 3.4 us per group of a workgroup's
        // 85.)  j is the same for the whole workgroup: the barriers are uniform.
        const int rb = (wq0 - q_tile0) / 32;   // this wave's first row block inside the workgroup's rows
        if (diag_first > 0)
#pragma unroll
            for (int qb = 0; qb < QB; ++qb) m[qb] = fmaxf(m[qb], -FLT_MAX);   // no key of this group so far, or all of score -inf
        int base = 1, at = KS * GROUP_BYTES;
        for (int nb = diag_first; nb > 0;) {
            const int other = at == 0 ? KS * GROUP_BYTES : 0;
            const int more = min(j + 1 - base - nb, at == 0 ? a.diag_slots : KS * GROUP_BYTES / slot_bytes);
            request_diag(base + nb, more, other);
            if (active) {
                for (int i = kg; i < nb; i += KS) {
                    const uint32_t drow = at + i * slot_bytes - kg * GROUP_BYTES;
                    frag dk[QB][DC], dv[QB][DC];
#pragma unroll
                    for (int qb = 0; qb < QB; ++qb)
#pragma unroll
                        for (int t = 0; t < DC; ++t) {
                            dk[qb][t] = row_frag(drow, rb + qb, t);
                            dv[qb][t] = row_frag(drow + diag_bytes, rb + qb, t);
                        }
                    diag_key(dk, dv, IntC<0>{});
                }
            }
            wait_async_copies();
            __syncthreads();
            base += nb;
            nb = more;
            at = other;
        }
    }

    // normalise; rows go through a wave-private LDS patch (carved out of the tile stages, which
    // everybody has finished reading) so that every global store is a full 16-byte piece of a row and a
    // wave instruction covers whole rows
    if constexpr (KS == 2) {
        // The second key group's rows join the first one's: reference maximum, sum and O of the same lane of wave
        // gwave, as 16-byte pieces side by side.  A group that saw no key of a row brings m = -inf, l = 0, O = 0.
        static_assert(NWG * QB * (DB * 4 + 1) * 1024 <= KS * GROUP_BYTES, "one group's rows fit in the tile stages");
        f32x4* piece = reinterpret_cast<f32x4*>(smem) + gwave * (QB * (DB * 4 + 1) * 64) + lane;
        if (kg == 1) {
#pragma unroll
            for (int qb = 0; qb < QB; ++qb) {
#pragma unroll
                for (int db = 0; db < DB; ++db)
#pragma unroll
                    for (int i4 = 0; i4 < 4; ++i4)
                        piece[(qb * (DB * 4 + 1) + db * 4 + i4) * 64] =
                            f32x4{oacc[qb][db][4 * i4], oacc[qb][db][4 * i4 + 1], oacc[qb][db][4 * i4 + 2], oacc[qb][db][4 * i4 + 3]};
                piece[(qb * (DB * 4 + 1) + DB * 4) * 64] = f32x4{m[qb], l[qb], 0.f, 0.f};
            }
        }
        __syncthreads();
        if (kg == 1) return;
        if (active) {
#pragma unroll
            for (int qb = 0; qb < QB; ++qb) {
                const f32x4 ml = piece[(qb * (DB * 4 + 1) + DB * 4) * 64];
                const float m_new = fmaxf(m[qb], ml[0]), off = m_new == -INFINITY ? 0.f : m_new;   // (-inf: every score of the row is)
                const float a0 = fast_exp2((m[qb] - off) * c), a1 = fast_exp2((ml[0] - off) * c);
                m[qb] = m_new;
                l[qb] = l[qb] * a0 + ml[1] * a1;
#pragma unroll
                for (int db = 0; db < DB; ++db)
#pragma unroll
                    for (int i4 = 0; i4 < 4; ++i4) {
                        const f32x4 o4 = piece[(qb * (DB * 4 + 1) + db * 4 + i4) * 64];
#pragma unroll
                        for (int x = 0; x < 4; ++x) oacc[qb][db][4 * i4 + x] = oacc[qb][db][4 * i4 + x] * a0 + o4[x] * a1;
                    }
            }
        }
    }
    if (!active) return;
    char* patch = smem + (KS == 1 ? 0 : NWG * QB * (DB * 4 + 1) * 1024) + gwave * (32 * D * E::kBytes);
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
        const float lt = half_sum(l[qb]);
        const float inv = 1.f / lt;
        if (hh == 0 && qi[qb] < Tn) a.lse[j][(int64_t)h * geo.T + qi[qb]] = m[qb] * geo.scale + __logf(lt);
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int i4 = 0; i4 < 4; ++i4) {
                T* dst = reinterpret_cast<T*>(patch + Tile<T, D>::offset(n, db * 32 + i4 * 8 + hh * 4));
                typename E::vec4 pk;
#pragma unroll
                for (int e = 0; e < 4; ++e) pk[e] = (T)(oacc[qb][db][i4 * 4 + e] * inv);
                *reinterpret_cast<typename E::vec4*>(dst) = pk;
            }
        // the patch is private to the wave: LDS operations of one wave complete in order
        constexpr int PIECES = Tile<T, D>::kPieces;
        T* obase = static_cast<T*>(a.o[j]) + (int64_t)h * geo.q_sh;
#pragma unroll
        for (int it = 0; it < 32 * PIECES / 64; ++it) {
            const int pidx = it * 64 + lane;
            const int r = pidx / PIECES, piece = pidx % PIECES;
            const int row = wq0 + 32 * qb + r;
            const f32x4 val = *reinterpret_cast<const f32x4*>(patch + r * Tile<T, D>::kRowBytes + ((piece ^ Tile<T, D>::swz(r)) * 16));
            if (row < Tn) *reinterpret_cast<f32x4*>(obase + (int64_t)row * geo.q_st + piece * Tile<T, D>::kElemsPerPiece) = val;
        }
    }
}

// ------------------------------------------------------------------------------------------------
// fp32: operands straight from memory
// ------------------------------------------------------------------------------------------------
// One workgroup = 32 tokens x one query head x one step; its eight waves take every eighth block of 32 keys (and every
// eighth diagonal key) and meet once, in LDS.  fp32 matrix instructions are a sixteenth as fast as 16-bit ones, so a block's
// operands (32 KB at head_dim 128) need no LDS to keep up with them, and without tiles to share the waves need no
// barrier before the end: what bounds a short call is one wave's chain of matrix instructions, and this split makes it
// as short as the keys allow (us, tiles in LDS -> so: 128 tokens, 4/4 heads of 64, three steps 13.7 -> 10.2; 247 tokens, 8/1 heads
// of 128, one step 56 -> 21; 444 tokens, 8/2 of 128 113 -> 37).  fwd_f32_direct has the rule.  (Two waves to a SIMD: with head_dim 128 two registers are spilled.)
template <int D, int N>
__global__ __launch_bounds__(512) void ttt_fwd_f32_kernel(const FwdArgs<N> a) {
    constexpr int NW = 8;
    constexpr int DC = D / 16, DB = D / 32;
    constexpr float kLazy = 8.f;                     // as in ttt_fwd_kernel
    constexpr int WAVE_PIECES = DB * 4 + 1;          // 16-byte pieces of a lane: O, and reference maximum and sum
    extern __shared__ __align__(16) char smem[];

    const Geometry& geo = a.geo;
    const FwdSlice& sl = slice_of(a, &FwdSlice::first, blockIdx.x);
    int g, rest;
    if (!decode_block(a.map, sl.rest_count, blockIdx.x - sl.first, g, rest)) return;
    const int h = g * geo.G + rest % geo.G;
    rest /= geo.G;
    const int j = geo.step_begin + rest % sl.n_steps;
    const int tile = sl.n_tiles - 1 - rest / sl.n_steps;   // long-prefix tiles first
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n = lane & 31, hh = lane >> 5;
    const int t0 = sl.t0, Tn = sl.t1;
    const int q0 = t0 + tile * 32, hi = min(q0 + 31, Tn - 1);
    const int qi = q0 + n, qc = min(qi, Tn - 1);

    // document starts of the first row, of the last one and of this lane's
    int lo, st_hi, st;
    if (a.tok_start) {
        st = a.tok_start[qc];
        lo = uniform_load(a.tok_start + q0);
        st_hi = uniform_load(a.tok_start + hi);
    } else {
        const int starts = a.cu[sl.doc0 + min(lane, sl.n_docs - 1)];   // one per lane
        int r = __popcll(__ballot(lane < sl.n_docs && starts <= q0)) - 1;
        lo = st = st_hi = __builtin_amdgcn_readlane(starts, r);
        for (++r; r < sl.n_docs; ++r) {
            const int s = __builtin_amdgcn_readlane(starts, r);
            if (s > hi) break;
            st = s <= qc ? s : st;
            st_hi = s;
        }
    }

    const float* qrow = static_cast<const float*>(a.q[j]) + (int64_t)h * geo.q_sh + (int64_t)qc * geo.q_st + hh * 8;
    f32x8 qf[DC];
#pragma unroll
    for (int t = 0; t < DC; ++t) qf[t] = gload_frag<float>(qrow + t * 16);
    f32x16 oacc[DB];
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int i = 0; i < 16; ++i) oacc[db][i] = 0.f;
    float m = -INFINITY, l = 0.f;
    const float c = geo.scale_log2;
    auto raise = [&](float mx) {   // the reference maximum moves when it is exceeded by 2^kLazy
        const bool grow = (mx - m) * c > kLazy;
        if (__any(grow)) {
            const float m_new = grow ? mx : m;
            const float alpha = grow ? fast_exp2((m - m_new) * c) : 1.f;
            m = m_new;
            l *= alpha;
#pragma unroll
            for (int db = 0; db < DB; ++db)
#pragma unroll
                for (int i = 0; i < 16; ++i) oacc[db][i] *= alpha;
        }
    };

    const float* K0 = static_cast<const float*>(a.k[0]) + (int64_t)g * geo.kv_sh;
    const float* V0 = static_cast<const float*>(a.v[0]) + (int64_t)g * geo.kv_sh;
    for (int kv0 = t0 + ((lo - t0) / 32 + wave) * 32; kv0 <= hi; kv0 += NW * 32) {
        const int last = min(31, Tn - 1 - kv0);
        const float* krow = K0 + (int64_t)(kv0 + min(n, last)) * geo.kv_st + hh * 8;
        const float* v0 = V0 + (int64_t)kv0 * geo.kv_st;
        // S^T[kv, q] = K Q^T; the first half of V is requested behind K and arrives under it
        f32x8 kf[DC], vf[DB];
#pragma unroll
        for (int t = 0; t < DC; ++t) kf[t] = gload_frag<float>(krow + t * 16);
#pragma unroll
        for (int db = 0; db < DB; ++db) vf[db] = gload_cols(v0, geo.kv_st, last, 0, db, n, hh);
        issue_fence();
        f32x16 s;
#pragma unroll
        for (int i = 0; i < 16; ++i) s[i] = 0.f;
#pragma unroll
        for (int t = 0; t < DC; ++t) s = mma(kf[t], qf[t], s);
        f32x8 vg[DB];
#pragma unroll
        for (int db = 0; db < DB; ++db) vg[db] = gload_cols(v0, geo.kv_st, last, 1, db, n, hh);
        issue_fence();
        if (kv0 + 31 > q0 || kv0 < st_hi) {
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const int kv = kv0 + acc_row(i, hh);
                s[i] = kv <= qi && kv >= st ? s[i] : -INFINITY;
            }
        }
        float mx = s[0];
#pragma unroll
        for (int i = 1; i < 16; ++i) mx = fmaxf(mx, s[i]);
        raise(half_max(mx));
        const float mc = m == -INFINITY ? 0.f : m * c;
        float sum = 0.f;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            s[i] = fast_exp2(fmaf(s[i], c, -mc));
            sum += s[i];
        }
        l += sum;
        // O^T[d, q] += V^T P^T
        const f32x8 p0 = acc_chunk<float>(s, 0), p1 = acc_chunk<float>(s, 1);
#pragma unroll
        for (int db = 0; db < DB; ++db) oacc[db] = mma(vf[db], p0, oacc[db]);
#pragma unroll
        for (int db = 0; db < DB; ++db) oacc[db] = mma(vg[db], p1, oacc[db]);
    }
    for (int lb = 1 + wave; lb <= j; lb += NW) {
        const int64_t at = (int64_t)g * geo.kv_sh + (int64_t)qc * geo.kv_st + hh * 8;
        const float *krow = static_cast<const float*>(a.k[lb]) + at, *vrow = static_cast<const float*>(a.v[lb]) + at;
        f32x8 vf[DC];
        float s = 0.f, vv[DB][16];
#pragma unroll
        for (int t = 0; t < DC; ++t) vf[t] = gload_frag<float>(vrow + t * 16);
#pragma unroll
        for (int t = 0; t < DC; ++t) s = dot8(qf[t], gload_frag<float>(krow + t * 16), s);
        frags_to_acc_order<float, DC>(vf, vv);
        s = half_sum(s);
        raise(s);
        const float p = fast_exp2((s - (m == -INFINITY ? 0.f : m)) * c);   // m = -inf: no key of the row yet but of score -inf (p = 0) or NaN
        l += 0.5f * p;   // the two lane halves are added at the end
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int i = 0; i < 16; ++i) oacc[db][i] = fmaf(p, vv[db][i], oacc[db][i]);
    }

    // The waves meet: what each has of a row is scaled to the row's maximum and added, wave w doing pieces w, w + 8, ... of O.
    // A wave that saw no key of a row brings m = -inf, l = 0, O = 0.
    f32x4* const mine = reinterpret_cast<f32x4*>(smem) + wave * (WAVE_PIECES * 64) + lane;
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int i4 = 0; i4 < 4; ++i4)
            mine[(db * 4 + i4) * 64] = f32x4{oacc[db][4 * i4], oacc[db][4 * i4 + 1], oacc[db][4 * i4 + 2], oacc[db][4 * i4 + 3]};
    mine[DB * 4 * 64] = f32x4{m, half_sum(l), 0.f, 0.f};
    __syncthreads();
    const f32x4* const all = reinterpret_cast<const f32x4*>(smem) + lane;
    float wm[NW], wl[NW];
    float m_all = -INFINITY, lt = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
        const f32x4 ml = all[(w * WAVE_PIECES + DB * 4) * 64];
        wm[w] = ml[0];
        wl[w] = ml[1];
        m_all = fmaxf(m_all, wm[w]);
    }
    const float off = m_all == -INFINITY ? 0.f : m_all;   // (-inf: every score of the row is)
#pragma unroll
    for (int w = 0; w < NW; ++w) {
        wm[w] = fast_exp2((wm[w] - off) * c);
        lt += wl[w] * wm[w];
    }
    if (qi >= Tn) return;
    const float inv = 1.f / lt;
    if (wave == 0 && hh == 0) a.lse[j][(int64_t)h * geo.T + qi] = m_all * geo.scale + __logf(lt);
    float* orow = static_cast<float*>(a.o[j]) + (int64_t)h * geo.q_sh + (int64_t)qi * geo.q_st + hh * 4;
    for (int p = wave; p < DB * 4; p += NW) {
        f32x4 o = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            const f32x4 x = all[(w * WAVE_PIECES + p) * 64];
#pragma unroll
            for (int e = 0; e < 4; ++e) o[e] = fmaf(x[e], wm[w], o[e]);
        }
        *reinterpret_cast<f32x4*>(orow + p * 8) = o * inv;
    }
}

template <int D, int N>
static hipError_t launch_fwd_f32_n(const FwdCommon& common, const Slice* slices, int n_slices, hipStream_t stream) {
    constexpr int LDS = 8 * (D / 8 + 1) * 1024;
    auto kern = ttt_fwd_f32_kernel<D, N>;
    static LdsOptIn lds_opt_in;
    if (hipError_t e = lds_opt_in.ensure((const void*)kern, LDS); e != hipSuccess) return e;
    FwdArgs<N> a;
    static_cast<FwdCommon&>(a) = common;
    a.map = head_map(a.geo.hkv);
    int64_t grid = 0;
    for (int i = 0; i < n_slices; ++i) {
        const CallShape& shape = slices[i].shape;
        FwdSlice& sl = a.slices[i];
        sl.first = (int)grid;
        sl.t0 = slices[i].t0;
        sl.t1 = sl.t0 + shape.T;
        sl.n_steps = shape.n_steps;
        sl.doc0 = slices[i].doc0;
        sl.n_docs = shape.n_docs;
        sl.n_tiles = (shape.T + 31) / 32;
        const int64_t rest = (int64_t)sl.n_tiles * shape.n_steps * a.geo.G;
        grid += head_map_grid(a.map, rest);
        if (grid > 0x7fffffffLL) return hipErrorInvalidValue;
        sl.rest_count = (int)rest;
    }
    a.n_slices = n_slices;
    ProfileScope prof("ttt_fwd_f32_kernel", stream);
    hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(512), LDS, stream, a);
    return hipGetLastError();
}

// first / one-past-last token of each token's document
__global__ void ttt_tok_bounds_kernel(const int* __restrict__ cu, int n_docs, int T, int* __restrict__ tok_start,
                                      int* __restrict__ tok_end) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < T) write_doc_bounds(cu, n_docs, i, tok_start, tok_end);
}

hipError_t launch_tok_bounds(const int* cu_dev, int n_docs, int T, int* tok_start, int* tok_end, hipStream_t stream) {
    if (T <= 0) return hipSuccess;
    ProfileScope prof("ttt_tok_bounds_kernel", stream);
    hipLaunchKernelGGL(ttt_tok_bounds_kernel, dim3((T + 255) / 256), dim3(256), 0, stream, cu_dev, n_docs, T, tok_start, tok_end);
    return hipGetLastError();
}

template <typename T, int D, int QB, int NW, int KS, int WPE, int N>
static hipError_t launch_fwd_n(const FwdCommon& common, const Slice* slices, int n_slices, hipStream_t stream) {
    constexpr int PER_CU = WPE * 4 / NW;   // workgroups that share a compute unit
    constexpr int LDS_TILES = fwd_lds_tiles(D, sizeof(T), KS), LDS_MAX = fwd_lds_max(PER_CU);
    auto kern = ttt_fwd_kernel<T, D, QB, NW, KS, WPE, N>;
    static LdsOptIn lds_opt_in;
    if (hipError_t e = lds_opt_in.ensure((const void*)kern, LDS_MAX); e != hipSuccess) return e;
    FwdArgs<N> a;
    static_cast<FwdCommon&>(a) = common;
    const Geometry& geo = a.geo;
    const int qt_rows = (NW / KS * QB * 32) >> a.pack_log2;
    const DiagSlots diag = sizeof(T) == 2 ? fwd_diag_slots(D, NW, KS, PER_CU, qt_rows) : DiagSlots{0, 0};
    a.diag_rows = diag.rows;
    a.diag_slots = diag.slots;
    const int lds_bytes = LDS_TILES + diag.slots * 2 * diag.rows * D * (int)sizeof(T);
    a.map = head_map(geo.hkv);
    int64_t grid = 0;
    for (int i = 0; i < n_slices; ++i) {
        const CallShape& shape = slices[i].shape;
        FwdSlice& sl = a.slices[i];
        sl.first = (int)grid;
        sl.t0 = slices[i].t0;
        sl.t1 = sl.t0 + shape.T;
        sl.n_steps = shape.n_steps;
        sl.doc0 = slices[i].doc0;
        sl.n_docs = shape.n_docs;
        sl.n_tiles = (shape.T + qt_rows - 1) / qt_rows;
        const int64_t rest = (int64_t)sl.n_tiles * shape.n_steps * (geo.G >> a.pack_log2);
        grid += head_map_grid(a.map, rest);
        if (grid > 0x7fffffffLL) return hipErrorInvalidValue;
        sl.rest_count = (int)rest;
    }
    a.n_slices = n_slices;
    // the 16-bit kernels address the pieces of up to 64 rows of K or V with 32-bit byte offsets
    if (sizeof(T) == 2 && geo.kv_st * 64 * (int64_t)sizeof(T) >= (int64_t)1 << 32) return hipErrorInvalidValue;
    ProfileScope prof("ttt_fwd_kernel", stream);
    hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(NW * 64), lds_bytes, stream, a);
    return hipGetLastError();
}

template <typename T, int D, int QB, int NW, int KS, int WPE = NW / 4>
static hipError_t launch_fwd_t(const FwdCommon& a, const Slice* slices, int n_slices, hipStream_t stream) {
    return n_slices > 1 ? launch_fwd_n<T, D, QB, NW, KS, WPE, kMaxSlices>(a, slices, n_slices, stream)
                        : launch_fwd_n<T, D, QB, NW, KS, WPE, 1>(a, slices, n_slices, stream);
}

hipError_t launch_fwd(int dtype, int head_dim, const FwdCommon& common, const Slice* slices, int n_slices, hipStream_t stream) {
    int n_cu = 0;
    if (hipError_t e = current_device_cu_count(n_cu); e != hipSuccess) return e;
    CallShape shapes[kMaxSlices];
    for (int i = 0; i < n_slices; ++i) shapes[i] = slices[i].shape;
    const FwdPlan plan = plan_fwd(shapes, n_slices, dtype == 1, head_dim, n_cu);
    FwdCommon a = common;
    a.pack_log2 = plan.pack_log2;
    const bool two_groups = plan.split == kFwdTwoKeyGroups;
    if (dtype == 1 && head_dim == 128)
        return two_groups ? launch_fwd_t<__bf16, 128, 1, 8, 2>(a, slices, n_slices, stream) : launch_fwd_t<__bf16, 128, 1, 8, 1>(a, slices, n_slices, stream);
    if (dtype == 1 && head_dim == 64) {
        if (two_groups) return launch_fwd_t<__bf16, 64, 1, 8, 2>(a, slices, n_slices, stream);
        if (plan.split == kFwdFourWaves) return launch_fwd_t<__bf16, 64, 1, 4, 1, 3>(a, slices, n_slices, stream);
        return launch_fwd_t<__bf16, 64, 1, 8, 1, 4>(a, slices, n_slices, stream);
    }
    if (dtype == 0 && fwd_f32_direct(shapes, n_slices, head_dim, n_cu, plan, a.geo.kv_st)) {   // operands straight from memory
        if (head_dim == 128) return n_slices > 1 ? launch_fwd_f32_n<128, kMaxSlices>(a, slices, n_slices, stream) : launch_fwd_f32_n<128, 1>(a, slices, n_slices, stream);
        return n_slices > 1 ? launch_fwd_f32_n<64, kMaxSlices>(a, slices, n_slices, stream) : launch_fwd_f32_n<64, 1>(a, slices, n_slices, stream);
    }
    if (dtype == 0 && head_dim == 128) return launch_fwd_t<float, 128, 1, 4, 1>(a, slices, n_slices, stream);
    if (dtype == 0 && head_dim == 64)
        return two_groups ? launch_fwd_t<float, 64, 1, 4, 2>(a, slices, n_slices, stream) : launch_fwd_t<float, 64, 1, 4, 1>(a, slices, n_slices, stream);
    return hipErrorInvalidValue;
}

}  // namespace ttt
