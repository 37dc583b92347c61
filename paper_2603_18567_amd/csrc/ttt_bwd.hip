// Backward TTT attention kernels (gfx950).  Nothing but O and LSE was kept by the forward
// (Sec. 4.2.1), so every kernel here recomputes p = exp(s - LSE) from Q and K tile by tile and
// applies the softmax-attention VJP:  D = <dO,O>, dp = <dO,V>, ds = p (dp - D).
//
//   ttt_bwd_delta_kernel   D for every (step, head, token); 16-bit: -D, from which the dP sums start
//   ttt_bwd_pre_regs_kernel  the same and the complete dK_l, dV_l of the later blocks (16-bit, by a rule on sizes)
//   ttt_bwd_main_kernel    both streaming passes in one launch (ttt_bwd_main_f32_kernel for fp32):
//     dkv_p8_tile, dkv_tile   key-stationary over block 0: dK, dV accumulators of 32 keys per wave in registers
//                          while every (step, head of the group, query block at or below the diagonal) streams
//                          past through LDS; partial sums of the splits meet in fp32 atomics
//     dq_pipe_tile, dq_tile   query-stationary, same streaming structure as the forward: dQ_j
//     diag_unit            the complete dK_l, dV_l of the later cache blocks l >= 1, which are only ever read on the
//                          diagonal (suffix part of Alg. 2), so one small group of lanes owns each (token, kv
//                          head) -- no atomics
//   ttt_bwd_finish_kernel  fp32 block-0 sums -> dK_0, dV_0 in the tensor dtype

#include <algorithm>

#include "ttt_args.hpp"

namespace ttt {

constexpr float kLog2e = 1.44269504088896340736f;

// ------------------------------------------------------------------------------------------------
// D and the diagonal blocks' dK_l, dV_l
// ------------------------------------------------------------------------------------------------
// What the streaming passes need besides, done by further workgroups of the same launch (as launches of their own
// these took longer to start than to run: three of the five or six launches of a short call): document bounds per
// token, and cleared block-0 sums.
TTT_DEV void bwd_pre_side_work(const BwdCommon& a, int blk) {
    const Geometry& geo = a.geo;
    if (blk < a.bounds_blocks) {
        const int i = blk * 256 + threadIdx.x;
        if (i < geo.T) write_doc_bounds(a.cu, a.n_docs, i, a.tok_start, a.tok_end);
        return;
    }
    const int clear_blocks = (int)gridDim.x - a.pre_blocks - a.bounds_blocks;
    for (int64_t i = (int64_t)(blk - a.bounds_blocks) * 256 + threadIdx.x; i < a.clear_n4; i += (int64_t)clear_blocks * 256) {
        reinterpret_cast<f32x4*>(a.dk0_acc)[i] = f32x4{0.f, 0.f, 0.f, 0.f};
        reinterpret_cast<f32x4*>(a.dv0_acc)[i] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
}

// Sum over an aligned group of LPR (4, 8 or 16) lanes with DPP moves only (no LDS traffic):
// quad butterflies, then the half-row and the row mirror pair up quads and half-rows.
template <int LPR> TTT_DEV float group_sum_dpp(float v) {
    auto mv = [](float x, auto ctrl) {
        return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), decltype(ctrl)::value, 0xf, 0xf, true));
    };
    v += mv(v, IntC<0xB1>{});                              // quad_perm [1,0,3,2]
    v += mv(v, IntC<0x4E>{});                              // quad_perm [2,3,0,1]
    if constexpr (LPR >= 8) v += mv(v, IntC<0x141>{});     // row_half_mirror
    if constexpr (LPR >= 16) v += mv(v, IntC<0x140>{});    // row_mirror
    return v;
}

// D and, 16-bit, LSE * log2(e) (the fp32 passes read LSE itself): all that the streaming passes wait for.  Bound by memory (16-bit, 16384
// tokens, 32 heads, one step: 52 us, 5.2 TB/s); one workgroup takes 32 tokens x kDeltaHeads heads of one step: its loads
// are all requested at once (whole rows of neighbouring heads), its results leave as runs of 32 tokens.
constexpr int kDeltaTokens = 32, kDeltaHeads = 4;

template <typename T, int D, int N>
__global__ __launch_bounds__(256) void ttt_bwd_delta_kernel(const BwdArgs<N> a) {
    if ((int)blockIdx.x >= a.pre_blocks) {
        bwd_pre_side_work(a, (int)blockIdx.x - a.pre_blocks);
        return;
    }
    using frag = typename Elem<T>::frag;
    constexpr int LPR = D / 8;
    constexpr int RPP = 256 / LPR;                                   // rows per pass
    constexpr int NP = kDeltaTokens * kDeltaHeads / RPP;
    __shared__ float sum[kDeltaHeads * kDeltaTokens];

    const Geometry& geo = a.geo;
    const BwdSlice& sl = slice_of(a, &BwdSlice::pre_first, blockIdx.x);
    const int n_hc = (geo.hq + kDeltaHeads - 1) / kDeltaHeads;
    const int wg = (int)blockIdx.x - sl.pre_first;
    const int h0 = wg % n_hc * kDeltaHeads;
    const int rest = wg / n_hc;
    const int js = rest % sl.n_steps, t0 = sl.t0 + rest / sl.n_steps * kDeltaTokens;
    const int j = geo.step_begin + js;
    const int grp = threadIdx.x / LPR, sub = threadIdx.x % LPR;
    const T* go_base = static_cast<const T*>(a.d_o[j]) + sub * 8;
    const T* oo_base = static_cast<const T*>(a.o[j]) + sub * 8;

    frag go[NP], oo[NP];
#pragma unroll
    for (int p = 0; p < NP; ++p) {
        const int r = p * RPP + grp;                                 // neighbouring rows are heads of one token
        const int i = min(t0 + r / kDeltaHeads, sl.t1 - 1), h = min(h0 + r % kDeltaHeads, geo.hq - 1);
        const int64_t off = (int64_t)i * geo.q_st + (int64_t)h * geo.q_sh;
        go[p] = gload_frag<T>(go_base + off);
        oo[p] = gload_frag<T>(oo_base + off);
    }
    const int wt = threadIdx.x % kDeltaTokens, wh = threadIdx.x / kDeltaTokens;   // what this thread writes
    const bool writes = wh < kDeltaHeads && h0 + wh < geo.hq && t0 + wt < sl.t1;
    float lse = 0.f;
    if (sizeof(T) == 2 && writes) lse = a.lse[j][(int64_t)(h0 + wh) * geo.T + t0 + wt];
#pragma unroll
    for (int p = 0; p < NP; ++p) {
        const float d = group_sum_dpp<LPR>(dot8(go[p], oo[p], 0.f));
        const int r = p * RPP + grp;
        if (sub == 0) sum[r % kDeltaHeads * kDeltaTokens + r / kDeltaHeads] = d;
    }
    __syncthreads();
    if (writes) {
        const int64_t at = ((int64_t)js * geo.hq + h0 + wh) * geo.T + t0 + wt;
        a.delta[at] = sizeof(T) == 2 ? -sum[wh * kDeltaTokens + wt] : sum[wh * kDeltaTokens + wt];
        if constexpr (sizeof(T) == 2) a.lse2[at] = lse * kLog2e;
    }
}

// dK_l, dV_l of the later blocks: the K_l, V_l rows of a (token, kv head) and their fp32 gradients stay
// in registers while one sweep over (step, head of the group) feeds all of them (the suffix part of Alg. 2 read from
// the key's side: key (l, i) is seen only by the queries (j >= l, i) of Sec. 2.4's unrolled steps).
// kDiagRegBlocks blocks fit (fp32: kDiagRegBlocksF32); with more steps the blocks are taken so many at a time by further workgroups, whose sweeps
// start at the first step that sees one of theirs.  Either workgroups of the streaming launch, with D and LSE at hand,
// or (MAKE_D) the preprocess launch, whose first pass makes these from O on the way.  Bound by memory; the rows of the
// next two pairs are requested before a pair is worked on (4096 tokens, MAKE_D, 0.98 GB: none ahead 4.45 TB/s, one
// 4.75, two 5.07; four, with two blocks fewer in registers, no more).
template <typename T, int D, int THREADS, bool MAKE_D>
TTT_DEV void diag_unit(const BwdCommon& a, const BwdSlice& sl, const int wg) {
    using frag = typename Elem<T>::frag;
    constexpr int NL = sizeof(T) == 2 ? kDiagRegBlocks : kDiagRegBlocksF32, PF = 2;
    constexpr bool kExactLse = sizeof(T) == 4;   // fp32: the difference to the LSE before the factor log2(e), which is the more exact
    constexpr int LPR = D / 8;        // lanes that share one (token, kv head): 8 elements each
    constexpr int UPB = THREADS / LPR;

    const Geometry& geo = a.geo;
    const int Tn = geo.T, G = geo.G, b = geo.step_begin, e = b + sl.n_steps;
    const int per_pass = sl.diag_units / sl.diag_passes;
    const int pass = wg / per_pass;
    const int l0 = 1 + pass * NL;                                 // first block of this pass
    const int j0 = MAKE_D && pass == 0 ? b : max(b, l0);          // first step of its sweep
    const int grp = threadIdx.x / LPR, sub = threadIdx.x % LPR;
    const int64_t unit = (int64_t)(wg % per_pass) * UPB + grp;
    if (unit >= (int64_t)(sl.t1 - sl.t0) * geo.hkv) return;   // whole aligned lane groups leave together
    const int i = sl.t0 + (int)(unit / geo.hkv);
    const int g = (int)(unit % geo.hkv);
    const int64_t kvoff = (int64_t)i * geo.kv_st + (int64_t)g * geo.kv_sh + sub * 8;
    // this lane's place in a block of the carry: two quads D / 2 apart, so that a wave's 16-byte accesses are side by side
    const int64_t coff = ((int64_t)i * geo.hkv + g) * D + sub * 4;
    const int64_t cblk = (int64_t)Tn * geo.hkv * D;

    const int n_pairs = (e - j0) * G;
    frag qf[PF], go[PF], oo[PF];
    float lse[PF], dl[PF];
    auto request = [&](int n, int s) {
        const int j = j0 + n / G, h = g * G + n % G;
        const int64_t off = (int64_t)i * geo.q_st + (int64_t)h * geo.q_sh + sub * 8;
        qf[s] = gload_frag<T>(static_cast<const T*>(a.q[j]) + off);
        go[s] = gload_frag<T>(static_cast<const T*>(a.d_o[j]) + off);
        if constexpr (MAKE_D) {
            oo[s] = gload_frag<T>(static_cast<const T*>(a.o[j]) + off);
            lse[s] = a.lse[j][(int64_t)h * geo.T + i];
        } else {
            const int64_t at = ((int64_t)(j - b) * geo.hq + h) * Tn + i;
            lse[s] = kExactLse ? a.lse[j][(int64_t)h * geo.T + i] : a.lse2[at];
            dl[s] = a.delta[at];
        }
    };
#pragma unroll
    for (int s = 0; s < PF; ++s)
        if (s < n_pairs) request(s, s);

    frag kf[NL], vf[NL];
    float dk[NL][8], dv[NL][8];
#pragma unroll
    for (int l = 0; l < NL; ++l) {
        if (l0 + l < e) {
            kf[l] = gload_frag<T>(static_cast<const T*>(a.k[l0 + l]) + kvoff);
            vf[l] = gload_frag<T>(static_cast<const T*>(a.v[l0 + l]) + kvoff);
        }
#pragma unroll
        for (int x = 0; x < 8; ++x) dk[l][x] = dv[l][x] = 0.f;
    }
    // The carry of the later steps' calls.  16-bit: the sums start from it, so that everything that a unit reads is in flight at
    // once; fp32: it is added to this call's sums, which is the more exact by 1 %.
    auto add_carry = [&]() {
#pragma unroll
        for (int l = 0; l < NL; ++l) {
            if (!a.accumulate || a.carry_reset || l0 + l >= e) break;
            const float* ck = a.dkl_acc + (l0 + l - 1) * cblk + coff;
            const float* cv = a.dvl_acc + (l0 + l - 1) * cblk + coff;
#pragma unroll
            for (int half = 0; half < 2; ++half) {
                const f32x4 k4 = gload_vec4<float>(ck + half * (D / 2)), v4 = gload_vec4<float>(cv + half * (D / 2));
#pragma unroll
                for (int x = 0; x < 4; ++x) {
                    dk[l][4 * half + x] += k4[x];
                    dv[l][4 * half + x] += v4[x];
                }
            }
        }
    };
    if constexpr (sizeof(T) == 2) add_carry();

    for (int n = 0; n < n_pairs; ++n) {
        const int j = j0 + n / G;
        const frag cq = qf[0], cg = go[0], co = oo[0];
        const float lse2 = MAKE_D ? lse[0] * kLog2e : lse[0];
        float dsum = sizeof(T) == 2 ? -dl[0] : dl[0];
#pragma unroll
        for (int s = 0; s + 1 < PF; ++s) {
            qf[s] = qf[s + 1];
            go[s] = go[s + 1];
            oo[s] = oo[s + 1];
            lse[s] = lse[s + 1];
            dl[s] = dl[s + 1];
        }
        if (n + PF < n_pairs) request(n + PF, PF - 1);
        if constexpr (MAKE_D) {
            dsum = group_sum_dpp<LPR>(dot8(cg, co, 0.f));
            if (sub == 0 && pass == 0) {
                const int64_t at = ((int64_t)(j - b) * geo.hq + g * G + n % G) * Tn + i;
                a.delta[at] = -dsum;
                a.lse2[at] = lse2;
            }
        }
        float qx[8], gx[8];
#pragma unroll
        for (int x = 0; x < 8; ++x) {
            qx[x] = to_f32<T>(cq[x]);
            gx[x] = to_f32<T>(cg[x]);
        }
#pragma unroll
        for (int l = 0; l < NL; ++l) {
            if (l0 + l > j) break;             // a block is visible from the step of its own number on
            const float s = group_sum_dpp<LPR>(dot8(cq, kf[l], 0.f));
            const float dp = group_sum_dpp<LPR>(dot8(cg, vf[l], 0.f));
            const float p = fast_exp2(kExactLse ? (s * geo.scale - lse2) * kLog2e : s * geo.scale_log2 - lse2);
            const float ds = p * (dp - dsum) * geo.scale;
#pragma unroll
            for (int x = 0; x < 8; ++x) {
                dk[l][x] = fmaf(ds, qx[x], dk[l][x]);
                dv[l][x] = fmaf(p, gx[x], dv[l][x]);
            }
        }
    }

    if constexpr (sizeof(T) == 4) add_carry();
#pragma unroll
    for (int l = 0; l < NL; ++l) {
        const int lb = l0 + l;
        if (lb >= e) break;
        if (a.accumulate && lb < b) {   // not complete yet: earlier steps' calls have not run
            float* ck = a.dkl_acc + (lb - 1) * cblk + coff;
            float* cv = a.dvl_acc + (lb - 1) * cblk + coff;
#pragma unroll
            for (int half = 0; half < 2; ++half) {
                gstore_vec4<float>(ck + half * (D / 2), dk[l][4 * half], dk[l][4 * half + 1], dk[l][4 * half + 2], dk[l][4 * half + 3]);
                gstore_vec4<float>(cv + half * (D / 2), dv[l][4 * half], dv[l][4 * half + 1], dv[l][4 * half + 2], dv[l][4 * half + 3]);
            }
            continue;
        }
        gstore_frag<T>(static_cast<T*>(a.dk[lb]) + kvoff, dk[l]);
        gstore_frag<T>(static_cast<T*>(a.dv[lb]) + kvoff, dv[l]);
    }
}

template <typename T, int D, int N>
__global__ __launch_bounds__(256) void ttt_bwd_pre_regs_kernel(const BwdArgs<N> a) {
    if ((int)blockIdx.x >= a.pre_blocks) {
        bwd_pre_side_work(a, (int)blockIdx.x - a.pre_blocks);
        return;
    }
    const BwdSlice& sl = slice_of(a, &BwdSlice::pre_first, blockIdx.x);
    diag_unit<T, D, 256, true>(a, sl, (int)blockIdx.x - sl.pre_first);
}

// ------------------------------------------------------------------------------------------------
// dQ: query-stationary
// ------------------------------------------------------------------------------------------------
// fp32, with tiles in LDS
template <typename T, int D, int QB, int NW>
TTT_DEV void dq_tile(const BwdCommon& a, const BwdSlice& sl, char* smem, const int wg) {
    using E = Elem<T>;
    using frag = typename E::frag;
    constexpr int KT = 64;
    constexpr int KB = KT / 32;
    constexpr int QT = NW * QB * 32;
    constexpr int DC = D / 16;
    constexpr int DB = D / 32;
    constexpr int NT = NW * 64;
    constexpr int TILE_BYTES = KT * D * E::kBytes;

    // LDS: K stage 0, K stage 1, V stage 0, V stage 1
    auto sK = [&](int s) -> char* { return smem + s * TILE_BYTES; };
    auto sV = [&](int s) -> char* { return smem + (2 + s) * TILE_BYTES; };

    const Geometry& geo = a.geo;
    int g, rest;
    if (!decode_block(a.map, sl.q_rest, wg, g, rest)) return;
    const int hg = rest % geo.G;
    rest /= geo.G;
    const int js = rest % sl.n_steps;
    const int j = geo.step_begin + js;
    const int t0 = sl.t0, Tn = sl.t1;   // first token of the slice, one past its last
    const int tile = (Tn - t0 + QT - 1) / QT - 1 - rest / sl.n_steps;
    const int h = g * geo.G + hg;

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int n = lane & 31, hh = lane >> 5;
    const int q_tile0 = t0 + tile * QT;
    const int wq0 = q_tile0 + wave * (QB * 32);
    const bool active = wq0 < Tn;

    const T* Qj = static_cast<const T*>(a.q[j]) + (int64_t)h * geo.q_sh;
    const T* dOj = static_cast<const T*>(a.d_o[j]) + (int64_t)h * geo.q_sh;
    const T* K0 = static_cast<const T*>(a.k[0]) + (int64_t)g * geo.kv_sh;
    const T* V0 = static_cast<const T*>(a.v[0]) + (int64_t)g * geo.kv_sh;

    int qi[QB], qc[QB], st[QB];
    float lse2[QB], dl[QB];
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
        qi[qb] = wq0 + 32 * qb + n;
        qc[qb] = qi[qb] < Tn ? qi[qb] : Tn - 1;
        st[qb] = a.tok_start[qc[qb]];
        lse2[qb] = a.lse[j][(int64_t)h * geo.T + qc[qb]] * kLog2e;
        dl[qb] = a.delta[((int64_t)js * geo.hq + h) * geo.T + qc[qb]];
    }
    const int hi_w = min(wq0 + QB * 32 - 1, Tn - 1);
    const int lo_w = active ? __builtin_amdgcn_readfirstlane(a.tok_start[min(wq0, Tn - 1)]) : 0;
    const int st_hi = active ? __builtin_amdgcn_readfirstlane(a.tok_start[hi_w]) : 0;
    const int lo = __builtin_amdgcn_readfirstlane(a.tok_start[q_tile0]);
    const int hi = min(q_tile0 + QT - 1, Tn - 1);
    const int u_lo = (lo - t0) / KT, u_hi = (hi - t0) / KT;   // key tiles, counted from t0

    frag qf[QB][DC], gof[QB][DC];
#pragma unroll
    for (int qb = 0; qb < QB; ++qb)
#pragma unroll
        for (int t = 0; t < DC; ++t) {
            qf[qb][t] = gload_frag<T>(Qj + (int64_t)qc[qb] * geo.q_st + t * 16 + hh * 8);
            gof[qb][t] = gload_frag<T>(dOj + (int64_t)qc[qb] * geo.q_st + t * 16 + hh * 8);
        }

    f32x16 dqacc[QB][DB];
#pragma unroll
    for (int qb = 0; qb < QB; ++qb)
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int i = 0; i < 16; ++i) dqacc[qb][db][i] = 0.f;
    const float c = geo.scale_log2;

    auto load = [&](int s, int u) {
        tile_load_async<T, D, KT, NT>(sK(s), K0, geo.kv_st, t0 + u * KT, Tn - 1, tid);
        tile_load_async<T, D, KT, NT>(sV(s), V0, geo.kv_st, t0 + u * KT, Tn - 1, tid);
    };
    load(0, u_lo);
    int stage = 0;
    for (int u = u_lo; u <= u_hi; ++u) {
        wait_async_copies();
        __syncthreads();
        if (u < u_hi) load(stage ^ 1, u + 1);
        const int kv0 = t0 + u * KT;
        if (active && kv0 <= hi_w && kv0 + KT - 1 >= lo_w) {
            const char* tk = sK(stage);
            const char* tv = sV(stage);
            f32x16 sacc[KB][QB], pacc[KB][QB];
#pragma unroll
            for (int kb = 0; kb < KB; ++kb)
#pragma unroll
                for (int qb = 0; qb < QB; ++qb)
#pragma unroll
                    for (int i = 0; i < 16; ++i) sacc[kb][qb][i] = pacc[kb][qb][i] = 0.f;
            // S^T = K Q^T and dP^T = V dO^T
#pragma unroll
            for (int t = 0; t < DC; ++t) {
#pragma unroll
                for (int kb = 0; kb < KB; ++kb) {
                    const frag kf = frag_rowwise<T, D>(tk, kb * 32 + n, t * 16 + hh * 8);
                    const frag vf = frag_rowwise<T, D>(tv, kb * 32 + n, t * 16 + hh * 8);
#pragma unroll
                    for (int qb = 0; qb < QB; ++qb) {
                        sacc[kb][qb] = mma(kf, qf[qb][t], sacc[kb][qb]);
                        pacc[kb][qb] = mma(vf, gof[qb][t], pacc[kb][qb]);
                    }
                }
            }
            const bool need_mask = kv0 + KT - 1 > wq0 || kv0 < st_hi;
#pragma unroll
            for (int kb = 0; kb < KB; ++kb)
#pragma unroll
                for (int qb = 0; qb < QB; ++qb)
#pragma unroll
                    for (int i = 0; i < 16; ++i) {
                        float p = fast_exp2(fmaf(sacc[kb][qb][i], c, -lse2[qb]));
                        if (need_mask) {
                            const int kv = kv0 + kb * 32 + acc_row(i, hh);
                            p = (kv <= qi[qb] && kv >= st[qb]) ? p : 0.f;
                        }
                        sacc[kb][qb][i] = p * (pacc[kb][qb][i] - dl[qb]);   // dS^T
                    }
            // dQ^T[d, q] += K^T dS^T
#pragma unroll
            for (int c4 = 0; c4 < KT / 16; ++c4) {
                frag sf[QB];
#pragma unroll
                for (int qb = 0; qb < QB; ++qb) sf[qb] = acc_chunk<T>(sacc[c4 / 2][qb], c4 % 2);
#pragma unroll
                for (int db = 0; db < DB; ++db) {
                    const frag kt = frag_transposed<T, D>(tk, c4 * 16, db * 32, lane);
#pragma unroll
                    for (int qb = 0; qb < QB; ++qb) dqacc[qb][db] = mma(kt, sf[qb], dqacc[qb][db]);
                }
            }
        }
        stage ^= 1;
    }
    if (!active) return;

    // diagonal keys of blocks 1..j
    for (int lb = 1; lb <= j; ++lb) {
        const T* Kl = static_cast<const T*>(a.k[lb]) + (int64_t)g * geo.kv_sh;
        const T* Vl = static_cast<const T*>(a.v[lb]) + (int64_t)g * geo.kv_sh;
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) {
            const T* krow = Kl + (int64_t)qc[qb] * geo.kv_st;
            const T* vrow = Vl + (int64_t)qc[qb] * geo.kv_st;
            float s = 0.f, dp = 0.f;
#pragma unroll
            for (int t = 0; t < DC; ++t) {
                const frag kf = gload_frag<T>(krow + t * 16 + hh * 8);
                const frag vf = gload_frag<T>(vrow + t * 16 + hh * 8);
#pragma unroll
                for (int x = 0; x < 8; ++x) {
                    s = fmaf(to_f32<T>(qf[qb][t][x]), to_f32<T>(kf[x]), s);
                    dp = fmaf(to_f32<T>(gof[qb][t][x]), to_f32<T>(vf[x]), dp);
                }
            }
            s += xor32(s);
            dp += xor32(dp);
            const float p = fast_exp2(fmaf(s, c, -lse2[qb]));
            const float ds = p * (dp - dl[qb]);
#pragma unroll
            for (int db = 0; db < DB; ++db)
#pragma unroll
                for (int i4 = 0; i4 < 4; ++i4) {
                    const typename E::vec4 kk = gload_vec4<T>(krow + db * 32 + i4 * 8 + hh * 4);
#pragma unroll
                    for (int x = 0; x < 4; ++x)
                        dqacc[qb][db][i4 * 4 + x] = fmaf(ds, to_f32<T>(kk[x]), dqacc[qb][db][i4 * 4 + x]);
                }
        }
    }

#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
        if (qi[qb] < Tn) {
            T* row = static_cast<T*>(a.dq[j]) + (int64_t)h * geo.q_sh + (int64_t)qi[qb] * geo.q_st;
#pragma unroll
            for (int db = 0; db < DB; ++db)
#pragma unroll
                for (int i4 = 0; i4 < 4; ++i4)
                    gstore_vec4<T>(row + db * 32 + i4 * 8 + hh * 4, dqacc[qb][db][i4 * 4 + 0] * geo.scale,
                                   dqacc[qb][db][i4 * 4 + 1] * geo.scale, dqacc[qb][db][i4 * 4 + 2] * geo.scale,
                                   dqacc[qb][db][i4 * 4 + 3] * geo.scale);
        }
    }
}

// ------------------------------------------------------------------------------------------------
// dQ: query-stationary, 128-row kv tiles (16-bit element types)
//
// One wave = 32 query rows with Q and dO as stationary B operands; a kv tile has 128 rows = 4
// blocks of 32, each taken through S^T, dP^T, dS^T and the dQ^T update in turn, with the LDS
// fragments of the next matrix instructions requested ahead.  Eight waves (two per SIMD) overlap
// one wave's vector work with the other's matrix work.
// With two key groups (KS = 2, short launches: plan_short_bwd) a workgroup has 128 rows and its halves take the two halves of
// every key tile and every second diagonal key, and add up in LDS: a chain half as long for a launch that lasts as long as
// its longest tile (493 tokens, 12/2 heads, the fifth of five steps: backward 34.4 -> 26.5 us).
// LDS: two stages of [K tile | V tile], which differ in one bit of the per-lane addresses.
// ------------------------------------------------------------------------------------------------
template <typename T, int D, int NW, int KS>
TTT_DEV void dq_pipe_tile(const BwdCommon& a, const BwdSlice& sl, char* smem, const int wg) {
    static_assert(sizeof(T) == 2, "this dQ kernel is for 16-bit elements");
    static_assert(NW == 8, "two waves per SIMD supply the overlap; no other wave count is built");
    using E = Elem<T>;
    using frag = typename E::frag;
    using TL = Tile<T, D>;
    constexpr int KT = 128;
    constexpr int KW = KT / KS;       // keys of a tile that a wave works on
    constexpr int NB = KW / 32;
    constexpr int NWG = NW / KS;      // waves of a key group
    constexpr int QT = NWG * 32;
    constexpr int DC = D / 16;
    constexpr int DB = D / 32;
    constexpr int NT = NW * 64;
    constexpr int TILE_BYTES = KT * D * E::kBytes;
    constexpr int STAGE_BYTES = 2 * TILE_BYTES;
    static_assert((STAGE_BYTES & (STAGE_BYTES - 1)) == 0, "the stages differ in one address bit");
    constexpr int NE = 2 * DB;   // matrix instructions of one dQ block update
    constexpr int PDR = 2;       // row-wise K / V fragments requested ahead of their matrix instruction
    constexpr int PDT = 2;       // K^T fragments requested ahead
    typedef __attribute__((address_space(3))) char lds_char;

    const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_char*)smem;

    const Geometry& geo = a.geo;
    int g, rest;
    if (!decode_block(a.map, sl.q_rest, wg, g, rest)) return;
    const int hg = rest % geo.G;
    rest /= geo.G;
    const int js = rest % sl.n_steps;
    const int j = geo.step_begin + js;
    const int t0 = sl.t0, Tn = sl.t1;   // first token of the slice, one past its last
    const int tile = (Tn - t0 + QT - 1) / QT - 1 - rest / sl.n_steps;
    const int h = g * geo.G + hg;

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int n = lane & 31, hh = lane >> 5;
    const int q_tile0 = t0 + tile * QT;
    // key group, wave within it
    const int kg = KS == 1 ? 0 : __builtin_amdgcn_readfirstlane(wave / NWG), gwave = KS == 1 ? wave : wave % NWG;
    const int wq0 = q_tile0 + gwave * 32;
    const bool active = wq0 < Tn;

    const T* Qj = static_cast<const T*>(a.q[j]) + (int64_t)h * geo.q_sh;
    const T* dOj = static_cast<const T*>(a.d_o[j]) + (int64_t)h * geo.q_sh;
    const T* K0 = static_cast<const T*>(a.k[0]) + (int64_t)g * geo.kv_sh;
    const T* V0 = static_cast<const T*>(a.v[0]) + (int64_t)g * geo.kv_sh;

    const int qi = wq0 + n;
    const int qc = qi < Tn ? qi : Tn - 1;
    const int st = a.tok_start[qc];
    const int64_t at = ((int64_t)js * geo.hq + h) * geo.T + qc;
    const float lse2 = a.lse2[at];
    const float ndl = a.delta[at];   // -D
    const int hi_w = min(wq0 + 31, Tn - 1);
    const int first_row = __builtin_amdgcn_readfirstlane(min(wq0, Tn - 1));
    int lo_w = uniform_load(a.tok_start + first_row);
    int st_hi = uniform_load(a.tok_start + max(__builtin_amdgcn_readfirstlane(hi_w), first_row));
    asm volatile("" : "+v"(lo_w), "+v"(st_hi));
    const int lo = uniform_load(a.tok_start + q_tile0);
    const int hi = min(q_tile0 + QT - 1, Tn - 1);
    const int u_lo = (lo - t0) / KT, u_hi = (hi - t0) / KT;   // key tiles, counted from t0

    f32x16 dqacc[DB];
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int i = 0; i < 16; ++i) dqacc[db][i] = 0.f;
    const float c = geo.scale_log2;
    // The dP sums start from -D, which has registers of its own for that: sixteen vector instructions less per block (4096 tokens, 32/8
    // heads, seven steps 4161 -> 4120 us; head_dim 64, 8192 tokens, four steps 5114 -> 5077).
    f32x16 minus_d;
#pragma unroll
    for (int i = 0; i < 16; ++i) minus_d[i] = ndl;
    asm volatile("" : "+v"(minus_d));

    uint32_t ra[DC], ta[DB][2];
    {
        LaneFrags<T, D> lf;
        lf.init(lane);
#pragma unroll
        for (int t = 0; t < DC; ++t) ra[t] = lds0 + lf.row[t] + kg * (KW * TL::kRowBytes);
#pragma unroll
        for (int db = 0; db < DB; ++db) {
            ta[db][0] = lds0 + lf.tr[db][0] + kg * (KW * TL::kRowBytes);
            ta[db][1] = lds0 + lf.tr[db][1] + kg * (KW * TL::kRowBytes);
        }
    }
    auto ld_row = [&](int which, int kb, int t) -> frag {   // which: 0 = K tile, 1 = V tile
        return *reinterpret_cast<const __attribute__((address_space(3))) frag*>(
            (uintptr_t)(ra[t] + which * TILE_BYTES + kb * 32 * TL::kRowBytes));
    };
    auto ld_ktr = [&](int kb, int x) -> frag {   // K^T fragment x = c2 * DB + db of block kb
        typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
        const int c2 = x / DB, db = x % DB;
        const uint32_t off = (kb * 32 + c2 * 16) * TL::kRowBytes;
        union { s16x4 s[2]; frag v; } u;
        u.s[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(uintptr_t)(ta[db][0] + off));
        u.s[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(uintptr_t)(ta[db][1] + off));
        return u.v;
    };
    TileCopy<T, D, KT, NT> tile_copy;
    tile_copy.init(geo.kv_st, tid);
    auto issue = [&](int u, int s) {
        if (t0 + (u + 1) * KT <= Tn) {
            const int64_t first = (int64_t)(t0 + u * KT) * geo.kv_st;
            tile_copy.copy(lds0 + s * STAGE_BYTES, K0 + first);
            tile_copy.copy(lds0 + s * STAGE_BYTES + TILE_BYTES, V0 + first);
        } else {
            char* stg = smem + s * STAGE_BYTES;
            int tid_here = tid;
            asm volatile("" : "+v"(tid_here));   // computed here, not carried through the main loop
            tile_load_async<T, D, KT, NT>(stg, K0, geo.kv_st, t0 + u * KT, Tn - 1, tid_here);
            tile_load_async<T, D, KT, NT>(stg + TILE_BYTES, V0, geo.kv_st, t0 + u * KT, Tn - 1, tid_here);
        }
    };

    // The wave's Q rows, and then its dO rows, come through a region of the stage that the second tile will take, as
    // whole rows: loaded as fragments from global memory they touch 32 rows per instruction and hold up the
    // copies of the first tile behind them (start of a workgroup to its first scores, one step: 128 tokens 4.4 -> 3.5 us,
    // 1024 tokens 6.7 -> 4.5; all seven steps at 4096 tokens, forward and backward 0.5 % less).
    frag qf[DC], gof[DC];
    {
        constexpr int NCP = 32 * TL::kPieces / 64;
        constexpr int ROWS_BYTES = 32 * TL::kRowBytes;
        static_assert(NW * ROWS_BYTES <= STAGE_BYTES, "one region per wave");
        const uint32_t region = __builtin_amdgcn_readfirstlane(lds0 + STAGE_BYTES + wave * ROWS_BYTES);
        int lane_here = lane;
        asm volatile("" : "+v"(lane_here));   // computed here, not carried through the main loop
        uint32_t roff[NCP];
#pragma unroll
        for (int it = 0; it < NCP; ++it) {
            const int pidx = it * 64 + lane_here;
            const int r = pidx / TL::kPieces, pos = pidx % TL::kPieces;   // rows past the end repeat the last one
            roff[it] = (uint32_t)((min(r, Tn - 1 - first_row) * geo.q_st + (pos ^ TL::swz(r)) * TL::kElemsPerPiece) * (int64_t)sizeof(T));
        }
        auto request = [&](const T* base) {
#pragma unroll
            for (int it = 0; it < NCP; ++it) async_copy16(base + (int64_t)first_row * geo.q_st, roff[it], region + it * 1024);
        };
        LaneFrags<T, D> lf;
        lf.init(lane_here);
        const char* rows = smem + STAGE_BYTES + wave * ROWS_BYTES;
        request(Qj);
        issue(u_lo, 0);
        wait_copies_but(IntC<2 * TILE_BYTES / (NT * 16)>{});
#pragma unroll
        for (int t = 0; t < DC; ++t) qf[t] = lf.rowwise(rows, 0, t);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // the region is read out: refill it
        request(dOj);
        wait_async_copies();
#pragma unroll
        for (int t = 0; t < DC; ++t) gof[t] = lf.rowwise(rows, 0, t);
    }
    int stage = 0;
    for (int u = u_lo; u <= u_hi; ++u) {
        wait_async_copies();
        __syncthreads();
        if (u < u_hi) issue(u + 1, stage ^ 1);
        const int kv0 = t0 + u * KT + kg * KW;
        if (active && kv0 <= hi_w && kv0 + KW - 1 >= lo_w) {
            frag ka[DC], va[DC];   // row-wise K / V fragments of the block being scored
            frag tfr[NE];          // K^T fragments of the block being accumulated
            frag sfr[2];           // dS^T operands of the previous block
            f32x16 sacc, pacc;
            auto prime_rows = [&](int kb) {
#pragma unroll
                for (int t = 0; t < PDR; ++t) {
                    ka[t] = ld_row(0, kb, t);
                    va[t] = ld_row(1, kb, t);
                }
            };
            // S^T[kv, q] = K Q^T and dP^T[kv, q] = V dO^T (lane = query row)
            auto score = [&](int kb) {
#pragma unroll
                for (int i = 0; i < 16; ++i) sacc[i] = 0.f;
                pacc = minus_d;
#pragma unroll
                for (int t = 0; t < DC; ++t) {
                    if (t + PDR < DC) {
                        ka[t + PDR] = ld_row(0, kb, t + PDR);
                        va[t + PDR] = ld_row(1, kb, t + PDR);
                    }
                    issue_fence();
                    sacc = mma(ka[t], qf[t], sacc);
                    pacc = mma(va[t], gof[t], pacc);
                }
            };
            {
                // Two waves per SIMD: no pipelining inside the wave.  One wave's vector work runs
                // while the other wave of the SIMD uses the matrix core (they fall into opposite
                // phases by themselves); blocks that this wave's rows cannot see are skipped.
                bool primed = false;
#pragma unroll
                for (int kb = 0; kb < NB; ++kb) {
                    const int kb0 = kv0 + kb * 32;
                    if (kb0 > hi_w || kb0 + 31 < lo_w) {
                        primed = false;
                        continue;
                    }
                    if (!primed) prime_rows(kb);
                    score(kb);
                    // requests that do not depend on the vector work below
#pragma unroll
                    for (int x = 0; x < PDT; ++x) tfr[x] = ld_ktr(kb, x);
                    primed = kb + 1 < NB && !(kb0 + 32 > hi_w || kb0 + 63 < lo_w);
                    if (primed) prime_rows(kb + 1);
                    issue_fence();
                    const bool need_mask = kb0 + 31 > wq0 || kb0 < st_hi;
                    if (need_mask) {
#pragma unroll
                        for (int x = 0; x < 16; ++x) {
                            const int kv = kb0 + acc_row(x, hh);
                            float p = fast_exp2(fmaf(sacc[x], c, -lse2));
                            p = (kv <= qi && kv >= st) ? p : 0.f;
                            pacc[x] *= p;   // dS^T
                        }
                    } else {
#pragma unroll
                        for (int x = 0; x < 16; ++x) pacc[x] *= fast_exp2(fmaf(sacc[x], c, -lse2));
                    }
                    sfr[0] = acc_chunk<T>(pacc, 0);
                    sfr[1] = acc_chunk<T>(pacc, 1);
#pragma unroll
                    for (int x = 0; x < NE; ++x) {
                        if (x + PDT < NE) tfr[x + PDT] = ld_ktr(kb, x + PDT);
                        issue_fence();
                        dqacc[x % DB] = mma(tfr[x], sfr[x / DB], dqacc[x % DB]);
                    }
                }
            }
        }
#pragma unroll
        for (int t = 0; t < DC; ++t) ra[t] ^= STAGE_BYTES;
#pragma unroll
        for (int db = 0; db < DB; ++db) {
            ta[db][0] ^= STAGE_BYTES;
            ta[db][1] ^= STAGE_BYTES;
        }
        stage ^= 1;
    }
    __syncthreads();   // everybody is done with the tile stages: they become the store patches
    if (KS == 1 && !active) return;

    // Diagonal keys of blocks 1..j.  The workgroup's LDS is free now and every wave has 16 KB of it to
    // itself (its store patch lies inside): the K_l / V_l rows of the wave's 32 tokens are copied there
    // by LDS-DMA as whole 256-byte rows (fragment loads straight from global memory would touch 32 rows
    // with 32 bytes each per instruction) and read back as fragments; the copy of block lb + 1 is
    // requested as soon as the fragments of block lb are in registers.
    constexpr int WAVE_LDS = 2 * 32 * D * E::kBytes;
    static_assert(NW * WAVE_LDS <= 2 * STAGE_BYTES, "one region per wave");
    char* wbuf = smem + wave * WAVE_LDS;
    if (active && j >= 1 + kg) {
        frag dk[DC], dv[DC];
        auto request = [&](int lb) {   // straight from global memory (rows past the end clamped)
            const T* krow = static_cast<const T*>(a.k[lb]) + (int64_t)g * geo.kv_sh + (int64_t)qc * geo.kv_st;
            const T* vrow = static_cast<const T*>(a.v[lb]) + (int64_t)g * geo.kv_sh + (int64_t)qc * geo.kv_st;
#pragma unroll
            for (int t = 0; t < DC; ++t) {
                dk[t] = gload_frag<T>(krow + t * 16 + hh * 8);
                dv[t] = gload_frag<T>(vrow + t * 16 + hh * 8);
            }
        };
        auto apply = [&]() {
            float s = 0.f, dp = 0.f;
            uint32_t kk[DC][4];   // the key row in accumulator order, still packed
#pragma unroll
            for (int t = 0; t < DC; ++t) {
                s = dot8(qf[t], dk[t], s);
                dp = dot8(gof[t], dv[t], dp);
            }
            frags_to_acc_order_packed<T, DC>(dk, kk);
            s = half_sum(s);
            dp = half_sum(dp);
            const float p = fast_exp2(fmaf(s, c, -lse2));
            const float ds = p * (dp + ndl);
#pragma unroll
            for (int db = 0; db < DB; ++db)
#pragma unroll
                for (int i = 0; i < 16; ++i) dqacc[db][i] = fmaf(ds, acc_order_elem<DC>(kk, db, i), dqacc[db][i]);
        };
        if (wq0 + 32 <= Tn) {
            constexpr int NCP = 32 * TL::kPieces / 64;   // copy instructions per 32-row matrix
            uint32_t doff[NCP];                          // this lane's piece: bytes from the first row
            int lane_here = lane;
            asm volatile("" : "+v"(lane_here));          // computed here, not carried through the main loop
#pragma unroll
            for (int it = 0; it < NCP; ++it) {
                const int pidx = it * 64 + lane_here;
                const int r = pidx / TL::kPieces, pos = pidx % TL::kPieces;
                doff[it] = (uint32_t)((r * geo.kv_st + (pos ^ TL::swz(r)) * TL::kElemsPerPiece) * (int64_t)sizeof(T));
            }
            const uint32_t wl = __builtin_amdgcn_readfirstlane(lds0 + wave * WAVE_LDS);
            const int wq0u = __builtin_amdgcn_readfirstlane(wq0);   // wave-uniform copies of per-wave values
            auto copy = [&](int lb) {
                const T* kb = static_cast<const T*>(a.k[lb]) + (int64_t)g * geo.kv_sh + (int64_t)wq0u * geo.kv_st;
                const T* vb = static_cast<const T*>(a.v[lb]) + (int64_t)g * geo.kv_sh + (int64_t)wq0u * geo.kv_st;
#pragma unroll
                for (int it = 0; it < NCP; ++it) {
                    async_copy16(kb, doff[it], wl + it * 1024);
                    async_copy16(vb, doff[it], wl + WAVE_LDS / 2 + it * 1024);
                }
            };
            LaneFrags<T, D> lf;
            lf.init(lane_here);
            copy(1 + kg);
            for (int lb = 1 + kg; lb <= j; lb += KS) {
                wait_async_copies();
#pragma unroll
                for (int t = 0; t < DC; ++t) {
                    dk[t] = lf.rowwise(wbuf, 0, t);
                    dv[t] = lf.rowwise(wbuf + WAVE_LDS / 2, 0, t);
                }
                if (lb + KS <= j) {
                    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // the region is read out: refill it
                    copy(lb + KS);
                }
                apply();
            }
        } else {
            for (int lb = 1 + kg; lb <= j; lb += KS) {
                request(lb);
                apply();
            }
        }
    }

    if constexpr (KS == 2) {
        // the second group's rows join the first one's: 16-byte pieces of the same lane of wave gwave
        static_assert(DB * 4 * 1024 <= WAVE_LDS, "a wave's rows fit in its region");
        f32x4* piece = reinterpret_cast<f32x4*>(smem + gwave * WAVE_LDS) + lane;
        __syncthreads();   // everybody is done with the diagonal keys
        if (kg == 1) {
#pragma unroll
            for (int db = 0; db < DB; ++db)
#pragma unroll
                for (int i4 = 0; i4 < 4; ++i4)
                    piece[(db * 4 + i4) * 64] = f32x4{dqacc[db][4 * i4], dqacc[db][4 * i4 + 1], dqacc[db][4 * i4 + 2], dqacc[db][4 * i4 + 3]};
        }
        __syncthreads();
        if (kg == 1 || !active) return;
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int i4 = 0; i4 < 4; ++i4) {
                const f32x4 o4 = piece[(db * 4 + i4) * 64];
#pragma unroll
                for (int x = 0; x < 4; ++x) dqacc[db][4 * i4 + x] += o4[x];
            }
    }

    // scaled rows go through a wave-private LDS patch so that global stores are whole 16-byte pieces
    char* patch = wbuf;
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int i4 = 0; i4 < 4; ++i4) {
            typename E::vec4 pk;
#pragma unroll
            for (int x = 0; x < 4; ++x) pk[x] = (T)(dqacc[db][i4 * 4 + x] * geo.scale);
            *reinterpret_cast<typename E::vec4*>(patch + TL::offset(n, db * 32 + i4 * 8 + hh * 4)) = pk;
        }
    T* obase = static_cast<T*>(a.dq[j]) + (int64_t)h * geo.q_sh;
#pragma unroll
    for (int it = 0; it < 32 * TL::kPieces / 64; ++it) {
        const int pidx = it * 64 + lane;
        const int r = pidx / TL::kPieces, piece = pidx % TL::kPieces;
        const int row = wq0 + r;
        const f32x4 val = *reinterpret_cast<const f32x4*>(patch + r * TL::kRowBytes + ((piece ^ TL::swz(r)) * 16));
        if (row < Tn) *reinterpret_cast<f32x4*>(obase + (int64_t)row * geo.q_st + piece * TL::kElemsPerPiece) = val;
    }
}

// ------------------------------------------------------------------------------------------------
// dK_0, dV_0: key-stationary
// ------------------------------------------------------------------------------------------------
template <typename T, int D, int NW>
TTT_DEV void dkv_tile(const BwdCommon& a, const BwdSlice& sl, char* smem, const int wg) {
    using E = Elem<T>;
    using frag = typename E::frag;
    constexpr int KVT = NW * 32;   // kv rows per workgroup, 32 per wave
    constexpr int QTL = 64;        // query rows per LDS tile
    constexpr int DC = D / 16;
    constexpr int DB = D / 32;
    constexpr int NT = NW * 64;
    constexpr int TILE_BYTES = QTL * D * E::kBytes;
    constexpr int ROWV_BYTES = QTL * 4;
    constexpr int STAGE_BYTES = 2 * TILE_BYTES + 3 * ROWV_BYTES;

    auto sQ = [&](int s) -> char* { return smem + s * STAGE_BYTES; };
    auto sG = [&](int s) -> char* { return smem + s * STAGE_BYTES + TILE_BYTES; };
    auto sLse = [&](int s) -> float* { return reinterpret_cast<float*>(smem + s * STAGE_BYTES + 2 * TILE_BYTES); };
    auto sDl = [&](int s) -> float* { return sLse(s) + QTL; };
    auto sSt = [&](int s) -> int* { return reinterpret_cast<int*>(sLse(s) + 2 * QTL); };

    const Geometry& geo = a.geo;
    int g, rest;
    if (!decode_block(a.map, sl.kv_rest, wg, g, rest)) return;
    const int sp = rest % sl.n_split;
    const int tile = rest / sl.n_split;   // low tiles of a document have the longest query range: first

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int n = lane & 31, hh = lane >> 5;
    const int t0 = sl.t0, Tn = sl.t1;   // first token of the slice, one past its last
    const int kv_tile0 = t0 + tile * KVT;
    const int wk0 = kv_tile0 + wave * 32;          // first kv row of this wave
    const bool active = wk0 < Tn;
    const int wk_hi = min(wk0 + 31, Tn - 1);
    // query rows that can see this workgroup's / this wave's keys
    const int q_end = __builtin_amdgcn_readfirstlane(a.tok_end[min(kv_tile0 + KVT - 1, Tn - 1)]);
    const int wq_end = active ? __builtin_amdgcn_readfirstlane(a.tok_end[wk_hi]) : 0;
    const int qt_lo = tile * (KVT / QTL), nqt = (q_end - 1 - t0) / QTL - qt_lo + 1;   // query tiles, counted from t0
    if (nqt <= 0) return;
    const int n_jh = sl.n_steps * geo.G;
    const int n_c = (n_jh - sp + sl.n_split - 1) / sl.n_split;   // (step, head) pairs of this split
    const int n_it = n_c * nqt;

    const T* K0 = static_cast<const T*>(a.k[0]) + (int64_t)g * geo.kv_sh;
    const T* V0 = static_cast<const T*>(a.v[0]) + (int64_t)g * geo.kv_sh;
    const int kc = min(wk0 + n, Tn - 1);
    const int kvi = wk0 + n;   // this lane's kv row (accumulator column)
    // K_0, V_0 rows as stationary B operands: lane (n,hh) holds row n, elements 16t + 8hh .. +8
    frag kf[DC], vf[DC];
#pragma unroll
    for (int t = 0; t < DC; ++t) {
        kf[t] = gload_frag<T>(K0 + (int64_t)kc * geo.kv_st + t * 16 + hh * 8);
        vf[t] = gload_frag<T>(V0 + (int64_t)kc * geo.kv_st + t * 16 + hh * 8);
    }
    f32x16 dkacc[DB], dvacc[DB];
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int i = 0; i < 16; ++i) dkacc[db][i] = dvacc[db][i] = 0.f;
    const float c = geo.scale_log2;

    // stage loader: query tile `qt` of (step, head) pair number `ci` of this split
    auto issue = [&](int it, int s) {
        const int ci = it / nqt, qt = qt_lo + it % nqt;
        const int jh = sp + ci * sl.n_split;
        const int js = jh / geo.G, h = g * geo.G + jh % geo.G;
        const int j = geo.step_begin + js;
        const T* Qj = static_cast<const T*>(a.q[j]) + (int64_t)h * geo.q_sh;
        const T* dOj = static_cast<const T*>(a.d_o[j]) + (int64_t)h * geo.q_sh;
        tile_load_async<T, D, QTL, NT>(sQ(s), Qj, geo.q_st, t0 + qt * QTL, Tn - 1, tid);
        tile_load_async<T, D, QTL, NT>(sG(s), dOj, geo.q_st, t0 + qt * QTL, Tn - 1, tid);
        if (tid < QTL) {
            const int q = t0 + qt * QTL + tid;
            const bool in = q < Tn;
            const int qq = in ? q : Tn - 1;
            // rows past the end get LSE = +inf so that p = 0
            sLse(s)[tid] = in ? a.lse[j][(int64_t)h * geo.T + qq] * kLog2e : INFINITY;
            sDl(s)[tid] = in ? a.delta[((int64_t)js * geo.hq + h) * geo.T + qq] : 0.f;
            sSt(s)[tid] = a.tok_start[qq];
        }
    };

    if (n_it > 0) issue(0, 0);
    int stage = 0;
    for (int it = 0; it < n_it; ++it) {
        wait_async_copies();
        __syncthreads();
        if (it + 1 < n_it) issue(it + 1, stage ^ 1);
        const int q0 = t0 + (qt_lo + it % nqt) * QTL;
        // this wave's keys are seen by query rows [wk0, wq_end)
        if (active && q0 + QTL - 1 >= wk0 && q0 < wq_end) {
            const char* tq = sQ(stage);
            const char* tg = sG(stage);
            const float* tl = sLse(stage);
            const float* td = sDl(stage);
            const int* ts = sSt(stage);
#pragma unroll
            for (int qb = 0; qb < QTL / 32; ++qb) {
                const int qb0 = q0 + qb * 32;
                if (qb0 + 31 < wk0 || qb0 >= wq_end) continue;
                // fragments are read where they are used (this kernel serves the fp32 instantiation;
                // 16-bit types take dkv_p8_tile)
                frag qa[DC], ga[DC], gt[2][DB], qt[2][DB];
                // S[q, kv] = Q K^T and dP[q, kv] = dO V^T : lane = kv column, values = query rows
                f32x16 sacc, pacc;
#pragma unroll
                for (int i = 0; i < 16; ++i) sacc[i] = pacc[i] = 0.f;
#pragma unroll
                for (int t = 0; t < DC; ++t) {
                    qa[t] = frag_rowwise<T, D>(tq, qb * 32 + n, t * 16 + hh * 8);
                    ga[t] = frag_rowwise<T, D>(tg, qb * 32 + n, t * 16 + hh * 8);
                    sacc = mma(qa[t], kf[t], sacc);
                    pacc = mma(ga[t], vf[t], pacc);
                }
                // every row of the block sees every key of the wave iff the block is below the
                // wave's last key and starts its document at or before the wave's first key
                const bool need_mask = qb0 < wk0 + 31 || ts[min(qb * 32 + 31, QTL - 1)] > wk0 || qb0 + 31 >= wq_end;
#pragma unroll
                for (int i4 = 0; i4 < 4; ++i4) {
                    const int r = qb * 32 + i4 * 8 + hh * 4;
                    const f32x4 l4 = *reinterpret_cast<const f32x4*>(tl + r);
                    const f32x4 d4 = *reinterpret_cast<const f32x4*>(td + r);
#pragma unroll
                    for (int x = 0; x < 4; ++x) {
                        const int i = i4 * 4 + x;
                        float p = fast_exp2(fmaf(sacc[i], c, -l4[x]));
                        if (need_mask) {
                            const int q = q0 + r + x;
                            p = (kvi <= q && kvi >= ts[r + x]) ? p : 0.f;
                        }
                        sacc[i] = p;                       // P
                        pacc[i] = p * (pacc[i] - d4[x]);   // dS
                    }
                }
                // dV[kv, d] += P^T dO ;  dK[kv, d] += dS^T Q
#pragma unroll
                for (int c2 = 0; c2 < 2; ++c2) {
                    const frag pf = acc_chunk<T>(sacc, c2);
                    const frag sf = acc_chunk<T>(pacc, c2);
#pragma unroll
                    for (int db = 0; db < DB; ++db) {
                        gt[c2][db] = frag_transposed<T, D>(tg, qb * 32 + c2 * 16, db * 32, lane);
                        qt[c2][db] = frag_transposed<T, D>(tq, qb * 32 + c2 * 16, db * 32, lane);
                        dvacc[db] = mma(pf, gt[c2][db], dvacc[db]);
                        dkacc[db] = mma(sf, qt[c2][db], dkacc[db]);
                    }
                }
            }
        }
        stage ^= 1;
    }
    if (!active) return;

    // fp32 partial sums of this split -> block-0 accumulators [T][hkv][D]
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const int kv = wk0 + acc_row(i, hh);
            if (kv < Tn) {
                const int64_t off = ((int64_t)kv * geo.hkv + g) * D + db * 32 + n;
                atomicAdd(a.dk0_acc + off, dkacc[db][i]);
                atomicAdd(a.dv0_acc + off, dvacc[db][i]);
            }
        }
}

// ------------------------------------------------------------------------------------------------
// dK_0, dV_0: key-stationary, eight equal waves (16-bit element types)
//
// Measured on MI355X: a wave issues at most one instruction (of any kind) every ~8 cycles, so the
// time of a step is close to 8 cycles x the instructions a wave executes in it, and the two waves of
// a SIMD are worth most as two independent instruction streams doing the same work on different
// data.  Hence: eight equal waves, and as few instructions per block as the arithmetic allows (stage
// offsets as immediates in an unrolled pair of steps, pointers advanced instead of recomputed, LDS
// reads and waits in pairs).  Workgroup = 128
// key rows; wave w owns the 32 keys of pair w & 3 (fp32 dK, dV accumulators in registers) and takes
// every second query block: group w >> 2 = parity of the block.  The K_0 / V_0 rows of the tile sit
// in LDS for the whole tile (row-wise B operands of S = Q K^T and dP = dO V^T); query blocks (Q and
// dO rows, LSE*log2e, D, document start) stream through a two-stage LDS ring, each group copying the
// blocks it will use.  P and dS never leave the registers: the 16 accumulator values of a lane are
// already two A-operand chunks of dV += P^T dO and dK += dS^T Q, whose B operands are read
// transposed from the same stage.  One workgroup barrier per pair of blocks.  The two waves that
// share a key range both add their partial sums to the fp32 accumulators in global memory.
// ------------------------------------------------------------------------------------------------
template <typename T, int D> struct DkvP8 {
    static constexpr int kKeys = 128;
    static constexpr int kBlk = 32 * D * (int)sizeof(T);      // one 32-row block of one matrix
    static constexpr int kSlot = 2 * kBlk;                    // Q block + dO block of one query block
    static constexpr int kStage = 2 * kSlot;                  // one query block per wave group
    static constexpr int kStages = 2;
    static constexpr int kKBase = kStages * kStage;
    static constexpr int kVBase = kKBase + kKeys * D * (int)sizeof(T);
    static constexpr int kVecBase = kVBase + kKeys * D * (int)sizeof(T);
    static constexpr int kVecSlot = 3 * 32 * 4;               // LSE*log2e, D, first token of the document
    static constexpr int kVecStage = 2 * kVecSlot;
    static constexpr int kLds = kVecBase + kStages * kVecStage;
    // K and V rows, operand-major: [32 columns][16 keys][16-byte piece of the columns][key].  Where the row fragment of
    // chunk t (16 columns) starts, from a lane's place on:
    static constexpr int chunk_at(int t) { return (t >> 1) * kKeys * 64 + (t & 1) * 512; }
};

template <typename T, int D>
__device__ __forceinline__ void dkv_p8_tile(const BwdCommon& a, const BwdSlice& sl, char* smem, const int g, const int sp,
                                            const int tile, const int chunk) {
    static_assert(sizeof(T) == 2, "this dK/dV kernel is for 16-bit elements");
    using E = Elem<T>;
    using frag = typename E::frag;
    using TL = Tile<T, D>;
    using C = DkvP8<T, D>;
    constexpr int KVT = C::kKeys;
    constexpr int DC = D / 16;
    constexpr int DB = D / 32;
    constexpr int NE = 4 * DB;                // dV / dK matrix instructions per block
    static_assert((C::kStage & (C::kStage - 1)) == 0, "the stage bit is toggled with XOR");
    typedef __attribute__((address_space(3))) char lds_char;
    typedef __attribute__((address_space(3))) frag lds_frag;
    typedef __attribute__((address_space(3))) s16x4 lds_s16x4;

    const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_char*)smem;
    const Geometry& geo = a.geo;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int pair = wave & 3, grp = wave >> 2;
    const int n = lane & 31, hh = lane >> 5;
    const int t0 = sl.t0, Tn = sl.t1;   // first token of the slice, one past its last
    const int kv_tile0 = t0 + tile * KVT;
    const int wk0 = kv_tile0 + pair * 32;
    const bool active = wk0 < Tn;
    const int wk_hi = min(wk0 + 31, Tn - 1);
    const int q_end = uniform_load(a.tok_end + min(kv_tile0 + KVT - 1, Tn - 1));
    const int wk_end = uniform_load(a.tok_end + wk_hi), wk_start = uniform_load(a.tok_start + wk_hi);   // of the last key's document
    const int kvi = wk0 + n;
    // K_0, V_0 rows of the tile -> LDS, while the document bounds are on their way.  The layout gives a lane one address
    // register for all its row fragments of K and V, consecutive lanes consecutive 16-byte pieces, and a copy
    // instruction 64 bytes of each of 16 rows (after the bounds, with 32 bytes of 32 rows, the requests end 2.1 us after the
    // workgroup's start, 1.4 so; 128 tokens, 32/8 heads, a pass of seven steps one by one 208 -> 204 us).
    {
        const int row = min(kv_tile0 + wave * 16 + (lane & 15), Tn - 1);
        const int64_t off = (int64_t)row * geo.kv_st + (int64_t)g * geo.kv_sh + (lane >> 4) * 8;
        const T* K0 = static_cast<const T*>(a.k[0]) + off;
        const T* V0 = static_cast<const T*>(a.v[0]) + off;
        const uint32_t dst = __builtin_amdgcn_readfirstlane(lds0 + wave * 1024);
#pragma unroll
        for (int t = 0; t < DC; t += 2) {
            async_copy16(K0 + t * 16, dst + C::kKBase + C::chunk_at(t));
            async_copy16(V0 + t * 16, dst + C::kVBase + C::chunk_at(t));
        }
    }

    const int wq_end = active ? wk_end : 0;
    const bool wave_split = active && wk_start > wk0;
    // query blocks of this chunk that see a key of this tile, counted from t0
    const int qb_lo = max(tile * (KVT / 32), chunk * sl.chunk_blocks);
    const int nqb = min((q_end - 1 - t0) / 32, (chunk + 1) * sl.chunk_blocks - 1) - qb_lo + 1;
    if (nqb <= 0) {
        wait_async_copies();   // nothing may land in LDS that is the next workgroup's
        return;
    }
    const int wq_lim = min(wq_end, t0 + (qb_lo + nqb) * 32);   // blocks from here on are not this unit's
    const int n_split = sl.n_split;
    const int n_jh = sl.n_steps * geo.G;
    const int n_c = (n_jh - sp + n_split - 1) / n_split;
    const int nqb2 = (nqb + 1) / 2;           // steps per (step, head) pair: one block per wave group
    const int n_steps2 = n_c * nqb2;
    const float c = geo.scale_log2;

    // per-lane LDS addresses: query-block fragments (this group's slot of stage 0), the pair's K rows
    uint32_t ra[DC], ta[DB][2];
    const uint32_t ka = lds0 + C::kKBase + pair * 2048 + (n >> 4) * 1024 + hh * 256 + (n & 15) * 16;
    static_assert(C::chunk_at(DC - 1) + C::kVBase - C::kKBase < 65536, "LDS offsets are 16-bit immediates");
    {
        LaneFrags<T, D> lf;
        lf.init(lane);
#pragma unroll
        for (int t = 0; t < DC; ++t) ra[t] = lds0 + lf.row[t] + grp * C::kSlot;
#pragma unroll
        for (int db = 0; db < DB; ++db) {
            ta[db][0] = lds0 + lf.tr[db][0] + grp * C::kSlot;
            ta[db][1] = lds0 + lf.tr[db][1] + grp * C::kSlot;
        }
    }
    const uint32_t va = lds0 + C::kVecBase + grp * C::kVecSlot + hh * 16;
    auto ld = [&](uint32_t addr) -> frag { return *reinterpret_cast<const lds_frag*>((uintptr_t)addr); };
    auto ld_tr = [&](uint32_t stage_off, int which, int c2, int db) -> frag {
        const uint32_t off = stage_off + which * C::kBlk + c2 * 16 * TL::kRowBytes;
        union { s16x4 s[2]; frag v; } u;
        u.s[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(uintptr_t)(ta[db][0] + off));
        u.s[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(uintptr_t)(ta[db][1] + off));
        return u.v;
    };
    auto ld_vec = [&](uint32_t off, int i4) -> f32x4 {
        return *reinterpret_cast<const __attribute__((address_space(3))) f32x4*>((uintptr_t)(va + off + i4 * 32));
    };

    // ---- copies: the 256 threads of a group copy the group's next block (32 x kPieces 16-byte
    // pieces per matrix) and its three per-row vectors.  Group grp takes the query blocks
    // qb_lo + 2 nqb2 - 1 - grp - 2 i, i < nqb2, of one (step, head) pair after the other; if the number
    // of blocks is odd, the first block of group 0 lies past every query that sees the tile and is
    // skipped.  The sweep runs from the last query block down to the tile's own: all key tiles of a
    // (kv head, split) start a pair at the same block, so the workgroups that share an XCD read the
    // same Q / dO rows at about the same time and find them in its L2.
    constexpr int NLD = 32 * TL::kPieces / 256;
    const int gw = wave & 3, gt = tid & 255;
    uint32_t src_off[NLD];
#pragma unroll
    for (int i = 0; i < NLD; ++i) {
        const int pidx = (i * 4 + gw) * 64 + lane;
        const int r = pidx / TL::kPieces, pos = pidx % TL::kPieces;
        src_off[i] = (uint32_t)((r * geo.q_st + (pos ^ TL::swz(r)) * TL::kElemsPerPiece) * (int64_t)sizeof(T));
    }
    const uint32_t vec_off = (uint32_t)(lane & 31) * 4;
    const uint32_t dst0 = __builtin_amdgcn_readfirstlane(lds0 + grp * C::kSlot + gw * 1024);
    const uint32_t vdst0 = __builtin_amdgcn_readfirstlane(lds0 + C::kVecBase + grp * C::kVecSlot);
    const int64_t blk2_stride = (int64_t)64 * geo.q_st;       // two blocks, in elements
    const int row_top = t0 + (qb_lo + 2 * nqb2 - 1 - grp) * 32;   // this group's first block: the sweep runs downwards
    struct Pos {
        int i, ci;             // block 2 i + grp of (step, head) pair number ci of this split
        const T *q, *g;        // first row of the block in Q_j and dO_j of that head
    };
    const T *head_q = nullptr, *head_g = nullptr;             // of the pair the next request is in
    const float *head_l = nullptr, *head_d = nullptr;
    auto enter_pair = [&](Pos& ps) {
        const int jh = sp + ps.ci * n_split;
        const int js = jh / geo.G, h = g * geo.G + jh % geo.G;
        const int j = geo.step_begin + js;
        head_q = static_cast<const T*>(a.q[j]) + (int64_t)h * geo.q_sh;
        head_g = static_cast<const T*>(a.d_o[j]) + (int64_t)h * geo.q_sh;
        const int64_t at = ((int64_t)js * geo.hq + h) * geo.T;
        head_l = a.lse2 + at;
        head_d = a.delta + at;
        const int64_t first = (int64_t)row_top * geo.q_st;
        ps.q = head_q + first;
        ps.g = head_g + first;
    };
    auto advance = [&](Pos& ps) {
        if (++ps.i == nqb2) {
            ps.i = 0;
            ++ps.ci;
            if (ps.ci < n_c) enter_pair(ps);
        } else {
            ps.q -= blk2_stride;
            ps.g -= blk2_stride;
        }
    };
    auto request = [&](const Pos& ps, auto stage_c) {
        constexpr int ST = decltype(stage_c)::value;
        const uint32_t st = dst0 + ST * C::kStage;
        const uint32_t vec = vdst0 + ST * C::kVecStage;
        const int row0 = row_top - 64 * ps.i;
        if (row0 + 32 <= Tn) {
#pragma unroll
            for (int i = 0; i < NLD; ++i) {
                async_copy16(ps.q, src_off[i], st + i * 4096);
                async_copy16(ps.g, src_off[i], st + C::kBlk + i * 4096);
            }
            if (gt < 32) {
                async_copy4(head_l + row0, vec_off, vec);
                async_copy4(head_d + row0, vec_off, vec + 128);
                async_copy4(a.tok_start + row0, vec_off, vec + 256);
            }
        } else {
#pragma unroll
            for (int i = 0; i < NLD; ++i) {
                const int pidx = (i * 4 + gw) * 64 + lane;
                const int r = pidx / TL::kPieces, pos = pidx % TL::kPieces;
                const int row = min(row0 + r, Tn - 1);            // rows past the end are masked later
                const int64_t off = (int64_t)row * geo.q_st + (pos ^ TL::swz(r)) * TL::kElemsPerPiece;
                async_copy16(head_q + off, st + i * 4096);
                async_copy16(head_g + off, st + C::kBlk + i * 4096);
            }
            if (gt < 32) {
                const int qq = min(row0 + gt, Tn - 1);
                async_copy4(head_l + qq, vec);
                async_copy4(head_d + qq, vec + 128);
                async_copy4(a.tok_start + qq, vec + 256);
            }
        }
    };
    Pos nxt{0, 0, nullptr, nullptr};
    enter_pair(nxt);
    request(nxt, IntC<0>{});

    f32x16 dkacc[DB], dvacc[DB];
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int i = 0; i < 16; ++i) dkacc[db][i] = dvacc[db][i] = 0.f;

    wait_async_copies();
    __syncthreads();

    // KR of the pair's K row fragments stay in registers, as many as there is room for: the scores' operand reads
    // are what loads LDS most (1.5 KB per matrix instruction, 1.34 with these: 4096 tokens, seven steps, six of them 3480 -> 3415 us;
    // with six beside the dP sums that start from -D four registers spill and everything is 3 to 5 % slower, with five or four
    // none does and they are equal)
    constexpr int KR = DC < 5 ? DC : 5;
    frag kreg[KR];
#pragma unroll
    for (int t = 0; t < KR; ++t) kreg[t] = ld(ka + C::chunk_at(t));

    // One step: request the blocks of the next step into the other stage, then this wave's block from
    // stage ST (a compile-time constant, so that every LDS address is a register plus an immediate).
    auto step = [&](const bool more, auto stage_c) {
        constexpr int ST = decltype(stage_c)::value;
        constexpr uint32_t SO = ST * C::kStage;
        constexpr uint32_t VO = ST * C::kVecStage;
        const int q0 = row_top - 64 * nxt.i;
        if (more) {
            advance(nxt);
            request(nxt, IntC<1 - ST>{});
        }
        if (active && q0 + 31 >= wk0 && q0 < wq_lim) {
            // ---- S = Q K^T, dP - D = dO V^T - D for the pair's 32 keys, two contraction chunks at a time.  The dP sums start
            // from -D, read before the scores: read where dP begins it is waited for (the backward 3 % slower than with the
            // subtraction), so it takes the place of sixteen vector instructions a block (forward and backward of 4096 tokens, 32/8
            // heads, one step a call 0.5 % faster; head_dim 64, 4431 tokens, eight steps 3768 -> 3683 us).
            f32x16 sacc, pacc;
#pragma unroll
            for (int i4 = 0; i4 < 4; ++i4) {
                const f32x4 d4 = ld_vec(VO + 128, i4);
#pragma unroll
                for (int x = 0; x < 4; ++x) pacc[4 * i4 + x] = d4[x];
            }
            {
                frag qa[DC], kf[DC];
#pragma unroll
                for (int t = 0; t < 2; ++t) {
                    qa[t] = ld(ra[t] + SO);
                    kf[t] = t < KR ? kreg[t < KR ? t : 0] : ld(ka + C::chunk_at(t));
                }
#pragma unroll
                for (int i = 0; i < 16; ++i) sacc[i] = 0.f;
#pragma unroll
                for (int t = 0; t < DC; t += 2) {
                    if (t + 2 < DC) {
#pragma unroll
                        for (int u = t + 2; u < t + 4; ++u) {
                            qa[u] = ld(ra[u] + SO);
                            kf[u] = u < KR ? kreg[u < KR ? u : 0] : ld(ka + C::chunk_at(u));
                        }
                    }
                    issue_fence();
                    sacc = mma(qa[t], kf[t], sacc);
                    sacc = mma(qa[t + 1], kf[t + 1], sacc);
                }
            }
            {
                frag ga[DC], vf[DC];
#pragma unroll
                for (int t = 0; t < 2; ++t) {
                    ga[t] = ld(ra[t] + SO + C::kBlk);
                    vf[t] = ld(ka + C::chunk_at(t) + (C::kVBase - C::kKBase));
                }
#pragma unroll
                for (int t = 0; t < DC; t += 2) {
                    if (t + 2 < DC) {
#pragma unroll
                        for (int u = t + 2; u < t + 4; ++u) {
                            ga[u] = ld(ra[u] + SO + C::kBlk);
                            vf[u] = ld(ka + C::chunk_at(u) + (C::kVBase - C::kKBase));
                        }
                    }
                    issue_fence();
                    pacc = mma(ga[t], vf[t], pacc);
                    pacc = mma(ga[t + 1], vf[t + 1], pacc);
                }
            }
            // ---- P and dS.  Every row of the block sees every key of the pair iff the block lies at
            // or below the pair's last key, ends before that key's document does, and the pair's keys
            // are all in one document
            const bool need_mask = q0 < wk0 + 31 || q0 + 31 >= wq_end || wave_split;
            {
                f32x4 l4[4];
#pragma unroll
                for (int i4 = 0; i4 < 4; ++i4) l4[i4] = ld_vec(VO, i4);
                if (need_mask) {
                    f32x4 s4[4];
#pragma unroll
                    for (int i4 = 0; i4 < 4; ++i4) s4[i4] = ld_vec(VO + 256, i4);
#pragma unroll
                    for (int x = 0; x < 16; ++x) {
                        const int q = q0 + acc_row(x, hh);
                        const float p = fast_exp2(fmaf(sacc[x], c, -l4[x / 4][x % 4]));
                        const bool see = (kvi <= q) & (q < wq_end) & (kvi >= __float_as_int(s4[x / 4][x % 4]));
                        sacc[x] = see ? p : 0.f;
                    }
                } else {
#pragma unroll
                    for (int x = 0; x < 16; ++x) sacc[x] = fast_exp2(fmaf(sacc[x], c, -l4[x / 4][x % 4]));
                }
            }
            issue_fence();
            frag tfr[NE];
#pragma unroll
            for (int x = 0; x < 2; ++x) tfr[x] = ld_tr(SO, 1 - (x & 1), (x >> 1) / DB, (x >> 1) % DB);
#pragma unroll
            for (int x = 0; x < 16; ++x) pacc[x] *= sacc[x];
            // ---- dV += P^T dO, dK += dS^T Q: the accumulator chunks are the A operands as they are
            frag pfr[2], sfr[2];
#pragma unroll
            for (int c2 = 0; c2 < 2; ++c2) {
                pfr[c2] = acc_chunk<T>(sacc, c2);
                sfr[c2] = acc_chunk<T>(pacc, c2);
            }
            // transposed fragment x = (c2 * DB + db) * 2 + (0: dO for dV, 1: Q for dK), two at a time
#pragma unroll
            for (int x = 0; x < NE; x += 2) {
                if (x + 2 < NE) {
#pragma unroll
                    for (int y = x + 2; y < x + 4; ++y) tfr[y] = ld_tr(SO, 1 - (y & 1), (y >> 1) / DB, (y >> 1) % DB);
                }
                issue_fence();
                const int c2 = (x >> 1) / DB, db = (x >> 1) % DB;
                dvacc[db] = mma(pfr[c2], tfr[x], dvacc[db]);
                dkacc[db] = mma(sfr[c2], tfr[x + 1], dkacc[db]);
            }
        }
        wait_async_copies();
        lds_barrier();   // the blocks of the next step are in LDS; everybody is done with those of this one
    };
    for (int s = 0; s < n_steps2; s += 2) {
        step(s + 1 < n_steps2, IntC<0>{});
        if (s + 1 < n_steps2) step(s + 2 < n_steps2, IntC<1>{});
    }
    // The two waves of a key range add their sums in LDS (the last barrier of the loop has freed all of it): group 0 hands
    // its dV over and ends with the sums of dK, group 1 the other way round, so that eight waves request the atomics
    // (from four waves, each row's address worked out per lane: 5.1 us of a unit's end, 2.3 so; 128 tokens, 32/8 heads, a
    // pass of seven steps one by one 216 -> 210 us).  Quad q of what a lane hands over sits at
    // (q * 256 + pair * 64 + lane) * 16 bytes of its group's half.
    constexpr int HALF_BYTES = DB * 4 * 256 * 16;
    static_assert(2 * HALF_BYTES <= C::kLds, "the sums that change hands fit in LDS");
    typedef __attribute__((address_space(3))) f32x4 lds_f32x4;
    const uint32_t sum_addr = lds0 + (pair * 64 + lane) * 16;
    if (grp == 1) {
#pragma unroll
        for (int db = 0; db < DB; ++db) {
            const f32x16 t = dkacc[db];
            dkacc[db] = dvacc[db];
            dvacc[db] = t;
        }
    }
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int i4 = 0; i4 < 4; ++i4)
            *(lds_f32x4*)(uintptr_t)(sum_addr + grp * HALF_BYTES + (db * 4 + i4) * 4096) =
                f32x4{dvacc[db][4 * i4], dvacc[db][4 * i4 + 1], dvacc[db][4 * i4 + 2], dvacc[db][4 * i4 + 3]};
    __syncthreads();
    if (!active) return;
    // rows of the block-0 sums: a uniform base per row and a lane's place in it
    float* const acc = (grp == 0 ? a.dk0_acc : a.dv0_acc) + ((int64_t)wk0 * geo.hkv + g) * D;
    const int64_t row = (int64_t)geo.hkv * D;
    const uint32_t lane_at = (uint32_t)(4 * hh) * (uint32_t)row + n;
    auto flush = [&](auto whole) {
#pragma unroll
        for (int i4 = 0; i4 < 4; ++i4)
#pragma unroll
            for (int db = 0; db < DB; ++db) {
                const f32x4 s4 = *(const lds_f32x4*)(uintptr_t)(sum_addr + (grp ^ 1) * HALF_BYTES + (db * 4 + i4) * 4096);
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (decltype(whole)::value || wk0 + acc_row(4 * i4 + e, hh) < Tn)
                        atomicAdd(acc + (8 * i4 + e) * row + lane_at + db * 32, dkacc[db][4 * i4 + e] + s4[e]);
            }
    };
    if (wk0 + 32 <= Tn) flush(IntC<1>{});
    else flush(IntC<0>{});
}

// One workgroup = one key tile x one chunk of `chunk_blocks` query blocks x one split of the
// (step, head) list of the kv head.  Units are numbered chunk by chunk, the tiles that a chunk can
// see (those that begin at or before its last row) side by side: workgroups with consecutive numbers
// stream the same Q / dO rows, (step, head) pair after pair, each pair costing all of them the same
// number of blocks -- except the few tiles on the chunk's diagonal -- so they stay together and the
// rows are read from HBM once per XCD, not once per workgroup.
template <typename T, int D>
TTT_DEV void dkv_p8_unit(const BwdCommon& a, const BwdSlice& sl, char* smem, const int wg) {
    int g, rest;
    if (!decode_block(a.map, sl.kv_rest, wg, g, rest)) return;
    const int sp = rest / sl.n_units;
    int r = rest % sl.n_units;
    const int n_tiles = (sl.t1 - sl.t0 + 127) / 128;
    int chunk = 0;
    for (;; ++chunk) {
        const int tiles = min(n_tiles, (chunk + 1) * sl.chunk_blocks / 4);   // 128-key tiles = 4 blocks
        if (r < tiles) break;
        r -= tiles;
    }
    dkv_p8_tile<T, D>(a, sl, smem, g, sp, r, chunk);
}

// ------------------------------------------------------------------------------------------------
// One launch for both streaming passes: the dK/dV units first (they are the longer ones), then the dQ
// tiles in order of falling length.  Neither needs anything from the other, so what one pass leaves of
// the device while its last units finish is filled by the other -- and, unless the preprocess launch has made them
// (diag_blocks_apart), by the units of the later blocks' dK, dV, which are short and come last (spread over the
// launch, or between its two parts, they keep the dK/dV units of an XCD from streaming the same rows together: one
// step, 32/8 heads, 512 and 2048 tokens 66 and 227 us at the end, 83 and 232 elsewhere).
// ------------------------------------------------------------------------------------------------
template <typename T, int D, int N, int KS>
__global__ __launch_bounds__(512) void ttt_bwd_main_kernel(const BwdArgs<N> a) {
    extern __shared__ __align__(16) char smem[];
    const int wg = blockIdx.x;
    if (wg >= a.grid_stream) {
        const BwdSlice& sl = slice_of(a, &BwdSlice::diag_first, wg);
        diag_unit<T, D, 512, false>(a, sl, wg - sl.diag_first);
        return;
    }
    const BwdSlice& sl = slice_of(a, &BwdSlice::kv_first, wg);
    if (wg < sl.q_first) dkv_p8_unit<T, D>(a, sl, smem, wg - sl.kv_first);
    else dq_pipe_tile<T, D, 8, KS>(a, sl, smem, wg - sl.q_first);
}

template <typename T, int D, int N>
__global__ __launch_bounds__(256) void ttt_bwd_main_f32_kernel(const BwdArgs<N> a) {
    extern __shared__ __align__(16) char smem[];
    const int wg = blockIdx.x;
    if (wg >= a.grid_stream) {
        const BwdSlice& sl = slice_of(a, &BwdSlice::diag_first, wg);
        diag_unit<T, D, 256, false>(a, sl, wg - sl.diag_first);
        return;
    }
    const BwdSlice& sl = slice_of(a, &BwdSlice::kv_first, wg);
    if (wg < sl.q_first) dkv_tile<T, D, 4>(a, sl, smem, wg - sl.kv_first);
    else dq_tile<T, D, 1, 4>(a, sl, smem, wg - sl.q_first);
}

// ------------------------------------------------------------------------------------------------
// fp32: operands straight from memory
// ------------------------------------------------------------------------------------------------
// As in the forward, fp32 matrix instructions are slow enough for operands that come from memory, and without tiles to share
// a workgroup's four waves need no barrier until their sums meet in LDS.  A dQ tile is 32 rows of one (step, head)
// whose key blocks (and diagonal keys) the waves take in turn; a dK/dV unit 32 keys of a kv head whose (step, head, query
// block) items are dealt to the waves of all its splits.  A wave has a part of LDS to itself, into which the next block's rows are
// copied once the operands of this one are in registers: they arrive under its last matrix instructions, half of all (read as
// fragments from global memory instead, an item of head_dim 128 took 12.4 us, so 8.5, 7.0 of them matrix instructions).  Whole backward, tiles
// shared in LDS -> so: 247 tokens, 8/1 heads of 128, one step 67 -> 38 us; 444 tokens, 8/2 of 128, the last of seven 129 -> 63; 128
// tokens, 4/4 heads of 64, three steps 24.2 -> 18.7.  Errors against 64 bits are smaller too (dQ 4.6e-7, 4.8e-7 before; dK, dV as before or less).
// With head_dim 128 the rows, sums and operands of a unit are more than 512 registers hold: 32 are spilled (124 bytes of scratch per lane; tiles
// shared in LDS spill 43), with 64 none.
template <int D> struct BwdF32 {
    static constexpr int kRows = 32, kWaves = 4;
    static constexpr int kVec = 3 * 32 * 4;                                   // LSE*log2e, D, first token of the document of 32 rows
    static constexpr int kPieces = 2 * (D / 8);                               // 16-byte pieces of a lane's dK and dV
    static constexpr int kLds = kWaves * (kPieces * 1024 + kVec);
};

template <int D>
TTT_DEV void dq_f32_tile(const BwdCommon& a, const BwdSlice& sl, char* smem, const int wg) {
    constexpr int NW = BwdF32<D>::kWaves;
    constexpr int DC = D / 16, DB = D / 32;
    const Geometry& geo = a.geo;
    int g, rest;
    if (!decode_block(a.map, sl.q_rest, wg, g, rest)) return;
    const int h = g * geo.G + rest % geo.G;
    rest /= geo.G;
    const int js = rest % sl.n_steps, j = geo.step_begin + js;
    const int t0 = sl.t0, Tn = sl.t1;
    const int tile = (Tn - t0 + 31) / 32 - 1 - rest / sl.n_steps;   // long-prefix tiles first
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n = lane & 31, hh = lane >> 5;
    const int q0 = t0 + tile * 32, hi = min(q0 + 31, Tn - 1);
    const int qi = q0 + n, qc = min(qi, Tn - 1);
    const int lo = uniform_load(a.tok_start + q0), st_hi = uniform_load(a.tok_start + hi);

    const int64_t qoff = (int64_t)h * geo.q_sh + (int64_t)qc * geo.q_st + hh * 8;
    const float *qrow = static_cast<const float*>(a.q[j]) + qoff, *grow = static_cast<const float*>(a.d_o[j]) + qoff;
    f32x8 qf[DC], gof[DC];
#pragma unroll
    for (int t = 0; t < DC; ++t) {
        qf[t] = gload_frag<float>(qrow + t * 16);
        gof[t] = gload_frag<float>(grow + t * 16);
    }
    const int st = a.tok_start[qc];
    const float lse2 = a.lse[j][(int64_t)h * geo.T + qc] * kLog2e;
    const float dl = a.delta[((int64_t)js * geo.hq + h) * geo.T + qc];
    const float c = geo.scale_log2;
    f32x16 dqacc[DB];
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int i = 0; i < 16; ++i) dqacc[db][i] = 0.f;

    const float* K0 = static_cast<const float*>(a.k[0]) + (int64_t)g * geo.kv_sh;
    const float* V0 = static_cast<const float*>(a.v[0]) + (int64_t)g * geo.kv_sh;
    char* const tk = smem + wave * (BwdF32<D>::kPieces * 1024);
    char* const tv = tk + 32 * D * 4;
    const uint32_t lds = lds_addr(smem) + wave * (BwdF32<D>::kPieces * 1024);
    auto request = [&](int kv0) {   // K and V rows of a block
        const int last = min(31, Tn - 1 - kv0);
        wave_rows_async<D>(lds, K0 + (int64_t)kv0 * geo.kv_st, geo.kv_st, last, lane);
        wave_rows_async<D>(lds + 32 * D * 4, V0 + (int64_t)kv0 * geo.kv_st, geo.kv_st, last, lane);
    };
    const int kv_first = t0 + ((lo - t0) / 32 + wave) * 32;
    if (kv_first <= hi) request(kv_first);
    for (int kv0 = kv_first; kv0 <= hi; kv0 += NW * 32) {
        wait_async_copies();
        // S^T = K Q^T and dP^T = V dO^T
        f32x16 s, dp;
#pragma unroll
        for (int i = 0; i < 16; ++i) s[i] = dp[i] = 0.f;
#pragma unroll
        for (int t = 0; t < DC; ++t) {
            s = mma(frag_rowwise<float, D>(tk, n, t * 16 + hh * 8), qf[t], s);
            dp = mma(frag_rowwise<float, D>(tv, n, t * 16 + hh * 8), gof[t], dp);
        }
        f32x8 kt[2][DB];
#pragma unroll
        for (int x = 0; x < 2; ++x)
#pragma unroll
            for (int db = 0; db < DB; ++db) kt[x][db] = frag_transposed<float, D>(tk, x * 16, db * 32, lane);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // the block is read out: the next one arrives under what follows
        if (kv0 + NW * 32 <= hi) request(kv0 + NW * 32);
        const bool need_mask = kv0 + 31 > q0 || kv0 < st_hi;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            float p = fast_exp2(fmaf(s[i], c, -lse2));
            if (need_mask) {
                const int kv = kv0 + acc_row(i, hh);
                p = kv <= qi && kv >= st ? p : 0.f;
            }
            dp[i] = p * (dp[i] - dl);   // dS^T
        }
        // dQ^T[d, q] += K^T dS^T
#pragma unroll
        for (int x = 0; x < 2; ++x) {
            const f32x8 sf = acc_chunk<float>(dp, x);
#pragma unroll
            for (int db = 0; db < DB; ++db) dqacc[db] = mma(kt[x][db], sf, dqacc[db]);
        }
    }
    for (int lb = 1 + wave; lb <= j; lb += NW) {
        const int64_t at = (int64_t)g * geo.kv_sh + (int64_t)qc * geo.kv_st;
        const float *krow = static_cast<const float*>(a.k[lb]) + at, *vrow = static_cast<const float*>(a.v[lb]) + at;
        float s = 0.f, dp = 0.f;
#pragma unroll
        for (int t = 0; t < DC; ++t) {
            s = dot8(qf[t], gload_frag<float>(krow + t * 16 + hh * 8), s);
            dp = dot8(gof[t], gload_frag<float>(vrow + t * 16 + hh * 8), dp);
        }
        s = half_sum(s);
        dp = half_sum(dp);
        const float p = fast_exp2(fmaf(s, c, -lse2));
        const float ds = p * (dp - dl);
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int i4 = 0; i4 < 4; ++i4) {
                const f32x4 kk = gload_vec4<float>(krow + db * 32 + i4 * 8 + hh * 4);
#pragma unroll
                for (int x = 0; x < 4; ++x) dqacc[db][i4 * 4 + x] = fmaf(ds, kk[x], dqacc[db][i4 * 4 + x]);
            }
    }

    // the waves meet: piece p of a lane's row is added up by wave p % 4
    f32x4* const mine = reinterpret_cast<f32x4*>(tk) + lane;   // each in its own part of LDS: the others may still read theirs
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int i4 = 0; i4 < 4; ++i4)
            mine[(db * 4 + i4) * 64] = f32x4{dqacc[db][4 * i4], dqacc[db][4 * i4 + 1], dqacc[db][4 * i4 + 2], dqacc[db][4 * i4 + 3]};
    __syncthreads();
    if (qi >= Tn) return;
    const f32x4* const all = reinterpret_cast<const f32x4*>(smem) + lane;
    float* row = static_cast<float*>(a.dq[j]) + (int64_t)h * geo.q_sh + (int64_t)qi * geo.q_st + hh * 4;
    for (int p = wave; p < DB * 4; p += NW) {
        f32x4 sum = all[p * 64];
#pragma unroll
        for (int w = 1; w < NW; ++w) sum += all[(w * BwdF32<D>::kPieces + p) * 64];
        *reinterpret_cast<f32x4*>(row + p * 8) = sum * geo.scale;
    }
}

template <int D>
TTT_DEV void dkv_f32_unit(const BwdCommon& a, const BwdSlice& sl, char* smem, const int wg) {
    using C = BwdF32<D>;
    constexpr int NW = C::kWaves;
    constexpr int DC = D / 16, DB = D / 32;
    const Geometry& geo = a.geo;
    int g, rest;
    if (!decode_block(a.map, sl.kv_rest, wg, g, rest)) return;
    const int sp = rest % sl.n_split, tile = rest / sl.n_split;   // low tiles of a document have the longest query range: first
    const int t0 = sl.t0, Tn = sl.t1;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n = lane & 31, hh = lane >> 5;
    const int wk0 = t0 + tile * 32, kvi = wk0 + n;
    const int nqb = (uniform_load(a.tok_end + min(wk0 + 31, Tn - 1)) - 1 - t0) / 32 - tile + 1;   // query blocks that see a key
    const int n_items = sl.n_steps * geo.G * nqb;

    const int64_t kvoff = (int64_t)g * geo.kv_sh + (int64_t)min(kvi, Tn - 1) * geo.kv_st + hh * 8;
    f32x8 kf[DC], vf[DC];
#pragma unroll
    for (int t = 0; t < DC; ++t) {
        kf[t] = gload_frag<float>(static_cast<const float*>(a.k[0]) + kvoff + t * 16);
        vf[t] = gload_frag<float>(static_cast<const float*>(a.v[0]) + kvoff + t * 16);
    }
    f32x16 dkacc[DB], dvacc[DB];
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int i = 0; i < 16; ++i) dkacc[db][i] = dvacc[db][i] = 0.f;
    const float c = geo.scale_log2;
    float* const vec = reinterpret_cast<float*>(smem + NW * C::kPieces * 1024 + wave * C::kVec);

    char* const tq = smem + wave * (C::kPieces * 1024);
    char* const tg = tq + 32 * D * 4;
    const uint32_t lds = lds_addr(smem) + wave * (C::kPieces * 1024);
    float lse2_n = 0.f, dl_n = 0.f;   // of the item requested last, one row per lane
    int st_n = 0;
    auto request = [&](int it) {      // Q and dO rows of an item
        const int jh = it / nqb, qb = tile + it % nqb;
        const int js = jh / geo.G, j = geo.step_begin + js, h = g * geo.G + jh % geo.G;
        const int q0 = t0 + qb * 32, last = min(31, Tn - 1 - q0), qq = q0 + min(n, last);
        const int64_t first = (int64_t)h * geo.q_sh + (int64_t)q0 * geo.q_st;
        const float l = a.lse[j][(int64_t)h * geo.T + qq];
        dl_n = a.delta[((int64_t)js * geo.hq + h) * geo.T + qq];
        st_n = a.tok_start[qq];
        wave_rows_async<D>(lds, static_cast<const float*>(a.q[j]) + first, geo.q_st, last, lane);
        wave_rows_async<D>(lds + 32 * D * 4, static_cast<const float*>(a.d_o[j]) + first, geo.q_st, last, lane);
        lse2_n = n <= last ? l * kLog2e : INFINITY;   // rows past the end: p = 0
    };
    const int stride = sl.n_split * NW;
    int it = sp * NW + wave;
    if (it < n_items) request(it);
    for (; it < n_items; it += stride) {
        const int q0 = t0 + (tile + it % nqb) * 32;
        wait_async_copies();
        __builtin_amdgcn_wave_barrier();
        vec[n] = lse2_n;   // to be read by accumulator row
        vec[32 + n] = dl_n;
        vec[64 + n] = __int_as_float(st_n);
        __builtin_amdgcn_wave_barrier();
        // S[q, kv] = Q K^T and dP[q, kv] = dO V^T: lane = key
        f32x16 s, dp;
#pragma unroll
        for (int i = 0; i < 16; ++i) s[i] = dp[i] = 0.f;
#pragma unroll
        for (int t = 0; t < DC; ++t) {
            s = mma(frag_rowwise<float, D>(tq, n, t * 16 + hh * 8), kf[t], s);
            dp = mma(frag_rowwise<float, D>(tg, n, t * 16 + hh * 8), vf[t], dp);
        }
        f32x8 gt[2][DB], qt[2][DB];
#pragma unroll
        for (int x = 0; x < 2; ++x)
#pragma unroll
            for (int db = 0; db < DB; ++db) {
                gt[x][db] = frag_transposed<float, D>(tg, x * 16, db * 32, lane);
                qt[x][db] = frag_transposed<float, D>(tq, x * 16, db * 32, lane);
            }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // the item is read out: the next one arrives under what follows
        if (it + stride < n_items) request(it + stride);
#pragma unroll
        for (int i4 = 0; i4 < 4; ++i4) {
            const int r = 8 * i4 + 4 * hh;
            const f32x4 l4 = *reinterpret_cast<const f32x4*>(vec + r), d4 = *reinterpret_cast<const f32x4*>(vec + 32 + r);
            const f32x4 s4 = *reinterpret_cast<const f32x4*>(vec + 64 + r);
#pragma unroll
            for (int x = 0; x < 4; ++x) {
                const int i = i4 * 4 + x;
                const float p = fast_exp2(fmaf(s[i], c, -l4[x]));
                s[i] = kvi <= q0 + r + x && kvi >= __float_as_int(s4[x]) ? p : 0.f;   // P
                dp[i] = s[i] * (dp[i] - d4[x]);                                       // dS
            }
        }
        // dV[kv, d] += P^T dO;  dK[kv, d] += dS^T Q
#pragma unroll
        for (int x = 0; x < 2; ++x) {
            const f32x8 pf = acc_chunk<float>(s, x), sf = acc_chunk<float>(dp, x);
#pragma unroll
            for (int db = 0; db < DB; ++db) {
                dvacc[db] = mma(pf, gt[x][db], dvacc[db]);
                dkacc[db] = mma(sf, qt[x][db], dkacc[db]);
            }
        }
    }

    // the waves meet: piece p of a lane's sums (dK's first) is added up by wave p % 4 and joins the block-0 sums
    f32x4* const mine = reinterpret_cast<f32x4*>(tq) + lane;
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int i4 = 0; i4 < 4; ++i4) {
            mine[(db * 4 + i4) * 64] = f32x4{dkacc[db][4 * i4], dkacc[db][4 * i4 + 1], dkacc[db][4 * i4 + 2], dkacc[db][4 * i4 + 3]};
            mine[(DB * 4 + db * 4 + i4) * 64] = f32x4{dvacc[db][4 * i4], dvacc[db][4 * i4 + 1], dvacc[db][4 * i4 + 2], dvacc[db][4 * i4 + 3]};
        }
    __syncthreads();
    const f32x4* const all = reinterpret_cast<const f32x4*>(smem) + lane;
    for (int p = wave; p < C::kPieces; p += NW) {
        f32x4 sum = all[p * 64];
#pragma unroll
        for (int w = 1; w < NW; ++w) sum += all[(w * C::kPieces + p) * 64];
        float* const acc = p < DB * 4 ? a.dk0_acc : a.dv0_acc;
        const int db = p % (DB * 4) / 4, row0 = wk0 + 8 * (p % 4) + 4 * hh;
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (row0 + e < Tn) atomicAdd(acc + ((int64_t)(row0 + e) * geo.hkv + g) * D + db * 32 + n, sum[e]);
    }
}

template <int D, int N>
__global__ __launch_bounds__(256) void ttt_bwd_f32_kernel(const BwdArgs<N> a) {
    extern __shared__ __align__(16) char smem[];
    const int wg = blockIdx.x;
    if (wg >= a.grid_stream) {
        const BwdSlice& sl = slice_of(a, &BwdSlice::diag_first, wg);
        diag_unit<float, D, 256, false>(a, sl, wg - sl.diag_first);
        return;
    }
    const BwdSlice& sl = slice_of(a, &BwdSlice::kv_first, wg);
    if (wg < sl.q_first) dkv_f32_unit<D>(a, sl, smem, wg - sl.kv_first);
    else dq_f32_tile<D>(a, sl, smem, wg - sl.q_first);
}

// ------------------------------------------------------------------------------------------------
// small helper: the block-0 sums in the output dtype
// ------------------------------------------------------------------------------------------------
template <typename T, int D, int N>
__global__ void ttt_bwd_finish_kernel(const BwdArgs<N> a) {
    const Geometry& geo = a.geo;
    const BwdSlice& sl = slice_of(a, &BwdSlice::finish_first, blockIdx.x);
    const int64_t row4 = (int64_t)geo.hkv * (D / 4), end4 = sl.t1 * row4;
    const int64_t stride = (int64_t)sl.finish_blocks * blockDim.x;
    for (int64_t x = sl.t0 * row4 + (int64_t)((int)blockIdx.x - sl.finish_first) * blockDim.x + threadIdx.x; x < end4; x += stride) {
        const int d4 = (int)(x % (D / 4));
        const int64_t tg = x / (D / 4);
        const int g = (int)(tg % geo.hkv);
        const int64_t t = tg / geo.hkv;
        const f32x4 k4 = reinterpret_cast<const f32x4*>(a.dk0_acc)[x];
        const f32x4 v4 = reinterpret_cast<const f32x4*>(a.dv0_acc)[x];
        const int64_t off = t * geo.kv_st + (int64_t)g * geo.kv_sh + d4 * 4;
        gstore_vec4<T>(static_cast<T*>(a.dk[0]) + off, k4[0] * geo.scale, k4[1] * geo.scale, k4[2] * geo.scale,
                       k4[3] * geo.scale);
        gstore_vec4<T>(static_cast<T*>(a.dv[0]) + off, v4[0], v4[1], v4[2], v4[3]);
    }
}

// ------------------------------------------------------------------------------------------------
// launch sequence
// ------------------------------------------------------------------------------------------------
template <typename T, int D, int N>
static hipError_t launch_bwd_n(const BwdCommon& common, const Slice* slices, int n_slices, hipStream_t stream) {
    constexpr bool k16 = sizeof(T) == 2;      // streaming launch: eight waves; fp32: four
    constexpr int kMaxGrid = 0x7fffffff;
    BwdArgs<N> a;
    static_cast<BwdCommon&>(a) = common;
    const Geometry& geo = a.geo;
    hipError_t e;
    int n_cu = 0;
    if ((e = current_device_cu_count(n_cu)) != hipSuccess) return e;
    a.map = head_map(geo.hkv);
    CallShape shapes[kMaxSlices];
    for (int i = 0; i < n_slices; ++i) {
        shapes[i] = slices[i].shape;
        BwdSlice& sl = a.slices[i];
        sl.t0 = slices[i].t0;
        sl.t1 = sl.t0 + shapes[i].T;
        sl.n_steps = shapes[i].n_steps;
        sl.diag_units = 0;
        sl.diag_passes = 1;
    }
    a.n_slices = n_slices;

    // 1. D and, here or beside the streaming passes, the diagonal blocks; the tokens' document bounds; and cleared block-0
    // sums unless a carry from later steps is being continued
    const bool apart = k16 && diag_blocks_apart(shapes, n_slices, D, n_cu);
    {
        constexpr int UPB = 256 / (D / 8);
        int64_t grid = 0;
        for (int i = 0; i < n_slices; ++i) {
            BwdSlice& sl = a.slices[i];
            const int64_t tokens = shapes[i].T;
            sl.pre_first = (int)grid;
            sl.diag_passes = diag_passes(shapes[i], k16 ? kDiagRegBlocks : kDiagRegBlocksF32);
            int64_t blocks = (tokens + kDeltaTokens - 1) / kDeltaTokens * sl.n_steps * ((geo.hq + kDeltaHeads - 1) / kDeltaHeads);
            if (apart) {
                blocks = (tokens * geo.hkv + UPB - 1) / UPB * sl.diag_passes;
                if (blocks <= kMaxGrid) sl.diag_units = (int)blocks;
            }
            if ((grid += blocks) > kMaxGrid) return hipErrorInvalidValue;
        }
        a.pre_blocks = (int)grid;
        grid += a.bounds_blocks + std::min<int64_t>((a.clear_n4 + 1023) / 1024, 2048);
        if (grid > kMaxGrid) return hipErrorInvalidValue;
        ProfileScope prof(apart ? "ttt_bwd_pre_regs_kernel" : "ttt_bwd_delta_kernel", stream);
        auto kern = ttt_bwd_delta_kernel<T, D, N>;
        if constexpr (k16)
            if (apart) kern = ttt_bwd_pre_regs_kernel<T, D, N>;
        hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(256), 0, stream, a);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }

    // 2. dQ and block 0's dK, dV in one launch
    {
        const bool direct = !k16 && bwd_f32_direct(shapes, n_slices, D, geo.q_st, geo.kv_st);   // fp32: operands straight from memory, or tiles in LDS
        constexpr int NW = k16 ? 8 : 4;
        constexpr int KVT = 128;
        constexpr int LDS_Q = k16 ? 2 * 2 * 128 * D * (int)sizeof(T) : 4 * 64 * D * (int)sizeof(T);
        constexpr int LDS_KV = k16 ? DkvP8<T, D>::kLds : 2 * (2 * 64 * D * (int)sizeof(T) + 3 * 64 * 4);
        constexpr int LDS = LDS_Q > LDS_KV ? LDS_Q : LDS_KV;
        constexpr int LDS_DIRECT = BwdF32<D>::kLds;
        DkvPlan plans[N];
        int direct_split[N];
        if (direct) plan_dkv_f32_direct(shapes, n_slices, D, n_cu, direct_split);
        int dq_key_groups = 1;
        if constexpr (k16) dq_key_groups = plan_dkv_launch(shapes, n_slices, D, n_cu, plans);
        void (*kern)(BwdArgs<N>);
        if constexpr (!k16) kern = direct ? ttt_bwd_f32_kernel<D, N> : ttt_bwd_main_f32_kernel<T, D, N>;
        else if constexpr (N == 1) kern = dq_key_groups == 2 ? ttt_bwd_main_kernel<T, D, N, 2> : ttt_bwd_main_kernel<T, D, N, 1>;
        else kern = ttt_bwd_main_kernel<T, D, N, 1>;   // (several slices: one key group)
        const int lds_bytes = direct ? LDS_DIRECT : LDS;
        static LdsOptIn lds_opt_in[2];   // one per kernel
        if ((e = lds_opt_in[dq_key_groups == 2 || direct ? 1 : 0].ensure((const void*)kern, lds_bytes)) != hipSuccess) return e;
        // the 16-bit passes address the pieces of up to 64 rows of K or V and 32 rows of Q or dO with
        // 32-bit byte offsets
        if (k16 && geo.kv_st * 64 * (int64_t)sizeof(T) >= (int64_t)1 << 32) return hipErrorInvalidValue;
        if (k16 && geo.q_st * 32 * (int64_t)sizeof(T) >= (int64_t)1 << 32) return hipErrorInvalidValue;
        // dK/dV: split the (step, head) list of a unit so that the grid fills the device evenly
        const int q_rows = direct ? 32 : NW * 32 / dq_key_groups, kv_rows = direct ? 32 : KVT;
        int64_t grid = 0;
        for (int i = 0; i < n_slices; ++i) {
            BwdSlice& sl = a.slices[i];
            const int n_tiles = (shapes[i].T + kv_rows - 1) / kv_rows;
            int64_t n_units = n_tiles;   // units per kv head and split: key tiles, or (key tile, query chunk) pairs
            if constexpr (k16) {
                sl.chunk_blocks = plans[i].chunk_blocks;
                sl.n_split = plans[i].n_split;
                n_units = dkv_units_of(shapes[i].T, n_tiles, sl.chunk_blocks);
            } else if (direct) {
                sl.n_split = direct_split[i];
            } else {
                sl.n_split = plan_dkv_split_f32(shapes[i]);
            }
            if (n_units * sl.n_split > kMaxGrid) return hipErrorInvalidValue;
            sl.n_units = (int)n_units;
            sl.kv_rest = (int)(n_units * sl.n_split);
            sl.kv_first = (int)grid;
            if ((grid += head_map_grid(a.map, sl.kv_rest)) > kMaxGrid) return hipErrorInvalidValue;
            const int64_t rest = (int64_t)((shapes[i].T + q_rows - 1) / q_rows) * sl.n_steps * geo.G;
            sl.q_first = (int)grid;
            if ((grid += head_map_grid(a.map, rest)) > kMaxGrid) return hipErrorInvalidValue;
            sl.q_rest = (int)rest;
        }
        a.grid_stream = (int)grid;
        if (!apart) {
            constexpr int UPB = NW * 64 / (D / 8);
            for (int i = 0; i < n_slices; ++i) {
                BwdSlice& sl = a.slices[i];
                const int64_t units = geo.step_begin + sl.n_steps > 1 ? ((int64_t)shapes[i].T * geo.hkv + UPB - 1) / UPB * sl.diag_passes : 0;
                sl.diag_first = (int)grid;
                if ((grid += units) > kMaxGrid) return hipErrorInvalidValue;
                sl.diag_units = (int)units;
            }
        }
        {
            ProfileScope prof(k16 ? "ttt_bwd_main_kernel" : direct ? "ttt_bwd_f32_kernel" : "ttt_bwd_main_f32_kernel", stream);
            hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(NW * 64), lds_bytes, stream, a);
        }
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }

    // 3. block-0 sums -> output dtype, once the sweep has covered step 0
    if (!a.accumulate || geo.step_begin == 0) {
        int blocks = 0;
        for (int i = 0; i < n_slices; ++i) {
            BwdSlice& sl = a.slices[i];
            sl.finish_first = blocks;
            sl.finish_blocks = (int)std::min<int64_t>(((int64_t)shapes[i].T * geo.hkv * (D / 4) + 255) / 256, 4096);
            blocks += sl.finish_blocks;
        }
        {
            ProfileScope prof("ttt_bwd_finish_kernel", stream);
            hipLaunchKernelGGL((ttt_bwd_finish_kernel<T, D, N>), dim3(blocks), dim3(256), 0, stream, a);
        }
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    return hipSuccess;
}

// the slices (those with the longest work first) in launches of one or of many
template <typename T, int D> static hipError_t launch_bwd_slices(BwdCommon a, const Slice* slices, int n_slices, hipStream_t stream) {
    int n_cu = 0;
    if (hipError_t e = current_device_cu_count(n_cu); e != hipSuccess) return e;
    for (int i = 0, n; i < n_slices; i += n) {
        n = 1;
        if (sizeof(T) == 4 || !bwd_slice_alone(slices[i].shape, D, n_cu))
            while (n < kMaxSlices && i + n < n_slices && (sizeof(T) == 4 || !bwd_slice_alone(slices[i + n].shape, D, n_cu))) ++n;
        const hipError_t e = n > 1 ? launch_bwd_n<T, D, kMaxSlices>(a, slices + i, n, stream) : launch_bwd_n<T, D, 1>(a, slices + i, n, stream);
        if (e != hipSuccess) return e;
        a.bounds_blocks = 0;   // the first launch wrote and cleared them for the whole batch
        a.clear_n4 = 0;
    }
    return hipSuccess;
}

hipError_t launch_bwd(int dtype, int head_dim, const BwdCommon& a, const Slice* slices, int n_slices, hipStream_t stream) {
    if (dtype == 1 && head_dim == 128) return launch_bwd_slices<__bf16, 128>(a, slices, n_slices, stream);
    if (dtype == 1 && head_dim == 64) return launch_bwd_slices<__bf16, 64>(a, slices, n_slices, stream);
    if (dtype == 0 && head_dim == 128) return launch_bwd_slices<float, 128>(a, slices, n_slices, stream);
    if (dtype == 0 && head_dim == 64) return launch_bwd_slices<float, 64>(a, slices, n_slices, stream);
    return hipErrorInvalidValue;
}

}  // namespace ttt
