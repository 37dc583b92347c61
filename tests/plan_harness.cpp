// The launch rules of the library (csrc/ttt_plan.hpp) behind C functions, built by a plain C++ compiler: which kernel
// variant and work split a call takes on a device of n_cu compute units.
#include "../paper_2603_18567_amd/csrc/ttt_plan.hpp"

extern "C" {

void plan_forward(int T, int step_begin, int n_steps, int G, int hkv, int n_docs, const int32_t* cu, int is_bf16, int head_dim,
                  int n_cu, int* split, int* pack_log2) {
    const ttt::FwdPlan p = ttt::plan_fwd(ttt::CallShape{T, step_begin, n_steps, G, hkv, n_docs, cu, cu[0]}, is_bf16 != 0, head_dim, n_cu);
    *split = p.split;
    *pack_log2 = p.pack_log2;
}

void plan_backward(int T, int step_begin, int n_steps, int G, int hkv, int n_docs, const int32_t* cu, int head_dim, int n_cu,
                   int* chunk_blocks, int* n_split) {
    const ttt::DkvPlan p = ttt::plan_dkv_split(ttt::CallShape{T, step_begin, n_steps, G, hkv, n_docs, cu, cu[0]}, head_dim, n_cu);
    *chunk_blocks = p.chunk_blocks;
    *n_split = p.n_split;
}

// the work splits of runs of documents [first, first + n_docs) that take n_steps steps, 16 to a launch
void plan_backward_runs(int n_runs, const int* first, const int* n_docs, const int* n_steps, const int32_t* cu, int G, int hkv,
                        int head_dim, int n_cu, int* chunk_blocks, int* n_split) {
    for (int i = 0; i < n_runs; i += 16) {
        ttt::CallShape calls[16];
        ttt::DkvPlan plans[16];
        const int n = n_runs - i < 16 ? n_runs - i : 16;
        for (int x = 0; x < n; ++x) {
            const int32_t* c = cu + first[i + x];
            calls[x] = ttt::CallShape{c[n_docs[i + x]] - c[0], 0, n_steps[i + x], G, hkv, n_docs[i + x], c, c[0]};
        }
        ttt::plan_dkv_launch(calls, n, head_dim, n_cu, plans);
        for (int x = 0; x < n; ++x) {
            chunk_blocks[i + x] = plans[x].chunk_blocks;
            n_split[i + x] = plans[x].n_split;
        }
    }
}

// the work split and the key groups of the dQ tiles of a launch of one run of documents
void plan_backward_launch(int T, int step_begin, int n_steps, int G, int hkv, int n_docs, const int32_t* cu, int head_dim, int n_cu,
                          int* chunk_blocks, int* n_split, int* dq_groups) {
    const ttt::CallShape call{T, step_begin, n_steps, G, hkv, n_docs, cu, cu[0]};
    ttt::DkvPlan p;
    *dq_groups = ttt::plan_dkv_launch(&call, 1, head_dim, n_cu, &p);
    *chunk_blocks = p.chunk_blocks;
    *n_split = p.n_split;
}

int plan_later_blocks(int T, int step_begin, int n_steps, int G, int hkv, int head_dim, int n_cu) {
    return ttt::diag_blocks_apart(ttt::CallShape{T, step_begin, n_steps, G, hkv, 0, nullptr, 0}, head_dim, n_cu);
}

// whether the fp32 passes take their operands straight from memory (q_st, kv_st: elements from row to row)
void plan_f32_direct(int T, int step_begin, int n_steps, int G, int hkv, int n_docs, const int32_t* cu, int head_dim, int n_cu, int64_t q_st,
                     int64_t kv_st, int* fwd, int* bwd) {
    const ttt::CallShape call{T, step_begin, n_steps, G, hkv, n_docs, cu, cu[0]};
    *fwd = ttt::fwd_f32_direct(&call, 1, head_dim, n_cu, ttt::plan_fwd(call, false, head_dim, n_cu), kv_st);
    *bwd = ttt::bwd_f32_direct(&call, 1, head_dim, q_st, kv_st);
}

// tile sizes and workgroups per compute unit of the launches of a projection; returns how many there are
int plan_projection(int64_t tokens, int hidden_in, int features, int largest_fits, int n_cu, int* mt_nt_per_cu, int* f_first) {
    const ttt::QkvPlan p = ttt::plan_qkv(tokens, hidden_in, features, largest_fits != 0, n_cu);
    int n = 0;
    for (int kind : {p.first, p.second}) {
        if (kind < 0) continue;
        const ttt::QkvTile& t = ttt::kQkvTiles[kind];
        mt_nt_per_cu[3 * n] = t.mt;
        mt_nt_per_cu[3 * n + 1] = t.nt;
        mt_nt_per_cu[3 * n + 2] = t.per_cu;
        ++n;
    }
    *f_first = p.f_first;
    return n;
}

// token tiles of one feature tile that a launch of tiles of `kind` deals to an XCD together
int plan_projection_group(int64_t tokens, int kind, int features, int n_cu) {
    const ttt::QkvTile& t = ttt::kQkvTiles[kind];
    return ttt::qkv_group(t, (tokens + t.mt - 1) / t.mt, (features + t.nt - 1) / t.nt, n_cu);
}

}
