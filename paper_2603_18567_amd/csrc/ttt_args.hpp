// Kernel argument blocks (host fills, device reads) and the launcher prototypes that connect the
// C-ABI file to the kernel files.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <atomic>

#include "ttt_device.hpp"
#include "ttt_plan.hpp"

namespace ttt {

constexpr int kMaxSteps = 32;

struct Geometry {
    int T;               // packed tokens of the whole batch
    int k;               // cache blocks
    int step_begin;
    int hq, hkv, G;
    float scale;         // softmax_scale
    float scale_log2;    // softmax_scale * log2(e)
    int64_t q_st, q_sh;  // strides (elements) of Q/O/dO/dQ
    int64_t kv_st, kv_sh;
};

// A launch covers up to kMaxSlices slices of the batch: tokens [t0, t1) = whole documents that take n_steps steps from
// geo.step_begin on.  Tiles count from t0, tokens from the batch's first; each part of a launch lists where the
// workgroups of a slice start (a multiple of 8 where workgroups are dealt to the XCDs by kv head).
constexpr int kMaxSlices = 16;

struct FwdSlice {
    int first;              // first workgroup
    int t0, t1, n_steps;
    int doc0, n_docs;
    int n_tiles;            // query tiles
    int rest_count;         // work items per kv head
};

struct FwdCommon {   // what every workgroup reads first stands together
    Geometry geo;
    const int* tok_start;   // [T] first token of each token's document, or null: at most 64 documents a slice, found in `cu`
    const int* cu;          // device cu_seqlens
    int pack_log2;          // log2 of the query heads (of one kv group) that share a workgroup
    int diag_rows;          // rows of a workgroup's diagonal keys that go through LDS, 0: straight from global memory
    int diag_slots;         // blocks that have LDS for these rows behind the tile stages
    HeadMap map;
    int n_slices;
    const void* q[kMaxSteps];
    const void* k[kMaxSteps];
    const void* v[kMaxSteps];
    void* o[kMaxSteps];
    float* lse[kMaxSteps];
};
template <int N> struct FwdArgs : FwdCommon {
    FwdSlice slices[N];
};

struct BwdSlice {
    int t0, t1, n_steps;
    int pre_first;          // first workgroup of its D (and diagonal blocks) in the preprocess launch
    int kv_first;           // of its dK/dV units in the streaming launch,
    int q_first;            // of its dQ tiles, which follow them,
    int diag_first;         // and of its later blocks, which follow the tiles of all slices
    int finish_first, finish_blocks;   // of its block-0 results in the last launch
    int kv_rest, q_rest;    // work items per kv head
    int n_split;            // dK/dV: ways the (step, head) list of one kv tile is split
    int n_units;            // dK/dV (16-bit): (key tile, query chunk) units per kv head and split
    int chunk_blocks;       // dK/dV (16-bit): 32-row query blocks per chunk (a multiple of 4)
    int diag_units;         // workgroups that make the later blocks' dK, dV,
    int diag_passes;        // in so many passes over these blocks
};

struct BwdCommon {
    Geometry geo;
    HeadMap map;
    int grid_stream;        // workgroups of the streaming launch for dK/dV units and dQ tiles; after them: the later blocks' dK, dV
    int pre_blocks;         // workgroups of the preprocess launch that do its main work; after them:
    int bounds_blocks;      // those that write tok_start, tok_end; and the rest clear the block-0 sums
    int64_t clear_n4;       // 16-byte pieces of each block-0 sum to clear
    int accumulate;         // 0/1
    int carry_reset;        // accumulate mode: this call starts the sweep (carry is overwritten, not read)
    int* tok_start;         // [T] first token of each token's document
    int* tok_end;           // [T] one past its last token
    float* delta;           // [steps][hq][T]  D = <dO, O>; 16-bit: -D
    float* lse2;            // [steps][hq][T]  LSE * log2(e), the exponent offset of the 16-bit kernels
    float* dk0_acc;         // [T][hkv][d] fp32, block-0 partial sums (atomics)
    float* dv0_acc;
    float* dkl_acc;         // [k-1][T][hkv][d] fp32 carry for blocks l>=1 (accumulate mode), else null
    float* dvl_acc;
    const int* cu;          // device cu_seqlens
    int n_docs;
    int n_slices;
    const void* q[kMaxSteps];
    const void* k[kMaxSteps];
    const void* v[kMaxSteps];
    const void* o[kMaxSteps];
    const float* lse[kMaxSteps];
    const void* d_o[kMaxSteps];
    void* dq[kMaxSteps];
    void* dk[kMaxSteps];
    void* dv[kMaxSteps];
};
template <int N> struct BwdArgs : BwdCommon {
    BwdSlice slices[N];
};
static_assert(sizeof(BwdArgs<kMaxSlices>) <= 4096 && sizeof(FwdArgs<kMaxSlices>) <= 4096, "kernel arguments");

// The slice whose workgroups, counted by `first`, include number wg.  Launches of one slice (N = 1) are instantiations of
// their own: the search costs a kernel 0.3 us before its first load (128 tokens, forward and backward in four launches: 45.7
// us, 46.5 with it), the longer arguments cost the host.
template <template <int> class Args, int N, typename S> TTT_DEV const S& slice_of(const Args<N>& a, int S::* first, int wg) {
    int s = 0;
    if constexpr (N > 1)
        while (s + 1 < a.n_slices && wg >= a.slices[s + 1].*first) ++s;
    return a.slices[s];
}

// host side: a slice as the launch rules see it, and its place in the batch
struct Slice {
    CallShape shape;
    int doc0, t0;
};

// launchers (defined in the kernel files); all enqueue on `stream` and return the launch status
hipError_t launch_tok_bounds(const int* cu_dev, int n_docs, int T, int* tok_start, int* tok_end, hipStream_t stream);
constexpr int kMaxInlineDocs = 64;   // documents whose bounds the forward kernel finds by itself (one per lane)
hipError_t launch_fwd(int dtype, int head_dim, const FwdCommon& a, const Slice* slices, int n_slices, hipStream_t stream);
hipError_t launch_bwd(int dtype, int head_dim, const BwdCommon& a, const Slice* slices, int n_slices, hipStream_t stream);
hipError_t launch_loss_bwd(int dtype, void* logits, const void* target, const float* grad, int64_t n_rows, int vocab,
                           int64_t logits_row_stride, int64_t target_row_stride, hipStream_t stream);

hipError_t launch_qkv_rope(const void* x, const void* w, const float* cos_tab, const float* sin_tab, const int* pos, void* q,
                           void* k, void* v, int64_t tokens, int hidden_in, int n_q, int n_k, int n_v, int64_t x_st,
                           int64_t w_st, int n_pos, hipStream_t stream);

// Per-device host-side state of the launchers.  A kernel's opt-in to more than 48 KB of dynamic LDS
// is an attribute of (kernel, device): LdsOptIn sets it the first time a kernel instantiation is
// launched on each device (one bit per device index; indices past 63 simply set it every time).
struct LdsOptIn {
    std::atomic<uint64_t> done{0};
    hipError_t ensure(const void* kernel, int bytes) {
        int dev = 0;
        hipError_t e = hipGetDevice(&dev);
        if (e != hipSuccess) return e;
        const bool tracked = dev >= 0 && dev < 64;
        if (tracked && ((done.load(std::memory_order_acquire) >> dev) & 1u)) return hipSuccess;
        e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
        if (e == hipSuccess && tracked) done.fetch_or((uint64_t)1 << dev, std::memory_order_release);
        return e;
    }
};
// compute units of the current device (cached per device index; 256 if the runtime reports none)
inline hipError_t current_device_cu_count(int& n_cu) {
    static std::atomic<int> cache[64];
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    const bool tracked = dev >= 0 && dev < 64;
    if (tracked && (n_cu = cache[dev].load(std::memory_order_relaxed)) > 0) return hipSuccess;
    if ((e = hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev)) != hipSuccess) return e;
    if (n_cu <= 0) n_cu = 256;
    if (tracked) cache[dev].store(n_cu, std::memory_order_relaxed);
    return hipSuccess;
}

// Diagnostics (off by default): brackets one kernel launch with HIP events on its stream so that
// a caller can read per-kernel durations afterwards (ttt_attn_profile_totals).
void profile_begin(const char* kernel_name, hipStream_t stream);
void profile_end(hipStream_t stream);
struct ProfileScope {
    hipStream_t stream;
    ProfileScope(const char* name, hipStream_t s) : stream(s) { profile_begin(name, s); }
    ~ProfileScope() { profile_end(stream); }
};

}  // namespace ttt
