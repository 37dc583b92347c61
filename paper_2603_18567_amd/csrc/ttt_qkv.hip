// Producer of Q_j, K_j, V_j (gfx950): the draft layer's query / key / value projection with the
// rotary position embedding applied in the epilogue, written in the layout the attention kernels
// read ([token, head, head_dim]) -- the tensors that Sec. 4.2.1 takes as given.
//
//   y[t, f] = sum_c x[t, c] w[f, c]            bf16 operands, fp32 accumulation on the matrix cores
//   Q, K heads: (y[i], y[i + d/2]) turned by the angle whose cos / sin the table holds at pos[t]
//   V heads:    y as it is
// With no rotated heads at all the same kernel is the plain projection y = x w^T (the output
// projection that reads O_j).
//
// Two kernels.  ttt_qkv_rope_kernel, for many tokens: one workgroup = 256 tokens x 2 heads (256 features), four waves
// of 128 tokens x the 128 features of one head, one to a SIMD: 4 x 4 accumulator blocks of 32 x 32 fill one half
// of its 512 registers.  What bounds it is LDS traffic and, with all compute units at work, the clock under the
// board's power cap: a wave reads half an operand fragment per matrix instruction (eight waves of 64 x 128
// read three quarters) and 64-column slices of both tiles stream through two LDS stages by LDS-DMA copies.
// Measured against that eight-wave form: 4096 x 4096 x 4096 126 -> 109 us (1.26 PFLOP/s), 8192 tokens x 8192 x
// 9216 1.26 PFLOP/s, 1500 tokens x 4096 x 9216 221 -> 100 us (there mostly by dealing out the tiles evenly).
// ttt_qkv_rope_splitk_kernel, for few tokens or the features that the large tiles leave over: smaller tiles, see
// there; kQkvTiles has their times and the choice.
//
// Both compute y^T (row = feature, lane = token).  Both operands are contraction-contiguous in memory, so
// both are read from their LDS tiles as row fragments.  The token tiles of one feature tile go to one XCD
// in groups: each x and w slice that enters that XCD's L2 is used by several workgroups.
#include "ttt_args.hpp"

namespace ttt {

struct QkvArgs {
    const void* x;
    const void* w;
    const float* cos_tab;
    const float* sin_tab;
    const int* pos;
    void* q;
    void* k;
    void* v;
    int T, Hin, n_pos;
    int n_q, n_k, n_v;    // heads written to q (rotated), k (rotated), v (as they are); weight rows in this order
    int64_t x_st, w_st;   // row strides in elements
    int m_tiles, n_tiles;
    int m_per;            // token tiles of one feature tile that go to one XCD together
    int f_first, f_count; // features of this launch (a call may be carried out as two launches)
};

template <typename T>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1))) void ttt_qkv_rope_kernel(const QkvArgs a) {
    static_assert(sizeof(T) == 2, "16-bit operands");
    using E = Elem<T>;
    using frag = typename E::frag;
    constexpr int D = 128;         // head_dim
    constexpr int MB = 4;          // blocks of 32 tokens per wave
    constexpr int MT = MB * 64;    // tokens per workgroup
    constexpr int NT = 256;        // features per workgroup (two heads)
    constexpr int KT = 64;         // contraction slice per stage
    using TL = Tile<T, KT>;
    constexpr int X_BYTES = MT * KT * E::kBytes;
    constexpr int STAGE_BYTES = X_BYTES + NT * KT * E::kBytes;
    typedef __attribute__((address_space(3))) char lds_char;

    extern __shared__ __align__(16) char smem[];
    const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_char*)smem;

    // groups of up to 4 token tiles of one feature tile on one XCD, as in the kernel below
    const int slot = blockIdx.x >> 3;
    const int m_per = a.m_per, m_groups = (a.m_tiles + m_per - 1) / m_per;
    const int grp = slot / m_per * 8 + (blockIdx.x & 7);
    const int tm = grp % m_groups * m_per + slot % m_per, tn = grp / m_groups;
    if (tm >= a.m_tiles || tn >= a.n_tiles) return;
    const int m0 = tm * MT;
    const int n0 = a.f_first + tn * NT;
    const int n_feat = a.f_first + a.f_count;

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave & 1, wn = wave >> 1;
    const int n = lane & 31, hh = lane >> 5;

    // ---- copies of one slice (KT columns) of the two tiles: 8 rows per wave and instruction, 16 instructions
    const T* xs = static_cast<const T*>(a.x) + (int64_t)m0 * a.x_st;
    const T* ws = static_cast<const T*>(a.w) + (int64_t)n0 * a.w_st;
    uint32_t off_x[8], off_w[8];
#pragma unroll
    for (int it = 0; it < 8; ++it) {
        const int r = it * 32 + wave * 8 + (lane >> 3);
        const uint32_t piece = 16 * ((lane & 7) ^ TL::swz(r));
        // rows past the end repeat the last one and are not stored
        off_x[it] = (uint32_t)min(r, a.T - 1 - m0) * (uint32_t)(a.x_st * 2) + piece;
        off_w[it] = (uint32_t)min(r, n_feat - 1 - n0) * (uint32_t)(a.w_st * 2) + piece;
    }
    auto copy = [&](int ks, int s, int i) {
        const uint32_t dst = lds0 + s * STAGE_BYTES + wave * 1024;
        if (i < 8) async_copy16(xs + ks * KT, off_x[i], dst + i * 4096);
        else async_copy16(ws + ks * KT, off_w[i - 8], dst + X_BYTES + (i - 8) * 4096);
    };

    // ---- per-lane LDS addresses of the row fragments: chunk t of row n of this wave's first block, in the
    // stage that is read next (the two stages differ in one address bit)
    constexpr int BLK = 32 * TL::kRowBytes;   // one 32-row block of a tile
    static_assert(STAGE_BYTES == 65536, "stages are told apart by bit 16 of an LDS address");
    uint32_t rx[KT / 16], rw[KT / 16];
    {
        LaneFrags<T, KT> lf;
        lf.init(lane);
#pragma unroll
        for (int t = 0; t < KT / 16; ++t) {
            rx[t] = lds0 + lf.row[t] + wm * MB * BLK;
            rw[t] = lds0 + lf.row[t] + X_BYTES + wn * 4 * BLK;
        }
    }
    auto ld = [&](uint32_t addr) -> frag {
        return *reinterpret_cast<const __attribute__((address_space(3))) frag*>((uintptr_t)addr);
    };

    f32x16 acc[MB][4];
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int nb = 0; nb < 4; ++nb)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[mb][nb][i] = 0.f;

    const int n_k = a.Hin / KT;
    frag xf[2][MB], wf[2][4];   // of the chunk at work and of the next one
    auto request = [&](int buf, int t, int i) {   // fragment i of chunk t
        if (i < 4) wf[buf][i] = ld(rw[t] + i * BLK);
        else xf[buf][i - 4] = ld(rx[t] + (i - 4) * BLK);
    };
    // One slice.  Between its third and last chunk the next slice is in LDS for everyone and everyone has the
    // last fragments of this one, so its stage is requested again (the slice after the next) and the first
    // fragments of the next slice are, too: no wave waits for LDS with its matrix core idle.
    auto step = [&](int ks, auto fill_c, auto next_c) {
        constexpr bool FILL = decltype(fill_c)::value, NEXT = decltype(next_c)::value;
#pragma unroll
        for (int t = 0; t < KT / 16; ++t) {
            const bool last = t == KT / 16 - 1;
            if (last && NEXT) {
                wait_async_copies();
                lds_barrier();
#pragma unroll
                for (int u = 0; u < KT / 16; ++u) {
                    rx[u] ^= STAGE_BYTES;
                    rw[u] ^= STAGE_BYTES;
                }
            }
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                if (!last || NEXT) request((t + 1) & 1, last ? 0 : t + 1, i);
                if (last && FILL) {
                    copy(ks + 2, ks & 1, 2 * i);
                    copy(ks + 2, ks & 1, 2 * i + 1);
                }
                issue_fence();
                acc[i / 2][2 * (i & 1)] = mma(wf[t & 1][2 * (i & 1)], xf[t & 1][i / 2], acc[i / 2][2 * (i & 1)]);
                acc[i / 2][2 * (i & 1) + 1] = mma(wf[t & 1][2 * (i & 1) + 1], xf[t & 1][i / 2], acc[i / 2][2 * (i & 1) + 1]);
                issue_fence();
            }
        }
    };
    auto pin = [&]() {   // the accumulators' home is the accumulation half of the register file
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
            for (int nb = 0; nb < 4; ++nb) asm volatile("" : "+a"(acc[mb][nb]));
    };
#pragma unroll
    for (int i = 0; i < 16; ++i) copy(0, 0, i);
    if (n_k > 1) {
#pragma unroll
        for (int i = 0; i < 16; ++i) copy(1, 1, i);
        wait_copies_but(IntC<16>{});
    } else {
        wait_async_copies();
    }
    lds_barrier();
#pragma unroll
    for (int i = 0; i < 8; ++i) request(0, 0, i);
    pin();
    for (int ks = 0; ks < n_k - 2; ++ks) {
        step(ks, IntC<1>{}, IntC<1>{});
        pin();
    }
    if (n_k > 1) step(n_k - 2, IntC<0>{}, IntC<1>{});
    step(n_k - 1, IntC<0>{}, IntC<0>{});
    pin();
    lds_barrier();   // the stages are free

    // ---- epilogue, 32 tokens of a wave at a time through LDS: a lane puts the features 32 nb + 8 k4 + 4 hh + 0..3 of
    // token n there and takes 8 pairs of a token, so that eight lanes read one row of the angle table and write
    // 128 consecutive bytes (storing from the accumulators, 8 bytes in each of 32 rows per instruction, cost a
    // tile 10 us).  The table rows of the next 32 tokens are requested ahead.
    const int head = n0 / D + wn;
    if (head * D >= n_feat) return;
    const bool rotate = head < a.n_q + a.n_k;
    T* out;
    int64_t out_st;
    if (head < a.n_q) {
        out = static_cast<T*>(a.q) + (int64_t)head * D;
        out_st = (int64_t)a.n_q * D;
    } else if (head < a.n_q + a.n_k) {
        out = static_cast<T*>(a.k) + (int64_t)(head - a.n_q) * D;
        out_st = (int64_t)a.n_k * D;
    } else {
        out = static_cast<T*>(a.v) + (int64_t)(head - a.n_q - a.n_k) * D;
        out_st = (int64_t)a.n_v * D;
    }
    constexpr int PITCH = D + 4;   // floats: rows 16 bytes apart modulo the banks
    float* part = reinterpret_cast<float*>(smem) + wave * (32 * PITCH);
    const int t8 = lane >> 3, i0 = 8 * (lane & 7);
    const int m_wave = m0 + wm * (32 * MB);
    int p[MB][4];
    f32x8 c8[2][4], s8[2][4];
    auto angles = [&](int mb) {
#pragma unroll
        for (int it = 0; it < 4; ++it) {
            c8[mb & 1][it] = gload_frag<float>(a.cos_tab + (int64_t)p[mb][it] * (D / 2) + i0);
            s8[mb & 1][it] = gload_frag<float>(a.sin_tab + (int64_t)p[mb][it] * (D / 2) + i0);
        }
    };
    if (rotate) {
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
            for (int it = 0; it < 4; ++it) {
                const int v = a.pos[min(m_wave + mb * 32 + it * 8 + t8, a.T - 1)];
                p[mb][it] = v < 0 ? 0 : (v >= a.n_pos ? a.n_pos - 1 : v);
            }
        angles(0);
    }
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
        issue_fence();   // one block of rows at a time leaves the accumulators
        if (rotate && mb + 1 < MB) angles(mb + 1);
#pragma unroll
        for (int nb = 0; nb < 4; ++nb)
#pragma unroll
            for (int k4 = 0; k4 < 4; ++k4)
                *reinterpret_cast<f32x4*>(part + n * PITCH + nb * 32 + 8 * k4 + 4 * hh) =
                    f32x4{acc[mb][nb][4 * k4], acc[mb][nb][4 * k4 + 1], acc[mb][nb][4 * k4 + 2], acc[mb][nb][4 * k4 + 3]};
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int it = 0; it < 4; ++it) {
            const int m = m_wave + mb * 32 + it * 8 + t8;
            const f32x8 y0 = gload_frag<float>(part + (it * 8 + t8) * PITCH + i0);
            const f32x8 y1 = gload_frag<float>(part + (it * 8 + t8) * PITCH + D / 2 + i0);
            bf16x8 lo, hi;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                lo[e] = (__bf16)(rotate ? y0[e] * c8[mb & 1][it][e] - y1[e] * s8[mb & 1][it][e] : y0[e]);
                hi[e] = (__bf16)(rotate ? y1[e] * c8[mb & 1][it][e] + y0[e] * s8[mb & 1][it][e] : y1[e]);
            }
            if (m < a.T) {
                T* row = out + (int64_t)m * out_st + i0;
                *reinterpret_cast<bf16x8*>(row) = lo;
                *reinterpret_cast<bf16x8*>(row + D / 2) = hi;
            }
        }
        __builtin_amdgcn_wave_barrier();
    }
}

// ------------------------------------------------------------------------------------------------
// Few tokens: the weights outweigh the activations
// ------------------------------------------------------------------------------------------------
// Tiles of MT tokens x NT features, so small that even a short batch makes about one workgroup per compute unit;
// what keeps the matrix work of such a tile apart is the contraction: the eight waves are KG groups of
// MW x NW waves, wave group kg taking every KG-th 16-column chunk of the slices that stream through LDS
// (each wave has 64 x 64 accumulators or fewer, and reads one operand fragment from LDS per matrix
// instruction where a split of the tile would read two).  The groups' partial sums meet once, in LDS, at
// the end.  NST stages of SUB 64-column slices, requested NST - 1 ahead: the copies are the bound here.
// A tile of NT < 128 features holds both elements of its rotary pairs: NT / 2 features of the lower half
// of one head and the NT / 2 that they are paired with.
template <typename T, int MT, int NT, int KG, int MW, int NW, int SUB, int NST>
struct QkvSplitK {
    static constexpr int KT = 64;
    static constexpr int ROW_BYTES = KT * 2;
    static constexpr int SLICE_ROWS = MT + NT;
    static constexpr int STAGE_BYTES = SUB * SLICE_ROWS * ROW_BYTES;
    static constexpr int MB = MT / (32 * MW), NB = NT / (32 * NW);   // 32 x 32 blocks of a wave
    static constexpr int PITCH = NB * 32 + 4;                        // floats; rows 16 bytes apart modulo the banks
    static constexpr int PART_BYTES = MB * 32 * PITCH * 4;
    // Where the partial sums of all eight waves would need more LDS than the stages, the upper half of the
    // contraction groups hands its sums to the lower half first.
    static constexpr bool FOLD = 8 * PART_BYTES > NST * STAGE_BYTES;
    static constexpr int KGE = FOLD ? KG / 2 : KG;                   // partial sums that the outputs are added up from
    static constexpr int EPI_BYTES = KGE * MW * NW * PART_BYTES;
    static constexpr int LDS = NST * STAGE_BYTES > EPI_BYTES ? NST * STAGE_BYTES : EPI_BYTES;
    static_assert(KG * MW * NW == 8 && SUB * 4 % KG == 0 && SUB * SLICE_ROWS % 64 == 0 && LDS <= 160 * 1024, "work split");
};

template <typename T, int MT, int NT, int KG, int MW, int NW, int SUB, int NST>
__global__ __launch_bounds__(512) void ttt_qkv_rope_splitk_kernel(const QkvArgs a) {
    static_assert(sizeof(T) == 2, "16-bit operands");
    using C = QkvSplitK<T, MT, NT, KG, MW, NW, SUB, NST>;
    using frag = typename Elem<T>::frag;
    using TL = Tile<T, C::KT>;
    constexpr int D = 128;
    constexpr int MB = C::MB, NB = C::NB;
    constexpr int CH = SUB * 4 / KG;                      // chunks of a stage that a wave works on
    constexpr int PASSES = SUB * C::SLICE_ROWS / 64;      // copy instructions of a wave per stage, 8 rows each
    typedef __attribute__((address_space(3))) char lds_char;

    extern __shared__ __align__(16) char smem[];
    const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_char*)smem;

    // Groups of up to 8 token tiles of one feature tile are consecutive workgroups of one XCD (workgroup ids go
    // round-robin over the 8): with few tokens its weight rows enter that L2 once; with many the groups are
    // dealt out token group by token group, so that an XCD keeps to the same x rows.
    const int slot = blockIdx.x >> 3;
    const int m_per = a.m_per, m_groups = (a.m_tiles + m_per - 1) / m_per;
    const int grp = slot / m_per * 8 + (blockIdx.x & 7);
    const int tm = grp % m_groups * m_per + slot % m_per, tn = grp / m_groups;
    if (tm >= a.m_tiles || tn >= a.n_tiles) return;
    const int m0 = tm * MT;
    constexpr int TILES_PER_HEAD = D / NT;
    const int head = a.f_first / D + tn / TILES_PER_HEAD, pair0 = tn % TILES_PER_HEAD * (NT / 2);

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wn = wave % NW, wm = wave / NW % MW, kg = wave / (NW * MW);
    const int n = lane & 31, hh = lane >> 5;

    // ---- copies: 8 stage rows per wave and pass; a lane's source row stays the same from stage to stage
    const T* src[PASSES];
    int sub_of[PASSES];
#pragma unroll
    for (int p = 0; p < PASSES; ++p) {
        const int rr = p * 64 + wave * 8 + (lane >> 3);
        const int r = rr % C::SLICE_ROWS, piece = (lane & 7) ^ TL::swz(r);   // MT is a multiple of 16: swz(r) == swz(r - MT)
        sub_of[p] = __builtin_amdgcn_readfirstlane(rr / C::SLICE_ROWS);
        if (r < MT) {
            const int m = m0 + r < a.T ? m0 + r : a.T - 1;   // rows past the end repeat the last one and are not stored
            src[p] = static_cast<const T*>(a.x) + (int64_t)m * a.x_st;
        } else {
            const int f = r - MT;
            const int row = head * D + pair0 + (f < NT / 2 ? f : D / 2 + f - NT / 2);
            src[p] = static_cast<const T*>(a.w) + (int64_t)row * a.w_st;
        }
        src[p] += sub_of[p] * C::KT + piece * 8;
    }
    const int n_slices = a.Hin / C::KT;
    const int n_stages = (n_slices + SUB - 1) / SUB;
    auto issue = [&](int st, int slot_bytes) {
#pragma unroll
        for (int p = 0; p < PASSES; ++p) {
            if (SUB == 1 || st * SUB + sub_of[p] < n_slices)
                async_copy16(src[p], lds0 + slot_bytes + (p * 64 + wave * 8) * C::ROW_BYTES);
            src[p] += SUB * C::KT;
        }
    };

    uint32_t ra[CH];   // this wave's chunks: row n of the tile's first block, in stage 0
#pragma unroll
    for (int c = 0; c < CH; ++c) {
        const int chunk = kg + KG * c;
        ra[c] = lds0 + chunk / 4 * (C::SLICE_ROWS * C::ROW_BYTES) + TL::offset(n, chunk % 4 * 16 + hh * 8);
    }
    auto ld = [&](uint32_t addr) -> frag {
        return *reinterpret_cast<const __attribute__((address_space(3))) frag*>((uintptr_t)addr);
    };
    constexpr int BLK = 32 * C::ROW_BYTES;
    const uint32_t xo = wm * MB * BLK, wo = MT * C::ROW_BYTES + wn * NB * BLK;

    f32x16 acc[MB][NB];
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[mb][nb][i] = 0.f;

#pragma unroll
    for (int s = 0; s < NST - 1; ++s)
        if (s < n_stages) issue(s, s * C::STAGE_BYTES);
    int cur = 0;                                   // byte offset of the stage to read
    int nxt = (NST - 1) * C::STAGE_BYTES;          // and of the one to fill: the stage read in the step before
    for (int s = 0; s < n_stages; ++s) {
        // stage s has landed; the NST - 2 stages behind it stay in flight while all of them are whole ones
        const bool more = s + NST - 1 < n_stages;
        if (more) wait_copies_but(IntC<(NST - 2) * PASSES>{});
        else wait_async_copies();
        lds_barrier();
        if (more) issue(s + NST - 1, nxt);
        frag xf[CH][MB], wf[CH][NB];
#pragma unroll
        for (int c = 0; c < CH; ++c) {
            const uint32_t base = ra[c] + cur;
#pragma unroll
            for (int mb = 0; mb < MB; ++mb) xf[c][mb] = ld(base + xo + mb * BLK);
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) wf[c][nb] = ld(base + wo + nb * BLK);
        }
#pragma unroll
        for (int c = 0; c < CH; ++c)
            if (SUB == 1 || s * SUB + (kg + KG * c) / 4 < n_slices) {
#pragma unroll
                for (int mb = 0; mb < MB; ++mb)
#pragma unroll
                    for (int nb = 0; nb < NB; ++nb) acc[mb][nb] = mma(wf[c][nb], xf[c][mb], acc[mb][nb]);
            }
        nxt = cur;
        cur = cur + C::STAGE_BYTES == NST * C::STAGE_BYTES ? 0 : cur + C::STAGE_BYTES;
    }

    // ---- partial sums to LDS (as [token][feature] per wave), then 16 outputs per thread: 8 features of the
    // lower half of the tile and the 8 that they are paired with
    lds_barrier();
    float* part = reinterpret_cast<float*>(smem + wave % (C::KGE * MW * NW) * C::PART_BYTES) + n * C::PITCH + 4 * hh;
    auto each_piece = [&](auto&& f) {   // 4 consecutive features of one token
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
#pragma unroll
                for (int k4 = 0; k4 < 4; ++k4)
                    f(*reinterpret_cast<f32x4*>(part + mb * 32 * C::PITCH + nb * 32 + 8 * k4), acc[mb][nb], 4 * k4);
    };
    auto put = [](f32x4& at, const f32x16& v, int i) { at = f32x4{v[i], v[i + 1], v[i + 2], v[i + 3]}; };
    if constexpr (C::FOLD) {
        if (kg >= C::KGE) each_piece(put);
        __syncthreads();
        if (kg < C::KGE) {
            each_piece([](const f32x4& at, f32x16& v, int i) {
#pragma unroll
                for (int e = 0; e < 4; ++e) v[i + e] += at[e];
            });
            each_piece(put);   // the same lane wrote and read this place: nobody else's sums are touched
        }
    } else {
        each_piece(put);
    }
    __syncthreads();
    const bool rotate = head < a.n_q + a.n_k;
    T* out;
    int64_t out_st;
    if (head < a.n_q) {
        out = static_cast<T*>(a.q) + (int64_t)head * D;
        out_st = (int64_t)a.n_q * D;
    } else if (rotate) {
        out = static_cast<T*>(a.k) + (int64_t)(head - a.n_q) * D;
        out_st = (int64_t)a.n_k * D;
    } else {
        out = static_cast<T*>(a.v) + (int64_t)(head - a.n_q - a.n_k) * D;
        out_st = (int64_t)a.n_v * D;
    }
    constexpr int PER_ROW = NT / 16;
    for (int it = tid; it < MT * PER_ROW; it += 512) {
        const int t = it / PER_ROW, u = it % PER_ROW, m = m0 + t;
        if (m >= a.T) break;
        float y[2][8];
#pragma unroll
        for (int half = 0; half < 2; ++half) {
            const int f = half * (NT / 2) + 8 * u;
            const char* at = smem + (t / (MB * 32) * NW + f / (NB * 32)) * C::PART_BYTES;
            const int within = t % (MB * 32) * C::PITCH + f % (NB * 32);
#pragma unroll
            for (int e = 0; e < 8; ++e) y[half][e] = 0.f;
#pragma unroll
            for (int k = 0; k < C::KGE; ++k) {
                const float* row = reinterpret_cast<const float*>(at + k * (MW * NW) * C::PART_BYTES) + within;
                const f32x4 v0 = *reinterpret_cast<const f32x4*>(row), v1 = *reinterpret_cast<const f32x4*>(row + 4);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    y[half][e] += v0[e];
                    y[half][4 + e] += v1[e];
                }
            }
        }
        const int i0 = pair0 + 8 * u;
        bf16x8 lo, hi;
        if (rotate) {
            int p = a.pos[m];
            p = p < 0 ? 0 : (p >= a.n_pos ? a.n_pos - 1 : p);
            const f32x8 c8 = gload_frag<float>(a.cos_tab + (int64_t)p * (D / 2) + i0);
            const f32x8 s8 = gload_frag<float>(a.sin_tab + (int64_t)p * (D / 2) + i0);
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                lo[e] = (__bf16)(y[0][e] * c8[e] - y[1][e] * s8[e]);
                hi[e] = (__bf16)(y[1][e] * c8[e] + y[0][e] * s8[e]);
            }
        } else {
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                lo[e] = (__bf16)y[0][e];
                hi[e] = (__bf16)y[1][e];
            }
        }
        T* row = out + (int64_t)m * out_st + i0;
        *reinterpret_cast<bf16x8*>(row) = lo;
        *reinterpret_cast<bf16x8*>(row + D / 2) = hi;
    }
}

template <int MT, int NT, int KG, int MW, int NW, int SUB, int NST>
static hipError_t launch_qkv_rope_splitk(QkvArgs& a, hipStream_t stream) {
    using C = QkvSplitK<__bf16, MT, NT, KG, MW, NW, SUB, NST>;
    auto kern = ttt_qkv_rope_splitk_kernel<__bf16, MT, NT, KG, MW, NW, SUB, NST>;
    static LdsOptIn lds_opt_in;
    if (hipError_t e = lds_opt_in.ensure((const void*)kern, C::LDS); e != hipSuccess) return e;
    a.m_tiles = (a.T + MT - 1) / MT;
    a.n_tiles = a.f_count / NT;
    const int64_t m_per = a.m_per, m_groups = (a.m_tiles + m_per - 1) / m_per;
    const int64_t grid = 8 * m_per * ((m_groups * a.n_tiles + 7) / 8);
    if (grid > 0x7fffffffLL) return hipErrorInvalidValue;
    ProfileScope prof("ttt_qkv_rope_kernel", stream);
    hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(512), C::LDS, stream, a);
    return hipGetLastError();
}

static hipError_t launch_qkv_rope_256(QkvArgs& a, hipStream_t stream) {
    constexpr int LDS = 2 * (256 + 256) * 64 * 2;
    auto kern = ttt_qkv_rope_kernel<__bf16>;
    static LdsOptIn lds_opt_in;
    if (hipError_t e = lds_opt_in.ensure((const void*)kern, LDS); e != hipSuccess) return e;
    a.m_tiles = (a.T + 255) / 256;
    a.n_tiles = (a.f_count + 255) / 256;
    const int64_t m_per = a.m_per, m_groups = (a.m_tiles + m_per - 1) / m_per;
    const int64_t grid = 8 * m_per * ((m_groups * a.n_tiles + 7) / 8);
    if (grid > 0x7fffffffLL) return hipErrorInvalidValue;
    ProfileScope prof("ttt_qkv_rope_kernel", stream);
    hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(256), LDS, stream, a);
    return hipGetLastError();
}

// in the order of kQkvTiles
static hipError_t (*const kQkvLaunchers[])(QkvArgs&, hipStream_t) = {
    launch_qkv_rope_256,
    launch_qkv_rope_splitk<128, 128, 2, 2, 2, 1, 2>,
    launch_qkv_rope_splitk<128, 128, 2, 2, 2, 1, 4>,
    launch_qkv_rope_splitk<128, 64, 4, 2, 1, 1, 6>,
    launch_qkv_rope_splitk<64, 64, 4, 1, 2, 1, 4>,
    launch_qkv_rope_splitk<64, 32, 4, 2, 1, 2, 3>,
    launch_qkv_rope_splitk<32, 32, 8, 1, 1, 2, 4>,
};
static_assert(sizeof(kQkvLaunchers) / sizeof(kQkvLaunchers[0]) == kQkvTileKinds, "one launcher per kind of tile");

// n_q + n_k heads are rotated and go to q and k, n_v heads go to v as they are.  With n_q = n_k = 0 the
// call is a plain projection y = x w^T into v ([tokens, n_v * 128]).
hipError_t launch_qkv_rope(const void* x, const void* w, const float* cos_tab, const float* sin_tab, const int* pos, void* q,
                           void* k, void* v, int64_t tokens, int hidden_in, int n_q, int n_k, int n_v, int64_t x_st,
                           int64_t w_st, int n_pos, hipStream_t stream) {
    QkvArgs a;
    a.x = x;
    a.w = w;
    a.cos_tab = cos_tab;
    a.sin_tab = sin_tab;
    a.pos = pos;
    a.q = q;
    a.k = k;
    a.v = v;
    a.T = (int)tokens;
    a.Hin = hidden_in;
    a.n_q = n_q;
    a.n_k = n_k;
    a.n_v = n_v;
    a.n_pos = n_pos;
    a.x_st = x_st;
    a.w_st = w_st;
    int n_cu = 0;
    if (hipError_t e = current_device_cu_count(n_cu); e != hipSuccess) return e;
    // the largest kind addresses its 256 rows with 32-bit byte offsets (the others with a 64-bit address per row)
    const bool largest_fits = x_st < (int64_t)1 << 23 && w_st < (int64_t)1 << 23;
    const int features = (n_q + n_k + n_v) * 128;
    const QkvPlan plan = plan_qkv(tokens, hidden_in, features, largest_fits, n_cu);
    auto launch = [&](int kind, int f_first, int f_count) {
        const QkvTile& t = kQkvTiles[kind];
        a.f_first = f_first;
        a.f_count = f_count;
        a.m_per = qkv_group(t, (a.T + t.mt - 1) / t.mt, (f_count + t.nt - 1) / t.nt, n_cu);
        return kQkvLaunchers[kind](a, stream);
    };
    if (hipError_t e = launch(plan.first, 0, plan.f_first); e != hipSuccess || plan.second < 0) return e;
    return launch(plan.second, plan.f_first, features - plan.f_first);
}

}  // namespace ttt
