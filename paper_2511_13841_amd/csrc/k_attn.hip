// Ragged causal GQA attention over the paged KV cache (split-KV).  The cache holds bf16-rounded values in
// binary16 containers (see rope_kv_kernel): the MFMAs here are the f16 ones, whose 11-bit operands let the rotated
// query and the probabilities go in as ONE term each (as bf16 each needed a hi + lo pair to keep the scores and the
// weighted sum at fp32-like accuracy, which doubled the matrix work).
//
// One workgroup = one (sequence, KV head, chunk of pm.chunk tokens: 2048, or 1024 for models with two KV heads).
// All G*(1+k_i) query rows that share the KV head are served by ONE pass over the chunk's KV: arithmetic per KV
// byte is G*(1+k) <= 231 flop/B, below the machine's ridge, so the kernel is built around streaming pages at HBM rate:
//   * pages are stored in MFMA operand order, so a 32-token tile (2 pages of K and of V) is four contiguous runs
//     copied to LDS with coalesced 16-byte loads (asynchronous, non-temporal, a ring of four tiles that never
//     drains) and read back lane-linearly (no bank conflicts);
//   * S^T = K Q^T with v_mfma_f32_16x16x32_f16 puts 8 tokens of one query row in each lane, so the row max needs
//     two cross-lane steps and the probabilities are already laid out as the B operand of O^T += V^T P^T;
//   * chunks start at absolute multiples of the chunk length and each chunk is reduced from scratch, then chunks
//     are merged in ascending order: a row's result does not depend on the batch it is verified in (speculative
//     verification and one-token decoding give bit-identical rows).
// Wave w of 8 owns query-row block w (16 rows); more than 8 row blocks go to attn_rows_kernel.
#include "das_internal.h"

// ring depth: four 16 KiB stages per workgroup (one tile in use, three in flight), two workgroups per CU.  Five stages
// (2 x 80 KiB = all of the CU's LDS) leave room for one workgroup only and are slower (320 against 299 us per layer
// on contexts of 32k-64k tokens).
#define DAS_ATTN_STAGES 4
// ring of attn_rows_kernel, which has a CU to itself: two tiles in use, five in flight, one being left
#define DAS_ATTN_ROWS_STAGES 8

typedef __attribute__((ext_vector_type(8))) _Float16 f16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;

// two floats -> packed fp16 pair (round to nearest even), and back
__device__ __forceinline__ uint32_t pack_h2(float a, float b) {
    typedef __attribute__((ext_vector_type(2))) _Float16 h2;
    h2 v = {(_Float16)a, (_Float16)b};
    return *reinterpret_cast<uint32_t *>(&v);
}
__device__ __forceinline__ float2 unpack_h2(uint32_t u) {
    typedef __attribute__((ext_vector_type(2))) _Float16 h2;
    h2 v = *reinterpret_cast<h2 *>(&u);
    return make_float2((float)v[0], (float)v[1]);
}

// 16-byte-per-lane asynchronous copy HBM -> LDS (no VGPR staging): lane l's 16 bytes land at
// lds_wave_base + 16*l.  Inline assembly, so that the copies are ordered only by the explicit
// s_waitcnt/s_barrier of the tile loop (M0 carries the LDS address; 1 wait state before its use).  The KV stream is
// read once per launch: the non-temporal hint keeps it from pushing the split-KV partials, which are written here and
// read back by the merge kernel, out of the caches (measured: attention -10 %, merge -20 %).
__device__ __forceinline__ void dma16(const void *g, uint32_t lds_wave_base) {
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off nt" ::"v"(g), "s"(lds_wave_base) : "memory", "m0");
}

// The same copy with a scalar base and a 32-bit lane offset; `shared` != 0 (the same for the whole workgroup): without the hint,
// for a stream that several workgroups read side by side.  The choice is made inside the assembly, so that the tile step stays
// one basic block.
__device__ __forceinline__ void dma16_s(uint32_t voff, const void *base, uint32_t lds_wave_base, int shared) {
    asm volatile("s_mov_b32 m0, %2\n\ts_cmp_lg_u32 %3, 0\n\ts_cbranch_scc1 .Lshared%=\n\tglobal_load_lds_dwordx4 %0, %1 nt\n\ts_branch .Lissued%=\n"
                 ".Lshared%=:\n\tglobal_load_lds_dwordx4 %0, %1\n.Lissued%=:"
                 ::"v"(voff), "s"(base), "s"(lds_wave_base), "s"(shared) : "memory", "m0", "scc");
}

// Up to 128 query rows per KV head.  Four waves per SIMD are asked for: besides the occupancy, it
// makes the compiler keep the MFMA accumulators in ordinary VGPRs, where the (rare) rescale can reach them
// without copies out of the accumulation register file on every tile.
template <int D, int NS>
__global__ __launch_bounds__(512, 4) void attn_partial_kernel(PassMeta pm, const int *__restrict__ items,
                                                           const f16_t *__restrict__ q_h,
                                                           const f16_t *__restrict__ kpool,
                                                           const f16_t *__restrict__ vpool,
                                                           uint16_t *__restrict__ part_o, float *__restrict__ part_ml,
                                                           bf16_t *__restrict__ out,
                                                           int Hkv, int G, int qstride, float scale_log2e) {
    constexpr int KFR = D / 32;            // K fragments (1 KiB) per page
    constexpr int VDB = D / 16;            // V dim blocks (512 B) per page
    constexpr int PAGE_E = DAS_PAGE * D;   // elements of one (page, head) block
    constexpr int PAGE_B = PAGE_E * 2;
    constexpr int TILE_B = 4 * PAGE_B;     // K page0, K page1, V page0, V page1
    constexpr int UNITS_PER_SEG = PAGE_B / 16;
    constexpr int NT = 512, RBW = 1;
    constexpr int NLOAD = (TILE_B / 16) / NT;
    static_assert((TILE_B / 16) % NT == 0, "tile must divide over the threads");
    // ring of NS tile stages: one being read, NS-1 being filled
    extern __shared__ __align__(16) unsigned char smem[];      // NS * TILE_B bytes
    const uint32_t lds_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char *)smem;

    // work items arrive sorted longest first: sequence, chunk | KV head << 20
    const int b = items[2 * blockIdx.x], chunk = items[2 * blockIdx.x + 1] & 0xFFFFF;
    const int kvh = items[2 * blockIdx.x + 1] >> 20;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int ctx = pm.b_start[b], n = pm.b_n[b], row0 = pm.b_row0[b];
    const int R = G * n;
    const int tok_begin = chunk * pm.chunk;
    const int tok_total = ctx + n;
    const int tok_end = min(tok_begin + pm.chunk, tok_total);
    const int ntiles = (tok_end - tok_begin + DAS_ATTN_TILE - 1) / DAS_ATTN_TILE;
    const int npages = (tok_total + DAS_PAGE - 1) / DAS_PAGE;
    const int *pt = pm.page_table + (size_t)pm.b_slot[b] * pm.max_pages;
    // the chunk's (at most 64) page ids, one per lane, fetched once: the tile loop then takes them with
    // v_readlane and never waits on a vector load of its own (which would also wait for every copy in flight)
    const int first_page = tok_begin >> 4;
    constexpr int NPREG = DAS_ATTN_CHUNK_MAX / DAS_PAGE / 64;      // registers of 64 page ids each
    int my_page[NPREG];
#pragma unroll
    for (int q = 0; q < NPREG; ++q) my_page[q] = pt[min(first_page + q * 64 + lane, npages - 1)];

    // ---- query fragments (B operand: lane l = query row l%16, dims 8*(l/16)..+7 of each 32-dim step)
    f16x8 qf[RBW][KFR];
    int lim[RBW];           // last KV position this lane's query row may see (-1: padding row)
    bool any_active = false;
#pragma unroll
    for (int i = 0; i < RBW; ++i) {
        const int rr = (wave * RBW + i) * 16 + (lane & 15);
        const bool valid = rr < R;
        const int j = valid ? rr / G : 0, g = valid ? rr % G : 0;
        lim[i] = valid ? ctx + j : -1;
        any_active |= ((wave * RBW + i) * 16 < R);
        const size_t qo = (size_t)(row0 + j) * qstride + (size_t)(kvh * G + g) * D + 8 * (lane >> 4);
#pragma unroll
        for (int ks = 0; ks < KFR; ++ks) {
            uint4 v = valid ? *reinterpret_cast<const uint4 *>(q_h + qo + ks * 32) : make_uint4(0, 0, 0, 0);
            qf[i][ks] = *reinterpret_cast<f16x8 *>(&v);
        }
    }

    float m_run[RBW], l_run[RBW];
    f32x4 acc[RBW][VDB];
#pragma unroll
    for (int i = 0; i < RBW; ++i) {
        m_run[i] = -INFINITY; l_run[i] = 0.f;
#pragma unroll
        for (int db = 0; db < VDB; ++db) acc[i][db] = (f32x4){0.f, 0.f, 0.f, 0.f};
    }

    // ---- tile loader: 16-byte unit u of the tile belongs to segment u / UNITS_PER_SEG
    auto issue = [&](int ti, int stage) {
        // pages 2*ti and 2*ti+1 of the chunk (the second one was clamped to the last page at load)
        static_assert(NPREG <= 2, "at most two registers of 64 page ids per chunk");
        const int li = (2 * ti) & 63;
        int pg0 = __builtin_amdgcn_readlane(my_page[0], li), pg1 = __builtin_amdgcn_readlane(my_page[0], li + 1);
        if (NPREG == 2) {
            const int qg0 = __builtin_amdgcn_readlane(my_page[NPREG - 1], li), qg1 = __builtin_amdgcn_readlane(my_page[NPREG - 1], li + 1);
            if (2 * ti >= 64) { pg0 = qg0; pg1 = qg1; }
        }
#pragma unroll
        for (int jn = 0; jn < NLOAD; ++jn) {
            const int u = tid + jn * NT;
            const int seg = u / UNITS_PER_SEG, off = u % UNITS_PER_SEG;
            const int pg = (seg & 1) ? pg1 : pg0;
            const f16_t *base = (seg < 2 ? kpool : vpool) + ((size_t)pg * Hkv + kvh) * PAGE_E;
            dma16(reinterpret_cast<const uint4 *>(base) + off, lds_base + stage * TILE_B + jn * NT * 16 + wave * 1024);
        }
    };

    // ---- the three phases of a tile, kept apart so that two tiles can be interleaved below
    struct Scores { f32x4 v[RBW][2]; };
    struct Probs { f16x8 v[RBW]; };

    // S^T = K Q^T : s[i][pg][r] = score of token 16*pg + 4*(lane/16) + r for query row lane%16
    auto qk = [&](const unsigned char *cur, Scores &s) {
#pragma unroll
        for (int i = 0; i < RBW; ++i) { s.v[i][0] = (f32x4){0.f, 0.f, 0.f, 0.f}; s.v[i][1] = (f32x4){0.f, 0.f, 0.f, 0.f}; }
#pragma unroll
        for (int ks = 0; ks < KFR; ++ks) {
            const f16x8 k0 = *reinterpret_cast<const f16x8 *>(cur + (ks * 64 + lane) * 16);
            const f16x8 k1 = *reinterpret_cast<const f16x8 *>(cur + PAGE_B + (ks * 64 + lane) * 16);
#pragma unroll
            for (int i = 0; i < RBW; ++i) {
                s.v[i][0] = __builtin_amdgcn_mfma_f32_16x16x32_f16(k0, qf[i][ks], s.v[i][0], 0, 0, 0);
                s.v[i][1] = __builtin_amdgcn_mfma_f32_16x16x32_f16(k1, qf[i][ks], s.v[i][1], 0, 0, 0);
            }
        }
    };

    // Softmax with a lazily updated reference: p = exp2(s * scale - m_ref).  m_ref only moves when the row's
    // maximum in this tile exceeds it by more than 8 (a factor 256), which after a row's first tile almost never
    // happens: the common path needs no cross-lane step and no rescaling of the accumulators.  The decision is
    // taken per ROW (from the row's own maximum), so a row's arithmetic never depends on its neighbours;
    // softmax is shift-invariant, the result is exact.
    // row_check: causal mask (only the chunk's last tiles need one), row maximum, and the rare move of m_ref.
    auto row_check = [&](int ti, Scores &s) {
        const int tile_tok0 = tok_begin + ti * DAS_ATTN_TILE;
        const bool need_mask = tile_tok0 + DAS_ATTN_TILE - 1 > ctx;
#pragma unroll
        for (int i = 0; i < RBW; ++i) {
            if (need_mask) {
                const int pbase = tile_tok0 + 4 * (lane >> 4);
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    if (pbase + r > lim[i]) s.v[i][0][r] = -INFINITY;
                    if (pbase + 16 + r > lim[i]) s.v[i][1][r] = -INFINITY;
                }
            }
            float mt = fmaxf(s.v[i][0][0], s.v[i][1][0]);
#pragma unroll
            for (int r = 1; r < 4; ++r) mt = fmaxf(mt, fmaxf(s.v[i][0][r], s.v[i][1][r]));
            mt *= scale_log2e;
            if (__any(mt > m_run[i] + 8.f)) {          // some row of this block may have to move its reference
                mt = fmaxf(mt, __shfl_xor(mt, 16));
                mt = fmaxf(mt, __shfl_xor(mt, 32));    // the row's maximum, same in its four lanes
                const float mn = (mt > m_run[i] + 8.f) ? mt : m_run[i];
                const float alpha = exp2f(m_run[i] - ((mn == -INFINITY) ? 0.f : mn));   // 1 for rows that stay
                const bool had_sum = m_run[i] != -INFINITY && alpha != 1.f;            // a first tile has nothing to rescale
                l_run[i] *= alpha;
                m_run[i] = mn;
                if (__any(had_sum)) {                  // rare: a reference moving after the row's first tile
#pragma unroll
                    for (int db = 0; db < VDB; ++db) acc[i][db] *= alpha;
                }
            }
        }
    };
    // probabilities of a checked tile, rounded to binary16 (at most 256 by the rule above; what falls below the
    // format's 6e-8 is lost against a row sum of at least 1), and the row sums of the unrounded values
    auto probs = [&](const Scores &s, Probs &p) {
#pragma unroll
        for (int i = 0; i < RBW; ++i) {
            const float ms = (m_run[i] == -INFINITY) ? 0.f : m_run[i];
            float ps = 0.f;
            float pv[8];
#pragma unroll
            for (int r = 0; r < 8; ++r) {
                pv[r] = __builtin_amdgcn_exp2f(__builtin_fmaf(s.v[i][r >> 2][r & 3], scale_log2e, -ms));
                ps += pv[r];
            }
            l_run[i] += ps;
            typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
            const u32x4 hv = {pack_h2(pv[0], pv[1]), pack_h2(pv[2], pv[3]), pack_h2(pv[4], pv[5]), pack_h2(pv[6], pv[7])};
            p.v[i] = *reinterpret_cast<const f16x8 *>(&hv);
        }
    };

    // O^T += V^T P^T : A = V fragment (dims x 32 token slots), B = probabilities
    auto pv = [&](const unsigned char *cur, const Probs &p) {
#pragma unroll
        for (int db = 0; db < VDB; ++db) {
            // the two halves of a fragment (tokens of the first and of the second page) are read by separate
            // 8-byte loads straight into its registers; left to itself the compiler pairs the loads of
            // neighbouring dim blocks instead and pays for it with register moves
            typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;
            typedef const volatile __attribute__((address_space(3))) u32x2 *lds_u32x2_ptr;
            const u32x2 lo = *(lds_u32x2_ptr)(cur + 2 * PAGE_B + (db * 64 + lane) * 8);
            const u32x2 hi = *(lds_u32x2_ptr)(cur + 3 * PAGE_B + (db * 64 + lane) * 8);
            typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
            u32x4 vv = {lo[0], lo[1], hi[0], hi[1]};
            const f16x8 vf = *reinterpret_cast<f16x8 *>(&vv);
#pragma unroll
            for (int i = 0; i < RBW; ++i) acc[i][db] = __builtin_amdgcn_mfma_f32_16x16x32_f16(vf, p.v[i], acc[i][db], 0, 0, 0);
        }
    };

    // (Matrix and vector instructions of one SIMD do not overlap on this chip -- measured: their times add even with
    // four waves per SIMD -- so nothing is gained by interleaving the score MFMAs of one tile with the exponentials of
    // another; what counts is the instruction count per tile.)
    const bool work = any_active;
    {
        // One tile per barrier, ring of NS stages: tile ti in use, tiles ti+1 .. ti+NS-1 in flight.  Copies are issued
        // unconditionally (past the end: the last tile again, into a stage nobody reads any more), so "tile ti has
        // landed" is the same s_waitcnt in every iteration and the copy queue never drains at a barrier.
        const int last = ntiles - 1;
#pragma unroll
        for (int s0 = 0; s0 < NS - 1; ++s0) issue(min(s0, last), s0);
        int stage = 0;
        for (int ti = 0; ti < ntiles; ++ti) {
            constexpr int NEWER = (NS - 2) * NLOAD;
            __builtin_amdgcn_s_waitcnt(0xF70 | (NEWER & 15) | ((NEWER >> 4) << 14));
            __builtin_amdgcn_s_barrier();      // tile ti visible to all waves; all waves are done with tile ti-1
            asm volatile("" ::: "memory");
            issue(min(ti + NS - 1, last), stage == 0 ? NS - 1 : stage - 1);
            if (work) {
                const unsigned char *c0 = smem + stage * TILE_B;
                Scores s0;
                Probs p0;
                qk(c0, s0);
                row_check(ti, s0);
                probs(s0, p0);
                pv(c0, p0);
            }
            stage = stage == NS - 1 ? 0 : stage + 1;
        }
    }
    __builtin_amdgcn_s_waitcnt(0xF70);     // vmcnt(0): no copy may land in LDS after this workgroup is gone

    // ---- partial results per 16-row block: (m, l) per row in fp32 and the chunk's normalised output acc / l in
    // fp16 (values bounded by the largest |v|; 11 significant bits, well below the bf16 rounding of the merged
    // result), in the lane order the accumulators are held in: dim blocks 2q and 2q+1 share one 16-byte store, a
    // contiguous KiB per instruction.  HBM writes cost this kernel about three times their bytes in read
    // bandwidth, hence the narrow format.
    const int nrb = (R + 15) >> 4;
    // Partials of a long sequence (many chunks) leave with non-temporal stores: they are many, the merge reads each once,
    // and kept in the caches they cost the KV stream more than the merge gains (contexts of 32k-64k: attention -20 us,
    // merge +7 us per layer); the few partials of short sequences stay cached for the merge.
    const int nchunk_b = pm.b_nchunk[b];
    const bool stream_out = nchunk_b >= 8;
    // A sequence of one chunk needs no merge: its rows are finished here with the arithmetic attn_merge_kernel would
    // apply to that one chunk ((o * l) * (1 / l) on the binary16-rounded o, then bf16), so a row comes out the same
    // whether its sequence had one chunk or more (later chunks that the row cannot see are skipped by the merge).
    const bool single = nchunk_b == 1;
#pragma unroll
    for (int i = 0; i < RBW; ++i) {
        float l = l_run[i];
        l += __shfl_xor(l, 16);
        l += __shfl_xor(l, 32);
        const int rb = wave * RBW + i;
        if (rb < nrb) {
            const size_t id = ((size_t)pm.b_prow[b] + (size_t)chunk * nrb + rb) * Hkv + kvh;
            const float inv = l > 0.f ? 1.f / l : 0.f;
            if (single) {
                const int rr = rb * 16 + (lane & 15);
                if (rr < R) {
                    const int t = pm.b_row0[b] + rr / G, a = kvh * G + rr % G;
                    const float invden = 1.f / l;
                    auto fin = [&](float x, float y) -> uint32_t {      // two neighbouring dims -> two bf16
                        const float2 o = unpack_h2(pack_h2(x, y));
                        uint32_t u0 = __float_as_uint((o.x * l) * invden), u1 = __float_as_uint((o.y * l) * invden);
                        u0 += 0x7FFFu + ((u0 >> 16) & 1u);
                        u1 += 0x7FFFu + ((u1 >> 16) & 1u);
                        return (u0 >> 16) | (u1 & 0xFFFF0000u);
                    };
#pragma unroll
                    for (int db = 0; db < VDB; ++db) {
                        const f32x4 o = acc[i][db] * inv;
                        *reinterpret_cast<uint2 *>(out + frag_off(t, a * D + 16 * db + 4 * (lane >> 4), qstride)) =
                            make_uint2(fin(o[0], o[1]), fin(o[2], o[3]));
                    }
                }
                continue;
            }
            if ((lane >> 4) == 0) *reinterpret_cast<float2 *>(part_ml + id * 32 + 2 * lane) = make_float2(m_run[i], l);
            uint4 *dst = reinterpret_cast<uint4 *>(part_o + id * (16 * D)) + lane;
#pragma unroll
            for (int q = 0; q < VDB / 2; ++q) {
                const f32x4 lo = acc[i][2 * q] * inv, hi = acc[i][2 * q + 1] * inv;
                typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
                const u32x4 val = {pack_h2(lo[0], lo[1]), pack_h2(lo[2], lo[3]), pack_h2(hi[0], hi[1]), pack_h2(hi[2], hi[3])};
                // (inline assembly: written with the builtin, the two branches are merged into one plain store.  The wait
                // states cover the hazard between a 16-byte store and a later write of its data registers, which the
                // compiler handles for its own stores only.  No load may follow these stores in this kernel: the compiler's
                // s_waitcnt bookkeeping does not count them.)
                if (stream_out) asm volatile("global_store_dwordx4 %0, %1, off nt\n\ts_nop 4" ::"v"(dst + q * 64), "v"(val) : "memory");
                else *reinterpret_cast<u32x4 *>(dst + q * 64) = val;
            }
        }
    }
}

// ---------------------------------------------------------------- shared by the attention kernels and the merge
// One finished chunk of a row -- normalised output o (binary16 values), row sum l, reference m -- folded into the running
// (M, den, num) of the row; ascending chunk order.  Written out so that every caller rounds at the same places.
struct ChunkScale { float a0, a1; };
__device__ __forceinline__ ChunkScale chunk_fold(float &M, float &den, float m, float l) {
    const float mn = fmaxf(M, m);
    const ChunkScale c = {exp2f(M - mn), l * exp2f(m - mn)};
    den = __builtin_fmaf(den, c.a0, c.a1);
    M = mn;
    return c;
}
__device__ __forceinline__ float chunk_num(float num, float o, ChunkScale c) { return __builtin_fmaf(c.a0, num, c.a1 * o); }
__device__ __forceinline__ uint32_t rne_bf16(float f) {
    uint32_t u = __float_as_uint(f);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return u >> 16;
}

// ---------------------------------------------------------------- many query rows per KV head (129 .. 256)
// Prompt blocks and long drafts: up to 16 row blocks share a KV head, and the launch is bound by its matrix and vector
// instructions, not by its copies.  Three things follow:
//   * 8 waves of two row blocks (16 waves of one read every K and V fragment from LDS twice as often, and V's 8-byte reads
//     alone then take longer than the MFMAs);
//   * the tile loop is pipelined by hand: while the softmax of tile t runs, the same wave's MFMAs are the scores of tile t+1
//     and the weighted sum of tile t-1, so every MFMA has vector instructions of the same wave to cover.  On this chip a
//     16x16x32 MFMA hides about two vector instructions (or one v_exp) of its OWN wave placed behind it, and none of another
//     wave: 16 MFMAs 130 ns, 64 FMAs 101 ns, the two dealt out one to four 169 ns, in two runs one after the other 186 ns;
//   * an item may cover ALL chunks of its block (chunk field 0xFFFFF): the chunk results are then folded one after the other
//     with the merge kernel's arithmetic and the finished rows leave here.  The running sums rest in a workspace of fixed size
//     between chunks (the registers are full), so a prefill pass is not limited by the partial buffers (27k prompt tokens of
//     the 7B shape: passes of up to 2048 rows instead of 36 .. 290).
// The ring holds NS tiles: V of tile t-1, tile t, K of tile t+1 in use, the others in flight.
// Measured on the last pass of a 16k prompt (7B heads, 228 items of 512 tiles): 1.15 us per tile and CU, of which the MFMAs
// alone with their barriers take 0.87 (clock lowered by their power draw), LDS reads and softmax the rest; taking the copies
// out saves 0.1.  16 waves of one row block with nothing pipelined: 1.2.  Behind it stands the size of the passes: 27k prompt
// tokens (7B, 28 layers) 1125 -> 450 ms.
template <int D>
__global__ __launch_bounds__(512, 2) void attn_rows_kernel(PassMeta pm, const int *__restrict__ items, const f16_t *__restrict__ q_h,
                                                          const f16_t *__restrict__ kpool, const f16_t *__restrict__ vpool,
                                                          uint16_t *__restrict__ part_o, float *__restrict__ part_ml, float4 *__restrict__ fold,
                                                          bf16_t *__restrict__ out, int Hkv, int G, int qstride, float scale_log2e) {
    constexpr int KFR = D / 32, VDB = D / 16, PAGE_E = DAS_PAGE * D, PAGE_B = PAGE_E * 2, TILE_B = 4 * PAGE_B;
    constexpr int UNITS_PER_SEG = PAGE_B / 16, NT = 512, NLOAD = (TILE_B / 16) / NT, RBW = 2, NS = DAS_ATTN_ROWS_STAGES, AHEAD = NS - 2;
    static_assert((TILE_B / 16) % NT == 0 && UNITS_PER_SEG % 64 == 0 && NT == 2 * UNITS_PER_SEG * (NLOAD == 1 ? 2 : 1), "whole waves per page segment");
    extern __shared__ __align__(16) unsigned char smem[];      // NS * TILE_B bytes
    const uint32_t lds_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char *)smem;

    const int b = items[2 * blockIdx.x], chunk = items[2 * blockIdx.x + 1] & 0xFFFFF, kvh = items[2 * blockIdx.x + 1] >> 20;
    const bool whole = chunk == 0xFFFFF;
    const int shared_stream = (chunk + 1) >> 20;      // 1: whole (kept an integer in a scalar register)
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int ctx = pm.b_start[b], n = pm.b_n[b], row0 = pm.b_row0[b];
    const int R = G * n, nrb = (R + 15) >> 4, tok_total = ctx + n;
    const int last_page = (tok_total - 1) >> 4, tiles_per_chunk = pm.chunk / DAS_ATTN_TILE;
    const int t_begin = whole ? 0 : chunk * tiles_per_chunk;
    const int t_end = whole ? (tok_total + DAS_ATTN_TILE - 1) / DAS_ATTN_TILE : min((chunk + 1) * tiles_per_chunk, (tok_total + DAS_ATTN_TILE - 1) / DAS_ATTN_TILE);
    // page ids come through scalar loads, one tile ahead of the copies that need them (a vector load would wait for every
    // copy in flight); the table was written by earlier kernels of the stream
    typedef const __attribute__((address_space(4))) int *const_int_ptr;
    const const_int_ptr pt = (const_int_ptr)(uintptr_t)(pm.page_table + (size_t)pm.b_slot[b] * pm.max_pages);

    f16x8 qf[RBW][KFR];
    int lim[RBW];           // last KV position this lane's query row may see (-1: padding row)
#pragma unroll
    for (int i = 0; i < RBW; ++i) {
        const int rr = (wave * RBW + i) * 16 + (lane & 15);
        const bool valid = rr < R;
        const int j = valid ? rr / G : 0, g = valid ? rr % G : 0;
        lim[i] = valid ? ctx + j : -1;
        const size_t qo = (size_t)(row0 + j) * qstride + (size_t)(kvh * G + g) * D + 8 * (lane >> 4);
#pragma unroll
        for (int ks = 0; ks < KFR; ++ks) {
            uint4 v = valid ? *reinterpret_cast<const uint4 *>(q_h + qo + ks * 32) : make_uint4(0, 0, 0, 0);
            qf[i][ks] = *reinterpret_cast<f16x8 *>(&v);
        }
    }
    // This wave's copies of a tile: 1 KiB pieces of the K page and of the V page of one of the tile's two pages (head dim 64:
    // of the K or the V page), always at the same place inside the page.
    constexpr bool KV_WAVES = NLOAD == 1;                        // (head dim 64: waves 0-3 copy K, waves 4-7 V)
    const int seg0 = wave * 64 / UNITS_PER_SEG, odd = seg0 & 1;
    const uint32_t voff = (uint32_t)((wave * 64) % UNITS_PER_SEG + lane) * 16;
    const size_t page_stride = (size_t)Hkv * PAGE_B;
    const char *base0 = reinterpret_cast<const char *>(KV_WAVES && seg0 >= 2 ? vpool : kpool) + (size_t)kvh * PAGE_B;
    const char *base1 = reinterpret_cast<const char *>(vpool) + (size_t)kvh * PAGE_B;
    auto page_of = [&](int t) { return pt[min(2 * min(t, t_end - 1) + odd, last_page)]; };
    // (whole items are read by many workgroups side by side.  A split item's stream is read once and carries the hint: without
    // it the residual and the activations of the O projection behind it are pushed out of the last-level cache, 57 -> 66 us)
    auto issue = [&](uint32_t stage_off, int page) {
        const size_t o = (size_t)(uint32_t)page * page_stride;
        const uint32_t dst = lds_base + stage_off + wave * 1024;
        dma16_s(voff, base0 + o, dst, shared_stream);
        if (!KV_WAVES) dma16_s(voff, base1 + o, dst + NT * 16, shared_stream);
    };

    struct Scores { f32x4 v[RBW][2]; };
    struct Probs { f16x8 v[RBW]; };
    float m_run[RBW], l_run[RBW], mt[RBW];
    f32x4 acc[RBW][VDB];
    float M[RBW], den[RBW];      // whole items: the rows' running maximum and sum over the finished chunks
#pragma unroll
    for (int i = 0; i < RBW; ++i) {
        m_run[i] = -INFINITY; l_run[i] = 0.f; M[i] = -INFINITY; den[i] = 0.f;
#pragma unroll
        for (int db = 0; db < VDB; ++db) acc[i][db] = (f32x4){0.f, 0.f, 0.f, 0.f};
    }

    auto k_frag = [&](const unsigned char *cur, int pg, int ks) { return *reinterpret_cast<const f16x8 *>(cur + pg * PAGE_B + (ks * 64 + lane) * 16); };
    auto v_frag = [&](const unsigned char *cur, int db) {
        typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;
        typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
        typedef const volatile __attribute__((address_space(3))) u32x2 *lds_u32x2_ptr;
        const u32x2 lo = *(lds_u32x2_ptr)(cur + 2 * PAGE_B + (db * 64 + lane) * 8);
        const u32x2 hi = *(lds_u32x2_ptr)(cur + 3 * PAGE_B + (db * 64 + lane) * 8);
        const u32x4 vv = {lo[0], lo[1], hi[0], hi[1]};
        return *reinterpret_cast<const f16x8 *>(&vv);
    };
    auto tile_max = [&](const Scores &s, int i) {
        float x = fmaxf(s.v[i][0][0], s.v[i][1][0]);
#pragma unroll
        for (int r = 1; r < 4; ++r) x = fmaxf(x, fmaxf(s.v[i][0][r], s.v[i][1][r]));
        return x * scale_log2e;
    };
    auto scores = [&](const unsigned char *cur, Scores &s) {
#pragma unroll
        for (int i = 0; i < RBW; ++i) { s.v[i][0] = (f32x4){0.f, 0.f, 0.f, 0.f}; s.v[i][1] = (f32x4){0.f, 0.f, 0.f, 0.f}; }
#pragma unroll
        for (int ks = 0; ks < KFR; ++ks)
#pragma unroll
            for (int pg = 0; pg < 2; ++pg) {
                const f16x8 k = k_frag(cur, pg, ks);
#pragma unroll
                for (int i = 0; i < RBW; ++i) s.v[i][pg] = __builtin_amdgcn_mfma_f32_16x16x32_f16(k, qf[i][ks], s.v[i][pg], 0, 0, 0);
            }
    };
    auto weigh = [&](const unsigned char *cur, const Probs &p) {
#pragma unroll
        for (int db = 0; db < VDB; ++db) {
            const f16x8 vf = v_frag(cur, db);
#pragma unroll
            for (int i = 0; i < RBW; ++i) acc[i][db] = __builtin_amdgcn_mfma_f32_16x16x32_f16(vf, p.v[i], acc[i][db], 0, 0, 0);
        }
    };
    // the result of a finished chunk: normalised output rounded to binary16, folded into the row's running sums, which leave
    // as the finished row after the last chunk
    auto fold_chunk = [&](const float *m_c, const float *l_c, bool first, bool final) {
        int ln = lane;
        asm volatile("" : "+v"(ln));      // (addresses are computed here and not kept over the tile loop, which has no register left for them)
        float4 *const num_ws = fold + (((size_t)pm.b_prow[b] * Hkv + kvh) * 16 + wave * RBW) * (VDB * 64) + ln;
#pragma unroll
        for (int i = 0; i < RBW; ++i) {
            float l = l_c[i];
            l += __shfl_xor(l, 16);
            l += __shfl_xor(l, 32);
            const float inv = l > 0.f ? 1.f / l : 0.f;
            const bool seen = m_c[i] != -INFINITY;      // (a chunk a row cannot see leaves its sums alone)
            ChunkScale c = {1.f, 0.f};
            if (seen) c = chunk_fold(M[i], den[i], m_c[i], l);
            const int rr = (wave * RBW + i) * 16 + (ln & 15);
            const int t = row0 + rr / G, a = kvh * G + rr % G;
            const float invden = 1.f / den[i];
#pragma unroll
            for (int db = 0; db < VDB; ++db) {
                float4 *ws = num_ws + (i * VDB + db) * 64;
                float4 x = make_float4(0.f, 0.f, 0.f, 0.f);
                if (!first) x = *ws;
                const f32x4 o = acc[i][db] * inv;
                const float2 o01 = unpack_h2(pack_h2(o[0], o[1])), o23 = unpack_h2(pack_h2(o[2], o[3]));
                if (seen) x = make_float4(chunk_num(x.x, o01.x, c), chunk_num(x.y, o01.y, c), chunk_num(x.z, o23.x, c), chunk_num(x.w, o23.y, c));
                if (!final) *ws = x;
                else if (rr < R)
                    *reinterpret_cast<uint2 *>(out + frag_off(t, a * D + 16 * db + 4 * (ln >> 4), qstride)) =
                        make_uint2(rne_bf16(x.x * invden) | (rne_bf16(x.y * invden) << 16), rne_bf16(x.z * invden) | (rne_bf16(x.w * invden) << 16));
            }
        }
    };

    int first_pages[AHEAD];
#pragma unroll
    for (int s0 = 0; s0 < AHEAD; ++s0) first_pages[s0] = page_of(t_begin + s0);
#pragma unroll
    for (int s0 = 0; s0 < AHEAD; ++s0) issue(s0 * TILE_B, first_pages[s0]);
    int page = page_of(t_begin + AHEAD);
    Scores sa, sb;
    Probs pa, pb;
#pragma unroll
    for (int i = 0; i < RBW; ++i) pa.v[i] = pb.v[i] = (f16x8){0, 0, 0, 0, 0, 0, 0, 0};
    {
        constexpr int NEWER = (AHEAD - 1) * NLOAD;
        __builtin_amdgcn_s_waitcnt(0xF70 | (NEWER & 15) | ((NEWER >> 4) << 14));
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    }
    static_assert((NS & (NS - 1)) == 0, "the ring wraps with a mask");
    uint32_t o_fill = AHEAD * TILE_B;      // ring offset of tile t+AHEAD
    auto advance = [&]() {                 // tile t+1 visible to all waves; all waves are done with tile t-2 ...
        constexpr int NEWER = (AHEAD - 2) * NLOAD;
        __builtin_amdgcn_s_waitcnt(0xF70 | (NEWER & 15) | ((NEWER >> 4) << 14));
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };
    auto refill = [&](int t) {             // ... and its stage is filled again
        issue(o_fill, page);
        page = page_of(t + AHEAD + 1);
        o_fill = (o_fill + TILE_B) & (NS * TILE_B - 1);
    };
    if (wave * RBW >= nrb) {               // a wave without rows copies and keeps step
        for (int t = t_begin; t < t_end; ++t) { advance(); refill(t); }
        __builtin_amdgcn_s_waitcnt(0xF70);
        return;
    }
    scores(smem, sa);
#pragma unroll
    for (int i = 0; i < RBW; ++i) mt[i] = tile_max(sa, i);
    uint32_t o_prev = 0, o_cur = 0, o_next = TILE_B;      // ring offsets of tiles t-1 (t for the first tile: its weights are zero), t, t+1
    // first tile that is not plain: the first of a new chunk, or one that needs the causal mask
    const int t_mask = (ctx + 1) / DAS_ATTN_TILE;
    int t_chunk = t_begin + tiles_per_chunk, t_plain_end = min(t_chunk, t_mask);
    float thr[RBW], nms[RBW];      // m_run + 8; -(reference of the exponentials)
#pragma unroll
    for (int i = 0; i < RBW; ++i) { thr[i] = -INFINITY; nms[i] = 0.f; }
    constexpr int SLOTS = VDB + 2 * KFR, FRONT = 3, PER_SLOT = RBW * 8 / SLOTS;
    static_assert(RBW == 2 && SLOTS * PER_SLOT == RBW * 8 && SLOTS % 4 == 0 && SLOTS - FRONT - 2 * KFR >= 1, "slot plan of a tile step");
    auto slot_frag = [&](const unsigned char *kc, const unsigned char *vc, int q) {
        if (q >= FRONT && q < FRONT + 2 * KFR) return k_frag(kc, (q - FRONT) & 1, (q - FRONT) >> 1);
        return v_frag(vc, q < FRONT ? q : q - 2 * KFR);
    };
    f16x8 frag[4];
#pragma unroll
    for (int q = 0; q < 3; ++q) frag[q] = v_frag(smem, q);
    // one tile: s, m_run etc. of tile t; p = probabilities of tile t-1; s_next, p_new are produced
    auto step = [&](int t, Scores &s, const Probs &p, Scores &s_next, Probs &p_new) {
        advance();
        float m_old[RBW], l_old[RBW], alpha[RBW];
        bool new_chunk = false, rescale = false;
        if (t >= t_plain_end || __builtin_amdgcn_ballot_w64(mt[0] > thr[0] || mt[1] > thr[1]) != 0) {
            // a new chunk, the causal mask, the rare move of a row's reference (see attn_partial_kernel: same rules, same
            // arithmetic).  The sums of tile t-1 are still to be added: the accumulators are rescaled behind them.
            new_chunk = t == t_chunk;      // the chunk of tile t-1 is complete after this step
            if (new_chunk) {
                t_chunk += tiles_per_chunk;
                t_plain_end = min(t_chunk, t_mask);
            }
            const bool need_mask = t >= t_mask;
#pragma unroll
            for (int i = 0; i < RBW; ++i) {
                m_old[i] = m_run[i]; l_old[i] = l_run[i];
                if (new_chunk) { m_run[i] = -INFINITY; l_run[i] = 0.f; }
                if (need_mask) {
                    const int pbase = t * DAS_ATTN_TILE + 4 * (lane >> 4);
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        if (pbase + r > lim[i]) s.v[i][0][r] = -INFINITY;
                        if (pbase + 16 + r > lim[i]) s.v[i][1][r] = -INFINITY;
                    }
                }
                float x = tile_max(s, i);
                x = fmaxf(x, __shfl_xor(x, 16));
                x = fmaxf(x, __shfl_xor(x, 32));
                const float mn = (x > m_run[i] + 8.f) ? x : m_run[i];
                alpha[i] = exp2f(m_run[i] - ((mn == -INFINITY) ? 0.f : mn));
                rescale |= __any(m_run[i] != -INFINITY && alpha[i] != 1.f) != 0;
                l_run[i] *= alpha[i];
                m_run[i] = mn;
                thr[i] = mn + 8.f;
                nms[i] = mn == -INFINITY ? 0.f : -mn;
            }
        }
        const unsigned char *kc = smem + o_next, *vc = smem + o_prev, *vn = smem + o_cur;
        float ps[RBW], pv[RBW * 8];
        uint32_t hv[RBW][4];
#pragma unroll
        for (int i = 0; i < RBW; ++i) {
            s_next.v[i][0] = (f32x4){0.f, 0.f, 0.f, 0.f}; s_next.v[i][1] = (f32x4){0.f, 0.f, 0.f, 0.f};
        }
        // Slots of two MFMAs: a few of the weighted sum of tile t-1 (their V fragments were read before the barrier), the
        // scores of tile t+1, the rest of the weighted sum.  Each slot also reads the fragment that the slot three
        // places on needs and takes its share of the softmax of tile t; order pinned by scheduling barriers.
#pragma unroll
        for (int q = 0; q < SLOTS; ++q) {
            __builtin_amdgcn_sched_barrier(0);
            const f16x8 f = frag[q & 3];
            const bool qk = q >= FRONT && q < FRONT + 2 * KFR;
#pragma unroll
            for (int i = 0; i < RBW; ++i) {
                if (qk) {
                    const int ks = (q - FRONT) >> 1, pg = (q - FRONT) & 1;
                    s_next.v[i][pg] = __builtin_amdgcn_mfma_f32_16x16x32_f16(f, qf[i][ks], s_next.v[i][pg], 0, 0, 0);
                } else {
                    const int db = q < FRONT ? q : q - 2 * KFR;
                    acc[i][db] = __builtin_amdgcn_mfma_f32_16x16x32_f16(f, p.v[i], acc[i][db], 0, 0, 0);
                }
            }
            frag[(q + 3) & 3] = slot_frag(kc, q + 3 < SLOTS ? vc : vn, (q + 3) % SLOTS);
            if (q == 1) refill(t);
#pragma unroll
            for (int e = q * PER_SLOT; e < (q + 1) * PER_SLOT; ++e) {
                const int i = e >> 3, r = e & 7;
                pv[e] = __builtin_amdgcn_exp2f(__builtin_fmaf(s.v[i][r >> 2][r & 3], scale_log2e, nms[i]));
                asm volatile("" : "+v"(pv[e]));      // (keeps the softmax in its slots: it would sink below the branches that follow)
                // the sum and the packing trail by one element: v_exp's result is not there for the next instruction
                const int e1 = e - 1, fi = e1 >> 3, fr = e1 & 7;
                if (e > 0) {
                    if (fr == 0) ps[fi] = pv[e1];
                    else { ps[fi] += pv[e1]; asm volatile("" : "+v"(ps[fi])); }
                    if (fr & 1) { hv[fi][fr >> 1] = pack_h2(pv[e1 - 1], pv[e1]); asm volatile("" : "+v"(hv[fi][fr >> 1])); }
                }
            }
            if (q == SLOTS - 2 || q == SLOTS - 1) {
                const int i = q - (SLOTS - 2);
                mt[i] = tile_max(s_next, i);
                asm volatile("" : "+v"(mt[i]));
            }
        }
        __builtin_amdgcn_sched_barrier(0);
        ps[RBW - 1] += pv[RBW * 8 - 1];
        hv[RBW - 1][3] = pack_h2(pv[RBW * 8 - 2], pv[RBW * 8 - 1]);
#pragma unroll
        for (int i = 0; i < RBW; ++i) {
            l_run[i] += ps[i];
            p_new.v[i] = *reinterpret_cast<const f16x8 *>(hv[i]);
        }
        if (rescale) {
#pragma unroll
            for (int i = 0; i < RBW; ++i)
#pragma unroll
                for (int db = 0; db < VDB; ++db) acc[i][db] *= alpha[i];
        }
        if (new_chunk) {
            fold_chunk(m_old, l_old, t == tiles_per_chunk, false);
#pragma unroll
            for (int i = 0; i < RBW; ++i)
#pragma unroll
                for (int db = 0; db < VDB; ++db) acc[i][db] = (f32x4){0.f, 0.f, 0.f, 0.f};
        }
        o_prev = o_cur;
        o_cur = o_next;
        o_next = (o_next + TILE_B) & (NS * TILE_B - 1);
    };
    for (int t = t_begin;;) {
        step(t, sa, pa, sb, pb);
        if (++t == t_end) break;
        step(t, sb, pb, sa, pa);
        if (++t == t_end) { pb = pa; break; }
    }
    __builtin_amdgcn_s_waitcnt(0xF70);     // vmcnt(0): no copy may land in LDS after this workgroup is gone
    weigh(smem + o_prev, pb);

    if (whole) {
        fold_chunk(m_run, l_run, t_end <= tiles_per_chunk, true);
        return;
    }
    // one chunk of several: partial results for the merge, as attn_partial_kernel leaves them
#pragma unroll
    for (int i = 0; i < RBW; ++i) {
        float l = l_run[i];
        l += __shfl_xor(l, 16);
        l += __shfl_xor(l, 32);
        const int rb = wave * RBW + i;
        if (rb >= nrb) continue;
        const size_t id = ((size_t)pm.b_prow[b] + (size_t)chunk * nrb + rb) * Hkv + kvh;
        const float inv = l > 0.f ? 1.f / l : 0.f;
        if ((lane >> 4) == 0) *reinterpret_cast<float2 *>(part_ml + id * 32 + 2 * lane) = make_float2(m_run[i], l);
        uint4 *dst = reinterpret_cast<uint4 *>(part_o + id * (16 * D)) + lane;
#pragma unroll
        for (int q = 0; q < VDB / 2; ++q) {
            const f32x4 lo = acc[i][2 * q] * inv, hi = acc[i][2 * q + 1] * inv;
            dst[q * 64] = make_uint4(pack_h2(lo[0], lo[1]), pack_h2(lo[2], lo[3]), pack_h2(hi[0], hi[1]), pack_h2(hi[2], hi[3]));
        }
    }
}

template <int D>
static void launch_attn_cfg(const PassMeta &pm, const int *items, int n_items, const f16_t *q_h, const f16_t *kpool_layer,
                            const f16_t *vpool_layer, uint16_t *part_o, float *part_ml, bf16_t *out_frag, const DasDims &dm, float sc, hipStream_t st) {
    // 8 waves per workgroup: the 8 query-row blocks of a KV head are spread one per wave, two workgroups per CU, so that
    // MFMA, exp and LDS work of different waves overlap
    auto kern = attn_partial_kernel<D, DAS_ATTN_STAGES>;
    constexpr int LDS = DAS_ATTN_STAGES * 4 * DAS_PAGE * D * 2;
    static bool configured = false;
    if (!configured) {
        (void)hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, LDS);
        configured = true;
    }
    kern<<<dim3(n_items), dim3(512), LDS, st>>>(pm, items, q_h, kpool_layer, vpool_layer, part_o, part_ml, out_frag, dm.Hkv, dm.G, dm.Hq * dm.D, sc);
}
template <int D>
static void launch_attn_rows(const PassMeta &pm, const int *items, int n_items, const f16_t *q_h, const f16_t *kpool_layer,
                             const f16_t *vpool_layer, uint16_t *part_o, float *part_ml, float4 *fold, bf16_t *out_frag, const DasDims &dm, float sc, hipStream_t st) {
    auto kern = attn_rows_kernel<D>;
    constexpr int LDS = DAS_ATTN_ROWS_STAGES * 4 * DAS_PAGE * D * 2;
    static bool configured = false;
    if (!configured) {
        (void)hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, LDS);
        configured = true;
    }
    kern<<<dim3(n_items), dim3(512), LDS, st>>>(pm, items, q_h, kpool_layer, vpool_layer, part_o, part_ml, fold, out_frag, dm.Hkv, dm.G, dm.Hq * dm.D, sc);
}

void launch_attn(const PassMeta &pm, const int *items, int n_items, bool many_rows, const f16_t *q_h,
                 const f16_t *kpool_layer, const f16_t *vpool_layer, uint16_t *part_o, float *part_ml, float4 *fold, bf16_t *out_frag,
                 const DasDims &dm, hipStream_t st) {
    if (n_items <= 0) return;
    const float sc = 1.4426950408889634f / sqrtf((float)dm.D);
    if (many_rows) (dm.D == 128 ? launch_attn_rows<128> : launch_attn_rows<64>)(pm, items, n_items, q_h, kpool_layer, vpool_layer, part_o, part_ml, fold, out_frag, dm, sc, st);
    else (dm.D == 128 ? launch_attn_cfg<128> : launch_attn_cfg<64>)(pm, items, n_items, q_h, kpool_layer, vpool_layer, part_o, part_ml, out_frag, dm, sc, st);
}

// ---------------------------------------------------------------- merge of the chunk partials
// One workgroup per (sequence, 16-row block, KV head), one wave per pair of dim blocks: lane l holds row l%16 and dims
// 16*db + 4*(l/16) .. +3 of its two dim blocks, as the attention kernel left them.  A chunk contributes its
// normalised output with weight l * 2^(m - M); ascending chunk order, fp32; chunks a row cannot see carry
// m = -inf and are skipped.  Output: bf16, fragment order, K = Hq*D.
template <int D>
__global__ __launch_bounds__(64 * (D / 32)) void attn_merge_kernel(PassMeta pm, const uint16_t *__restrict__ part_o,
                                                        const float *__restrict__ part_ml, bf16_t *__restrict__ out,
                                                        int Hq, int Hkv, int G) {
    const int b = pm.mblk[2 * blockIdx.x], rb = pm.mblk[2 * blockIdx.x + 1];
    const int kvh = blockIdx.y, q = threadIdx.y, lane = threadIdx.x;     // this wave: dim blocks 2q and 2q+1
    const int n = pm.b_n[b];
    const int R = G * n, nrb = (R + 15) >> 4, nchunk = pm.b_nchunk[b];
    const int rr = rb * 16 + (lane & 15);
    float M = -INFINITY, den = 0.f;
    float num[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) num[e] = 0.f;
    const size_t id0 = ((size_t)pm.b_prow[b] + rb) * Hkv + kvh, idstep = (size_t)nrb * Hkv;
    auto load = [&](int c, float2 &ml, uint4 &v) {
        const size_t id = id0 + (size_t)c * idstep;
        ml = *reinterpret_cast<const float2 *>(part_ml + id * 32 + 2 * (lane & 15));
        v = (reinterpret_cast<const uint4 *>(part_o + id * (16 * D)) + q * 64)[lane];
    };
    // Four chunks in flight: the merge of a long sequence is one dependent chain of loads, and its partials come from
    // HBM (they were written past the caches), so the depth of this ring is what its duration follows.
    constexpr int PF = 4;
    float2 ml_q[PF];
    uint4 v_q[PF];
#pragma unroll
    for (int u = 0; u < PF; ++u)
        if (u < nchunk) load(u, ml_q[u], v_q[u]);
    for (int c0 = 0; c0 < nchunk; c0 += PF) {
#pragma unroll
        for (int u = 0; u < PF; ++u) {
            const int c = c0 + u;
            if (c >= nchunk) break;
            const float2 ml = ml_q[u];
            const uint4 v = v_q[u];
            if (c + PF < nchunk) load(c + PF, ml_q[u], v_q[u]);
            if (ml.x == -INFINITY) continue;
            const ChunkScale cs = chunk_fold(M, den, ml.x, ml.y);
            const float2 o0 = unpack_h2(v.x), o1 = unpack_h2(v.y), o2 = unpack_h2(v.z), o3 = unpack_h2(v.w);
            const float o[8] = {o0.x, o0.y, o1.x, o1.y, o2.x, o2.y, o3.x, o3.y};
#pragma unroll
            for (int e = 0; e < 8; ++e) num[e] = chunk_num(num[e], o[e], cs);
        }
    }
    if (rr >= R) return;
    const int j = rr / G, g = rr % G;
    const int t = pm.b_row0[b] + j, a = kvh * G + g;
    const float inv = 1.f / den;
    const int K = Hq * D;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        // four consecutive dims: they share one 8-element group of the fragment layout
        const uint32_t lo = rne_bf16(num[4 * h] * inv) | (rne_bf16(num[4 * h + 1] * inv) << 16);
        const uint32_t hi = rne_bf16(num[4 * h + 2] * inv) | (rne_bf16(num[4 * h + 3] * inv) << 16);
        *reinterpret_cast<uint2 *>(out + frag_off(t, a * D + 16 * (2 * q + h) + 4 * (lane >> 4), K)) = make_uint2(lo, hi);
    }
}

void launch_attn_merge(const PassMeta &pm, const uint16_t *part_o, const float *part_ml, bf16_t *out_frag,
                       const DasDims &dm, hipStream_t st) {
    if (pm.n_mblk <= 0) return;
    dim3 g(pm.n_mblk, dm.Hkv), blk(64, dm.D / 32);      // one wave per pair of dim blocks
    if (dm.D == 128) attn_merge_kernel<128><<<g, blk, 0, st>>>(pm, part_o, part_ml, out_frag, dm.Hq, dm.Hkv, dm.G);
    else attn_merge_kernel<64><<<g, blk, 0, st>>>(pm, part_o, part_ml, out_frag, dm.Hq, dm.Hkv, dm.G);
}
