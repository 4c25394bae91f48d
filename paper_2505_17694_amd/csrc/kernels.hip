// gfx950 kernels: partial attention computation (paper Alg. 2) over the scheduled
// task lists, and partial output reduction (Alg. 3) per query (Alg. 4).
//
// Partial attention.  One persistent workgroup per (slot, KV head) walks the
// slot's task list (256 threads in the narrow launch variant, 512 in the wide one).
// A task is a KV slice of a node together with the query rows of the requests
// below the node: rows = requests x heads of the GQA group, gathered straight from
// the query tensor into MFMA operand registers (the on-chip query assembly of
// Sec. 4.1).  Every K and V byte of the slice is fetched from HBM once per task and
// serves all rows.
//
// Arithmetic of one 32-token block, per wave: S^T = K Q^T (tokens x rows) on the
// matrix unit, K rows as the A operand, Q as the B operand.  The accumulator
// layout (a query row per lane column, several tokens per lane) is already the
// B-operand layout of the second product O^T = V^T P^T once the tokens a lane
// holds are taken as its k-slice, so P never moves between lanes; V is brought in
// with the matching token-to-lane map.  Softmax statistics stay in fp32, in log2
// units.
//
// Three task shapes share that arithmetic:
//  * "stream" (tasks of at most 16 rows, in both launch variants): 16 x 16 x 32
//    tiles; the waves of the workgroup take interleaved 32-token blocks of the
//    slice as one team, each with all rows; K and V go from HBM straight to
//    registers (no LDS in the loop; V becomes an A operand by an 8x8 16-bit
//    transpose inside each lane, v_perm_b32); the waves' states are merged through
//    LDS at the end.  Runs of short tasks are handed out one wave each instead.
//  * "dense" (tasks of 17..256 rows, wide variant): 32 x 32 x 16 tiles; eight waves
//    split the rows (32 each) and walk the slice together; blocks are copied HBM ->
//    LDS asynchronously into a ring of 16 KB slots (five blocks in flight, four with two-block intervals)
//    and read by all waves, V through transposing LDS reads (ds_read_b64_tr_b16).
//    Long slices under at most 128 rows put two waves on each row group, on
//    alternate blocks.
//  * "tile" (64 and 256 channels): sibling row tiles of one slice packed into one
//    task of up to 256 (128) rows; 16 x 16 x 32 tiles, blocks shared through LDS.
//
// K and V slices that a single task reads, in plans that read little twice, are
// loaded with the streaming (nontemporal) hint; the plan marks those tasks.
#include <hip/hip_runtime.h>

#include <mutex>
#include <type_traits>

#include "kernels.hpp"

namespace codec {
namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(8))) _Float16 f16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) unsigned int u32x4;

constexpr int kHeadDim = 128;       // the dense path; the stream path and the reduction take the head
                                    // dimension D (64, 128 or 256) as a template parameter
constexpr int kNarrowWaves = 4;     // stream-only kernel variant: 4 waves, two workgroups per CU
constexpr int kWideWaves = 8;       // all task shapes: 8 waves (two per SIMD), one workgroup per CU
// Forms of the attention kernel: stream tasks only; all task shapes (dense, or tile with 64 and 256 channels);
// stream tasks whose rows go out finished (store_finished).
enum { kFormNarrow = 0, kFormWide = 1, kFormFinish = 2 };
// Waves of a workgroup: with 256 channels a wave needs a SIMD's registers for itself
constexpr int kernel_waves(int form, int d) { return form == kFormWide && d <= 128 ? kWideWaves : kNarrowWaves; }
// Row tiles of the stream path in the narrow variant: one tile of 16 rows, or two (32 rows) with 64
// channels, where the accumulators of a second tile still fit the registers.
constexpr int stream_tiles(int d) { return d == 64 ? 2 : 1; }
constexpr int kMergeWaves = 2;      // reduction kernel (workgroups of two waves: measured against one and four, the
                                    // launch that follows a reduction starts up to 3 us sooner)
// Channel tiles of 16 that a stream task accumulates: 8 per 128 channels (with 64 channels half of each
// tile's rows are idle, see BlockRegs).
constexpr int channel_tiles(int d) { return d <= 128 ? 8 : d / 16; }
// LDS for merging the waves' states at the end of a stream task: W/2 states of NT row tiles
constexpr int merge_bytes(int waves, int nt, int d) { return (waves / 2) * (nt * channel_tiles(d) * 64 * 4 + nt * 64 * 2) * 4; }
// LDS of a wave that runs a task on its own: its 16 partial rows, fp32, 16 bytes between rows (the 16
// lanes of a row group then cover all banks).  256 channels: none (the rows go out as the lanes hold them).
constexpr int solo_stage_pitch(int d) { return d * 4 + 16; }
constexpr int solo_stage_bytes(int d) { return d <= 128 ? 16 * solo_stage_pitch(d) : 0; }

template <int DT>
__device__ __forceinline__ f32x4 mfma16(u32x4 a, u32x4 b, f32x4 c)
{
    if constexpr (DT == CODEC_DTYPE_FP16)
        return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, a),
                                                       __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
    else
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a),
                                                        __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

// Two fp32 values -> one dword of two 16-bit values (round to nearest even), lo in bits 0..15.
template <int DT>
__device__ __forceinline__ unsigned int pack2(float lo, float hi)
{
    if constexpr (DT == CODEC_DTYPE_FP16) {
        typedef __attribute__((ext_vector_type(2))) _Float16 h2;
        h2 v = {(_Float16)lo, (_Float16)hi};
        return __builtin_bit_cast(unsigned int, v);
    } else {
        typedef __attribute__((ext_vector_type(2))) __bf16 b2;
        b2 v = {(__bf16)lo, (__bf16)hi};
        return __builtin_bit_cast(unsigned int, v);
    }
}

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// acc + lo + hi of a dword of two 16-bit values (a two-element dot product with ones, exact products,
// fp32 sum).  Row sums are taken over the probabilities as rounded for the second product: the
// normaliser then matches the numerator, and a pair costs one instruction.
template <int DT>
__device__ __forceinline__ float add_pair(unsigned int packed, float acc)
{
    if constexpr (DT == CODEC_DTYPE_FP16) {
        typedef __attribute__((ext_vector_type(2))) _Float16 h2;
        const h2 ones = {(_Float16)1.0f, (_Float16)1.0f};
        return __builtin_amdgcn_fdot2(__builtin_bit_cast(h2, packed), ones, acc, false);
    } else {
        typedef __attribute__((ext_vector_type(2))) __bf16 b2;
        const b2 ones = {(__bf16)1.0f, (__bf16)1.0f};
        return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(b2, packed), ones, acc, false);
    }
}

__device__ __forceinline__ u32x4 ld16(const char *p) { return *reinterpret_cast<const u32x4 *>(p); }
// The same load with the streaming hint (the `nt` bit).  K and V slices that one task alone reads are
// fetched this way: bytes on their way through then do not displace each other, nor the slices that
// several tasks read, in the caches.  Slices with several readers keep plain loads: their re-reads live
// on cache hits.
__device__ __forceinline__ u32x4 ld16_once(const char *p)
{
    return __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(p));
}

// Accesses that are coherent across the whole device without cache maintenance: relaxed atomic
// accesses at device scope go past the caches that are not coherent at that scope (the `sc1` forms of
// the load and store instructions).  The single-launch mode moves partial results between workgroups
// of one launch through them; everywhere else partial results cross a kernel boundary and use plain
// accesses.
__device__ __forceinline__ void st8_device(float *p, float a, float b)
{
    const float2 v = {a, b};
    __hip_atomic_store(reinterpret_cast<unsigned long long *>(p), __builtin_bit_cast(unsigned long long, v),
                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ float2 ld8_device(const float *p)
{
    const unsigned long long v = __hip_atomic_load(reinterpret_cast<const unsigned long long *>(p),
                                                   __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return __builtin_bit_cast(float2, v);
}
// How the partial rows of a task are stored.
//  kRowsPlain     read by a later launch; the lines stay in the L2 of the XCD until something pushes them out
//  kRowsThrough   the same, written through at once (the `sc1` form): rows of dense and tile tasks in plans that
//                 have many (kEarlyThroughBytes, last_rows_through)
//  kRowsCoherent  read by other workgroups of this launch (single-launch mode)
// Lines that wait in L2 for their write-back are pushed out by the K and V that stream through it, a few at a
// time, and HBM turns around between reads and writes for each.  Rows written through are not in L2, though, when
// the reduction reads them.  Which of the two costs more depends on how many rows the plan has; both sides are
// measured at the rules.  Stream tasks keep plain stores.  Rows of a wave that ran a task on its own, 1 KB of
// consecutive memory per instruction: written through, 117 drawn plans of 64 and 128 channels take 1.008 of the
// time, the worst 1.096.  Rows of a team, 16 bytes of each of up to 64 lines per instruction, which only L2 puts
// together: 150 plans 1.023, the worst 1.155.
enum RowStore { kRowsPlain, kRowsThrough, kRowsCoherent };
// Rows behind a buffer descriptor (base the same for the wave, `bytes` long; stores behind its end are dropped):
// the compiler has no other 16-byte store that is written through, and it keeps the distance that this target wants
// between a store of this width and the next write to its data registers (inline assembly would not).  Dense tasks
// store plain rows like that as well, as no row then needs a branch: 92 drawn plans whose dense rows stay plain take
// 0.993 of the time with pointers, the best 0.949, the worst 1.009.
typedef __amdgpu_buffer_rsrc_t Rows;
__device__ __forceinline__ Rows rows_at(float *base, int bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(base, 0, bytes, 0x00027000);   // word 3: 32-bit raw data
}
template <RowStore HOW>
__device__ __forceinline__ void st16_rows(Rows rows, int offset, f32x4 v)
{
    static_assert(HOW != kRowsCoherent, "two 8-byte stores: st16_partial");
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), rows, offset, 0, HOW == kRowsThrough ? 16 /* sc1 */ : 0);
}
// The same through a pointer: plain or coherent.
template <RowStore HOW>
__device__ __forceinline__ void st16_partial(float *p, f32x4 v)
{
    static_assert(HOW != kRowsThrough, "st16_rows");
    if constexpr (HOW == kRowsCoherent) {
        st8_device(p, v[0], v[1]);
        st8_device(p + 2, v[2], v[3]);
    } else {
        *reinterpret_cast<f32x4 *>(p) = v;
    }
}
template <RowStore HOW>
__device__ __forceinline__ void st8_partial(float *p, float a, float b)
{
    if constexpr (HOW != kRowsPlain) st8_device(p, a, b);
    else                             *reinterpret_cast<float2 *>(p) = float2{a, b};
}
// body(integral constant): one branch around all stores of a task, whose LDS reads then travel together
template <class Body>
__device__ __forceinline__ void with_row_store(RowStore how, Body body)
{
    if (how == kRowsCoherent)     body(std::integral_constant<RowStore, kRowsCoherent>{});
    else if (how == kRowsThrough) body(std::integral_constant<RowStore, kRowsThrough>{});
    else                          body(std::integral_constant<RowStore, kRowsPlain>{});
}

// The lane index as a value the optimiser cannot trace back to the thread id.  Each task path derives
// its lane constants (operand addresses, row and channel positions) from it, which keeps them inside
// the path: hoisted out of the task loop they would stay live across all paths and cost the dense
// path, which needs nearly every register, a dozen spills.
__device__ __forceinline__ int opaque_lane()
{
    int lane = threadIdx.x & 63;
    asm volatile("" : "+v"(lane));
    return lane;
}

// Slice being processed: wave-uniform values only, so that addresses are SGPR base + 32-bit lane offset.
struct SliceCtx {
    const char *k_head;         // K pool + KV-head offset
    const char *v_head;
    const int32_t *pages;       // page ids of the slice, first page first
    uint32_t page_bytes;
    uint32_t token_bytes;
    int32_t kv_len;
    int32_t page_shift;         // log2(page_size)
    int32_t page_mask;
    int32_t read_once;          // no other task reads this slice
};

// Page ids are read through the scalar data path (s_load_dword, a read-only access): a vector load
// would sit in the same in-order return queue as the K/V traffic, and waiting for it would drain every
// prefetched block.  The page table does not change while a launch runs, so the load goes through a
// pointer to the constant address space; with a wave-uniform index the compiler then picks the scalar
// path and places the wait at the first use, which lets callers load an id a whole step ahead.
__device__ __forceinline__ int uniform_load(const int32_t *p, int index)
{
    typedef const int32_t __attribute__((address_space(4))) *const_i32_ptr;
    return ((const_i32_ptr)(uintptr_t)p)[uint32_t(__builtin_amdgcn_readfirstlane(index))];
}

// Byte offset of a page slot: page id `pg`, token slot `slot` inside the page (wave-uniform).
__device__ __forceinline__ int64_t page_offset(const SliceCtx &c, int pg, int slot)
{
    return int64_t(uint64_t(uint32_t(pg)) * c.page_bytes + uint64_t(uint32_t(slot) * c.token_bytes));
}

// K and V registers of one 32-token block (stream path), head dimension D.
template <int D>
struct BlockRegs {
    static constexpr int KS = D / 32;                   // k-steps of the scores
    static constexpr int VU = D <= 128 ? 1 : D / 128;   // 16-byte V pieces per token and lane
    u32x4 k[2][KS];     // [tile][k-step]: token = tile*16 + lane%16, channels 32*ks + 8*(lane/16)..+7
    u32x4 v[8][VU];     // [e][u]: token = (e/4)*16 + 4*(lane/16) + e%4, channels 128*u + 8*(lane%16)..+7;
                        // D = 64: lanes 8..15 repeat the pieces of lanes 0..7 (their rows of the
                        // accumulated tiles stand for channels that do not exist and are never stored)
    uint32_t visible;   // masked tasks: bit t = the lane's row sees token t of the block
};

// Issue the loads of block `tb`.  A tile that starts beyond the slice is not loaded (its registers are
// cleared; its scores are masked later): no address leaves the slice's pages, and the sixteen load
// instructions of a block, each of which holds a place in the CU's queue of memory instructions in
// flight whatever it fetches, become eight for the last tile of a ragged slice and for one-token
// nodes.  ONCE: with the streaming hint.
template <bool ONCE, int D>
__device__ __forceinline__ void load_block(const SliceCtx &c, int tb, uint32_t koff, uint32_t voff, BlockRegs<D> &r,
                                           bool masked, const uint32_t *mask_row)
{
    // the word of the row's visibility mask for this block (a slice with masks starts at token 0 of its
    // node; a row without a mask sees everything)
    if (masked) r.visible = mask_row ? mask_row[tb] : 0xFFFFFFFFu;
    int tok[2], pg[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        tok[j] = tb * 32 + j * 16;
        pg[j] = tok[j] < c.kv_len ? uniform_load(c.pages, tok[j] >> c.page_shift) : 0;
    }
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        if (j == 1 && tok[j] >= c.kv_len) {     // wave-uniform: the slice ends inside the first tile
#pragma unroll
            for (int ks = 0; ks < BlockRegs<D>::KS; ++ks) r.k[j][ks] = u32x4{0u, 0u, 0u, 0u};
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int u = 0; u < BlockRegs<D>::VU; ++u) r.v[j * 4 + e][u] = u32x4{0u, 0u, 0u, 0u};
            continue;
        }
        const int64_t off = page_offset(c, pg[j], tok[j] & c.page_mask);
        const char *kt = c.k_head + off;
        const char *vt = c.v_head + off;
#pragma unroll
        for (int ks = 0; ks < BlockRegs<D>::KS; ++ks)
            r.k[j][ks] = ONCE ? ld16_once(kt + koff + ks * 64) : ld16(kt + koff + ks * 64);
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int u = 0; u < BlockRegs<D>::VU; ++u) {
                const char *p = vt + size_t(e) * c.token_bytes + voff + u * 256;
                r.v[j * 4 + e][u] = ONCE ? ld16_once(p) : ld16(p);
            }
    }
}

// Initial reference of a row.  Finite, so that a block in which a row sees no token at all (every score
// -inf under its visibility mask) yields exp2(-inf - m) = 0 and not exp2(-inf + inf); so low that the
// first finite score raises the reference and wipes (multiplies by exp2 of -1e30) whatever it scaled.
constexpr float kNoReference = -1e30f;

template <int NT, int D, int CTILES = channel_tiles(D)>
struct RowState {
    static constexpr int CT = CTILES;
    f32x4 o[NT][CT];    // [row tile][dt]: row = 16*nt + lane%16; channel of component e is
                        // 128*(dt/8) + 32*(lane/16) + 8*e + dt%8 (tile path: 16*dt + 4*(lane/16) + e)
    float m[NT];        // reference subtracted before exponentiation, log2 units (same in the 4 lanes
                        // that share a row); kNoReference until the row has seen a score above -inf
    float l[NT];        // the lane's share of the row sum; the row sum after finish()

    __device__ __forceinline__ void clear()
    {
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            m[nt] = kNoReference;
            l[nt] = 0.f;
#pragma unroll
            for (int dt = 0; dt < CT; ++dt) o[nt][dt] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
    }
    // each lane summed its own 8 tokens per block: the four lanes of a row are added up
    __device__ __forceinline__ void finish()
    {
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            l[nt] += __shfl_xor(l[nt], 16);
            l[nt] += __shfl_xor(l[nt], 32);
        }
    }
};

// ---- one 32-token block of online softmax, in pieces so that callers can interleave them ---------
//
// The reference m of a row is allowed to lag behind the row's true running maximum by up to kLag
// (log2 units): softmax is invariant to the reference, and with the lag bounded every exponential
// stays <= 2^kLag, well inside fp16/bf16 and fp32 range.  A block therefore only needs each lane's own
// maximum over its 8 scores and one wave-wide vote; the cross-lane maximum and the rescaling of the
// accumulators run only when some row's scores outgrow the lag (always on a wave's first block,
// rarely afterwards).
constexpr float kLag = 8.f;

// Scores of tokens past `valid` become -inf (ragged last block of a slice).
template <int NT>
__device__ __forceinline__ void mask_scores(f32x4 (&s)[2][NT], int valid, int grp)
{
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const bool dead = j * 16 + grp * 4 + e >= valid;
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) s[j][nt][e] = dead ? -INFINITY : s[j][nt][e];
        }
}

// Scores of tokens the row does not see become -inf (visibility mask, Sec. 4.1): bit t of `visible` is
// token t of the block.
template <int NT>
__device__ __forceinline__ void mask_invisible(f32x4 (&s)[2][NT], uint32_t visible, int grp)
{
    static_assert(NT == 1, "one mask word per lane: one row per lane");
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const bool seen = (visible >> (j * 16 + grp * 4 + e)) & 1u;
            s[j][0][e] = seen ? s[j][0][e] : -INFINITY;
        }
}

// V rows of tokens past `valid` count as zero (their memory may hold anything).
template <int VU>
__device__ __forceinline__ void mask_values(u32x4 (&v)[8][VU], int valid, int grp)
{
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const bool dead = (e >> 2) * 16 + grp * 4 + (e & 3) >= valid;
#pragma unroll
        for (int u = 0; u < VU; ++u)
#pragma unroll
            for (int c = 0; c < 4; ++c) v[e][u][c] = dead ? 0u : v[e][u][c];
    }
}

// Each lane's maximum over its 8 scores per row tile, in log2 units.
template <int NT>
__device__ __forceinline__ void lane_maxima(const f32x4 (&s)[2][NT], float scale_log2e, float (&lm)[NT])
{
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        float a = fmaxf(fmaxf(s[0][nt][0], s[0][nt][1]), s[0][nt][2]);
        a = fmaxf(fmaxf(a, s[0][nt][3]), s[1][nt][0]);
        a = fmaxf(fmaxf(a, s[1][nt][1]), s[1][nt][2]);
        lm[nt] = fmaxf(a, s[1][nt][3]) * scale_log2e;
    }
}

template <int NT, class State>
__device__ __forceinline__ bool outgrown(const float (&lm)[NT], const State &st)
{
    bool any = false;
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) any |= lm[nt] > st.m[nt] + kLag;
    return any;
}

// Move every row's reference up to its true running maximum and rescale its accumulators.
template <int NT, class State>
__device__ __forceinline__ void raise_reference(const float (&lm)[NT], State &st)
{
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        float mx = lm[nt];
        mx = fmaxf(mx, __shfl_xor(mx, 16));
        mx = fmaxf(mx, __shfl_xor(mx, 32));
        const float m_new = fmaxf(st.m[nt], mx);
        const float alpha = fast_exp2(st.m[nt] - m_new);       // 0 on the first block (m = -inf)
        st.l[nt] *= alpha;
#pragma unroll
        for (int dt = 0; dt < State::CT; ++dt) st.o[nt][dt] *= alpha;
        st.m[nt] = m_new;
    }
}

// P = exp2(scale * S - m), rounded to 16 bits in B-operand layout; the lane adds its 8 exponentials to
// its share of the row sum.
template <int DT, int NT, class State>
__device__ __forceinline__ void probabilities(const f32x4 (&s)[2][NT], State &st,
                                              float scale_log2e, u32x4 (&pb)[NT])
{
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        float p[2][4];
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e)
                p[j][e] = fast_exp2(__builtin_fmaf(s[j][nt][e], scale_log2e, -st.m[nt]));
        pb[nt] = u32x4{pack2<DT>(p[0][0], p[0][1]), pack2<DT>(p[0][2], p[0][3]),
                       pack2<DT>(p[1][0], p[1][1]), pack2<DT>(p[1][2], p[1][3])};
#pragma unroll
        for (int d = 0; d < 4; ++d) st.l[nt] = add_pair<DT>(pb[nt][d], st.l[nt]);
    }
}

// O^T += V^T P^T for the channel tiles dt = 8*U + 4*HALF .. +3.  `vh[e]` holds dwords 2*HALF and
// 2*HALF+1 (channels 4*HALF .. 4*HALF+3 of the lane's 8) of token e's V row piece U; the 16-bit
// transpose inside each lane turns them into A operands.
template <int DT, int NT, int D, int U, int HALF>
__device__ __forceinline__ void accumulate_half(const unsigned int (&vh)[8][2], const u32x4 (&pb)[NT],
                                                RowState<NT, D> &st)
{
#pragma unroll
    for (int d = 0; d < 4; ++d) {
        const int dt = 8 * U + 4 * HALF + d;
        const unsigned int sel = (d & 1) ? 0x07060302u : 0x05040100u;
        u32x4 va;
#pragma unroll
        for (int k = 0; k < 4; ++k)
            va[k] = __builtin_amdgcn_perm(vh[2 * k + 1][d >> 1], vh[2 * k][d >> 1], sel);
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) st.o[nt][dt] = mfma16<DT>(va, pb[nt], st.o[nt][dt]);
    }
}

// Same for V row piece U of every token (16 bytes each) held in registers.
template <int DT, int NT, int D, int U>
__device__ __forceinline__ void accumulate_piece(const u32x4 (&v)[8][BlockRegs<D>::VU], const u32x4 (&pb)[NT],
                                                 RowState<NT, D> &st)
{
    unsigned int lo[8][2], hi[8][2];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        lo[e][0] = v[e][U][0]; lo[e][1] = v[e][U][1];
        hi[e][0] = v[e][U][2]; hi[e][1] = v[e][U][3];
    }
    accumulate_half<DT, NT, D, U, 0>(lo, pb, st);
    accumulate_half<DT, NT, D, U, 1>(hi, pb, st);
}
template <int DT, int NT, int D>
__device__ __forceinline__ void accumulate(const u32x4 (&v)[8][BlockRegs<D>::VU], const u32x4 (&pb)[NT],
                                           RowState<NT, D> &st)
{
    accumulate_piece<DT, NT, D, 0>(v, pb, st);
    if constexpr (BlockRegs<D>::VU > 1) accumulate_piece<DT, NT, D, 1>(v, pb, st);
    static_assert(BlockRegs<D>::VU <= 2, "head dimensions up to 256");
}

// Gather the wave's query rows (task rows row0 .. row0 + 16*NT) into B-operand registers.
template <int NT, int D>
__device__ __forceinline__ void gather_q(const PacParams &P, const DevTask &t, int head, int row0, int rows,
                                         int l16, int grp, u32x4 (&qb)[NT][D / 32])
{
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        const int row = row0 + nt * 16 + l16;
        const bool live = row < rows;
        const int qi = live ? row / P.group : 0;
        const int hj = live ? row - qi * P.group : 0;
        const int req = t.single_req >= 0 ? t.single_req : P.node_q[t.q_off + qi];
        const char *qp = static_cast<const char *>(P.q)
                         + (int64_t(req) * P.h_q + int64_t(head) * P.group + hj) * (D * 2) + grp * 16;
#pragma unroll
        for (int ks = 0; ks < D / 32; ++ks) qb[nt][ks] = live ? ld16(qp + ks * 64) : u32x4{0u, 0u, 0u, 0u};
    }
}

// The same for a wave that ran the task on its own, through its staging area in LDS.  In registers a
// lane holds 16-byte pieces of one row, so a store instruction of the wave would carry 16 bytes for each
// of 16 lines, and a task of `group` rows would take eight of them however few its rows; every
// vector-memory instruction takes a place in the CU's queue of instructions in flight, and a short task
// has few to spare.  Staged, the task's rows (they are neighbours in the partial array) go out 1 KB of
// consecutive memory per instruction: two instructions for four rows of 128 channels.
template <RowStore HOW, int D>
__device__ __forceinline__ void store_partial_staged(const PacParams &P, const DevTask &t, int head, int rows,
                                                     int lane, const RowState<1, D> &st, char *stage)
{
    static_assert(D <= 128, "staging area is sized for up to 128 channels");
    constexpr int PITCH = solo_stage_pitch(D), ROW = D * 4;
    const int l16 = lane & 15, grp = lane >> 4;
    char *put = stage + l16 * PITCH + grp * 128;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        if (grp * 32 + e * 8 >= D) continue;            // channels the head does not have
        const f32x4 lo = {st.o[0][0][e], st.o[0][1][e], st.o[0][2][e], st.o[0][3][e]};
        const f32x4 hi = {st.o[0][4][e], st.o[0][5][e], st.o[0][6][e], st.o[0][7][e]};
        *reinterpret_cast<f32x4 *>(put + e * 32) = lo;
        *reinterpret_cast<f32x4 *>(put + e * 32 + 16) = hi;
    }
    const int64_t prow = int64_t(head) * P.part_rows + t.part_row_base;
    if (grp == 0 && l16 < rows) st8_partial<HOW>(P.part_ml + (prow + l16) * 2, st.m[0], st.l[0]);
    __builtin_amdgcn_wave_barrier();                    // LDS serves a wave's accesses in order: no wait needed
    float *po = P.part_o + prow * D;
    const int bytes = rows * ROW;
#pragma unroll
    for (int i = 0; i < 16 * ROW / 1024; ++i) {
        if (i * 1024 >= bytes) break;                   // wave-uniform
        const int off = i * 1024 + lane * 16;
        if (off < bytes) {
            const f32x4 x = *reinterpret_cast<const f32x4 *>(stage + (off / ROW) * PITCH + off % ROW);
            st16_partial<HOW>(po + off / 4, x);
        }
    }
    __builtin_amdgcn_wave_barrier();                    // the area is read before the wave's next task writes it
}

// Write one wave's rows of the partial result: unnormalised output, (reference, sum) per row.
template <RowStore HOW, int NT, int D>
__device__ __forceinline__ void store_partial(const PacParams &P, const DevTask &t, int head, int row0, int rows,
                                              int l16, int grp, const RowState<NT, D> &st)
{
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        const int row = row0 + nt * 16 + l16;
        if (row < rows) {
            const int64_t prow = int64_t(head) * P.part_rows + t.part_row_base + row;
            float *po = P.part_o + prow * D + grp * 32;
#pragma unroll
            for (int u = 0; u < BlockRegs<D>::VU; ++u)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    if (D < 128 && grp * 32 + e * 8 >= D) continue;     // channels the head does not have
                    const f32x4 lo = {st.o[nt][8 * u + 0][e], st.o[nt][8 * u + 1][e], st.o[nt][8 * u + 2][e], st.o[nt][8 * u + 3][e]};
                    const f32x4 hi = {st.o[nt][8 * u + 4][e], st.o[nt][8 * u + 5][e], st.o[nt][8 * u + 6][e], st.o[nt][8 * u + 7][e]};
                    st16_partial<HOW>(po + u * 128 + e * 8, lo);
                    st16_partial<HOW>(po + u * 128 + e * 8 + 4, hi);
                }
            if (grp == 0) st8_partial<HOW>(P.part_ml + prow * 2, st.m[nt], st.l[nt]);
        }
    }
}

// The rows of a task whose requests have no other partial result, finished: normalised and rounded as the
// reduction does it (its fold of one partial multiplies by 1), straight into the output.  Plans in which
// every request has a single partial, unshared contexts that the plan does not divide, save the partial
// rows, the reduction launch and the gap in front of it: 256 unshared contexts of 100 .. 4000 tokens, 28 / 4
// heads, 207.2 -> 200.7 us per step.
template <int DT, int D>
__device__ __forceinline__ void store_finished(const PacParams &P, const DevTask &t, int head, int rows, int l16, int grp,
                                               const RowState<1, D> &st)
{
    if (l16 >= rows) return;
    const int qi = l16 / P.group, hj = l16 - qi * P.group;
    const int req = t.single_req >= 0 ? t.single_req : P.node_q[t.q_off + qi];
    const float inv = 1.f / st.l[0];
    char *out = static_cast<char *>(P.merge.out) + ((int64_t(req) * P.h_q + int64_t(head) * P.group + hj) * D + grp * 32) * 2;
#pragma unroll
    for (int u = 0; u < BlockRegs<D>::VU; ++u)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            if (D < 128 && grp * 32 + e * 8 >= D) continue;             // channels the head does not have
            u32x4 x;
#pragma unroll
            for (int d = 0; d < 4; ++d) x[d] = pack2<DT>(st.o[0][8 * u + 2 * d][e] * inv, st.o[0][8 * u + 2 * d + 1][e] * inv);
            *reinterpret_cast<u32x4 *>(out + u * 256 + e * 16) = x;
        }
}

__device__ __forceinline__ SliceCtx make_ctx(const PacParams &P, const DevTask &t, int head)
{
    SliceCtx c;
    c.k_head = static_cast<const char *>(P.k_pages) + int64_t(head) * P.head_stride * 2;
    c.v_head = static_cast<const char *>(P.v_pages) + int64_t(head) * P.head_stride * 2;
    c.pages = P.page_ids + t.page_off;
    c.page_bytes = uint32_t(P.page_stride * 2);
    c.token_bytes = uint32_t(P.token_stride * 2);
    c.kv_len = t.kv_len;
    c.page_shift = P.page_shift;
    c.page_mask = (1 << P.page_shift) - 1;
    c.read_once = t.flags & kTaskReadOnce;
    return c;
}

// exp2(a - m) with the convention that the side holding the maximum weighs exactly 1
// (keeps "-inf minus -inf" of a wave that saw no token out of the arithmetic).
__device__ __forceinline__ float weight(float a, float m) { return a == m ? 1.f : fast_exp2(a - m); }

// ---- stream path: rows <= 16*NT (NT = 2 for 17 .. 32 rows of 64 channels, else 1), a team of W waves splits the tokens
// `wave` is the wave's index in its team.  A team of one wave (W = 1) uses no LDS and no barrier, so
// several such waves may work on different tasks at the same time.
// FINISH: the task's rows go out finished (store_finished).
template <int DT, bool ONCE, int NT, int W, int D, bool FINISH = false>
__device__ __forceinline__ void run_stream(const PacParams &P, const DevTask &t, int head, char *lds_raw, int wave,
                                           char *stage = nullptr)   // W = 1, up to 128 channels: the wave's staging area
{
    constexpr int KS = D / 32, CT = channel_tiles(D);
    const int lane = opaque_lane();
    const int l16 = lane & 15, grp = lane >> 4;
    const int rows = t.n_req * P.group;

    u32x4 qb[NT][KS];
    gather_q<NT, D>(P, t, head, 0, rows, l16, grp, qb);
    const SliceCtx c = make_ctx(P, t, head);
    const uint32_t koff = uint32_t(l16) * c.token_bytes + grp * 16;
    const uint32_t voff = uint32_t(grp * 4) * c.token_bytes + (D < 128 ? (l16 & (D / 8 - 1)) : l16) * 16;

    // visibility mask of the lane's row, if the task has any (masked tasks hold at most 16 rows and are
    // never slices of a node: block tb of the task is word tb of the mask)
    const bool masked = (t.flags & kTaskMasked) != 0;
    const uint32_t *mask_row = nullptr;
    if (masked && l16 < rows) {
        const int off = P.nodeq_mask[t.q_off + l16 / P.group];
        if (off >= 0) mask_row = P.mask_words + off;
    }

    RowState<NT, D> st;
    st.clear();

    auto compute = [&](int tb, BlockRegs<D> &r) {
        f32x4 s[2][NT];
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) acc = mfma16<DT>(r.k[j][ks], qb[nt][ks], acc);
                s[j][nt] = acc;
            }
        const int valid = c.kv_len - tb * 32;
        if (valid < 32) {
            mask_scores<NT>(s, valid, grp);
            mask_values<BlockRegs<D>::VU>(r.v, valid, grp);
        }
        if constexpr (NT == 1) {            // tasks with masks are planned as tiles of at most 16 rows
            if (masked) mask_invisible<NT>(s, r.visible, grp);
        }
        float lm[NT];
        lane_maxima<NT>(s, P.scale_log2e, lm);
        if (__any(outgrown<NT>(lm, st))) raise_reference<NT>(lm, st);
        u32x4 pb[NT];
        probabilities<DT, NT>(s, st, P.scale_log2e, pb);
        accumulate<DT, NT, D>(r.v, pb, st);
    };

    // software pipeline: the loads of the wave's next block are in flight while it computes this one
    const int nblk = (t.kv_len + 31) >> 5;
    BlockRegs<D> ra, rb;
    int tb = wave;
    if (tb < nblk) load_block<ONCE, D>(c, tb, koff, voff, ra, masked, mask_row);
    while (tb < nblk) {
        int nb = tb + W;
        if (nb < nblk) load_block<ONCE, D>(c, nb, koff, voff, rb, masked, mask_row);
        compute(tb, ra);
        tb = nb;
        if (tb >= nblk) break;
        nb = tb + W;
        if (nb < nblk) load_block<ONCE, D>(c, nb, koff, voff, ra, masked, mask_row);
        compute(tb, rb);
        tb = nb;
    }

    st.finish();

    // merge the waves' states pairwise through LDS: waves [h, 2h) hand theirs to waves [0, h), h = W/2 .. 1
    constexpr int kState = NT * CT * 64 * 4 + NT * 64 * 2;             // floats per handed-over state
    float *lds = reinterpret_cast<float *>(lds_raw);
#pragma unroll 1
    for (int h = W / 2; h >= 1; h >>= 1) {
        if (wave >= h && wave < 2 * h) {
            float *base = lds + (wave - h) * kState;
            f32x4 *lo = reinterpret_cast<f32x4 *>(base);                // [NT][CT][64]
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
#pragma unroll
                for (int dt = 0; dt < CT; ++dt) lo[(nt * CT + dt) * 64 + lane] = st.o[nt][dt];
                base[NT * CT * 64 * 4 + nt * 64 + lane] = st.m[nt];
                base[NT * CT * 64 * 4 + NT * 64 + nt * 64 + lane] = st.l[nt];
            }
        }
        __syncthreads();
        if (wave < h) {
            const float *base = lds + wave * kState;
            const f32x4 *lo = reinterpret_cast<const f32x4 *>(base);
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                const float m2 = base[NT * CT * 64 * 4 + nt * 64 + lane];
                const float l2 = base[NT * CT * 64 * 4 + NT * 64 + nt * 64 + lane];
                const float mm = fmaxf(st.m[nt], m2);
                const float a = weight(st.m[nt], mm), b = weight(m2, mm);
                st.l[nt] = st.l[nt] * a + l2 * b;
                st.m[nt] = mm;
#pragma unroll
                for (int dt = 0; dt < CT; ++dt)
                    st.o[nt][dt] = st.o[nt][dt] * a + lo[(nt * CT + dt) * 64 + lane] * b;
            }
        }
        __syncthreads();
    }
    if constexpr (FINISH) {
        if (wave == 0) store_finished<DT, D>(P, t, head, rows, l16, grp, st);
    } else if constexpr (W == 1 && NT == 1 && D <= 128) {
        if (P.arrive) store_partial_staged<kRowsCoherent, D>(P, t, head, rows, lane, st, stage);
        else          store_partial_staged<kRowsPlain, D>(P, t, head, rows, lane, st, stage);
    } else {
        if (wave == 0) {
            if (P.arrive) store_partial<kRowsCoherent, NT, D>(P, t, head, 0, rows, l16, grp, st);
            else          store_partial<kRowsPlain, NT, D>(P, t, head, 0, rows, l16, grp, st);
        }
    }
}

// ---- dense path: 1..256 rows, the 8 waves split the rows (32 each) and share each block ------------
//
// Blocks travel HBM -> LDS without passing through registers (global_load_lds_dwordx4: every lane
// moves 16 bytes, a wave fills 1 KB of consecutive LDS).  A ring of kRing block slots (16 KB each:
// 32 K rows then 32 V rows of 256 B) keeps five (four with two-block intervals) blocks in flight per
// workgroup.  Rows are stored unpadded; the 16-byte column index is XORed with a function of the row so
// that the operand reads spread over all banks.  The swizzle is applied on the global side: the lane that fills LDS
// column c of a row fetches column c ^ f(row).
//
// The compiler does not see these loads (inline asm), so the waits are explicit: loads complete in
// issue order, block b is in LDS once at most 2 * (blocks issued after b) of the wave's loads are
// outstanding, and the barrier that follows publishes all eight waves' parts.
constexpr int kRing = 10;                    // slots allocated; a path may cycle through fewer
constexpr int kBlockBytes = 16384;
constexpr int kRingBytes = kRing * kBlockBytes;
constexpr int kSplitBlocksMaxRows = 128;     // dense tasks up to this many rows, and at least
constexpr int kSplitBlocksMinLen = 1024;     // this many tokens: two waves per row group
// s_waitcnt immediate that waits for the vector-memory counter only (gfx9 encoding: bits 3:0 and 15:14)
constexpr int vmcnt_imm(int n) { return (n & 15) | ((n >> 4) << 14) | 0x0F70; }

// One block's K piece and V piece for this wave: each lane fetches 16 bytes at gk + voff_k (gv + voff_v)
// and the wave's 64 pieces land in 1 KB of consecutive LDS at lds_addr (the V piece 8 KB behind).  M0
// holds the LDS address for the instruction and is put back afterwards.
__device__ __forceinline__ void dma16_pair(uint32_t lds_addr, uint32_t voff_k, uint32_t voff_v, const char *gk,
                                           const char *gv, int read_once)
{
    uint32_t m0_saved;
    if (read_once) {
        asm volatile("s_mov_b32 %0, m0\n\t"
                     "s_mov_b32 m0, %1\n\t"
                     "s_nop 0\n\t"
                     "global_load_lds_dwordx4 %2, %4 nt\n\t"
                     "s_add_u32 m0, m0, 0x2000\n\t"
                     "s_nop 0\n\t"
                     "global_load_lds_dwordx4 %3, %5 nt\n\t"
                     "s_mov_b32 m0, %0\n"
                     : "=&s"(m0_saved)
                     : "s"(lds_addr), "v"(voff_k), "v"(voff_v), "s"(gk), "s"(gv)
                     : "memory", "scc");
    } else {
        asm volatile("s_mov_b32 %0, m0\n\t"
                     "s_mov_b32 m0, %1\n\t"
                     "s_nop 0\n\t"
                     "global_load_lds_dwordx4 %2, %4\n\t"
                     "s_add_u32 m0, m0, 0x2000\n\t"
                     "s_nop 0\n\t"
                     "global_load_lds_dwordx4 %3, %5\n\t"
                     "s_mov_b32 m0, %0\n"
                     : "=&s"(m0_saved)
                     : "s"(lds_addr), "v"(voff_k), "v"(voff_v), "s"(gk), "s"(gv)
                     : "memory", "scc");
    }
}

// One 16-byte piece per lane from a per-lane address: lane i's piece lands at lds_addr + 16 * i.  Used for
// the query rows of a dense task, which are queued between the copies of K/V blocks: a load into
// registers there would have to be waited for by the compiler, which counts the copies as its own loads
// and would wait for all of them; through LDS the rows take the same asynchronous path as the blocks,
// no register is written behind the compiler's back, and the rows are read from LDS by ordinary loads
// once the hand-placed wait has passed.
__device__ __forceinline__ void dma16_rows(uint32_t lds_addr, const char *gp)
{
    uint32_t m0_saved;
    asm volatile("s_mov_b32 %0, m0\n\t"
                 "s_mov_b32 m0, %1\n\t"
                 "s_nop 0\n\t"
                 "global_load_lds_dwordx4 %2, off\n\t"
                 "s_mov_b32 m0, %0\n"
                 : "=&s"(m0_saved)
                 : "s"(lds_addr), "v"(gp)
                 : "memory", "scc");
}

// ---- dense path with 32 query rows per wave ---------------------------------------------------------
//
// v_mfma_f32_32x32x16: A operand lane = (row lane%32, k-group lane/32), 8 k-values per lane; B operand
// lane = (column lane%32, k-group lane/32); result register r of lane (column lane%32, group lane/32)
// is row 8*(r/4) + 4*(lane/32) + r%4.  As in the 16-row tiles, S^T = K Q^T comes out with a query row
// per lane column, which is the layout the B operand of O^T += V^T P^T wants: register 8t + i of the
// scores becomes k-value i of k-step t, and the A operand (V^T) is read with the same token order.
// Compared with 16 x 16 x 32 tiles a block costs half as many matrix instructions for the same
// arithmetic; the path is bound by the instructions a wave can issue, not by the matrix unit.
typedef __attribute__((ext_vector_type(16))) float f32x16;

template <int DT>
__device__ __forceinline__ f32x16 mfma32(u32x4 a, u32x4 b, f32x16 c)
{
    if constexpr (DT == CODEC_DTYPE_FP16)
        return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, a),
                                                       __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
    else
        return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a),
                                                        __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

// Keeps the computation of `x` where it is written (the compiler otherwise sinks work whose result
// is only used after the next barrier below that barrier).
__device__ __forceinline__ void pin(u32x4 &x) { asm volatile("" : "+v"(x)); }
__device__ __forceinline__ void pin(int &x) { asm volatile("" : "+v"(x)); }

// Roles of a wave in a dense task.  A wave with rows owns 32 of them; in the two live roles the halves
// of a step come in opposite orders, for the two waves of a SIMD.  Waves without rows only help moving
// blocks.  All eight waves run the same barriers.
//
// STRIDE = 1: a live wave takes every block (tasks of more than 128 rows, up to eight row groups; and
// short slices of any task, see run_dense32).
// STRIDE = 2: tasks of at most 128 rows have at most four row groups; waves w and w+4 (one SIMD) share
// group w, the first takes the even blocks, the second the odd ones, and their two states are merged
// through LDS when the slice is done.  An interval then covers two blocks.  Without the split a SIMD
// would hold a single computing wave and the other one would idle.
enum { kHelper = 0, kMatrixFirst = 1, kVectorFirst = 2 };

// One wave's share of a dense task: task rows row0 .. row0+31 (none for a helper).
template <int DT, int ROLE, int STRIDE>
__device__ __forceinline__ void dense32_wave(const PacParams &P, const DevTask &t, int head, char *lds,
                                             int wave, int row0, int rows, RowStore how)
{
    constexpr bool LIVE = ROLE != kHelper;
    static_assert(STRIDE == 1 || STRIDE == 2, "a row group is shared by one or two waves");
    // slots in use: an interval of two blocks wants a deeper ring to keep as many bytes in flight
    constexpr int RING = STRIDE == 2 ? kRing : 8;
    // the wave's blocks are first, first + STRIDE, ...
    const int first = (STRIDE == 2 && ROLE == kVectorFirst) ? 1 : 0;
    auto blk = [&](int k) { return first + k * STRIDE; };
    const int lane = opaque_lane();
    const int l32 = lane & 31, kg = lane >> 5;
    const int l16 = lane & 15, grp = lane >> 4;

    u32x4 qb[8];            // B operand of the scores: row l32, channels 16*ks + 8*kg .. +7
    f32x16 o[4];            // O^T: row l32, channel 32*ct + 8*(r/4) + 4*kg + r%4
    float m = -INFINITY;    // reference, log2 units, integer-valued (same in the two lanes of a row)
    float l4[4] = {0.f, 0.f, 0.f, 0.f};     // this lane's share of the row sum, in four partial sums
    if constexpr (LIVE) {
#pragma unroll
        for (int ct = 0; ct < 4; ++ct)
#pragma unroll
            for (int r = 0; r < 16; ++r) o[ct][r] = 0.f;
    }
    const SliceCtx c = make_ctx(P, t, head);

    // Asynchronous copies.  Wave w moves tokens 4w .. 4w+3 of every block, 1 KB of K and 1 KB of V;
    // lane (grp, l16) writes the 16-byte slot l16 of LDS row 4w + grp.  A K row keeps its 16-byte
    // column g in slot g ^ (token & 15), a V row in slot g ^ 4*(token & 3): the swizzles that make
    // the operand reads below free of bank conflicts (a transposing V read takes, per 32 lanes, 4 rows
    // x 64 bytes: the four rows must land in four different quarters of the 256 bytes of banks).
    const uint32_t lds_base = uint32_t(uintptr_t(lds));
    const int tok_w = wave * 4 + grp;
    const uint32_t voff_k = uint32_t(grp) * c.token_bytes + uint32_t((l16 ^ (tok_w & 15)) << 4);
    const uint32_t voff_v = uint32_t(grp) * c.token_bytes + uint32_t((l16 ^ ((tok_w & 3) << 2)) << 4);
    // a group of four tokens past the end of the slice is redirected to token 0 (its rows are masked
    // later) so that no address leaves the slice's pages
    auto first_token = [&](int bb) {
        const int tok0 = bb * 32 + wave * 4;
        return tok0 >= c.kv_len ? 0 : tok0;
    };
    auto page_issue = [&](int bb) { return uniform_load(c.pages, first_token(bb) >> c.page_shift); };
    auto dma_block = [&](int bb, int pg) {                              // pg: page id from page_issue(bb)
        const int64_t off = page_offset(c, pg, first_token(bb) & c.page_mask);
        const uint32_t slot = lds_base + uint32_t(bb % RING) * kBlockBytes + uint32_t(wave) * 1024;
        dma16_pair(slot, voff_k, voff_v, c.k_head + off, c.v_head + off, c.read_once);
    };

    // Operand reads.
    // K (A operand of the scores): lane (l32, kg) reads column 2*ks + kg of token row l32; with the
    // swizzle its address is the ks = 0 address with (ks << 5) XORed in.
    // V (A operand of the accumulation, channel tile ct, k-step t): ds_read_b64_tr_b16 hands lane i of a
    // 16-lane group column i of the 4 x 16 tile whose row k the group's lanes 4k .. 4k+3 address 8 bytes
    // apiece.  Lane group (kg, ch) = (lane/32, lane/16 % 2), lane (k, q) in it, addresses token
    // 16*t + 8*h + 4*kg + k, channels 32*ct + 16*ch + 4*q .. +3: two reads (h = 0, 1) give the lane its
    // channel 32*ct + lane%32 for the 8 tokens of its k-group.  ct is XORed into the address like ks.
    const uint32_t ka_lane = uint32_t(l32 * 256 + ((kg ^ (l32 & 15)) << 4));
    const int vk = l16 >> 2, vq = l16 & 3, vch = grp & 1;
    const int vrow = 4 * kg + vk;
    const uint32_t va_lane =
        uint32_t(8192 + vrow * 256 + ((((2 * vch + (vq >> 1)) ^ ((vrow & 3) << 2)) & 15) << 4) + 8 * (vq & 1));
    u32x4 kr[8];            // K operands of one block, by k-step
    u32x4 vr[4][2];         // V operands of one block, by channel tile and k-step
    auto key_base = [&](int bb) { return lds_base + uint32_t(bb % RING) * kBlockBytes + ka_lane; };
    auto value_base = [&](int bb) { return lds_base + uint32_t(bb % RING) * kBlockBytes + va_lane; };
    auto load_key = [&](uint32_t base, int ks) {                        // K operand of k-step ks
        kr[ks] = *reinterpret_cast<const u32x4 __attribute__((address_space(3))) *>(uintptr_t(base ^ uint32_t(ks << 5)));
    };
    typedef __attribute__((ext_vector_type(4))) short s16x4;
    typedef s16x4 __attribute__((address_space(3))) *lds_s16x4_ptr;
    auto load_value = [&](uint32_t base, int ct, int tt) {              // V operand of channel tile ct, k-step tt
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const uint32_t addr = (base ^ uint32_t(ct << 6)) + tt * 4096 + h * 2048;
            const s16x4 x = __builtin_amdgcn_ds_read_tr16_b64_v4i16(reinterpret_cast<lds_s16x4_ptr>(uintptr_t(addr)));
            const uint2 w = __builtin_bit_cast(uint2, x);
            vr[ct][tt][2 * h] = w.x;
            vr[ct][tt][2 * h + 1] = w.y;
        }
    };
    auto load_keys = [&](int bb) {
        const uint32_t base = key_base(bb);
#pragma unroll
        for (int ks = 0; ks < 8; ++ks) load_key(base, ks);
    };
    auto load_values = [&](int bb) {
        const uint32_t base = value_base(bb);
#pragma unroll
        for (int ct = 0; ct < 4; ++ct)
#pragma unroll
            for (int tt = 0; tt < 2; ++tt) load_value(base, ct, tt);
    };
    // tokens past `valid` count as zero in V (the slot may hold anything there, NaN patterns included)
    // and as -inf in the scores
    auto mask_values = [&](int valid) {
#pragma unroll
        for (int tt = 0; tt < 2; ++tt)
#pragma unroll
            for (int d = 0; d < 4; ++d) {
                const int tok = 16 * tt + 8 * (d >> 1) + 4 * kg + 2 * (d & 1);  // low half; high half tok+1
                const unsigned int keep = (tok < valid ? 0x0000FFFFu : 0u) | (tok + 1 < valid ? 0xFFFF0000u : 0u);
#pragma unroll
                for (int ct = 0; ct < 4; ++ct) vr[ct][tt][d] &= keep;
            }
    };
    auto mask_scores32 = [&](f32x16 &s, int valid) {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const bool dead = 8 * (r >> 2) + 4 * kg + (r & 3) >= valid;
            s[r] = dead ? -INFINITY : s[r];
        }
    };

    f32x16 s;               // scores: row l32, token 8*(r/4) + 4*kg + r%4
    u32x4 p[2];             // probabilities, B operand: k-step t holds registers 8t .. 8t+7 of the scores
    auto scores32 = [&]() {
        f32x16 acc;
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[r] = 0.f;
#pragma unroll
        for (int i = 0; i < 8; ++i) acc = mfma32<DT>(kr[i], qb[i], acc);
        s = acc;
    };
    auto accumulate32 = [&]() {
#pragma unroll
        for (int i = 0; i < 8; ++i) o[i & 3] = mfma32<DT>(vr[i & 3][i >> 2], p[i >> 2], o[i & 3]);
    };
    // The matrix half of a FULL step: O^T += V^T P^T of the block in vr and the scores of the block in
    // kr; the two alternate so that no instruction waits for the one before it.  With one wave per row
    // group (compute-bound tasks) each pair is followed by the LDS reads that refill the operand
    // registers it has just consumed (K of block kb, V of block vb): the reads are issued while the
    // matrix unit works on the pair.
    auto matrix_half = [&](int kb, int vb, auto after_first_pair) {
        const uint32_t kbase = key_base(kb), vbase = value_base(vb);
        // the wave in its matrix half goes first when both waves of the SIMD have an instruction ready:
        // measured, the other order starves the matrix instructions (1150 against 1010 clk per half)
        __builtin_amdgcn_s_setprio(3);
        f32x16 acc;
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[r] = 0.f;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            o[i & 3] = mfma32<DT>(vr[i & 3][i >> 2], p[i >> 2], o[i & 3]);
            acc = mfma32<DT>(kr[i], qb[i], acc);
            if constexpr (STRIDE == 1) {
                load_value(vbase, i & 3, i >> 2);
                load_key(kbase, i);
            }
            if (i == 0) after_first_pair();
            __builtin_amdgcn_sched_barrier(0);
        }
        __builtin_amdgcn_s_setprio(0);
        if constexpr (STRIDE == 2) {        // memory-bound tasks: measured faster with the reads in one go
            load_keys(kb);
            load_values(vb);
            __builtin_amdgcn_sched_barrier(0);
        }
        s = acc;
    };
    // The vector work of a block, in three pieces.  reference(): the lane's maximum over its 16 scores;
    // when a row has outgrown its reference by more than the lag, the reference moves up to the
    // (rounded-up) row maximum and everything accumulated against the old one is rescaled.
    // probabilities(t): P = exp2(scale * S - m) for k-step t in B-operand layout, and the lane's share
    // of the row sum.
    auto reference = [&]() {
        float a = __builtin_fmaxf(__builtin_fmaxf(s[0], s[1]), s[2]);
#pragma unroll
        for (int r = 3; r + 1 < 16; r += 2) a = __builtin_fmaxf(__builtin_fmaxf(a, s[r]), s[r + 1]);
        const float lm = __builtin_fmaxf(a, s[15]) * P.scale_log2e;
        if (__any(lm > m + kLag)) {
            const float mx = fmaxf(lm, __shfl_xor(lm, 32));
            const float m_new = __builtin_ceilf(fmaxf(m, mx));
            const float alpha = fast_exp2(m - m_new);                   // 0 on the first block (m = -inf)
#pragma unroll
            for (int d = 0; d < 4; ++d) l4[d] *= alpha;
#pragma unroll
            for (int ct = 0; ct < 4; ++ct)
#pragma unroll
                for (int r = 0; r < 16; ++r) o[ct][r] *= alpha;
            m = m_new;
        }
    };
    auto probabilities32 = [&](int tt) {
        float e[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) e[i] = fast_exp2(__builtin_fmaf(s[8 * tt + i], P.scale_log2e, -m));
#pragma unroll
        for (int d = 0; d < 4; ++d) {
            p[tt][d] = pack2<DT>(e[2 * d], e[2 * d + 1]);
            l4[d] = add_pair<DT>(p[tt][d], l4[d]);
        }
        pin(p[tt]);
    };

    // Common to all roles.  All but S = STRIDE blocks of the ring are requested up front; interval j
    // (j = 0 .. nint-1) starts with a barrier behind which S blocks are requested into the slots of the
    // blocks of interval j-1.  Those were consumed before the barrier; the LDS reads issued last, of blocks
    // that interval j uses, may still be under way: the barrier waits for no LDS read.  Against one that did,
    // with the slots of interval j's own blocks refilled, which kept a block (two) more in flight: 32 layers of
    // 64 requests of 4 rows below a 4096-token root 853 -> 835 us, a six-level binary tree of 32 .. 1024 rows
    // 40.0 -> 39.2, three-level documents 161.4 -> 160.5, long slices under 64 and 128 rows 0.5-1.5 % faster
    // (109.7 -> 108.7), nothing on a 131072-token root under 512 rows, whose rate the clock sets.  The LDS
    // reads of interval j reach up to block S*j + 3*S - 1, which must have landed at its barrier: each wave
    // issues 2 loads per block and loads complete in order, so a block has landed once at most 2 * (blocks
    // issued after it) loads are outstanding; near the end of the slice, where fewer blocks follow, the
    // wait is for everything.
    const int nblk = (t.kv_len + 31) >> 5;
    const int nint = (nblk + STRIDE - 1) / STRIDE - 1;                  // the same for every wave
    // Start of the task.  What the first matrix instruction waits for is a chain of dependent reads:
    // page ids and the rows' requests, then the first blocks and the query rows.  The two reads of a
    // stage are issued together; the query rows (32 rows of 32 bytes per instruction, the slowest
    // requests to issue) are queued behind the copies of the first 2S blocks only.  They travel through
    // LDS like the blocks (dma16_rows): each wave parks its 8 KB in the last four slots of the ring,
    // whose blocks are requested once every wave has taken its rows into registers, behind the barrier
    // that ends this start-up; the other blocks of the ring are requested right behind the rows.
    constexpr int LAG = STRIDE;                                         // slots left free when an interval starts
    constexpr int EARLY = RING - 4;                                     // blocks requested ahead of that barrier
    static_assert(EARLY >= 2 * STRIDE && 8 * 8192 == 4 * kBlockBytes, "the rows' parking space is the last four slots");
    int pg_late[4];
    {
        int pg[RING];
#pragma unroll
        for (int d = 0; d < RING; ++d) pg[d] = page_issue(d < nblk ? d : 0);
        const char *qp = nullptr;
        bool live = false;
        if constexpr (LIVE) {
            const int row = row0 + l32;
            live = row < rows;
            const int qi = live ? row / P.group : row0 / P.group;       // a dead row reads row0's
            const int hj = live ? row - qi * P.group : row0 - qi * P.group;
            int req = t.single_req >= 0 ? t.single_req : P.node_q[t.q_off + qi];
            pin(req);                           // the wait for it stands here, ahead of the copies
            qp = static_cast<const char *>(P.q)
                 + (int64_t(req) * P.h_q + int64_t(head) * P.group + hj) * (kHeadDim * 2) + kg * 16;
        }
#pragma unroll
        for (int d = 0; d < 4; ++d) pg_late[d] = pg[EARLY + d];
#pragma unroll
        for (int d = 0; d < 2 * STRIDE; ++d)
            if (d < nblk) dma_block(d, pg[d]);
        const uint32_t park = lds_base + uint32_t(EARLY) * kBlockBytes + uint32_t(wave) * 8192;   // wave-uniform
        const uint32_t parked = park + uint32_t(lane) * 16;
        if constexpr (LIVE) {
#pragma unroll
            for (int ks = 0; ks < 8; ++ks) dma16_rows(park + ks * 1024, qp + ks * 32);
        }
#pragma unroll
        for (int d = 2 * STRIDE; d < EARLY; ++d)
            if (d < nblk) dma_block(d, pg[d]);
        // loads complete in order: with at most the copies of blocks 2S .. EARLY-1 outstanding, blocks
        // 0 .. 2S-1 and the query rows have landed
        if (nblk >= EARLY) __builtin_amdgcn_s_waitcnt(vmcnt_imm(2 * (EARLY - 2 * STRIDE)));
        else                __builtin_amdgcn_s_waitcnt(0x0F70);
        if constexpr (LIVE) {
            typedef const u32x4 __attribute__((address_space(3))) *lds_u32x4_ptr;
#pragma unroll
            for (int ks = 0; ks < 8; ++ks) {
                const u32x4 x = *reinterpret_cast<lds_u32x4_ptr>(uintptr_t(parked + ks * 1024));   // the piece this lane sent
                qb[ks] = live ? x : u32x4{0u, 0u, 0u, 0u};
            }
            // the rows are in registers before this wave passes the barrier below, behind which the
            // parking space is overwritten
            __builtin_amdgcn_s_waitcnt(0xC07F);
        }
    }
    int pg_next[STRIDE];                                                // pages of the blocks interval 0 requests
#pragma unroll
    for (int u = 0; u < STRIDE; ++u) pg_next[u] = pg_late[4 - LAG + u];
    __syncthreads();
#pragma unroll
    for (int d = 0; d < 4 - LAG; ++d)
        if (EARLY + d < nblk) dma_block(EARLY + d, pg_late[d]);

    // more: the blocks that interval j requests all exist
    auto wait_and_sync = [&](auto more) {   // then blocks up to S*j+3S-1 are complete, and everyone is done with those below S*j
        if constexpr (decltype(more)::value) {
            asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" : : "n"(2 * (RING - LAG - 3 * STRIDE)) : "memory");
        } else {
            __builtin_amdgcn_s_waitcnt(0x0F70);
            __syncthreads();
        }
    };
    auto request_blocks = [&](int j, auto more) {                       // any time inside interval j
        if constexpr (decltype(more)::value) {
#pragma unroll
            for (int u = 0; u < STRIDE; ++u) dma_block(STRIDE * j + RING - LAG + u, pg_next[u]);
#pragma unroll
            for (int u = 0; u < STRIDE; ++u) pg_next[u] = page_issue(STRIDE * (j + 1) + RING - LAG + u);
        } else if constexpr (STRIDE == 2) {
            if (2 * j + RING - LAG < nblk) dma_block(2 * j + RING - LAG, pg_next[0]);         // an odd block left over
        }
    };
    auto enter_interval = [&](int j, auto more) {                       // j < nint
        wait_and_sync(more);
        request_blocks(j, more);
    };
    using yes = std::true_type;
    using no = std::false_type;
    auto short_block = [&](int b) { return c.kv_len - b * 32; };        // valid tokens if below 32
    auto more_follow = [&](int j) { return STRIDE * j + RING - LAG + STRIDE - 1 < nblk; };

    if constexpr (LIVE) {
        // The wave's k-th block is b_k = blk(k), nmine of them.  Per block a vector half V(b_k) (scores
        // of the block -> probabilities) and a matrix half M(b_k) (accumulation of b_k, alternating with
        // the scores of b_k+1), in the order V(b_0) M(b_0) V(b_1) M(b_1) ...; right after M(b_k) has read
        // its operands the operands of M(b_k+1) (K of block b_k+2, V of block b_k+1) are requested from
        // LDS, to arrive during V(b_k+1).  A vector-first wave places the barrier of interval k before
        // V(b_k), a matrix-first wave before M(b_k): the two waves of a SIMD run in opposite phases,
        // one's matrix work beside the other's vector work.
        constexpr bool VFIRST = ROLE == kVectorFirst;
        const int nmine = nblk > first ? (nblk - first + STRIDE - 1) / STRIDE : 0;
        auto vector_half_of = [&](int b) {
            if (short_block(b) < 32) mask_scores32(s, short_block(b));
            reference();
            probabilities32(0);
            probabilities32(1);
        };
        // With one wave per row group the copies of the interval are requested from inside the matrix
        // half: their address arithmetic issues while the matrix unit works, instead of ahead of it.
        constexpr bool REQUEST_INSIDE = STRIDE == 1;
        auto matrix_half_and_loads = [&](int k, auto more) {            // M(b_k), k + 1 < nmine
            matrix_half(blk(k + 2), blk(k + 1), [&]() {
                if constexpr (REQUEST_INSIDE) request_blocks(k, more);
            });
            __builtin_amdgcn_sched_barrier(0);
        };
        auto interval = [&](int k, auto more) {
            wait_and_sync(more);
            if constexpr (!REQUEST_INSIDE) request_blocks(k, more);
            if (STRIDE == 1 || k + 1 < nmine) {                         // else: the other wave's last block only
                if constexpr (VFIRST) {
                    vector_half_of(blk(k));
                    __builtin_amdgcn_sched_barrier(0);
                    matrix_half_and_loads(k, more);
                } else {
                    matrix_half_and_loads(k, more);
                    vector_half_of(blk(k + 1));
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
        };
        if (STRIDE == 1 || nmine > 0) {
            load_keys(blk(0));
            scores32();
            __builtin_amdgcn_sched_barrier(0);
            load_keys(blk(1));
            load_values(blk(0));
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (!VFIRST) {
                vector_half_of(blk(0));
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        int k = 0;
#pragma unroll 1
        for (; k < nint && more_follow(k); ++k) interval(k, yes{});
#pragma unroll 1
        for (; k < nint; ++k) interval(k, no{});
        if (STRIDE == 1 || nmine > 0) {
            const int last = blk(nmine - 1);
            if constexpr (VFIRST) vector_half_of(last);
            if (short_block(last) < 32) mask_values(short_block(last));
            accumulate32();
        }
    } else {
        int k = 0;
#pragma unroll 1
        for (; k < nint && more_follow(k); ++k) enter_interval(k, yes{});
#pragma unroll 1
        for (; k < nint; ++k) enter_interval(k, no{});
    }

    __syncthreads();                        // every block has been read: the ring is free
    float l = (l4[0] + l4[1]) + (l4[2] + l4[3]);
    if constexpr (STRIDE == 2) {
        // The odd-block wave hands its state to the even-block wave of its row group: 64 accumulator
        // registers, reference and sum share per lane, register-major so that a wave's store or load
        // covers consecutive words.
        float *x = reinterpret_cast<float *>(lds) + (wave & 3) * (66 * 64) + lane;
        if constexpr (ROLE == kVectorFirst) {
#pragma unroll
            for (int ct = 0; ct < 4; ++ct)
#pragma unroll
                for (int r = 0; r < 16; ++r) x[(ct * 16 + r) * 64] = o[ct][r];
            x[64 * 64] = m;
            x[65 * 64] = l;
        }
        __syncthreads();
        if constexpr (ROLE == kMatrixFirst) {
            const float m2 = x[64 * 64], l2 = x[65 * 64];
            const float m_new = fmaxf(m, m2);
            const float a1 = weight(m, m_new), a2 = weight(m2, m_new);
            l = l * a1 + l2 * a2;
#pragma unroll
            for (int ct = 0; ct < 4; ++ct)
#pragma unroll
                for (int r = 0; r < 16; ++r) o[ct][r] = o[ct][r] * a1 + x[(ct * 16 + r) * 64] * a2;
            m = m_new;
        }
    }

    // The partial rows go out through LDS: in registers a lane holds 16-byte pieces of one row, and a
    // store instruction of the wave would touch 32 rows with 32 bytes each (measured: 3.1 us to issue
    // the 128 KB of a 256-row task, the address unit taking one such piece about every two cycles).
    // Each wave writes its 32 x 128 floats into an area of its own (rows 528 bytes apart: 16 lanes
    // then cover all banks) and reads them back row by row: a store instruction covers two whole rows,
    // 1 KB of consecutive memory.  With two waves per row group the area is the one the hand-over
    // above has just used, and only its own wave touches it from here on.
    constexpr int kStageRow = 528, kStageWave = 66 * 64 * 4;
    static_assert(32 * kStageRow <= kStageWave && 8 * kStageWave <= kRingBytes, "staging areas fit the ring");
    if constexpr (ROLE == kMatrixFirst || (STRIDE == 1 && LIVE)) {
        l += __shfl_xor(l, 32);
        typedef f32x4 __attribute__((address_space(3))) *lds_f32x4_ptr;
        const uint32_t area = lds_base + uint32_t(STRIDE == 2 ? (wave & 3) : wave) * kStageWave;
        const uint32_t put = area + uint32_t(l32) * kStageRow + uint32_t(kg) * 16;
#pragma unroll
        for (int ct = 0; ct < 4; ++ct)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const f32x4 x4 = {o[ct][4 * q], o[ct][4 * q + 1], o[ct][4 * q + 2], o[ct][4 * q + 3]};
                *reinterpret_cast<lds_f32x4_ptr>(uintptr_t(put + ct * 128 + q * 32)) = x4;
            }
        const uint32_t get = area + uint32_t(kg) * kStageRow + uint32_t(l32) * 16;
        const int64_t prow = int64_t(head) * P.part_rows + t.part_row_base + row0;
        float *po = P.part_o + prow * kHeadDim;
        with_row_store(how, [&](auto h) __attribute__((always_inline)) {
            constexpr RowStore HOW = decltype(h)::value;
            if (row0 + l32 < rows && kg == 0) st8_partial<HOW>(P.part_ml + (prow + l32) * 2, m, l);
            const Rows out = rows_at(po, (rows - row0) * kHeadDim * 4);         // rows the task does not have are dropped
#pragma unroll
            for (int j = 0; j < 16; ++j) {
                const f32x4 x4 = *reinterpret_cast<lds_f32x4_ptr>(uintptr_t(get + j * 2 * kStageRow));
                if constexpr (HOW != kRowsCoherent) st16_rows<HOW>(out, lane * 16 + j * 2 * kHeadDim * 4, x4);
                else if (row0 + 2 * j + kg < rows) st16_partial<HOW>(po + (2 * j + kg) * kHeadDim + l32 * 4, x4);
            }
        });
    }
    __syncthreads();                        // the staging areas (and the hand-over area) are free for the next task
}

// Dense task.  More than 128 rows: wave w owns rows 32w .. 32w+31; waves 4 .. 7 share their SIMDs with
// waves 0 .. 3 and run in the opposite phase.  Up to 128 rows: waves w and w+4 share rows 32w .. 32w+31
// and take alternate blocks, again in opposite phases; short slices, for which the hand-over at the end
// costs more than the overlap gains (about 1 us per task), keep one wave per row group.
template <int DT>
__device__ __forceinline__ void run_dense32(const PacParams &P, const DevTask &t, int head, char *lds, RowStore how)
{
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int rows = t.n_req * P.group;
    if (rows > kSplitBlocksMaxRows || t.kv_len < kSplitBlocksMinLen) {
        const int row0 = wave * 32;
        if (row0 >= rows)  dense32_wave<DT, kHelper, 1>(P, t, head, lds, wave, 0, 0, how);
        else if (wave & 4) dense32_wave<DT, kVectorFirst, 1>(P, t, head, lds, wave, row0, rows, how);
        else               dense32_wave<DT, kMatrixFirst, 1>(P, t, head, lds, wave, row0, rows, how);
    } else {
        const int row0 = (wave & 3) * 32;
        if (row0 >= rows)  dense32_wave<DT, kHelper, 2>(P, t, head, lds, wave, 0, 0, how);
        else if (wave & 4) dense32_wave<DT, kVectorFirst, 2>(P, t, head, lds, wave, row0, rows, how);
        else               dense32_wave<DT, kMatrixFirst, 2>(P, t, head, lds, wave, row0, rows, how);
    }
}

// ---- tile path: 17 .. 256 rows of 64 channels, 17 .. 128 rows of 256 ------------------------------------
//
// With 64 and 256 channels the plan tiles query sets 32 (16) rows at a time.  Sibling row tiles of one KV
// slice run here as ONE task (the device image packs them, DevTask): the slice then travels HBM -> LDS once
// for all of them instead of once per tile through the CU's memory pipeline, which is what bounds such
// plans (a CU streams 24-27 GB/s from HBM whatever its waves do).  Measured, whole step, a tree of a
// 2048-token root, 16 nodes of 8192 tokens and ragged leaves of 32 .. 512: 128 requests with 64 / 8 heads of
// 64 channels 100.6 -> 74.7 us, 256 requests with 16 / 8 heads of 256 channels 370 -> 290 us.  A task of up to
// 64 rows streams at 5.2 (64 channels) and 6.0 TB/s (256) where its row tiles took 4.1 and 3.0; 128 rows
// at 3.8 and 4.8 where they took 2.4 and 1.6 (4096 tokens, all CUs busy).
//
// One workgroup per CU: eight waves with 64 channels, four (one per SIMD, for its registers) with 256.
// 16 x 16 x 32 tiles and the arithmetic of the stream path; a wave owns NT row tiles of 16, which share
// every operand read.  K is the A operand by 16-byte LDS reads, V by transposing LDS reads, so that
// register e of channel tile dt is channel 16*dt + 4*(lane/16) + e.  Blocks are copied asynchronously
// (dma16_pair's instruction) into a ring of 128 KB, an interval of 32 KB (four blocks of 64 channels, one
// of 256) per barrier and all but one interval of the ring requested ahead.
template <int D>
struct TilePath {
    static constexpr int kWaves = kernel_waves(kFormWide, D);
    static constexpr int kRowBytes = D * 2;
    static constexpr int kHalf = 32 * kRowBytes;            // K (or V) of a block
    static constexpr int kBlock = 2 * kHalf;
    static constexpr int kBlocks = D == 64 ? 4 : 1;         // blocks of an interval
    static constexpr int kInterval = kBlocks * kBlock;
    static constexpr int kMine = kBlocks * 4 / kWaves;      // blocks of an interval of which a wave copies eight tokens
    static constexpr int kIntervals = 131072 / kInterval;   // slots of the ring
    static constexpr int kRingBytes = kIntervals * kInterval;
    static constexpr int kPieces = 8 * kRowBytes / 1024;    // 1 KB copies of eight tokens of one pool
    static constexpr int kCopies = kMine * 2 * kPieces;     // copies per wave and interval
    static constexpr int CT = D / 16;
    // state of NT row tiles as a wave hands it to another, in floats
    static constexpr int state_floats(int nt) { return nt * CT * 64 * 4 + nt * 64 * 2; }
    static_assert((kIntervals - 2) * kCopies < 64, "outstanding copies fit the wait counter");
};

// Copies 1 KB: each lane 16 bytes from gbase + voff to lds_addr + 16 * lane.
__device__ __forceinline__ void dma16(uint32_t lds_addr, uint32_t voff, const char *gbase, int read_once)
{
    // wave-uniform: kept in scalar registers also where the compiler has lost track of that
    const uint64_t g = uint64_t(uintptr_t(gbase));
    gbase = reinterpret_cast<const char *>(uintptr_t(
        uint64_t(uint32_t(__builtin_amdgcn_readfirstlane(uint32_t(g >> 32)))) << 32 | uint32_t(__builtin_amdgcn_readfirstlane(uint32_t(g)))));
    uint32_t m0_saved;
    if (read_once)
        asm volatile("s_mov_b32 %0, m0\n\t"
                     "s_mov_b32 m0, %1\n\t"
                     "s_nop 0\n\t"
                     "global_load_lds_dwordx4 %2, %3 nt\n\t"
                     "s_mov_b32 m0, %0\n"
                     : "=&s"(m0_saved)
                     : "s"(lds_addr), "v"(voff), "s"(gbase)
                     : "memory");
    else
        asm volatile("s_mov_b32 %0, m0\n\t"
                     "s_mov_b32 m0, %1\n\t"
                     "s_nop 0\n\t"
                     "global_load_lds_dwordx4 %2, %3\n\t"
                     "s_mov_b32 m0, %0\n"
                     : "=&s"(m0_saved)
                     : "s"(lds_addr), "v"(voff), "s"(gbase)
                     : "memory");
}

// NT: row tiles of 16 per wave.  SHARE: waves that share a row group; they take turns with the blocks of
// every interval and merge their states at the end.
template <int DT, int D, int NT, int SHARE>
__device__ __forceinline__ void run_tile_of(const PacParams &P, const DevTask &t, int head, char *lds, RowStore how)
{
    using T = TilePath<D>;
    constexpr int RB = T::kRowBytes, KS = D / 32, CT = T::CT;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = opaque_lane();
    const int l16 = lane & 15, grp = lane >> 4;
    const int rows = t.n_req * P.group;
    constexpr int GROUPS = T::kWaves / SHARE;
    const int group = wave % GROUPS, phase = wave / GROUPS;
    const int row0 = group * 16 * NT;
    const bool live = row0 < rows;                          // else: the wave only helps moving blocks
    const SliceCtx c = make_ctx(P, t, head);
    const int nblk = (t.kv_len + 31) >> 5;
    constexpr int NB = T::kBlocks, R = T::kIntervals;
    static_assert(NB % SHARE == 0 && (SHARE & (SHARE - 1)) == 0, "every wave of a group takes as many blocks of an interval");
    static_assert(SHARE == 1 || T::kWaves / 2 * T::state_floats(NT) * 4 <= T::kRingBytes, "hand-over areas fit the ring");
    const int nint = (nblk + NB - 1) / NB;
    // what the wave copies of every interval: eight tokens of block my_block and, with kMine = 2, of my_block + 2
    const int my_block = wave >> 2, my_token = (wave & 3) * 8;
    constexpr int MINE = T::kMine, STEP = T::kWaves / 4;

    // Copies, 1024 / RB tokens each.  A K row keeps its
    // 16-byte column g in slot g ^ fk(token), a V row in slot g ^ fv(token), applied on the global side:
    // the sixteen rows of a K read, and the eight rows (32 bytes each) that 32 lanes of a transposing V
    // read take, then lie in different banks.
    //   256 channels (a row is twice the 256 bytes of banks):  fk = token % 16,        fv = 2 * (token % 8)
    //    64 channels (a row is half of them):                  fk = (token / 2) % 8,   fv = 2 * ((token / 2) % 4)
    constexpr int LPR = RB / 16;                            // lanes per row of a copy
    constexpr int TPC = 64 / LPR;                           // tokens per copy
    auto fk = [](int token) { return D == 256 ? token & 15 : (token >> 1) & 7; };
    auto fv = [](int token) { return D == 256 ? 2 * (token & 7) : 2 * ((token >> 1) & 3); };
    const uint32_t lds_base = uint32_t(uintptr_t(lds));
    uint32_t voff_k[T::kPieces], voff_v[T::kPieces];
#pragma unroll
    for (int i = 0; i < T::kPieces; ++i) {
        const int in_copy = lane / LPR, token = my_token + i * TPC + in_copy;
        voff_k[i] = uint32_t(i * TPC + in_copy) * c.token_bytes + uint32_t(((lane % LPR) ^ fk(token)) << 4);
        voff_v[i] = uint32_t(i * TPC + in_copy) * c.token_bytes + uint32_t(((lane % LPR) ^ fv(token)) << 4);
    }
    // eight tokens past the end of the slice are redirected to its first ones (masked later): no address
    // leaves the slice's pages, and every interval has the same number of copies
    auto first_token = [&](int i, int u) {
        const int tok0 = (NB * i + my_block + u * STEP) * 32 + my_token;
        return tok0 >= c.kv_len ? 0 : tok0;
    };
    auto page_issue = [&](int i, int u) { return uniform_load(c.pages, first_token(i, u) >> c.page_shift); };
    const uint32_t my_slot = lds_base + uint32_t(my_block) * T::kBlock + uint32_t(my_token) * RB;
    auto request = [&](int i, const int (&pg)[MINE]) __attribute__((always_inline)) {  // interval i; pg: page_issue(i, .)
#pragma unroll
        for (int u = 0; u < MINE; ++u) {
            const uint32_t at = my_slot + uint32_t(i % R) * T::kInterval + uint32_t(u * STEP) * T::kBlock;
            const int64_t off = page_offset(c, pg[u], first_token(i, u) & c.page_mask);
#pragma unroll
            for (int n = 0; n < T::kPieces; ++n) dma16(at + n * 1024, voff_k[n], c.k_head + off, c.read_once);
#pragma unroll
            for (int n = 0; n < T::kPieces; ++n) dma16(at + T::kHalf + n * 1024, voff_v[n], c.v_head + off, c.read_once);
        }
    };

    // Operand reads.  K, token tile j, k-step ks: lane (l16, grp) reads 16-byte column 4*ks + grp of token
    // 16*j + l16.  V, channel tile dt, h: lane (k, q) of lane group grp addresses token 16*h + 4*grp + k,
    // channels 16*dt + 4*q .. +3, and receives channel 16*dt + l16 of tokens 16*h + 4*grp .. +3.
    const uint32_t k_lane = uint32_t(l16 * RB + ((grp ^ fk(l16)) << 4));
    const int vtok = 4 * grp + (l16 >> 2), vq = l16 & 3;
    const uint32_t v_lane = uint32_t(vtok * RB + (((vq >> 1) ^ fv(vtok)) << 4) + 8 * (vq & 1));
    typedef const u32x4 __attribute__((address_space(3))) *lds_u32x4_ptr;
    typedef __attribute__((ext_vector_type(4))) short s16x4;
    typedef s16x4 __attribute__((address_space(3))) *lds_s16x4_ptr;

    u32x4 qb[NT][KS];
    RowState<NT, D, CT> st;
    st.clear();

    auto compute = [&](int b, uint32_t kb) __attribute__((always_inline)) {
        f32x4 s[2][NT];
#pragma unroll
        for (int j = 0; j < 2; ++j) {
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) s[j][nt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                const u32x4 kr = reinterpret_cast<lds_u32x4_ptr>(uintptr_t(kb + (k_lane ^ uint32_t(ks << 6))))[j * RB];
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) s[j][nt] = mfma16<DT>(kr, qb[nt][ks], s[j][nt]);
            }
        }
        // the V operands of the first half of the channel tiles travel during the softmax
        u32x4 va[CT];
        auto load_value = [&](int dt) {
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const lds_s16x4_ptr at = reinterpret_cast<lds_s16x4_ptr>(uintptr_t(kb + (v_lane ^ uint32_t(dt << 5))));
                const uint2 w = __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16(at + (T::kHalf + h * 16 * RB) / 8));
                va[dt][2 * h] = w.x;
                va[dt][2 * h + 1] = w.y;
            }
        };
        constexpr int AHEAD = NT == 1 ? CT : CT / 2;
#pragma unroll
        for (int dt = 0; dt < AHEAD; ++dt) load_value(dt);
        __builtin_amdgcn_sched_barrier(0);
        const int valid = c.kv_len - b * 32;
        if (valid < 32) mask_scores<NT>(s, valid, grp);
        float lm[NT];
        lane_maxima<NT>(s, P.scale_log2e, lm);
        if (__any(outgrown<NT>(lm, st))) raise_reference<NT>(lm, st);
        u32x4 pb[NT];
        probabilities<DT, NT>(s, st, P.scale_log2e, pb);
#pragma unroll
        for (int dt = AHEAD; dt < CT; ++dt) load_value(dt);
#pragma unroll
        for (int dt = 0; dt < CT; ++dt)
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) st.o[nt][dt] = mfma16<DT>(va[dt], pb[nt], st.o[nt][dt]);
    };

    // V rows of the last block past the end of the slice count as zero (their memory may hold anything):
    // each wave clears the ones that it copied
    auto clear_tail = [&]() __attribute__((always_inline)) {
        const int valid = c.kv_len - (nblk - 1) * 32, last = (nblk - 1) % NB;
        if (last % STEP != my_block) return;
        const uint32_t at = lds_base + uint32_t((nint - 1) % R) * T::kInterval + uint32_t(last) * T::kBlock + T::kHalf
                            + uint32_t(my_token) * RB + uint32_t(lane) * 16;
#pragma unroll
        for (int n = 0; n < T::kPieces; ++n)
            if (my_token + n * TPC + lane / LPR >= valid)
                *reinterpret_cast<u32x4 __attribute__((address_space(3))) *>(uintptr_t(at + n * 1024)) = u32x4{0u, 0u, 0u, 0u};
    };

    // Start: the rows' requests and the page ids, read together; then the first interval's copies and the query
    // rows.  Waiting for the rows (the compiler waits for every load in flight) waits for that interval too, so
    // the others are requested behind it.
    int pg[R][MINE];
#pragma unroll
    for (int i = 0; i < R; ++i)
#pragma unroll
        for (int u = 0; u < MINE; ++u) pg[i][u] = page_issue(i, u);
    const char *qp[NT];
    bool row_live[NT];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        const int row = row0 + nt * 16 + l16;
        row_live[nt] = row < rows;
        const int qi = row_live[nt] ? row / P.group : 0;    // a dead row reads the task's first
        const int hj = row_live[nt] ? row - qi * P.group : 0;
        int req = P.node_q[t.q_off + qi];
        pin(req);                                           // the wait for it stands here, ahead of the copies
        qp[nt] = static_cast<const char *>(P.q) + (int64_t(req) * P.h_q + int64_t(head) * P.group + hj) * (D * 2) + grp * 16;
    }
    request(0, pg[0]);
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            qb[nt][ks] = ld16(qp[nt] + ks * 64);
            if (!row_live[nt]) qb[nt][ks] = u32x4{0u, 0u, 0u, 0u};
        }
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) pin(qb[nt][ks]);
#pragma unroll
    for (int i = 1; i + 1 < R; ++i)
        if (i < nint) request(i, pg[i]);
    int pg_next[MINE];
#pragma unroll
    for (int u = 0; u < MINE; ++u) pg_next[u] = pg[R - 1][u];
    auto enter_interval = [&](int i) __attribute__((always_inline)) {
        // interval i has landed once at most the copies of the intervals requested after it are outstanding
        if (i + R - 2 < nint) __builtin_amdgcn_s_waitcnt(vmcnt_imm((R - 2) * T::kCopies));
        else                  __builtin_amdgcn_s_waitcnt(0x0F70);
        if (i == nint - 1 && (c.kv_len & 31)) clear_tail();
        __syncthreads();                    // everyone's part has landed; interval i - 1 has been read by all
        if (i + R - 1 < nint) {
            request(i + R - 1, pg_next);
#pragma unroll
            for (int u = 0; u < MINE; ++u) pg_next[u] = page_issue(i + R, u);
        }
    };
    if (live) {
#pragma unroll 1
        for (int i = 0; i < nint; ++i) {
            enter_interval(i);
            const uint32_t kb = lds_base + uint32_t(i % R) * T::kInterval;
            if constexpr (NB == 1) {
                compute(i, kb);
            } else {
                const int end = nblk - NB * i < NB ? nblk - NB * i : NB;
#pragma unroll 1
                for (int u = phase; u < end; u += SHARE) compute(NB * i + u, kb + uint32_t(u) * T::kBlock);
            }
        }
    } else {
#pragma unroll 1
        for (int i = 0; i < nint; ++i) enter_interval(i);
    }
    st.finish();
    // the waves of a row group hand their states over pairwise: phases [h, 2h) to phases [0, h)
    if constexpr (SHARE > 1) {
        __syncthreads();                    // every block has been read: the ring is free
#pragma unroll 1
        for (int h = SHARE / 2; h >= 1; h >>= 1) {
            float *x = reinterpret_cast<float *>(lds) + (phase % h * GROUPS + group) * T::state_floats(NT);
            f32x4 *xo = reinterpret_cast<f32x4 *>(x);       // [NT][CT][64]
            float *xs = x + NT * CT * 64 * 4;
            if (phase >= h && phase < 2 * h) {
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) {
#pragma unroll
                    for (int dt = 0; dt < CT; ++dt) xo[(nt * CT + dt) * 64 + lane] = st.o[nt][dt];
                    xs[nt * 64 + lane] = st.m[nt];
                    xs[(NT + nt) * 64 + lane] = st.l[nt];
                }
            }
            __syncthreads();
            if (phase < h) {
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) {
                    const float m2 = xs[nt * 64 + lane], mm = fmaxf(st.m[nt], m2);
                    const float a = weight(st.m[nt], mm), b = weight(m2, mm);
                    st.l[nt] = st.l[nt] * a + xs[(NT + nt) * 64 + lane] * b;
                    st.m[nt] = mm;
#pragma unroll
                    for (int dt = 0; dt < CT; ++dt) st.o[nt][dt] = st.o[nt][dt] * a + xo[(nt * CT + dt) * 64 + lane] * b;
                }
            }
            __syncthreads();
        }
    }
    if (live && phase == 0) {
        const int tile_rows = (t.flags >> kTaskTileShift) & 255, stride = ~t.single_req;
        const int last_tile = (rows - 1) / tile_rows, last_back = t.flags >> kTaskLastShift;
        float *po = P.part_o + (int64_t(head) * P.part_rows + t.part_row_base) * D;
        float *pml = P.part_ml + (int64_t(head) * P.part_rows + t.part_row_base) * 2;
        // The descriptor spans the rows of all tiles, which lie apart, and drops none: rows that a tile does not have
        // are left out by a branch.  An offset reaches 2^31 bytes: more slices of a node than any but a forced
        // division has.
        if (how == kRowsThrough && int64_t(last_tile + 1) * stride * (D * 4) >= int64_t(1) << 31) how = kRowsPlain;
        with_row_store(how, [&](auto h) __attribute__((always_inline)) {
            constexpr RowStore HOW = decltype(h)::value;
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                const int row = row0 + nt * 16 + l16;
                if (row < rows) {
                    const int tile = row / tile_rows;
                    const int64_t at = int64_t(tile) * stride + (row - tile * tile_rows) - (tile == last_tile ? last_back : 0);
#pragma unroll
                    for (int dt = 0; dt < CT; ++dt) {
                        const int64_t off = at * D + grp * 4 + dt * 16;
                        if constexpr (HOW == kRowsThrough) st16_rows<HOW>(rows_at(po, -1), int(off) * 4, st.o[nt][dt]);
                        else                               st16_partial<HOW>(po + off, st.o[nt][dt]);
                    }
                    if (grp == 0) st8_partial<HOW>(pml + at * 2, st.m[nt], st.l[nt]);
                }
            }
        });
    }
    __syncthreads();                        // every block has been read: the ring is free for the next task
}

template <int DT, int D>
__device__ __forceinline__ void run_tile(const PacParams &P, const DevTask &t, int head, char *lds, RowStore how)
{
    const int rows = t.n_req * P.group;
    if constexpr (D == 64) {            // row groups of 32: up to two, four, eight
        if (rows <= 64)       run_tile_of<DT, D, 2, 4>(P, t, head, lds, how);
        else if (rows <= 128) run_tile_of<DT, D, 2, 2>(P, t, head, lds, how);
        else                  run_tile_of<DT, D, 2, 1>(P, t, head, lds, how);
    } else {                            // a row group per wave, of 16 or of 32 rows
        if (rows <= 64) run_tile_of<DT, D, 1, 1>(P, t, head, lds, how);
        else            run_tile_of<DT, D, 2, 1>(P, t, head, lds, how);
    }
}

// Partial output reduction (Alg. 3), n-ary: one wave folds the partials of RPW consecutive query heads
// of one request (hq .. hq + RPW - 1, all of one KV head) in list order.  Partials are taken in chunks, the first fifteen
// of a list, then eight at a time: their loads are issued together, they are summed up against the maximum so far, and
// the sum is added to what the chunks before came to (by associativity of the reduction this equals any binary
// bracketing).  All forms of the reduction have the same chunks and the same rounding and agree bit for bit, but
// for fp16 of 64 channels: the forms with one row per wave multiply and round a value in one instruction, those with
// four rows in two (68 of 1064960 values differ, in their last bit).
//
constexpr int kFoldChunk = 8;

// A chunk of a row's partials.
template <int N, int CPL>
struct Chunk {
    float2 ml[N];
    float o[N][CPL];

    // those that exist
    template <class Rows>
    __device__ __forceinline__ void load(const MergeParams &P, const Rows &at, const int *rows, int cnt)
    {
#pragma unroll
        for (int j = 0; j < N; ++j) {
            ml[j] = float2{0.f, 0.f};
#pragma unroll
            for (int c = 0; c < CPL; ++c) o[j][c] = 0.f;
            if (j < cnt) at.load(P, rows[j], ml[j], o[j]);      // wave-uniform
        }
    }
    // every slot
    template <class Rows>
    __device__ __forceinline__ void load_all(const MergeParams &P, const Rows &at, const int *rows)
    {
#pragma unroll
        for (int j = 0; j < N; ++j) at.load(P, rows[j], ml[j], o[j]);
    }
    __device__ __forceinline__ float top(float m, int cnt) const
    {
#pragma unroll
        for (int j = 0; j < N; ++j)
            if (j < cnt) m = fmaxf(m, ml[j].x);
        return m;
    }
    // against a reference.  (fmaf written out here and in add_chunk: the compiler has no choice to make.)
    __device__ __forceinline__ void sum_up(int cnt, float reference, float &l, float (&sum)[CPL]) const
    {
        l = 0.f;
#pragma unroll
        for (int c = 0; c < CPL; ++c) sum[c] = 0.f;
#pragma unroll
        for (int j = 0; j < N; ++j)
            if (j < cnt) {
                const float w = weight(ml[j].x, reference);
                l = __builtin_fmaf(ml[j].y, w, l);
#pragma unroll
                for (int c = 0; c < CPL; ++c) sum[c] = __builtin_fmaf(o[j][c], w, sum[c]);
            }
    }
};

// What the chunks before came to, l and sum against m, and a chunk's sums against mm, the maximum so far.
template <int CPL>
__device__ __forceinline__ void add_chunk(float m, float &l, float (&sum)[CPL], float mm, float chunk_l, const float (&chunk_sum)[CPL])
{
    const float before = weight(m, mm);
    l = __builtin_fmaf(l, before, chunk_l);
#pragma unroll
    for (int c = 0; c < CPL; ++c) sum[c] = __builtin_fmaf(sum[c], before, chunk_sum[c]);
}

// A lane's channels of a finished row: normalised, rounded.
template <int DT, int CPL>
__device__ __forceinline__ void store_finished(char *out, float l, const float (&sum)[CPL])
{
    const float inv = 1.f / l;
    if constexpr (CPL == 1) {
        *reinterpret_cast<unsigned short *>(out) = static_cast<unsigned short>(pack2<DT>(sum[0] * inv, 0.f) & 0xFFFFu);
    } else {
#pragma unroll
        for (int c = 0; c < CPL; c += 2)
            *reinterpret_cast<unsigned int *>(out + c * 2) = pack2<DT>(sum[c] * inv, sum[c + 1] * inv);
    }
}

// The form inside the attention kernel (single-launch mode): one row per wave, each lane owns D / 64 channels of it, and
// every slot of a round is loaded: rows behind the end of a list read as row 0, which is valid memory, and the
// straight-line code keeps that kernel as it is.
template <int D>
struct DeliveredRows {
    static constexpr int CPL = D / 64;          // channels per lane: 1, 2 or 4
    int64_t head_base;
    int lane;

    // rows written by other workgroups of this launch
    __device__ __forceinline__ void load(const MergeParams &P, int entry, float2 &ml, float (&o)[CPL]) const
    {
        const int64_t prow = head_base + entry;
        const float *src = P.part_o + prow * D + lane * CPL;
        ml = ld8_device(P.part_ml + prow * 2);
        if constexpr (CPL == 1) {
            o[0] = __builtin_bit_cast(float, __hip_atomic_load(reinterpret_cast<const unsigned int *>(src),
                                                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
        } else {
#pragma unroll
            for (int c = 0; c < CPL; c += 2) {
                const float2 x = ld8_device(src + c);
                o[c] = x.x;
                o[c + 1] = x.y;
            }
        }
    }
};

template <int DT, int D>
__device__ __forceinline__ void merge_one(const MergeParams &P, int r, int hq, int wave_lane)
{
    constexpr int CPL = DeliveredRows<D>::CPL;
    const int head = hq / P.group, hj = hq - head * P.group;
    // The request's line: its number of partial rows and the first kInlineParts of them, read together
    // (no address waits for another read).  Lists of up to eight rows, and of up to kInlineParts, are
    // folded in one round of loads; what lies beyond comes from the CSR arrays, eight rows a round.
    const int32_t *line = P.req_inline + int64_t(r) * (kInlineParts + 1);
    const int total = line[0];
    int first[kInlineParts];
#pragma unroll
    for (int j = 0; j < kInlineParts; ++j) first[j] = line[1 + j];  // zero behind the end: a valid row
    const DeliveredRows<D> at{int64_t(head) * P.part_rows + hj, wave_lane};
    float M, L, acc[CPL];
    if (total <= kFoldChunk) {
        Chunk<kFoldChunk, CPL> x;
        x.load_all(P, at, first);
        x.sum_up(total, x.top(-INFINITY, total), L, acc);
    } else {
        Chunk<kInlineParts, CPL> x;
        const int cnt = total < kInlineParts ? total : kInlineParts;
        x.load_all(P, at, first);
        M = x.top(-INFINITY, cnt);
        x.sum_up(cnt, M, L, acc);
        if (total > kInlineParts) {
            const int32_t *list = P.req_part + P.req_part_off[r];
#pragma unroll 1
            for (int base = kInlineParts; base < total; base += kFoldChunk) {
                const int cnt = total - base < kFoldChunk ? total - base : kFoldChunk;
                int rows[kFoldChunk];
#pragma unroll
                for (int j = 0; j < kFoldChunk; ++j) rows[j] = list[base + (j < cnt ? j : 0)];
                Chunk<kFoldChunk, CPL> y;
                y.load_all(P, at, rows);
                const float mm = y.top(M, cnt);
                float l, sum[CPL];
                y.sum_up(cnt, mm, l, sum);
                add_chunk(M, L, acc, mm, l, sum);
                M = mm;
            }
        }
    }
    store_finished<DT>(static_cast<char *>(P.out) + ((int64_t(r) * P.h_q + hq) * D + wave_lane * CPL) * 2, L, acc);
}

// The reduction kernels.  A wave takes RPW = 256 / D consecutive query heads of a request where the rows of a KV head's
// group divide that evenly (else RPW = 1, as above): each lane owns four channels of one of the rows; they are
// neighbours in the partial arrays and in the output, so every load of partial rows is one full 1 KB instruction and a
// reduction costs half (a quarter for 64 channels) the memory instructions per row.  Large launches are bound by those: each
// takes a place in the CU's queue of memory instructions in flight whatever it moves.  For the same reason only the
// partials that exist are loaded.  Small launches are bound by the chain of dependent reads and by the code between them:
// merge_kernel has what is the same for the wave, the request's line and the addresses of its rows, read and worked out by
// the scalar unit, and reads rows sixteen to 23 beside the first fifteen.  Time against a form with all of that in vector
// registers and rows in rounds, whole steps of drawn plans: lists of up to eight rows, steps of 8 .. 16 us 0.986 (40
// plans, the best 0.956), 16 .. 32 us 0.990; 16 .. 23 rows 0.979 and 0.986 (the best 0.932); larger steps 0.997 .. 1.000.

// The rows of a wave and the place of its lanes in them.
template <int DT, int D, int RPW>
struct WaveRows {
    static constexpr int LPR = 64 / RPW;        // lanes per row
    static constexpr int CPL = D / LPR;         // channels per lane
    static_assert(CPL == 1 || CPL == 2 || CPL == 4, "channels per lane");
    int lane, row;                              // the lane's place in its row, which is row `row` of the wave
    uint32_t off_o, off_ml;                     // bytes behind the first of the wave's rows
    int64_t head_base;                          // the first of the wave's rows lies at head_base + an entry of the list
    char *out;

    __device__ __forceinline__ WaveRows(const MergeParams &P, int head, int r, int hj)
    {
        const int wave_lane = threadIdx.x & 63;
        lane = wave_lane % LPR;
        row = wave_lane / LPR;
        off_o = uint32_t(row * D + lane * CPL) * 4;
        off_ml = uint32_t(row) * 8;
        head_base = int64_t(head) * P.part_rows + hj;
        out = static_cast<char *>(P.out) + (int64_t(r) * P.h_q + int64_t(head) * P.group + hj) * (D * 2) + off_o / 2;
    }
    __device__ __forceinline__ void load(const MergeParams &P, int entry, float2 &ml, float (&o)[CPL]) const
    {
        const int64_t prow = head_base + entry;
        ml = *reinterpret_cast<const float2 *>(reinterpret_cast<const char *>(P.part_ml + prow * 2) + off_ml);
        const char *src = reinterpret_cast<const char *>(P.part_o + prow * D) + off_o;
        if constexpr (CPL == 1) {
            o[0] = *reinterpret_cast<const float *>(src);
        } else if constexpr (CPL == 2) {
            const float2 x = *reinterpret_cast<const float2 *>(src);
            o[0] = x.x;
            o[1] = x.y;
        } else {
            const f32x4 x = *reinterpret_cast<const f32x4 *>(src);
#pragma unroll
            for (int c = 0; c < 4; ++c) o[c] = x[c];
        }
    }
    __device__ __forceinline__ void store(float l, const float (&sum)[CPL]) const { store_finished<DT>(out, l, sum); }
};

// blockIdx.x is the KV head.  Workgroups are dealt to the eight XCDs in turn, here and in the attention kernel, so
// with eight heads the rows of a head are read through the L2 that holds them.  In order of requests that is so only
// where the rows of a request fill eight workgroups.  us per step, by request / by head: a lone request of
// 8191 tokens with 64 / 8 heads 16.4 / 14.5, with 8 / 8 heads 15.5 / 13.7, with 28 / 4 14.9 / 14.5; a 4096-token root under
// 16 requests with 64 / 8 heads 19.4 / 16.5, with 32 / 4 16.2 / 15.5; 32 / 8 heads of 128 channels, where both are so, alike.
// Drawn plans, time by head over by request: 193 with KV heads that eight divides 0.991 (0.858 .. 1.013), 7 with four
// heads 0.988, 51 with one head, for which the order is the same, 1.002 (0.987 .. 1.020).
//
// LONG: what of a list follows its first fifteen rows.  0: nothing, in no list of the plan.  1: rows sixteen to 23 are read
// beside the first fifteen.  2: one after the other, for large launches, most of whose lists are short as a rule: 1 takes 110
// registers, 2 at most 98, of which a SIMD holds a wave more.  us, reduction alone, 0.1 % of the lists of 20 rows
// and the others of three, 1 / 2: 1040 requests with 32 / 8 heads 11.6 / 10.8, with 28 / 4 15.1 / 11.7, 2080 with 32 / 8
// 20.2 / 18.8; half of them of 20 rows 29.9 / 30.5, 29.4 / 29.7, 77.6 / 78.8; all of 16 rows and 28 / 4 heads 37.3 / 39.7.
// Lists of more than fifteen rows have a branch and a Chunk of their own: with the chunk of the lists of nine to fifteen rows, and its
// loads under a condition, both forms took up to 165 registers and three waves fit on a SIMD (13.3, 17.5, 22.9 in the
// first three of these cases).
template <int DT, int D, int RPW, int LONG>
__global__ void __launch_bounds__(kMergeWaves * 64) merge_kernel(const MergeParams P)
{
    using W = WaveRows<DT, D, RPW>;
    constexpr int CPL = W::CPL;
    const int per_req = P.group / RPW;          // the launch has checked that RPW divides the group size
    const int unit = (blockIdx.z * gridDim.y + blockIdx.y) * kMergeWaves + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (unit >= P.num_requests * per_req) return;
    const int r = unit / per_req;
    const W at(P, blockIdx.x, r, (unit - r * per_req) * RPW);
    // see merge_one
    const int32_t *line = P.req_inline + int64_t(r) * (kInlineParts + 1);
    const int total = line[0], list_off = LONG ? P.req_part_off[r] : 0;
    int first[kInlineParts];
#pragma unroll
    for (int j = 0; j < kInlineParts; ++j) first[j] = line[1 + j];
#pragma unroll
    for (int j = 0; j < kInlineParts; ++j) asm volatile("" : : "s"(first[j]));  // the line is read whole, not its second half when it is wanted
    if constexpr (LONG != 0) asm volatile("" : : "s"(list_off));
    float M, L, acc[CPL];
    if (total <= kFoldChunk) {
        Chunk<kFoldChunk, CPL> x;
        x.load(P, at, first, total);
        x.sum_up(total, x.top(-INFINITY, total), L, acc);
    } else if (LONG == 0 || total <= kInlineParts) {
        Chunk<kInlineParts, CPL> x;
        x.load(P, at, first, total);
        x.sum_up(total, x.top(-INFINITY, total), L, acc);
    } else {
        const int32_t *list = P.req_part + list_off;
        auto load_next = [&](Chunk<kFoldChunk, CPL> &y, int base) {
            int rows[kFoldChunk];
#pragma unroll
            for (int j = 0; j < kFoldChunk; ++j) rows[j] = list[base + j];  // behind the list: what follows it in the metadata, unused
            y.load(P, at, rows, total - base);
        };
        auto add_next = [&](const Chunk<kFoldChunk, CPL> &y, int cnt) {
            const float mm = y.top(M, cnt);
            float l, sum[CPL];
            y.sum_up(cnt, mm, l, sum);
            add_chunk(M, L, acc, mm, l, sum);
            M = mm;
        };
        int base = kInlineParts;
        Chunk<kInlineParts, CPL> x;
        x.load_all(P, at, first);
        if constexpr (LONG == 1) {
            Chunk<kFoldChunk, CPL> y;
            load_next(y, base);
            M = x.top(-INFINITY, kInlineParts);
            x.sum_up(kInlineParts, M, L, acc);
            add_next(y, total - base);
            base += kFoldChunk;
        } else {
            M = x.top(-INFINITY, kInlineParts);
            x.sum_up(kInlineParts, M, L, acc);
        }
#pragma unroll 1
        for (; base < total; base += kFoldChunk) {
            Chunk<kFoldChunk, CPL> y;
            load_next(y, base);
            add_next(y, total - base);
        }
    }
    at.store(L, acc);
}

// The same for plans with lists of 24 rows and more whose launch is small (split_waves), which is bound by its chain of
// dependent reads: one wave makes four or five for a list of 32 (line, fifteen rows, CSR entries and eight rows, twice).
// Here WAVES waves take a chunk each, wave 0 the first, after two dependent reads (line, rows), and their sums meet in LDS.
// The references of all rows up to the end of its chunk, whose maximum a chunk's sum refers to, are read by every wave, a
// row per lane and each once.  us per step, one wave / split: a lone request of 8191 tokens, 32 / 8 heads, 32 partials 14.9 / 13.5;
// one KV head, a two-level tree of three requests, 58 partials 21.6 / 13.4; 24 requests, 48 partials 31.6 / 27.2.  Measured
// and dropped: the sums of the waves against references of their own (12.9, but the single launch, which has to round
// alike, then took up to 16 % longer); the rows handed over through LDS as they are and folded there (14.4).
template <int DT, int D, int RPW, int WAVES>
__global__ void __launch_bounds__(WAVES * 64) merge_split_kernel(const MergeParams P)
{
    using W = WaveRows<DT, D, RPW>;
    constexpr int CPL = W::CPL;
    __shared__ float sums[WAVES - 1][CPL + 2][64];
    const int per_req = P.group / RPW;
    const int unit = blockIdx.z * gridDim.y + blockIdx.y;
    if (unit >= P.num_requests * per_req) return;
    const int r = unit / per_req;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), wave_lane = threadIdx.x & 63;
    const W at(P, blockIdx.x, r, (unit - r * per_req) * RPW);
    const int32_t *line = P.req_line + int64_t(r) * split_line_words(WAVES);
    const int total = line[0];
    const int32_t *list = line + 1;
    float M, L, acc[CPL];                               // the wave's chunk; wave 0: all chunks so far
    float top = -INFINITY;                              // maximum of the references of rows 0 .. seen - 1
    int seen = 0;

    // rows begin .. begin + cnt - 1 of the list, cnt at most N
    auto fold = [&](int begin, int cnt, auto width) {
        constexpr int N = decltype(width)::value;
        int rows[N];
#pragma unroll
        for (int j = 0; j < N; ++j) rows[j] = list[begin + j];      // behind the list: see merge_kernel
        Chunk<N, CPL> x;
        x.load(P, at, rows, cnt);
#pragma unroll 1
        for (int j = seen + at.lane; j < begin + cnt; j += W::LPR) top = fmaxf(top, P.part_ml[(at.head_base + at.row + list[j]) * 2]);
#pragma unroll
        for (int d = 1; d < W::LPR; d *= 2) top = fmaxf(top, __shfl_xor(top, d));
        seen = begin + cnt;
        M = top;
        x.sum_up(cnt, M, L, acc);
    };
    int base = kInlineParts;                            // first row of wave 1's chunk
    if (wave == 0) fold(0, kInlineParts < total ? kInlineParts : total, std::integral_constant<int, kInlineParts>{});
#pragma unroll 1
    for (;;) {                                          // one round, but for lists of more than split_rows(WAVES)
        if (wave > 0) {
            const int begin = base + (wave - 1) * kFoldChunk, cnt = total - begin < kFoldChunk ? total - begin : kFoldChunk;
            if (cnt > 0) {
                fold(begin, cnt, std::integral_constant<int, kFoldChunk>{});
                float (*put)[64] = sums[wave - 1];
                put[CPL][wave_lane] = L;
                put[CPL + 1][wave_lane] = M;
#pragma unroll
                for (int c = 0; c < CPL; ++c) put[c][wave_lane] = acc[c];
            }
        }
        __syncthreads();
        if (wave == 0) {
#pragma unroll
            for (int w = 0; w < WAVES - 1; ++w) {
                if (base + w * kFoldChunk >= total) break;
                const float m = sums[w][CPL + 1][wave_lane];
                float sum[CPL];
#pragma unroll
                for (int c = 0; c < CPL; ++c) sum[c] = sums[w][c][wave_lane];
                add_chunk(M, L, acc, m, sums[w][CPL][wave_lane], sum);
                M = m;
            }
        }
        base += (WAVES - 1) * kFoldChunk;
        if (base >= total) break;
        list = P.req_part + P.req_part_off[r];
        __syncthreads();                                // the sums of this round have been read
    }
    if (wave == 0) at.store(L, acc);
}

// ---- single-launch mode: the reduction inside the attention launch (Sec. 4.3, parallel reduction) ----
//
// Every task delivers one partial result to each of its requests.  arrive[head][request] counts them
// (device-scope atomics); the delivery that completes a request's reduction list (its length is the
// first word of the request's line) makes the delivering workgroup reduce that request's rows of this
// KV head right away, and put the counter back to zero for the next launch.  In this mode partial rows
// are written and read with device-coherent accesses (st8_device / ld8_device), so no cache has to be
// written back or invalidated: every wave that has stored rows waits until its stores have been acknowledged
// (they are then visible device-wide), and only then is the delivery counted; the workgroup that sees the
// last count reads the rows after that.  (Fences at device scope instead, with plain accesses, cost a write-back and an
// invalidation of the whole L2 per task: measured, several times the launch they were to save.)
//
// expect(): request i of the task and the length of its list, read ahead of the wait for the stores so that the
// two reads travel beside them.  deliver(): counts; true for the delivery that completes the list.
__device__ __forceinline__ int2 expect(const PacParams &P, const DevTask &t, int i)
{
    const int req = t.single_req >= 0 ? t.single_req : P.node_q[t.q_off + i];
    return int2{req, P.merge.req_inline[int64_t(req) * (kInlineParts + 1)]};
}
__device__ __forceinline__ bool deliver(const PacParams &P, int head, int2 expected)
{
    int32_t *c = P.arrive + int64_t(head) * P.merge.num_requests + expected.x;
    const int old = __hip_atomic_fetch_add(c, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (old + 1 != expected.y) return false;
    __hip_atomic_store(c, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);   // nobody else counts on it in this launch
    return true;
}

// Waits until the wave's stores have been acknowledged.  No barrier or fence at workgroup scope does that on
// this target: they order LDS, and the wave's own path to the vector cache keeps global stores in order for
// the workgroup; rows that another workgroup will read need the wait of every wave that has stored some.
__device__ __forceinline__ void stores_acknowledged() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// A task that the whole workgroup ran (every thread calls this after the task).  Inline without fail, as all
// device functions here: one real call makes the compiler keep the kernel's parameters in scratch memory.
template <int DT, int D>
__device__ __forceinline__ void task_delivered_by_workgroup(const PacParams &P, const DevTask &t, int head, char *lds_raw, int waves)
{
    int *count = reinterpret_cast<int *>(lds_raw), *ready = count + 1;
    const bool mine = int(threadIdx.x) < t.n_req;
    int2 expected{0, 0};
    if (mine) expected = expect(P, t, threadIdx.x);
    stores_acknowledged();              // the rows of a task may come from every wave (dense and tile path)
    __syncthreads();                    // ... and all have waited when a thread counts; LDS is free
    if (threadIdx.x == 0) *count = 0;
    __syncthreads();
    if (mine && deliver(P, head, expected)) ready[atomicAdd(count, 1)] = expected.x;
    __syncthreads();
    const int n = *count * P.group;
    if (n > 0) {
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");     // no load of a partial row moves above the count
        const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
#pragma unroll 1
        for (int i = wave; i < n; i += waves) {
            const int k = i / P.group;
            merge_one<DT, D>(P.merge, ready[k], head * P.group + (i - k * P.group), threadIdx.x & 63);
        }
    }
    __syncthreads();                    // the list is done with before LDS is used again
}

// A task that one wave ran on its own (no barrier: the other waves are inside other tasks).
template <int DT, int D>
__device__ __forceinline__ void task_delivered_by_wave(const PacParams &P, const DevTask &t, int head)
{
    const int lane = threadIdx.x & 63;
    int2 expected{0, 0};
    if (lane < t.n_req) expected = expect(P, t, lane);
    stores_acknowledged();
    const bool last = lane < t.n_req && deliver(P, head, expected);
    unsigned long long ready = __ballot(last);
    if (ready == 0) return;
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
#pragma unroll 1
    while (ready) {
        const int src = __builtin_ctzll(ready);
        ready &= ready - 1;
        const int r = __shfl(expected.x, src);
#pragma unroll 1
        for (int hj = 0; hj < P.group; ++hj) merge_one<DT, D>(P.merge, r, head * P.group + hj, lane);
    }
}

// WIDE: a ring of dynamic LDS (kRingBytes, TilePath::kRingBytes).  The dense and tile paths XOR channel
// tiles into operand addresses, so the ring must start on a 512-byte boundary (no static LDS there).
extern __shared__ __attribute__((aligned(1024))) char dyn_lds[];

// FUSED: with the code of the single-launch mode (used if P.arrive).  The kernels without it are shorter and
// need fewer registers, which shows where a step is a few dozen microseconds (both builds in turn on one card,
// whose runs differ by 0.1-0.7 %): 32 layers of document questions 842 -> 833 us, a six-level tree with one KV
// head 39.7 -> 39.1, a lone request 15.1 -> 14.8, documents of 64 channels 75.8 -> 74.9, three-level documents
// 161.5 -> 160.2; nothing on steps of 250 us and more.  Only the tile path of 256 channels was allocated worse without it (three-level
// documents 289 -> 299 us), so its one kernel serves both modes (one_kernel).
constexpr bool one_kernel(int form, int d) { return form == kFormWide && d == 256; }
// TURNS: stream tasks that alone read their slice go round the KV heads (head_of); two launches, up to 128 channels.  In a
// kernel of its own: a choice at run time costs small plans, which do not make it, about 1 us.
template <int DT, int FORM, int D, bool TURNS, bool FUSED>
__global__ void __launch_bounds__(kernel_waves(FORM, D) * 64, D > 128 ? 1 : 2)
pac_kernel(const PacParams params)     // 256 channels: two blocks of K and V in registers need a wave per SIMD
{
    PacParams P = params;
    if constexpr (!FUSED) P.arrive = nullptr;
    // kFormWide: the dense path (128 channels, eight waves) or the tile path (64 and 256 channels)
    constexpr bool WIDE = FORM == kFormWide, DENSE = WIDE && D == kHeadDim, TILES = WIDE && D != kHeadDim;
    constexpr bool FINISH = FORM == kFormFinish;
    constexpr int W = kernel_waves(FORM, D);
    char *lds;
    if constexpr (WIDE) {
        lds = dyn_lds;
    } else {
        __shared__ __attribute__((aligned(16))) char static_lds[merge_bytes(kNarrowWaves, stream_tiles(D), D) + kNarrowWaves * solo_stage_bytes(D)];
        lds = static_lds;
    }
    const int head = blockIdx.x % P.h_kv;
    const int slot = blockIdx.x / P.h_kv;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // staging area of this wave for tasks it runs on its own: behind the area in which a team merges its
    // states (in the wide variant both lie in the ring, which only dense tasks fill)
    static_assert(merge_bytes(kWideWaves, 1, kHeadDim) + kWideWaves * solo_stage_bytes(kHeadDim) <= kRingBytes, "staging areas fit the ring");
    if constexpr (TILES)
        static_assert(merge_bytes(W, stream_tiles(D), D) + W * solo_stage_bytes(D) <= TilePath<D>::kRingBytes,
                      "staging areas fit the ring");
    char *stage = lds + merge_bytes(W, DENSE ? 1 : stream_tiles(D), D) + wave * solo_stage_bytes(D);
    // How dense and tile tasks store their rows with tasks to follow, and as the last of the workgroup (in
    // single-launch mode all alike).
    constexpr bool ARRIVES = FUSED && !one_kernel(FORM, D);             // P.arrive for certain
    const bool many_rows = int64_t(P.part_rows) * P.h_kv * (D * 4) > kEarlyThroughBytes;
    const RowStore early = ARRIVES || P.arrive ? kRowsCoherent : many_rows ? kRowsThrough : kRowsPlain;
    const RowStore late = ARRIVES || P.arrive ? kRowsCoherent : last_rows_through(P.h_kv) ? kRowsThrough : kRowsPlain;
    // The KV head for which the workgroup runs record i.  Where the heads of a token lie side by side ([token][head]
    // pools), the rows of one head meet a subset of the memory channels, and not all heads as many: with a head
    // of its own a workgroup of a slow head ends up to 20 % after the others.  In plans whose rows go out finished the
    // workgroups, and with TURNS those of larger plans in two launches, therefore take record i for the head i places on: every (record, head) is still run once, by the
    // workgroups that run record i, and the slow heads are spread over all of them.  (Slices that other tasks read as
    // well keep their head, whose L2 may hold them.)  Drawn plans of 100 .. 500 unshared contexts, time against fixed heads,
    // [token][head] pools: 64 channels 8 plans 0.816 (0.756 .. 0.908), 128 channels and four or eight heads 30 plans 0.902
    // (0.877 .. 0.961), 256 channels 11 plans 0.961; one head, or [head][token] pools, 142 plans 0.997 (0.985 .. 1.005).
    // 256 contexts of 100 .. 4000 tokens, 28 / 4 heads 199.8 -> 185.5 us.
    auto head_of = [&](const DevTask &t, int i) __attribute__((always_inline)) {
        if constexpr (FINISH || TURNS) {
            if (t.flags & kTaskReadOnce) return int(uint32_t(head + i) % uint32_t(P.h_kv));
        }
        return head;
    };
    // Runs the task records recs[t0 .. t1).  Tasks of more than 16 rows take the dense path (wide variant
    // only).  Tasks of at most 16 rows take the stream path, as a rule with all waves of the workgroup
    // as one team.  Runs of two or more short ones are handed out one wave each through a counter in
    // LDS: the latencies of a short task (descriptor, query rows, page ids, first blocks, merge of a
    // team) then overlap with the other tasks' instead of adding up.  In a slot's list the plan marks
    // such runs (they are neighbours there, the list being sorted by cost); an entry of the run-time
    // queue with several tasks is one such run.  `more`: other records may follow these.
    auto run_tasks = [&](const DevTask *recs, int t0, int t1, bool marked, bool more) __attribute__((always_inline)) {
        int i = t0;
#pragma unroll 1
        while (i < t1) {
            const DevTask t = recs[i];
            const int n = marked ? t.solo_run : t1 - i;
            if (n >= 2) {
                // Wave w starts with task w of the run, every further task is the next one nobody has
                // taken.  The run is in order of decreasing cost and the first waves are the older ones
                // of the pairs that share a SIMD, which the hardware serves first (measured: in a run
                // they move two to three times the tokens of their partners), so the longest tasks start
                // on the fastest waves.
                int *next = reinterpret_cast<int *>(lds);
                if (threadIdx.x == 0) *next = W;
                __syncthreads();
                int k = wave;
#pragma unroll 1
                while (k < n) {
                    const DevTask mine = recs[i + k];
                    const int own = head_of(mine, i + k);
                    if (mine.flags & kTaskReadOnce) run_stream<DT, true, 1, 1, D, FINISH>(P, mine, own, lds, 0, stage);
                    else                run_stream<DT, false, 1, 1, D, FINISH>(P, mine, own, lds, 0, stage);
                    if constexpr (FUSED)
                        if (P.arrive) task_delivered_by_wave<DT, D>(P, mine, head);
                    k = 0;
                    if ((threadIdx.x & 63) == 0) k = atomicAdd(next, 1);
                    k = __builtin_amdgcn_readfirstlane(k);
                }
                __syncthreads();                // the counter is done with before LDS is used again
                i += n;
            } else {
                bool tiles = false;             // sibling row tiles packed into one task
                if constexpr (TILES) tiles = (t.flags & kTaskTiles) != 0;
                const RowStore how = i + 1 < t1 || more ? early : late;
                if (tiles) {
                    if constexpr (TILES) run_tile<DT, D>(P, t, head, lds, how);
                } else if (t.n_req * P.group <= 16) {
                    const int own = head_of(t, i);
                    if (t.flags & kTaskReadOnce) run_stream<DT, true, 1, W, D, FINISH>(P, t, own, lds, wave);
                    else             run_stream<DT, false, 1, W, D, FINISH>(P, t, own, lds, wave);
                }
                else if constexpr (DENSE) run_dense32<DT>(P, t, head, lds, how);
                else if constexpr (stream_tiles(D) == 2 && !FINISH) {   // 17 .. 32 rows of 64 channels: two row tiles
                    if (t.flags & kTaskReadOnce) run_stream<DT, true, 2, W, D>(P, t, head_of(t, i), lds, wave);
                    else             run_stream<DT, false, 2, W, D>(P, t, head, lds, wave);
                }
                if constexpr (FUSED)
                    if (P.arrive) task_delivered_by_workgroup<DT, D>(P, t, head, lds, W);
                ++i;
            }
        }
    };

    // Static schedule: the slot's own list, once.  Run-time queue: entry `slot` is this workgroup's
    // first; every further one is the next entry nobody has taken, fetched by one thread (one atomic)
    // and spread to the waves through LDS.  Every path through run_tasks ends with a barrier behind
    // its last LDS access, so the word can be written right away; the second barrier keeps the next
    // task's block copies from overwriting it before everyone has read it.
    const bool queued = P.queue_off != nullptr;
    const bool fetching = queued && P.num_entries > P.num_slots;        // else: an entry per workgroup at most
    const DevTask *recs = queued ? P.queue_recs : P.slot_recs;
    const int32_t *off = queued ? P.queue_off : P.slot_off;
    const int limit = queued ? P.num_entries : slot + 1;
    int32_t *taken = P.counters + 2 * head, *finished = taken + 1;
    int *word = reinterpret_cast<int *>(lds);
    int e = slot;
#pragma unroll 1
    while (e < limit) {
        run_tasks(recs, off[e], off[e + 1], !queued, fetching);
        if (!fetching) break;
        // taken when the workgroup is free, not ahead of time: an entry reserved early would wait for
        // the end of a long task while other workgroups idle
        if (threadIdx.x == 0) *word = P.num_slots + atomicAdd(taken, 1);
        __syncthreads();
        e = __builtin_amdgcn_readfirstlane(*word);
        __syncthreads();
    }
    // the last workgroup of this KV head to get here leaves the counters at zero for the next launch
    if (fetching && threadIdx.x == 0 && atomicAdd(finished, 1) == P.num_slots - 1) {
        atomicExch(taken, 0);
        atomicExch(finished, 0);
    }
}

// Read-only streaming kernel (measurement support): every thread sums 16-byte loads; a workgroup takes
// whole 4 KB chunks, chunk c of the walk being chunk perm(c) of the buffer, so that the order can be
// that of a paged pool.  One value per workgroup is written so that the loads cannot be dropped.
template <bool ONCE>
__global__ void __launch_bounds__(256) stream_read_kernel(const char *buf, uint64_t chunks, uint64_t mult,
                                                          uint32_t *sink)
{
    u32x4 acc = {0u, 0u, 0u, 0u};
    for (uint64_t c = blockIdx.x; c < chunks; c += gridDim.x) {
        const uint64_t at = (c * mult) & (chunks - 1);          // chunks is a power of two, mult odd: a permutation
        const char *p = buf + at * 4096 + threadIdx.x * 16;
        const u32x4 x = ONCE ? ld16_once(p) : ld16(p);
        acc ^= x;
    }
    const uint32_t v = acc[0] ^ acc[1] ^ acc[2] ^ acc[3];
    if (v == 0x9E3779B9u && threadIdx.x == 0) sink[blockIdx.x] = v;       // practically never: keeps the loads alive
}

}  // namespace

// Scratch for callers that cannot provide a workspace (codec_decode_attention_static): partial outputs
// and their softmax statistics of one decode call.  Every GPU the library is loaded on holds one copy
// of this array at an address of its own until the process ends.  In host code the name below is only a
// handle for hipGetSymbolAddress; kernels get the address that call returns, as an ordinary argument.
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

// dynamic LDS of the forms with the dense and the tile path
template <int D>
constexpr int wide_lds_bytes()
{
    if constexpr (D == kHeadDim) return kRingBytes;
    else                         return TilePath<D>::kRingBytes;
}

int static_scratch_address(void **ptr)
{
    // one lookup per device, with that device current; the table is filled under a lock and read-only after
    constexpr int kMaxDevices = 64;
    static void *address[kMaxDevices] = {};
    static std::mutex lock;
    int dev = -1;
    if (hipError_t e = hipGetDevice(&dev)) return int(e);
    if (dev < 0 || dev >= kMaxDevices) return int(hipErrorInvalidDevice);
    std::lock_guard<std::mutex> guard(lock);
    if (!address[dev]) {
        void *p = nullptr;
        if (hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch))) return int(e);
        address[dev] = p;
    }
    *ptr = address[dev];
    return 0;
}

// The wide variant needs more dynamic LDS than the 64 KB a kernel gets by default.  Set once per
// process and device, outside any stream capture (codec_plan_upload calls this).
int prepare_kernels()
{
    constexpr int kMaxDevices = 64;
    static bool done[kMaxDevices] = {};
    static std::mutex lock;
    int dev = -1;
    if (hipError_t e = hipGetDevice(&dev)) return int(e);
    if (dev < 0 || dev >= kMaxDevices) return int(hipErrorInvalidDevice);
    std::lock_guard<std::mutex> guard(lock);
    if (done[dev]) return 0;
    struct Kernel { const void *kernel; int bytes; };
    auto wide = [](auto dt, auto d, auto fused) {
        constexpr int D = decltype(d)::value;
        return Kernel{reinterpret_cast<const void *>(pac_kernel<decltype(dt)::value, kFormWide, D, false, decltype(fused)::value>), wide_lds_bytes<D>()};
    };
    auto turns = [](auto dt, auto d) {
        constexpr int D = decltype(d)::value;
        return Kernel{reinterpret_cast<const void *>(pac_kernel<decltype(dt)::value, kFormWide, D, true, false>), wide_lds_bytes<D>()};
    };
    using f16 = std::integral_constant<int, CODEC_DTYPE_FP16>;
    using b16 = std::integral_constant<int, CODEC_DTYPE_BF16>;
    using d64 = std::integral_constant<int, 64>;
    using d128 = std::integral_constant<int, 128>;
    using d256 = std::integral_constant<int, 256>;
    using no = std::false_type;
    using yes = std::true_type;
    const Kernel kernels[] = {
        wide(f16{}, d128{}, no{}), wide(b16{}, d128{}, no{}), wide(f16{}, d128{}, yes{}), wide(b16{}, d128{}, yes{}),
        wide(f16{}, d64{}, no{}),  wide(b16{}, d64{}, no{}),  wide(f16{}, d64{}, yes{}),  wide(b16{}, d64{}, yes{}),
        wide(f16{}, d256{}, yes{}), wide(b16{}, d256{}, yes{}),
        turns(f16{}, d64{}), turns(b16{}, d64{}), turns(f16{}, d128{}), turns(b16{}, d128{}),
    };
    for (const auto &k : kernels)
        if (hipError_t e = hipFuncSetAttribute(k.kernel, hipFuncAttributeMaxDynamicSharedMemorySize, k.bytes)) return int(e);
    done[dev] = true;
    return 0;
}

template <int DT, int D>
void launch_pac_of(const PacParams &p, dim3 grid, bool wide, bool turns, hipStream_t s)
{
    constexpr bool kTurns = D <= 128;

    const bool fused = p.arrive != nullptr;
    constexpr bool kOne = one_kernel(kFormWide, D);
    const dim3 block((wide ? kernel_waves(kFormWide, D) : kNarrowWaves) * 64);
    const size_t lds = wide ? wide_lds_bytes<D>() : 0;
    if (!p.part_o)          hipLaunchKernelGGL((pac_kernel<DT, kFormFinish, D, false, false>), grid, block, lds, s, p);
    else if (wide && fused) hipLaunchKernelGGL((pac_kernel<DT, kFormWide, D, false, true>), grid, block, lds, s, p);
    else if (wide && turns) hipLaunchKernelGGL((pac_kernel<DT, kFormWide, D, kTurns, kOne>), grid, block, lds, s, p);
    else if (wide)          hipLaunchKernelGGL((pac_kernel<DT, kFormWide, D, false, kOne>), grid, block, lds, s, p);
    else if (fused)         hipLaunchKernelGGL((pac_kernel<DT, kFormNarrow, D, false, true>), grid, block, lds, s, p);
    else if (turns)         hipLaunchKernelGGL((pac_kernel<DT, kFormNarrow, D, kTurns, false>), grid, block, lds, s, p);
    else                    hipLaunchKernelGGL((pac_kernel<DT, kFormNarrow, D, false, false>), grid, block, lds, s, p);
}

int launch_pac(const PacParams &p, int dtype, int head_dim, int num_slots, int max_rows_in_plan, bool tiles, bool turns, void *stream)
{
    if (head_dim != 64 && head_dim != 128 && head_dim != 256) return int(hipErrorInvalidValue);
    // all task shapes: dense tasks with 128 channels, packed row tiles with 64 and 256
    const bool wide = head_dim == kHeadDim ? max_rows_in_plan > 16 : tiles;
    // the planner never builds a plan with more rows per task than the kernel runs
    if (!wide && max_rows_in_plan > 16 * stream_tiles(head_dim)) return int(hipErrorInvalidValue);
    if (!p.part_o && (wide || max_rows_in_plan > 16)) return int(hipErrorInvalidValue);
    const dim3 grid(unsigned(num_slots) * unsigned(p.h_kv));
    hipStream_t s = static_cast<hipStream_t>(stream);
    const bool half = dtype == CODEC_DTYPE_FP16;
    if (head_dim == 64)       half ? launch_pac_of<CODEC_DTYPE_FP16, 64>(p, grid, wide, turns, s) : launch_pac_of<CODEC_DTYPE_BF16, 64>(p, grid, wide, turns, s);
    else if (head_dim == 128) half ? launch_pac_of<CODEC_DTYPE_FP16, 128>(p, grid, wide, turns, s) : launch_pac_of<CODEC_DTYPE_BF16, 128>(p, grid, wide, turns, s);
    else                      half ? launch_pac_of<CODEC_DTYPE_FP16, 256>(p, grid, wide, false, s) : launch_pac_of<CODEC_DTYPE_BF16, 256>(p, grid, wide, false, s);
    return int(hipGetLastError());
}

int launch_stream_read(const void *buf, uint64_t chunks, uint64_t mult, int once, int blocks, void *sink, void *stream)
{
    hipStream_t s = static_cast<hipStream_t>(stream);
    const char *b = static_cast<const char *>(buf);
    uint32_t *k = static_cast<uint32_t *>(sink);
    if (once) hipLaunchKernelGGL(stream_read_kernel<true>, dim3(unsigned(blocks)), dim3(256), 0, s, b, chunks, mult, k);
    else      hipLaunchKernelGGL(stream_read_kernel<false>, dim3(unsigned(blocks)), dim3(256), 0, s, b, chunks, mult, k);
    return int(hipGetLastError());
}

template <int DT, int D>
int launch_merge_of(const MergeParams &p, hipStream_t s)
{
    // a wave reduces 256 / D rows at a time where the rows of a KV head's group divide that evenly
    constexpr int kWide = 256 / D;
    const bool wide = kWide > 1 && p.group % kWide == 0;
    const int units = p.num_requests * (p.group / (wide ? kWide : 1));     // per KV head
    constexpr unsigned kMaxY = 32768;
    auto launch = [&](auto kernel, int units_of, int waves) {               // of a workgroup
        const unsigned groups = unsigned((units + units_of - 1) / units_of), y = groups < kMaxY ? groups : kMaxY;
        const dim3 grid(unsigned(p.h_q / p.group), y, (groups + y - 1) / y), block(waves * 64);
        hipLaunchKernelGGL(kernel, grid, block, 0, s, p);
    };
    auto split = [&](auto waves) {
        constexpr int W = decltype(waves)::value;
        if (wide) launch(merge_split_kernel<DT, D, kWide, W>, 1, W);
        else      launch(merge_split_kernel<DT, D, 1, W>, 1, W);
    };
    auto one = [&](auto form) {
        constexpr int LONG = decltype(form)::value;
        if (wide) launch(merge_kernel<DT, D, kWide, LONG>, kMergeWaves, kMergeWaves);
        else      launch(merge_kernel<DT, D, 1, LONG>, kMergeWaves, kMergeWaves);
    };
    switch (p.split_waves) {
    case 0: one(std::integral_constant<int, 0>{}); break;
    case 1: one(std::integral_constant<int, 1>{}); break;
    case 2: one(std::integral_constant<int, 2>{}); break;
    case 4: split(std::integral_constant<int, 4>{}); break;
    case 8: split(std::integral_constant<int, 8>{}); break;
    default: return int(hipErrorInvalidValue);
    }
    return int(hipGetLastError());
}

int launch_merge(const MergeParams &p, int dtype, int head_dim, void *stream)
{
    hipStream_t s = static_cast<hipStream_t>(stream);
    const bool half = dtype == CODEC_DTYPE_FP16;
    if (head_dim == 64)  return half ? launch_merge_of<CODEC_DTYPE_FP16, 64>(p, s) : launch_merge_of<CODEC_DTYPE_BF16, 64>(p, s);
    if (head_dim == 128) return half ? launch_merge_of<CODEC_DTYPE_FP16, 128>(p, s) : launch_merge_of<CODEC_DTYPE_BF16, 128>(p, s);
    if (head_dim == 256) return half ? launch_merge_of<CODEC_DTYPE_FP16, 256>(p, s) : launch_merge_of<CODEC_DTYPE_BF16, 256>(p, s);
    return int(hipErrorInvalidValue);
}

}  // namespace codec
