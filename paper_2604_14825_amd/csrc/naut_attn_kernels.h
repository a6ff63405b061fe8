// naut_attn_kernels.h -- the fused attention forward kernels for gfx950 (MI355X) and their launcher.
//
// Included by naut_attn.hip (the C ABI, which only declares the launcher instantiations) and by
// naut_attn_inst.hip (compiled once per storage-type pair, which defines them): splitting the
// instantiations over translation units lets them compile in parallel.
//
// One kernel computes O = softmax(scale * Q K^T + causal mask) V for a
// (batch, head, query tile) per work-group; two kernels share the formulation
// below and are picked per shape (pick_form): kernel 1 (this file; the smallest and shortest
// launches, and heads wider than 128) and kernel 2 (naut_attn_pipe.h, software-pipelined over 32-key blocks, in
// four forms).  The reductions over the key
// axis (row max, row sum, weighted sum of V) are fused with the rolling-update
// scheme of Section 4.2/4.3 of the paper: a running maximum m and running sum l
// are kept per query, and whenever m grows the partial results are repaired by
// the factor exp2(m_old - m_new).  The S x S scores never leave registers.
// Hand-applied rewrites (table of Section 5): scale*log2(e) folded into one
// constant, exp -> exp2, and a single division by l in the epilogue instead of
// one per step.
//
// Work decomposition (bi-level tiling, Section 4.2): outer loops (batch, head,
// query tile) -> work-groups; inner tile = 128 or 256 queries x 64 keys.  A
// wavefront owns 32 (or 64) queries.  Per key tile and wavefront:
//
//   S^T[key][query] = K_tile . Q^T     v_mfma_f32_32x32x16 (A = K from LDS, B = Q in registers)
//   online softmax over keys           each lane owns ONE query (column) and 16 keys per 32-key block,
//                                      so row max / row sum are in-lane plus one exchange between the
//                                      two 32-lane halves
//   O^T[d][query] += V^T . P^T         A = V^T (LDS transpose read), B = P^T taken straight from the
//                                      S^T accumulator registers (no shuffle: the MFMA k-slot <-> key
//                                      assignment is chosen to match the accumulator layout)
//
// K and V tiles are multi-buffered in LDS, one barrier per tile, and go straight from
// global memory into LDS (the swizzle applied to the source
// address): one tile ahead over two buffers in kernel 1, three over four
// buffers in kernel 2 and for heads wider than 128.
#ifndef NAUT_ATTN_KERNELS_H
#define NAUT_ATTN_KERNELS_H
#include <cfloat>
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <type_traits>

#include "naut_attn.h"
#include "naut_common.h"

#ifndef NAUT_KPF
#define NAUT_KPF 2
#endif
#ifndef NAUT_K1_NBUF
#define NAUT_K1_NBUF 2
#endif

namespace naut_k {

using namespace naut;


constexpr int BM = 128;  // queries per work-group
constexpr int BM2 = 256; // queries per work-group of the eight-wavefront kernels
constexpr int BN = 64;   // keys per step
#ifndef NAUT_HAO
#define NAUT_HAO 8
#endif
constexpr int HEADS_AT_ONCE = NAUT_HAO;  // (batch, head) pairs an XCD works on at a time (eight-wavefront kernels)
constexpr int NWAVES = 4;
constexpr int NTHREADS = NWAVES * 64;
constexpr float RESCALE_TAU = 6.0f;  // log2 units

// The kernels are compiled for head dimensions 64, 80, 96, 128, 192 and 256; a head in between runs on the next
// wider one.  In LDS a row of K or V always takes 64, 128 or 256 values, so that the swizzles (which need a power
// of two) are those of the wide head; a narrower head leaves the rest of the row out of its MFMAs and fragment
// reads.  At D = 80 that is 11 MFMAs for every 16 of the 128-wide head, at 96 it is 12, at 192 24 for 32.  Measured
// against the next wider kernel: 4x16 heads, S = 1777, D = 80 108 -> 88 us; 4x64/8 heads, S = 3835, D = 192, causal
// 2.67 -> 2.28 ms (outputs bit-identical).
constexpr int layout_width(int D) { return D <= 64 ? 64 : D <= 128 ? 128 : 256; }
constexpr int compiled_width(int D) { return D <= 64 ? 64 : D <= 80 ? 80 : D <= 96 ? 96 : D <= 128 ? 128 : D <= 192 ? 192 : 256; }

struct Params {
    const void* q;
    const void* k;
    const void* v;
    void* o;
    float* lse;
    int B, Hq, Hkv, S;
    int nqt;       // number of 128-query tiles = ceil(S / BM)
    int nqt2;      // number of 256-query tiles
    float c;       // scale * log2(e), > 0
    float p_limit; // kernel 2: a block's row sum of P above this moves the reference maximum (set at the launch)
    // Byte strides of batch, head and sequence position (the D axis is contiguous).  The kernels are
    // compiled for a few head dimensions; others run on the next wider one: cpr 16-byte
    // chunks of every row are real, the chunks of Q beyond them read as zero, those of K and V repeat
    // a real chunk (they meet zeros of Q, or end in columns of O that are not stored).
    long long q_bs, q_hs, k_bs, k_hs, v_bs, v_hs, o_bs, o_hs;
    int q_rs, k_rs, v_rs, o_rs;
    int cpr;       // real 16-byte chunks per row = head dimension / 8
};

// The order of work-groups that keeps an XCD to few heads: work-groups are dealt to the 8 XCDs round-robin by block id, and
// each XCD has its own L2.  Every XCD gets a contiguous run of an eighth of the (batch, head) pairs, in `groups` groups of
// nearly one size, one group after the other, each with its heaviest (last) query tiles first.  Pairs that eight does not
// divide are taken all at once, heaviest tiles first: dealing only those left over to all XCDs was between 6 % slower and
// 4 % faster (7 x 12 heads, S = 9088, D = 80, causal 1223 -> 1286 us; 12 heads, S = 16384, D = 256 1536 -> 1467).
struct QueryTile {
    int qt, bh;
};
__device__ __forceinline__ QueryTile tile_by_head(int bid, int nbh, int nqt, int groups)
{
    if (nbh & 7)
        return {nqt - 1 - bid / nbh, bid % nbh};
    const int xcd = bid & 7, s = bid >> 3;
    const int hpx = nbh >> 3;
    const int G = (hpx + groups - 1) / groups, per_group = nqt * G;
    const int g = s / per_group, sg = s % per_group;
    const int ng = hpx - g * G < G ? hpx - g * G : G;
    return {nqt - 1 - sg / ng, xcd * hpx + g * G + sg % ng};
}

// S^T MFMAs of the shape that needs more than 256 registers per lane (wide heads on four wavefronts),
// written as asm so that their accumulator is an ordinary vector
// register tuple while O and Q live in the accumulation registers (the compiler's own MFMA form
// would then put the scores there too and copy each one out for the softmax).  The compiler's hazard handling does not look inside asm, so the wait states the
// hardware does not interlock are owed by hand:
//   - a vector instruction that writes an MFMA source (the register allocator may route a
//     fragment through a copy) must be 2 wait states ahead of the MFMA: each asm starts with them;
//   - an MFMA result may be read by a vector instruction only 11 wait states after the issue of
//     this 8-pass MFMA: see `settle`.
// Everything that fits the ordinary vector registers uses the compiler's MFMA throughout.
template <int DT>
struct XMfma;
// Puts every later reader of an asm MFMA's result `d` the owed wait states behind that MFMA.
__device__ __forceinline__ void settle(f32x16_t& d) { asm volatile(NAUT_NOP_SETTLE : "+v"(d)); }
template <>
struct XMfma<NAUT_BF16> {
    static __device__ __forceinline__ void first(f32x16_t& d, i32x4_t a, i32x4_t b)
    {
        asm volatile(NAUT_NOP_SHORT "v_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" NAUT_NOP_AFTER_MFMA : "=&v"(d) : "v"(a), "a"(b));
    }
    static __device__ __forceinline__ void acc(f32x16_t& d, i32x4_t a, i32x4_t b)
    {
        asm volatile(NAUT_NOP_SHORT "v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" NAUT_NOP_AFTER_MFMA : "+v"(d) : "v"(a), "a"(b));
    }
};
template <>
struct XMfma<NAUT_F16> {
    static __device__ __forceinline__ void first(f32x16_t& d, i32x4_t a, i32x4_t b)
    {
        asm volatile(NAUT_NOP_SHORT "v_mfma_f32_32x32x16_f16 %0, %1, %2, 0" NAUT_NOP_AFTER_MFMA : "=&v"(d) : "v"(a), "a"(b));
    }
    static __device__ __forceinline__ void acc(f32x16_t& d, i32x4_t a, i32x4_t b)
    {
        asm volatile(NAUT_NOP_SHORT "v_mfma_f32_32x32x16_f16 %0, %1, %2, %0" NAUT_NOP_AFTER_MFMA : "+v"(d) : "v"(a), "a"(b));
    }
};

// ---- kernel 1: 32 queries per wavefront, 4 wavefronts (D > 128: 4 or 8) per work-group ----
// Two work-groups per CU (four at D = 64) and 64 keys per step for D <= 128.  A wider head doubles the O accumulator
// and the Q fragments of a lane (192 registers between them at D = 256) and runs one work-group per CU with 32 keys per
// step (four K and four V buffers of 16 KB), in two shapes:
//   NWV = 8: two wavefronts per SIMD.  With O and Q, 16 scores that become P in place, and fragment addresses that
//       share their two halves (k_at, v_at) a lane needs 246 of its 256 registers (D = 192: 218), all ordinary ones, so
//       the compiler schedules every MFMA; while one wavefront of a SIMD does its softmax or waits for LDS the other's
//       MFMAs run, and a K/V tile serves 256 queries.
//   NWV = 4: one wavefront per SIMD on the 512-register budget, O and Q in the accumulation registers and the score
//       MFMAs in asm.  It is bound by the dependences of its one instruction stream (46 % of the wavefront time is
//       waiting), but one work-group of it takes 0.8 times as long as one of the other, so it stays for grids that do
//       not fill the chip (see wide_variant).
// NG key groups of NWV wavefronts (D <= 128: two of four or four of two; see pick_form): group g takes key tiles g, g + NG, ... through tile
// buffers of its own, and the partial (O, m, l) of the groups are merged through LDS at the end.
// S = 16384, 32 heads, causal, D = 256: 5282 us (833 TFLOP/s) on four wavefronts, 4173 us (1054) on eight under sustained
// load (three launches at a time, before the clock falls, 5026 / 3922); the D = 128 kernel reaches 1150 to 1190.  D = 192,
// 4x64/8 heads, S = 3835: 2106 / 1387 us.  Outputs are bit-identical (same tiles, same order).

template <int D, int DT_IN, int DT_OUT, bool CAUSAL, int NWV = NWAVES, int NG = 1>
__global__ __launch_bounds__(NWV * NG * 64, D > 128 ? 1 : 2) void naut_fwd_kernel_bm128(const Params p)
{
    using T = In<DT_IN>;
    constexpr int BM = NWV * 32;             // queries per work-group (hides the file-scope value)
    constexpr int W = layout_width(D);       // row width of the LDS layouts
    // keys per step of a group (hides the file-scope value used by kernel 2); four groups: what their rings leave room for
    constexpr int BN = D > 128 || (NG == 4 && W == 128) ? 32 : 64;
    constexpr int ROWB = W * 2;              // bytes per K/V row in LDS
    constexpr int TILEB = BN * ROWB;         // bytes per K or V tile
    constexpr int CPR = W / 8;               // 16-byte chunks per row
    constexpr int KS = D / 16;               // MFMA k-steps of Q.K^T
    constexpr int DB = (D + 31) / 32;        // 32-row blocks of O^T
    constexpr int KB = BN / 32;              // 32-key blocks of S^T

    // Tiles are filled by direct global->LDS loads, each wavefront its share of every tile.  D = 256: four K
    // buffers, then four V buffers, filled three steps ahead (one wavefront per SIMD has nothing else to
    // hide the load latency behind).  D <= 128: K0 V0 K1 V1 ..., a ring of NB2 buffers filled NB2 - 1 steps
    // ahead (the key loop is unrolled over the ring, so a tile's LDS offsets are instruction immediates).
    constexpr bool WIDE = D > 128;
    constexpr bool ACC = WIDE && NWV == 4;         // O and Q live in the accumulation registers
    constexpr bool PAIR = WIDE && NWV == 8;        // two wavefronts per SIMD on 256 ordinary registers each
    static_assert(WIDE ? NG == 1 && NWV >= 4 : (NWV == 4 && NG <= 2) || (NWV == 2 && NG == 4), "the shapes that are launched");
    constexpr int NB = 4;                          // buffers per operand (wide)
    constexpr int NB2 = NAUT_K1_NBUF;              // buffers per operand (D <= 128)
    constexpr int LDW = TILEB / 1024 / NWV;        // direct loads (1 KB each) per wavefront per tile
    static_assert(LDW >= 1 && (NB2 - 1) * 2 * LDW < 64, "every wavefront loads; vmcnt field");
    constexpr int RINGB = (WIDE ? 2 * NB : 2 * NB2) * TILEB;  // bytes of a key group's tile buffers
    __shared__ __attribute__((aligned(1024))) unsigned char smem[NG * RINGB];
    __shared__ float dl_lds[NG * NWV * 64];
    __shared__ float ml_lds[NG > 1 ? (NG - 1) * NWV * 64 * 2 : 1];

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave_wg = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave-uniform: it feeds scalar operands of the tile loads
    const int wave = NG == 1 ? wave_wg : wave_wg % NWV;           // inside its key group
    const int grp = NG == 1 ? 0 : wave_wg / NWV;
    const int l32 = lane & 31;
    const int h = lane >> 5;

    // Tile scheduler: heaviest (last) query tiles first; consecutive block ids walk the
    // (batch, head) axis so that each XCD (block id mod 8) keeps to a fixed subset of heads.
    const int nbh = p.B * p.Hq;
    const int nqt = NWV == 4 ? p.nqt : NWV == 8 ? p.nqt2 : (p.S + BM - 1) / BM;
    const int bid = blockIdx.x;
    int qt, bh;
    if (NWV == 8) {
        // About HEADS_AT_ONCE heads at a time in groups of nearly one size: a last group of one or two heads would start its
        // heaviest tiles when everything else is done (D = 256, causal, S = 1536, 72 heads, nine to an XCD: eight and one 153
        // us, nine 113; S = 2048, 136 heads: eight, eight and one 392, nine and eight 327; all at once costs 2 to 4 % of
        // larger grids).
        const int hpx = nbh >> 3;
        const QueryTile t = tile_by_head(bid, nbh, nqt, hpx < HEADS_AT_ONCE ? 1 : (hpx + HEADS_AT_ONCE / 2) / HEADS_AT_ONCE);
        qt = t.qt;
        bh = t.bh;
    } else {
        qt = nqt - 1 - bid / nbh;
        bh = bid % nbh;
    }
    const int b = bh / p.Hq;
    const int hq = bh % p.Hq;
    const int hk = hq / (p.Hq / p.Hkv);
    const int S = p.S;

    const unsigned char* qg = (const unsigned char*)p.q + b * p.q_bs + hq * p.q_hs;
    const unsigned char* kg = (const unsigned char*)p.k + b * p.k_bs + hk * p.k_hs;
    const unsigned char* vg = (const unsigned char*)p.v + b * p.v_bs + hk * p.v_hs;
    const int cpr = p.cpr;

    const int q_wave0 = qt * BM + wave * 32;  // first query of this wavefront
    const int my_q = q_wave0 + l32;           // the query this lane owns
    const int my_q_ld = my_q < S ? my_q : S - 1;

    // Q^T fragments (MFMA B operand): lane holds q[my_q][16*ks + 8*h .. +8].
    i32x4_t qf[KS];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
        // Unconditional, from a chunk that exists (a load under a condition becomes a branch); the padding
        // chunks of a narrower head are zeroed when Q is pinned.
        const int ch = ks * 2 + h < cpr ? ks * 2 + h : cpr - 1;
        qf[ks] = *(const i32x4_t*)(qg + (size_t)my_q_ld * p.q_rs + ch * 16);
    }
    // Keep Q resident: without this the compiler re-issues the global loads inside the key loop.
    // The wide instantiation keeps it, and O, in the accumulation registers.  D <= 128 pins it only
    // after the first tile's loads are out, so that the two share one round trip to memory.
    auto pin_acc = [](f32x16_t& x) {
        if constexpr (ACC)
            asm volatile("" : "+a"(x));
    };
    auto pin_q = [&](int cpr_now) {
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            if (ks * 2 + h >= cpr_now)
                qf[ks] = i32x4_t{0, 0, 0, 0};
            if constexpr (ACC)
                asm volatile("" : "+a"(qf[ks]));
            else
                asm volatile("" : "+v"(qf[ks]));
        }
    };
    if constexpr (WIDE)
        pin_q(cpr);

    const int kv_end = CAUSAL ? (S < (qt + 1) * BM ? S : (qt + 1) * BM) : S;
    const int ntiles = (kv_end + BN - 1) / BN;

    // Lane i of direct load n fills physical chunk P = (wave*LDW + n)*64 + i of the tile, so it fetches the
    // logical (row, chunk) that k_off / v_off place there (chunks beyond a narrower head repeat a real one).
    auto source_of = [&](int n, int& krow, int& kcol, int& vrow, int& vcol) {
        const int P = (wave * LDW + n) * 64 + lane;
        int kc, vc;
        if constexpr (WIDE) {
            const int line = P >> 4;
            krow = line >> 1;
            kc = ((line & 1) << 4) | ((P & 15) ^ (krow & 15));
            vrow = P >> 5;
            vc = (P & 31) ^ ((vrow & 3) << 2);
        } else {
            const int line = P >> 4, pos = P & 15;
            const int off = ((line << 4) + (pos ^ (line & 15))) * 16;  // the inverse of k_off: byte offset in a dense tile
            krow = off / ROWB;
            kc = off % ROWB / 16;
            vrow = P / CPR;                                              // the inverse of v_off
            vc = W == 128 ? (P % CPR) ^ ((vrow & 3) << 2) : (P % CPR) ^ (((vrow >> 1) & 1) << 2);
        }
        kcol = (kc < cpr ? kc : cpr - 1) * 16;
        vcol = (vc < cpr ? vc : cpr - 1) * 16;
    };
    // wide: (row, byte in the row) per load; D <= 128: the byte offset inside a whole tile
    int wk_row[LDW], wk_col[LDW], wv_row[LDW], wv_col[LDW];
    const unsigned smem_base = (unsigned)(uintptr_t)(NAUT_LDS unsigned char*)smem + (unsigned)(grp * RINGB);
#pragma unroll
    for (int n = 0; n < LDW; ++n) {
        source_of(n, wk_row[n], wk_col[n], wv_row[n], wv_col[n]);
        if constexpr (!ACC) {
            wk_col[n] += wk_row[n] * p.k_rs;
            wv_col[n] += wv_row[n] * p.v_rs;
        }
    }
    const int last_tile = (S + BN - 1) / BN - 1;  // of the sequence: the only one that can be ragged
    const int my_tiles = (ntiles - grp + NG - 1) / NG;  // of this key group: grp, grp + NG, ...
    // The address of a load is the tile's base, a 64-bit wave-uniform pointer, plus a 32-bit lane offset inside
    // the tile (at most BN rows of the largest row stride the entry point admits); rows beyond the end of the
    // sequence re-read its last row.
    // (D <= 128: `buf`, the tile's place in the ring, is a constant at every call)
    auto issue_tile = [&](int tile, int buf = 0) {
        const unsigned kd = smem_base + (unsigned)((ACC ? (tile % NB) * TILEB : WIDE ? buf * TILEB : buf * 2 * TILEB) + wave * LDW * 1024);
        const unsigned vd = kd + (WIDE ? NB * TILEB : TILEB);
        const unsigned char* const kt = kg + (size_t)tile * BN * p.k_rs;
        const unsigned char* const vt = vg + (size_t)tile * BN * p.v_rs;
        const int last_row = S - 1 - tile * BN;  // of this tile, counted from its first row; >= 0
        if constexpr (ACC) {
#pragma unroll
            for (int n = 0; n < LDW; ++n) {
                const int row = wk_row[n] < last_row ? wk_row[n] : last_row;
                const int off = row * p.k_rs + wk_col[n];
                load_to_lds(kd + n * 1024, off, kt);
            }
#pragma unroll
            for (int n = 0; n < LDW; ++n) {
                const int row = wv_row[n] < last_row ? wv_row[n] : last_row;
                const int off = row * p.v_rs + wv_col[n];
                load_to_lds(vd + n * 1024, off, vt);
            }
        } else if (tile == last_tile) {  // once per work-group: the offsets of the ragged tile are formed on the spot
#pragma unroll
            for (int n = 0; n < LDW; ++n) {
                int kr, kcol, vr, vcol;
                source_of(n, kr, kcol, vr, vcol);
                load_to_lds(kd + n * 1024, (kr < last_row ? kr : last_row) * p.k_rs + kcol, kt);
                load_to_lds(vd + n * 1024, (vr < last_row ? vr : last_row) * p.v_rs + vcol, vt);
            }
        } else {
#pragma unroll
            for (int n = 0; n < LDW; ++n) {
                load_to_lds(kd + n * 1024, wk_col[n], kt);
                load_to_lds(vd + n * 1024, wv_col[n], vt);
            }
        }
    };
    // Waits until at most `ahead` later tiles of this wavefront's loads are still in flight.
    auto wait_tiles = [&](int ahead) {
        if (ahead >= 2)
            wait_loads<WIDE ? 2 * 2 * LDW : 0>();
        else if (ahead == 1)
            wait_loads<WIDE ? 2 * LDW : 0>();
        else
            wait_loads<0>();
    };

    // fixed LDS addresses of this lane's fragment reads in buffer 0 (K: per k-step; V: per 32-row block
    // of O^T, first of the two transposed reads); buffer, key-block and key-step offsets are immediates
    // (adding 8, 16 or 32 to a row changes no swizzle key)
    // (wide: the swizzles stay inside 256 bytes, so the second half of a row is the first plus 256)
    constexpr int NRK = WIDE ? 8 : KS, NRV = WIDE ? 4 : DB;
    int rd_k[NRK], rd_v[NRV];
#pragma unroll
    for (int ks = 0; ks < NRK; ++ks) {
        rd_k[ks] = (int)smem_base + k_off<W>(l32, ks * 2 + h);
        asm volatile("" : "+v"(rd_k[ks]));
    }
    {
        const int i16 = lane & 15;
        const int key = 4 * h + (i16 >> 2);
#pragma unroll
        for (int db = 0; db < NRV; ++db) {
            const int d = 32 * db + 16 * ((lane >> 4) & 1) + 4 * (i16 & 3);
            rd_v[db] = (int)smem_base + v_off<W>(key, d >> 3) + (d & 7) * 2 + (PAIR ? NB * TILEB : 0);
            asm volatile("" : "+v"(rd_v[db]));
        }
    }
    auto k_at = [&](int ks) { return rd_k[ks % NRK] + ks / NRK * 256; };
    auto v_at = [&](int db) { return rd_v[db % NRV] + db / NRV * 256; };

    f32x16_t oacc[DB];
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int r = 0; r < 16; ++r)
            oacc[db][r] = 0.f;
    // running max, in the exp2 domain (already times c).  A key group may see nothing but masked keys of a row, so
    // with several the start is finite: the lowest value there is, below any score that is itself finite.
    float m_run = NG == 1 ? -INFINITY : -FLT_MAX;
    float l_run = 0.f;        // this lane's share of the running sum (its 16 of every 32 keys)
    // What the sum of P as rounded for the second product, the divisor of O, has over l (this lane's share; see
    // "the two sums" in kernel 2).  It is touched only in rare blocks and in the epilogue, so it lives in a word
    // of LDS per lane instead of a register: the D = 64 instantiation fits four wavefronts per SIMD on exactly
    // 128 registers.
    // (its index is re-derived from the hardware lane count where it is used: no register holds it either)
    auto dl_slot = [&]() -> float& {
        const int ln = (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
        return dl_lds[wave_wg * 64 + ln];
    };
    dl_slot() = 0.f;
    const float c = p.c;

    if constexpr (WIDE) {
        // Q must be in its registers before the tile loads start: the compiler's own wait for Q would
        // otherwise also wait for every tile load issued before it.
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        static_for<0, NB - 1>([&](auto TC) {
            if (decltype(TC)::value < ntiles)
                issue_tile(decltype(TC)::value, decltype(TC)::value);
        });
        wait_tiles(ntiles - 1);
        tile_barrier();
    } else {
        static_for<0, NB2 - 1>([&](auto TC) {
            if (decltype(TC)::value < my_tiles)
                issue_tile(decltype(TC)::value * NG + grp, decltype(TC)::value);
        });
        int cpr_late = cpr;
        asm volatile("" : "+s"(cpr_late));  // ordered after the asm of the tile loads: so is everything that uses it
        pin_q(cpr_late);                    // Q and the first tiles share one round trip to memory
    }

    // One key tile.  UC = j mod the number of buffers as a constant -- the driver loop below is unrolled over
    // the LDS buffers, so the tile's LDS offsets are immediates.  The four-wavefront wide shape keeps one copy of
    // its (long) body and adds the buffer offset at run time.
    constexpr int NU = ACC ? 1 : PAIR ? NB : NB2;
    auto step = [&](auto UC, int j) {
        constexpr int U = decltype(UC)::value;
        const int KT = ACC ? (j % NB) * TILEB : PAIR ? U * TILEB : U * 2 * TILEB;   // byte offset of this step's K tile
        const int VT = ACC ? KT + NB * TILEB : PAIR ? KT : KT + TILEB;
        const int kv0 = (j * NG + grp) * BN;
        if constexpr (WIDE) {
            // buffer (j + NB - 1) % NB was last read in step j - 1, which every wavefront has left
            if (j + NB - 1 < ntiles)
                issue_tile(j + NB - 1, PAIR ? (U + NB - 1) % NB : 0);
            if constexpr (SAFE_SYNC)
                tile_barrier();  // checking build: nothing in flight while the step computes
        } else {
            // Tile j must have landed.  Loads complete in order, so with the tiles j+1 .. j+NB2-2 requested after
            // it this wavefront may leave theirs in flight; near the end fewer were requested and it waits for all.
            if (j + NB2 - 2 < my_tiles)
                wait_loads<(NB2 - 2) * 2 * LDW>();
            else
                wait_loads<0>();
            tile_barrier();  // publishes tile j; every wavefront has left step j-1, whose buffer is refilled next
            if (j + NB2 - 1 < my_tiles)
                issue_tile((j + NB2 - 1) * NG + grp, (U + NB2 - 1) % NB2);
            if constexpr (SAFE_SYNC) {  // checking build: nothing in flight while the step computes
                wait_loads<0>();
                tile_barrier();
            }
        }

        // Causal block skipping per wavefront: nothing to do if every key of the tile lies
        // beyond this wavefront's last query.
        const bool active = (!CAUSAL || kv0 <= q_wave0 + 31) && (NG == 1 || j < my_tiles);
        if (active) {
            f32x16_t sacc[KB];
#pragma unroll
            for (int kb = 0; kb < KB; ++kb) {
                if constexpr (ACC) {
                    // The compiler moves nothing across the asm MFMAs, so the fragment reads are put
                    // KPF MFMAs ahead of their use by hand.  Measured at S = 16384: reading each fragment
                    // right before its MFMA exposes the LDS latency 16 times per step (714 TFLOP/s), one
                    // ahead 829, two 850, three 846, four 843, six 839, eight 835, twelve 825, sixteen 812:
                    // two reads in flight cover the latency, more only lengthen the wait before the first
                    // MFMA of the step.
                    constexpr int KPF = NAUT_KPF;
                    i32x4_t kf[KS];
#pragma unroll
                    for (int ks = 0; ks < KPF; ++ks)
                        kf[ks] = *(const NAUT_LDS i32x4_t*)(uintptr_t)(k_at(ks) + KT + kb * 32 * ROWB);
#pragma unroll
                    for (int ks = 0; ks < KS; ++ks) {
                        if (ks + KPF < KS)
                            kf[ks + KPF] = *(const NAUT_LDS i32x4_t*)(uintptr_t)(k_at(ks + KPF) + KT + kb * 32 * ROWB);
                        if (ks == 0)
                            XMfma<DT_IN>::first(sacc[kb], kf[ks], qf[ks]);
                        else
                            XMfma<DT_IN>::acc(sacc[kb], kf[ks], qf[ks]);
                    }
                    settle(sacc[kb]);
                } else {
#pragma unroll
                    for (int r = 0; r < 16; ++r)
                        sacc[kb][r] = 0.f;
#pragma unroll
                    for (int ks = 0; ks < KS; ++ks) {
                        const i32x4_t kf = *(const NAUT_LDS i32x4_t*)(uintptr_t)(k_at(ks) + KT + kb * 32 * ROWB);
                        sacc[kb] = T::mfma(kf, qf[ks], sacc[kb]);
                    }
                }
            }
            // Mask only where the tile straddles the diagonal or the end of the sequence.
            const bool need_mask = (CAUSAL && kv0 + BN - 1 > q_wave0) || (kv0 + BN > S);
            if (need_mask) {
#pragma unroll
                for (int kb = 0; kb < KB; ++kb)
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        const int key = kv0 + kb * 32 + 8 * (r >> 2) + 4 * h + (r & 3);
                        const bool dead = (CAUSAL && key > my_q) || key >= S;
                        sacc[kb][r] = dead ? -INFINITY : sacc[kb][r];
                    }
            }
            // running max over keys: in-lane, then across the two 32-lane halves
            float mx = sacc[0][0];
#pragma unroll
            for (int kb = 0; kb < KB; ++kb)
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    mx = fmaxf(mx, sacc[kb][r]);
            mx = half_max(mx);
            // The reference maximum only has to be *a* bound shared by l and O, not the exact running
            // maximum: it is moved (and the partial sums repaired) only when some query of this
            // wavefront exceeds it by more than 2^RESCALE_TAU, which keeps every P below that factor.
            const float m_cand = mx * c;
            const bool grow = m_cand > m_run + RESCALE_TAU;
            if (__builtin_amdgcn_ballot_w64(grow) != 0) {
                const float m_new = fmaxf(m_run, m_cand);
                const float alpha = __builtin_amdgcn_exp2f(m_run - m_new);  // repair factor
                m_run = m_new;
                l_run *= alpha;
                dl_slot() *= alpha;
#pragma unroll
                for (int db = 0; db < DB; ++db) {
                    pin_acc(oacc[db]);  // the copy into vector registers for the multiply starts here, not at the loop top
#pragma unroll
                    for (int r = 0; r < 16; ++r)
                        oacc[db][r] *= alpha;
                    pin_acc(oacc[db]);
                }
            }
#pragma unroll
            for (int db = 0; db < DB; ++db)
                pin_acc(oacc[db]);
            const float m_new = m_run;
            float psum = 0.f;
#pragma unroll
            for (int kb = 0; kb < KB; ++kb)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const float pv = __builtin_amdgcn_exp2f(__builtin_fmaf(sacc[kb][r], c, -m_new));
                    sacc[kb][r] = pv;
                    psum = (kb | r) == 0 ? pv : psum + pv;
                }
            // O^T += V^T . P^T, 16 keys per MFMA
#pragma unroll
            for (int t = 0; t < BN / 16; ++t) {
                const int kb = t >> 1, r0 = (t & 1) * 8;
                i32x4_t pb = {T::pack2(sacc[kb][r0 + 0], sacc[kb][r0 + 1]), T::pack2(sacc[kb][r0 + 2], sacc[kb][r0 + 3]),
                              T::pack2(sacc[kb][r0 + 4], sacc[kb][r0 + 5]), T::pack2(sacc[kb][r0 + 6], sacc[kb][r0 + 7])};
#pragma unroll
                for (int db = 0; db < DB; ++db) {
                    const int a = v_at(db) + VT + t * 16 * ROWB;
                    const i16x4_t r0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((NAUT_LDS i16x4_t*)(uintptr_t)a);
                    const i16x4_t r1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((NAUT_LDS i16x4_t*)(uintptr_t)(a + 8 * ROWB));
                    const i32x2_t lo = __builtin_bit_cast(i32x2_t, r0), hi = __builtin_bit_cast(i32x2_t, r1);
                    const i32x4_t vf = {lo.x, lo.y, hi.x, hi.y};
                    oacc[db] = T::mfma(vf, pb, oacc[db]);
                }
            }
            // The divisor of O takes the sum of P as rounded for the second product only for a tile that at least
            // doubles some row's running sum (see "the two sums" in kernel 2); elsewhere the unrounded sum stands
            // in for it.  The test sits at the end of the tile, where it splits no schedule; a tile that passes
            // it rounds its P, still in their registers, once more (the pairs in the other order -- the sum does
            // not care -- so that these packs are not merged with those of the product loop above).
            if (__builtin_amdgcn_ballot_w64(psum > l_run) != 0) {
                float prsum = -psum;
#pragma unroll
                for (int kb = 0; kb < KB; ++kb)
#pragma unroll
                    for (int r = 0; r < 16; r += 2)
                        prsum = T::add_pair(T::pack2(sacc[kb][r + 1], sacc[kb][r]), prsum);
                dl_slot() += prsum;
            }
            l_run += psum;
        }
        if constexpr (WIDE) {
            // Tile j + 1 must have landed; the tiles after it may fly on.  A bare barrier: every LDS
            // read of this step has been consumed by its MFMA, and the fence of __syncthreads()
            // would wait for all tile loads in flight.
            wait_tiles(ntiles - 2 - j);
            if constexpr (PAIR)
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // nothing is left to wait for unless the compiler moved an MFMA
            tile_barrier();
        }
    };
    const int nsteps = (ntiles + NG - 1) / NG;  // of the first group, which has the most: all meet the same barriers
    for (int j0 = 0; j0 < nsteps; j0 += NU) {
        static_for<0, NU>([&](auto UC) {
            const int j = j0 + decltype(UC)::value;
            if (j < nsteps)  // uniform over the work-group
                step(UC, j);
        });
    }

    if constexpr (!WIDE)
        __syncthreads();  // every wavefront has left the last step: the tiles are dead, the epilogue stages O in them
    if constexpr (NG > 1) {
        // Split-merge of the key groups: the others leave O, m and l (dl is in LDS already) in the layout they hold
        // them in, lane by lane, each in its own dead tiles; the first group's wavefronts add them up and store.
        static_assert(NWV * DB * 16 * 64 * 4 <= RINGB, "a group's O fits its tile buffers");
        constexpr int OW = DB * 16 * 64;  // floats per wavefront
        int ln = lane;
        asm volatile("" : "+v"(ln));  // as in the epilogue: no address of the merge is held across the key loop
        if (grp > 0) {
            float* const mo = (float*)(smem + grp * RINGB) + wave * OW;
#pragma unroll
            for (int db = 0; db < DB; ++db)
#pragma unroll
                for (int g = 0; g < 4; ++g)
                    *(f32x4_t*)(mo + ((db * 4 + g) * 64 + ln) * 4) =
                        f32x4_t{oacc[db][4 * g], oacc[db][4 * g + 1], oacc[db][4 * g + 2], oacc[db][4 * g + 3]};
            float* const ml = ml_lds + ((grp - 1) * NWV + wave) * 128 + ln;
            ml[0] = m_run;
            ml[64] = l_run;
        }
        __syncthreads();
        if (grp > 0)
            return;
#pragma unroll 1  // one group's partials in registers at a time
        for (int o = 1; o < NG; ++o) {
            const float* const ml = ml_lds + ((o - 1) * NWV + wave) * 128 + ln;
            const float* const mo = (const float*)(smem + o * RINGB) + wave * OW;
            // The halves of a row hold the same maximum, and key 0, which every row sees, is the first group's.
            const float m_new = fmaxf(m_run, ml[0]);
            const float f0 = __builtin_amdgcn_exp2f(m_run - m_new), f1 = __builtin_amdgcn_exp2f(ml[0] - m_new);
            m_run = m_new;
            l_run = l_run * f0 + ml[64] * f1;
            float& dl = dl_slot();
            dl = dl * f0 + dl_lds[(o * NWV + wave) * 64 + ln] * f1;
#pragma unroll
            for (int db = 0; db < DB; ++db)
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const f32x4_t x = *(const f32x4_t*)(mo + ((db * 4 + g) * 64 + ln) * 4);
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        oacc[db][4 * g + i] = oacc[db][4 * g + i] * f0 + x[i] * f1;
                }
        }
    }
    // Epilogue: one division by l (the per-step divide/multiply pairs telescope away), lse, store.
    const float l_tot = l_run + __shfl_xor(l_run, 32);
    const float dl_run = dl_slot();
    const float inv_l = 1.0f / (l_tot + (dl_run + __shfl_xor(dl_run, 32)));
    if (my_q < S && p.lse != nullptr && h == 0)
        p.lse[(size_t)bh * S + my_q] = (m_run + __builtin_amdgcn_logf(l_tot)) * 0.6931471805599453f;
    unsigned char* const o_bh = (unsigned char*)p.o + b * p.o_bs + hq * p.o_hs;
    if constexpr (DT_OUT != NAUT_F32) {
        // 16-bit O leaves through LDS in whole rows: a lane owns 4 consecutive d of one query (8 bytes, 32
        // different rows per store instruction); after the exchange D/8 lanes write one row with 16 bytes
        // each.  The tiles are dead after the loop's last barrier (every tile load has landed, every
        // fragment has been consumed); each wavefront stages its 32 rows in its own part of them.
        constexpr int CPRO = CPR, R256 = ROWB >= 256 ? 1 : 256 / ROWB;
        static_assert(NWV * 32 * ROWB <= (int)sizeof(smem), "staging rows must fit the tile buffers");
        // Every address below derives from this copy of the lane id, which exists only from here on: nothing
        // of the epilogue can be computed before the key loop and held in registers across it.
        int ln = lane;
        asm volatile("" : "+v"(ln));
        const int l32e = ln & 31, he = ln >> 5;
        unsigned char* const stg = smem + wave * 32 * ROWB;
        auto staged = [&](int r, int ch) {  // swizzled so that neither the writes nor the reads conflict
            return stg + r * ROWB + ((ch ^ ((r / R256) & (CPRO - 1))) << 4);
        };
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const int d = 32 * db + 8 * g + 4 * he;
                const i32x2_t w = {In<DT_OUT>::pack2(oacc[db][4 * g + 0] * inv_l, oacc[db][4 * g + 1] * inv_l),
                                   In<DT_OUT>::pack2(oacc[db][4 * g + 2] * inv_l, oacc[db][4 * g + 3] * inv_l)};
                *(i32x2_t*)(staged(l32e, d >> 3) + (d & 7) * 2) = w;
            }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        constexpr int RPI = 64 / CPRO;    // rows per store instruction
        constexpr int BATCH = 8 < 32 / RPI ? 8 : 32 / RPI;  // reads in flight before their stores
        typedef i32x4_t __attribute__((aligned(8))) i32x4_a8;  // O rows are 8-byte aligned, not more
#pragma unroll
        for (int i0 = 0; i0 < 32 / RPI; i0 += BATCH) {
            i32x4_t rows[BATCH];
#pragma unroll
            for (int i = 0; i < BATCH; ++i)
                rows[i] = *(const i32x4_t*)staged((i0 + i) * RPI + ln / CPRO, ln % CPRO);
#pragma unroll
            for (int i = 0; i < BATCH; ++i) {
                const int q = q_wave0 + (i0 + i) * RPI + ln / CPRO;
                if (q < S && ln % CPRO < cpr)  // not the rows beyond S, not the padding columns of a narrower head
                    *(i32x4_a8*)(o_bh + (size_t)q * p.o_rs + (ln % CPRO) * 16) = rows[i];
            }
        }
    } else if (my_q < S) {
        unsigned char* og = o_bh + (size_t)my_q * p.o_rs;
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const int d = 32 * db + 8 * g + 4 * h;
                if (d >= cpr * 8)
                    continue;  // padding columns of a narrower head dimension
                f32x4_t w = {oacc[db][4 * g + 0] * inv_l, oacc[db][4 * g + 1] * inv_l,
                             oacc[db][4 * g + 2] * inv_l, oacc[db][4 * g + 3] * inv_l};
                *(f32x4_t*)(og + d * 4) = w;
            }
    }
}

#include "naut_attn_pipe.h"

// ---- host side: variant choice and launch -------------------------------------------

// Kernel variants (the tile shape / wavefront count / buffering choice the paper leaves to its
// auto-tuner, Section 4.4 and Section 7.2).  NAUT_ATTN_VARIANT overrides the shape-based choice for A/B runs (read at every
// call, so that one process can time all of them; any other non-empty value makes the call fail): kernel 2 as w8q32, w4q32,
// w4q32g2 or w4q64, kernel 1 as bm128g1, bm128g2 or bm128g4; bm128 is kernel 1 with the key groups of the class (key_groups).
enum Variant { V_W8Q32 = 0, V_W4Q64 = 1, V_BM128 = 2, V_W4Q32 = 3, V_UNKNOWN = -1, V_BY_SHAPE = -2 };
constexpr const char* kVariantName[4] = {"fwd_bm256_w8q32_bn64", "fwd_bm256_w4q64_bn64", "fwd_bm128_w4q32_bn64", "fwd_bm128_w4q32_bn32"};

// The variant that NAUT_ATTN_VARIANT names, and its key groups (0: by shape).
inline int named_variant(int* groups)
{
    static const struct { const char* name; int variant, groups; } names[] = {
        {"w8q32", V_W8Q32, 0}, {"w4q64", V_W4Q64, 0}, {"w4q32", V_W4Q32, 1}, {"w4q32g2", V_W4Q32, 2},
        {"bm128", V_BM128, 0}, {"bm128g1", V_BM128, 1}, {"bm128g2", V_BM128, 2}, {"bm128g4", V_BM128, 4}};
    *groups = 0;
    const char* e = getenv("NAUT_ATTN_VARIANT");
    if (!e || !e[0])
        return V_BY_SHAPE;
    for (const auto& n : names)
        if (!strcmp(e, n.name)) {
            *groups = n.groups;
            return n.variant;
        }
    return V_UNKNOWN;  // a name that selects nothing is an error, not a silent fall-back to the rule
}

// D > 128: eight wavefronts per work-group, or four (V_BM128).  Either runs one work-group per CU; one of four wavefronts
// covers 128 queries in 0.8 of the time that one of eight takes for 256.
//   No mask: whole rounds of 256 work-groups are what counts.  Four / eight wavefronts, D = 256 (us): 32 heads, S = 1024 (one
//   round of either) 49.0 / 58.1; S = 1536 (two / one) 119.4 / 85.5; 96 heads, S = 577 (two / two) 60.8 / 76.6; 64 heads, S =
//   1152 (three / two) 142.1 / 131.6.  Over 781 shapes of D = 192 and 256 the rule loses 1.1 % at most against the better of
//   the two (one round of four or none, as it was: up to 30 %).  At four rounds against three the two are level, and the
//   longer loops of D = 256 are faster on four wavefronts (104 heads, S = 1152 191 / 203, 320 heads, S = 300 82 / 76).
//   With the mask the second round's work-groups are short and start as the first ones end: two rounds still count as one.
//   S = 2048 (512 of four wavefronts) 94.3 / 105.5, 64 heads, S = 1024 (512) 60.9 / 61.5, S = 1536 (768) 119.8 / 92.2.
inline int wide_variant(int S, long long nbh, int D, int causal)
{
    int groups;
    const int named = named_variant(&groups);
    if (named == V_W8Q32 || (named == V_BM128 && groups <= 1) || named == V_UNKNOWN)
        return named;  // w4q64 and several key groups have no wide form: they choose nothing here
    const long long wgs = nbh * ((S + BM - 1) / BM), wgs2 = nbh * ((S + BM2 - 1) / BM2);
    if (causal)
        return wgs <= 512 ? V_BM128 : V_W8Q32;
    const long long r4 = (wgs + 255) / 256, r8 = (wgs2 + 255) / 256;
    return 4 * r4 <= 5 * r8 || (r4 == 4 && r8 == 3 && D == 256 && S >= 1024) ? V_BM128 : V_W8Q32;
}

// Whether a shape of D <= 128 runs long key loops with whole rounds of 256-query work-groups.
inline bool long_loops(int S, long long nbh, int D, int causal)
{
    const long long wg256 = nbh * ((S + BM2 - 1) / BM2);
    const int avg_keys = causal ? (S + 1) / 2 : S;
    return wg256 >= 256 && (D > 64 ? avg_keys >= (causal ? 2048 : 1024) : avg_keys >= 8192 && wg256 < 1024);
}

// Key groups of the shapes without long loops (D: the compiled width): four for grids of at most 256 work-groups of 64
// queries (512 with the mask on long sequences), two up to 256 work-groups of 128 queries; with the mask up to 512, along a
// line that rises with S, since the second round of work-groups is short only if few of them are heavy, which takes many
// query tiles.  A launch has at least these: every group has a reference maximum of its own, and the more keys there are
// whose P is exactly 1, the smaller the error of O (see pick_form).
inline int key_groups(int S, long long nbh, int D, int causal)
{
    const long long wgs64 = nbh * ((S + 63) / 64), wgs = nbh * ((S + BM - 1) / BM);
    if (S > 256 && (wgs64 <= 256 || (causal && wgs64 <= 512 && S >= 2048)))
        return 4;
    if (S <= 8 * BN || wgs > (causal ? 512 : 256))
        return 1;
    if (wgs <= 256)
        return 2;
    const int beyond = D <= 64   ? (S - 192) * 7 / 32  // work-groups beyond the first 256
                       : D <= 96 ? (S - 384) * 14 / 32
                       : nbh & 1 ? (S - 700) * 5 / 64
                                 : (S - 448) * (nbh & 7 ? 5 : 6) / 32;
    return wgs - 256 <= beyond ? 2 : 1;
}

// The class that a shape falls into, D <= 128, and the key groups of the class: V_W8Q32 for long loops, V_BM128 otherwise.
// It is what naut_attn_variant_name and naut_attn_key_groups tell; the kernel that a launch of either class runs is
// pick_form's choice.
inline int pick_variant(int S, long long nbh, int D, int causal, int* groups)
{
    int named_groups;
    const int named = named_variant(&named_groups);
    *groups = named_groups ? named_groups : key_groups(S, nbh, D, causal);
    if (named != V_BY_SHAPE && (named != V_W4Q64 || D <= 64)) {  // w4q64 has no wider form: it chooses nothing there
        if (named == V_W8Q32 || named == V_W4Q64)
            *groups = 1;
        return named;
    }
    if (!long_loops(S, nbh, D, causal))
        return V_BM128;
    *groups = 1;
    return V_W8Q32;
}

// What a launch with D <= 128 runs (D: the compiled width): kernel 1 (V_BM128) with one, two or four key groups, or kernel 2
// on 8 x 32 queries (V_W8Q32), 4 x 32 (V_W4Q32, one or two key groups) or 4 x 64 (V_W4Q64, D = 64 only).
// Fitted to timings of every form in turn over some 9500 shapes (D = 64, 80, 96 and 128, 1 to 768 heads, S = 128 to 16384,
// with and without the mask).  Kernel time, us:
//   Four key groups of kernel 1: where key_groups says four, and on a little shorter and larger grids: up to 256 work-groups
//   of 64 queries, one per CU, all in one round (8 heads, S = 1024, D = 128, causal 16.2; kernel 2 17.6).  With the mask also
//   two such rounds where the loops are long enough to even out: light tiles go to the CUs that are done first (16 heads, S =
//   1536, D = 64 16.3 / 19.9).  Fewer groups there would be as fast (causal, 22 shapes 0.96 of the time), but less accurate:
//   relative error against 64 bits of two for four 1.02 at the usual scale, up to 1.4 on keys with outliers.
//   Two key groups of kernel 2: where key_groups says two (fewer: error 1.04, up to 1.4 on keys with outliers), and: one
//   work-group of 128 queries per CU (129 to 256 of them) whose loop is worth halving (32 heads, S = 1003, causal, D = 128
//   19.4, one group 20.4, kernel 1 with two 21.6); with the mask up to 512 in two rounds, the more the longer the sequence, as
//   the second round has to be of light tiles (8 heads, S = 8192, D = 128 133 / 142 / 143).
//   Two key groups of kernel 1: with the mask, beyond one round, short: the second round's few light tiles are over sooner
//   (56 heads, S = 640, D = 128 17.5, kernel 2 19.2; D = 80 14.0 / 15.3; 64 heads, S = 640, D = 64 13.3 / 13.8).
//   Kernel 1 with one: sequences of at most 128 keys (two tiles; 2 heads, S = 128, D = 64 6.4 / 6.7), and short ones of very
//   many heads: at D = 64, of which it has four work-groups on a CU for three, between two rounds of the latter and two of the
//   former where the last query tile is more than half full (256 heads, S = 512, causal 19.7 / 21.2, 512 heads, S = 256 17.8
//   / 18.8); at D > 64, with the mask, the first work-groups beyond one round (144 heads, S = 512, D = 128 1.05 of its time
//   on kernel 2, 192 heads, S = 384 1.05).
//   256-query work-groups read K and V half as often as 128-query ones and are coarser.  No mask: by whole rounds, 256
//   slots of 8 x 32 against 512 of 4 x 32 (24 heads, S = 3072, D = 128: 288 work-groups 150 / 130; 32 heads, S = 4096: 512
//   243 / 249), at D = 64 512 slots of 4 x 64 against 768 of 4 x 32, where a fragment read from LDS that feeds two MFMAs
//   is worth 8 % (32 heads, S = 4096 135 / 145).  With the mask they pay where the loop is long or the rounds come out even
//   (32 heads, S = 16384, D = 128 1790 / 1850; 32 heads, S = 4096 129 / 136; 128 heads, S = 4096 536 / 529).
//   Where eight does not divide the heads, XCDs share them, and K and V pass through several L2s: an XCD sees
//   an eighth of 8 k heads, a quarter of 4 k, half of 2 k and all of an odd count.  Time of 4 x 32 over 8 x
//   32 queries at equal rounds (D = 128 / 96 / 80, more than two rounds): odd counts 1.22 / 1.09 / 1.00, 2 k 1.17 / 1.05 /
//   0.98, 4 k 1.07 / 1.00 / 0.97.  At D = 64 kernel 1 is the better one on odd counts with the mask (63 heads, S = 2700 84.8,
//   4 x 32 89.6, 93 heads, S = 1700 57.9 / 62.1).
inline int pick_form(int S, long long nbh, int D, int causal, int* groups)
{
    int named_groups;
    const int named = named_variant(&named_groups);
    if (named != V_BY_SHAPE && (named != V_W4Q64 || D <= 64)) {  // 4 x 64 has no wider form: the name chooses nothing there
        *groups = named_groups ? named_groups : named == V_BM128 ? key_groups(S, nbh, D, causal) : 1;
        return named == V_W8Q32 && D <= 64 ? V_W4Q64 : named;  // eight wavefronts are too many for the 4 KB tiles of D = 64
    }
    const int least = long_loops(S, nbh, D, causal) ? 1 : key_groups(S, nbh, D, causal);
    const long long w64 = nbh * ((S + 63) / 64), w = nbh * ((S + BM - 1) / BM), w2 = nbh * ((S + BM2 - 1) / BM2);
    *groups = 4;
    if (least == 4 || (w64 <= 256 && D <= 64 && causal && S > 192) ||
        (causal && w <= (D <= 64 ? 256 : 224) && S >= 1200 && S >= 1300 + 30 * (w - 160)))
        return V_BM128;
    *groups = 2;
    if (least == 2 && causal && w > 256 && (D > 64 ? S < 850 || (S <= 1024 && w > 296 && w <= 352) : S <= 600 || (S < 1150 && 5 * (w - 290) >= S - 640)))
        return V_BM128;
    if (least == 2 || (w > 128 && w <= 256 && S >= (causal ? 600 : D <= 64 ? 850 : 1000)) ||
        (causal && w > 256 && w <= 512 && S >= 900 + 11 * (w - 288)))
        return V_W4Q32;
    *groups = 1;
    if (S <= 128 || (D <= 64 && !causal && S <= 256) || (causal && w <= 256 && S <= (D <= 64 ? 192 : 144)))
        return V_BM128;
    if (causal) {
        if (D <= 64 && w > 780 && w <= 2000 && S <= 768 && (S <= 640 || w >= 1500) && (S - 1) % BM >= BM / 2)
            return V_BM128;
        if (D > 64 && w > 512 && S > 224 && S <= 640 && w <= (S % BM == 0 && S <= 512 ? 768 : 600))
            return V_BM128;
        if (D <= 64 && nbh % 2 && w >= 900 && S >= 750 && S < 6144)
            return V_BM128;
        if (D <= 64)
            return S >= 6144 && w2 >= 900 ? V_W4Q64 : V_W4Q32;
        if (D > 80 && S >= 1000 && w2 >= (nbh % 2 ? (D > 96 ? 270 : 480) : nbh % 4 ? (D > 96 ? 480 : 1000) : nbh % 8 && D > 96 ? 1000 : w2 + 1))
            return V_W8Q32;
        return (S >= 8192 && w2 >= 480) || (w2 > 448 && w2 <= 512 && S >= 1280) || (w2 > 928 && w2 <= 1024 && S >= 4096) ? V_W8Q32 : V_W4Q32;
    }
    if (D <= 64 ? nbh >= 192 && w > 512 && w <= 1024 && S == 512 : S == 256 && w > 416 && w <= 704)
        return V_BM128;
    if (S < 1000)
        return V_W4Q32;
    // rounds, in per cent of a full one; a last round that leaves every CU one work-group fewer is shorter
    if (D <= 64) {
        const long long r = w % 768, r2 = w2 % 512;
        const long long c32 = w / 768 * 300 + (r == 0 ? 0 : r <= 256 ? 130 : r <= 512 ? 210 : 300);
        const long long c64 = w2 / 512 * 368 + (r2 == 0 ? 0 : r2 <= 256 ? 202 : 368);
        return c64 < c32 && (w2 > 256 || S >= 4096) ? V_W4Q64 : V_W4Q32;
    }
    const int dear = nbh % 2 || (nbh % 4 && w2 >= 600) ? 4 * (D - 72) : nbh % 4 ? 2 * (D - 72) : nbh % 8 && D > 96 && w2 >= 1000 ? 80 : 0;
    const long long r = w % 512;
    const long long c4 = (w / 512 * 100 + (r == 0 ? 0 : r <= 256 ? 60 : 100)) * (1000 + dear) / 1000;
    const long long c8 = (w2 + 255) / 256 * (S >= 1250 ? 97 : 102);
    // beyond eight rounds the halves of that no longer matter -- unless XCDs share heads, and twice the loads count
    return nbh & 7 ? (c8 <= c4 || w2 > 2048 ? V_W8Q32 : V_W4Q32) : w2 <= 2048 && c8 < c4 ? V_W8Q32 : V_W4Q32;
}

template <int D, int DT_IN, int DT_OUT>
int launch(Params p, int causal, hipStream_t stream)
{
    const long long nbh = (long long)p.B * p.Hq;
    int groups = 1;
    int variant = D > 128 ? wide_variant(p.S, nbh, D, causal) : pick_form(p.S, nbh, D, causal, &groups);
    // Two key groups of kernel 2 step over twice the rows at a time: with rows of at most 8 MiB that is at most 2^29 bytes, as
    // the 32-bit offsets between two moves of the base need it (see rebase in the kernel).  Farther apart: those of kernel 1.
    if (D <= 128 && variant == V_W4Q32 && groups == 2 && (p.k_rs > p.v_rs ? p.k_rs : p.v_rs) > 8 << 20)
        variant = V_BM128;
    // How far a block's row sum of P (16 keys) may grow before kernel 2 moves the reference maximum.  Long loops take all the
    // range the type has: a move costs the block's softmax again.  Elsewhere 24, a lag of 1 to 4.6 binades for kernel 1's 6
    // (RESCALE_TAU): after a move the largest P of the row is exactly 1 and carries no rounding error into O, which shows in
    // rows that few keys dominate.  Relative error against 64 bits over that of kernel 1 with as many key groups (bf16, f32
    // O, 256 shapes) with limits of 32, 24 and 16: four times the usual scale 0.99, 0.94, 0.92; twice 0.97, 0.95, 0.91; usual
    // 0.997, 0.997, 0.996.  24 costs 0.1 % of the time on N(0,1) inputs, 16 1.2 %, 8 up to 13 %.
    p.p_limit = long_loops(p.S, nbh, D, causal) ? In<DT_IN>::P_LIMIT : 24.0f;  // by shape, whatever form is named
    if (variant < 0)
        return fail(NAUT_ERR_UNSUPPORTED, "NAUT_ATTN_VARIANT names no kernel variant (w8q32, w4q64, w4q32, w4q32g2, bm128, bm128g1, bm128g2 or bm128g4)");
    const long long nblocks = nbh * (groups == 4 ? (p.S + 63) / 64 : variant == V_BM128 || variant == V_W4Q32 ? p.nqt : p.nqt2);
    if (nblocks > 0x7fffffffLL)
        return fail(NAUT_ERR_UNSUPPORTED, "B*Hq*ceil(S/128) exceeds the 1-D grid limit");
    const dim3 grid((unsigned)nblocks);
#define NAUT_LAUNCH(THREADS, KERNEL, ...)                                                                              \
    do {                                                                                                               \
        if (causal)                                                                                                    \
            hipLaunchKernelGGL((KERNEL<D, DT_IN, DT_OUT, true __VA_ARGS__>), grid, dim3(THREADS), 0, stream, p);       \
        else                                                                                                           \
            hipLaunchKernelGGL((KERNEL<D, DT_IN, DT_OUT, false __VA_ARGS__>), grid, dim3(THREADS), 0, stream, p);      \
    } while (0)
#define NAUT_COMMA ,
    if constexpr (D > 128) {
        if (variant == V_W8Q32)
            NAUT_LAUNCH(512, naut_fwd_kernel_bm128, NAUT_COMMA 8);
        else
            NAUT_LAUNCH(256, naut_fwd_kernel_bm128, NAUT_COMMA 4);
    } else if (variant == V_BM128) {
        if (groups == 4)
            NAUT_LAUNCH(512, naut_fwd_kernel_bm128, NAUT_COMMA 2 NAUT_COMMA 4);
        else if (groups == 2)
            NAUT_LAUNCH(512, naut_fwd_kernel_bm128, NAUT_COMMA 4 NAUT_COMMA 2);
        else
            NAUT_LAUNCH(256, naut_fwd_kernel_bm128, NAUT_COMMA 4);
    } else if (variant == V_W4Q32) {
        if (groups == 2)
            NAUT_LAUNCH(512, naut_fwd_kernel_pipe, NAUT_COMMA 1 NAUT_COMMA 4 NAUT_COMMA 2);
        else
            NAUT_LAUNCH(256, naut_fwd_kernel_pipe, NAUT_COMMA 1 NAUT_COMMA 4);
    } else {
        if constexpr (D <= 64)
            NAUT_LAUNCH(256, naut_fwd_kernel_pipe, NAUT_COMMA 2 NAUT_COMMA 4);
        else
            NAUT_LAUNCH(512, naut_fwd_kernel_pipe, NAUT_COMMA 1 NAUT_COMMA 8);
    }
#undef NAUT_COMMA
#undef NAUT_LAUNCH
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess)
        return fail_launch(e);
    return NAUT_OK;
}

}  // namespace naut_k

#endif  // NAUT_ATTN_KERNELS_H
