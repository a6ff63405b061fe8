// naut_decode.hip -- decode-time attention for gfx950 (MI355X): a few new query positions per head
// against a long key/value cache (the paper's second workload, "DC", Section 6).
//
// The work is bound by reading K and V once from HBM, not by the matrix pipes, so the key axis is
// split across work-groups (and again across the eight wavefronts of a work-group): every wavefront
// streams its own 32-key blocks of K and V through a private buffer of each in LDS with direct
// global->LDS loads (no work-group barrier in the loop), runs the same transposed MFMA formulation
// as the prefill kernels on them (S^T = K.Q^T, online softmax with a lazily moved reference maximum,
// O^T += V^T.P^T), and the partial (O, m, l) triples are merged with the split-merge identity of
// softmax, first across the wavefronts through LDS, then, if there is more than one split, across the
// splits by a second small kernel that reads them from a caller-provided workspace.
//
// Query heads that share a K/V head (grouped-query attention) and the Sq positions of each form the
// rows of one MFMA tile: for a fixed (batch, K/V head) the Hq/Hkv * Sq query rows are contiguous in
// memory, so they are simply rows 0..R-1 of a [R][D] matrix, taken 32 at a time.
#include <hip/hip_runtime.h>

#include <atomic>
#include <cmath>
#include <cstdint>
#include <cstdio>

#include "naut_attn.h"
#include "naut_common.h"

namespace {

using namespace naut;

constexpr int DEC_WAVES = 8;               // wavefronts of a split kernel, each with LDS for a block of K and one of V
constexpr int MRG_WAVES = 4;               // wavefronts of the merge kernel
constexpr int MRG_THREADS = MRG_WAVES * 64;
constexpr int DEC_ROWS = 32;               // query rows per work-group (one MFMA tile)
constexpr int DEC_BLK = 32;                // keys per block
// The reference maximum of the 16-bit kernel moves whenever a row's maximum grows: the largest P of a row is
// then exactly 1 and carries no rounding error into O (with a reference that lags, the largest P is an
// arbitrary number whose rounding to 16 bit, up to 2^-8 relative in bf16, goes into O but not into l).  The
// rescaling this costs is vector work that a kernel bound by reading the cache has to spare.
constexpr float DEC_TAU = 0.0f;
constexpr float DEC_M_INIT = -1.0e30f;     // finite stand-in for "no maximum yet"
#ifndef NAUT_DEC_TARGET
#define NAUT_DEC_TARGET 256
#endif
constexpr int DEC_TARGET_WGS = NAUT_DEC_TARGET;  // work-groups of a round: one per CU (LDS; the 66 KB of D = 64 let two share one)

struct DecodeParams {
    const void* q;
    const void* k;
    const void* v;
    void* o;
    float* lse;
    float* ws;     // workspace: partial O [nparts][32][D], then m [nparts][32], then l [nparts][32]
    int B, Hq, Hkv, Sq, Sk;
    int R;         // query rows per (batch, K/V head) = Hq/Hkv * Sq
    int nchunks;   // ceil(R / 32)
    int nsplit;    // splits of the key axis
    int bps;       // blocks per split (a multiple of half the wavefronts)
    int causal;
    float c;       // scale * log2(e) (FP8: times descale_q * descale_k), > 0
    float dv;      // factor on O: 1 (16-bit inputs) or descale_v (FP8)
    int out_f32;   // O is fp32 (otherwise the 16-bit type of the inputs; FP8: bf16)
    // byte strides of batch, head and sequence position (the D axis is contiguous)
    long long q_bs, q_hs, k_bs, k_hs, v_bs, v_hs, o_bs, o_hs;
    int q_rs, k_rs, v_rs, o_rs;
    // The kernels are compiled for D = 64, 128 or 256 (FP8: 64 or 128); a smaller head dimension runs on the next wider one:
    // cpr 16-byte chunks of every row are real, the chunks of Q beyond them read as zero, those of K and
    // V repeat a real chunk (they meet zeros of Q, or end in columns of O that are not stored).
    int cpr;
};

__device__ __forceinline__ float half_sum_f(float x)
{
    float a = x, b = x;
    asm volatile(NAUT_NOP_SHORT "v_permlane32_swap_b32 %0, %1" : "+v"(a), "+v"(b));
    return a + b;
}

// Tail of a split kernel: the wavefronts' partial (O, m, l) are merged through LDS (each wavefront
// reuses its own, now idle, region of REGION bytes) and the work-group's partial goes to the workspace.
// m is the reference maximum the wavefront's l and O are relative to (log2 units).
// With a single split that partial is the result: it is divided by l and stored as O right here, and there is no merge
// kernel (32/8 heads, D = 128, 512 keys, B = 40, the same single split: 27.9 -> 24.5 us).
template <int D, int REGION, int NW, int DT_IN>
__device__ __forceinline__ void merge_wavefronts(unsigned char* smem, float (&ml_lds)[NW][2 * DEC_ROWS], const f32x16_t (&oacc)[D / 32],
                                                 float m_run, float l_run, const DecodeParams& p, int bhk, int chunk, int split)
{
    constexpr int DB = D / 32;
    constexpr int Q4 = D / 4;  // 16-byte pieces of a row of O
    static_assert(DEC_ROWS * D * 4 <= REGION, "the wavefront's partial fits its LDS region");
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31;
    const int h = lane >> 5;
    const int rows = p.R - chunk * DEC_ROWS < DEC_ROWS ? p.R - chunk * DEC_ROWS : DEC_ROWS;  // the rest is padding
    // ---- merge the wavefronts through LDS (each reuses its own, now idle, region) ----
    // piece q4 of row r; the position is XOR-ed with the row, so that neither side conflicts
    auto piece = [&](int w, int r, int q4) { return (f32x4_t*)(smem + w * REGION) + r * Q4 + (q4 ^ (r & 7)); };
    const float l_tot = half_sum_f(l_run);
    if (l32 < rows) {
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int gq = 0; gq < 4; ++gq)
                *piece(wave, l32, 8 * db + 2 * gq + h) =
                    f32x4_t{oacc[db][4 * gq + 0], oacc[db][4 * gq + 1], oacc[db][4 * gq + 2], oacc[db][4 * gq + 3]};
    }
    if (h == 0) {
        ml_lds[wave][l32] = m_run;
        ml_lds[wave][DEC_ROWS + l32] = l_tot;
    }
    __syncthreads();

    // (row, M pieces Q4 / M apart) items, dealt to the threads; partial written to the workspace
    const size_t nparts = (size_t)p.B * p.Hkv * p.nchunks * p.nsplit;
    const size_t part = ((size_t)bhk * p.nchunks + chunk) * p.nsplit + split;
    auto merge = [&](auto PIECES) {
        constexpr int M = decltype(PIECES)::value, G = Q4 / M;
        for (int item = tid; item < rows * G; item += NW * 64) {
            const int r_out = item / G, g = item % G;
            float mw[NW], lw[NW];
            f32x4_t x[NW][M];
            float m = DEC_M_INIT;
#pragma unroll
            for (int w = 0; w < NW; ++w) {
                mw[w] = ml_lds[w][r_out];
                lw[w] = ml_lds[w][DEC_ROWS + r_out];
#pragma unroll
                for (int i = 0; i < M; ++i)
                    x[w][i] = *piece(w, r_out, g + i * G);
                m = fmaxf(m, mw[w]);
            }
            float l = 0.f;
            f32x4_t acc[M];
#pragma unroll
            for (int i = 0; i < M; ++i)
                acc[i] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int w = 0; w < NW; ++w) {
                const float f = __builtin_amdgcn_exp2f(mw[w] - m);
                l += f * lw[w];
#pragma unroll
                for (int i = 0; i < M; ++i)
                    acc[i] += x[w][i] * f;
            }
            if (p.nsplit == 1) {
                const int r = chunk * DEC_ROWS + r_out;
                const float inv_l = p.dv / l;
                // lse is dense [B][Hq][Sq]: the R rows of (batch, K/V head) bhk are contiguous there
                if (p.lse != nullptr && g == 0)
                    p.lse[(size_t)bhk * p.R + r] = (m + __builtin_amdgcn_logf(l)) * 0.6931471805599453f;
                const int b = bhk / p.Hkv, hk = bhk % p.Hkv;
                const int head = hk * (p.Hq / p.Hkv) + r / p.Sq, pos = r % p.Sq;
                unsigned char* orow = (unsigned char*)p.o + b * p.o_bs + head * p.o_hs + (long long)pos * p.o_rs;
#pragma unroll
                for (int i = 0; i < M; ++i) {
                    const int d = 4 * (g + i * G);
                    if (d >= p.cpr * 8)
                        break;  // padding columns of a narrower head dimension
                    const f32x4_t y = acc[i] * inv_l;
                    if (p.out_f32)
                        *(f32x4_t*)(orow + d * 4) = y;
                    else
                        *(i32x2_t*)(orow + d * 2) = i32x2_t{In<DT_IN>::pack2(y.x, y.y), In<DT_IN>::pack2(y.z, y.w)};
                }
                continue;
            }
#pragma unroll
            for (int i = 0; i < M; ++i)
                *(f32x4_t*)(p.ws + (part * DEC_ROWS + r_out) * D + 4 * (g + i * G)) = acc[i];
            if (g == 0) {
                float* ws_m = p.ws + nparts * DEC_ROWS * D;
                float* ws_l = ws_m + nparts * DEC_ROWS;
                ws_m[part * DEC_ROWS + r_out] = m;
                ws_l[part * DEC_ROWS + r_out] = l;
            }
        }
    };
    // as few pieces per thread as take the rows in one pass, so that few threads are idle (a row's exponentials and latency
    // are shared by its pieces); at most four
    constexpr int FULL = DEC_ROWS * Q4 / (NW * 64);
    if (FULL == 1 || rows * Q4 <= NW * 64)
        merge(std::integral_constant<int, 1>{});
    else if (FULL == 2 || rows * Q4 <= 2 * NW * 64)
        merge(std::integral_constant<int, 2>{});
    else
        merge(std::integral_constant<int, 4>{});
}

// wavefronts of the split kernel (or half as many: see half_waves); the two LDS blocks of one are 32 KB at D = 256
constexpr int dec_waves(int D) { return D > 128 ? DEC_WAVES / 2 : DEC_WAVES; }

// Wavefronts per SIMD that a split kernel has to leave registers for: two work-groups of half the wavefronts share a CU (D =
// 64: four, D > 128: of two wavefronts each).  Left to itself the compiler took 260 registers for FP8 at D = 128, one
// work-group, and 136 and 144 at D = 64, three; with the bound 168, 113 and 112, none spilled.
constexpr int dec_waves_per_simd(int D) { return D > 128 ? 1 : D > 64 ? 2 : 4; }

// A wavefront has one buffer for K and one for V: the next block's K is requested when this block's K fragments are in
// registers, its V when the V fragments are.  Twice as many wavefronts as with two buffers of each keep as many bytes in
// flight (128 KB per CU), and cover a block's scores, softmax and P.V with each other's loads; the first block's loads
// are out before Q's.  Against four wavefronts with two buffers (us a call, 32/8 heads, D = 128): 20 caches of 2000 keys 34.1 ->
// 31.0, 40 of 500 24.9 -> 22.1; D = 256, 16/8 heads, 256 keys 11.6 -> 10.7.  Long caches gain nothing (8 of 16384 94.2 / 94.1).
template <int D, int DT_IN, int NW>
__global__ __launch_bounds__(NW * 64, (dec_waves_per_simd(D))) void naut_decode_split_kernel(const DecodeParams p)
{
    using T = In<DT_IN>;
    constexpr int REGION = 2 * DEC_BLK * D * 2;  // LDS of a wavefront
    constexpr int ROWB = D * 2;
    constexpr int BLKB = DEC_BLK * ROWB;   // one 32-key block of K or V
    constexpr int KS = D / 16;
    constexpr int DB = D / 32;
    constexpr int NLD = BLKB / 1024;       // direct loads (1 KB each) per block and operand

    __shared__ __attribute__((aligned(1024))) unsigned char smem[NW * REGION];  // per wavefront: K, V
    __shared__ float ml_lds[NW][2 * DEC_ROWS];

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31;
    const int h = lane >> 5;

    const int split = blockIdx.x, chunk = blockIdx.y, bhk = blockIdx.z;
    const int b = bhk / p.Hkv, hk = bhk % p.Hkv;
    const int g = p.Hq / p.Hkv;
    const int Sk = p.Sk;
    const float c = p.c;

    // The R rows of this (batch, K/V head): row r is position r % Sq of query head hk*g + r / Sq.
    const unsigned char* qg = (const unsigned char*)p.q + b * p.q_bs + (long long)(hk * g) * p.q_hs;
    const unsigned char* kg = (const unsigned char*)p.k + b * p.k_bs + hk * p.k_hs;
    const unsigned char* vg = (const unsigned char*)p.v + b * p.v_bs + hk * p.v_hs;

    const int row = chunk * DEC_ROWS + l32;                 // the query row this lane owns
    const int row_ld = row < p.R ? row : p.R - 1;
    // last key this row may see: the Sq queries are the last positions of a sequence of Sk
    const int lim = p.causal ? Sk - p.Sq + (row_ld % p.Sq) : Sk - 1;

    i32x4_t qf[KS];
    auto load_q = [&]() {
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
            qf[ks] = ks * 2 + h < p.cpr
                         ? *(const i32x4_t*)(qg + (row_ld / p.Sq) * p.q_hs + (long long)(row_ld % p.Sq) * p.q_rs + ks * 32 + h * 16)
                         : i32x4_t{0, 0, 0, 0};
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
            asm volatile("" : "+v"(qf[ks]));
    };
    // Direct global->LDS loads: instruction n fills physical chunks 64n..64n+63 of the block, lane i
    // the chunk 64n+i, so the lane fetches the logical chunk that the swizzle maps there.
    // (row of the block, byte inside the row) of that logical chunk:
    int k_row[NLD], k_col[NLD], v_row[NLD], v_col[NLD];
#pragma unroll
    for (int n = 0; n < NLD; ++n) {
        const int P = n * 64 + lane;
        {
            const int line = P >> 4, pos = P & 15;
            const int key = D > 128 ? line >> 1 : line;                // the inverse of k_off
            const int off = ((line << 4) + (pos ^ (key & 15))) * 16;   // byte offset in a dense [32][D] block
            k_row[n] = off / ROWB;
            const int kc = off % ROWB / 16;
            k_col[n] = (kc < p.cpr ? kc : p.cpr - 1) * 16;
        }
        if constexpr (D >= 128) {
            const int r = P / (D / 8), cc = P % (D / 8);
            const int vc = cc ^ ((r & 3) << 2);
            v_row[n] = r;
            v_col[n] = (vc < p.cpr ? vc : p.cpr - 1) * 16;
        } else {
            const int r = P >> 3, cc = P & 7;
            const int vc = cc ^ (((r >> 1) & 1) << 2);
            v_row[n] = r;
            v_col[n] = (vc < p.cpr ? vc : p.cpr - 1) * 16;
        }
    }
    const unsigned lds0 = (unsigned)(uintptr_t)(NAUT_LDS unsigned char*)smem + (unsigned)(wave * REGION);
    unsigned char* my_lds = smem + wave * REGION;

    const int nblk = (Sk + DEC_BLK - 1) / DEC_BLK;
    const int blk_begin = split * p.bps;
    const int blk_end = blk_begin + p.bps < nblk ? blk_begin + p.bps : nblk;

    // K (OP = 0) or V (OP = 1) of a block into its buffer
    auto issue = [&](auto OP, int blk) {
        constexpr bool V = decltype(OP)::value != 0;
        const int rs = V ? p.v_rs : p.k_rs;
        const unsigned char* const base = (V ? vg : kg) + (size_t)blk * DEC_BLK * rs;
        const int rows_left = Sk - blk * DEC_BLK;  // >= 1
        const unsigned dst = lds0 + (V ? BLKB : 0);
#pragma unroll
        for (int n = 0; n < NLD; ++n) {
            int r = V ? v_row[n] : k_row[n];
            if (rows_left < DEC_BLK)  // ragged last block: re-read the last row instead of running past the end
                r = r < rows_left ? r : rows_left - 1;
            load_to_lds(dst + n * 1024, r * rs + (V ? v_col[n] : k_col[n]), base);
        }
    };
    constexpr std::integral_constant<int, 0> OPK{};
    constexpr std::integral_constant<int, 1> OPV{};

    f32x16_t oacc[DB];
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int r = 0; r < 16; ++r)
            oacc[db][r] = 0.f;
    float m_run = DEC_M_INIT;  // reference maximum, log2 units (already times c)
    float l_run = 0.f;         // this lane's share of the running sum (its 16 of every 32 keys)

    // This wavefront's blocks: blk_begin + wave, + NW, ...
    static_assert(2 * NLD < 64, "vmcnt field");
    int blk = blk_begin + wave;
    if (blk < blk_end) {
        issue(OPK, blk);
        issue(OPV, blk);
    }
    load_q();
    for (; blk < blk_end; blk += NW) {
        const bool more = blk + NW < blk_end;
        wait_loads<NLD>();  // this block's K; its V may still be on its way
        const unsigned char* kt = my_lds;
        const unsigned char* vt = kt + BLKB;

        f32x16_t s_;
#pragma unroll
        for (int r = 0; r < 16; ++r)
            s_[r] = 0.f;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            const i32x4_t kf = *(const i32x4_t*)(kt + k_off<D>(l32, ks * 2 + h));
            s_ = T::mfma(kf, qf[ks], s_);
        }
        if (more) {
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // the K fragments are in registers
            issue(OPK, blk + NW);
        }
        const int key0 = blk * DEC_BLK;
        if (key0 + DEC_BLK - 1 > Sk - p.Sq || key0 + DEC_BLK > Sk) {  // some row's limit may fall inside the block
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int key = key0 + 8 * (r >> 2) + 4 * h + (r & 3);
                s_[r] = key > lim ? -INFINITY : s_[r];
            }
        }
        float mx = s_[0];
#pragma unroll
        for (int r = 1; r < 16; ++r)
            mx = fmaxf(mx, s_[r]);
        mx = half_max(mx);
        const float m_cand = mx * c;  // -inf if the whole block is masked for this row
        if (__builtin_amdgcn_ballot_w64(m_cand > m_run + DEC_TAU) != 0) {
            const float m_new = fmaxf(m_run, m_cand);
            const float alpha = __builtin_amdgcn_exp2f(m_run - m_new);  // repair factor
            m_run = m_new;
            l_run *= alpha;
#pragma unroll
            for (int db = 0; db < DB; ++db)
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    oacc[db][r] *= alpha;
        }
        float psum = 0.f;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            s_[r] = __builtin_amdgcn_exp2f(__builtin_fmaf(s_[r], c, -m_run));
            psum = r == 0 ? s_[r] : psum + s_[r];
        }
        l_run += psum;
        if (more)
            wait_loads<NLD>();  // this block's V; the next one's K may still be on its way
        else
            wait_loads<0>();
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const int r0 = t * 8;
            const i32x4_t pb = {T::pack2(s_[r0 + 0], s_[r0 + 1]), T::pack2(s_[r0 + 2], s_[r0 + 3]),
                                T::pack2(s_[r0 + 4], s_[r0 + 5]), T::pack2(s_[r0 + 6], s_[r0 + 7])};
#pragma unroll
            for (int db = 0; db < DB; ++db) {
                const i32x4_t vf = load_vt_frag<D>(vt, t * 16, db, lane);
                oacc[db] = T::mfma(vf, pb, oacc[db]);
            }
        }
        if (more) {
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // the V fragments too
            issue(OPV, blk + NW);
        }
    }

    merge_wavefronts<D, REGION, NW, DT_IN>(smem, ml_lds, oacc, m_run, l_run, p, bhk, chunk, split);
}

// The same split kernel on FP8 (E4M3) Q, K and V: 64-key blocks (one 32x32x64 MFMA covers 64 keys of
// P.V), the LDS layouts, transposed byte reads and the 2^7 scaling of P of the FP8 prefill kernel, the
// blocks dealt to the wavefronts and one buffer of K and V each, exactly as above; strides and narrower heads
// as above too, in 16-byte chunks of 16 values (p.cpr counts 8 values: two per chunk here).
// bps counts 64-key blocks here.  The partial's reference maximum is stored as m - 7, which makes its l
// and O (both carry the factor 2^7) relative to it in the plain sense the merge kernel expects.
constexpr int DEC8_BLK = 64;
constexpr float DEC8_TAU = 1.0f;      // P * 2^7 <= 2^(1+7) = 256 < 448, the largest E4M3 value
constexpr float DEC8_P_SHIFT = 7.0f;

template <int D, int NW>
__global__ __launch_bounds__(NW * 64, (dec_waves_per_simd(D))) void naut_decode_split_fp8_kernel(const DecodeParams p)
{
    constexpr int BLKB = DEC8_BLK * D;     // bytes of one 64-key block of K or V
    constexpr int REGION = 2 * BLKB;
    constexpr int KS = D / 64;
    constexpr int DB = D / 32;
    constexpr int CPR = D / 16;            // 16-byte chunks per row
    constexpr int NLD = BLKB / 1024;       // direct loads (1 KB each) per block and operand

    __shared__ __attribute__((aligned(1024))) unsigned char smem[NW * REGION];  // per wavefront: K, V
    __shared__ float ml_lds[NW][2 * DEC_ROWS];

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31;
    const int h = lane >> 5;

    const int split = blockIdx.x, chunk = blockIdx.y, bhk = blockIdx.z;
    const int b = bhk / p.Hkv, hk = bhk % p.Hkv;
    const int g = p.Hq / p.Hkv;
    const int Sk = p.Sk;
    const float c = p.c;

    // The R rows of this (batch, K/V head): row r is position r % Sq of query head hk*g + r / Sq.
    const unsigned char* qg = (const unsigned char*)p.q + b * p.q_bs + (long long)(hk * g) * p.q_hs;
    const unsigned char* kg = (const unsigned char*)p.k + b * p.k_bs + hk * p.k_hs;
    const unsigned char* vg = (const unsigned char*)p.v + b * p.v_bs + hk * p.v_hs;
    const int cpr16 = p.cpr >> 1;  // real 16-byte chunks per row

    const int row = chunk * DEC_ROWS + l32;                 // the query row this lane owns
    const int row_ld = row < p.R ? row : p.R - 1;
    const int lim = p.causal ? Sk - p.Sq + (row_ld % p.Sq) : Sk - 1;  // last key this row may see

    // Q^T fragments (MFMA B operand): lane holds q[row][64*ks + 32*h .. +32]
    i32x8_t qf[KS];
    auto load_q = [&]() {
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            const unsigned char* qrow = qg + (row_ld / p.Sq) * p.q_hs + (long long)(row_ld % p.Sq) * p.q_rs;
            const int c0 = ks * 4 + h * 2;  // this lane's two 16-byte chunks of the row
            const i32x4_t lo = c0 < cpr16 ? *(const i32x4_t*)(qrow + c0 * 16) : i32x4_t{0, 0, 0, 0};
            const i32x4_t hi = c0 + 1 < cpr16 ? *(const i32x4_t*)(qrow + c0 * 16 + 16) : i32x4_t{0, 0, 0, 0};
            qf[ks] = i32x8_t{lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
        }
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
            asm volatile("" : "+v"(qf[ks]));
    };
    // Direct global->LDS loads: instruction n fills physical 16-byte chunks 64n..64n+63 of the block, lane i
    // the chunk 64n+i, so the lane fetches the logical chunk that k8_off / v8_off place there.
    int k_row[NLD], k_col[NLD], v_row[NLD], v_col[NLD];
#pragma unroll
    for (int n = 0; n < NLD; ++n) {
        const int P = n * 64 + lane;
        const int r = P / CPR, pc = P % CPR;
        k_row[n] = r;
        const int kc = pc ^ ((r >> 1) & (CPR - 1));  // logical chunk that k8_off places at position pc
        k_col[n] = (kc < cpr16 ? kc : cpr16 - 1) * 16;
        const int key = D == 128 ? (((r >> 1) & 1) | (((r >> 3) & 1) << 1)) : ((r >> 3) & 1);
        v_row[n] = r;
        const int vc = (((pc >> 1) ^ key) << 1) + (pc & 1);  // likewise for v8_off (32-byte chunks, two halves)
        v_col[n] = (vc < cpr16 ? vc : cpr16 - 1) * 16;
    }
    const unsigned lds0 = (unsigned)(uintptr_t)(NAUT_LDS unsigned char*)smem + (unsigned)(wave * REGION);
    unsigned char* my_lds = smem + wave * REGION;

    const int nblk = (Sk + DEC8_BLK - 1) / DEC8_BLK;
    const int blk_begin = split * p.bps;
    const int blk_end = blk_begin + p.bps < nblk ? blk_begin + p.bps : nblk;

    // K (OP = 0) or V (OP = 1) of a block into its buffer
    auto issue = [&](auto OP, int blk) {
        constexpr bool V = decltype(OP)::value != 0;
        const int rs = V ? p.v_rs : p.k_rs;
        const unsigned char* const base = (V ? vg : kg) + (size_t)blk * DEC8_BLK * rs;
        const int rows_left = Sk - blk * DEC8_BLK;  // >= 1
        const unsigned dst = lds0 + (V ? BLKB : 0);
#pragma unroll
        for (int n = 0; n < NLD; ++n) {
            int r = V ? v_row[n] : k_row[n];
            if (rows_left < DEC8_BLK)  // ragged last block: re-read the last row instead of running past the end
                r = r < rows_left ? r : rows_left - 1;
            load_to_lds(dst + n * 1024, r * rs + (V ? v_col[n] : k_col[n]), base);
        }
    };
    constexpr std::integral_constant<int, 0> OPK{};
    constexpr std::integral_constant<int, 1> OPV{};

    // lane-constant parts of the transposed V reads (as in the FP8 prefill kernel)
    const int i16 = lane & 15;
    const int v_e = i16 >> 1;
    const int v_key = 4 * h + (v_e & 3) + ((v_e >> 2) << 3);
    const int v_byte = 16 * ((lane >> 4) & 1) + 8 * (i16 & 1);

    f32x16_t oacc[DB];
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int r = 0; r < 16; ++r)
            oacc[db][r] = 0.f;
    float m_run = DEC_M_INIT;
    float l_run = 0.f;
    i32x8_t pb = {0, 0, 0, 0, 0, 0, 0, 0};

    static_assert(2 * NLD < 64, "vmcnt field");
    int blk = blk_begin + wave;
    if (blk < blk_end) {
        issue(OPK, blk);
        issue(OPV, blk);
    }
    load_q();
    for (; blk < blk_end; blk += NW) {
        const bool more = blk + NW < blk_end;
        wait_loads<NLD>();  // this block's K; its V may still be on its way
        const unsigned char* kt = my_lds;
        const unsigned char* vt = kt + BLKB;

        f32x16_t sacc[2];
#pragma unroll
        for (int kb = 0; kb < 2; ++kb) {
#pragma unroll
            for (int r = 0; r < 16; ++r)
                sacc[kb][r] = 0.f;
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                const int rw = kb * 32 + l32, c0 = ks * 4 + h * 2;
                const i32x4_t lo = *(const i32x4_t*)(kt + k8_off<D>(rw, c0));
                const i32x4_t hi = *(const i32x4_t*)(kt + k8_off<D>(rw, c0 + 1));
                const i32x8_t kf = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
                sacc[kb] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(kf, qf[ks], sacc[kb], 0, 0, 0, 0, 0, 0);
            }
        }
        if (more) {
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // the K fragments are in registers
            issue(OPK, blk + NW);
        }
        const int key0 = blk * DEC8_BLK;
        if (key0 + DEC8_BLK - 1 > Sk - p.Sq || key0 + DEC8_BLK > Sk) {  // some row's limit may fall inside the block
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int key = key0 + kb * 32 + 8 * (r >> 2) + 4 * h + (r & 3);
                    sacc[kb][r] = key > lim ? -INFINITY : sacc[kb][r];
                }
        }
        float mx = sacc[0][0];
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
            for (int r = 0; r < 16; ++r)
                mx = fmaxf(mx, sacc[kb][r]);
        mx = half_max(mx);
        const float m_cand = mx * c;  // -inf if the whole block is masked for this row
        if (__builtin_amdgcn_ballot_w64(m_cand > m_run + DEC8_TAU) != 0) {
            const float m_new = fmaxf(m_run, m_cand);
            const float alpha = __builtin_amdgcn_exp2f(m_run - m_new);  // repair factor
            m_run = m_new;
            l_run *= alpha;
#pragma unroll
            for (int db = 0; db < DB; ++db)
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    oacc[db][r] *= alpha;
        }
        const float shift = DEC8_P_SHIFT - m_run;
        float psum = 0.f;
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const float pv = __builtin_amdgcn_exp2f(__builtin_fmaf(sacc[kb][r], c, shift));
                sacc[kb][r] = pv;
                psum = (kb | r) == 0 ? pv : psum + pv;
            }
        l_run += psum;
        if (more)
            wait_loads<NLD>();  // this block's V; the next one's K may still be on its way
        else
            wait_loads<0>();
#pragma unroll
        for (int w = 0; w < 8; ++w) {
            const int kb = w >> 2, r0 = (w & 3) * 4;
            pb[w] = pack4_fp8(sacc[kb][r0 + 0], sacc[kb][r0 + 1], sacc[kb][r0 + 2], sacc[kb][r0 + 3], pb[w]);
        }
#pragma unroll
        for (int db = 0; db < DB; ++db) {
            i32x8_t vf;
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const int key = 32 * (t >> 1) + 16 * (t & 1) + v_key;
                const i32x2_t x = __builtin_amdgcn_ds_read_tr8_b64_v2i32(
                    (NAUT_LDS i32x2_t*)(vt + v8_off<D>(key, db) + v_byte));
                vf[2 * t] = x.x;
                vf[2 * t + 1] = x.y;
            }
            oacc[db] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(vf, pb, oacc[db], 0, 0, 0, 0, 0, 0);
        }
        if (more) {
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // the V fragments too
            issue(OPV, blk + NW);
        }
    }
    merge_wavefronts<D, REGION, NW, NAUT_BF16>(smem, ml_lds, oacc, m_run - DEC8_P_SHIFT, l_run, p, bhk, chunk, split);
}

// One work-group (four wavefronts) per query row: merges the nsplit > 1 partials of the row, divides by l
// once, stores O and lse.  Wavefront w takes splits w, w+4, ...; lanes run over D.  Bound by the latency of its
// loads: with the maximum over all splits found in a pass of its own, as it was, 3.7 us for 17 splits of 32 rows and 6.4
// for 128 of 8 (D = 128), now 3.0 and 4.7.
// BATCH: the most splits that a wavefront loads at a time (see launch_merge).
template <int D, int DT_OUT, int BATCH>
__global__ __launch_bounds__(MRG_THREADS) void naut_decode_merge_kernel(const DecodeParams p)
{
    __shared__ float red_m[MRG_WAVES];
    __shared__ float red_l[MRG_WAVES];
    __shared__ __attribute__((aligned(16))) float red_o[MRG_WAVES][D];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int r = blockIdx.x;    // row inside the (batch, K/V head): 0 .. R-1
    const int bhk = blockIdx.y;
    const int chunk = r / DEC_ROWS, rr = r % DEC_ROWS;
    const size_t nparts = (size_t)p.B * p.Hkv * p.nchunks * p.nsplit;
    const size_t part0 = ((size_t)bhk * p.nchunks + chunk) * p.nsplit;
    const float* ws_m = p.ws + nparts * DEC_ROWS * D + part0 * DEC_ROWS + rr;   // stride DEC_ROWS per split
    const float* ws_l = ws_m + nparts * DEC_ROWS;
    const float* ws_o = p.ws + (part0 * DEC_ROWS + rr) * D;                      // stride DEC_ROWS*D per split

    // Every wavefront adds up its splits, BATCH at a time, relative to the largest m it has met; nothing of a batch
    // depends on another load, so up to MRG_WAVES * BATCH splits cost one round trip to memory.
    constexpr int EPT = D / 64;  // elements per lane
    typedef float fe_t __attribute__((ext_vector_type(EPT)));
    fe_t acc = (fe_t)(0.f);
    float M = DEC_M_INIT, L = 0.f;
    for (int s0 = wave; s0 < p.nsplit; s0 += MRG_WAVES * BATCH) {
        float m[BATCH], l[BATCH];
        fe_t x[BATCH];
#pragma unroll
        for (int u = 0; u < BATCH; ++u) {
            const int s = s0 + u * MRG_WAVES;
            const size_t sc = s < p.nsplit ? s : s0;  // past the end: repeats a split, not added
            m[u] = ws_m[sc * DEC_ROWS];
            l[u] = ws_l[sc * DEC_ROWS];
            x[u] = *(const fe_t*)(ws_o + sc * DEC_ROWS * D + lane * EPT);
        }
        float m_new = M;
#pragma unroll
        for (int u = 0; u < BATCH; ++u)
            m_new = fmaxf(m_new, m[u]);
        const float alpha = __builtin_amdgcn_exp2f(M - m_new);
        M = m_new;
        L *= alpha;
        acc *= alpha;
#pragma unroll
        for (int u = 0; u < BATCH; ++u) {
            const bool real = s0 + u * MRG_WAVES < p.nsplit;
            const float f = __builtin_amdgcn_exp2f(m[u] - M);
            L += real ? f * l[u] : 0.f;
            acc += real ? f * x[u] : (fe_t)(0.f);
        }
    }
    *(fe_t*)&red_o[wave][lane * EPT] = acc;
    if (lane == 0) {
        red_m[wave] = M;
        red_l[wave] = L;
    }
    __syncthreads();
    if (wave != 0)
        return;
#pragma unroll
    for (int w = 1; w < MRG_WAVES; ++w)
        M = fmaxf(M, red_m[w]);
    acc = (fe_t)(0.f);
    L = 0.f;
#pragma unroll
    for (int w = 0; w < MRG_WAVES; ++w) {
        const float f = __builtin_amdgcn_exp2f(red_m[w] - M);
        L += f * red_l[w];
        acc += f * *(const fe_t*)&red_o[w][lane * EPT];
    }
    const float inv_l = p.dv / L;
    // lse is dense [B][Hq][Sq]: the R rows of (batch, K/V head) bhk are contiguous there
    if (p.lse != nullptr && lane == 0)
        p.lse[(size_t)bhk * p.R + r] = (M + __builtin_amdgcn_logf(L)) * 0.6931471805599453f;
    const int b = bhk / p.Hkv, hk = bhk % p.Hkv;
    const int head = hk * (p.Hq / p.Hkv) + r / p.Sq, pos = r % p.Sq;
    unsigned char* orow = (unsigned char*)p.o + b * p.o_bs + head * p.o_hs + (long long)pos * p.o_rs;
    if (lane * EPT >= p.cpr * 8)
        return;  // padding columns of a narrower head dimension
    if constexpr (DT_OUT == NAUT_F32) {
        float* og = (float*)orow + lane * EPT;
#pragma unroll
        for (int e = 0; e < EPT; ++e)
            og[e] = acc[e] * inv_l;
    } else if constexpr (EPT == 4) {
        i32x2_t* og = (i32x2_t*)(orow + lane * EPT * 2);
        *og = i32x2_t{In<DT_OUT>::pack2(acc[0] * inv_l, acc[1] * inv_l), In<DT_OUT>::pack2(acc[2] * inv_l, acc[3] * inv_l)};
    } else if constexpr (EPT == 2) {
        int* og = (int*)(orow + lane * EPT * 2);
        *og = In<DT_OUT>::pack2(acc[0] * inv_l, acc[1] * inv_l);
    } else {
        unsigned short* og = (unsigned short*)orow + lane;
        *og = (unsigned short)(In<DT_OUT>::pack2(acc[0] * inv_l, 0.f) & 0xffff);
    }
}

// A batch reads a split again for each it has too many, so few splits take a small one.  Two or four splits, in a batch of
// eight / of one (us a call, D = 128): 5 caches of 8 heads, 1024 keys 11.8 / 11.2, 15 caches, 512 keys, 8 query heads to a
// K/V head 13.9 / 13.0 (13.5 before there were batches).  At 16 splits four are no better than eight.  A kernel of its own
// for each: one that picks the batch as it runs is 6 to 12 % of the call slower on many splits (one cache of one head,
// 131072 keys 24.5 / 27.3).
template <int D, int DT_OUT>
void launch_merge(const DecodeParams& p, hipStream_t stream)
{
    const dim3 grid((unsigned)p.R, (unsigned)(p.B * p.Hkv));
    if (p.nsplit <= MRG_WAVES)
        hipLaunchKernelGGL((naut_decode_merge_kernel<D, DT_OUT, 1>), grid, dim3(MRG_THREADS), 0, stream, p);
    else if (p.nsplit <= 2 * MRG_WAVES)
        hipLaunchKernelGGL((naut_decode_merge_kernel<D, DT_OUT, 2>), grid, dim3(MRG_THREADS), 0, stream, p);
    else
        hipLaunchKernelGGL((naut_decode_merge_kernel<D, DT_OUT, 8>), grid, dim3(MRG_THREADS), 0, stream, p);
}

struct Plan {
    int nchunks, nsplit, bps;
    size_t ws_bytes;    // workspace asked for
    size_t ws_least;    // the least that is taken (see make_plan)
};

// Scratch of naut_attn_decode_static: the split partials live in this file-scope device array instead of a
// caller-provided workspace.  Every GPU the library runs on holds its own copy at its own address for the
// life of the process.  In host code the array's name is only a handle for hipGetSymbolAddress: the device
// address it returns (taken once per device, with that device current) is what kernels and copies get.
constexpr size_t DEC_STATIC_BYTES = 16u << 20;
static __device__ __align__(256) unsigned char scratch[DEC_STATIC_BYTES];
constexpr int DEC_MAX_DEVICES = 64;
std::atomic<void*> g_scratch_ptr[DEC_MAX_DEVICES];

// Device address of `scratch` on the current device (NULL and an error message on failure).
void* static_scratch(int* err)
{
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) {
        *err = fail_launch(e);
        return nullptr;
    }
    if (dev < 0 || dev >= DEC_MAX_DEVICES) {
        *err = fail(NAUT_ERR_UNSUPPORTED, "device ordinal beyond the library's per-device table");
        return nullptr;
    }
    void* ptr = g_scratch_ptr[dev].load(std::memory_order_acquire);
    if (ptr == nullptr) {
        e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
        if (e != hipSuccess || ptr == nullptr) {
            snprintf(g_err, sizeof g_err, "hipGetSymbolAddress(scratch) failed: %s", hipGetErrorString(e));
            *err = NAUT_ERR_HIP;
            return nullptr;
        }
        g_scratch_ptr[dev].store(ptr, std::memory_order_release);  // every thread computes the same value
    }
    return ptr;
}

// D: the width the kernels are compiled for (64, 128 or 256); Sk counts keys in units that make a block DEC_BLK of them.
//
// How many splits: a work-group occupies a CU (LDS), so the work-groups run in rounds of 256 (at D = 64 two fit a CU; the
// rounds below price that width too, and where the first count is more than one round pick fewer splits than would be
// fastest: 33 caches of 8 heads, 4096 keys 61.7 us with two, 55.2 with eight, 68.0 before), and a last round of n of
// them lasts longer than its n/256 of a full round's bytes: one CU streams at most about 2.2 times its even share of the
// memory's rate.  The candidates are the counts that fill one, two, three or four rounds without starting another; the
// time of each is priced from three measurements: a full chip takes 2.9 us for 64 KB per CU, a further round about 2 us
// of fill and drain, the merge kernel with its launch about 7 us (a single split needs none).  Measured with the first
// count that reaches 256 work-groups, as it was / the one picked here (us a call, 32/8 heads, one position, D = 128):
// 4096 keys, B = 9 42.7 / 33.6, B = 12 52.0 / 43.2, B = 20 77.0 / 63.8, B = 33 133 / 113, B = 40 139 / 124.
// The first count stands, and nothing is priced, where it fills whole rounds (base divides 256) and where a fuller split would
// leave a wavefront without a block.
//
// A cache of at most two blocks for each of all wavefronts is one split, however few work-groups that makes: a second 128 KB
// takes one CU about 2.5 us, the merge kernel 7 us where the host paces the calls and 3 us on a stream that runs behind it.
// Two splits as it was / one (us a call, D = 128, 32/8 heads, one position): 512 keys 10.7 / 8.4 (from a graph 9.2 / 8.1), 12
// caches of 512 keys 11.9 / 10.1.  At 768 keys one split is no faster where a graph holds the calls (9.4 / 9.2) and slower
// with more of them (8 caches 11.6 / 12.4).  At D = 64 four blocks a wavefront would be as many bytes, but they are fewer
// partials than four splits of four wavefronts have, and every partial has a reference maximum of its own, whose key's P is
// exactly 1: error against 64 bits 1.06 of that of four splits at 1000 keys, 1.1 to 1.3 at four times the usual scale
// (kernel time 0.94 to 0.98 of it; FP8 at 2000 keys 1.08).
//
// The workspace must hold the least count's partials (the first count that reaches 256 work-groups); with less room than
// the picked count needs, the best candidate that fits is taken.  No count takes more than DEC_MAX_PARTS partials unless
// the least does, so the 16 MiB static scratch holds the picked count wherever it holds the least (D <= 128).  Both sizes
// are those of the counts above also where one split is taken and nothing is written there.
constexpr unsigned DEC_MAX_PARTS = 960;

bool make_plan(int B, int Hq, int Hkv, int Sq, int Sk, int D, int block_bytes, size_t room, Plan* pl)
{
    const unsigned W = dec_waves(D), G = W / 2;  // 8 or 4; a split is a multiple of G blocks
    const long long R = (long long)(Hq / Hkv) * Sq;
    const long long nchunks = (R + DEC_ROWS - 1) / DEC_ROWS;
    if (nchunks > 65535 || (long long)B * Hkv > 65535 || R > 0x7fffffffLL)
        return false;
    const unsigned nblk = ((unsigned)Sk + DEC_BLK - 1) / DEC_BLK;
    const unsigned base = (unsigned)B * Hkv * (unsigned)nchunks;
    const unsigned max_split = (nblk + W - 1) / W;  // a block per wavefront
    const unsigned part_bytes = DEC_ROWS * (D + 2) * sizeof(float);
    // a count without empty splits, and its blocks per split
    auto settle = [&](unsigned n, unsigned* bps) {
        n = n > max_split ? max_split : n < 1 ? 1 : n;
        if (n == 1) {
            *bps = (nblk + G - 1) / G * G;
            return 1u;
        }
        *bps = ((nblk + n - 1) / n + G - 1) / G * G;
        return (nblk + *bps - 1) / *bps;
    };
    unsigned bps;
    const unsigned first = DEC_TARGET_WGS / base, at_least = first * base == DEC_TARGET_WGS ? first : first + 1;
    const unsigned least = settle(at_least, &bps);
    const unsigned parts = base * least;
    pl->nchunks = (int)nchunks;
    pl->nsplit = (int)least;
    pl->bps = (int)bps;
    pl->ws_least = pl->ws_bytes = (size_t)parts * part_bytes;
    if (room < pl->ws_least)
        return true;  // the caller refuses it
    const bool one = nblk <= 2 * W;
    if (one) {
        pl->nsplit = 1;
        pl->bps = (int)((nblk + G - 1) / G * G);
    }
    // No other candidate: a fuller split would leave a wavefront without a block, or the least fills whole rounds.
    if (first >= max_split || first * base == DEC_TARGET_WGS)
        return true;
    const unsigned most = parts > DEC_MAX_PARTS ? parts : DEC_MAX_PARTS;
    const double block_us = block_bytes * (2.9 / 65536.0);  // a block per CU while the whole chip streams
    unsigned picked = least, picked_bps = bps;
    double best = 0.0;
    for (unsigned rounds = 1; rounds <= 4; ++rounds) {
        unsigned b;
        const unsigned n = settle(rounds * DEC_TARGET_WGS / base, &b);
        const unsigned wgs = base * n, full = wgs / DEC_TARGET_WGS, rest = wgs % DEC_TARGET_WGS;
        if (n > 1 && (wgs > most || (size_t)wgs * part_bytes > room))
            break;  // so is every later one
        const double turn = b * block_us, share = rest * (1.0 / DEC_TARGET_WGS);
        const double us = full * (turn + 2.0) + (rest ? turn * (share > 0.45 ? share : 0.45) + 2.0 : 0.0) + (n > 1 ? 7.0 : 0.0);
        if (rounds == 1 || us < best) {
            picked = n;
            picked_bps = b;
            best = us;
        }
        if (n >= max_split)
            break;
    }
    if (picked > least)
        pl->ws_bytes = (size_t)base * picked * part_bytes;
    if (!one) {
        pl->nsplit = (int)picked;
        pl->bps = (int)picked_bps;
    }
    return true;
}

constexpr int dec_width(int D) { return D <= 64 ? 64 : D <= 128 ? 128 : 256; }
constexpr int block_bytes16(int D) { return 2 * DEC_BLK * D * 2; }  // K and V of one block

// Whether the split kernel runs on half of its wavefronts, which lets two work-groups (D = 64: four) share a CU:
// - where the others would have no block, and at D <= 128 up to twice that (a block or two per wavefront: the merge of four
//   partials is shorter than that of eight by what the second block costs, and short caches fill the chip with twice the
//   work-groups; us a call before / all / half: 30 caches of 16 heads, 128 keys 15.0 / 13.2 / 10.1, 5 caches of 1326
//   keys, 2 heads, 32 rows 10.5 / 10.7 / 10.5; D = 256, 512 keys, 8 heads 11.8 / 10.9 / 12.5);
// - where there are more work-groups than CUs: the second one's loads fill the gaps of the first and the last round is
//   shorter (320 of 512 keys 25.0 / 22.1 / 19.6, D = 256 49.1 / 42.6 / 37.5; 288 of 3000 87.5 / 83.9 / 81.1).  Half / all
//   over grids of more than 256, kernel time: FP8, D = 128, 640 to 1000 keys 0.84 to 0.89, 1300 to 3000 0.91 to 0.97; FP8,
//   D = 64 0.92 to 0.98; 16 bits, D = 64 0.95 to 1.00 (16384 keys 1.008).
// D > 128, where half is two wavefronts:
// - a last round of at most one work-group a CU runs with half the bytes in flight, so it has to be another one (40 caches of
//   8 heads, 4096 keys, 640 work-groups: four wavefronts each before there was half 250, half 269; 33 caches, 792: 226 / 204);
// - the few threads take their time to merge and store many rows (64 keys, 16 rows 8.1 / 8.7, 32 rows 9.3 / 9.9).
template <int D>
bool half_waves(const DecodeParams& p)
{
    constexpr int W = dec_waves(D);
    const long long wgs = (long long)p.nsplit * p.nchunks * p.B * p.Hkv;
    if (D <= 128)
        return p.bps <= W || wgs > DEC_TARGET_WGS;
    const long long rest = wgs % (2 * DEC_TARGET_WGS);
    return (p.bps <= W / 2 && p.R < 8) || (wgs > DEC_TARGET_WGS && (rest == 0 || rest > DEC_TARGET_WGS));
}

template <int D, int DT_IN, int DT_OUT>
int launch_decode(const DecodeParams& p, hipStream_t stream)
{
    const dim3 g1((unsigned)p.nsplit, (unsigned)p.nchunks, (unsigned)(p.B * p.Hkv));
    constexpr int W = dec_waves(D);
    if (half_waves<D>(p))
        hipLaunchKernelGGL((naut_decode_split_kernel<D, DT_IN, W / 2>), g1, dim3(W / 2 * 64), 0, stream, p);
    else
        hipLaunchKernelGGL((naut_decode_split_kernel<D, DT_IN, W>), g1, dim3(W * 64), 0, stream, p);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess)
        return fail_launch(e);
    if (p.nsplit == 1)
        return NAUT_OK;
    launch_merge<D, DT_OUT>(p, stream);
    e = hipGetLastError();
    if (e != hipSuccess)
        return fail_launch(e);
    return NAUT_OK;
}

}  // namespace

extern "C" {

size_t naut_attn_decode_workspace_bytes(int B, int Hq, int Hkv, int Sq, int Sk, int D)
{
    Plan pl;
    if (B <= 0 || Hq <= 0 || Hkv <= 0 || Sq <= 0 || Sk <= 0 || Hq % Hkv != 0 || D <= 0 || D % 8 != 0 || D > 256 ||
        !make_plan(B, Hq, Hkv, Sq, Sk, dec_width(D), block_bytes16(dec_width(D)), SIZE_MAX, &pl))
        return 0;
    return pl.ws_bytes;
}

}  // extern "C"

namespace {

// The 16-bit decode path behind naut_attn_decode[_dt|_strided] and naut_attn_decode_static.  With
// `use_static` the split partials go to the library's static device array instead of `workspace`; its
// address is taken only after every argument check has passed (no HIP call before that).
int decode_16bit(const void* q, const void* k, const void* v, void* o, float* lse, int B, int Hq, int Hkv,
                 int Sq, int Sk, int D, int causal, float scale, void* workspace, size_t workspace_bytes,
                 bool use_static, void* stream, int in_dtype, int out_dtype, const naut_strides* st)
{
    if (!q || !k || !v || !o)
        return fail(NAUT_ERR_NULL, "q, k, v and o must be non-NULL device pointers");
    if (B <= 0 || Hq <= 0 || Hkv <= 0 || Sq <= 0 || Sk <= 0 || D <= 0)
        return fail(NAUT_ERR_SHAPE, "B, Hq, Hkv, Sq, Sk and D must be positive");
    if (Hq % Hkv != 0)
        return fail(NAUT_ERR_SHAPE, "Hq must be a multiple of Hkv");
    if (causal && Sk < Sq)
        return fail(NAUT_ERR_SHAPE, "with the causal mask the Sq queries are the last positions of Sk: Sk >= Sq");
    if (!std::isfinite(scale))
        return fail(NAUT_ERR_SHAPE, "scale must be finite");
    if (scale < 0.f)
        return fail(NAUT_ERR_UNSUPPORTED, "negative scale is not supported");
    if (D % 8 != 0 || D > 256)
        return fail(NAUT_ERR_UNSUPPORTED, "D must be a multiple of 8, at most 256");
    const int DK = dec_width(D);  // width the kernels are compiled for
    if ((in_dtype != NAUT_BF16 && in_dtype != NAUT_F16) || (out_dtype != in_dtype && out_dtype != NAUT_F32))
        return fail(NAUT_ERR_UNSUPPORTED, "supported dtypes: q/k/v bf16 or f16; o of the same type or f32");
    Plan pl;
    if (!make_plan(B, Hq, Hkv, Sq, Sk, DK, block_bytes16(DK), use_static ? DEC_STATIC_BYTES : workspace_bytes, &pl))
        return fail(NAUT_ERR_UNSUPPORTED, "shape exceeds the grid limits");
    if (use_static)
        workspace = nullptr;
    if (((uintptr_t)q | (uintptr_t)k | (uintptr_t)v | (uintptr_t)o | (uintptr_t)workspace) & 15)
        return fail(NAUT_ERR_ALIGN, "q, k, v, o and workspace must be 16-byte aligned");
    if ((uintptr_t)lse & 3)
        return fail(NAUT_ERR_ALIGN, "lse must be 4-byte aligned");
    if (use_static) {
        if (pl.ws_least > DEC_STATIC_BYTES) {
            snprintf(g_err, sizeof g_err,
                     "these sizes need %zu bytes of split partials, more than the %zu-byte static scratch of "
                     "naut_attn_decode_static: use naut_attn_decode with a workspace",
                     pl.ws_least, DEC_STATIC_BYTES);
            return NAUT_ERR_UNSUPPORTED;
        }
    } else {
        if (!workspace)
            return fail(NAUT_ERR_NULL, "workspace must be a non-NULL device pointer");
        if (workspace_bytes < pl.ws_least)
            return fail(NAUT_ERR_SHAPE, "workspace is smaller than naut_attn_decode_workspace_bytes()");
    }

    naut_strides cs;  // contiguous q, o [B][Hq][Sq][D] and k, v [B][Hkv][Sk][D]
    cs.q_s = cs.k_s = cs.v_s = cs.o_s = D;
    cs.q_h = cs.o_h = (long long)Sq * D;
    cs.k_h = cs.v_h = (long long)Sk * D;
    cs.q_b = cs.o_b = (long long)Hq * Sq * D;
    cs.k_b = cs.v_b = (long long)Hkv * Sk * D;
    if (!st)
        st = &cs;
    const long long in_strides[9] = {st->q_b, st->q_h, st->q_s, st->k_b, st->k_h, st->k_s, st->v_b, st->v_h, st->v_s};
    for (long long x : in_strides)
        if (x < 0 || x % 8 != 0)
            return fail(NAUT_ERR_ALIGN, "q/k/v strides must be non-negative multiples of 8 elements (16 bytes)");
    if (st->o_b <= 0 || st->o_h <= 0 || st->o_s <= 0 || st->o_b % 4 != 0 || st->o_h % 4 != 0 || st->o_s % 4 != 0)
        return fail(NAUT_ERR_ALIGN, "o strides must be positive multiples of 4 elements");
    if (st->q_s < D || st->k_s < D || st->v_s < D || st->o_s < D)
        return fail(NAUT_ERR_SHAPE, "a sequence stride is smaller than D: rows would overlap");
    const long long max_rs = 1LL << 23;  // elements: keeps 32 rows of byte offsets inside 32 bits
    if (st->q_s > max_rs || st->k_s > max_rs || st->v_s > max_rs || st->o_s > max_rs)
        return fail(NAUT_ERR_UNSUPPORTED, "sequence stride too large");
    const int out_b = out_dtype == NAUT_F32 ? 4 : 2;

    if (use_static) {  // every host-side check has passed: the first HIP calls of this path
        int err = NAUT_OK;
        workspace = static_scratch(&err);
        if (workspace == nullptr)
            return err;
    }
    DecodeParams p;
    p.q = q;
    p.k = k;
    p.v = v;
    p.o = o;
    p.lse = lse;
    p.ws = (float*)workspace;
    p.B = B;
    p.Hq = Hq;
    p.Hkv = Hkv;
    p.Sq = Sq;
    p.Sk = Sk;
    p.R = Hq / Hkv * Sq;
    p.nchunks = pl.nchunks;
    p.nsplit = pl.nsplit;
    p.bps = pl.bps;
    p.causal = causal ? 1 : 0;
    const float cc = scale * 1.4426950408889634f;
    p.c = cc > 0.f ? cc : 1.0e-30f;  // scale == 0: every score becomes (almost exactly) 0, the softmax uniform
    p.dv = 1.0f;
    p.out_f32 = out_dtype == NAUT_F32;
    p.q_bs = st->q_b * 2;
    p.q_hs = st->q_h * 2;
    p.q_rs = (int)(st->q_s * 2);
    p.k_bs = st->k_b * 2;
    p.k_hs = st->k_h * 2;
    p.k_rs = (int)(st->k_s * 2);
    p.v_bs = st->v_b * 2;
    p.v_hs = st->v_h * 2;
    p.v_rs = (int)(st->v_s * 2);
    p.o_bs = st->o_b * out_b;
    p.o_hs = st->o_h * out_b;
    p.o_rs = (int)(st->o_s * out_b);
    p.cpr = D / 8;
    hipStream_t hs = (hipStream_t)stream;
#define NAUT_DEC(DD, IN, OUT)                                  \
    if (DK == DD && in_dtype == IN && out_dtype == OUT)        \
        return launch_decode<DD, IN, OUT>(p, hs);
    NAUT_DEC(256, NAUT_BF16, NAUT_BF16)
    NAUT_DEC(256, NAUT_BF16, NAUT_F32)
    NAUT_DEC(256, NAUT_F16, NAUT_F16)
    NAUT_DEC(256, NAUT_F16, NAUT_F32)
    NAUT_DEC(128, NAUT_BF16, NAUT_BF16)
    NAUT_DEC(128, NAUT_BF16, NAUT_F32)
    NAUT_DEC(128, NAUT_F16, NAUT_F16)
    NAUT_DEC(128, NAUT_F16, NAUT_F32)
    NAUT_DEC(64, NAUT_BF16, NAUT_BF16)
    NAUT_DEC(64, NAUT_BF16, NAUT_F32)
    NAUT_DEC(64, NAUT_F16, NAUT_F16)
    NAUT_DEC(64, NAUT_F16, NAUT_F32)
#undef NAUT_DEC
    return fail(NAUT_ERR_UNSUPPORTED, "no kernel for this (D, dtype) combination");
}

}  // namespace

extern "C" {

int naut_attn_decode_strided(const void* q, const void* k, const void* v, void* o, float* lse, int B, int Hq, int Hkv,
                             int Sq, int Sk, int D, int causal, float scale, void* workspace, size_t workspace_bytes,
                             void* stream, int in_dtype, int out_dtype, const naut_strides* st)
{
    return decode_16bit(q, k, v, o, lse, B, Hq, Hkv, Sq, Sk, D, causal, scale, workspace, workspace_bytes, false, stream,
                        in_dtype, out_dtype, st);
}

int naut_attn_decode_fp8_strided(const void* q, const void* k, const void* v, void* o, float* lse, int B, int Hq,
                                 int Hkv, int Sq, int Sk, int D, int causal, float scale, float descale_q,
                                 float descale_k, float descale_v, void* workspace, size_t workspace_bytes, void* stream,
                                 const naut_strides* st)
{
    if (!q || !k || !v || !o)
        return fail(NAUT_ERR_NULL, "q, k, v and o must be non-NULL device pointers");
    if (B <= 0 || Hq <= 0 || Hkv <= 0 || Sq <= 0 || Sk <= 0 || D <= 0)
        return fail(NAUT_ERR_SHAPE, "B, Hq, Hkv, Sq, Sk and D must be positive");
    if (Hq % Hkv != 0)
        return fail(NAUT_ERR_SHAPE, "Hq must be a multiple of Hkv");
    if (causal && Sk < Sq)
        return fail(NAUT_ERR_SHAPE, "with the causal mask the Sq queries are the last positions of Sk: Sk >= Sq");
    if (!std::isfinite(scale) || !std::isfinite(descale_q) || !std::isfinite(descale_k) || !std::isfinite(descale_v))
        return fail(NAUT_ERR_SHAPE, "scale and the three descale factors must be finite");
    if (scale < 0.f || descale_q <= 0.f || descale_k <= 0.f || descale_v <= 0.f)
        return fail(NAUT_ERR_UNSUPPORTED, "scale must be >= 0 and the descale factors > 0");
    if (D % 16 != 0 || D > 128)
        return fail(NAUT_ERR_UNSUPPORTED, "D must be a multiple of 16, at most 128");
    const int DK = D <= 64 ? 64 : 128;  // width the kernels are compiled for
    Plan pl;  // over 64-key blocks: the plan of a cache half as long in 32-key blocks
    if (!make_plan(B, Hq, Hkv, Sq, (Sk + 1) / 2, DK, 2 * DEC8_BLK * DK, workspace_bytes, &pl))
        return fail(NAUT_ERR_UNSUPPORTED, "shape exceeds the grid limits");
    if (((uintptr_t)q | (uintptr_t)k | (uintptr_t)v | (uintptr_t)o | (uintptr_t)workspace) & 15)
        return fail(NAUT_ERR_ALIGN, "q, k, v, o and workspace must be 16-byte aligned");
    if ((uintptr_t)lse & 3)
        return fail(NAUT_ERR_ALIGN, "lse must be 4-byte aligned");
    if (!workspace)
        return fail(NAUT_ERR_NULL, "workspace must be a non-NULL device pointer");
    if (workspace_bytes < pl.ws_least)
        return fail(NAUT_ERR_SHAPE, "workspace is smaller than naut_attn_decode_workspace_bytes()");

    naut_strides cs;  // contiguous q, o [B][Hq][Sq][D] and k, v [B][Hkv][Sk][D]
    cs.q_s = cs.k_s = cs.v_s = cs.o_s = D;
    cs.q_h = cs.o_h = (long long)Sq * D;
    cs.k_h = cs.v_h = (long long)Sk * D;
    cs.q_b = cs.o_b = (long long)Hq * Sq * D;
    cs.k_b = cs.v_b = (long long)Hkv * Sk * D;
    if (!st)
        st = &cs;
    const long long in_strides[9] = {st->q_b, st->q_h, st->q_s, st->k_b, st->k_h, st->k_s, st->v_b, st->v_h, st->v_s};
    for (long long x : in_strides)
        if (x < 0 || x % 16 != 0)
            return fail(NAUT_ERR_ALIGN, "q/k/v strides must be non-negative multiples of 16 elements (16 bytes)");
    if (st->o_b <= 0 || st->o_h <= 0 || st->o_s <= 0 || st->o_b % 4 != 0 || st->o_h % 4 != 0 || st->o_s % 4 != 0)
        return fail(NAUT_ERR_ALIGN, "o strides must be positive multiples of 4 elements");
    if (st->q_s < D || st->k_s < D || st->v_s < D || st->o_s < D)
        return fail(NAUT_ERR_SHAPE, "a sequence stride is smaller than D: rows would overlap");
    const long long max_rs = 1LL << 23;  // elements: keeps 64 rows of byte offsets inside 32 bits
    if (st->q_s > max_rs || st->k_s > max_rs || st->v_s > max_rs || st->o_s > max_rs)
        return fail(NAUT_ERR_UNSUPPORTED, "sequence stride too large");

    DecodeParams p;
    p.q = q;
    p.k = k;
    p.v = v;
    p.o = o;
    p.lse = lse;
    p.ws = (float*)workspace;
    p.B = B;
    p.Hq = Hq;
    p.Hkv = Hkv;
    p.Sq = Sq;
    p.Sk = Sk;
    p.R = Hq / Hkv * Sq;
    p.nchunks = pl.nchunks;
    p.nsplit = pl.nsplit;
    p.bps = pl.bps;
    p.causal = causal ? 1 : 0;
    const float cc = scale * descale_q * descale_k * 1.4426950408889634f;
    p.c = cc > 0.f ? cc : 1.0e-30f;
    p.dv = descale_v;
    p.out_f32 = 0;
    // q, k, v: one byte per element; o: bf16
    p.q_bs = st->q_b;
    p.q_hs = st->q_h;
    p.q_rs = (int)st->q_s;
    p.k_bs = st->k_b;
    p.k_hs = st->k_h;
    p.k_rs = (int)st->k_s;
    p.v_bs = st->v_b;
    p.v_hs = st->v_h;
    p.v_rs = (int)st->v_s;
    p.o_bs = st->o_b * 2;
    p.o_hs = st->o_h * 2;
    p.o_rs = (int)(st->o_s * 2);
    p.cpr = D / 8;
    hipStream_t hs = (hipStream_t)stream;
    const dim3 g1((unsigned)p.nsplit, (unsigned)p.nchunks, (unsigned)(p.B * p.Hkv));
    constexpr int W = DEC_WAVES;
    const bool half = half_waves<128>(p);  // D = 64 has the same rule
    if (DK == 128 && half)
        hipLaunchKernelGGL((naut_decode_split_fp8_kernel<128, W / 2>), g1, dim3(W / 2 * 64), 0, hs, p);
    else if (DK == 128)
        hipLaunchKernelGGL((naut_decode_split_fp8_kernel<128, W>), g1, dim3(W * 64), 0, hs, p);
    else if (half)
        hipLaunchKernelGGL((naut_decode_split_fp8_kernel<64, W / 2>), g1, dim3(W / 2 * 64), 0, hs, p);
    else
        hipLaunchKernelGGL((naut_decode_split_fp8_kernel<64, W>), g1, dim3(W * 64), 0, hs, p);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess)
        return fail_launch(e);
    if (p.nsplit == 1)
        return NAUT_OK;
    if (DK == 128)
        launch_merge<128, NAUT_BF16>(p, hs);
    else
        launch_merge<64, NAUT_BF16>(p, hs);
    e = hipGetLastError();
    if (e != hipSuccess)
        return fail_launch(e);
    return NAUT_OK;
}

int naut_attn_decode_fp8(const void* q, const void* k, const void* v, void* o, float* lse, int B, int Hq, int Hkv,
                         int Sq, int Sk, int D, int causal, float scale, float descale_q, float descale_k,
                         float descale_v, void* workspace, size_t workspace_bytes, void* stream)
{
    if (D > 0 && D != 64 && D != 128)
        return fail(NAUT_ERR_UNSUPPORTED, "D must be 64 or 128 (naut_attn_decode_fp8_strided takes other head dimensions)");
    return naut_attn_decode_fp8_strided(q, k, v, o, lse, B, Hq, Hkv, Sq, Sk, D, causal, scale, descale_q, descale_k,
                                        descale_v, workspace, workspace_bytes, stream, nullptr);
}

int naut_attn_decode_static(const void* q, const void* k, const void* v, void* o, float* lse, int B, int Hq, int Hkv,
                              int Sq, int Sk, int D, int causal, float scale, void* stream)
{
    if (D > 0 && D != 64 && D != 128)
        return fail(NAUT_ERR_UNSUPPORTED, "D must be 64 or 128");
    return decode_16bit(q, k, v, o, lse, B, Hq, Hkv, Sq, Sk, D, causal, scale, nullptr, 0, true, stream, NAUT_BF16,
                        NAUT_BF16, nullptr);
}

int naut_attn_decode_dt(const void* q, const void* k, const void* v, void* o, float* lse, int B, int Hq, int Hkv,
                        int Sq, int Sk, int D, int causal, float scale, void* workspace, size_t workspace_bytes,
                        void* stream, int in_dtype, int out_dtype)
{
    if (D > 0 && D != 64 && D != 128)
        return fail(NAUT_ERR_UNSUPPORTED, "D must be 64 or 128 (naut_attn_decode_strided takes other head dimensions)");
    return naut_attn_decode_strided(q, k, v, o, lse, B, Hq, Hkv, Sq, Sk, D, causal, scale, workspace, workspace_bytes,
                                    stream, in_dtype, out_dtype, nullptr);
}

int naut_attn_decode(const void* q, const void* k, const void* v, void* o, float* lse, int B, int Hq, int Hkv, int Sq,
                     int Sk, int D, int causal, float scale, void* workspace, size_t workspace_bytes, void* stream)
{
    return naut_attn_decode_dt(q, k, v, o, lse, B, Hq, Hkv, Sq, Sk, D, causal, scale, workspace, workspace_bytes, stream,
                               NAUT_BF16, NAUT_BF16);
}

}  // extern "C"
