// naut_attn_pipe.h -- kernel 2, software-pipelined over 32-key blocks (included by naut_attn_kernels.h, D <= 128).
//
// Matrix and vector work overlap inside the wavefront: the key axis is processed in 32-key blocks, and stage k issues
//
//     MFMA:  Y(k-1) = O^T += V^T . P^T of block k-1      VALU:  SM(k) = online softmax of block k
//            X(k+1) = S^T of block k+1
//
// so the MFMAs of a stage never depend on its vector work.  A stage is laid out as a sequence of slots, one MFMA each,
// followed by a few vector instructions: the matrix pipe hides about six ordinary vector instructions per MFMA and no
// more, so the softmax is cut into pieces of that size.  K and V tiles are 32 keys, one barrier per stage, in four LDS
// buffers per operand, filled by direct global->LDS loads that are requested three stages before the one that
// reads them.
//
// What a wavefront owns (QH x 32 queries) and how many share a tile (NWV), with two wavefronts per SIMD throughout (three
// at D = 64, QH = 1):
//   4 x 32: two work-groups to a CU (64 KB of LDS each at D > 64), so that one's prologue, epilogue and waits are covered by
//       the other's loop, and the causal diagonal is followed in steps of 128 queries;
//   8 x 32: one work-group to a CU; a tile serves 256 queries, half the loads per FLOP;
//   4 x 64 (D = 64 only, where two halves fit 256 registers): a fragment read from LDS feeds two MFMAs;
//   4 x 32 with two key groups (NG): group g takes tiles g, g + 2, ... through buffers of its own, and the partial (O, m, l)
//       are merged through LDS.  For grids that leave a CU one work-group, whose loop it halves.
//
// Measured (kernel time, against the same pipeline over 64-key tiles on eight wavefronts, and against kernel 1): B = 4, 32
// heads, S = 4096, D = 128, causal 552 / 582 -> 528 us; S = 1024 53.5 -> 49.5, without the mask 78 -> 72; 32 heads, S =
// 16384 1904 -> 1900 (8 x 32); B = 4, 32 heads, S = 4096, D = 64 600 -> 534 (4 x 64).  Long launches are bound by power: at
// D = 64 4 x 32 takes 10 % fewer cycles than kernel 1 at a 5 % lower clock (1.67 GHz for 1.75), and the 4 x 64 form's gain
// is the LDS reads that it does not do.  Tried: five and six buffers (within 1 %, 20 KB more LDS), 2 and 5 fragments read
// ahead for 3 (both 1 % slower), four wavefronts per SIMD at D = 64 (128 registers spill, 32 % slower).
#ifndef NAUT_ATTN_PIPE_H
#define NAUT_ATTN_PIPE_H

// sum over the two 32-lane halves (same exchange as half_max)
__device__ __forceinline__ float half_sum(float x)
{
    float a = x, b = x;
    asm volatile(NAUT_NOP_SHORT "v_permlane32_swap_b32 %0, %1" : "+v"(a), "+v"(b));
    return a + b;
}

// The softmax of a stage is cut into two pieces per score: FE (fma + exp2) and AC (row-sum add, and
// for odd scores the pack to 16 bit).  FE of score e+1 is placed before AC of score e so that no
// add waits on the exponential just issued.  Approximate issue costs, in vector slots (an
// exponential counts 2), are dealt out to the MFMA slots greedily, at most `cap` per slot.
template <int QH>
struct Pieces {
    static constexpr int NE = 16 * QH, N = 2 * NE;
    // position -> (is_fe, score index)
    static constexpr bool is_fe(int pos) { return pos == 0 || (pos != N - 1 && pos % 2 == 1); }
    static constexpr int score(int pos)
    {
        return pos == 0 ? 0 : pos == N - 1 ? NE - 1 : pos % 2 == 1 ? (pos + 1) / 2 : pos / 2 - 1;
    }
    static constexpr int cost(int pos) { return is_fe(pos) ? 3 : (score(pos) % 2 == 1 ? 2 : 1); }
    template <int NSLOT>
    static constexpr int begin(int slot)
    {
        int total = 0;
        for (int pc = 0; pc < N; ++pc)
            total += cost(pc);
        const int cap = (total + NSLOT - 1) / NSLOT + 1;
        int pc = 0;
        for (int s = 0; s < slot && s < NSLOT; ++s) {
            int used = 0;
            while (pc < N && (s == NSLOT - 1 || used + cost(pc) <= cap || used == 0)) {
                used += cost(pc);
                ++pc;
            }
        }
        return slot >= NSLOT ? N : pc;
    }
};

template <int D, int QH, int NWV, int NG>
constexpr int pipe_waves_per_simd() { return D <= 64 && QH == 1 && NG == 1 ? 3 : 2; }

template <int D, int DT_IN, int DT_OUT, bool CAUSAL, int QH, int NWV, int NG = 1>
__global__ __launch_bounds__(NWV * NG * 64, (pipe_waves_per_simd<D, QH, NWV, NG>())) void naut_fwd_kernel_pipe(const Params p)
{
    using T = In<DT_IN>;
    using PC = Pieces<QH>;
    constexpr int WQ = 32 * QH;                // queries per wavefront
    constexpr int BM = NWV * WQ;               // queries per work-group
    constexpr int BN = 32;                     // keys per tile and stage
    constexpr int NBUF = 4;                    // LDS buffers per operand
    constexpr int LA = NBUF - 1;               // stage j requests K tile j + LA and V tile j + LA - 2 (read in stage j + LA)
    constexpr int W = layout_width(D);         // row width of the LDS layouts
    constexpr int ROWB = W * 2;
    constexpr int TILEB = BN * ROWB;           // one 32-key K or V tile
    constexpr int KS = D / 16;
    constexpr int DB = (D + 31) / 32;
    constexpr int LDW = TILEB / 1024 / NWV;    // direct loads per wavefront per tile (1 KB each)
    constexpr int NF = 2 * DB + KS;            // fragments per stage: even = V^T (Y), odd = K (X)
    constexpr int NS = NF * QH;                // slots (MFMAs) per stage
    constexpr int PREFETCH = 3;                // fragments in flight from LDS ahead of their MFMAs
    static_assert(QH == 1 || D <= 64, "what fits the ordinary vector registers");
    auto pin_acc = [](f32x16_t& x) { asm volatile("" : "+v"(x)); };
    static_assert(2 * DB == KS || 2 * DB == KS + 1, "Y and X fragments alternate, Y first");
    static_assert(LDW >= 1, "every wavefront must take part in the tile loads");
    static_assert(LA >= 3 && (LA - 2) * 2 * LDW < 64, "vmcnt field");

    constexpr int RINGB = 2 * NBUF * TILEB;    // a key group's buffers: K tiles, then V tiles
    __shared__ __attribute__((aligned(1024))) unsigned char smem[NG * RINGB];
    __shared__ float ml_lds[NG > 1 ? (NG - 1) * NWV * 64 * 3 : 1];

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave_wg = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wave = NG == 1 ? wave_wg : wave_wg % NWV;  // inside its key group
    const int grp = NG == 1 ? 0 : wave_wg / NWV;
    const int l32 = lane & 31;
    const int h = lane >> 5;

    // Tile scheduler: heaviest (last) query tiles first.  A launch that is resident all at once takes them over all heads; up
    // to two work-groups to each of an XCD's 32 CUs, causal, the second round in ascending order, so that a heavy tile shares
    // its CU with a light one (D = 128: 32 heads, S = 2048 45.9 -> 43.2 us, 128 heads, S = 512 21.5 -> 18.9).
    //   A larger one goes through the heads of an XCD about AT_ONCE at a time (query heads that share a K/V head sit next to
    // each other), all at once where they are few or small: each group starts with its heaviest tiles (96 heads, S = 2048,
    // causal, D = 64, twelve heads to an XCD: six and six 76.2 us, all at once 65.7; 128 heads, S = 4096, D = 128 eight at a time 529,
    // sixteen 540; 256 heads, S = 640, causal, D = 64 groups 30.8, all 27.2; without the mask a group's tiles are alike, and
    // groups cost nothing).
    const int nbh = p.B * p.Hq;
    const int nqt = BM == BM2 ? p.nqt2 : p.nqt;
    constexpr int PER_CU = NWV * NG == 8 ? 1 : pipe_waves_per_simd<D, QH, NWV, NG>();  // work-groups that share a CU
    constexpr int AT_ONCE = D <= 64 ? 2 * HEADS_AT_ONCE : HEADS_AT_ONCE;               // (their K and V are half the bytes)
    const int xcd = blockIdx.x & 7, n_xcd = (nbh * nqt - xcd + 7) >> 3;                // work-groups of this XCD
    int qt, bh;
    if (n_xcd <= 32 * PER_CU) {
        int s = (int)blockIdx.x >> 3;
        if (CAUSAL && PER_CU == 2 && s >= 32)
            s = 31 + n_xcd - s;
        const int bid = s * 8 + xcd;
        qt = nqt - 1 - bid / nbh;
        bh = bid % nbh;
    } else {
        const int hpx = nbh >> 3;
        const bool all = 2 * hpx <= 3 * AT_ONCE || (CAUSAL && (long long)hpx * p.S * ROWB <= 3 << 20);
        const QueryTile t = tile_by_head(blockIdx.x, nbh, nqt, all ? 1 : (hpx + AT_ONCE / 2) / AT_ONCE);
        qt = t.qt;
        bh = t.bh;
    }
    const int b = bh / p.Hq;
    const int hq = bh % p.Hq;
    const int hk = hq / (p.Hq / p.Hkv);
    const int S = p.S;
    const float c = p.c;
    const float p_limit = p.p_limit;
    float c_v = c;  // copy held in a vector register: an FMA with a scalar-register operand issues at the slower rate
    asm volatile("" : "+v"(c_v));

    const unsigned char* qg = (const unsigned char*)p.q + b * p.q_bs + hq * p.q_hs;
    const unsigned char* kg = (const unsigned char*)p.k + b * p.k_bs + hk * p.k_hs;
    const unsigned char* vg = (const unsigned char*)p.v + b * p.v_bs + hk * p.v_hs;
    const int cpr = p.cpr;

    const int Q0 = qt * BM + wave * WQ;  // first query of this wavefront
    int qrow[QH];
#pragma unroll
    for (int hf = 0; hf < QH; ++hf)
        qrow[hf] = Q0 + 32 * hf + l32;

    // Q^T fragments (MFMA B operands), resident for the whole kernel.
    i32x4_t qf[QH][KS];
#pragma unroll
    for (int hf = 0; hf < QH; ++hf) {
        const int q_ld = qrow[hf] < S ? qrow[hf] : S - 1;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            // Unconditional, from a chunk that exists; the padding chunks of a narrower head are zeroed when Q is pinned
            // below.  (A load under a condition becomes a branch, and the compiler then waited for the first loads in
            // the middle of issuing the rest.)
            const int ch = ks * 2 + h < cpr ? ks * 2 + h : cpr - 1;
            qf[hf][ks] = *(const i32x4_t*)(qg + (size_t)q_ld * p.q_rs + ch * 16);
        }
    }
    const int kv_end_wg = CAUSAL ? (S < (qt + 1) * BM ? S : (qt + 1) * BM) : S;
    const int kv_end_w = Q0 >= S ? 0 : (CAUSAL ? (S < Q0 + WQ ? S : Q0 + WQ) : S);
    const int ntiles = (kv_end_wg + BN - 1) / BN;
    // tiles and blocks below count those of a key group: grp, grp + NG, ...
    auto of_group = [&](int n) { return n > grp ? (n - grp + NG - 1) / NG : 0; };
    const int niter = (ntiles + NG - 1) / NG + 2;             // of the first group, which has the most: all meet the same barriers
    const int nblk = of_group((kv_end_w + BN - 1) / BN);      // key blocks of this wavefront

    // Direct global->LDS tile loads, 1 KB each: lane i fills physical chunk i of its KB, so it fetches the logical chunk
    // that the swizzle places there.  The address is that of the head plus the tile's byte offset (scalar) plus a
    // per-lane offset that never changes.  The loads go through a buffer descriptor whose range ends with the last row:
    // beyond it (the ragged end of the sequence) a lane gets zeros and touches no memory.
    int k_goff[LDW], v_goff[LDW];  // byte offset of the lane's chunk inside a tile
#pragma unroll
    for (int i = 0; i < LDW; ++i) {
        const int P = (wave * LDW + i) * 64 + lane;  // physical chunk index in the tile
        const int line = P >> 4, pos = P & 15;
        const int L = (line << 4) + (pos ^ (line & 15));
        const int krow = L / (W / 8), kch = L % (W / 8);
        k_goff[i] = krow * p.k_rs + (kch < cpr ? kch : cpr - 1) * 16;
        const int vrow = P / (W / 8), cc = P % (W / 8);
        const int lc = W == 128 ? cc ^ ((vrow & 3) << 2) : cc ^ (((vrow >> 1) & 1) << 2);
        v_goff[i] = vrow * p.v_rs + (lc < cpr ? lc : cpr - 1) * 16;
    }
    const unsigned smem_base = (unsigned)(uintptr_t)(NAUT_LDS unsigned char*)smem + (unsigned)(grp * RINGB);
    const unsigned ld_dst = smem_base + (unsigned)(wave * LDW * 1024);
    struct Tiles {
        i32x4_t rsrc;
        unsigned off, end;       // byte offsets of the tile requested next and of the work-group's last one
        uint64_t range64, end64; // what the descriptor's range and `end` stand for: both are cut off at 32 bits
    };
    auto tiles_of = [&](const unsigned char* g, int rs) {
        Tiles t;
        const uint64_t a = (uint64_t)g;
        t.rsrc.x = __builtin_amdgcn_readfirstlane((int)a);
        t.rsrc.y = __builtin_amdgcn_readfirstlane((int)(a >> 32) & 0xffff);
        t.rsrc.w = 0x00020000;
        t.off = (unsigned)(grp < ntiles ? grp : ntiles - 1) * (unsigned)(BN * rs);
        t.range64 = (uint64_t)(S - 1) * (unsigned)rs + (unsigned)(cpr * 16);
        // the group's last tile (a group without one: a tile that exists, for nobody)
        t.end64 = (uint64_t)(grp < ntiles ? ntiles - 1 - (ntiles - 1 - grp) % NG : ntiles - 1) * (unsigned)(BN * rs);
        t.rsrc.z = __builtin_amdgcn_readfirstlane((int)(unsigned)(t.range64 >> 32 ? 0xffffffffu : t.range64));
        t.end = __builtin_amdgcn_readfirstlane((int)(unsigned)(t.end64 >> 32 ? 0xffffffffu : t.end64));
        return t;
    };
    auto advance = [&](Tiles& t, unsigned step) { t.off = t.off + step < t.end ? t.off + step : t.end; };  // the last tile again past the end
    // Offsets stay below 2^32: a step is at most 2^29 bytes (32 rows of 16 MiB; 64 of 8 MiB, beyond which launch() does not
    // run two key groups), and this, called every four steps and first after five, moves the base past 2^30.
    auto rebase = [&](Tiles& t) {
        if (t.off >> 30) {
            const uint64_t a = ((uint64_t)(unsigned)t.rsrc.y << 32 | (unsigned)t.rsrc.x) + t.off;
            t.rsrc.x = __builtin_amdgcn_readfirstlane((int)a);
            t.rsrc.y = __builtin_amdgcn_readfirstlane((int)(a >> 32));
            t.range64 -= t.off;
            t.end64 -= t.off;
            t.rsrc.z = __builtin_amdgcn_readfirstlane((int)(unsigned)(t.range64 >> 32 ? 0xffffffffu : t.range64));
            t.end = __builtin_amdgcn_readfirstlane((int)(unsigned)(t.end64 >> 32 ? 0xffffffffu : t.end64));
            t.off = 0;
        }
    };
    auto issue = [&](const Tiles& t, int lds_tile, int off, int i) {
        buffer_to_lds(ld_dst + lds_tile * TILEB + i * 1024, off, t.rsrc, (int)t.off);
    };
    Tiles kt = tiles_of(kg, p.k_rs), vt = tiles_of(vg, p.v_rs);
    const unsigned k_step = NG * BN * (unsigned)p.k_rs, v_step = NG * BN * (unsigned)p.v_rs;

    // LDS byte addresses of the fragments in buffer 0 of K and of V; they stay as they are for the whole kernel (buffer
    // and step offsets are immediates)
    int k_it[KS], v_it[DB];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
        k_it[ks] = (int)smem_base + k_off<W>(l32, ks * 2 + h);
        asm volatile("" : "+v"(k_it[ks]));  // opaque: the compiler then adds nothing but instruction immediates to it
    }
    {
        const int i16 = lane & 15;
        const int key = 4 * h + (i16 >> 2);
#pragma unroll
        for (int db = 0; db < DB; ++db) {
            const int d = 32 * db + 16 * ((lane >> 4) & 1) + 4 * (i16 & 3);
            v_it[db] = (int)smem_base + NBUF * TILEB + v_off<W>(key, d >> 3) + (d & 7) * 2;
            asm volatile("" : "+v"(v_it[db]));
        }
    }

    f32x16_t oacc[QH][DB];
    // reference maximum (log2 units), its negation, a quarter of the running sum of P (kept as the quarter because that
    // is what a block's sum is compared with; the factor is exact), and what the sum of P as rounded for the second
    // product has over the unrounded sum (touched in heavy blocks only; see "the two sums" at the pieces of a stage)
    float m_run[QH], neg_m[QH], lq_run[QH], dl_run[QH];
#pragma unroll
    for (int hf = 0; hf < QH; ++hf) {
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int r = 0; r < 16; ++r)
                oacc[hf][db][r] = 0.f;
        m_run[hf] = -FLT_MAX;  // the lowest value there is, below any score that is itself finite
        neg_m[hf] = FLT_MAX;
        lq_run[hf] = 0.f;
        dl_run[hf] = 0.f;
    }

    // causal / tail masking of block kblk
    auto mask_block = [&](int kblk, f32x16_t (&s_)[QH]) {
        int key0 = (kblk * NG + grp) * BN + 4 * h;
        asm volatile("" : "+v"(key0));  // nothing of the masks is formed ahead of the loop and held across it
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int key = key0 + 8 * (r >> 2) + (r & 3);
#pragma unroll
            for (int hf = 0; hf < QH; ++hf)
                s_[hf][r] = (key >= kv_end_w || (CAUSAL && key > qrow[hf])) ? -INFINITY : s_[hf][r];
        }
    };
    // first block that needs masking: 32k+31 > Q0 (causal; Q0 is a multiple of 32) or 32k+32 > kv_end_w
    const int kc2 = kv_end_w / BN;
    const int k_mask_from = of_group(CAUSAL ? (Q0 / BN < kc2 ? Q0 / BN : kc2) : kc2);
    // max of three; the device code is compiled with NaNs assumed absent, so this is one v_max3_f32 with no quieting of
    // the operands
    auto max3 = [](float x, float y, float z) { return __builtin_fmaxf(__builtin_fmaxf(x, y), z); };

    // Fragment f of iteration U (mod NBUF): even f = V^T of tile U - 2 (two transposed 64-bit reads), odd f = K of tile U
    // (one 128-bit read).
    auto load_frag = [&](auto F, auto UC) -> i32x4_t {
        constexpr int f = decltype(F)::value, U = decltype(UC)::value;
        if constexpr (f % 2 == 0) {
            constexpr int y = f / 2, t = y / DB, db = y % DB;
            constexpr int off = ((U + NBUF - 2) % NBUF) * TILEB + 16 * t * ROWB;
            const i16x4_t r0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((NAUT_LDS i16x4_t*)(uintptr_t)(v_it[db] + off));
            const i16x4_t r1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((NAUT_LDS i16x4_t*)(uintptr_t)(v_it[db] + off + 8 * ROWB));
            const i32x2_t lo = __builtin_bit_cast(i32x2_t, r0), hi = __builtin_bit_cast(i32x2_t, r1);
            return i32x4_t{lo.x, lo.y, hi.x, hi.y};
        } else {
            return *(const NAUT_LDS i32x4_t*)(uintptr_t)(k_it[f / 2] + (U % NBUF) * TILEB);
        }
    };

    // Stage of iteration j (j mod NBUF = U): Y(j-2), SM(j-1), X(j); k = j-1.  HY / HS: it has a Y / an SM (the first two
    // iterations have not both); NHY: the next one has a Y; MASK: block k may need the mask.  The first PREFETCH
    // fragments arrive in `carry` (read during the previous stage) and the last slots read the next stage's first
    // fragments into it, so no stage starts with an empty LDS pipeline.
    float psum[QH];                    // of the block in SM, per lane: its 16 of the 32 keys
    unsigned long long test_mask = 0;  // see settle_block
    auto stage = [&](auto UC, auto HYC, auto HSC, auto NHYC, auto MASKC, int k, i32x4_t (&carry)[PREFETCH],
                     f32x16_t (&s_cur)[QH], f32x16_t (&s_nxt)[QH], const i32x4_t (&p_in)[QH][2], i32x4_t (&p_out)[QH][2],
                     auto&& side) {
        constexpr int U = decltype(UC)::value;
        constexpr bool HY = decltype(HYC)::value, HS = decltype(HSC)::value, NHY = decltype(NHYC)::value;
        if constexpr (HS && decltype(MASKC)::value)
            if (k >= k_mask_from)
                mask_block(k, s_cur);
        i32x4_t frag[NF];
        static_for<0, PREFETCH>([&](auto F) { frag[decltype(F)::value] = carry[decltype(F)::value]; });
        auto read_ahead = [&](auto F) {
            constexpr int f = decltype(F)::value;
            if constexpr (f < NF) {
                if constexpr (HY || f % 2 == 1)
                    frag[f] = load_frag(F, UC);
            } else if constexpr (NHY || (f - NF) % 2 == 1) {
                carry[f - NF] = load_frag(std::integral_constant<int, f - NF>{}, std::integral_constant<int, U + 1>{});
            }
        };
        float pe[QH][16];
        // Vector work of the stage, one piece at a time (see Pieces).  P is formed against the
        // reference maximum as it stands, with no look at this block's own maximum: as long as the
        // row sums stay below p_limit (Params) every P is below it too, and the reference need not move.
        // The two sums: lse needs l = sum of P to better than 16-bit accuracy, so P is summed in fp32 before it
        // is rounded; O, on the other hand, must be divided by the sum of the P that went into it, the rounded
        // ones.  With the reference lagging behind the maximum the largest P of a row is an arbitrary number,
        // not 1, and its rounding error (up to 2^-8 relative in bf16, whose significand has 8 bits) would otherwise
        // go into O but not into its divisor: for a row that one key dominates that is an error of up to 2^-8 |v|
        // on top of the rounding of O itself (as much again: together past the 2e-2 bar once |v| exceeds 2.6).
        // Divided by the rounded sum the weights add up to one exactly and such a row returns v (what is left is
        // 2^-8 w |v - O| per key of weight w, as in any kernel that rounds P).  Only keys of large weight matter for
        // this, so the rounded sum is formed (after the slots, from the packed P) only for a block that
        // adds a quarter or more to some row's running sum -- every key that ends with a fifth of its row's
        // weight or more is in such a block -- and the unrounded sum stands in for it otherwise: a key so
        // treated adds at most 0.2 * 2^-8 |v| to the error, and |O| near 4 would take several such keys with
        // |v| near 4 in one column, which N(0,1)-like values do not supply; the rounding errors of the many
        // light keys, independent and of either sign, average out in O.
        auto piece = [&](auto PCI) {
            constexpr int pos = decltype(PCI)::value, e = PC::score(pos), hf = e / 16, idx = e % 16;
            if constexpr (PC::is_fe(pos)) {
                pe[hf][idx] = __builtin_amdgcn_exp2f(__builtin_fmaf(s_cur[hf][idx], c_v, neg_m[hf]));
                // anchor: keeps this piece in its slot (the optimiser would otherwise sink it to the first use of P,
                // after the last MFMA of the stage).  Input-only: an asm that also defined the value would make the
                // compiler pad the next use with a wait state.
                asm volatile("" ::"v"(pe[hf][idx]));
            } else {
                // fp32 sum of the unrounded P: lse needs l to better than bf16 accuracy
                if constexpr (idx == 0)
                    psum[hf] = pe[hf][0];
                else
                    psum[hf] += pe[hf][idx];
                if constexpr (idx % 2 == 1) {
                    int w = T::pack2(pe[hf][idx - 1], pe[hf][idx]);
                    asm volatile("" ::"v"(w), "v"(psum[hf]));
                    p_out[hf][idx >> 3][(idx >> 1) & 3] = w;
                } else {
                    asm volatile("" ::"v"(psum[hf]));
                }
            }
        };
        static_for<0, NS>([&](auto I) {
            constexpr int i = decltype(I)::value, f = i / QH, hf = i % QH;
            if constexpr (hf == 0)
                read_ahead(std::integral_constant<int, f + PREFETCH>{});
            if constexpr (f % 2 == 0) {
                constexpr int y = f / 2, t = y / DB, db = y % DB;
                if constexpr (HY)
                    oacc[hf][db] = T::mfma(frag[f], p_in[hf][t], oacc[hf][db]);
            } else {
                constexpr int ks = f / 2;
                if constexpr (ks == 0)
                    s_nxt[hf] = T::mfma(frag[f], qf[hf][ks], f32x16_t{0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f});
                else
                    s_nxt[hf] = T::mfma(frag[f], qf[hf][ks], s_nxt[hf]);
            }
            constexpr int p0 = PC::template begin<NS>(i), p1 = PC::template begin<NS>(i + 1);
            side(I);
            if constexpr (HS)
                static_for<p0, p1>([&](auto PCI) { piece(PCI); });
            // one wait for two fragments: LDS reads return in order, so waiting at the end of an odd slot for the
            // fragment two slots on covers the next slot's too, and neither of the two coming slots needs a wait
            // instruction of its own
            if constexpr (hf == QH - 1 && f % 2 == 1 && f + 2 < NF)
                asm volatile("" ::"v"(frag[f + 2]));
            __builtin_amdgcn_sched_barrier(0);
        });
        if constexpr (HS) {
            // one comparison per half serves both tests of settle_block; its lane mask is on its way to a scalar register
            // while the wavefront waits at the barrier
            test_mask = 0;
#pragma unroll
            for (int hf = 0; hf < QH; ++hf)
                test_mask |= __builtin_amdgcn_ballot_w64(psum[hf] > __builtin_fminf(lq_run[hf], p_limit));
            asm volatile("" ::"s"(test_mask));
        }
#pragma unroll
        for (int hf = 0; hf < QH; ++hf)
#pragma unroll
            for (int db = 0; db < DB; ++db)
                pin_acc(oacc[hf][db]);
    };
    // What is left of SM once every P of the block exists, after the barrier: the rare move of the reference maximum, the
    // two sums.  Block k's scores are intact and its P not yet used; s_nxt holds those of block k + 1.  (Always inlined: a
    // call would put the whole state of the loop into memory.)
    auto settle_block = [&](int k, f32x16_t (&s_cur)[QH], f32x16_t (&s_nxt)[QH], i32x4_t (&p_out)[QH][2]) __attribute__((always_inline)) {
        if (test_mask != 0) {
            bool over = false;  // also true for +inf (first block of a row: the reference is still the lowest value)
#pragma unroll
            for (int hf = 0; hf < QH; ++hf)
                over = over || psum[hf] > p_limit;
            if (__builtin_amdgcn_ballot_w64(over) != 0) {
                // Some row of this wavefront met scores far above its reference maximum.  Move the reference of every
                // row to its true running maximum, apply the repair factor exp2(m_old - m_new) to l and O (after
                // Y(k-1), whose P was formed against the old maxima), and form this block's P again.
                //   The maximum is that of this block and the next, as kernel 1 takes it over tiles of 64 keys: the larger the
                // keys whose P is exactly 1, the smaller the error of O.  Relative error against 64 bits over that of kernel 1
                // with as many key groups, bf16, f32 O, usual scale: from this block alone 1.020 (190 shapes of one group)
                // and 1.011 (66 of two), from both 0.997 and 0.993.  It costs eight instructions a move, 0.3 % of the time
                // over 3693 shapes.
                if (k + 1 >= k_mask_from)
                    mask_block(k + 1, s_nxt);  // once more in its own stage, to the same values
#pragma unroll
                for (int hf = 0; hf < QH; ++hf) {
                    const f32x16_t& s_ = s_cur[hf];
                    float mx = max3(s_[0], s_[1], s_[2]);
#pragma unroll
                    for (int r = 3; r < 15; r += 2)
                        mx = max3(mx, s_[r], s_[r + 1]);
                    mx = max3(mx, s_[15], s_nxt[hf][15]);
#pragma unroll
                    for (int r = 0; r < 14; r += 2)
                        mx = max3(mx, s_nxt[hf][r], s_nxt[hf][r + 1]);
                    mx = max3(mx, s_nxt[hf][14], s_nxt[hf][14]);
                    float a2 = mx, b2 = mx;
                    asm volatile(NAUT_NOP_SHORT "v_permlane32_swap_b32 %0, %1" : "+v"(a2), "+v"(b2));
                    const float cand = max3(a2, b2, b2) * c;  // -inf if both blocks are masked for this row
                    const float m_new = max3(m_run[hf], cand, cand);
                    const float alpha = __builtin_amdgcn_exp2f(m_run[hf] - m_new);
                    lq_run[hf] *= alpha;
                    dl_run[hf] *= alpha;
#pragma unroll
                    for (int db = 0; db < DB; ++db) {
#pragma unroll
                        for (int r = 0; r < 16; ++r)
                            oacc[hf][db][r] *= alpha;
                        pin_acc(oacc[hf][db]);
                    }
                    m_run[hf] = m_new;
                    neg_m[hf] = -m_new;
                    float ps = 0.f;
#pragma unroll
                    for (int idx = 0; idx < 16; idx += 2) {
                        const float p0 = __builtin_amdgcn_exp2f(__builtin_fmaf(s_[idx], c_v, neg_m[hf]));
                        const float p1 = __builtin_amdgcn_exp2f(__builtin_fmaf(s_[idx + 1], c_v, neg_m[hf]));
                        ps += p0 + p1;
                        p_out[hf][idx >> 3][(idx >> 1) & 3] = T::pack2(p0, p1);
                    }
                    psum[hf] = ps;
                }
            }
            // the heavy block's sum of the rounded P; its difference to the unrounded sum goes to dl_run
#pragma unroll
            for (int hf = 0; hf < QH; ++hf) {
                float pr = -psum[hf];
#pragma unroll
                for (int t = 0; t < 2; ++t)
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        pr = T::add_pair(p_out[hf][t][e], pr);
                dl_run[hf] += pr;
            }
        }
#pragma unroll
        for (int hf = 0; hf < QH; ++hf)
            lq_run[hf] = __builtin_fmaf(psum[hf], 0.25f, lq_run[hf]);
    };

    // ---- prologue: K tiles 0 .. LA-1, V tiles 0 .. LA-3 ----
    static_for<0, LA>([&](auto TC) {
        constexpr int t = decltype(TC)::value;
#pragma unroll
        for (int i = 0; i < LDW; ++i)
            issue(kt, t, k_goff[i], i);
        advance(kt, k_step);
        if constexpr (t + 2 < LA) {
#pragma unroll
            for (int i = 0; i < LDW; ++i)
                issue(vt, NBUF + t, v_goff[i], i);
            advance(vt, v_step);
        }
    });
    // Q is pinned to its registers only here: its loads, issued at the top, and the tile loads share one round trip to
    // memory instead of taking one each.
    int cpr_late = cpr;
    asm volatile("" : "+s"(cpr_late));  // ordered after the tile loads above: so is everything that uses it
#pragma unroll
    for (int hf = 0; hf < QH; ++hf)
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            if (ks * 2 + h >= cpr_late)
                qf[hf][ks] = i32x4_t{0, 0, 0, 0};
            asm volatile("" : "+v"(qf[hf][ks]));
        }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();

    f32x16_t s_e[QH], s_o[QH];              // scores of the current even / odd block
    i32x4_t p_e[QH][2], p_o[QH][2];         // P of the last even / odd block
    i32x4_t carry[PREFETCH];                // first fragments of the coming stage

    // Iteration j (U = j mod NBUF): its stage, and the request of K tile j + LA and V tile j + LA - 2, dealt out over the
    // slots, into the buffers that the previous stage was the last to read.
    auto iteration = [&](auto UC, auto HYC, auto HSC, auto NHYC, auto MASKC, int j) {
        constexpr int U = decltype(UC)::value, KBUF = (U + LA) % NBUF, VBUF = NBUF + (U + LA - 2) % NBUF;
        auto side = [&](auto I) {
            constexpr int i = decltype(I)::value, NL = 2 * LDW, STEP = NS / NL;
            if constexpr (!SAFE_SYNC && i % STEP == STEP / 2 && i / STEP < NL) {
                constexpr int q = i / STEP;
                if constexpr (q < LDW)
                    issue(kt, KBUF, k_goff[q], q);
                else
                    issue(vt, VBUF, v_goff[q - LDW], q - LDW);
            }
        };
        if constexpr (SAFE_SYNC) {  // checking build: the iteration's loads are issued, awaited and published first
            tile_barrier();
#pragma unroll
            for (int i = 0; i < LDW; ++i) {
                issue(kt, KBUF, k_goff[i], i);
                issue(vt, VBUF, v_goff[i], i);
            }
            tile_barrier();
        }
        // even j: X(j) -> s_e, SM(j-1) of s_o -> p_o, Y(j-2) with p_e
        if constexpr (U % 2 == 0)
            stage(UC, HYC, HSC, NHYC, MASKC, j - 1, carry, s_o, s_e, p_e, p_o, side);
        else
            stage(UC, HYC, HSC, NHYC, MASKC, j - 1, carry, s_e, s_o, p_o, p_e, side);
        advance(kt, k_step);
        advance(vt, v_step);
        // The last slots of the next iteration already read the tiles of the one after it: everything but the loads
        // of the last LA - 2 iterations must have landed.  A bare barrier, not __syncthreads(): the fence in the latter
        // would first drain the LDS reads in flight, which are this wavefront's prefetch for the next stage.
        wait_loads<(LA - 2) * 2 * LDW>();
        tile_barrier();
        if constexpr (decltype(HSC)::value) {
            if constexpr (U % 2 == 0)
                settle_block(j - 1, s_o, s_e, p_o);
            else
                settle_block(j - 1, s_e, s_o, p_e);
        }
    };
    int j = 0;
    constexpr std::true_type yes{};
    constexpr std::false_type no{};
    if (nblk > 0) {
        static_for<0, PREFETCH>([&](auto F) {
            if constexpr (decltype(F)::value % 2 == 1)
                carry[decltype(F)::value] = load_frag(F, std::integral_constant<int, 0>{});
        });
        iteration(std::integral_constant<int, 0>{}, no, no, no, no, 0);
        iteration(std::integral_constant<int, 1>{}, no, yes, yes, yes, 1);
        // Iterations 2 .. nblk, each with a Y, an SM and an X (the last X is of no block: nobody reads it): first whole
        // rounds of NBUF whose blocks need no mask, without any test but the loop's own.
        int j0 = 2;
        for (; j0 + NBUF - 2 < k_mask_from; j0 += NBUF) {
            rebase(kt);
            rebase(vt);
            static_for<0, NBUF>([&](auto C) {
                constexpr int u = decltype(C)::value;
                iteration(std::integral_constant<int, (2 + u) % NBUF>{}, yes, yes, yes, no, j0 + u);
            });
        }
        for (; j0 <= nblk; j0 += NBUF) {
            rebase(kt);
            rebase(vt);
            static_for<0, NBUF>([&](auto C) {
                constexpr int u = decltype(C)::value;
                if (j0 + u <= nblk)
                    iteration(std::integral_constant<int, (2 + u) % NBUF>{}, yes, yes, yes, yes, j0 + u);
            });
        }
        j = nblk + 1;  // Y of the last block alone
        const bool odd = (nblk - 1) & 1;
        const int voff = (int)((unsigned)(nblk - 1) % NBUF) * TILEB;
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int db = 0; db < DB; ++db) {
                const int a = v_it[db] + voff + 16 * t * ROWB;
                const i16x4_t r0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((NAUT_LDS i16x4_t*)(uintptr_t)a);
                const i16x4_t r1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((NAUT_LDS i16x4_t*)(uintptr_t)(a + 8 * ROWB));
                const i32x2_t lo = __builtin_bit_cast(i32x2_t, r0), hi = __builtin_bit_cast(i32x2_t, r1);
#pragma unroll
                for (int hf = 0; hf < QH; ++hf) {
                    i32x4_t pl;
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        pl[e] = odd ? p_o[hf][t][e] : p_e[hf][t][e];
                    oacc[hf][db] = T::mfma(i32x4_t{lo.x, lo.y, hi.x, hi.y}, pl, oacc[hf][db]);
                }
            }
    }
    // With the causal mask the wavefronts of a work-group finish at different keys: what the others still read, this one's
    // part of it, one barrier for each of their iterations.
    for (; j + 1 < niter; ++j) {
        rebase(kt);
        rebase(vt);
        if constexpr (SAFE_SYNC)
            tile_barrier();
#pragma unroll
        for (int i = 0; i < LDW; ++i) {
            issue(kt, (j + LA) % NBUF, k_goff[i], i);
            issue(vt, NBUF + (j + LA - 2) % NBUF, v_goff[i], i);
        }
        if constexpr (SAFE_SYNC)
            tile_barrier();
        advance(kt, k_step);
        advance(vt, v_step);
        wait_loads<(LA - 2) * 2 * LDW>();
        tile_barrier();
    }
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    __syncthreads();  // every load has landed and the last Y of every wavefront has its fragments: the tiles are dead

    if constexpr (NG > 1) {
        // Split-merge of the key groups: the second leaves O, m and l in the layout it holds them in, lane by lane, O in
        // its own dead tiles; the first adds them up and stores.
        static_assert(QH == 1 && NG == 2 && NWV * DB * 16 * 64 * 4 <= RINGB, "a group's O fits its tile buffers");
        int ln = lane;
        asm volatile("" : "+v"(ln));  // no address of the merge is held across the key loop
        float* const mo = (float*)(smem + RINGB) + wave * (DB * 16 * 64) + ln * 4;
        float* const ml = ml_lds + wave * 192 + ln;
        if (grp > 0) {
#pragma unroll
            for (int db = 0; db < DB; ++db)
#pragma unroll
                for (int g = 0; g < 4; ++g)
                    *(f32x4_t*)(mo + (db * 4 + g) * 256) =
                        f32x4_t{oacc[0][db][4 * g], oacc[0][db][4 * g + 1], oacc[0][db][4 * g + 2], oacc[0][db][4 * g + 3]};
            ml[0] = m_run[0];
            ml[64] = lq_run[0];
            ml[128] = dl_run[0];
        }
        __syncthreads();
        if (grp > 0)
            return;
        // The halves of a row hold the same maximum, and key 0, which every row sees, is the first group's.
        const float m_new = __builtin_fmaxf(m_run[0], ml[0]);
        const float f0 = __builtin_amdgcn_exp2f(m_run[0] - m_new), f1 = __builtin_amdgcn_exp2f(ml[0] - m_new);
        m_run[0] = m_new;
        lq_run[0] = lq_run[0] * f0 + ml[64] * f1;
        dl_run[0] = dl_run[0] * f0 + ml[128] * f1;
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const f32x4_t x = *(const f32x4_t*)(mo + (db * 4 + g) * 256);
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    oacc[0][db][4 * g + i] = oacc[0][db][4 * g + i] * f0 + x[i] * f1;
            }
    }
    // ---- epilogue ----
    if (Q0 >= S)
        return;
    constexpr int OUTB = DT_OUT == NAUT_F32 ? 4 : 2;
    unsigned char* const o_bh = (unsigned char*)p.o + b * p.o_bs + hq * p.o_hs;
    // 16-bit O leaves through LDS in whole rows: a lane owns 4 consecutive d of one query (8 bytes, 32 different rows per
    // store instruction); after the exchange 16 lanes (D = 128) write one 256-byte row with 16 bytes each.
    constexpr int CPRO = W / 8, R256 = ROWB >= 256 ? 1 : 256 / ROWB;  // 16-byte chunks per row, rows per 256-byte bank line
    static_assert(OUTB == 4 || NWV * WQ * ROWB <= RINGB, "staging rows must fit the (first group's) tile buffers");
    unsigned char* const stg = smem + wave * WQ * ROWB;
    auto staged = [&](int r, int ch) {  // swizzled so that neither side conflicts
        return stg + r * ROWB + ((ch ^ ((r / R256) & (CPRO - 1))) << 4);
    };
#pragma unroll
    for (int hf = 0; hf < QH; ++hf) {
        const int q = qrow[hf];
        const float lt = 4.0f * half_sum(lq_run[hf]);
        const float inv_l = 1.0f / (lt + half_sum(dl_run[hf]));  // rows beyond S: never stored
        if (p.lse != nullptr && h == 0 && q < S)
            p.lse[(size_t)bh * S + q] = (m_run[hf] + __builtin_amdgcn_logf(lt)) * 0.6931471805599453f;
        unsigned char* const og = o_bh + (size_t)(q < S ? q : 0) * p.o_rs;
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const int d = 32 * db + 8 * g + 4 * h;
                const f32x4_t x = {oacc[hf][db][4 * g + 0] * inv_l, oacc[hf][db][4 * g + 1] * inv_l,
                                   oacc[hf][db][4 * g + 2] * inv_l, oacc[hf][db][4 * g + 3] * inv_l};
                if constexpr (OUTB == 2)
                    *(i32x2_t*)(staged(32 * hf + l32, d >> 3) + (d & 7) * 2) =
                        i32x2_t{In<DT_OUT>::pack2(x.x, x.y), In<DT_OUT>::pack2(x.z, x.w)};
                else if (q < S && d < cpr * 8)  // not the padding columns of a narrower head dimension
                    *(f32x4_t*)(og + d * 4) = x;
            }
    }
    if constexpr (OUTB == 2) {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        constexpr int RPI = 64 / CPRO;  // rows per store instruction
        typedef i32x4_t __attribute__((aligned(8))) i32x4_a8;  // O rows are 8-byte aligned, not more
        i32x4_t rows[WQ / RPI];
#pragma unroll
        for (int i = 0; i < WQ / RPI; ++i)  // all reads first: one LDS latency, not one per store
            rows[i] = *(const i32x4_t*)staged(i * RPI + lane / CPRO, lane % CPRO);
#pragma unroll
        for (int i = 0; i < WQ / RPI; ++i) {
            const int ch = lane % CPRO;
            const int q = Q0 + i * RPI + lane / CPRO;
            if (q < S && ch < cpr)  // not the rows beyond S, not the padding columns of a narrower head
                *(i32x4_a8*)(o_bh + (size_t)q * p.o_rs + ch * 16) = rows[i];
        }
    }
}
#endif
