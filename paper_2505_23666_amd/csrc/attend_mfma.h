// Chunk-parallel output kernel of the prefill for gfx950, bf16 storage (paper Sec. 3, y_t equation with the chunk sharing
// one state, "Chunkwise Inference"): any window, any sparse budget up to 1024, 64 or 128 head columns, 128 or 256 features.
//
// One workgroup takes one chunk (64 queries) of G query heads that read the same memories; wavefront w owns the 32 queries
// 32 (w % 2) .. of head w / 2.  Everything the workgroup reads besides its queries passes through LDS once for all of
// its heads, as one sequence of equal stages through two slots, each requested by direct global -> LDS loads
// while the one before it is worked on:
//   1. the keys and values: the chunk itself (causal), the window, the cache slots (gathered by virtual row): S^T = K Q^T,
//      weights e^(s - m) as bf16 high + low parts, out^T += V^T P^T with V^T through the transposing LDS read;
//   2. W_q (32 projections of every head per stage): z^T = W_q Q^T, then phi(q), scaled by the linear terms' weight e^-m, and
//      phi(q)^T s;
//   3. the chunk's snapshot of H^T (bf16 high + low parts in operand order, as the evolution kernel leaves it):
//      out^T += H^T phi(q)^T, three products.
// Then y = out / (sum of weights + e^-m phi(q)^T s).
//
// Products are 32x32x16 (A: row l % 32, contraction 8 (l / 32) + 0..7; B: column l % 32, same; C: column l % 32, rows
// 8 (i / 4) + 4 (l / 32) + i % 4) and transposed, so that a query's statistics live in two lanes and the C layout of one
// product is the B layout of the next: of a 32-row tile, registers {8 s .. 8 s + 7} serve as the B operand whose
// contraction slots are rows 16 s + 4 (l / 32) + {0..3, 8..11}; registers {0..3, 8..11} and {4..7, 12..15} match the pieces
// of the snapshot, whose operand order was made for 16-row products.
//
// What bounds it: vector instructions (weights, their split, addresses) and MFMAs of two wavefronts per SIMD, which hardly
// overlap (a 64-key step of a wavefront is 48 MFMAs of 32 cycles and about 350 vector instructions of 4); 16 queries per
// wavefront and one head per workgroup, as before, read every operand from LDS twice as often and the keys, the snapshot
// and W_q from L2 two to four times as often.  Whole launches on an empty chip, 3072 chunks of 4 heads (16 x 1536 tokens,
// 8B shape, budget 128): 545 us before, 370 - 390 now; 1024 chunks at eta = lambda = 256 with 256 features 560 -> 260; at eta 512 /
// lambda 1024 1290 -> 450 (534 TFLOP/s algorithmic).
// Tried: 64 queries per wavefront at one wavefront per SIMD (525 us for the first of these), three slots instead of two (the
// same or 10 % slower), several chunks per workgroup with the next one's first stages requested ahead (the scalar registers
// it takes cost more than the waits it hides), operands read from LDS a tile ahead by force (5 - 10 % slower).
#pragma once
#include "decode_mfma.h"
#include "generic_kernels.h"

namespace lola {
namespace fast {

typedef float f32x16 __attribute__((ext_vector_type(16)));
__device__ __forceinline__ f32x16 mfma32(bf16x8 a, bf16x8 b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ f32x16 zero_f32x16() {
    return (f32x16){0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
}
__device__ __forceinline__ float pair_sum(float v) { float x, y; swap32(v, x, y); return x + y; }
__device__ __forceinline__ float pair_max(float v) { float x, y; swap32(v, x, y); return fmaxf(x, y); }
__device__ __forceinline__ float pair_min(float v) { float x, y; swap32(v, x, y); return fminf(x, y); }

constexpr int ATTEND_MAXLAM = 1024;
static __device__ __attribute__((aligned(16))) const uint16_t attend_zero_row[128] = {0};   // the row of a position that holds no pair

template <int DH, int DF, int G>
struct AttendShape {
    static constexpr int M = DF / 2, NW = 2 * G, NTHR = 64 * NW;
    static constexpr int SB = G == 4 ? 32768 : 16384;      // bytes per stage
    static constexpr int NI = SB / 1024 / NW;              // direct loads per wavefront and stage
    static constexpr int QROWS = SB / (2 * DH), NQS = G * 64 / QROWS < 1 ? 1 : G * 64 / QROWS;   // queries per stage (rows beyond 64 G repeat)
    static constexpr int KB = SB / (4 * DH);               // keys per stage
    static constexpr int KSUB = KB < 64 ? KB : 64;         // keys per step of the running softmax
    static constexpr int PW = SB / (G * DH * 2);           // projections per head and W_q stage (rows beyond M repeat)
    static constexpr int NWS = PW >= M ? 1 : M / PW;
    static constexpr int FS = SB / (4 * DH), NHS = DF / FS;   // features per H^T stage (all rows, high + low parts)
    static constexpr int FC = 32;                          // features whose B operands are held at a time
    static constexpr int PR = DH / 8, RPI = 64 / PR;       // 16-byte pieces per row, rows per direct load
    // bytes of LDS: two slots, s, the cache's rows (LR: lambda in whole wavefronts, one at least: positions below the first key
    // look at row 0, also without a cache) and their addresses
    static constexpr int LR(int lam) { return lam < 64 ? 64 : (lam + 63) / 64 * 64; }
    static constexpr int lds(int lam) { return 2 * SB + DF * 4 + LR(lam) * (4 + 16); }
};

template <int DH, int DF, int G, typename TO>
__global__ __launch_bounds__((AttendShape<DH, DF, G>::NTHR), 2) void attend_group_kernel(generic::PrefillArgs<bf16_t> a) {
    using S = AttendShape<DH, DF, G>;
    constexpr int M = S::M, NI = S::NI, PR = S::PR, KS = DH / 16, NCT = DH / 32;
    static_assert((DH == 64 || DH == 128) && (DF == 128 || DF == 256), "shape");
    static_assert(S::LR(0) > 0, "row 0 exists");
    static_assert(DF % S::FS == 0 && S::FS % S::FC == 0 && M % S::FC == 0 && S::NI >= 2 && (S::NWS == 1 || S::NWS * S::PW == M), "stages");
    extern __shared__ __attribute__((aligned(1024))) unsigned char ring[];
    __shared__ int gneg_l;   // the chunk's cache has an empty slot

    const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, l32 = lane & 31, hi = lane >> 5;
    const int LAM = a.dm.lam, ETA = a.dm.eta, P = LAM + ETA, NKEYS = P + 64;
    const int LR = S::LR(LAM);
    float *s_l = reinterpret_cast<float *>(ring + 2 * S::SB);           // [DF]
    int *G_l = reinterpret_cast<int *>(s_l + DF);                       // [LR]
    ulonglong2 *adr_l = reinterpret_cast<ulonglong2 *>(G_l + LR);       // [LR] addresses of a slot's key and value row
    const int ns = a.dm.B * a.dm.Hkv;                // workgroups of one stream's head groups meet in one XCD when ns % 8 == 0
    const int j = a.j0 + (int)(blockIdx.z * gridDim.y + blockIdx.y);
    if (j >= a.j1) return;
    const int si = blockIdx.x % ns, b = si / a.dm.Hkv, h = si - b * a.dm.Hkv;
    const int hq0 = h * a.dm.g + (blockIdx.x / ns) * G, hl = w >> 1;
    const int64_t a0 = a.st.n_tokens[si];
    const int Tn = a.T_tokens;
    const int cl = min(64, Tn - j * 64);             // queries in this chunk
    const int64_t aj = a0 + (int64_t)j * 64;         // token index of the chunk's first query
    // filling chunks share one snapshot of H and s, that of the launch's first chunk, and have their rows in closed form
    const int spc_in = a.fill_closed ? a.st.sp_count[si] : 0;
    const bool filling = a.fill_closed && j < generic::first_scored_chunk(a, a0, spc_in);
    const size_t sj = (size_t)si * a.S + (j - a.jb), sh = filling ? (size_t)si * a.S + (a.j0 - a.jb) : sj;
    const uint16_t *Hsnap = reinterpret_cast<const uint16_t *>(a.snapH) + sh * (2 * DH * DF);
    const bf16_t *pK = a.prefK + (size_t)si * P * DH, *pV = a.prefV + (size_t)si * P * DH;
    const bf16_t *kc = a.k + (size_t)si * Tn * DH, *vc = a.v + (size_t)si * Tn * DH;
    const size_t qrow0 = ((size_t)b * a.dm.Hq + hq0) * Tn + (size_t)j * 64;
    const bf16_t *Wq = a.Wq + (size_t)hq0 * M * DH;   // [G][M][DH]
    const float scale2 = a.dm.scale * LOG2E;          // logits are kept in units of log2(e)
    const int wlo = aj < ETA ? -(int)aj : -ETA;      // first window position that holds a token, relative to the chunk
    // Stages of keys, from the chunk down to the cache (the last one's positions may begin below 0).  In a filling chunk the positions
    // from the first unused slot to the window's first token are empty: the stages that lie wholly among them, `gap` positions from
    // pskip + KB down, are passed over.  Read as zeros and masked, as before, they are work for nothing and all fetch the same
    // row: 8 x 32 ungrouped heads with 64 columns, 333 tokens at eta 512 / lambda 1024 412 us a call, 231 without them; 8 sequences of 1000
    // tokens of the 8B shape there 507 and 267.
    int NKS = (NKEYS + S::KB - 1) / S::KB, pskip = NKEYS, gap = 0;
    if (filling) {
        const int used = spc_in + generic::left_after(a, a0, j * 64);
        const int i0 = (NKEYS - P - wlo + S::KB - 1) / S::KB, nskip = max(0, (used > 0 ? (NKEYS - used) / S::KB : NKS) - i0);
        NKS -= nskip; gap = nskip * S::KB; pskip = NKEYS - (i0 + 1) * S::KB;
    }

    // Rows of Q, K, V and W_q lie row-major in their slot, their 16-byte pieces XOR-swizzled (a lane of a direct load chooses
    // which piece it fetches) so that neither the operand reads (16 rows, one piece each) nor the transposing reads
    // (4 rows x 32 columns) conflict, whether the banks are counted as 32 or as 64.
    auto kswz = [](int row) { return PR == 16 ? row & 15 : (row >> 1) & 7; };
    auto vswz = [](int key) { return PR == 16 ? ((key & 2) | ((key & 1) << 2) | ((key & 2) << 2)) : (key & 3) << 1; };

    // This wavefront's share of a stage.  (The lane number is made opaque in each: hoisted out of the key loop, the addresses
    // of all kinds of stages would occupy half of the registers.)
    auto opaque_lane = [&]() { int ln = lane; asm volatile("" : "+v"(ln)); return ln; };
    auto issue_q = [&](unsigned char *slot, int i) {
        const int ln = opaque_lane();
#pragma unroll
        for (int x0 = 0; x0 < NI; x0++) {
            const int x = w * NI + x0, rr = x * S::RPI + ln / PR, r = (i * S::QROWS + rr) % (64 * G);
            // rows past the chunk's end are read from row 0 (their results are never stored)
            const int q = (r & 63) < cl ? r & 63 : 0;
            lds_dma16(a.q + (qrow0 + (size_t)(r >> 6) * Tn + q) * DH + ((ln % PR) ^ kswz(rr)) * 8, slot + x * 1024);
        }
    };
    // row of a position, as the addresses of its key and value (selected as numbers: pointers would become branches)
    auto row_address = [&](int vr) -> ulonglong2 {
        const uintptr_t zr = (uintptr_t)attend_zero_row, off = (uintptr_t)(uint32_t)(vr < 0 ? 0 : (vr < P ? vr : vr - P)) * (2 * DH);
        const uintptr_t kr = vr < P ? (uintptr_t)pK : (uintptr_t)kc, vv = vr < P ? (uintptr_t)pV : (uintptr_t)vc;
        ulonglong2 r;
        r.x = (vr < 0 ? zr : kr) + off; r.y = (vr < 0 ? zr : vv) + off;
        return r;
    };
    auto issue_keys = [&](unsigned char *slot, int p0) {   // positions p0 ..
        const int tok0 = j * 64 + p0 - P;   // (call token of the stage's first position, behind the cache)
        const int ln = opaque_lane();
        if (p0 >= 0 && p0 + S::KB <= LAM) {
#pragma unroll
            for (int x0 = 0; x0 < NI / 2; x0++) {
                const int x = w * (NI / 2) + x0, kk = x * S::RPI + ln / PR;
                const ulonglong2 ad = adr_l[p0 + kk];
                lds_dma16((const void *)(ad.x + ((ln % PR) ^ kswz(kk)) * 16), slot + x * 1024);
                lds_dma16((const void *)(ad.y + ((ln % PR) ^ vswz(kk)) * 16), slot + S::SB / 2 + x * 1024);
            }
        } else if (p0 >= LAM && p0 - P >= wlo && p0 + S::KB - P <= cl && tok0 >= 0) {
            const char *k0 = reinterpret_cast<const char *>(kc + (size_t)tok0 * DH), *v0 = reinterpret_cast<const char *>(vc + (size_t)tok0 * DH);
#pragma unroll
            for (int x0 = 0; x0 < NI / 2; x0++) {
                const int x = w * (NI / 2) + x0, kk = x * S::RPI + ln / PR;
                lds_dma16(k0 + (uint32_t)(kk * (2 * DH) + ((ln % PR) ^ kswz(kk)) * 16), slot + x * 1024);
                lds_dma16(v0 + (uint32_t)(kk * (2 * DH) + ((ln % PR) ^ vswz(kk)) * 16), slot + S::SB / 2 + x * 1024);
            }
        } else {
#pragma unroll
            for (int x0 = 0; x0 < NI / 2; x0++) {
                const int x = w * (NI / 2) + x0, kk = x * S::RPI + ln / PR, pos = p0 + kk, wpos = pos - P;
                const int gr = LAM > 0 ? G_l[max(0, min(pos, LAM - 1))] : -1, wr = ((int)(wpos >= cl) | (int)(wpos < wlo)) ? -1 : P + j * 64 + wpos;
                const ulonglong2 ad = row_address(pos < 0 ? -1 : (pos < LAM ? gr : wr));
                lds_dma16((const void *)(ad.x + ((ln % PR) ^ kswz(kk)) * 16), slot + x * 1024);
                lds_dma16((const void *)(ad.y + ((ln % PR) ^ vswz(kk)) * 16), slot + S::SB / 2 + x * 1024);
            }
        }
    };
    auto issue_w = [&](unsigned char *slot, int i) {
        const int ln = opaque_lane();
#pragma unroll
        for (int x0 = 0; x0 < NI; x0++) {
            const int x = w * NI + x0, rr = x * S::RPI + ln / PR, pc = (ln % PR) ^ kswz(rr);
            const int pj = (i * S::PW + rr % S::PW) % M;
            lds_dma16(Wq + ((size_t)(rr / S::PW) * M + pj) * DH + pc * 8, slot + x * 1024);
        }
    };
    auto issue_h = [&](unsigned char *slot, int i) {
        const int ln = opaque_lane();
#pragma unroll
        for (int x0 = 0; x0 < NI; x0++) {
            const int x = w * NI + x0, rp = x / (S::FS / 32), ksl = x % (S::FS / 32);   // (part and row tile, k-step)
            lds_dma16(Hsnap + ((size_t)rp * (DF / 32) + i * (S::FS / 32) + ksl) * 512 + ln * 8, slot + x * 1024);
        }
    };
    // Stage n (of all) is complete in LDS and the stage before it has been read by all wavefronts; returns its slot, the other
    // one may be requested anew.
    auto begin = [&]() {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        lds_barrier();
    };
    auto slot_of = [&](int n) { return ring + (n & 1) * S::SB; };

    // the cache's rows (straight into LDS, or computed), s, and the queries; then the addresses of the cache's rows
    if (tid == 0) gneg_l = 0;
    if (filling) {
        for (int x = tid; x < LAM; x += S::NTHR) G_l[x] = generic::fill_row(a, a0, spc_in, j, x);
    } else {
        const int32_t *Gsnap = a.snapG + sj * LAM;
        for (int x = 64 * w; x < LAM; x += S::NTHR) lds_dma4(Gsnap + min(x + lane, LAM - 1), G_l + x);
    }
    for (int x = 64 * w; x < DF; x += S::NTHR) lds_dma4(a.snapS + sh * DF + x + lane, s_l + x);
    issue_q(slot_of(0), 0);
    const int hidec = (a.dm.hide & 2) ? -1 : 0;   // restricted query: no cache slot is read
    bf16x8 BQ[KS];   // queries as B operand (column = query, contraction = input index)
#pragma unroll
    for (int n = 0; n < S::NQS; n++) {
        begin();
        if (n == 0) {
            bool neg = false;
            for (int x = tid; x < LAM; x += S::NTHR) { const int vr = G_l[x]; neg |= vr < 0; adr_l[x] = row_address(vr); }
            if (neg) gneg_l = 1;
        }
        if (n + 1 < S::NQS) issue_q(slot_of(n + 1), n + 1);
        else {
            if (n == 0) lds_barrier();   // (the addresses are there)
            issue_keys(slot_of(n + 1), NKEYS - S::KB);
        }
        if (S::NQS == 1 || n == hl * 64 / S::QROWS) {
            const uint16_t *Ql = reinterpret_cast<const uint16_t *>(slot_of(n));
            const int rr = (hl * 64) % S::QROWS + 32 * (w & 1) + l32;
#pragma unroll
            for (int ks = 0; ks < KS; ks++) BQ[ks] = as_bf16x8(*reinterpret_cast<const uint4 *>(&Ql[rr * DH + (((2 * ks + hi) ^ kswz(rr)) << 3)]));
        }
    }
    const bool holes = gneg_l != 0 || hidec != 0;   // some cache slots are not read
    f32x16 out[NCT];
    float lsum = 0.f;   // this lane's part of the sum of weights
    // running maximum (units of log2 e): a query's largest weight is exactly 1.  Raising it only for logits 2^8 beyond it spares
    // most of the rescaling (5 % of the kernel), but the largest weights are then split inexactly: outputs off by 2.5e-6 (2-norm)
    // instead of 1.9e-6.
    float mrun = 0.f;
#pragma unroll
    for (int ct = 0; ct < NCT; ct++) out[ct] = zero_f32x16();
    int pnext = NKEYS - S::KB;   // first position of the stage that was requested last
#pragma unroll 1
    for (int n = 0; n < NKS; n++) {
        begin();
        const unsigned char *slot = slot_of(S::NQS + n);
        const int ps = pnext;
        pnext -= S::KB;
        if (pnext == pskip) pnext -= gap;
        if (n + 1 < NKS) issue_keys(slot_of(S::NQS + n + 1), pnext);
        else issue_w(slot_of(S::NQS + n + 1), 0);
        const uint16_t *Kl = reinterpret_cast<const uint16_t *>(slot), *Vl = Kl + S::SB / 4;
#pragma unroll
        for (int sub = 0; sub < S::KB / S::KSUB; sub++) {
            const int p0 = ps + sub * S::KSUB;
            if (p0 + S::KSUB <= 0) continue;
            f32x16 sc[S::KSUB / 32];
#pragma unroll
            for (int t = 0; t < S::KSUB / 32; t++) {
                const int kr = sub * S::KSUB + 32 * t + l32;
                sc[t] = zero_f32x16();
#pragma unroll
                for (int ks = 0; ks < KS; ks++) {
                    const bf16x8 A = as_bf16x8(*reinterpret_cast<const uint4 *>(&Kl[kr * DH + (((2 * ks + hi) ^ kswz(kr)) << 3)]));
                    sc[t] = mfma32(A, BQ[ks], sc[t]);
                }
            }
            // no masks in the cache and the window if every slot is in use, the window is full and the queries may read the
            // cache
            const bool whole = p0 >= (holes ? LAM : 0) && p0 + S::KSUB <= P && (aj >= ETA || p0 + S::KSUB <= LAM);
            if (!whole) {
                if (p0 >= LAM) {
#pragma unroll
                    for (int t = 0; t < S::KSUB / 32; t++)
#pragma unroll
                        for (int i = 0; i < 16; i++) {
                            const int wpos = p0 + 32 * t + 8 * (i >> 2) + 4 * hi + (i & 3) - P;
                            const int bad = (wpos - wlo) | (32 * (w & 1) + l32 - wpos);   // (sign bit)
                            sc[t][i] = bad < 0 ? -INFINITY : sc[t][i];
                        }
                } else {
#pragma unroll
                    for (int t = 0; t < S::KSUB / 32; t++)
#pragma unroll
                        for (int i = 0; i < 16; i++) {
                            const int pos = p0 + 32 * t + 8 * (i >> 2) + 4 * hi + (i & 3), wpos = pos - P;
                            const int gr = G_l[max(0, min(pos, LAM - 1))] | hidec | pos, incache = (pos - LAM) >> 31;   // (all ones: a cache slot)
                            const int bad = (incache & gr) | (~incache & ((wpos - wlo) | (32 * (w & 1) + l32 - wpos)));
                            sc[t][i] = bad < 0 ? -INFINITY : sc[t][i];
                        }
                }
            }
            float bmax = -INFINITY;
#pragma unroll
            for (int t = 0; t < S::KSUB / 32; t++)
#pragma unroll
                for (int i = 0; i < 16; i++) bmax = fmaxf(bmax, sc[t][i]);
            const float mnew = pair_max(bmax) * scale2;
            if (__any(mnew > mrun)) {
                const float mr = fmaxf(mrun, mnew), resc = fexp2(mrun - mr);
                mrun = mr;
                lsum *= resc;
#pragma unroll
                for (int ct = 0; ct < NCT; ct++) out[ct] *= resc;
            }
#pragma unroll
            for (int s = 0; s < S::KSUB / 16; s++) {
                bf16x8 Ph, Pl;
                float pw[8];
#pragma unroll
                for (int e = 0; e < 8; e++) pw[e] = fexp2(fmaf(sc[s >> 1][8 * (s & 1) + e], scale2, -mrun));
                lsum += ((pw[0] + pw[1]) + (pw[2] + pw[3])) + ((pw[4] + pw[5]) + (pw[6] + pw[7]));
                asm volatile("" : "+v"(lsum));   // (before the split, which may then work in place)
                split8_beside(pw, Ph, Pl);
                const int key = sub * S::KSUB + 16 * s + 4 * hi + ((lane & 15) >> 2);
                const uint16_t *vb = &Vl[key * DH + 4 * (lane & 1)];
#pragma unroll
                for (int ct = 0; ct < NCT; ct++) {
                    const int pc = ((4 * ct + 2 * ((lane >> 4) & 1) + ((lane & 3) >> 1)) ^ vswz(key)) << 3;
                    const bf16x4 b0 = tr_read(vb + pc), b1 = tr_read(vb + 8 * DH + pc);   // (key and key + 8 have one swizzle)
                    const bf16x8 Av = __builtin_shufflevector(b0, b1, 0, 1, 2, 3, 4, 5, 6, 7);
                    out[ct] = mfma32(Av, Ph, out[ct]);
                    out[ct] = mfma32(Av, Pl, out[ct]);
                }
            }
        }
    }
    const int nt = S::NQS + NKS;   // number of the first stage of W_q
    // ---- phi(q)
    f32x16 zt[M / 32];
#pragma unroll
    for (int n = 0; n < S::NWS; n++) {
        begin();
        if (n + 1 < S::NWS) issue_w(slot_of(nt + n + 1), n + 1);
        else issue_h(slot_of(nt + n + 1), 0);
        const uint16_t *Wl = reinterpret_cast<const uint16_t *>(slot_of(nt + n));
#pragma unroll
        for (int tt = 0; tt < (S::PW < M ? S::PW : M) / 32; tt++) {
            const int rr = hl * S::PW + 32 * tt + l32;
            zt[n * (S::PW / 32) + tt] = zero_f32x16();
#pragma unroll
            for (int ks = 0; ks < KS; ks++) {
                const bf16x8 A = as_bf16x8(*reinterpret_cast<const uint4 *>(&Wl[rr * DH + (((2 * ks + hi) ^ kswz(rr)) << 3)]));
                zt[n * (S::PW / 32) + tt] = mfma32(A, BQ[ks], zt[n * (S::PW / 32) + tt]);
            }
        }
    }
    {
        const float el = (a.dm.hide & 1) ? 0.f : fexp2(-mrun);   // weight of the linear terms (restricted query: none)
        float cp = 0.f, cn = 0.f, ip = el;
        if (a.dm.phi_kind != 1) {
            float zmax = zt[0][0], zmin = zt[0][0];
#pragma unroll
            for (int t = 0; t < M / 32; t++)
#pragma unroll
                for (int i = 0; i < 16; i++) { zmax = fmaxf(zmax, zt[t][i]); zmin = fminf(zmin, zt[t][i]); }
            cp = -pair_max(zmax) * LOG2E; cn = pair_min(zmin) * LOG2E;
        }
        // ---- linear part, FC features at a time: first the positive half, then the negative one
        const unsigned char *Hs = nullptr;
#pragma unroll
        for (int n = 0; n < S::NHS; n++) {
#pragma unroll
            for (int u = 0; u < S::FS / S::FC; u++) {
                const int F0 = n * S::FS + u * S::FC, t0 = F0 % M / 32;
                const bool neg = F0 >= M;
                bf16x8 Bh[S::FC / 16], Bl[S::FC / 16];   // per 32 features: registers {0..3, 8..11}, {4..7, 12..15} of their tile
                // (kept apart from the steps before and behind, and the features computed anew from z where they are needed:
                // otherwise it does not fit the registers)
                __builtin_amdgcn_sched_barrier(0);
                if (n + u > 0) {
#pragma unroll
                    for (int t = 0; t < M / 32; t++) asm volatile("" : "+v"(zt[t]));
                }
                auto feat = [&](int t, int i) { return neg ? fexp2(fmaf(zt[t][i], -LOG2E, cn)) : fexp2(fmaf(zt[t][i], LOG2E, cp)); };
                if (F0 % M == 0) {
                    float sum = 0.f;
#pragma unroll
                    for (int t = 0; t < M / 32; t++)
#pragma unroll
                        for (int i = 0; i < 16; i++) sum += feat(t, i);
                    ip = a.dm.phi_kind == 1 ? el : el * frcp(pair_sum(sum));
                    if (M > S::FC) {
#pragma unroll
                        for (int t = 0; t < M / 32; t++) asm volatile("" : "+v"(zt[t]));
                    }
                }
#pragma unroll
                for (int tt = 0; tt < S::FC / 32; tt++) {
                    const int t = t0 + tt;
                    float f[16];
#pragma unroll
                    for (int x = 0; x < 4; x++) {
                        const float4 s4 = *reinterpret_cast<const float4 *>(&s_l[(neg ? M : 0) + 32 * t + 8 * x + 4 * hi]);
#pragma unroll
                        for (int i = 0; i < 4; i++) f[4 * x + i] = feat(t, 4 * x + i) * ip;
                        lsum = fmaf(f[4 * x], s4.x, lsum); lsum = fmaf(f[4 * x + 1], s4.y, lsum);
                        lsum = fmaf(f[4 * x + 2], s4.z, lsum); lsum = fmaf(f[4 * x + 3], s4.w, lsum);
                    }
                    const float v0[8] = {f[0], f[1], f[2], f[3], f[8], f[9], f[10], f[11]};
                    const float v1[8] = {f[4], f[5], f[6], f[7], f[12], f[13], f[14], f[15]};
                    split8_beside(v0, Bh[2 * tt], Bl[2 * tt]);
                    split8_beside(v1, Bh[2 * tt + 1], Bl[2 * tt + 1]);
                }
                if (u == 0) {
                    begin();
                    if (n + 1 < S::NHS) issue_h(slot_of(nt + S::NWS + n + 1), n + 1);
                    Hs = slot_of(nt + S::NWS + n);
                }
                const unsigned char *Hl = Hs + u * (S::FC / 32) * 1024 + ((lane >> 4) & 1) * (S::FS * 32) + (lane & 15) * 16 + hi * 256;
#pragma unroll
                for (int ks = 0; ks < S::FC / 16; ks++) {
#pragma unroll
                    for (int ct = 0; ct < NCT; ct++) {
                        const unsigned char *p = Hl + 2 * ct * (S::FS * 32) + (ks >> 1) * 1024 + (ks & 1) * 512;
                        const bf16x8 Ah = as_bf16x8(*reinterpret_cast<const uint4 *>(p));
                        const bf16x8 Al = as_bf16x8(*reinterpret_cast<const uint4 *>(p + S::SB / 2));
                        out[ct] = mfma32(Ah, Bh[ks], out[ct]);
                        out[ct] = mfma32(Ah, Bl[ks], out[ct]);
                        out[ct] = mfma32(Al, Bh[ks], out[ct]);
                    }
                }
            }
        }
    }
    const int qi = 32 * (w & 1) + l32;
    const float inv = frcp(pair_sum(lsum));
    if (qi < cl) {
        TO *oh = (TO *)a.out + (qrow0 + (size_t)hl * Tn + qi) * DH + 4 * hi;
#pragma unroll
        for (int ct = 0; ct < NCT; ct++)
#pragma unroll
            for (int x = 0; x < 4; x++)
#pragma unroll
                for (int i = 0; i < 4; i++) stf(oh, 32 * ct + 8 * x + i, out[ct][4 * x + i] * inv);
    }
}

}  // namespace fast
}  // namespace lola
