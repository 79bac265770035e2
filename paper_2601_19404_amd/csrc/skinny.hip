// C[M,N] (op)= A[M,K] * W[N,K]^T for a handful of rows (bf16 operands, fp32 accumulation): the
// contractions of a decode step of a small batch, and the narrow ones of a larger batch in groups of 64 rows.
//
// What bounds them is how fast a CU can be fed: 64 rows use a weight 64 times, far from what the matrix
// cores need to be the limit, and every weight byte comes from HBM once per decode step (the layers
// together are larger than every cache).  Measured on this chip: loads of whole 128-byte lines, into LDS or
// into registers, reach 133 GB/s per CU from L2 (all CUs reading 2 MB) and 107 from HBM (16 CUs reading); the
// fragment layout (16 rows x 64 bytes per instruction) reaches 37 and 38 whatever is in flight.  All CUs together get
// 6.0 to 6.2 TB/s from HBM either way (6 GiB read once; 7.4 to 9.1 TB/s from 128 MB, which the 256 MB memory-side
// cache holds), so it is the activations, read again by every workgroup, that the layout decides over: a kernel built on
// fragments lost to the 64-row tiles from 16 rows on.  Hence:
//   * weights and activations go to LDS in pieces of 8 rows x 128 bytes, and every wave has a ring of
//     its own that only it reads: the main loop has no barrier, a wave waits for its own loads only;
//   * K is split over the NW waves of a workgroup (wave w takes slabs w, w + NW, ...), so a narrow
//     projection still puts every CU to work; the partial sums meet in LDS, in a fixed order;
//   * 8 rows of activations move 8 rows, not a padded tile of 64: the loads are what is paid for;
//   * the weight rows are the A operand of v_mfma_f32_16x16x32_bf16 and the activations the B operand:
//     a lane then holds one activation row and four consecutive columns of the result.
// Against the 32x128 / 64x64 / 64x128 tiles of gemm.hip, weights streamed from HBM, 8 / 32 / 64 rows, us:
//   K = 1536: N = 2048 (QKV) 8.1 / 8.3 / 8.3 -> 3.4 / 4.1 / 5.2; N = 17920 (gate/up) 15.3 / 16.7 / 18.7 ->
//   11.7 / 13.1 / 15.1; K = 8960, N = 1536 (down, with its reduction) 15.3 / 16.0 / 17.2 -> 12.0 / 13.3 / 14.3;
//   K = 3584: N = 3584 (O) 12.7 / 13.5 / 14.9 -> 7.6 / 11.0 / 12.8; N = 37888 (gate/up) 61.9 / 63.5 / 68.7 ->
//   49.8 / 51.3 / 57.4 (5.5 TB/s of weights at 8 rows).
// Weights from HBM asked for with the non-temporal hint, and no bank conflicts left in the fragment reads (42 % of the LDS cycles
// before), the same shapes, 8 / 30 / 64 rows: QKV 4.4 / 5.6 / 7.0 -> 3.8 / 4.9 / 6.4, gate/up 12.4 / 13.8 / 15.9 -> 11.0 / 12.7 /
// 14.9, down 11.9 / 12.9 / 14.5 -> 10.9 / 12.1 / 14.4; O (K = 3584) 7.7 / 9.9 / 13.2 -> 6.9 / 9.2 / 12.4; gate/up (N = 37888) 48.2 /
// 51.6 / 57.7 -> 42.7 / 46.9 / 54.6 (6.4 TB/s); LM head (N = 151936, K = 1536) 85.4 / 97.5 / 114 -> 73.0 / 89.8 / 111.
#include "kernels.hpp"

namespace rpo {

// 65 to 512 rows (QKV and O of a decode step): the 16-row weight blocks per workgroup, 0: not for this kernel.
// Every group of 64 rows reads the weights again, from L2, and a workgroup that waits for a second round costs more
// than all that is gained, so the groups are taken only where they fit the CUs in one round.  Weights from HBM,
// 64x64 tiles -> this kernel, us: N = 2048, K = 1536: 128 rows 8.6 -> 5.6 (one block), 256 rows 8.8 -> 6.5 (two),
// 512 rows 9.7 -> 8.2 (four); N = 1536: 8.9 -> 5.9, 9.2 -> 6.6, 9.8 -> 8.5; N = K = 3584: 128 rows 20.1 -> 14.7 (two),
// 256 rows 21.5 -> 19.2 (four).  Past one round: 512 rows of N = 2048 with two blocks 11.1; N = 4608, K = 3584, 256 rows
// with four 31.5 against 31.4.  A deep K (down) and a wide N (gate/up) lose: 22.9 -> 25.3, 34.1 -> 35.9 us at 256 rows.
// A round is counted per XCD: all groups of a column block go to one of them, so 35 blocks of 7 groups put 35
// workgroups on the 32 CUs of three XCDs and 28 on the others (N = 1100, 400 rows, K = 512 to 3584, accumulating: 6.1 ->
// 7.8, 9.5 -> 11.4, 16.5 -> 17.6 us with two blocks).  Less than four slabs leave waves without one (N = 5120,
// K = 64, 96 rows 3.4 -> 3.9), and over a shallow K four blocks have too little to do for the residual's read at their
// end (accumulating: 96 rows, N = 8192, K = 1536 10.7 -> 12.4; 512 rows, N = 1100, K = 512 6.2 -> 7.2).
int gemm_skinny_groups(const GemmArgs& a) {
    if (a.K > 4096 || a.K < 256 || a.M > 512 || (a.epilogue != kEpiStore && a.epilogue != kEpiAddF32)) return 0;
    const int groups = ceil_div(a.M, 64);
    for (int nb = 1; nb <= 4; nb *= 2)
        if ((int64_t)ceil_div(ceil_div(a.N, nb * 16), 8) * groups <= 32)
            return nb == 4 && a.epilogue == kEpiAddF32 && a.K < (groups == 2 ? 2048 : 1024) ? 0 : nb;
    return 0;
}

namespace {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef unsigned short u16x4_t __attribute__((ext_vector_type(4)));

template <int N>
__device__ inline void wait_loads() {  // all but the newest N loads of this wave have landed
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// MA 8-row blocks of activations, NB 16-row blocks of weights per workgroup, NW waves (K split), rings of S
// slabs of 64 K values.  The weight rows of block t:
//   kEpiSwiglu: gate rows 8 q .. 8 q + 7, then up rows F + 8 q .. F + 8 q + 7, q = NB blockIdx.x + t
//   kEpiRope:   of head u / 8 the channels i0 .. i0 + 7 and 64 + i0 .. 64 + i0 + 7, u = NB blockIdx.x + t,
//               i0 = 8 (u % 8): the rotation pairs sit in one block (head_dim 128)
//   otherwise:  16 (NB blockIdx.x + t) ..
// kEpiPartial: workgroup (b, z) multiplies K slabs [z slabs_per_split, ...) only and stores fp32 partial sums to
// Cv[z][M][N] (ldc is not used).
template <int MA, int NB, int NW, int S, int EPI, bool GROUPS, bool ONCE>
__global__ __launch_bounds__(NW * 64) void gemm_skinny_kernel(const bf16* __restrict__ A, int64_t lda,
                                                              const bf16* __restrict__ W, int64_t ldw,
                                                              void* __restrict__ Cv, int64_t ldc, int M, int N,
                                                              int K, int slabs_per_split, int blocks,
                                                              int row_groups, RopeKvArgs rk, LseFuse lf, NormFuse nf) {
    static_assert(EPI != kEpiLogitsMax || NB == 4, "row maxima are kept per 64 columns");
    constexpr int MB = (MA + 1) / 2;  // 16-column MFMA blocks of activations (MA = 1: rows 0 .. 7 twice)
    constexpr int ROWS = MB * 16, COLS = NB * 16;
    constexpr int LD = COLS + 4;      // fp32 row of the partial sums, 16-byte pieces
    constexpr int INST = 2 * NB + MA;  // loads per slab; each fills 1 KiB of LDS (8 rows x 128 bytes)
    constexpr int STAGE = INST * 1024;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];  // rings [NW][S][STAGE], then partial sums
    float* part = (float*)smem;                                          // [NW][ROWS][LD]

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r = lane & 15, g = lane >> 4;
    // Row groups of one column block sit next to each other on one XCD (workgroups go to the eight XCDs in turn):
    // the weights come from HBM once and from that XCD's L2 for the other groups.
    int b = blockIdx.x, m0 = 0;
    if constexpr (GROUPS) {
        const int t = b >> 3;
        m0 = t % row_groups * (MA * 8);
        b = (t / row_groups) * 8 + (b & 7);
        if (b >= blocks) return;  // the whole workgroup
    }
    const int F = N / 2;

    // Load addressing: an instruction fills 8 rows; lane l stores piece position l % 8 of row l / 8 and fetches
    // piece (l % 8) ^ (row % 8), which spreads the fragment reads over the LDS banks (a 16-byte read is served 16 lanes
    // at a time: 0-3, 12-15, 20-23 and 24-27 together, so two pieces of eight rows each).
    uint32_t off[INST];
#pragma unroll
    for (int j = 0; j < INST; ++j) {
        const int l8 = lane >> 3;                   // row in the 8-row group
        const int half = j < 2 * NB ? (j & 1) : ((j - 2 * NB) & 1);  // which half of a 16-row block
        const int piece = (lane & 7) ^ l8;
        if (j < 2 * NB) {
            const int t = j >> 1;
            int row;
            if (EPI == kEpiSwiglu)
                row = half * F + min((b * NB + t) * 8 + l8, F - 1);
            else if (EPI == kEpiRope)
                row = ((b * NB + t) >> 3) * 128 + half * 64 + ((b * NB + t) & 7) * 8 + l8;
            else
                row = min((b * NB + t) * 16 + half * 8 + l8, N - 1);
            off[j] = (uint32_t)(((int64_t)row * ldw + piece * 8) * 2);
        } else {
            off[j] = (uint32_t)(((int64_t)min(m0 + (j - 2 * NB) * 8 + l8, M - 1) * lda + piece * 8) * 2);
        }
    }
    const uint32_t ring = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)smem + wave * (S * STAGE);
    const unsigned char* ring_p = smem + wave * (S * STAGE);

    f32x4_t acc[MB][NB];
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int t = 0; t < NB; ++t) acc[i][t] = f32x4_t{0.f, 0.f, 0.f, 0.f};

    // this wave's slabs: wave + i * NW, i < n_my, counted from the workgroup's own first slab: every workgroup
    // reads the same activations, and those running together then ask the L2 for different lines
    const int slab0 = EPI == kEpiPartial ? (int)blockIdx.y * slabs_per_split : 0;
    const int n_slabs = EPI == kEpiPartial ? min(slabs_per_split, (K >> 6) - slab0) : K >> 6;
    const int n_my = n_slabs > wave ? (n_slabs - wave + NW - 1) / NW : 0;
    const int rot = (int)((unsigned)b * 5u % (unsigned)n_slabs);
    auto issue = [&](int i, int st) __attribute__((always_inline)) {
        int sl = wave + i * NW + rot;
        sl = sl >= n_slabs ? sl - n_slabs : sl;
        sl += slab0;
        const bf16* wb = W + sl * 64;
        const bf16* ab = A + sl * 64;
#pragma unroll
        for (int j = 0; j < INST; ++j) {
            if (j < 2 * NB)
                dma_load16_at<ONCE>(wb, off[j], ring + st * STAGE, j * 1024);
            else
                dma_load16_at<false>(ab, off[j], ring + st * STAGE, j * 1024);
        }
    };
    const int sw = r & 7;
    const int ar = MA == 1 ? (r & 7) : r;
    auto multiply = [&](int st) __attribute__((always_inline)) {
        const unsigned char* base = ring_p + st * STAGE;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            bf16x8_t wf[NB], af[MB];
#pragma unroll
            for (int t = 0; t < NB; ++t)
                wf[t] = *(const bf16x8_t*)(base + t * 2048 + r * 128 + (((4 * h + g) ^ sw) << 4));
#pragma unroll
            for (int m = 0; m < MB; ++m)
                af[m] = *(const bf16x8_t*)(base + NB * 2048 + m * 2048 + ar * 128 + (((4 * h + g) ^ sw) << 4));
#pragma unroll
            for (int m = 0; m < MB; ++m)
#pragma unroll
                for (int t = 0; t < NB; ++t)
                    acc[m][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[t], af[m], acc[m][t], 0, 0, 0);
        }
    };
    // No barrier in the loop: a wave loads and reads its own ring only.
#pragma unroll
    for (int i = 0; i < S - 1; ++i)
        if (i < n_my) issue(i, i);
    // h of a norm taken apart: the rows' sums of squares (wave w: rows w, w + NW, ..., up to 256 blocks) are asked for
    // behind the first slabs and used after the last.
    constexpr bool kNormIn = EPI == kEpiSwiglu && MA <= 4;
    constexpr int kRows = kNormIn ? ROWS / NW : 1;
    float sq[kRows][4] = {};
    if constexpr (kNormIn) {
        if (nf.part) {  // uniform: asked per load, a projection without one paid for the questions (24 rows of 512 x 512 3.19 -> 2.90 us)
#pragma unroll
            for (int i = 0; i < kRows; ++i)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int m = wave + i * NW, c = lane + 64 * q;
                    if (m < M && c < nf.blocks) sq[i][q] = nf.part[m * nf.blocks + c];
                }
        }
    }
    int st = 0;
#pragma clang loop unroll(disable)
    for (int i = 0; i < n_my; ++i) {
        const int ahead = n_my - 1 - i;  // slabs after this one
        if (ahead >= S - 1) {
            // the stage that slab i - 1 has left: its reads are done before new data can arrive
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            issue(i + S - 1, st == 0 ? S - 1 : st - 1);
            wait_loads<(S - 1) * INST>();
        } else if (S > 3 && ahead == 2) {
            wait_loads<2 * INST>();
        } else if (S > 2 && ahead == 1) {
            wait_loads<INST>();
        } else {
            wait_loads<0>();
        }
        multiply(st);
        st = st + 1 == S ? 0 : st + 1;
    }
    __syncthreads();  // the rings are free: the partial sums take their place
    {
        float* dst = part + ((size_t)wave * ROWS + r) * LD + 4 * g;
#pragma unroll
        for (int m = 0; m < MB; ++m)
#pragma unroll
            for (int t = 0; t < NB; ++t) *(f32x4_t*)(dst + m * 16 * LD + t * 16) = acc[m][t];
    }
    float* inv = part + NW * ROWS * LD;  // [ROWS]
    if constexpr (kNormIn) {
        if (nf.part) {
#pragma unroll
            for (int i = 0; i < kRows; ++i) {
                const float ss = wave_sum((sq[i][0] + sq[i][1]) + (sq[i][2] + sq[i][3]));
                if (lane == 0) inv[wave + i * NW] = 1.0f / sqrtf(ss / (float)K + nf.eps);
            }
        }
    }
    __syncthreads();

    // four consecutive columns of row m, summed over the waves in order
    auto total = [&](int m, int c) __attribute__((always_inline)) {
        f32x4_t v = *(const f32x4_t*)(part + m * LD + c);
#pragma unroll
        for (int w = 1; w < NW; ++w) v += *(const f32x4_t*)(part + (w * ROWS + m) * LD + c);
        return v;
    };

    if constexpr (EPI == kEpiSwiglu) {
        const bool vec = (ldc & 3) == 0 && ((uintptr_t)Cv & 7) == 0;
        for (int it = tid; it < ROWS * NB * 2; it += NW * 64) {
            const int m = m0 + it / (NB * 2), q = it % (NB * 2);
            const int c = (q >> 1) * 16 + (q & 1) * 4, oc = (b * NB + (q >> 1)) * 8 + (q & 1) * 4;
            if (m >= M) continue;
            f32x4_t gate = total(m - m0, c), up = total(m - m0, 8 + c);
            if (kNormIn && nf.part) {
                const float f = inv[m - m0];
                gate *= f;
                up *= f;
            }
            u16x4_t o;
#pragma unroll
            for (int e = 0; e < 4; ++e) o[e] = f32_to_bf16(silu_f(gate[e]) * up[e]).bits;
            bf16* dst = (bf16*)Cv + (int64_t)m * ldc + oc;
            if (vec && oc + 3 < F) {
                *(u16x4_t*)dst = o;
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (oc + e < F) dst[e].bits = o[e];
            }
        }
    } else if constexpr (EPI == kEpiRope) {
        const int pt = rk.geom.page_tokens;
        for (int it = tid; it < ROWS * NB * 2; it += NW * 64) {
            const int m = m0 + it / (NB * 2), q = it % (NB * 2);
            const int unit = b * NB + (q >> 1), head = unit >> 3;
            const int c = (q >> 1) * 16 + (q & 1) * 4, ch = (unit & 7) * 8 + (q & 1) * 4;
            if (m >= M) continue;
            const f32x4_t x1 = total(m - m0, c), x2 = total(m - m0, 8 + c);
            int pos = -1;
            int64_t page = 0;
            const int seq = rk.row_seq ? rk.row_seq[m] : m;
            if (seq >= 0 && !(rk.active && !rk.active[m])) {
                const SeqDesc sd = rk.seqs[seq];
                pos = sd.pos0 + (rk.single_row ? 0 : m - sd.row_start) + rk.pos_add;
                page = rk.tables[sd.table_off + pos / pt];
            }
            bf16* pool = (bf16*)rk.kv_pool;
            if (head >= rk.Hq + rk.Hkv) {
                if (pos < 0) continue;
                bf16* v = pool + rk.geom.v_block(rk.layer, page, head - rk.Hq - rk.Hkv);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    v[rk.geom.v_elem(pos % pt, ch + e)] = f32_to_bf16(x1[e]);
                    v[rk.geom.v_elem(pos % pt, ch + e + 64)] = f32_to_bf16(x2[e]);
                }
                continue;
            }
            u16x4_t y1, y2;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                float a1 = x1[e], a2 = x2[e];
                if (pos >= 0) {  // a finished rollout keeps an unrotated q
                    const float2 cs = *(const float2*)(rk.rope + ((int64_t)pos * 64 + ch + e) * 2);
                    a1 = x1[e] * cs.x - x2[e] * cs.y;
                    a2 = x2[e] * cs.x + x1[e] * cs.y;
                }
                y1[e] = f32_to_bf16(a1).bits;
                y2[e] = f32_to_bf16(a2).bits;
            }
            bf16* dst;
            if (head < rk.Hq) {
                dst = (bf16*)Cv + (int64_t)m * ldc + head * 128 + ch;
            } else {
                if (pos < 0) continue;
                dst = pool + rk.geom.k_block(rk.layer, page, head - rk.Hq) + (int64_t)(pos % pt) * 128 + ch;
            }
            *(u16x4_t*)dst = y1;
            *(u16x4_t*)(dst + 64) = y2;
        }
    } else {
        constexpr int QPR = COLS / 4;  // column quads per row
        if constexpr (EPI == kEpiPartial) {
            Cv = (float*)Cv + (int64_t)blockIdx.y * M * N;
            ldc = N;
        }
        const bool vec = EPI == kEpiStore ? (ldc & 3) == 0 && ((uintptr_t)Cv & 7) == 0
                                          : (ldc & 3) == 0 && ((uintptr_t)Cv & 15) == 0;
        for (int it = tid; it < ROWS * QPR; it += NW * 64) {
            const int m = m0 + it / QPR, c = (it % QPR) * 4, n = b * COLS + c;
            if (m >= M) continue;  // all lanes of a row's quads together
            const f32x4_t v = total(m - m0, c);
            if constexpr (EPI == kEpiStore) {
                bf16* dst = (bf16*)Cv + (int64_t)m * ldc + n;
                u16x4_t o;
#pragma unroll
                for (int e = 0; e < 4; ++e) o[e] = f32_to_bf16(v[e]).bits;
                if (vec && n + 3 < N) {
                    *(u16x4_t*)dst = o;
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (n + e < N) dst[e].bits = o[e];
                }
            } else {
                float* dst = (float*)Cv + (int64_t)m * ldc + n;
                if constexpr (EPI == kEpiAddF32 && NB == 1) {
                    if (nf.part) {  // the norm that follows, taken apart: whole 16-column blocks, 16-byte rows (launcher)
                        const f32x4_t x = *(const f32x4_t*)dst + v;
                        const u16x4_t gain = *(const u16x4_t*)(nf.gain + n);
                        *(f32x4_t*)dst = x;
                        u16x4_t o;
#pragma unroll
                        for (int e = 0; e < 4; ++e) o[e] = f32_to_bf16(x[e] * bf16_to_f32(bf16{gain[e]})).bits;
                        *(u16x4_t*)(nf.h + (int64_t)m * N + n) = o;
                        float ss = (x[0] * x[0] + x[1] * x[1]) + (x[2] * x[2] + x[3] * x[3]);
                        ss += __shfl_xor(ss, 1, 64);
                        ss += __shfl_xor(ss, 2, 64);
                        if (c == 0) nf.part[(int64_t)m * nf.blocks + b] = ss;
                        continue;
                    }
                }
                if (vec && n + 3 < N) {
                    *(f32x4_t*)dst = EPI == kEpiAddF32 ? *(const f32x4_t*)dst + v : v;
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (n + e < N) dst[e] = EPI == kEpiAddF32 ? dst[e] + v[e] : v[e];
                }
                if constexpr (EPI == kEpiLogitsMax) {  // N is a multiple of 4 (checked by the launcher): whole quads
                    float mx = n < N ? fmaxf(fmaxf(v[0], v[1]), fmaxf(v[2], v[3])) : -INFINITY;
#pragma unroll
                    for (int o = 1; o < QPR; o <<= 1) mx = fmaxf(mx, __shfl_xor(mx, o, 64));
                    if (c == 0) lf.part[(int64_t)m * lf.blocks + b] = mx;
                }
            }
        }
    }
}

// LDS of one workgroup: the rings, or the partial sums that follow them.
template <int MA, int NB, int NW, int S>
constexpr size_t skinny_lds() {
    constexpr size_t rings = (size_t)NW * S * (2 * NB + MA) * 1024;
    constexpr size_t rows = (size_t)((MA + 1) / 2) * 16;
    constexpr size_t sums = (NW * rows * (NB * 16 + 4) + rows) * sizeof(float);  // and a factor per row
    return rings > sums ? rings : sums;
}

// PER_CU workgroups share a CU's 160 KiB of LDS; the ring is as deep as that allows, at most four slabs.
template <int MA, int NB, int NW, int PER_CU, int EPI, bool GROUPS, bool ONCE>
hipError_t launch_kernel(const GemmArgs& a, int blocks, hipStream_t s, int splits, void* out) {
    constexpr int kFit = 160 / PER_CU / (NW * (2 * NB + MA));
    constexpr int S = kFit < 4 ? kFit : 4;
    static_assert(S >= 2, "the ring needs two slabs");
    constexpr size_t lds = skinny_lds<MA, NB, NW, S>();
    static_assert(lds * PER_CU <= 160 * 1024, "LDS");
    auto kern = gemm_skinny_kernel<MA, NB, NW, S, EPI, GROUPS, ONCE>;
    static bool attr_set = false;  // one flag per template instance
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    const int row_groups = GROUPS ? ceil_div(a.M, MA * 8) : 1;
    const int grid = GROUPS ? ceil_div(blocks, 8) * 8 * row_groups : blocks;
    kern<<<dim3((unsigned)grid, (unsigned)splits), dim3(NW * 64), lds, s>>>(
        (const bf16*)a.A, a.lda, (const bf16*)a.W, a.ldw, out ? out : a.C, a.ldc, a.M, a.N, a.K,
        ceil_div(a.K / 64, splits), blocks, row_groups,
        (EPI == kEpiRope && a.rope) ? *a.rope : RopeKvArgs{},
        (EPI == kEpiLogitsMax && a.block_max) ? *a.block_max : LseFuse{},
        (EPI == kEpiAddF32 && a.norm_split) ? *a.norm_split : (EPI == kEpiSwiglu && a.norm_in) ? *a.norm_in : NormFuse{});
    return hipGetLastError();
}

// One workgroup reads a weight row: weights from HBM come with the non-temporal hint (8 / 30 rows of K = 3584, N = 37888 48.1
// -> 42.7 / 51.5 -> 46.9 us = 6.4 / 5.8 TB/s).  Not where 64 rows of activations, read by every workgroup, outweigh them
// (down, K = 8960: 14.5 -> 14.9 us).  A kernel of its own: both kinds of load in one cost 0.1 us a launch.
template <int MA, int NB, int NW, int PER_CU, int EPI, bool GROUPS = false>
hipError_t launch_one(const GemmArgs& a, int blocks, hipStream_t s, int splits = 1, void* out = nullptr) {
    if constexpr (!GROUPS && !(EPI == kEpiPartial && MA == 8))
        if (gemm_weights_pass(a)) return launch_kernel<MA, NB, NW, PER_CU, EPI, GROUPS, true>(a, blocks, s, splits, out);
    return launch_kernel<MA, NB, NW, PER_CU, EPI, GROUPS, false>(a, blocks, s, splits, out);
}

template <int MA, int EPI>
hipError_t launch_rows(const GemmArgs& a, int splits, hipStream_t s) {
    // A workgroup reads all activations whatever its weight blocks are, and one that waits for a second round costs
    // a whole round: the fewest weight blocks per workgroup that put all of them on the CUs in one round.  Beyond
    // what six (gate/up) or three blocks hold: two smaller workgroups per CU, so that one's loads cover the other's
    // reduction.  us, five blocks always (gate/up) or one (store) -> this, weights from HBM: gate/up, F = 2048, K =
    // 3584, 8 / 64 rows 15.7 / 23.1 -> 7.9 / 13.3; F = 11008, K = 3584 39.9 / 51.2 -> 29.6 / 33.8; store, N = 12288, K =
    // 3584 17.0 / 33.3 -> 17.7 / 21.8; N = 8192, K = 1536 6.7 / 11.0 -> 6.8 / 9.1.
    if constexpr (EPI == kEpiSwiglu) {
        const int units = ceil_div(a.N / 2, 8);
        if (units <= 256) return launch_one<MA, 1, 8, 1, EPI>(a, units, s);
        if (units <= 256 * 2) return launch_one<MA, 2, 4, 1, EPI>(a, ceil_div(units, 2), s);
        if (units <= 256 * 3) return launch_one<MA, 3, 4, 1, EPI>(a, ceil_div(units, 3), s);
        if (units <= 256 * 4) return launch_one<MA, 4, 4, 1, EPI>(a, ceil_div(units, 4), s);
        if (units <= 256 * 5) return launch_one<MA, 5, 4, 1, EPI>(a, ceil_div(units, 5), s);
        if (units <= 256 * 6) return launch_one<MA, 6, 4, 1, EPI>(a, ceil_div(units, 6), s);
        if constexpr (MA <= 2) {  // more rows of these widths are not taken
            if (units <= 512 * 4) return launch_one<MA, 4, 2, 2, EPI>(a, ceil_div(units, 4), s);
        }
        if (units <= 512 * 5) return launch_one<MA, 5, 2, 2, EPI>(a, ceil_div(units, 5), s);
        return launch_one<MA, 6, 2, 2, EPI>(a, ceil_div(units, 6), s);
    } else if constexpr (EPI == kEpiRope) {
        // from 16 rows on the activations weigh as much as a block's weights: two blocks share them where that
        // still leaves half the CUs a workgroup
        if (MA >= 2 && a.N >= 4096) return launch_one<MA, 2, MA <= 2 ? 8 : 4, 1, EPI>(a, a.N / 32, s);
        return launch_one<MA, 1, MA <= 2 ? 8 : 4, 2, EPI>(a, a.N / 16, s);
    } else if constexpr (EPI == kEpiPartial) {
        return launch_one<MA, 4, 4, 1, EPI>(a, ceil_div(a.N, 64), s, splits, a.ws);
    } else if constexpr (EPI == kEpiLogitsMax) {
        return launch_one<MA, 4, 2, 2, EPI>(a, ceil_div(a.N, 64), s);
    } else {
        const int units = ceil_div(a.N, 16);
        if (units <= 256) return launch_one<MA, 1, 8, 1, EPI>(a, units, s);
        if constexpr (MA <= 4) {  // 64 rows leave no LDS for a second workgroup of two blocks
            if (units <= 256 * 2 || (units > 256 * 4 && units <= 512 * 3))
                return launch_one<MA, 2, 4, 2, EPI>(a, ceil_div(units, 2), s);
        } else {
            if (units <= 256 * 2) return launch_one<MA, 2, 4, 1, EPI>(a, ceil_div(units, 2), s);
        }
        if (units <= 256 * 3) return launch_one<MA, 3, 4, 1, EPI>(a, ceil_div(units, 3), s);
        return launch_one<MA, 4, 2, 2, EPI>(a, ceil_div(units, 4), s);
    }
}

// More than 64 rows: groups of 64, with the blocks that gemm_skinny_groups found to fit one round.
template <int EPI>
hipError_t launch_groups(const GemmArgs& a, hipStream_t s) {
    switch (gemm_skinny_groups(a)) {
        case 1: return launch_one<8, 1, 4, 2, EPI, true>(a, ceil_div(a.N, 16), s);
        case 2: return launch_one<8, 2, 4, 1, EPI, true>(a, ceil_div(a.N, 32), s);
        case 4: return launch_one<8, 4, 4, 1, EPI, true>(a, ceil_div(a.N, 64), s);
        default: return hipErrorInvalidValue;
    }
}

template <int EPI>
hipError_t launch_epi(const GemmArgs& a, hipStream_t s, int splits = 1) {
    if (a.M <= 8) return launch_rows<1, EPI>(a, splits, s);
    if (a.M <= 16) return launch_rows<2, EPI>(a, splits, s);
    if (a.M <= 32) return launch_rows<4, EPI>(a, splits, s);
    if (a.M <= 64) return launch_rows<8, EPI>(a, splits, s);
    if constexpr (EPI == kEpiStore || EPI == kEpiAddF32 || EPI == kEpiRope) return launch_groups<EPI>(a, s);
    return hipErrorInvalidValue;
}

}  // namespace

// A deep K over a narrow N (the down projection): one workgroup per 16 columns would read all activations K deep
// in each of them (N = 1536, K = 8960: 12.5 us at 8 rows but 25 us at 64).  Blocks of 64 columns and a K range
// per workgroup instead, about one workgroup per CU; the sums go through memory to the reduction that also takes
// the residual and the RMSNorm (12.0 / 14.3 us with that reduction).  A shallow K stays unsplit: its workgroups
// would get less than eight slabs.
int gemm_skinny_splits(const GemmArgs& a) {
    if (a.epilogue != kEpiAddF32 || !a.ws || a.K < 4096 || a.M > 64) return 1;
    const int tiles = ceil_div(a.N, 64), slabs = a.K / 64;
    int splits = 256 / tiles;
    splits = splits < slabs / 8 ? splits : slabs / 8;
    splits = splits < 16 ? splits : 16;
    while (splits > 1 && (size_t)splits * a.M * a.N * sizeof(float) > a.ws_bytes) --splits;
    if (splits < 2) return 1;
    return ceil_div(slabs, ceil_div(slabs, splits));  // every split has slabs of its own
}

// Where the tiles of gemm.hip are the faster ones, up to 64 rows.  All figures us with the weights from HBM, tiles
// against this kernel.
bool gemm_skinny_takes(const GemmArgs& a, bool tiles_split_k) {
    const bool few = a.M <= 16, some = a.M <= 32;
    // A K split that goes through memory: from 33 rows on the tiles feed a deep K better (N = 3584, K = 18944, 32 / 64
    // rows: 30.6, 29.8 / 31.7, 34.6; N = 4096, K = 12288, 64 rows: 27.2, 26.5; N = 8192, K = 28672, 32 rows: 86, 91;
    // N = K = 6144, 64 rows: 22.6, 24.2).
    if (gemm_skinny_splits(a) > 1) return few || a.K <= (some ? 20480 : a.N <= 4096 ? 12288 : 4096);
    // Tiles that split K over the CUs against workgroups that walk all of it (store, N = 1536: 64 rows, K = 4096 13.2,
    // 12.6, K = 8192 17.3, 21.4; 24 rows, K = 8192 14.8, 14.1, K = 16384 18.1, 24.9; 8 rows, K = 16384 18.0, 17.2).
    // A QKV projection whose tiles split K rotates in the reduction, one workgroup per row, which costs more
    // (a decode step of four layers, K = 5120, N = 7168, 48 rows 922, 808; K = 8192, N = 10240, 24 rows 1585, 1480, 64 rows
    // 1695, 1764).
    if (a.rope && tiles_split_k) return some || a.K <= 6144;
    if (tiles_split_k && a.K > (few ? 16384 : some ? 6144 : 4096)) return false;
    if (a.epilogue == kEpiSwiglu) {
        // F = 14336, K = 3584: 8 rows 37.6, 37.1; 32 rows 37.9, 41.2; F = 22016: 64 rows 71.5, 66.4; F = 28672: 8 rows
        // 72.8, 73.6; 64 rows 80.9, 91.4.
        const int F = a.N / 2;
        return F <= 12288 || (F <= 16384 ? few : F <= 24576);
    }
    if (a.N <= 8192) return true;
    // N = 16384: 32 rows, K = 512 6.3, 7.3 (accumulating); 64 rows, K = 1536 13.2, 14.1; K = 3584 34.7, 26.1
    if (a.N <= 16384) return (a.N <= 12288 ? some : few) || a.K >= 2048;
    // N = 32768, K = 3584: 32 rows 38.3, 35.7; 64 rows 38.3, 39.1; K = 6144, 64 rows 76, 85.  A vocabulary (N = 151936, 64
    // rows): K = 1536 117, 114; K = 3584 227, 244.  N = 24000, 20 rows: K = 128 4.6, 5.1; K = 256 the same.
    return few || (some && a.K >= 256) || (a.epilogue == kEpiStoreF32 && a.N > 24576 && a.K < 3072);
}

// Up to 32 rows: RMSNorm in a launch of its own is 3 to 5 us of a layer's 45 (1.5B shape, 8 rows) to 125 (7B, 16 rows); taken
// apart between the O and the gate/up projection it costs neither of them anything that shows.  One 16-column block
// per workgroup, at most 256 of them (the consumer's lanes hold four a row).
bool gemm_skinny_splits_norm(const GemmArgs& a) {
    return a.epilogue == kEpiAddF32 && a.norm_split && a.norm_out && a.M <= 32 && a.N % 16 == 0 && a.N <= 4096 && gemm_skinny_splits(a) == 1 && a.ldc % 4 == 0 &&
           ((uintptr_t)a.C & 15) == 0 && ((uintptr_t)a.norm_out & 7) == 0 && ((uintptr_t)a.norm_gain & 7) == 0;
}

hipError_t gemm_skinny_load_kernels() {
    hipFuncAttributes attr;
    return hipFuncGetAttributes(&attr, (const void*)gemm_skinny_kernel<1, 1, 8, 4, kEpiStore, false, false>);
}

hipError_t launch_gemm_skinny(const GemmArgs& a, int epi, int splits, hipStream_t s) {
    if (splits > 1) return launch_epi<kEpiPartial>(a, s, splits);
    switch (epi) {
        case kEpiStore: return launch_epi<kEpiStore>(a, s);
        case kEpiStoreF32: return launch_epi<kEpiStoreF32>(a, s);
        case kEpiAddF32: return launch_epi<kEpiAddF32>(a, s);
        case kEpiSwiglu: return launch_epi<kEpiSwiglu>(a, s);
        case kEpiRope: return launch_epi<kEpiRope>(a, s);
        case kEpiLogitsMax: return launch_epi<kEpiLogitsMax>(a, s);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace rpo
