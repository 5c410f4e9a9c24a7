// a1 for layers whose blocks read (nearly) whole feature rows of 4097 to 16384 columns, with any weights: whole rows
// side by side in LDS, just as they lie in memory.
//
// Such a pattern makes every workgroup stage the row, whatever neurons it owns, and what a CU can pull out of L2 is the
// scarce resource: 64 KB per row at 16384 neurons.  So a workgroup owns as many neurons as the register file holds --
// two per lane with their 32 weights and 16-bit column offsets (96 registers), four with one weight for the layer --
// and the rows go from memory straight into LDS (global_load_lds, 16 bytes per lane) without passing through
// registers, of which none are left, or through the LDS write path: 16.5 TB/s from L2 into the CUs for eight
// workgroups that share their rows, against 11.4 through registers (64-KB rows, 256 workgroups).  The price is that
// LDS holds plain rows, so a connection is one ds_read_b32 per row (2.3 clocks per wave free of conflicts, against
// 2.8 for the two rows of an 8-byte entry).  A tile is as many rows as fit twice: the next one lands while this one
// is read, and a step has one barrier.
//
// gfx950 serves a 4-byte read half a wave at a time from 32 banks (measured with the probe that gave the 8-byte
// rule: lanes l and l + 32 never collide, columns that are equal mod 32 do), so the set-up orders the connections of
// 32 neighbouring neurons like row2_pack_kernel, with bank = column mod 32 (flat_pack_kernel).  Every neuron's 32
// products are one chain of fused multiply-adds in that order, bias last.
#pragma once

namespace spdnn {

constexpr int kFlatCols = 16384;  // columns a row may have
constexpr int kFlatMisc = 1024;   // bytes of bookkeeping in front of the tiles
// Rows per tile and the bytes between them: whole kilobytes (what one load instruction of a wave fills), two tiles and the
// bookkeeping within 160 KB, the last row within the 16-bit immediate offset of a read.
SPDNN_HD inline int flat_rows(int N) { return N <= 4864 ? 4 : N <= 6656 ? 3 : N <= 9984 ? 2 : 1; }
SPDNN_HD constexpr int flat_stride(int rows) { return rows == 4 ? 4864 * 4 : rows == 3 ? 6656 * 4 : rows == 2 ? 9984 * 4 : 16384 * 4; }
SPDNN_HD inline int flat_lds_bytes(int rows) { return kFlatMisc + 2 * rows * flat_stride(rows); }

// Sixteen connections of one neuron on R rows: acc[r] += row r[column i] * w_i, i = 0..15 in that order.  c0..c7 hold the
// connections' byte offsets in a row, two to a register; an SDWA add makes a half an address in the tile at `base`; reads
// run G connections ahead (v118..v125).
#define SPDNN_FLAT_READ(I, C, H)                                                                                          \
    "v_add_u32_sdwa v[126+" I "%%2], %[base], %[" C "] dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:WORD_" H "\n\t" \
    ".set spdnn_r, 0\n\t"                                                                                                 \
    ".rept %[R]\n\t"                                                                                                      \
    "ds_read_b32 v[118+(" I "%%%[G])*%[R]+spdnn_r], v[126+" I "%%2] offset:%[S]*spdnn_r\n\t"                               \
    ".set spdnn_r, spdnn_r+1\n\t"                                                                                         \
    ".endr\n\t"
#define SPDNN_FLAT_STEP(I, W)                                   \
    ".if " I "+%[G] <= 16\n\t"                                  \
    "s_waitcnt lgkmcnt((%[G]-1)*%[R])\n\t"                      \
    ".else\n\t"                                                 \
    "s_waitcnt lgkmcnt((15-" I ")*%[R])\n\t"                    \
    ".endif\n\t"                                                \
    "v_fmac_f32 %[a0], " W ", v[118+(" I "%%%[G])*%[R]]\n\t"    \
    ".if %[R] > 1\n\t"                                          \
    "v_fmac_f32 %[a1], " W ", v[119+(" I "%%%[G])*%[R]]\n\t"    \
    ".endif\n\t"                                                \
    ".if %[R] > 2\n\t"                                          \
    "v_fmac_f32 %[a2], " W ", v[120+(" I "%%%[G])*%[R]]\n\t"    \
    ".endif\n\t"                                                \
    ".if %[R] > 3\n\t"                                          \
    "v_fmac_f32 %[a3], " W ", v[121+(" I "%%%[G])*%[R]]\n\t"    \
    ".endif\n\t"
#define SPDNN_FLAT_ASM_W8 \
    SPDNN_FLAT_READ("0", "c0", "0") SPDNN_FLAT_READ("1", "c0", "1") SPDNN_FLAT_READ("2", "c1", "0") SPDNN_FLAT_READ("3", "c1", "1") SPDNN_FLAT_READ("4", "c2", "0") SPDNN_FLAT_READ("5", "c2", "1") SPDNN_FLAT_READ("6", "c3", "0") SPDNN_FLAT_READ("7", "c3", "1") \
    SPDNN_FLAT_STEP("0", "%[w0]") SPDNN_FLAT_READ("8", "c4", "0") SPDNN_FLAT_STEP("1", "%[w1]") SPDNN_FLAT_READ("9", "c4", "1") \
    SPDNN_FLAT_STEP("2", "%[w2]") SPDNN_FLAT_READ("10", "c5", "0") SPDNN_FLAT_STEP("3", "%[w3]") SPDNN_FLAT_READ("11", "c5", "1") \
    SPDNN_FLAT_STEP("4", "%[w4]") SPDNN_FLAT_READ("12", "c6", "0") SPDNN_FLAT_STEP("5", "%[w5]") SPDNN_FLAT_READ("13", "c6", "1") \
    SPDNN_FLAT_STEP("6", "%[w6]") SPDNN_FLAT_READ("14", "c7", "0") SPDNN_FLAT_STEP("7", "%[w7]") SPDNN_FLAT_READ("15", "c7", "1") \
    SPDNN_FLAT_STEP("8", "%[w8]") SPDNN_FLAT_STEP("9", "%[w9]") \
    SPDNN_FLAT_STEP("10", "%[w10]") SPDNN_FLAT_STEP("11", "%[w11]") \
    SPDNN_FLAT_STEP("12", "%[w12]") SPDNN_FLAT_STEP("13", "%[w13]") \
    SPDNN_FLAT_STEP("14", "%[w14]") SPDNN_FLAT_STEP("15", "%[w15]")
#define SPDNN_FLAT_ASM_U8 \
    SPDNN_FLAT_READ("0", "c0", "0") SPDNN_FLAT_READ("1", "c0", "1") SPDNN_FLAT_READ("2", "c1", "0") SPDNN_FLAT_READ("3", "c1", "1") SPDNN_FLAT_READ("4", "c2", "0") SPDNN_FLAT_READ("5", "c2", "1") SPDNN_FLAT_READ("6", "c3", "0") SPDNN_FLAT_READ("7", "c3", "1") \
    SPDNN_FLAT_STEP("0", "%[w]") SPDNN_FLAT_READ("8", "c4", "0") SPDNN_FLAT_STEP("1", "%[w]") SPDNN_FLAT_READ("9", "c4", "1") \
    SPDNN_FLAT_STEP("2", "%[w]") SPDNN_FLAT_READ("10", "c5", "0") SPDNN_FLAT_STEP("3", "%[w]") SPDNN_FLAT_READ("11", "c5", "1") \
    SPDNN_FLAT_STEP("4", "%[w]") SPDNN_FLAT_READ("12", "c6", "0") SPDNN_FLAT_STEP("5", "%[w]") SPDNN_FLAT_READ("13", "c6", "1") \
    SPDNN_FLAT_STEP("6", "%[w]") SPDNN_FLAT_READ("14", "c7", "0") SPDNN_FLAT_STEP("7", "%[w]") SPDNN_FLAT_READ("15", "c7", "1") \
    SPDNN_FLAT_STEP("8", "%[w]") SPDNN_FLAT_STEP("9", "%[w]") \
    SPDNN_FLAT_STEP("10", "%[w]") SPDNN_FLAT_STEP("11", "%[w]") \
    SPDNN_FLAT_STEP("12", "%[w]") SPDNN_FLAT_STEP("13", "%[w]") \
    SPDNN_FLAT_STEP("14", "%[w]") SPDNN_FLAT_STEP("15", "%[w]")
#define SPDNN_FLAT_ASM_W4 \
    SPDNN_FLAT_READ("0", "c0", "0") SPDNN_FLAT_READ("1", "c0", "1") SPDNN_FLAT_READ("2", "c1", "0") SPDNN_FLAT_READ("3", "c1", "1") \
    SPDNN_FLAT_STEP("0", "%[w0]") SPDNN_FLAT_READ("4", "c2", "0") SPDNN_FLAT_STEP("1", "%[w1]") SPDNN_FLAT_READ("5", "c2", "1") \
    SPDNN_FLAT_STEP("2", "%[w2]") SPDNN_FLAT_READ("6", "c3", "0") SPDNN_FLAT_STEP("3", "%[w3]") SPDNN_FLAT_READ("7", "c3", "1") \
    SPDNN_FLAT_STEP("4", "%[w4]") SPDNN_FLAT_READ("8", "c4", "0") SPDNN_FLAT_STEP("5", "%[w5]") SPDNN_FLAT_READ("9", "c4", "1") \
    SPDNN_FLAT_STEP("6", "%[w6]") SPDNN_FLAT_READ("10", "c5", "0") SPDNN_FLAT_STEP("7", "%[w7]") SPDNN_FLAT_READ("11", "c5", "1") \
    SPDNN_FLAT_STEP("8", "%[w8]") SPDNN_FLAT_READ("12", "c6", "0") SPDNN_FLAT_STEP("9", "%[w9]") SPDNN_FLAT_READ("13", "c6", "1") \
    SPDNN_FLAT_STEP("10", "%[w10]") SPDNN_FLAT_READ("14", "c7", "0") SPDNN_FLAT_STEP("11", "%[w11]") SPDNN_FLAT_READ("15", "c7", "1") \
    SPDNN_FLAT_STEP("12", "%[w12]") SPDNN_FLAT_STEP("13", "%[w13]") \
    SPDNN_FLAT_STEP("14", "%[w14]") SPDNN_FLAT_STEP("15", "%[w15]")
#define SPDNN_FLAT_ASM_U4 \
    SPDNN_FLAT_READ("0", "c0", "0") SPDNN_FLAT_READ("1", "c0", "1") SPDNN_FLAT_READ("2", "c1", "0") SPDNN_FLAT_READ("3", "c1", "1") \
    SPDNN_FLAT_STEP("0", "%[w]") SPDNN_FLAT_READ("4", "c2", "0") SPDNN_FLAT_STEP("1", "%[w]") SPDNN_FLAT_READ("5", "c2", "1") \
    SPDNN_FLAT_STEP("2", "%[w]") SPDNN_FLAT_READ("6", "c3", "0") SPDNN_FLAT_STEP("3", "%[w]") SPDNN_FLAT_READ("7", "c3", "1") \
    SPDNN_FLAT_STEP("4", "%[w]") SPDNN_FLAT_READ("8", "c4", "0") SPDNN_FLAT_STEP("5", "%[w]") SPDNN_FLAT_READ("9", "c4", "1") \
    SPDNN_FLAT_STEP("6", "%[w]") SPDNN_FLAT_READ("10", "c5", "0") SPDNN_FLAT_STEP("7", "%[w]") SPDNN_FLAT_READ("11", "c5", "1") \
    SPDNN_FLAT_STEP("8", "%[w]") SPDNN_FLAT_READ("12", "c6", "0") SPDNN_FLAT_STEP("9", "%[w]") SPDNN_FLAT_READ("13", "c6", "1") \
    SPDNN_FLAT_STEP("10", "%[w]") SPDNN_FLAT_READ("14", "c7", "0") SPDNN_FLAT_STEP("11", "%[w]") SPDNN_FLAT_READ("15", "c7", "1") \
    SPDNN_FLAT_STEP("12", "%[w]") SPDNN_FLAT_STEP("13", "%[w]") \
    SPDNN_FLAT_STEP("14", "%[w]") SPDNN_FLAT_STEP("15", "%[w]")
#define SPDNN_FLAT_ASM_W2 \
    SPDNN_FLAT_READ("0", "c0", "0") SPDNN_FLAT_READ("1", "c0", "1") \
    SPDNN_FLAT_STEP("0", "%[w0]") SPDNN_FLAT_READ("2", "c1", "0") SPDNN_FLAT_STEP("1", "%[w1]") SPDNN_FLAT_READ("3", "c1", "1") \
    SPDNN_FLAT_STEP("2", "%[w2]") SPDNN_FLAT_READ("4", "c2", "0") SPDNN_FLAT_STEP("3", "%[w3]") SPDNN_FLAT_READ("5", "c2", "1") \
    SPDNN_FLAT_STEP("4", "%[w4]") SPDNN_FLAT_READ("6", "c3", "0") SPDNN_FLAT_STEP("5", "%[w5]") SPDNN_FLAT_READ("7", "c3", "1") \
    SPDNN_FLAT_STEP("6", "%[w6]") SPDNN_FLAT_READ("8", "c4", "0") SPDNN_FLAT_STEP("7", "%[w7]") SPDNN_FLAT_READ("9", "c4", "1") \
    SPDNN_FLAT_STEP("8", "%[w8]") SPDNN_FLAT_READ("10", "c5", "0") SPDNN_FLAT_STEP("9", "%[w9]") SPDNN_FLAT_READ("11", "c5", "1") \
    SPDNN_FLAT_STEP("10", "%[w10]") SPDNN_FLAT_READ("12", "c6", "0") SPDNN_FLAT_STEP("11", "%[w11]") SPDNN_FLAT_READ("13", "c6", "1") \
    SPDNN_FLAT_STEP("12", "%[w12]") SPDNN_FLAT_READ("14", "c7", "0") SPDNN_FLAT_STEP("13", "%[w13]") SPDNN_FLAT_READ("15", "c7", "1") \
    SPDNN_FLAT_STEP("14", "%[w14]") SPDNN_FLAT_STEP("15", "%[w15]")
#define SPDNN_FLAT_ASM_U2 \
    SPDNN_FLAT_READ("0", "c0", "0") SPDNN_FLAT_READ("1", "c0", "1") \
    SPDNN_FLAT_STEP("0", "%[w]") SPDNN_FLAT_READ("2", "c1", "0") SPDNN_FLAT_STEP("1", "%[w]") SPDNN_FLAT_READ("3", "c1", "1") \
    SPDNN_FLAT_STEP("2", "%[w]") SPDNN_FLAT_READ("4", "c2", "0") SPDNN_FLAT_STEP("3", "%[w]") SPDNN_FLAT_READ("5", "c2", "1") \
    SPDNN_FLAT_STEP("4", "%[w]") SPDNN_FLAT_READ("6", "c3", "0") SPDNN_FLAT_STEP("5", "%[w]") SPDNN_FLAT_READ("7", "c3", "1") \
    SPDNN_FLAT_STEP("6", "%[w]") SPDNN_FLAT_READ("8", "c4", "0") SPDNN_FLAT_STEP("7", "%[w]") SPDNN_FLAT_READ("9", "c4", "1") \
    SPDNN_FLAT_STEP("8", "%[w]") SPDNN_FLAT_READ("10", "c5", "0") SPDNN_FLAT_STEP("9", "%[w]") SPDNN_FLAT_READ("11", "c5", "1") \
    SPDNN_FLAT_STEP("10", "%[w]") SPDNN_FLAT_READ("12", "c6", "0") SPDNN_FLAT_STEP("11", "%[w]") SPDNN_FLAT_READ("13", "c6", "1") \
    SPDNN_FLAT_STEP("12", "%[w]") SPDNN_FLAT_READ("14", "c7", "0") SPDNN_FLAT_STEP("13", "%[w]") SPDNN_FLAT_READ("15", "c7", "1") \
    SPDNN_FLAT_STEP("14", "%[w]") SPDNN_FLAT_STEP("15", "%[w]")
#define SPDNN_FLAT_IO                                                                                                   \
    : [a0] "+v"(acc[0]), [a1] "+v"(acc[1]), [a2] "+v"(acc[2]), [a3] "+v"(acc[3])                                          \
    : [c0] "v"(c[0]), [c1] "v"(c[1]), [c2] "v"(c[2]), [c3] "v"(c[3]), [c4] "v"(c[4]), [c5] "v"(c[5]), [c6] "v"(c[6]),       \
      [c7] "v"(c[7]), [base] "s"(base), [R] "n"(R), [G] "n"(G), [S] "n"(flat_stride(R))
#define SPDNN_FLAT_WEIGHTS                                                                                              \
    , [w0] "v"(w[0]), [w1] "v"(w[1]), [w2] "v"(w[2]), [w3] "v"(w[3]), [w4] "v"(w[4]), [w5] "v"(w[5]), [w6] "v"(w[6]),       \
        [w7] "v"(w[7]), [w8] "v"(w[8]), [w9] "v"(w[9]), [w10] "v"(w[10]), [w11] "v"(w[11]), [w12] "v"(w[12]),               \
        [w13] "v"(w[13]), [w14] "v"(w[14]), [w15] "v"(w[15])
#define SPDNN_FLAT_CLOBBER : "v118", "v119", "v120", "v121", "v122", "v123", "v124", "v125", "v126", "v127", "memory"
#define SPDNN_FLAT_CASE(Q)                                                                      \
    if constexpr (G == Q) {                                                                     \
        if constexpr (UNI)                                                                      \
            asm volatile(SPDNN_FLAT_ASM_U##Q SPDNN_FLAT_IO, [w] "s"(wu) SPDNN_FLAT_CLOBBER);     \
        else                                                                                    \
            asm volatile(SPDNN_FLAT_ASM_W##Q SPDNN_FLAT_IO SPDNN_FLAT_WEIGHTS SPDNN_FLAT_CLOBBER); \
    }
template <int R, bool UNI>
__device__ __forceinline__ void fma_flat16(float (&acc)[4], const uint32_t* c, const float* w, float wu, uint32_t base) {
    constexpr int G = R == 1 ? 8 : R == 2 ? 4 : 2;
    SPDNN_FLAT_CASE(8)
    SPDNN_FLAT_CASE(4)
    SPDNN_FLAT_CASE(2)
}

// A launch: ncb units of at most `gpu` groups of 64 neurons times Q chunks of tiles of R rows; wave w of a workgroup owns
// the unit's groups w, 16 + w, ... (at most SLOTS).
template <int R, bool UNI>
__global__ __launch_bounds__(kBlk) void fused_flat_kernel(const float* __restrict__ Yin, float* __restrict__ Yout,
                                                          uint8_t* __restrict__ flags, RowLists rl, LayerWeights lw,
                                                          const float* __restrict__ bias, int N, int ncb, int G, int Q, int gpu,
                                                          float wuni) {
    constexpr int SLOTS = UNI ? 4 : 2;
    constexpr uint32_t S = flat_stride(R);
    extern __shared__ __align__(16) char flat_lds[];  // all dynamic: addresses are counted from the start of the LDS
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    WorkItem wi;
    int* red = reinterpret_cast<int*>(flat_lds);
    if (!derive_work(rl, ncb, G, Q, wi, R, red, red + 32)) return;
    const int A = wi.A, g0 = wi.g0, T = wi.g1 - wi.g0;

    // my neurons and their connections
    const int first = wi.cb * gpu;
    const int ng = min(gpu, ((N + 63) >> 6) - first);  // the unit's groups
    const int nslots = wave < ng ? (ng - wave + 15) >> 4 : 0;
    uint32_t code[SLOTS][kNnz / 2];
    float wv[UNI ? 1 : SLOTS][kNnz];
    float bj[SLOTS];
#pragma unroll
    for (int s = 0; s < SLOTS; ++s) {
        const int g = s < nslots ? first + 16 * s + wave : first;  // (a group that exists, for waves with fewer)
        const int b = g >> 4, ln = (g & 15) * 64 + lane;
        const uint4* q = reinterpret_cast<const uint4*>(lw.rel + rel_entry(b, 0, ln));
#pragma unroll
        for (int c = 0; c < kNnz / 8; ++c) {
            const uint4 v = q[c * kBlk];
            code[s][4 * c] = v.x;
            code[s][4 * c + 1] = v.y;
            code[s][4 * c + 2] = v.z;
            code[s][4 * c + 3] = v.w;
        }
        if constexpr (!UNI) load_weights(wv[s], lw.val, b, ln);
        const int j = 64 * g + lane;
        bj[s] = j < N ? bias[j] : 0.0f;
    }

    ListWindow rows_of(rl.cat, g0 * R, min(A, wi.g1 * R), wi.identity);
    const int nload = (N + 255) >> 8;            // kilobytes of a row
    const uint32_t row_end = 4u * N - 16u;       // the last lanes of a row's last kilobyte read its end again
    // tile t into buffer p: wave w takes the row's kilobytes w, 16 + w, ...
    auto load_tile = [&](int t, int p) {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int row = rows_of.get1(min((g0 + t) * R + r, rows_of.end - 1));
            const char* src = reinterpret_cast<const char*>(Yin + (size_t)row * N);
            for (int k = wave; k < nload; k += 16)
                __builtin_amdgcn_global_load_lds(
                    (const __attribute__((address_space(1))) void*)(src + min((uint32_t)k * 1024u + 16u * lane, row_end)),
                    (__attribute__((address_space(3))) void*)(flat_lds + kFlatMisc + (p * R + r) * S + k * 1024), 16, 0, 0);
        }
    };
    {  // waves of one SIMD take turns rather than meet at the LDS all at once (see fused_layer_kernel)
        const int pw = __builtin_amdgcn_readfirstlane(3 - ((threadIdx.x >> 8) & 3));
        if (pw == 1) __builtin_amdgcn_s_setprio(1);
        else if (pw == 2) __builtin_amdgcn_s_setprio(2);
        else if (pw == 3) __builtin_amdgcn_s_setprio(3);
    }
    __syncthreads();  // the lists' scratch in front of the tiles is not touched again; rows_of has been read
    load_tile(0, 0);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    for (int t = 0; t < T; ++t) {
        if (t + 1 < T) load_tile(t + 1, (t + 1) & 1);
        const uint32_t base = kFlatMisc + (t & 1) * R * S;
        const int row0 = (g0 + t) * R;
        unsigned pos = 0;
#pragma unroll
        for (int s = 0; s < SLOTS; ++s) {
            if (s < nslots) {
                float acc[4] = {0.f, 0.f, 0.f, 0.f};
                fma_flat16<R, UNI>(acc, &code[s][0], UNI ? nullptr : &wv[UNI ? 0 : s][0], wuni, base);
                fma_flat16<R, UNI>(acc, &code[s][8], UNI ? nullptr : &wv[UNI ? 0 : s][16], wuni, base);
                const int j = 64 * (first + 16 * s + wave) + lane;
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    const float y = j < N ? fminf(fmaxf(acc[r] + bj[s], 0.0f), kClip) : 0.0f;
                    if (__builtin_amdgcn_ballot_w64(y > 0.0f) != 0ull) pos |= 1u << r;
                    if (j < N && row0 + r < A) __builtin_nontemporal_store(y, Yout + (size_t)(row0 + r) * N + j);
                }
            }
        }
        if (lane < R && row0 + lane < A && ((pos >> lane) & 1u)) flags[row0 + lane] = 1;  // lane r speaks for row r of the tile
        // The next tile has landed when at most the stores behind its loads are still under way.
        if (nslots == SLOTS && row0 + R <= A) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(SLOTS * R) : "memory");
        else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
    }
}

// Set-up: the connections of 32 neighbouring neurons ordered for the 32 banks, one wave per group, written as
// LayerWeights::rel (byte offsets in a row) and ::val.
__global__ __launch_bounds__(kRow2PackThreads) void flat_pack_kernel(const int32_t* __restrict__ idx, const float* __restrict__ val,
                                                                     int N, uint16_t* __restrict__ rel, float* __restrict__ wval) {
    __shared__ Pack32Scratch S;
    const int lane = threadIdx.x, l = lane & 31;
    const int j = blockIdx.x * kGroup32 + l;
    const bool exists = j < N;
    const int b = j / kBlk, ln = j - b * kBlk;
    const int32_t* mine = idx + (size_t)min(j, N - 1) * kNnz;
    auto column = [&](int k) -> int {  // out-of-range columns were reported; keep them harmless
        const int c = mine[k];
        return c < 0 || c >= N ? 0 : c;
    };
    if (!exists && lane < 32)
        for (int k = 0; k < kNnz; ++k) {
            rel[rel_entry(b, k, ln)] = 0;
            wval[val_entry(b, k, ln)] = 0.0f;
        }
    order32_wave(S, exists, [&](int k) { return (uint32_t)column(k) & 31u; },
                 [&](int step, int k) {
                     rel[rel_entry(b, step, ln)] = (uint16_t)(4 * column(k));
                     wval[val_entry(b, step, ln)] = val[(size_t)j * kNnz + k];
                 });
}

}  // namespace spdnn
