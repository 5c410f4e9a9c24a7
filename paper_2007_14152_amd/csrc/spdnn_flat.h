// a1 for layers whose blocks read more than one LDS stage of feature rows of 4097 to 16384 columns, with any weights: whole
// rows side by side in LDS, just as they lie in memory.
//
// A pattern that reads the whole row makes every workgroup stage the row, whatever neurons it owns, and what a CU can pull out of L2 is the
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
//
// What bounds it: the LDS reads, 3.1 clocks each with the conflicts the ordering leaves, and next to them the rows'
// way into LDS.  16384 neurons with weights of their own, 6 layers, 8000 rows: 5.42 -> 2.75 ms (one neuron per lane and
// the row in four stages before, so every row went to 16 workgroups).  Blocks that read less take it too: 4 layers on
// 8000 rows, windows -> whole rows, weights of their own: 16384 neurons, 5000 columns 2.69 -> 2.07 ms, 8192 neurons, 4300
// columns 1.34 -> 1.12, 10240 neurons, 5000 columns 1.78 -> 1.30 (one weight and windows of two stages: see create_impl).
#pragma once

namespace spdnn {

constexpr int kFlatCols = 16384;  // columns a row may have
constexpr int kFlatMisc = 1024;   // bytes of bookkeeping in front of the tiles
// Rows per tile and the bytes between them: whole kilobytes (what one load instruction of a wave fills), two tiles and the
// bookkeeping within 160 KB, the last row within the 16-bit immediate offset of a read.
SPDNN_HD inline int flat_rows(int N) { return N <= 4864 ? 4 : N <= 6656 ? 3 : N <= 9984 ? 2 : 1; }
SPDNN_HD constexpr int flat_stride(int rows) { return rows == 4 ? 4864 * 4 : rows == 3 ? 6656 * 4 : rows == 2 ? 9984 * 4 : 16384 * 4; }
SPDNN_HD inline int flat_lds_bytes(int rows) { return kFlatMisc + 2 * rows * flat_stride(rows); }

// All connections of a lane's NS neurons on R rows, one pipeline of reads from the first to the last: acc[s * R + r] +=
// row r[column] * weight over neuron s's 32 connections, in order.  Everything sits in fixed registers, so that the
// assembler's own loop can number it: byte offsets in a row in v[16..], two to a register (an SDWA add makes a half an
// address in the tile at `base`), weights in v[48..111], sums in v[8..15] -- with one weight per layer, of four neurons,
// offsets in v[16..79] and sums in v[80..95] -- and reads, G connections ahead, from v112 on.  (As blocks of 16
// connections with a drained pipeline between them a layer of 16384 neurons on 7000 rows took 0.52 ms.)
#define SPDNN_FLAT_READ(K)                                                                                                 \
    ".if ((" K ")&1)==0\n\t"                                                                                               \
    "v_add_u32_sdwa v[126+((" K ")&1)], %[base], v[16+(" K ")/2] dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:WORD_0\n\t" \
    ".else\n\t"                                                                                                            \
    "v_add_u32_sdwa v[126+((" K ")&1)], %[base], v[16+(" K ")/2] dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:WORD_1\n\t" \
    ".endif\n\t"                                                                                                           \
    ".set spdnn_r, 0\n\t"                                                                                                  \
    ".rept %[R]\n\t"                                                                                                       \
    "ds_read_b32 v[112+((" K ")%%%[G])*%[R]+spdnn_r], v[126+((" K ")&1)] offset:%[S]*spdnn_r\n\t"                           \
    ".set spdnn_r, spdnn_r+1\n\t"                                                                                          \
    ".endr\n\t"
#define SPDNN_FLAT_ASM(ACC, W)                                                                                             \
    ".set spdnn_k, 0\n\t"                                                                                                  \
    ".rept %[G]\n\t" SPDNN_FLAT_READ("spdnn_k") ".set spdnn_k, spdnn_k+1\n\t"                                               \
    ".endr\n\t"                                                                                                            \
    ".set spdnn_k, 0\n\t"                                                                                                  \
    ".rept 32*%[NS]\n\t"                                                                                                   \
    ".if (spdnn_k%%(8*%[NS]))==0\n\t"                                                                                      \
    "s_setprio 3-spdnn_k/(8*%[NS])\n\t" /* see set_wave_prio */                                                           \
    ".endif\n\t"                                                                                                         \
    ".if spdnn_k+%[G] <= 32*%[NS]\n\t"                                                                                     \
    "s_waitcnt lgkmcnt((%[G]-1)*%[R])\n\t"                                                                                 \
    ".else\n\t"                                                                                                            \
    "s_waitcnt lgkmcnt((32*%[NS]-1-spdnn_k)*%[R])\n\t"                                                                     \
    ".endif\n\t"                                                                                                           \
    ".set spdnn_r, 0\n\t"                                                                                                  \
    ".rept %[R]\n\t"                                                                                                       \
    "v_fmac_f32 v[" ACC "+(spdnn_k/32)*%[R]+spdnn_r], " W ", v[112+(spdnn_k%%%[G])*%[R]+spdnn_r]\n\t"                       \
    ".set spdnn_r, spdnn_r+1\n\t"                                                                                          \
    ".endr\n\t"                                                                                                            \
    ".if spdnn_k+%[G] < 32*%[NS]\n\t" SPDNN_FLAT_READ("spdnn_k+%[G]") ".endif\n\t"                                          \
    ".set spdnn_k, spdnn_k+1\n\t"                                                                                          \
    ".endr\n\t"
#define SPDNN_FLAT_CLOBBER                                                                                                 \
    "v112", "v113", "v114", "v115", "v116", "v117", "v118", "v119", "v120", "v121", "v122", "v123", "v126", "v127", "memory"
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x32 __attribute__((ext_vector_type(32)));
constexpr int flat_ahead(int R) { return 12 / R; }
#define SPDNN_FLAT_W(SUMS, REGS)                                                                                           \
    template <int R, int NS>                                                                                               \
    __device__ __forceinline__ void fma_flat(SUMS& acc, const u32x16 (&c)[2], const f32x32 (&w)[2], uint32_t base) {        \
        asm volatile(SPDNN_FLAT_ASM("8", "v[48+spdnn_k]")                                                                  \
                     : "+{" REGS "}"(acc)                                                                                  \
                     : "{v[16:31]}"(c[0]), "{v[32:47]}"(c[1]), "{v[48:79]}"(w[0]), "{v[80:111]}"(w[1]), [base] "s"(base),   \
                       [R] "n"(R), [G] "n"(flat_ahead(R)), [S] "n"(flat_stride(R)), [NS] "n"(NS)                            \
                     : SPDNN_FLAT_CLOBBER);                                                                                \
    }
SPDNN_FLAT_W(f32x2, "v[8:9]")    // sums of two neurons on one row,
SPDNN_FLAT_W(f32x4, "v[8:11]")   // on two,
SPDNN_FLAT_W(f32x8, "v[8:15]")   // on three or four
template <int R, int NS>
__device__ __forceinline__ void fma_flat(f32x16& acc, const u32x16 (&c)[4], float wu, uint32_t base) {
    asm volatile(SPDNN_FLAT_ASM("80", "%[w]")
                 : "+{v[80:95]}"(acc)
                 : "{v[16:31]}"(c[0]), "{v[32:47]}"(c[1]), "{v[48:63]}"(c[2]), "{v[64:79]}"(c[3]), [w] "s"(wu), [base] "s"(base),
                   [R] "n"(R), [G] "n"(flat_ahead(R)), [S] "n"(flat_stride(R)), [NS] "n"(NS)
                 : SPDNN_FLAT_CLOBBER);
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
    u32x16 code[SLOTS];
    f32x32 wv[2];  // (not with one weight per layer)
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
        if constexpr (!UNI) {
            const f32x4* p = reinterpret_cast<const f32x4*>(lw.val + val_entry(b, 0, ln));
#pragma unroll
            for (int c = 0; c < kNnz / 4; ++c) {
                const f32x4 v = p[c * kBlk];
                wv[s][4 * c] = v.x;
                wv[s][4 * c + 1] = v.y;
                wv[s][4 * c + 2] = v.z;
                wv[s][4 * c + 3] = v.w;
            }
        }
        const int j = 64 * g + lane;
        bj[s] = j < N ? bias[j] : 0.0f;
    }

    ListWindow<(R > 1)> rows_of(rl.cat, g0 * R, min(A, wi.g1 * R), wi.identity);
    const int nload = (N + 255) >> 8;            // kilobytes of a row
    const uint32_t row_end = 4u * N - 16u;       // the last lanes of a row's last kilobyte read its end again
    // Tile t into buffer p: wave w takes the row's kilobytes w, 16 + w, ...  The rows' loads are under way together: a slot's
    // number comes from a register that ListWindow has waited for where it filled it.  (With that wait left to the use, every
    // row of a tile but the first stood behind the one before: 6 layers with weights of their own, 8000 rows, 8000 neurons, two
    // rows to a tile, 1.47 -> 1.29 ms; 6000, three, 1.34 -> 1.17; one weight, 6144 neurons, 0.83 -> 0.75.  One row to a tile has
    // nothing to gain from it and lost 1 %: 10 layers of 16384 neurons, 1187 rows 816 -> 823 us.)
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
    __syncthreads();  // the lists' scratch in front of the tiles is not touched again; rows_of has been read
    load_tile(0, 0);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    for (int t = 0; t < T; ++t) {
        if (t + 1 < T) load_tile(t + 1, (t + 1) & 1);
        const uint32_t base = kFlatMisc + (t & 1) * R * S;
        const int row0 = (g0 + t) * R;
        unsigned pos = 0;
        const auto run = [&](auto NStag) {
            constexpr int NS = decltype(NStag)::value;
            std::conditional_t<UNI, f32x16, std::conditional_t<R == 1, f32x2, std::conditional_t<R == 2, f32x4, f32x8>>> acc = {};
            if constexpr (UNI) fma_flat<R, NS>(acc, code, wuni, base);
            else fma_flat<R, NS>(acc, code, wv, base);
            set_wave_prio(3);
#pragma unroll
            for (int s = 0; s < NS; ++s) {
                const int j = 64 * (first + 16 * s + wave) + lane;
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    const float y = j < N ? fminf(fmaxf(acc[s * R + r] + bj[s], 0.0f), kClip) : 0.0f;
                    if (__builtin_amdgcn_ballot_w64(y > 0.0f) != 0ull) pos |= 1u << r;
                    if (j < N && row0 + r < A) __builtin_nontemporal_store(y, Yout + (size_t)(row0 + r) * N + j);
                }
            }
        };
        if (nslots == SLOTS) run(std::integral_constant<int, SLOTS>{});
        else if (nslots == 1) run(std::integral_constant<int, 1>{});
        else if constexpr (UNI) {
            if (nslots == 2) run(std::integral_constant<int, 2>{});
            else if (nslots == 3) run(std::integral_constant<int, 3>{});
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
