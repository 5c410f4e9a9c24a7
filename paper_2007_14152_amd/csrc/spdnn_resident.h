// a1 + a2 + a3 for networks of at most 4096 neurons per layer: feature rows stay in LDS from layer to layer.
//
// A workgroup that computes EVERY neuron of the rows it is given has the next layer's input in its own hands: rows
// are independent (Eq. 1), so it can take a few rows through many layers without touching memory in between.  Up to
// 4096 columns fit: a pass holds 4 * P feature rows as P planes of 4 rows (an entry = 4 rows of one column, 16
// bytes), P = 4 for 1 and 2, 2 for 3 and 4 output blocks of 1024 neurons: at most 128 KB of LDS.  What moves instead are
// the connections, which every workgroup reads once per layer and pass (64 KB per 1024 neurons where the layer has
// one weight, 192 KB otherwise) straight into registers, a neuron-group ahead of their use.  A layer is
//
//   compute   lane = output neuron, for each of its NB blocks: 32 connections x P ds_read_b128 x 4 FMAs, summed in the
//             order the set-up chose, bias last -- the same operations in the same order as the per-layer kernels;
//             the clipped results stay in registers (NB * P * 4 <= 32)
//   barrier   every wave is done reading the rows
//   write     the results go over the input, each to the slot its column has in the NEXT layer's tile layout
//   barrier
//
// The rows that still have a positive output are a bit mask; rows that died stay in place as zeros (bias <= 0 keeps
// them zero) until so many are dead that the survivors need fewer planes: then the write packs them together
// (Listing 1's pruning inside the pass).  A pass whose rows have all died is over.
//
// A workgroup's share of the rows is a number of passes, and a pass reads a layer's connections whole whatever lives in
// it.  So rows that die later make passes worth merging: a pass that has lost 3/8 of its rows stops behind that layer,
// its survivors' rows go to memory, and the share's other passes stop there too; as soon as a pass's worth of rows
// waits there, it goes on from that layer.  A pass of those may stop again further on (kResLevels).  Nothing of this
// happens, or costs anything, as long as rows live.  Shares are dealt out quad by quad, so that rows that die together
// because they came in together are spread over the workgroups.  Whole passes, 24 layers on 60 000 rows of 4096 neurons
// with weights of their own: nine in ten die in layer 3 6.97 -> 3.41 ms; seven in ten, the first of the batch, 8.36 -> 4.44.
//
// What bounds it.  One weight per layer: LDS reads (16 bytes per connection, plane and lane; 256 B per clock and CU) and
// the FMAs behind them, which take nearly the same time (counters, 30 000 rows: LDS active 90 % of the clocks at
// 1024 neurons and 82 % at 4096, a fifth of that bank conflicts, vector instructions 80 and 78 %).  Weights of their own: the same two
// (74 and 71 %; neurons of any length 66 and 70), at 30 000 clocks per layer and pass of 4096 neurons, of which the reads would take 16 400 without conflicts (without any one of reads, FMAs and connection loads a layer takes 10 to 18 %
// less), and the rows' way in and out, 33 000 clocks per pass; the connections, 768 KB per layer and pass, are not what it
// waits for: a CU gets 53 bytes per clock out of its L2, in loads or beside LDS reads.  One workgroup on its own: latency.
// The copies between LDS and memory happen once per launch instead of once per layer.  What a wave can find out before the
// barrier -- which rows have a positive output -- it does group by group, not behind the last one: 12 layers of 4096 neurons
// with weights, 10 007 rows 889 -> 853 us with that and with buffer loads for the connections (load_lanes).
// Whole passes, one launch per layer -> this kernel: 120 layers of 1024 neurons, 1000 rows 0.85 -> 0.27 ms, 60 000 rows
// 7.40 -> 4.70; 24 layers of 4096 neurons, 60 000 rows 5.85 -> 4.53 (the first two layers one by one); 12 of them with
// weights of their own, 10 007 rows 1.19 -> 0.85; 6 with 16 to 64 connections per neuron, 10 000 rows 1.26 -> 0.68 (several
// lanes per neuron and two launches per layer before).  Few rows are few_kernel's.
//
// Workgroups.  Networks of one block whose rows are more than a quad per CU run two workgroups per CU of eight waves
// (two groups of 64 neurons per wave), so that one computes while the other writes or waits at a barrier (120 layers,
// 60 000 rows, when this was chosen: 5.12 ms against 5.19 for one workgroup with eight planes); fewer rows, one of sixteen waves.
#pragma once

namespace spdnn {

// Most rows a workgroup may own when networks of one output block run all their layers in one launch.
constexpr int kShareRows = 128;

struct ResidentLayer {   // one layer, in device memory
    const uint16_t* rel;   // LayerWeights::rel, slots as entry codes (res_code)
    const float* val;
    const uint32_t* qsel;  // quads of the columns of this layer's input (LayerWeights::qsel, block 0: all blocks share it)
    float wuni;            // kResUniform: the layer's weight
    // kResParts:
    const uint16_t* perm;  // neuron of every lane (64 to a group), 0xFFFF: none
    const uint32_t* nch;   // chunks of 8 connections that a group of 64 lanes has
};
// What the layers of a network have in common.  kResWeights: 32 connections per neuron.  kResUniform: the same, one weight
// per layer (it takes a scalar register, and half the bytes are read).  kResParts: any number of connections; the neurons
// are given to the lanes by length, longest first, so that the 64 lanes of a group have about equally many, and a group
// runs the chunks of 8 that its longest lane needs (the zero padding of Section III-A-3, per wave).  Every 32 connections
// are summed by themselves and added to the neuron's sum, in order.
enum { kResWeights = 0, kResUniform = 1, kResParts = 2 };
struct ResidentArgs {
    const ResidentLayer* layers;
    int l0, lmid, l1;  // layers l0 .. l1-1; passes stop and are merged at lmid (l1: only where rows die)
    int L;             // layers of the network
    int A;             // rows on entry, if the lists are not there yet (rl.count == NULL): row i is in slot i
    uint32_t part_stride;  // kResParts: bytes from a group's connections 32p .. 32p+31 to the next 32, slots and weights alike
    int* layer_rows;   // NULL, or [L + 1] counters: [l] += rows alive on entry to layer l
};

// Bytes of LDS: the planes, then the bookkeeping.
constexpr int kResMiscBytes = 1024;
constexpr int kResLevels = 6;  // layers a launch's passes may start at: l0, and five where they were stopped
// A pass stops where 5/8 of its rows or fewer live and at least three layers are left.  (Stopping costs the survivors' way
// through memory, about a layer's time.  Half and two layers, 24 layers of 4096 neurons on 30 000 rows that die evenly: 3.24
// instead of 3.17 ms; of 2048 neurons, 30 layers: 1.92 instead of 1.88; three quarters and four layers: 3.19, 1.92.)
constexpr int kStopNum = 5, kStopDen = 8, kStopLeft = 3;
SPDNN_HD inline uint32_t res_chunk_bytes(int planes) { return 256u * (uint32_t)planes; }
SPDNN_HD inline uint32_t res_tile_bytes(int N, int planes) { return (uint32_t)((N + 255) / 256) * 16u * res_chunk_bytes(planes); }

// A lane's 16 bytes of an array that the wave reads at a scalar place: base + scalar offset + the lane's.  As a buffer load it
// takes no vector instruction and no vector register for the address, where a pointer of the lane's own takes one and two.
__device__ __forceinline__ u32x4 load_lanes(const __attribute__((address_space(1))) char* base, uint32_t offset, uint32_t lane_offset) {
    const auto rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)base, 0, 0xffffffff, 0x00027000);
    return __builtin_amdgcn_raw_buffer_load_b128(rsrc, lane_offset, offset, 0);
}

// Eight connections of one neuron on P planes: acc[p] += tile[plane p][column i] * w_i, i = 0..7 in that order.  codes =
// the eight entry codes, two to a register; an SDWA shift makes a half an LDS address, which serves all planes through
// the read's immediate offset.  The reads of all (connection, plane) pairs form one pipeline of D in flight.  The
// accumulators and addresses sit in fixed registers so that the assembler's own loop can number them: plane p in
// v[80+4p .. 83+4p], address i in v[72+i], reads in v[112:127].
#define SPDNN_RES_ADDR(I, C, H) \
    "v_lshlrev_b32_sdwa v[72+" I "], %[s4], %[" C "] dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:WORD_" H "\n\t"
#define SPDNN_RES_READ(K)                                                                                        \
    "ds_read_b128 v[112+4*((" K ")%%%[D]):115+4*((" K ")%%%[D])], v[72+(" K ")/%[P]] offset:256*((" K ")%%%[P])\n\t"
#define SPDNN_RES_CONN_(ADD, W, FROM)                        \
    ".set spdnn_p, 0\n\t"                                    \
    ".rept %[P]\n\t"                                         \
    ".if 8*%[P]-spdnn_k > %[D]\n\t"                             \
    "s_waitcnt lgkmcnt(%[D]-1)\n\t"                          \
    ".else\n\t"                                              \
    "s_waitcnt lgkmcnt(8*%[P]-spdnn_k-1)\n\t"                \
    ".endif\n\t"                                             \
    ADD " v[80+4*spdnn_p], " W ", v[112+4*(spdnn_k%%%[D])]" FROM "\n\t" \
    ADD " v[81+4*spdnn_p], " W ", v[113+4*(spdnn_k%%%[D])]" FROM "\n\t" \
    ADD " v[82+4*spdnn_p], " W ", v[114+4*(spdnn_k%%%[D])]" FROM "\n\t" \
    ADD " v[83+4*spdnn_p], " W ", v[115+4*(spdnn_k%%%[D])]" FROM "\n\t" \
    ".if spdnn_k+%[D] < 8*%[P]\n\t"                          \
    SPDNN_RES_READ("spdnn_k+%[D]")                           \
    ".endif\n\t"                                             \
    ".set spdnn_p, spdnn_p+1\n\t"                            \
    ".set spdnn_k, spdnn_k+1\n\t"                            \
    ".endr\n\t"
#define SPDNN_RES_CONN(W) SPDNN_RES_CONN_("v_fmac_f32", W, "")
#define SPDNN_RES_CONN0(W) SPDNN_RES_CONN_("v_fma_f32", W, ", 0")  // the first of all: sums start at 0
#define SPDNN_RES_HEAD                                                                                                 \
    SPDNN_RES_ADDR("0", "c0", "0") SPDNN_RES_ADDR("1", "c0", "1") SPDNN_RES_ADDR("2", "c1", "0") SPDNN_RES_ADDR("3", "c1", "1") \
    ".set spdnn_k, 0\n\t" SPDNN_RES_READ("0") SPDNN_RES_READ("1") SPDNN_RES_READ("2") ".if %[D] > 3\n\t" SPDNN_RES_READ("3") ".endif\n\t" \
    SPDNN_RES_ADDR("4", "c2", "0") SPDNN_RES_ADDR("5", "c2", "1") SPDNN_RES_ADDR("6", "c3", "0") SPDNN_RES_ADDR("7", "c3", "1")
#define SPDNN_RES_ASM_U(FIRST)                                                                                         \
    SPDNN_RES_HEAD FIRST("%[w]") SPDNN_RES_CONN("%[w]") SPDNN_RES_CONN("%[w]") SPDNN_RES_CONN("%[w]")                    \
    SPDNN_RES_CONN("%[w]") SPDNN_RES_CONN("%[w]") SPDNN_RES_CONN("%[w]") SPDNN_RES_CONN("%[w]")
#define SPDNN_RES_ASM_W(FIRST)                                                                                         \
    SPDNN_RES_HEAD FIRST("%[w0]") SPDNN_RES_CONN("%[w1]") SPDNN_RES_CONN("%[w2]") SPDNN_RES_CONN("%[w3]")                \
    SPDNN_RES_CONN("%[w4]") SPDNN_RES_CONN("%[w5]") SPDNN_RES_CONN("%[w6]") SPDNN_RES_CONN("%[w7]")
#define SPDNN_RES_ACC1(D) D "{v[80:83]}"(acc[0])
#define SPDNN_RES_ACC2(D) SPDNN_RES_ACC1(D), D "{v[84:87]}"(acc[1])
#define SPDNN_RES_ACC3(D) SPDNN_RES_ACC2(D), D "{v[88:91]}"(acc[2])
#define SPDNN_RES_ACC4(D) SPDNN_RES_ACC3(D), D "{v[92:95]}"(acc[3])
#define SPDNN_RES_IN [c0] "v"(codes.x), [c1] "v"(codes.y), [c2] "v"(codes.z), [c3] "v"(codes.w), [s4] "s"(4), [P] "n"(P), [D] "n"(D)
#define SPDNN_RES_CLOBBER3                                                                                           \
    "v72", "v73", "v74", "v75", "v76", "v77", "v78", "v79", "v112", "v113", "v114", "v115", "v116", "v117", "v118", "v119",  \
        "v120", "v121", "v122", "v123", "memory"
#define SPDNN_RES_CLOBBER4 SPDNN_RES_CLOBBER3, "v124", "v125", "v126", "v127"
#define SPDNN_RES_RUN(Q, OUT, FIRST_CONN, CLOBBER)                                                                      \
    if constexpr (UNI)                                                                                               \
        asm volatile(SPDNN_RES_ASM_U(FIRST_CONN) : SPDNN_RES_ACC##Q(OUT) : SPDNN_RES_IN, [w] "s"(wu) : CLOBBER);        \
    else                                                                                                             \
        asm volatile(SPDNN_RES_ASM_W(FIRST_CONN)                                                                       \
                     : SPDNN_RES_ACC##Q(OUT)                                                                           \
                     : SPDNN_RES_IN, [w0] "v"(wa.x), [w1] "v"(wa.y), [w2] "v"(wa.z), [w3] "v"(wa.w), [w4] "v"(wb.x),     \
                       [w5] "v"(wb.y), [w6] "v"(wb.z), [w7] "v"(wb.w)                                                  \
                     : CLOBBER);
#define SPDNN_RES_CASE(Q)                                                                                             \
    if constexpr (P == Q && D == 3) {                                                                                \
        if constexpr (FIRST) { SPDNN_RES_RUN(Q, "=&", SPDNN_RES_CONN0, SPDNN_RES_CLOBBER3) }                            \
        else { SPDNN_RES_RUN(Q, "+", SPDNN_RES_CONN, SPDNN_RES_CLOBBER3) }                                              \
    } else if constexpr (P == Q) {                                                                                   \
        if constexpr (FIRST) { SPDNN_RES_RUN(Q, "=&", SPDNN_RES_CONN0, SPDNN_RES_CLOBBER4) }                            \
        else { SPDNN_RES_RUN(Q, "+", SPDNN_RES_CONN, SPDNN_RES_CLOBBER4) }                                              \
    }
// FIRST: acc need not be set, the sums start at 0.  D: reads in flight, 3 or 4.
template <int P, bool UNI, bool FIRST, int D>
__device__ __forceinline__ void res_fma8(f32x4 (&acc)[P], u32x4 codes, float wu, f32x4 wa, f32x4 wb) {
    SPDNN_RES_CASE(1)
    SPDNN_RES_CASE(2)
    SPDNN_RES_CASE(3)
    SPDNN_RES_CASE(4)
}

// NB = most groups of 64 neurons a wave owns, PM = most planes.  blockDim.x = 64 * W with W = ceil(U / NB),
// U = ceil(N / 64) groups of 64 neurons; wave w owns the groups w, w + W, ...  Workgroup i has the quads of rows i,
// i + gridDim.x, ... of the list on entry; a row keeps its place in the list in Yout, where it also waits while its pass
// is stopped.
template <int NB, int PM, int MODE>
__global__ __launch_bounds__(kBlk) void resident_kernel(const float* __restrict__ Yin, float* Yout,
                                                        uint8_t* __restrict__ flags, RowLists rl, ResidentArgs ra,
                                                        const float* __restrict__ bias, int N) {
    // The entry codes are addresses from the start of the workgroup's LDS: everything is dynamic, nothing static.
    extern __shared__ __align__(16) char res_lds[];
    using lds_f4 = __attribute__((address_space(3))) f32x4;
    // Three reads in flight leave registers that the weights take; four are better only where there is room for them (three / four:
    // 8 layers of 2048 neurons with weights, 20 000 rows 562 / 575 us, 120 layers of 1024 neurons, 60 000 rows 4594 / 4627; 24 layers
    // of 4096 neurons, one weight, 60 000 rows 4443 / 4431, 16 to 64 connections 670 / 665).
    constexpr int D = PM == 2 && MODE != kResWeights ? 4 : 3;
    constexpr uint32_t CH = 256u * PM;  // bytes of a chunk: 16 columns x PM planes
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int T = blockDim.x, W = T >> 6, U = (N + 63) >> 6;
    const uint32_t misc = res_tile_bytes(N, PM);
    uint32_t* live_word = reinterpret_cast<uint32_t*>(res_lds + misc);             // [2], raised by the layers in turn
    const uint32_t live_at = misc;                                                 // its LDS address
    int* row_at = reinterpret_cast<int*>(res_lds + misc + 16);                     // [4 * PM] row to copy to or from, per slot; -1: none
    constexpr int F = kRows * PM;  // rows of a full pass
    int* level_at = row_at + 16;               // [kResLevels + 1]
    int* level_n = level_at + kResLevels + 1;  // [kResLevels + 1]
    int* waiting = level_n + kResLevels + 1;   // [kResLevels - 1][2 * F] rows that wait, per level
    static_assert(16 + 4 * (16 + 2 * (kResLevels + 1) + (kResLevels - 1) * 2 * 16) <= kResMiscBytes, "the lists fit behind the planes");

    // my rows: `quads` quads, the last one of the list perhaps ragged
    const int A = rl.count ? __builtin_amdgcn_readfirstlane(*rl.count) : ra.A;
    const bool identity = !rl.count;
    const int groups = (A + kRows - 1) / kRows;
    const int wg = blockIdx.x, nwg = gridDim.x;
    if (wg >= groups) return;
    const int quads = (groups - wg + nwg - 1) / nwg;
    const int nrows = quads * kRows - ((groups - 1) % nwg == wg ? groups * kRows - A : 0);

    const int nb_w = (U - wave + W - 1) / W;  // my groups of 64 neurons (at least one: W <= U)
    float bj[NB];  // lanes without a neuron: minus infinity, which makes their outputs 0
    float* bias_lds = reinterpret_cast<float*>(res_lds + misc + kResMiscBytes);  // kResParts: [N]
    if constexpr (MODE == kResParts) {
        for (int j = tid; j < N; j += T) bias_lds[j] = bias[j];
    } else {
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            const int j = 64 * (b * W + wave) + lane;
            bj[b] = j < N ? bias[j] : -__builtin_inff();
        }
    }
    // Connections, fetched ahead: slots a whole group of 64 neurons (4 chunks of 8), weights two chunks.  Neurons of any
    // length: two chunks of both, and where the next layer's neurons are.
    // (Address spaces are spelled out: as generic pointers these loads would wait, and be waited for, with the LDS reads.)
    u32x4 cbuf[4];
    f32x4 wbuf[4] = {};
    using gchar = const __attribute__((address_space(1))) char;
    using gu32 = const __attribute__((address_space(1))) uint32_t;
    using gu16 = const __attribute__((address_space(1))) uint16_t;
    using cu32 = const __attribute__((address_space(4))) uint32_t;
    struct Item {  // a layer's connections of one group of 64 neurons
        gchar *c, *w;
        int nch;  // chunks of 8
    };
    auto item = [&](const ResidentLayer& d, int b) -> Item {
        const int u = b * W + wave;
        const uint32_t at = ((u >> 4) * (kNnz / 8) * kBlk + (u & 15) * 64) * 16;
        const uint32_t wat = ((u >> 4) * (kNnz / 4) * kBlk + (u & 15) * 64) * 16;
        const int nch = MODE == kResParts ? (int)((cu32*)(uintptr_t)d.nch)[u] : kNnz / 8;
        return Item{(gchar*)(uintptr_t)d.rel + at, (gchar*)(uintptr_t)d.val + wat, nch};
    };
    const uint32_t lane16 = 16u * lane;
    // chunk c (0..3) of the 32 connections that start at part_off bytes from the group's first
    auto fetch_codes = [&](const Item& it, int c) { cbuf[c] = load_lanes(it.c, (uint32_t)c * (16 * kBlk), lane16); };
    auto fetch_weights = [&](const Item& it, int c) {
        if constexpr (MODE == kResUniform) return;
        wbuf[2 * (c & 1)] = __builtin_bit_cast(f32x4, load_lanes(it.w, (uint32_t)(2 * c) * (16 * kBlk), lane16));
        wbuf[2 * (c & 1) + 1] = __builtin_bit_cast(f32x4, load_lanes(it.w, (uint32_t)(2 * c + 1) * (16 * kBlk), lane16));
    };
    auto fetch_chunk = [&](const Item& it, int slot, uint32_t c) {  // chunk c of the part that starts at `it`
        cbuf[slot] = load_lanes(it.c, c * (16 * kBlk), lane16);
        wbuf[2 * slot] = __builtin_bit_cast(f32x4, load_lanes(it.w, 2u * c * (16 * kBlk), lane16));
        wbuf[2 * slot + 1] = __builtin_bit_cast(f32x4, load_lanes(it.w, (2u * c + 1u) * (16 * kBlk), lane16));
    };
    // The descriptors are constant while the kernel runs: scalar loads.
    using clayer = const __attribute__((address_space(4))) ResidentLayer;
    auto layer_at = [&](int l) -> ResidentLayer {
        clayer* d = (clayer*)(uintptr_t)(ra.layers + l);
        return ResidentLayer{d->rel, d->val, d->qsel, d->wuni, d->perm, d->nch};
    };

    // Level v: rows that have come to layer level_at[v] and wait there for a pass (level 0: my rows on entry).
    const int npass = (quads + PM - 1) / PM;
    if (tid <= kResLevels) {  // seen from the second pass on
        level_at[tid] = tid == 0 ? ra.l0 : tid == 1 ? ra.lmid : ra.l1;
        level_n[tid] = 0;
    }
    int own = 0, i1 = 0;  // passes and rows of level 0 so far
    int jn_ahead[NB];     // kResParts: the next layer's neurons
    const auto neurons_of = [&](const ResidentLayer& d) {
        if constexpr (MODE == kResParts)
#pragma unroll
            for (int b = 0; b < NB; ++b) jn_ahead[b] = b < nb_w ? ((gu16*)(uintptr_t)d.perm)[64 * (b * W + wave) + lane] : 0;
    };
    int primed = -1;      // the layer whose first group's connections cbuf / wbuf hold ...
    Item ahead{};         // ... which is this (in general: the group whose connections come next)
    for (;;) {
        // the furthest level with a full pass; when my own rows are used up, the nearest with any
        int v = 0, la = ra.l0, lb = ra.lmid, n = 0;
        bool more = npass > 1;  // rows to come at this level or before it, which this pass could be merged with
        bool lower = false;     // rows that wait at a level before this one
        if (own > 0) {
            const int at = level_at[min(lane, kResLevels)], w = level_n[min(lane, kResLevels)];
            const uint32_t full = (uint32_t)__builtin_amdgcn_ballot_w64(lane < kResLevels && w >= F);
            const uint32_t any = (uint32_t)__builtin_amdgcn_ballot_w64(lane < kResLevels && w > 0);
            if (full) v = 31 - __builtin_clz(full);
            else if (own == npass && any) v = __builtin_ctz(any);
            else if (own == npass) break;
            la = __builtin_amdgcn_readlane(at, v);
            lb = __builtin_amdgcn_readlane(at, v + 1);
            n = __builtin_amdgcn_readlane(w, v);
            lower = (any & ((1u << v) - 1u)) != 0u;
            more = own + (v == 0) < npass || lower || n > F;
        }
        int n0;   // rows of this pass
        int rid;  // lane s (of every wave): place in the list of the row in slot s
        if (v == 0) {
            // (the shorter passes first in one half of the workgroups, last in the other: the passes get out of step, and
            // with them the workgroups' turns at the memory)
            const int upto = (wg & 1) ? quads - ((npass - 1 - own) * quads) / npass : ((own + 1) * quads) / npass;
            const int i0 = i1;
            i1 = min(nrows, upto * kRows);
            n0 = i1 - i0;
            const int i = i0 + min(lane, n0 - 1);
            rid = ((i / kRows) * nwg + wg) * kRows + i % kRows;
            ++own;
        } else {
            // a full pass as long as more rows come; the last ones are shared out evenly, quad by quad (17 rows as 16 and 1
            // take 8 % longer than as 12 and 5: 97 layers of 1024 neurons on 13 326 rows, half of them dead, 1.33 -> 1.29 ms)
            n0 = F;
            if (own == npass && !lower) {
                const int left = (n + kRows - 1) / kRows, passes = (left + PM - 1) / PM;
                n0 = min(n, (left + passes - 1) / passes * kRows);
            }
            n -= n0;
            rid = waiting[(v - 1) * 2 * F + n + min(lane, n0 - 1)];
        }
        // So few rows stop the pass, if there is a level left and rows it could be merged with.
        const int few = more && v < kResLevels - 1 && lb == ra.l1 ? n0 * kStopNum / kStopDen : 0;
        {
            const float* src = v == 0 ? Yin : Yout;
            const ResidentLayer first = layer_at(la);
            const uint32_t* q_in = first.qsel;
            const uint32_t* q_out = layer_at(min(lb, ra.L - 1)).qsel;  // any layout does for the last layer's output
            int P = (n0 + kRows - 1) / kRows;
            uint32_t live = n0 >= 32 ? 0xffffffffu : (1u << n0) - 1u;
            if (tid < F) row_at[tid] = tid >= n0 ? -1 : v == 0 && !identity ? rl.cat[rid] : rid;
            if (v == 0 && tid < n0) flags[rid] = 0;  // wave 0, like every other store to the flags
            if (tid < 2) live_word[tid] = 0u;
            if (primed != la) {
                ahead = item(first, 0);
                neurons_of(first);
#pragma unroll
                for (int c = 0; c < (MODE == kResParts ? 2 : 4); ++c) fetch_codes(ahead, c);
                fetch_weights(ahead, 0);
                fetch_weights(ahead, 1);
            }
            __syncthreads();  // also: the pass before has left the tile
            const int n4 = N >> 2;
            for (int e = tid; e < P * n4; e += T) {  // 4 rows x 4 columns per turn
                const int p = e / n4, t = e - p * n4;
                const int4 at = *reinterpret_cast<const int4*>(row_at + 4 * p);
                const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
                const size_t col = (size_t)t * 4;
                const f32x4 a0 = *reinterpret_cast<const f32x4*>(src + (size_t)at.x * N + col);
                const f32x4 a1 = at.y < 0 ? zero : *reinterpret_cast<const f32x4*>(src + (size_t)at.y * N + col);
                const f32x4 a2 = at.z < 0 ? zero : *reinterpret_cast<const f32x4*>(src + (size_t)at.z * N + col);
                const f32x4 a3 = at.w < 0 ? zero : *reinterpret_cast<const f32x4*>(src + (size_t)at.w * N + col);
                const uint32_t qp = q_in[t];
                const uint32_t base = (store_group((uint32_t)t * 4u)) * CH + 256u * p;
                *reinterpret_cast<lds_f4*>(base + (qp & 0xffu)) = f32x4{a0.x, a1.x, a2.x, a3.x};
                *reinterpret_cast<lds_f4*>(base + CH + ((qp >> 8) & 0xffu)) = f32x4{a0.y, a1.y, a2.y, a3.y};
                *reinterpret_cast<lds_f4*>(base + 2u * CH + ((qp >> 16) & 0xffu)) = f32x4{a0.z, a1.z, a2.z, a3.z};
                *reinterpret_cast<lds_f4*>(base + 3u * CH + (qp >> 24)) = f32x4{a0.w, a1.w, a2.w, a3.w};
            }
            __syncthreads();

            // Layers l .. as long as PP planes are needed: a loop of its own for every number of planes.
            int l = la, stop = lb;
            ResidentLayer cur = first, nxt = layer_at(la + 1 < lb ? la + 1 : la);
            auto layers = [&](auto Ptag) {
                constexpr int PP = decltype(Ptag)::value;
                const int enough = max(kRows * (PP - 1), few);  // as long as more rows live, all stays as it is
                while (l < stop && P == PP) {
                    gu32* q_next = (gu32*)(uintptr_t)(l + 1 < lb ? nxt.qsel : q_out);
                    int jn[NB];       // my neurons
                    uint32_t at[NB];  // where their outputs go
#pragma unroll
                    for (int b = 0; b < NB; ++b) {
                        jn[b] = MODE == kResParts ? jn_ahead[b] : 64 * (b * W + wave) + lane;
                        at[b] = q_next[min(jn[b], N - 1) >> 2];
                    }
                    neurons_of(nxt);
                    auto place = [&]() {  // out of the way of the first chunk's arithmetic
#pragma unroll
                        for (int b = 0; b < NB; ++b) at[b] = store_group((uint32_t)jn[b]) * CH + ((at[b] >> (8 * (jn[b] & 3))) & 0xffu);
                    };
                    f32x4 res[NB][PP];
                    uint32_t pos = 0;  // rows that have a positive output in my neurons
#pragma unroll
                    for (int b = 0; b < NB; ++b) {
#pragma unroll
                        for (int p = 0; p < PP; ++p) res[b][p] = f32x4{0.f, 0.f, 0.f, 0.f};
                        if (b < nb_w) {
                            f32x4 acc[PP];
                            const Item mine = ahead;
                            const Item next = b + 1 < nb_w ? item(cur, b + 1) : item(nxt, 0);
                            ahead = next;
                            if constexpr (MODE != kResParts) {
#pragma unroll
                                for (int c = 0; c < 4; ++c) {
                                    if ((b * 4 + c) % NB == 0) set_wave_prio(3 - (b * 4 + c) / NB);
                                    if (c == 0) res_fma8<PP, MODE == kResUniform, true, D>(acc, cbuf[0], cur.wuni, wbuf[0], wbuf[1]);
                                    else res_fma8<PP, MODE == kResUniform, false, D>(acc, cbuf[c], cur.wuni, wbuf[2 * (c & 1)], wbuf[2 * (c & 1) + 1]);
                                    fetch_codes(next, c);
                                    if (c < 2) fetch_weights(mine, c + 2);
                                    else fetch_weights(next, c - 2);
                                    if (b == 0 && c == 0) place();
                                }
#pragma unroll
                                for (int p = 0; p < PP; ++p) res[b][p] = acc[p];
                            } else {
                                // Two chunks per turn, each refilled behind its arithmetic, whether it had any or not: what is on
                                // its way at any point is the same on every path, so a chunk's wait is for that chunk (with
                                // refills on some paths only, for all that had been asked for: 10 000 rows, 6 layers of 4096
                                // neurons of 16 to 64 connections 701 us, 670 so).
#pragma unroll
                                for (int p = 0; p < PP; ++p) acc[p] = f32x4{0.f, 0.f, 0.f, 0.f};
                                set_wave_prio(3 - b * 4 / NB);
                                uint32_t off = 0;  // of the part of 32 connections that the next two chunks are of
                                for (int c = 0; c == 0 || c < mine.nch; c += 2) {
                                    const bool last = c + 2 >= mine.nch;
                                    if (c & 2) off += ra.part_stride;
                                    const uint32_t half = last || (c & 2) ? 0u : 2u;  // the next chunks' place in their part
                                    const Item from = last ? Item{next.c, next.w, 0} : Item{mine.c + off, mine.w + off, 0};
#pragma unroll
                                    for (int i = 0; i < 2; ++i) {
                                        if (c + i < mine.nch) res_fma8<PP, false, false, D>(acc, cbuf[i], 0.0f, wbuf[2 * i], wbuf[2 * i + 1]);
                                        fetch_chunk(from, i, half + i);
                                    }
                                    if (last || (c & 2))
#pragma unroll
                                        for (int p = 0; p < PP; ++p) {
                                            res[b][p] += acc[p];
                                            acc[p] = f32x4{0.f, 0.f, 0.f, 0.f};
                                        }
                                }
                                bj[b] = jn[b] < N ? bias_lds[min(jn[b], N - 1)] : -__builtin_inff();
                                if (b == 0) place();
                            }
#pragma unroll
                            for (int p = 0; p < PP; ++p)
#pragma unroll
                                for (int r = 0; r < kRows; ++r) {
                                    res[b][p][r] = fminf(fmaxf(res[b][p][r] + bj[b], 0.0f), kClip);
                                    pos = __builtin_amdgcn_ballot_w64(res[b][p][r] > 0.0f) != 0ull ? pos | 1u << (kRows * p + r) : pos;
                                }
                        }
                    }
                    set_wave_prio(3);
                    // Descriptors are asked for a layer ahead, and not before the arithmetic: its waits for the LDS would wait
                    // for them too.  After the last layer comes, for the connections, the next pass's first.
                    const ResidentLayer after = layer_at(l + 2 < lb ? l + 2 : la);
                    // (a plain LDS operation of one lane: the compiler's atomic would look for the first active lane on its own)
                    if (lane == 0) asm volatile("ds_or_b32 %0, %1" ::"v"(live_at + 4u * (uint32_t)(l & 1)), "v"(pos) : "memory");
                    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                    __syncthreads();  // every wave has read what it needs of the rows
                    const uint32_t raised = live_word[l & 1];  // (on its way while the results go out)
#pragma unroll
                    for (int b = 0; b < NB; ++b) {
                        if (b < nb_w && jn[b] < N)
#pragma unroll
                            for (int p = 0; p < PP; ++p) *reinterpret_cast<lds_f4*>(at[b] + 256u * p) = res[b][p];
                    }
                    live &= __builtin_amdgcn_readfirstlane(raised);
                    if (tid == 0) live_word[(l + 1) & 1] = 0u;
                    const int n = __popc(live);
                    if (n <= enough) {
                        P = (n + kRows - 1) / kRows;
                        if (P < PP && n > 0) {  // fewer planes will do: the survivors move together, over what was just written
                            using lds_f = __attribute__((address_space(3))) float;
#pragma unroll
                            for (int b = 0; b < NB; ++b) {
                                if (b < nb_w && jn[b] < N) {
#pragma unroll
                                    for (int s = 0; s < kRows * PP; ++s)
                                        if ((live >> s) & 1u) {
                                            const int to = __popc(live & ((1u << s) - 1u));
                                            *reinterpret_cast<lds_f*>(at[b] + 256u * (to >> 2) + 4u * (to & 3)) = res[b][s >> 2][s & 3];
                                        }
                                    for (int s = n; s < kRows * P; ++s) *reinterpret_cast<lds_f*>(at[b] + 256u * (s >> 2) + 4u * (s & 3)) = 0.0f;
                                }
                            }
                            // slot s now holds what the s-th live slot held
                            int from = 0;
                            for (uint32_t rest = live, k = 0; rest; rest &= rest - 1u, ++k)
                                if (lane == (int)k) from = __builtin_ctz(rest);
                            rid = __shfl(rid, from, 64);
                            live = n >= 32 ? 0xffffffffu : (1u << n) - 1u;
                        }
                        if (n > 0 && n <= few && l + 1 + kStopLeft <= ra.l1) stop = l + 1;
                    }
                    __syncthreads();
                    if (tid == 0 && n > 0 && ra.layer_rows) atomicAdd(&ra.layer_rows[l + 1], n);
                    cur = nxt;
                    nxt = after;
                    ++l;
                }
            };
            if constexpr (PM >= 4) {
                layers(std::integral_constant<int, 4>{});
                layers(std::integral_constant<int, 3>{});
            }
            layers(std::integral_constant<int, 2>{});
            layers(std::integral_constant<int, 1>{});
            if (!live) {
                primed = -1;
                if (v > 0) {
                    if (tid == 0) level_n[v] = n;
                    __syncthreads();
                }
                continue;
            }
            // a stopped pass asked for the next layer's connections, one that ran through for those of its first layer
            primed = stop < lb ? stop : la;
            if (stop < lb) q_out = cur.qsel;

            // the survivors' rows go to memory; those of a stopped pass wait for the next level's
            if (tid < F) row_at[tid] = (live >> tid) & 1u ? rid : -1;
            if (wave == 0) {
                const int before = l < ra.l1 ? level_n[v + 1] : 0;
                if (lane < 32 && ((live >> lane) & 1u)) {
                    if (l == ra.l1) flags[rid] = 1;
                    else waiting[v * 2 * F + before + __popc(live & ((1u << lane) - 1u))] = rid;
                }
                if (lane == 0) {
                    if (v > 0) level_n[v] = n;
                    if (l < ra.l1) level_n[v + 1] = before + __popc(live);
                    if (stop < lb) level_at[v + 1] = stop;
                }
            }
            __syncthreads();
            for (int e = tid; e < P * n4; e += T) {
                const int p = e / n4, t = e - p * n4;
                const int4 at = *reinterpret_cast<const int4*>(row_at + 4 * p);
                const size_t col = (size_t)t * 4;
                const uint32_t qp = q_out[t];
                const uint32_t base = (store_group((uint32_t)t * 4u)) * CH + 256u * p;
                const f32x4 c0 = *reinterpret_cast<const lds_f4*>(base + (qp & 0xffu));
                const f32x4 c1 = *reinterpret_cast<const lds_f4*>(base + CH + ((qp >> 8) & 0xffu));
                const f32x4 c2 = *reinterpret_cast<const lds_f4*>(base + 2u * CH + ((qp >> 16) & 0xffu));
                const f32x4 c3 = *reinterpret_cast<const lds_f4*>(base + 3u * CH + (qp >> 24));
                if (at.x >= 0) *reinterpret_cast<f32x4*>(Yout + (size_t)at.x * N + col) = f32x4{c0.x, c1.x, c2.x, c3.x};
                if (at.y >= 0) *reinterpret_cast<f32x4*>(Yout + (size_t)at.y * N + col) = f32x4{c0.y, c1.y, c2.y, c3.y};
                if (at.z >= 0) *reinterpret_cast<f32x4*>(Yout + (size_t)at.z * N + col) = f32x4{c0.z, c1.z, c2.z, c3.z};
                if (at.w >= 0) *reinterpret_cast<f32x4*>(Yout + (size_t)at.w * N + col) = f32x4{c0.w, c1.w, c2.w, c3.w};
            }
            __syncthreads();  // row_at is free for the next pass, and the rows that wait are in place
        }
    }
}

}  // namespace spdnn
