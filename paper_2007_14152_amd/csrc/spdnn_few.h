// Networks of at most 4096 neurons on few rows -- at most four per workgroup, a workgroup per CU: the rows stay in LDS from
// layer to layer as in resident_kernel, and with so few of them a layer is a matter of latency and instruction issue.
//
// A workgroup has R = 1 to 4 rows, as few as the batch allows: an entry is a column's R values (4, 8 or 16 bytes), and a
// connection costs one read of R values and R multiply-adds, where resident_kernel always computes four.  The rows are kept
// twice, a layer reads one copy and writes the other, so that it has one barrier instead of two, results go out as each
// group of 64 neurons is done, and which rows still live is looked at while the next layer is computed.  The copies are
// planes 0 and 1 of resident_kernel's tile layout at a quarter, half or (three rows too) all of its size: the connections' entry
// codes are the same, and the sums are the same products in the same order (kResParts: parts of 32 likewise), so the results have the same bits.
//
// The connections of a group are on their way while the group before is computed, all 32 with their weights: 12 KB per wave,
// which is what it takes for the 47 to 60 bytes per clock that a CU gets out of its L2 (two groups ahead, one row: 12 layers of 1024
// neurons 49.0 -> 48.7 us, 3100 neurons 87 -> 91).  (Neurons of any length: 16 of them.)
//
// Two rows or one, an entry of 8 or 4 bytes: such reads are served for two sets of 16 lanes at a time, and the order of the connections
// is that of 16-byte entries, which keeps a set's lanes apart and knows nothing of the other set.  The rows are there twice
// therefore, in planes that lie in different banks, a plane for each set: with one weight, 120 layers of 1024
// neurons on 1000 rows 218 -> 201 us, of 2048 on 300 rows 340 -> 281; 24 layers of 4096 on 200 rows 142 -> 119.
//
// What bounds it: latency -- 700 to 1000 clocks of a layer's 3300 (1024 neurons) to 17 000
// (4096 with weights) are the barrier and the waits at its ends -- and with weights of their own the stream of connections (one row, 12
// layers of 1024: LDS 21 %, vector instructions 23 % of the one CU's clocks).  With one weight and two rows: instructions, of which a
// wave issues one every 5 clocks and has 290 in a layer.
// Whole calls, resident_kernel -> this kernel when it was new: one row
// through 12 layers of 1024 neurons with weights 57 -> 51 us, of 4096 neurons 130 -> 116; 1000 rows, half of which die, through
// 120 layers of 1024 neurons with one weight 261 -> 228; 100 rows through 24 layers of 4096 neurons 179 -> 147.
//
// A deep network in which rows die shares them out anew behind two layers: the second launch's workgroups find their rows by
// counting the first one's flags themselves (FewArgs::flags_prev), so nothing runs between the two and the host does not wait.
// A batch that a single workgroup holds is finished there too: survivors numbered, counted and written to the caller.
#pragma once

namespace spdnn {

constexpr int kFewRows = 4;        // rows per workgroup, at most
constexpr int kFewCount = 1024;    // rows whose flags a second launch counts, at most
constexpr int kFewMiscBytes = 256;

struct FewArgs {
    const ResidentLayer* layers;
    int l0, l1;            // layers l0 .. l1-1
    int A;                 // rows on entry, without flags_prev; else rows that flags_prev speaks about (at most kFewCount)
    uint32_t part_stride;  // see ResidentArgs
    int planes_log2;
    int* layer_rows;       // see ResidentArgs
    const uint8_t* flags_prev;  // NULL: row i is in slot i of Yin.  Else its rows are the slots whose flag is set, ...
    int* gid;                   // ... whose numbers (row_offset + slot) go here ...
    int* count;                 // ... and how many there are here
    int row_offset;
    float* Yout;
    uint8_t* flags;        // whose rows live
    int* rows_out;         // not NULL: the workgroup is the only one and finishes the call: the survivors' numbers, ...
    int* host_count;       // ... their count; their rows are the first ones of Yout
};

template <int R>
struct FewEntry;
template <>
struct FewEntry<1> {
    typedef float T __attribute__((ext_vector_type(1)));
};
template <>
struct FewEntry<2> {
    typedef float T __attribute__((ext_vector_type(2)));
};
template <>
struct FewEntry<3> {  // as for four, the last value unused
    typedef float T __attribute__((ext_vector_type(4)));
};
template <>
struct FewEntry<4> {
    typedef float T __attribute__((ext_vector_type(4)));
};

// The two entry codes of a register as LDS addresses of entries of 4 << LOG2R bytes, from `base` on: an instruction for each, where
// adding a plane and a copy to both codes first took half a one more (one weight, 120 layers of 1024 neurons, 500 rows 188 -> 181 us, of
// 2048 on 300 rows, 60 layers, 175 -> 167; 24 layers of 4096 on 500 rows 145 -> 136).  Without a base: 16-byte entries, whose copy
// is in the read's offset.
template <int LOG2R>
__device__ __forceinline__ void few_address(uint32_t codes, uint32_t base, uint32_t& lo, uint32_t& hi) {
    asm("v_mad_u32_u16 %0, %1, %2, %3" : "=v"(lo) : "v"(codes), "n"(4 << LOG2R), "v"(base));
    asm("v_mad_u32_u16 %0, %1, %2, %3 op_sel:[1,0,0,0]" : "=v"(hi) : "v"(codes), "n"(4 << LOG2R), "v"(base));
}
template <int LOG2R>
__device__ __forceinline__ void few_address(uint32_t codes, uint32_t& lo, uint32_t& hi) {
    asm("v_lshlrev_b32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:WORD_0" : "=v"(lo) : "s"(2 + LOG2R), "v"(codes));
    asm("v_lshlrev_b32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:WORD_1" : "=v"(hi) : "s"(2 + LOG2R), "v"(codes));
}

template <int R, int MODE>
__device__ __forceinline__ void few_layers(const FewArgs& fa, const float* __restrict__ Yin, const float* __restrict__ bias, int N, int A, const int* row_at,
                                           uint32_t* live_word) {
    using T = typename FewEntry<R>::T;
    using lds_T = __attribute__((address_space(3))) T;
    using gchar = const __attribute__((address_space(1))) char;
    using gf32 = const __attribute__((address_space(1))) float;
    using gu32 = const __attribute__((address_space(1))) uint32_t;
    using gu16 = const __attribute__((address_space(1))) uint16_t;
    using cu32 = const __attribute__((address_space(4))) uint32_t;
    using clayer = const __attribute__((address_space(4))) ResidentLayer;
    constexpr int LOG2R = R == 1 ? 0 : R == 2 ? 1 : 2;
    // Entries of 4 and 8 bytes are read for two sets of 16 lanes at once, whose connections were ordered for 16-byte entries, each
    // set's by itself: the sets find the rows in planes of their own.  Of 8-byte entries one plane lies in the lower half of the banks, the other in
    // the upper.  Of 4-byte entries 16 take 16 banks: up to 2048 columns the two planes of one copy lie in banks 0 to 15 and 16 to 31, those of
    // the other copy in 32 to 47 and 48 to 63; of more columns a copy's planes alternate, 16 banks each, through all 64.
    constexpr bool TWICE = LOG2R < 2;
    constexpr uint32_t PLANE = 16u << (2 + LOG2R);  // bytes from an entry to its place in the next plane
    const int tid = threadIdx.x, lane = tid & 63, T_ = blockDim.x, W = T_ >> 6, U = (N + 63) >> 6;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int row0 = (int)blockIdx.x * R, nrow = min(R, A - row0);
    const int nb_w = (U - wave + W - 1) / W;
    const uint32_t lane16 = 16u * lane;
    // bytes from an entry to its place in the other copy of the rows: a layer reads one and writes the other
    const uint32_t copy = !TWICE ? PLANE : fa.planes_log2 == 2 ? 2 * PLANE : ((uint32_t)(N + 255) / 256u * 512u) << (2 + LOG2R);
    const uint32_t my_plane = TWICE && (set_of_lane((uint32_t)lane) & 1u) ? PLANE : 0u;
    // LDS address of column j of a row laid out by q = its quads' word
    const auto entry = [&](int j, uint32_t q) -> uint32_t {
        return ((store_group((uint32_t)j) << (8 + fa.planes_log2)) | ((q >> (8 * (j & 3))) & 0xffu)) >> (2 - LOG2R);
    };
    struct Item {  // a layer's connections of one group of 64 neurons
        gchar *c, *w;
        int nch;  // chunks of 8
    };
    const auto layer_at = [&](int l) -> ResidentLayer {
        clayer* d = (clayer*)(uintptr_t)(fa.layers + l);
        return ResidentLayer{d->rel, d->val, d->qsel, d->wuni, d->perm, d->nch};
    };
    const auto item = [&](const ResidentLayer& d, int b) -> Item {
        const int u = b * W + wave;
        const uint32_t at = ((u >> 4) * (kNnz / 8) * kBlk + (u & 15) * 64) * 16;
        const uint32_t wat = ((u >> 4) * (kNnz / 4) * kBlk + (u & 15) * 64) * 16;
        const int nch = MODE == kResParts ? (int)((cu32*)(uintptr_t)d.nch)[u] : kNnz / 8;
        return Item{(gchar*)(uintptr_t)d.rel + at, (gchar*)(uintptr_t)d.val + wat, nch};
    };
    u32x4 cbuf[4];
    f32x4 wbuf[8] = {};
    const auto fetch = [&](const Item& it, int slot, uint32_t c) {  // chunk c of the 32 connections that start at `it`
        cbuf[slot] = load_lanes(it.c, c * (16 * kBlk), lane16);
        if constexpr (MODE != kResUniform) {
            wbuf[2 * slot] = __builtin_bit_cast(f32x4, load_lanes(it.w, 2u * c * (16 * kBlk), lane16));
            wbuf[2 * slot + 1] = __builtin_bit_cast(f32x4, load_lanes(it.w, (2u * c + 1u) * (16 * kBlk), lane16));
        }
    };
    // the neuron of this lane in its wave's group b of a layer, what comes with it
    const auto neuron = [&](const ResidentLayer& d, int b) -> int {
        const int i = 64 * (b * W + wave) + lane;
        if constexpr (MODE == kResParts) return ((gu16*)(uintptr_t)d.perm)[i];
        else return i;
    };

    // the rows
    ResidentLayer cur = layer_at(fa.l0), nxt = layer_at(fa.l0 + 1 < fa.l1 ? fa.l0 + 1 : fa.l0);
    const int n4 = N >> 2;
    int slot[R];
#pragma unroll
    for (int r = 0; r < R; ++r) slot[r] = r < nrow ? (row_at ? row_at[r] : row0 + r) : -1;
    Item ahead = item(cur, 0);
#pragma unroll
    for (int c = 0; c < (MODE == kResParts ? 2 : 4); ++c) fetch(ahead, c, c);
    int jn = neuron(cur, 0);
    for (int t = tid; t < n4; t += T_) {
        f32x4 a[R];
#pragma unroll
        for (int r = 0; r < R; ++r)
            a[r] = slot[r] < 0 ? f32x4{0.f, 0.f, 0.f, 0.f} : *reinterpret_cast<const f32x4*>(Yin + (size_t)slot[r] * N + 4 * (size_t)t);
        const uint32_t q = ((gu32*)(uintptr_t)cur.qsel)[t];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            T e = {};
#pragma unroll
            for (int r = 0; r < R; ++r) e[r] = a[r][i];
            *(lds_T*)(entry(4 * t + i, q)) = e;
            if constexpr (TWICE) *(lds_T*)(entry(4 * t + i, q) + PLANE) = e;
        }
    }
    __syncthreads();

    uint32_t live = (1u << nrow) - 1u;
    const uint32_t live_at = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint32_t*)live_word;
    bool other = false;  // the copy that holds the rows
    const auto layer = [&](int l, auto from) {
        constexpr bool OTHER = decltype(from)::value;
        constexpr uint32_t FROM = TWICE || !OTHER ? 0u : PLANE;  // (16-byte entries: the other copy is a constant away)
        const uint32_t rows_at = my_plane + (OTHER ? copy : 0u);  // (TWICE)
        const uint32_t to_copy = OTHER ? 0u : copy;
        // (scalar loads are waited for with the first reads of the rows, so not any later than this)
        const ResidentLayer after = layer_at(l + 2 < fa.l1 ? l + 2 : fa.l1 - 1);
        gchar* q_next = (gchar*)(uintptr_t)nxt.qsel;  // (any layout does for the last layer's output: its own)
        const uint32_t raised = l > fa.l0 ? live_word[(l + 2) % 3] : live;  // (looked at behind the arithmetic)
        uint32_t pos = 0;
#pragma unroll 1
        for (int b = 0; b < nb_w; ++b) {
            const int j = jn;
            const bool mine = j < N;
            const uint32_t near = (uint32_t)min(j, N - 1);
            const uint32_t q = *(gu32*)(q_next + (near & ~3u));
            const float bias_j = *(gf32*)((gchar*)(uintptr_t)bias + 4u * near);
            const Item it = ahead;
            ahead = b + 1 < nb_w ? item(cur, b + 1) : item(nxt, 0);
            jn = b + 1 < nb_w ? neuron(cur, b + 1) : neuron(nxt, 0);
            T sum = {}, acc = {};
            const auto read = [&](T (&y)[8], const u32x4& c) {
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    uint32_t lo, hi;
                    if constexpr (TWICE) few_address<LOG2R>(c[k], rows_at, lo, hi);
                    else few_address<LOG2R>(c[k], lo, hi);
                    y[2 * k] = *(const lds_T*)(lo + FROM);
                    y[2 * k + 1] = *(const lds_T*)(hi + FROM);
                }
            };
            const auto add = [&](const T (&y)[8], int i) {
#pragma unroll
                for (int k = 0; k < 8; ++k) {
                    const float w = MODE == kResUniform ? cur.wuni : wbuf[2 * i + (k >> 2)][k & 3];
#pragma unroll
                    for (int r = 0; r < R; ++r) acc[r] = __builtin_fmaf(w, y[k][r], acc[r]);
                }
            };
            if constexpr (MODE != kResParts) {
                T y[2][8];  // a chunk's values are asked for before the chunk before is added up
                read(y[0], cbuf[0]);
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    if (i < 3) read(y[(i + 1) & 1], cbuf[i + 1]);
                    add(y[i & 1], i);
                    fetch(ahead, i, i);
                }
                sum = acc;
            } else {
                // Two chunks per turn, as in resident_kernel.  (Four, so that more is on its way: 1500 neurons of 0 to 40
                // connections, 12 layers, 300 rows 71 -> 79 us, for all that is fetched in vain.)
                uint32_t off = 0;  // of the part of 32 connections that the next two chunks are of
                for (int c = 0; c == 0 || c < it.nch; c += 2) {
                    const bool last = c + 2 >= it.nch;
                    if (c & 2) off += fa.part_stride;
                    const uint32_t half = last || (c & 2) ? 0u : 2u;  // the next chunks' place in their part
                    const Item from = last ? Item{ahead.c, ahead.w, 0} : Item{it.c + off, it.w + off, 0};
#pragma unroll
                    for (int i = 0; i < 2; ++i) {
                        if (c + i < it.nch) {
                            T y[8];
                            read(y, cbuf[i]);
                            add(y, i);
                        }
                        fetch(from, i, half + i);
                    }
                    if (last || (c & 2)) {
                        sum += acc;
                        acc = T{};
                    }
                }
            }
            const float bj = mine ? bias_j : -__builtin_inff();  // lanes without a neuron have no output
#pragma unroll
            for (int r = 0; r < R; ++r) {
                sum[r] = fminf(fmaxf(sum[r] + bj, 0.0f), kClip);
                if (__builtin_amdgcn_ballot_w64(sum[r] > 0.0f) != 0ull) pos |= 1u << r;
            }
            uint32_t to = entry(j, q) + to_copy;
            asm volatile("" : "+v"(to));  // (or its load would be moved behind the branch, and wait for all that were asked for since)
            if (mine) {
                *(lds_T*)to = sum;
                if constexpr (TWICE) *(lds_T*)(to + PLANE) = sum;
            }
        }
        cur = nxt;
        nxt = after;
        live &= __builtin_amdgcn_readfirstlane(raised);
        if (tid == 0) {
            if (fa.layer_rows && l > fa.l0 && live) atomicAdd(&fa.layer_rows[l], __popc(live));
            live_word[(l + 1) % 3] = 0u;
        }
        // (a plain LDS operation of one lane: the compiler's atomic would look for the first active lane on its own)
        if (lane == 0) asm volatile("ds_or_b32 %0, %1" ::"v"(live_at + 4u * (uint32_t)(l % 3)), "v"(pos) : "memory");
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __syncthreads();
    };
    int l = fa.l0;
    while (l < fa.l1 && live) {
        layer(l++, std::false_type{});
        other = true;
        if (l == fa.l1 || !live) break;
        layer(l++, std::true_type{});
        other = false;
    }
    if (live) live &= __builtin_amdgcn_readfirstlane(live_word[(l + 2) % 3]);  // the last layer's
    if (tid == 0 && live && fa.layer_rows) atomicAdd(&fa.layer_rows[l], __popc(live));
    // What is needed only now is read again (the kernel's first argument): kept over the layers these would be scalar registers
    // too many, and every layer would fetch others back from vector registers.
    using cargs = const __attribute__((address_space(4))) FewArgs;
    cargs* late = (cargs*)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(late));
    float* const Yout = late->Yout;
    int* const rows_out = late->rows_out;
    if (rows_out) {
        if (tid < R && ((live >> tid) & 1u)) rows_out[__popc(live & ((1u << tid) - 1u))] = late->row_offset + tid;
        if (tid == 0) __hip_atomic_store(late->host_count, __popc(live), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    } else if (tid < nrow) {
        late->flags[row0 + tid] = (live >> tid) & 1u;
    }
    if (!live || !Yout) return;
    gu32* q_out = (gu32*)(uintptr_t)nxt.qsel;
    for (int t = tid; t < n4; t += T_) {
        const uint32_t q = q_out[t];
        T e[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) e[i] = *(const lds_T*)(entry(4 * t + i, q) + (other ? copy : 0u));
#pragma unroll
        for (int r = 0; r < R; ++r)
            if ((live >> r) & 1u) {
                const int to = rows_out ? __popc(live & ((1u << r) - 1u)) : row0 + r;
                *reinterpret_cast<f32x4*>(Yout + (size_t)to * N + 4 * (size_t)t) = f32x4{e[0][r], e[1][r], e[2][r], e[3][r]};
            }
    }
}

// blockDim.x = 64 * W, W = min(16, U), U = ceil(N / 64) groups of 64 neurons; wave w owns the groups w, w + W, ...
template <int MODE>
__global__ __launch_bounds__(kBlk) void few_kernel(FewArgs fa, const float* __restrict__ Yin, const float* __restrict__ bias, int N) {
    // The entry codes are addresses from the start of the workgroup's LDS: everything is dynamic, nothing static.
    extern __shared__ __align__(16) char few_lds[];
    char* misc = few_lds + res_tile_bytes(N, 1 << fa.planes_log2);
    uint32_t* live_word = reinterpret_cast<uint32_t*>(misc);    // [3], raised by the layers in turn
    int* row_at = reinterpret_cast<int*>(misc + 16);            // [4] slots of my rows
    int* kept = row_at + kFewRows;                              // flags set
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int nwg = gridDim.x;
    int A = fa.A;
    const auto rows_per = [&](int a) { return (a + nwg - 1) / nwg; };  // 1 to 4: a is at most kFewRows * nwg
    if (tid < 3) live_word[tid] = 0u;
    if (fa.flags_prev) {  // at most kFewCount flags: a wave counts and numbers them all
        if (wave == 0) {
            uint32_t f[4] = {0u, 0u, 0u, 0u};
            if (16 * lane < fa.A) {
                const uint4 v = flags16(fa.flags_prev, 16 * lane, fa.A);
                f[0] = v.x; f[1] = v.y; f[2] = v.z; f[3] = v.w;
            }
            const int mine = __popc(f[0]) + __popc(f[1]) + __popc(f[2]) + __popc(f[3]);
            int upto = mine;
#pragma unroll
            for (int d = 1; d < 64; d <<= 1) {
                const int before = __shfl_up(upto, d, 64);
                if (lane >= d) upto += before;
            }
            const int total = __builtin_amdgcn_readlane(upto, 63), per = rows_per(total);
            const int r0 = (int)blockIdx.x * per;
            int rank = upto - mine;
#pragma unroll
            for (int i = 0; i < 16; ++i)
                if ((f[i >> 2] >> (8 * (i & 3))) & 1u) {
                    if (rank >= r0 && rank < r0 + per) {
                        row_at[rank - r0] = 16 * lane + i;
                        fa.gid[rank] = fa.row_offset + 16 * lane + i;
                    }
                    ++rank;
                }
            if (lane == 0) *kept = total;
        }
        __syncthreads();
        A = __builtin_amdgcn_readfirstlane(*kept);
        if (blockIdx.x == 0 && tid == 0) *fa.count = A;
    } else {
        __syncthreads();
    }
    const int R = rows_per(A);
    if ((int)blockIdx.x * R >= A) return;
    const int* at = fa.flags_prev ? row_at : nullptr;
    if (R == 1) few_layers<1, MODE>(fa, Yin, bias, N, A, at, live_word);
    else if (R == 2) few_layers<2, MODE>(fa, Yin, bias, N, A, at, live_word);
    else if (R == 3) few_layers<3, MODE>(fa, Yin, bias, N, A, at, live_word);
    else few_layers<4, MODE>(fa, Yin, bias, N, A, at, live_word);
}

}  // namespace spdnn
