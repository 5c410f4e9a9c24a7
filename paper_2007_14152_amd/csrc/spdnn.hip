// Host side of the spdnn C-ABI (see include/spdnn.h): argument checks, arena
// carving, weight set-up, and the per-layer launch loop.  Every arithmetic step
// of the inference runs in the kernels of spdnn_kernels.h.
#include "../../include/spdnn.h"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstdarg>
#include <cstdint>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <new>
#include <numeric>
#include <string>
#include <vector>

#include "spdnn_kernels.h"
#include "spdnn_cut.h"
#include "spdnn_profile.h"

// Work memory of spdnn_infer_static, the entry point for callers that cannot allocate: a fixed array in
// every GPU's memory instead of a caller-made work arena.  In host code this name is only a stand-in for
// the symbol; the device address comes from hipGetSymbolAddress (see static_scratch()).
constexpr size_t kStaticScratchBytes = SPDNN_STATIC_SCRATCH_BYTES;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

namespace {

thread_local std::string g_err;

int fail(int code, const char* fmt, ...) {
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    g_err = buf;
    return code;
}

int static_scratch(void** out);  // defined below

#define HIP_TRY(expr)                                                                         \
    do {                                                                                      \
        hipError_t e_ = (expr);                                                               \
        if (e_ != hipSuccess)                                                                 \
            return fail(SPDNN_EHIP, "%s failed: %s (%s:%d)", #expr, hipGetErrorString(e_),    \
                        __FILE__, __LINE__);                                                  \
    } while (0)

constexpr size_t kAlign = 256;
inline size_t up(size_t x) { return (x + kAlign - 1) / kAlign * kAlign; }

// Columns of the rows of strided_kernel.  Most: two of them fit the LDS.  Fewest: a layer takes it 1.6 us (orbits of 32) to 3.2
// however few the rows are, resident_kernel 1.2 (256 columns) to 2.6 (1152).  Deep networks on few rows, resident_kernel ->
// strided_kernel, 200 layers of stride 1, 60 and 500 rows: 512 columns 287 -> 650 and 285 -> 586 us, 1024 411 -> 645 and 417 ->
// 584, 1088 477 -> 527 and 482 -> 530, 1152 532 -> 527 and 539 -> 530, 1536 (60 layers) 191 -> 178; 60 000 rows, 1 layer: 64 columns
// 52 -> 99, 512 133 -> 150.  (Large batches of 384 columns and more lose by it -- 60 layers of 1024, strides 1 and 32, 60 000 rows 867 ->
// 2510 -- but a choice by the batch would make a row's bits depend on the rows beside it.)
constexpr int32_t kStridedColumns = 16384, kStridedFewest = 1152;
constexpr int kLag = 2;  // the host runs at most this many layers ahead of the GPU
// Set-up of device-resident layers runs on this many streams, a layer per stream in turn: its kernels
// are single-wave, latency-bound searches that fill a fraction of the chip, so several layers overlap.
constexpr int kSetupStreams = 8;

enum LayerMode { kSingle = 0, kStaged = 1, kWide = 2, kPair = 3, kWidePair = 4, kRow2 = 5, kFlat = 6 };
struct LayerDesc {
    spdnn::LayerWeights w;
    spdnn::WideWeights ww;
    spdnn::Row2Weights r2;
    uint16_t* r2_codes = nullptr;  // arena room for the two-row-tile format (NULL: none)
    int32_t* r2_map = nullptr;
    int* r2_ngroups = nullptr;
    // kRow2: one weight for the whole layer, N a multiple of 4096, every 4096-neuron unit's window within 16384
    // columns but wider than one LDS stage: four neurons per lane, two rows per tile (fused_row2_kernel);
    // kSingle: every window fits one LDS stage; kStaged: 2 stages (or fallback); kWide: 3+ stages;
    // kPair: one stage, one weight for the whole layer, two output neurons per lane; kWidePair: the same for 2-8 stages;
    // kFlat: whole rows of at most 16384 columns in LDS (fused_flat_kernel)
    int mode;
    int lds_cols;  // columns the LDS tile must hold for this layer
    float wuni;    // kPair, kWidePair, kRow2, kFlat with one weight: the layer's weight
    bool pair4;    // kWidePair: 2 to 4 stages -> slot lists resident in registers
    bool multi;    // one of several launches of a layer with more than 32 connections per neuron: each computes the
                   // outputs of a slice of the neurons, several lanes per neuron (spdnn::VirtInfo)
    spdnn::VirtInfo virt;
    int virt_lanes = 1;  // multi: lanes of the layer's longest neuron (the layer's passes)
    int virt_blocks = 0;  // multi: workgroups of this launch that have neurons
    bool flat_uniform = false;  // kFlat: one weight for the whole layer
    bool relabel = false;  // kPair under new names for neurons and columns (spdnn::PairRelabel)
    spdnn::PairRelabel rn{};
};

}  // namespace

constexpr int kInEvents = 2 + 3;  // pieces of inputs under way: one per input buffer, and the last batch's other pieces

struct spdnn_model {
    int32_t N = 0, L = 0, nblk = 0, G = 1;
    hipStream_t stream = nullptr;
    int num_cu = 256;
    const float* bias_dev = nullptr;
    std::vector<LayerDesc> layers;     // one per pass (launch); a layer is one pass unless some neuron has more than 32 connections
    std::vector<int32_t> first_pass;   // L+1 entries: layer l is passes first_pass[l] .. first_pass[l+1]-1
    int* host_counts = nullptr;  // pinned, L+2 entries: rows active on entry to layer l; [L + 1]: rows that survive a
                                 // resident_kernel run
    // rows that stay in LDS from layer to layer (resident_kernel): networks of at most 4096 neurons
    const spdnn::ResidentLayer* res_layers = nullptr;  // device copy of the layers' descriptors (NULL: not possible)
    int* res_rows = nullptr;                           // device, L + 1 counters
    int res_mode = spdnn::kResWeights;
    uint32_t res_part_stride = 0;                      // kResParts
    // every layer a strided sum, one bias: strided_kernel
    const spdnn::StridedLayer* strided = nullptr;  // device copy of the layers' descriptors (NULL: not such a network)
    int32_t strided_lanes = 0;                     // lanes a pair of rows takes in the layer that takes most
    float strided_bias = 0.0f;
    bool strided_known = false;  // all strides are among those that strided_kernel has code of its own for
    // out-of-core weights: pass p's block lives in host memory and is copied into device slot p & 1
    const char* ooc_host = nullptr;
    char* ooc_slot[2] = {nullptr, nullptr};
    size_t ooc_block = 0;
    hipStream_t ooc_stream = nullptr;
    hipEvent_t ooc_ready[2] = {nullptr, nullptr};  // the copy into the slot has landed
    hipEvent_t ooc_freed[2] = {nullptr, nullptr};  // the kernels that read the slot are done
    // inputs in host memory (spdnn_infer_host): copy stream and "batch has landed" events, made on first use
    hipStream_t in_stream = nullptr;
    hipEvent_t in_ready[kInEvents] = {};
    int32_t launches = 0, res_launches = 0;  // of fused kernels in the last inference; among them of those that keep rows on the chip
    int32_t row_kernel = SPDNN_ROWS_NONE;    // ... and which of these was the last
    // profiling
    int profiling = 0;
    std::vector<hipEvent_t> t0, t1;
    int32_t prof_layers = 0;
    std::vector<float> prof_ms;
    std::vector<int32_t> prof_rows;
};

namespace {

bool valid_n(int32_t N) { return N >= 32 && N <= 65536 && (N % 4) == 0; }

size_t layer_bytes(int32_t nblk) {
    const size_t e = (size_t)nblk * spdnn::kNnz * spdnn::kBlk;
    return up((size_t)nblk * sizeof(int2)) + up(e * sizeof(uint16_t)) + up(e * sizeof(float)) +
           up((size_t)nblk * spdnn::kBlk * sizeof(uint32_t)) +
           // several lanes per neuron: slots, steps per wave, neurons per workgroup, slots per neuron
           up((size_t)nblk * spdnn::kBlk * sizeof(uint16_t)) + up((size_t)nblk * 16) + up((size_t)nblk * sizeof(int2)) +
           up((size_t)nblk * spdnn::kBlk * sizeof(uint32_t));
}
int stages_of(int32_t window) { return (window + spdnn::kCap - 1) / spdnn::kCap; }
// extra bytes per layer for the wide format with up to `nstage` stages (0 if not needed)
// Steps per neuron the wide format needs at most, for a layer of 2 .. nstage stages (an
// arena sized for nstage stages also holds layers with fewer, which may use more steps per stage).
size_t wide_steps_max(int nstage) {
    size_t m = 0;
    for (int n = 2; n <= nstage; ++n) m = std::max(m, (size_t)n * spdnn::wide_steps(n));
    return m;
}
bool wide_has_slots(int nstage) { return nstage <= 8; }  // the compact 16-bit form exists for 2..8 stages
// the two-row-tile format (fused_row2_kernel): step codes, gathered-footprint list, groups per unit
size_t row2_bytes(int32_t nblk) {
    if (nblk % 4) return 0;
    const size_t nunit = nblk / 4;
    return up((size_t)nblk * spdnn::kBlk * spdnn::kNnz * sizeof(uint16_t)) +
           up(nunit * (spdnn::kRow2Cols / 4) * sizeof(int32_t)) + up(nunit * sizeof(int));
}
size_t wide_bytes(int32_t nblk, int nstage) {
    if (nstage < 2) return 0;
    const size_t e = (size_t)nblk * wide_steps_max(nstage) * spdnn::kBlk;
    const size_t sp = (size_t)nblk * spdnn::kSpill * spdnn::kBlk;
    return up(e * sizeof(uint2)) + up((size_t)nblk * nstage * 16) + up(sp * sizeof(uint16_t)) +
           up(sp * sizeof(float)) + up((size_t)nblk * 16) +
           (wide_has_slots(nstage) ? up(e * sizeof(uint16_t)) + up(sp * sizeof(uint16_t))
                                   : 0) +  // compact slots and spills
           row2_bytes(nblk);
}
size_t staging_bytes(int32_t N, int32_t L) {
    const int32_t nblk = (N + spdnn::kBlk - 1) / spdnn::kBlk;
    const size_t lanes = (size_t)nblk * spdnn::kBlk;  // rows of the staging arrays: the lanes of a launch
    return up(lanes * spdnn::kNnz * sizeof(int32_t)) + up(lanes * spdnn::kNnz * sizeof(float)) + up(lanes) +
           kSetupStreams * up((size_t)nblk * spdnn::kCap * sizeof(uint16_t)) +  // column -> LDS slot tables of the layers being set up
           up(sizeof(int) * (size_t)nblk) +                     // general layers: smallest column of every block
           up(sizeof(int) * (size_t)(5 * L + 1));  // error flag; per layer: wide failure, widest window, weights differ, pair info[2]
}
size_t block_bytes(int32_t N, int nstage_cap) {  // one pass's re-laid weights
    const int32_t nblk = (N + spdnn::kBlk - 1) / spdnn::kBlk;
    return layer_bytes(nblk) + wide_bytes(nblk, nstage_cap);
}
size_t res_bytes(int32_t L) {  // resident_kernel: the layers' descriptors and the rows-per-layer counters
    return up((size_t)L * sizeof(spdnn::ResidentLayer)) + up(((size_t)L + 1) * sizeof(int));
}
size_t arena_bytes_for(int32_t N, int32_t L, int nstage_cap) {
    return up((size_t)N * sizeof(float)) + (size_t)L * block_bytes(N, nstage_cap) + staging_bytes(N, L) + res_bytes(L);
}
// out-of-core: the device holds the bias, two blocks and the staging area; the host holds all blocks
size_t ooc_device_bytes_for(int32_t N, int32_t L, int nstage_cap) {
    return up((size_t)N * sizeof(float)) + 2 * block_bytes(N, nstage_cap) + staging_bytes(N, L);
}

struct WorkView {
    float* Y[2];
    int* cat[2];        // layer l writes and reads cat[l & 1]: slots, in layer l-1's buffer, of the rows active on entry
    int* gid[2];        // gid[l & 1]: their original row numbers (derived from gid[(l + 1) & 1], layer l-1's)
    uint8_t* flags[3];  // one byte per row; layer l raises flags[l % 3], reads flags[(l + 2) % 3] (layer l-1's) and
                        // clears flags[(l + 1) % 3] for layer l+1
    int* count[2];      // count[l & 1]: rows active on entry to layer l, written by layer l's kernel
};
size_t carve_work(int32_t N, int32_t batch, char* base, WorkView* v) {
    size_t o = 0;
    const size_t yb = up((size_t)batch * N * sizeof(float));
    const size_t lb = up(((size_t)batch + 4) * sizeof(int));  // lists are read 4 entries at a time
    for (int i = 0; i < 2; ++i) {
        if (v) v->Y[i] = reinterpret_cast<float*>(base + o);
        o += yb;
    }
    for (int i = 0; i < 2; ++i) {
        if (v) v->cat[i] = reinterpret_cast<int*>(base + o);
        o += lb;
    }
    for (int i = 0; i < 2; ++i) {
        if (v) v->gid[i] = reinterpret_cast<int*>(base + o);
        o += lb;
    }
    const size_t fb = up((size_t)batch + 16);  // flags are read 16 bytes at a time
    for (int i = 0; i < 3; ++i) {
        if (v) v->flags[i] = reinterpret_cast<uint8_t*>(base + o);
        o += fb;
    }
    for (int i = 0; i < 2; ++i) {
        if (v) v->count[i] = reinterpret_cast<int*>(base + o);
        o += kAlign;
    }
    return o;
}

constexpr int kVirtLds = 2 * spdnn::kBlk * 16;  // two sets of slots for the lanes' sums (spdnn::VirtInfo)
template <bool MULTI, bool VIRT, bool WHOLE = false>
hipError_t allow_big_lds() {
    return hipFuncSetAttribute(reinterpret_cast<const void*>(&spdnn::fused_layer_kernel<MULTI, VIRT, WHOLE>),
                               hipFuncAttributeMaxDynamicSharedMemorySize,
                               (int)spdnn::tile_pair_bytes(spdnn::kCap) + (VIRT ? kVirtLds : 0));
}
template <int R>
hipError_t allow_flat_lds() {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&spdnn::fused_flat_kernel<R, false>),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, spdnn::flat_lds_bytes(R));
    return e != hipSuccess ? e : hipFuncSetAttribute(reinterpret_cast<const void*>(&spdnn::fused_flat_kernel<R, true>),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, spdnn::flat_lds_bytes(R));
}
constexpr int kLdsBytes = 160 * 1024;
template <bool PAIRS, bool KNOWN>
hipError_t allow_strided_lds() {
    const void* const both[2] = {reinterpret_cast<const void*>(&spdnn::strided_kernel<PAIRS, KNOWN, false>),
                                 reinterpret_cast<const void*>(&spdnn::strided_kernel<PAIRS, KNOWN, true>)};
    const hipError_t e = hipFuncSetAttribute(both[0], hipFuncAttributeMaxDynamicSharedMemorySize, kLdsBytes);
    return e != hipSuccess ? e : hipFuncSetAttribute(both[1], hipFuncAttributeMaxDynamicSharedMemorySize, kLdsBytes);
}
int few_lds(int32_t N, int32_t nblk) {
    return (int)spdnn::res_tile_bytes(N, 1 << spdnn::res_planes_log2(nblk)) + spdnn::kFewMiscBytes;
}
hipError_t allow_few_lds() {
    for (const void* f : {reinterpret_cast<const void*>(&spdnn::few_kernel<spdnn::kResWeights>),
                          reinterpret_cast<const void*>(&spdnn::few_kernel<spdnn::kResUniform>),
                          reinterpret_cast<const void*>(&spdnn::few_kernel<spdnn::kResParts>)}) {
        const hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, few_lds(spdnn::kCap, 4));
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}
template <int NB, int PM>
hipError_t allow_resident_lds(int bytes) {
    for (const void* f : {reinterpret_cast<const void*>(&spdnn::resident_kernel<NB, PM, spdnn::kResWeights>),
                          reinterpret_cast<const void*>(&spdnn::resident_kernel<NB, PM, spdnn::kResUniform>),
                          reinterpret_cast<const void*>(&spdnn::resident_kernel<NB, PM, spdnn::kResParts>)}) {
        const hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// The fused kernels and set-up kernels use more dynamic LDS than the default limit allows.
int allow_large_lds() {
    constexpr size_t wide_lds = spdnn::kOrderThreads * sizeof(spdnn::WideScratch);
    const int tile_lds = (int)spdnn::tile_pair_bytes(spdnn::kCap);
    HIP_TRY(allow_few_lds());
    HIP_TRY((allow_strided_lds<false, false>()));
    HIP_TRY((allow_strided_lds<true, false>()));
    HIP_TRY((allow_strided_lds<false, true>()));
    HIP_TRY((allow_strided_lds<true, true>()));
    HIP_TRY((allow_big_lds<false, false>()));
    HIP_TRY((allow_big_lds<true, false>()));
    HIP_TRY((allow_big_lds<false, true>()));
    HIP_TRY((allow_big_lds<true, true>()));
    HIP_TRY((allow_big_lds<false, false, true>()));
    HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void*>(&spdnn::wide_pack_kernel),
                                hipFuncAttributeMaxDynamicSharedMemorySize, (int)wide_lds));
    HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void*>(&spdnn::balance_kernel<1>),
                                hipFuncAttributeMaxDynamicSharedMemorySize, (int)sizeof(spdnn::BalanceScratch<1>)));
    HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void*>(&spdnn::balance_kernel<2>),
                                hipFuncAttributeMaxDynamicSharedMemorySize, (int)sizeof(spdnn::BalanceScratch<2>)));
    HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void*>(&spdnn::fused_pair_kernel<false>),
                                hipFuncAttributeMaxDynamicSharedMemorySize, tile_lds));
    HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void*>((&spdnn::fused_pair_kernel<false, true>)),
                                hipFuncAttributeMaxDynamicSharedMemorySize, tile_lds));
    HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void*>(&spdnn::fused_pair_kernel<true>),
                                hipFuncAttributeMaxDynamicSharedMemorySize, tile_lds));
    HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void*>(&spdnn::fused_wide_pair_kernel),
                                hipFuncAttributeMaxDynamicSharedMemorySize, tile_lds + spdnn::kPadLds));
    HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void*>(&spdnn::fused_wide_pair4_kernel<4, 16>),
                                hipFuncAttributeMaxDynamicSharedMemorySize, tile_lds + spdnn::kPair4LdsExtra));
    HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void*>(&spdnn::fused_wide_pair4_kernel<2, 32>),
                                hipFuncAttributeMaxDynamicSharedMemorySize, tile_lds + spdnn::kPair4LdsExtra));
    HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void*>(&spdnn::fused_row2_kernel),
                                hipFuncAttributeMaxDynamicSharedMemorySize, spdnn::kRow2LdsBytes));
    HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void*>(&spdnn::fused_wide_kernel<16>),
                                hipFuncAttributeMaxDynamicSharedMemorySize, tile_lds));
    HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void*>(&spdnn::fused_wide_kernel<8>),
                                hipFuncAttributeMaxDynamicSharedMemorySize, tile_lds));
    HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void*>(&spdnn::balance_kernel<4>),
                                hipFuncAttributeMaxDynamicSharedMemorySize, (int)sizeof(spdnn::BalanceScratch<4>)));
    const int res_lds = (int)spdnn::res_tile_bytes(spdnn::kCap, 2) + spdnn::kResMiscBytes + 4 * spdnn::kCap;
    HIP_TRY((allow_flat_lds<1>()));
    HIP_TRY((allow_flat_lds<2>()));
    HIP_TRY((allow_flat_lds<3>()));
    HIP_TRY((allow_flat_lds<4>()));
    HIP_TRY((allow_resident_lds<1, 4>(res_lds)));
    HIP_TRY((allow_resident_lds<2, 4>(res_lds)));
    HIP_TRY((allow_resident_lds<4, 2>(res_lds)));
    return SPDNN_OK;
}

// Longest neuron of every layer of a general model -> passes of 32 connections; with idx also the
// widest column window of any 1024-neuron block (of any aligned pair of blocks when N is a multiple
// of 2048, as spdnn_scan_windows counts).  scratch: device, 8*L + 8*ceil(N/1024) bytes.
int scan_csr(int32_t N, int32_t L, const int32_t* const* ptr, void* scratch_dev, size_t scratch_bytes,
             hipStream_t stream, std::vector<int32_t>* passes_of, const int32_t* const* idx = nullptr,
             int32_t* widest_window = nullptr) {
    const int32_t nblk = (N + spdnn::kBlk - 1) / spdnn::kBlk;
    const size_t need = sizeof(int) * 2 * (size_t)L + sizeof(int2) * (size_t)nblk;
    if (scratch_bytes < need) return fail(SPDNN_ESIZE, "scratch has %zu bytes, %zu needed", scratch_bytes, need);
    if (reinterpret_cast<uintptr_t>(scratch_dev) % 8) return fail(SPDNN_EINVAL, "scratch must be 8-byte aligned");
    int* out = static_cast<int*>(scratch_dev);
    int2* win = reinterpret_cast<int2*>(out + 2 * (size_t)L);
    HIP_TRY(hipMemsetAsync(out, 0, sizeof(int) * 2 * (size_t)L, stream));
    for (int32_t l = 0; l < L; ++l) {
        if (!ptr[l]) return fail(SPDNN_EINVAL, "ptr[%d] is NULL", l);
        spdnn::csr_scan_kernel<<<(N + 255) / 256, 256, 0, stream>>>(ptr[l], N, out + 2 * l);
    }
    HIP_TRY(hipGetLastError());
    std::vector<int> h(2 * (size_t)L);
    HIP_TRY(hipMemcpyAsync(h.data(), out, sizeof(int) * h.size(), hipMemcpyDeviceToHost, stream));
    HIP_TRY(hipStreamSynchronize(stream));
    passes_of->assign((size_t)L, 1);
    for (int32_t l = 0; l < L; ++l) {
        if (h[2 * l + 1]) return fail(SPDNN_EINVAL, "ptr[%d] is negative somewhere or decreases", l);
        // parts of 32 connections per neuron, rounded up to a power of two (lanes per neuron)
        const int parts = std::max(1, (h[2 * l] + spdnn::kNnz - 1) / spdnn::kNnz);
        int p2 = 1;
        while (p2 < parts) p2 *= 2;
        if (p2 > spdnn::kBlk / 4)
            return fail(SPDNN_EINVAL, "layer %d has a neuron of %d connections; at most %d are supported", l, h[2 * l],
                        spdnn::kNnz * spdnn::kBlk / 4);
        (*passes_of)[l] = p2;
    }
    if (idx && widest_window) {  // after the ptr arrays are known to be sound
        std::vector<int2> hw(nblk);
        int widest = 4;
        for (int32_t l = 0; l < L; ++l) {
            if (!idx[l]) return fail(SPDNN_EINVAL, "idx[%d] is NULL", l);
            spdnn::csr_block_window_kernel<<<nblk, spdnn::kBlk, 0, stream>>>(ptr[l], idx[l], N, win);
            HIP_TRY(hipGetLastError());
            HIP_TRY(hipMemcpyAsync(hw.data(), win, sizeof(int2) * nblk, hipMemcpyDeviceToHost, stream));
            HIP_TRY(hipStreamSynchronize(stream));
            for (int32_t b = 0; b < nblk; ++b) {
                const int lo = hw[b].x & ~3;  // windows start at a multiple of 4 columns
                widest = std::max(widest, (hw[b].x + hw[b].y - lo + 3) & ~3);
            }
            if (N % (2 * spdnn::kBlk) == 0)
                for (int32_t b = 0; b + 1 < nblk; b += 2) {
                    if (!hw[b].y || !hw[b + 1].y) continue;
                    const int lo = std::min(hw[b].x, hw[b + 1].x) & ~3;
                    const int hi = std::max(hw[b].x + hw[b].y, hw[b + 1].x + hw[b + 1].y);
                    widest = std::max(widest, (hi - lo + 3) & ~3);
                }
        }
        *widest_window = widest;
    }
    return SPDNN_OK;
}

// resident_kernel: the most groups of 64 neurons a wave owns -- one if there is at most a quad of rows per CU and
// sixteen waves can own all there are -- and the workgroup's waves.
int resident_groups_per_wave(int32_t nblk, bool few_rows) { return nblk > 2 ? 4 : nblk == 1 && few_rows ? 1 : 2; }
int resident_waves(int32_t N, int nb) { return ((N + 63) / 64 + nb - 1) / nb; }

// Set-up shared by spdnn_create (ptr == NULL: every layer is [N][32]) and spdnn_create_csr
// (device arrays; layer l is cut into passes_of[l] passes of 32 connections per neuron).
int create_impl(spdnn_t* out, int32_t N, int32_t L, const std::vector<int32_t>& passes_of, const int32_t* const* ptr,
                const int32_t* const* idx, const float* const* val, const float* bias, int32_t where,
                void* weights_arena, size_t weights_arena_bytes, hipStream_t stream, void* host_arena = nullptr,
                size_t host_arena_bytes = 0) {
    const bool ooc = host_arena != nullptr;
    int32_t P = 0;  // passes = layers as the kernels see them
    std::vector<int32_t> layer_of, round_of, first_pass((size_t)L + 1, 0);
    for (int32_t l = 0; l < L; ++l) {
        first_pass[l] = P;
        for (int32_t r = 0; r < passes_of[l]; ++r) {
            layer_of.push_back(l);
            round_of.push_back(r);
        }
        P += passes_of[l];
    }
    first_pass[L] = P;
    // The arena decides how many stages the wide format may use (0 = none: layers with
    // wide windows then run the staged kernel, which is slower but needs no extra room).
    auto fits = [&](int cap) {
        return ooc ? ooc_device_bytes_for(N, P, cap) <= weights_arena_bytes &&
                         (size_t)P * block_bytes(N, cap) <= host_arena_bytes
                   : arena_bytes_for(N, P, cap) <= weights_arena_bytes;
    };
    int nstage_cap = stages_of(N);
    while (nstage_cap > 1 && !fits(nstage_cap)) --nstage_cap;
    if (nstage_cap < 2) nstage_cap = 0;
    if (!fits(nstage_cap)) {
        if (ooc)
            return fail(SPDNN_ESIZE, "out-of-core arenas have %zu (device) and %zu (host) bytes, at least %zu and %zu needed",
                        weights_arena_bytes, host_arena_bytes, ooc_device_bytes_for(N, P, 0),
                        (size_t)P * block_bytes(N, 0));
        return fail(SPDNN_ESIZE, "weights arena has %zu bytes, at least %zu needed", weights_arena_bytes,
                    arena_bytes_for(N, P, 0));
    }

    const int32_t nblk = (N + spdnn::kBlk - 1) / spdnn::kBlk;

    // bias: must be <= 0 everywhere, otherwise a dropped (all-zero) row would not stay zero
    std::vector<float> hb(N);
    if (where == SPDNN_HOST) {
        std::memcpy(hb.data(), bias, sizeof(float) * N);
    } else {
        // on the model's stream: the caller may have produced the bias there
        HIP_TRY(hipMemcpyAsync(hb.data(), bias, sizeof(float) * N, hipMemcpyDeviceToHost, stream));
        HIP_TRY(hipStreamSynchronize(stream));
    }
    for (int32_t j = 0; j < N; ++j)
        if (!(hb[j] <= 0.0f) || !std::isfinite(hb[j]))
            return fail(SPDNN_EBIAS, "bias[%d] = %g: every bias must be finite and <= 0", j, (double)hb[j]);

    spdnn_model* m = new (std::nothrow) spdnn_model;
    if (!m) return fail(SPDNN_EHIP, "out of host memory");
    struct Guard {
        spdnn_model* m;
        ~Guard() {
            if (m) spdnn_destroy(m);
        }
    } guard{m};

    m->N = N;
    m->L = L;
    m->first_pass = first_pass;
    m->nblk = nblk;
    m->G = (nblk % 4 == 0) ? 4 : (nblk % 3 == 0) ? 3 : (nblk % 2 == 0) ? 2 : 1;
    m->stream = stream;
    int dev = 0;
    HIP_TRY(hipGetDevice(&dev));
    hipDeviceProp_t prop;
    HIP_TRY(hipGetDeviceProperties(&prop, dev));
    m->num_cu = prop.multiProcessorCount > 0 ? prop.multiProcessorCount : 256;
    if (allow_large_lds() != SPDNN_OK) return SPDNN_EHIP;
    {  // set-up is also where this device's copy of the static scratch array is looked up
        void* unused = nullptr;
        if (static_scratch(&unused) != SPDNN_OK) return SPDNN_EHIP;
    }
    constexpr size_t wide_lds = spdnn::kOrderThreads * sizeof(spdnn::WideScratch);
    HIP_TRY(hipHostMalloc(reinterpret_cast<void**>(&m->host_counts), sizeof(int) * (size_t)(L + 2),  // [L + 1]: see infer_impl
                          hipHostMallocDefault));

    // carve the arena: bias | P x (win, rel, val) | staging (raw idx, raw val, error flag)
    char* base = static_cast<char*>(weights_arena);
    size_t o = 0;
    float* bias_dev = reinterpret_cast<float*>(base + o);
    o += up((size_t)N * sizeof(float));
    HIP_TRY(hipMemcpyAsync(bias_dev, hb.data(), sizeof(float) * N, hipMemcpyHostToDevice, stream));
    m->bias_dev = bias_dev;
    const size_t e = (size_t)nblk * spdnn::kNnz * spdnn::kBlk;
    std::vector<int2*> win_dev(P);
    m->layers.resize(P);
    const size_t blk_bytes = block_bytes(N, nstage_cap);
    if (ooc) {  // two device slots; pass p is built in slot p & 1 and runs from there
        m->ooc_host = static_cast<const char*>(host_arena);
        m->ooc_block = blk_bytes;
        m->ooc_slot[0] = base + o;
        m->ooc_slot[1] = base + o + blk_bytes;
        HIP_TRY(hipStreamCreateWithFlags(&m->ooc_stream, hipStreamNonBlocking));
        for (int i = 0; i < 2; ++i) {
            HIP_TRY(hipEventCreateWithFlags(&m->ooc_ready[i], hipEventDisableTiming));
            HIP_TRY(hipEventCreateWithFlags(&m->ooc_freed[i], hipEventDisableTiming));
        }
    }
    const size_t blocks_at = o;
    for (int32_t l = 0; l < P; ++l) {
        o = blocks_at + (size_t)(ooc ? (l & 1) : l) * blk_bytes;
        int2* win = reinterpret_cast<int2*>(base + o);
        o += up((size_t)nblk * sizeof(int2));
        uint16_t* rel = reinterpret_cast<uint16_t*>(base + o);
        o += up(e * sizeof(uint16_t));
        float* wv = reinterpret_cast<float*>(base + o);
        o += up(e * sizeof(float));
        uint32_t* qsel = reinterpret_cast<uint32_t*>(base + o);
        o += up((size_t)nblk * spdnn::kBlk * sizeof(uint32_t));
        m->layers[l].virt.slot = reinterpret_cast<const uint16_t*>(base + o);
        o += up((size_t)nblk * spdnn::kBlk * sizeof(uint16_t));
        m->layers[l].virt.nb8 = reinterpret_cast<const uint8_t*>(base + o);
        o += up((size_t)nblk * 16);
        m->layers[l].virt.range = reinterpret_cast<const int2*>(base + o);
        o += up((size_t)nblk * sizeof(int2));
        m->layers[l].virt.fin = reinterpret_cast<const uint32_t*>(base + o);
        o += up((size_t)nblk * spdnn::kBlk * sizeof(uint32_t));
        m->layers[l].w = spdnn::LayerWeights{rel, wv, win, qsel, 0};
        win_dev[l] = win;
        spdnn::WideWeights ww{};
        ww.win = win;
        if (nstage_cap >= 2) {  // room for the wide format; the layer's own stage count strides the arrays
            const size_t we = (size_t)nblk * wide_steps_max(nstage_cap) * spdnn::kBlk;
            const size_t sp = (size_t)nblk * spdnn::kSpill * spdnn::kBlk;
            ww.pk = reinterpret_cast<uint2*>(base + o);
            o += up(we * sizeof(uint2));
            ww.nb8 = reinterpret_cast<uint8_t*>(base + o);
            o += up((size_t)nblk * nstage_cap * 16);
            ww.spill_col = reinterpret_cast<uint16_t*>(base + o);
            o += up(sp * sizeof(uint16_t));
            ww.spill_val = reinterpret_cast<float*>(base + o);
            o += up(sp * sizeof(float));
            ww.spill_n = reinterpret_cast<uint8_t*>(base + o);
            o += up((size_t)nblk * 16);
            if (wide_has_slots(nstage_cap)) {
                ww.ps = reinterpret_cast<uint4*>(base + o);
                o += up(we * sizeof(uint16_t));
                ww.sp16 = reinterpret_cast<uint16_t*>(base + o);
                o += up(sp * sizeof(uint16_t));
            }
            if (nblk % 4 == 0) {
                const size_t nunit = nblk / 4;
                m->layers[l].r2_codes = reinterpret_cast<uint16_t*>(base + o);
                o += up((size_t)nblk * spdnn::kBlk * spdnn::kNnz * sizeof(uint16_t));
                m->layers[l].r2_map = reinterpret_cast<int32_t*>(base + o);
                o += up(nunit * (spdnn::kRow2Cols / 4) * sizeof(int32_t));
                m->layers[l].r2_ngroups = reinterpret_cast<int*>(base + o);
                o += up(nunit * sizeof(int));
            }
        }
        m->layers[l].ww = ww;
    }
    o = blocks_at + (size_t)(ooc ? 2 : P) * blk_bytes;
    const size_t lanes = (size_t)nblk * spdnn::kBlk;
    int32_t* st_idx = reinterpret_cast<int32_t*>(base + o);
    o += up(lanes * spdnn::kNnz * sizeof(int32_t));
    float* st_val = reinterpret_cast<float*>(base + o);
    o += up(lanes * spdnn::kNnz * sizeof(float));
    uint8_t* st_len = reinterpret_cast<uint8_t*>(base + o);  // several lanes per neuron: connections of every lane
    o += up(lanes);
    uint16_t* slot_tabs = reinterpret_cast<uint16_t*>(base + o);  // one table per set-up stream
    const size_t slot_tab_elems = up((size_t)nblk * spdnn::kCap * sizeof(uint16_t)) / sizeof(uint16_t);
    o += kSetupStreams * up((size_t)nblk * spdnn::kCap * sizeof(uint16_t));
    int* blockmin = reinterpret_cast<int*>(base + o);
    o += up(sizeof(int) * (size_t)nblk);
    // [0] bad column seen; [1 + p] pass p could not use the wide format; [1 + P + p] pass p's widest window;
    // [1 + 2P + p] pass p has more than one weight value; [1 + 3P + 2p] {two neurons per lane possible, weight bits}
    int* err_dev = reinterpret_cast<int*>(base + o);
    HIP_TRY(hipMemsetAsync(err_dev, 0, sizeof(int) * (size_t)(5 * P + 1), stream));
    o += up(sizeof(int) * (size_t)(5 * P + 1));
    spdnn::ResidentLayer* res_layers_dev = reinterpret_cast<spdnn::ResidentLayer*>(base + o);  // (not with out-of-core weights)
    o += up((size_t)P * sizeof(spdnn::ResidentLayer));
    int* res_rows_dev = reinterpret_cast<int*>(base + o);

    // Layers that are already on the device and need no staging are set up on several streams in turn.
    struct SetupStreams {
        hipStream_t s[kSetupStreams] = {};
        hipEvent_t start = nullptr;
        int n = 1;
        ~SetupStreams() {
            for (int i = 1; i < n; ++i)
                if (s[i]) (void)hipStreamDestroy(s[i]);
            if (start) (void)hipEventDestroy(start);
        }
    } ss;
    ss.s[0] = stream;
    if (!ptr && where == SPDNN_DEVICE && !ooc && P > 1) {
        HIP_TRY(hipEventCreateWithFlags(&ss.start, hipEventDisableTiming));
        HIP_TRY(hipEventRecord(ss.start, stream));  // bias and cleared flags are in place
        for (int i = 1; i < kSetupStreams; ++i) {
            HIP_TRY(hipStreamCreateWithFlags(&ss.s[i], hipStreamNonBlocking));
            ss.n = i + 1;
            HIP_TRY(hipStreamWaitEvent(ss.s[i], ss.start, 0));
        }
    }

    // Do rows stay in LDS from layer to layer (resident_kernel)?  General layers, not all of them of exactly 32
    // connections per neuron: neurons by length (kResParts), unless they are too uneven for a lane per neuron.
    bool resident = N <= spdnn::kCap && !ooc;
    bool parts = false;
    std::vector<int32_t> hp((size_t)N + 1);
    std::vector<std::vector<uint16_t>> perm;  // kResParts, per layer: order_by_length()
    std::vector<std::vector<uint32_t>> nch;
    if (ptr && resident) {
        double uneven = 0.0;
        perm.resize((size_t)L);
        nch.resize((size_t)L);
        for (int32_t ll = 0; ll < L; ++ll) {
            HIP_TRY(hipMemcpyAsync(hp.data(), ptr[ll], sizeof(int32_t) * hp.size(), hipMemcpyDeviceToHost, stream));
            HIP_TRY(hipStreamSynchronize(stream));
            for (int32_t j = 0; j < N && !parts; ++j) parts = hp[j + 1] - hp[j] != spdnn::kNnz;
            spdnn::order_by_length(hp.data(), N, nblk * spdnn::kBlk, resident_waves(N, resident_groups_per_wave(nblk, false)), perm[ll], nch[ll]);
            uneven += spdnn::uneven_chunks(hp.data(), N, nch[ll], resident_waves(N, resident_groups_per_wave(nblk, true)));
        }
        // A single layer of at most 32 connections per neuron: what one_by_one() says of one layer, for any batch (the
        // layouts differ).  8 to 32 connections, 30 000 rows: 2048 neurons 319 -> 253 us, 4096 600 -> 472; 100 rows 48 ->
        // 54, 53 -> 55.
        // (The offsets of a neuron's parts are 32-bit numbers: at most 256 passes of about 1 MB.)
        if (uneven > 0.0 || (parts && P == 1 && (nblk == 2 || nblk == 4))) resident = parts = false;
    }

    const size_t raw = (size_t)N * spdnn::kNnz;
    // A network of strided sums?  Looked at layer by layer until one is not.  (The descriptors and the rows-per-layer counters
    // take the place of the staged weights, which is free once the set-up is over.)
    std::vector<spdnn::StridedLayer> strided;
    bool all_strided = !ptr && N >= kStridedFewest && N <= kStridedColumns && std::all_of(hb.begin(), hb.end(), [&](float b) { return b == hb[0]; }) &&
                       (size_t)L * (sizeof(spdnn::StridedLayer) + sizeof(int)) + sizeof(int) <= lanes * spdnn::kNnz * sizeof(float);
    std::vector<int2> hw((size_t)P * nblk);
    std::vector<int2> virt_ranges;  // several lanes per neuron: {first neuron, neurons} of the current layer's workgroups
    for (int32_t l = 0; l < P; ++l) {  // l = pass; it belongs to layer ll
        hipStream_t stream = ss.s[l % ss.n];  // everything of this pass goes to one stream
        uint16_t* slot_tab = slot_tabs + (size_t)(l % ss.n) * slot_tab_elems;
        const int32_t ll = layer_of[l];
        const int32_t* di = idx[ll];
        const float* dv = val[ll];
        LayerDesc& d = m->layers[l];
        d.multi = passes_of[ll] > 1;
        if (parts) {
            const int32_t r = round_of[l], first = l - r;  // the layer's tables are under its first pass
            uint16_t* perm_dev = const_cast<uint16_t*>(m->layers[first].virt.slot);
            const int nlanes = nblk * spdnn::kBlk;
            if (r == 0) {
                HIP_TRY(hipMemcpyAsync(perm_dev, perm[ll].data(), sizeof(uint16_t) * perm[ll].size(), hipMemcpyHostToDevice, stream));
                HIP_TRY(hipMemcpyAsync(const_cast<uint32_t*>(d.virt.fin), nch[ll].data(), sizeof(uint32_t) * nch[ll].size(), hipMemcpyHostToDevice, stream));
            }
            spdnn::csr_part_kernel<<<(unsigned)((size_t)nlanes * spdnn::kNnz / 256), 256, 0, stream>>>(ptr[ll], idx[ll], val[ll], perm_dev, nlanes, r,
                                                                                                 st_idx, st_val, st_len);
            int* widest_dev = err_dev + 1 + P + l;
            int* pair_dev = err_dev + 1 + 3 * P + 2 * l;
            spdnn::block_window_kernel<<<nblk, spdnn::kBlk, 0, stream>>>(st_idx, N, win_dev[l], err_dev, widest_dev, st_val,
                                                                         err_dev + 1 + 2 * P + l, nlanes);
            spdnn::whole_row_window_kernel<<<1, 64, 0, stream>>>(win_dev[l], const_cast<int2*>(d.virt.range), nblk, N, widest_dev);
            d.w.planes_log2 = spdnn::res_planes_log2(nblk);
            int pair_info[2] = {0, 0};
            if (r == 0) {
                if (!d.multi) {  // what a layer of at most 32 connections reports as its kernel
                    spdnn::pair_merge_kernel<<<1, 64, 0, stream>>>(win_dev[l], nblk, N, st_val, err_dev + 1 + 2 * P + l, widest_dev, pair_dev);
                    HIP_TRY(hipMemcpyAsync(pair_info, pair_dev, sizeof(pair_info), hipMemcpyDeviceToHost, stream));
                    HIP_TRY(hipStreamSynchronize(stream));
                }
                // the tile layout, balanced for every neuron's first 32 connections
                uint32_t* qsel = const_cast<uint32_t*>(d.w.qsel);
                if (nblk > 2)
                    spdnn::balance_kernel<4><<<1, spdnn::kBalanceThreads, sizeof(spdnn::BalanceScratch<4>), stream>>>(
                        st_idx, N, win_dev[l], widest_dev, slot_tab, qsel, nlanes, st_len);
                else if (nblk == 2)
                    spdnn::balance_kernel<2><<<1, spdnn::kBalanceThreads, sizeof(spdnn::BalanceScratch<2>), stream>>>(
                        st_idx, N, win_dev[l], widest_dev, slot_tab, qsel, nlanes, st_len);
                else
                    spdnn::balance_kernel<1><<<1, spdnn::kBalanceThreads, sizeof(spdnn::BalanceScratch<1>), stream>>>(
                        st_idx, N, win_dev[l], widest_dev, slot_tab, qsel, nlanes, st_len);
            }
            spdnn::order_pack_kernel<<<nblk * spdnn::kOrderThreads, spdnn::kOrderPackThreads, 0, stream>>>(
                st_idx, st_val, N, win_dev[l], widest_dev, slot_tab, nblk, d.w.planes_log2, const_cast<uint16_t*>(d.w.rel),
                const_cast<float*>(d.w.val), nlanes, st_len);
            HIP_TRY(hipGetLastError());
            d.mode = pair_info[0] == 1 ? kPair : kSingle;
            d.lds_cols = N;
            d.virt_lanes = passes_of[ll];
            continue;
        }
        int nrows = -1;                 // rows of di / dv if not N
        const uint8_t* lens = nullptr;  // connections per row if not 32
        if (ptr && d.multi) {
            // More than 32 connections somewhere: a neuron takes as many lanes as it has parts of 32 connections, and
            // a workgroup as many neighbouring neurons (in fours) as fill its 1024 lanes -- fewer where the next
            // four would widen its column window beyond one LDS stage.  The layer's workgroups
            // are cut into launches of nblk; launch r is pass r.  Their lanes are set up like the neurons of a
            // fixed-32 layer.
            if (round_of[l] == 0) {
                std::vector<int2> qw((size_t)N / 4);  // columns of every four neurons (the staging area as scratch)
                int2* qw_dev = reinterpret_cast<int2*>(st_idx);
                spdnn::csr_quartet_window_kernel<<<(N / 4 + 255) / 256, 256, 0, stream>>>(ptr[ll], idx[ll], N, qw_dev);
                HIP_TRY(hipGetLastError());
                HIP_TRY(hipMemcpyAsync(hp.data(), ptr[ll], sizeof(int32_t) * hp.size(), hipMemcpyDeviceToHost, stream));
                HIP_TRY(hipMemcpyAsync(qw.data(), qw_dev, sizeof(int2) * qw.size(), hipMemcpyDeviceToHost, stream));
                HIP_TRY(hipStreamSynchronize(stream));
                // how the layer's neurons are cut into workgroups: spdnn_cut.h (host code, tested without a GPU)
                const std::vector<spdnn::NeuronRange> cut =
                    spdnn::cut_workgroups(hp.data(), reinterpret_cast<const int*>(qw.data()), N, passes_of[ll], nblk, m->G,
                                          spdnn::kBlk, spdnn::kNnz, spdnn::kCap);
                virt_ranges.clear();
                for (const spdnn::NeuronRange& r : cut) virt_ranges.push_back(make_int2(r.first, r.count));
            }
            std::vector<int2> mine((size_t)nblk, make_int2(N, 0));
            for (int32_t b = 0; b < nblk; ++b) {
                const size_t vb = (size_t)round_of[l] * nblk + b;
                if (vb < virt_ranges.size()) {
                    mine[b] = virt_ranges[vb];
                    d.virt_blocks = b + 1;
                }
            }
            HIP_TRY(hipMemcpyAsync(const_cast<int2*>(d.virt.range), mine.data(), sizeof(int2) * (size_t)nblk, hipMemcpyHostToDevice, stream));
            HIP_TRY(hipStreamSynchronize(stream));  // `mine` goes out of scope
            d.virt_lanes = passes_of[ll];
            spdnn::csr_virtual_kernel<<<nblk, spdnn::kBlk, 0, stream>>>(ptr[ll], idx[ll], val[ll], N, d.virt.range, st_idx, st_val,
                                                                        st_len, const_cast<uint16_t*>(d.virt.slot),
                                                                        const_cast<uint32_t*>(d.virt.fin));
            HIP_TRY(hipGetLastError());
            di = st_idx;
            dv = st_val;
            nrows = nblk * spdnn::kBlk;
            lens = st_len;
        } else if (ptr) {  // general layer of at most 32 connections per neuron, padded with zero weights
            const int r = round_of[l];
            spdnn::csr_block_min_kernel<<<nblk, spdnn::kBlk, 0, stream>>>(ptr[ll], idx[ll], N, r, blockmin);
            spdnn::csr_round_kernel<<<(unsigned)((raw + 255) / 256), 256, 0, stream>>>(ptr[ll], idx[ll], val[ll], N, r,
                                                                                     blockmin, st_idx, st_val);
            HIP_TRY(hipGetLastError());
            di = st_idx;
            dv = st_val;
        } else if (where == SPDNN_HOST) {
            HIP_TRY(hipMemcpyAsync(st_idx, idx[ll], raw * sizeof(int32_t), hipMemcpyHostToDevice, stream));
            HIP_TRY(hipMemcpyAsync(st_val, val[ll], raw * sizeof(float), hipMemcpyHostToDevice, stream));
            di = st_idx;
            dv = st_val;
        }
        int* widest_dev = err_dev + 1 + P + l;
        int* pair_dev = err_dev + 1 + 3 * P + 2 * l;
        spdnn::block_window_kernel<<<nblk, spdnn::kBlk, 0, stream>>>(di, N, win_dev[l], err_dev, widest_dev, dv,
                                                                       err_dev + 1 + 2 * P + l, nrows);
        // A row that fits one LDS stage: the blocks share one tile layout, that of the whole row, which is what
        // resident_kernel needs (out-of-core weights, which it does not take, are laid out the same: same sums).
        const bool whole = resident || (ooc && N <= spdnn::kCap);
        if (whole) {
            spdnn::whole_row_window_kernel<<<1, 64, 0, stream>>>(win_dev[l], const_cast<int2*>(d.virt.range), nblk, N, widest_dev);
            d.w.planes_log2 = spdnn::res_planes_log2(nblk);
        }
        // a layer of several passes runs the one-neuron-per-lane kernels, whose epilogue knows about passes
        if (!d.multi)
            spdnn::pair_merge_kernel<<<1, 64, 0, stream>>>(win_dev[l], nblk, N, dv, err_dev + 1 + 2 * P + l, widest_dev,
                                                           pair_dev);
        HIP_TRY(hipGetLastError());
        // the windows decide the layer's kernel and its set-up; they are small, so read them back now
        int pair_info[2] = {0, 0};
        // Layers that may run on two-row tiles: how many groups of four columns a 4096-neuron unit touches, for
        // every segment length of unit_neuron, asked for now so that it comes back with the windows (the list
        // area serves as the kernel's output).
        constexpr int kCand = spdnn::kSegLog2Max - spdnn::kSegLog2Min + 1;
        const bool r2_room = !d.multi && N % spdnn::kUnit4 == 0 && d.r2_codes != nullptr &&
                             (size_t)(nblk / 4) * (N / 4) <= slot_tab_elems;
        std::vector<int> ngr;
        if (r2_room) {
            ngr.resize((size_t)(nblk / 4) * kCand);
            spdnn::row2_footprint_kernel<<<dim3(nblk / 4, kCand), spdnn::kBlk, 0, stream>>>(di, N, reinterpret_cast<int*>(d.r2_map));
            HIP_TRY(hipGetLastError());
            HIP_TRY(hipMemcpyAsync(ngr.data(), d.r2_map, sizeof(int) * ngr.size(), hipMemcpyDeviceToHost, stream));
        }
        HIP_TRY(hipMemcpyAsync(&hw[(size_t)l * nblk], whole ? d.virt.range : win_dev[l], sizeof(int2) * nblk, hipMemcpyDeviceToHost, stream));
        HIP_TRY(hipMemcpyAsync(pair_info, pair_dev, sizeof(pair_info), hipMemcpyDeviceToHost, stream));
        int strided_info[4] = {1, 0, 0, 0};
        if (all_strided) {
            int* info_dev = reinterpret_cast<int*>(slot_tab);  // this stream's table as scratch
            HIP_TRY(hipMemsetAsync(info_dev, 0, sizeof(strided_info), stream));
            spdnn::strided_detect_kernel<<<(N + 255) / 256, 256, 0, stream>>>(di, dv, N, info_dev);
            HIP_TRY(hipGetLastError());
            HIP_TRY(hipMemcpyAsync(strided_info, info_dev, sizeof(strided_info), hipMemcpyDeviceToHost, stream));
        }
        HIP_TRY(hipStreamSynchronize(stream));
        if (all_strided && (all_strided = strided_info[0] == 0)) {
            spdnn::StridedLayer sl{strided_info[1], strided_info[2], std::gcd(N, strided_info[1]), 0, 1, 0.0f};
            sl.T = N / sl.orbits;
            if (sl.T > spdnn::kNnz) sl.per = (sl.T + spdnn::kStrideOut - 1) / spdnn::kStrideOut;
            std::memcpy(&sl.w, &strided_info[3], sizeof(float));
            // (infinity times an input of 0 is NaN: the sum has to be taken after the multiplication)
            all_strided = spdnn::strided_lanes(sl) <= spdnn::kStrideThreads && std::isfinite(sl.w);
            strided.push_back(sl);
        }
        // One weight, but the windows are too wide for two neurons per lane.  If units of 2048 neurons in segments
        // (unit_neuron) read columns that do not overlap, at most 2048 each -- the strided patterns that RadiX-Net
        // layers are (Section II-A) -- neurons and columns get new names under which every unit has a contiguous
        // window, and the layer is set up again as an ordinary one for the two-neurons-per-lane kernel.
        if (pair_info[0] == 2 && r2_room && d.ww.pk != nullptr && N % spdnn::kPairUnit == 0) {
            const int32_t nunit2 = N / spdnn::kPairUnit;
            constexpr int kCand2 = spdnn::kSegLog2Max - 1 - 5 + 1;  // segments of 2048 down to 32 neurons
            std::vector<int> ngr2((size_t)nunit2 * kCand2);
            int* cnt_dev = reinterpret_cast<int*>(d.r2_map);
            spdnn::row2_footprint_kernel<<<dim3(nunit2, kCand2), spdnn::kBlk, 0, stream>>>(di, N, cnt_dev, spdnn::kPairUnit);
            HIP_TRY(hipGetLastError());
            HIP_TRY(hipMemcpyAsync(ngr2.data(), cnt_dev, sizeof(int) * ngr2.size(), hipMemcpyDeviceToHost, stream));
            HIP_TRY(hipStreamSynchronize(stream));
            int best_a = -1, best = spdnn::kPairUnit / 4 + 1;
            for (int y = 0; y < kCand2; ++y) {
                const int most = *std::max_element(ngr2.begin() + (size_t)y * nunit2, ngr2.begin() + (size_t)(y + 1) * nunit2);
                if (most < best) {
                    best = most;
                    best_a = spdnn::kSegLog2Max - 1 - y;
                }
            }
            if (best_a >= 0) {  // every unit within 2048 columns: do they overlap?
                const int stride2 = nunit2 << best_a;
                int* owner = reinterpret_cast<int*>(slot_tab);  // this stream's table as scratch: N/4 owners, N/4 new names, a flag
                int* newname = owner + N / 4;
                int* conflict = newname + N / 4;
                HIP_TRY(hipMemsetAsync(owner, 0xff, sizeof(int) * (size_t)(N / 4), stream));
                HIP_TRY(hipMemsetAsync(conflict, 0, sizeof(int), stream));
                spdnn::relabel_owner_kernel<<<nunit2, spdnn::kBlk, 0, stream>>>(di, N, best_a, stride2, owner, conflict);
                spdnn::relabel_rank_kernel<<<nunit2, spdnn::kBlk, 0, stream>>>(owner, N, newname, d.r2_map, conflict);
                HIP_TRY(hipGetLastError());
                int clash = 1;
                HIP_TRY(hipMemcpyAsync(&clash, conflict, sizeof(int), hipMemcpyDeviceToHost, stream));
                HIP_TRY(hipStreamSynchronize(stream));
                if (!clash) {
                    // the layer under its new names is written where its wide format would go (it will not have one):
                    // room for 32 steps of 8 bytes per neuron, of which 4 bytes per connection are needed
                    int32_t* renamed = reinterpret_cast<int32_t*>(const_cast<uint2*>(d.ww.pk));
                    spdnn::relabel_apply_kernel<<<(unsigned)((raw + 255) / 256), 256, 0, stream>>>(di, N, best_a, stride2, newname, renamed);
                    HIP_TRY(hipGetLastError());
                    di = renamed;
                    d.relabel = true;
                    d.rn = spdnn::PairRelabel{d.r2_map, best_a, stride2};
                    // the windows, and whether pairs of blocks fit one stage, under the new names
                    HIP_TRY(hipMemsetAsync(widest_dev, 0, sizeof(int), stream));
                    spdnn::block_window_kernel<<<nblk, spdnn::kBlk, 0, stream>>>(di, N, win_dev[l], err_dev, widest_dev, dv,
                                                                                   err_dev + 1 + 2 * P + l, nrows);
                    spdnn::pair_merge_kernel<<<1, 64, 0, stream>>>(win_dev[l], nblk, N, dv, err_dev + 1 + 2 * P + l, widest_dev,
                                                                   pair_dev);
                    HIP_TRY(hipGetLastError());
                    HIP_TRY(hipMemcpyAsync(&hw[(size_t)l * nblk], win_dev[l], sizeof(int2) * nblk, hipMemcpyDeviceToHost, stream));
                    HIP_TRY(hipMemcpyAsync(pair_info, pair_dev, sizeof(pair_info), hipMemcpyDeviceToHost, stream));
                    HIP_TRY(hipStreamSynchronize(stream));
                    if (pair_info[0] != 1) return fail(SPDNN_EHIP, "layer %d: relabelled units do not fit one stage", ll);
                }
            }
        }
        const int pair = pair_info[0] == 1;        // two neurons per lane, single stage
        const bool wide_pair = pair_info[0] == 2;  // ... if the layer also fits the wide format
        // one weight, every block wider than one stage, and every 4096-neuron unit within 16384 columns:
        // four neurons per lane on two-row tiles; needs nothing of the other formats
        const bool row2_ok = wide_pair && !d.multi && N % spdnn::kUnit4 == 0 && d.r2_codes != nullptr;
        bool row2 = row2_ok;
        for (int32_t u = 0; row2 && u < nblk / 4; ++u) {
            int x = 0, y = 0;  // the unit's window: the union of its blocks' cyclic windows
            for (int i = 0; i < 4; ++i)
                spdnn::win_union(x, y, hw[(size_t)l * nblk + 4 * u + i].x, hw[(size_t)l * nblk + 4 * u + i].y, N, x, y);
            row2 = y <= spdnn::kRow2Cols;
        }
        // Windows too wide for the tile, or much wider than the unit itself: the gathered footprint (Section
        // III-A-2's preload list at 4-column granularity) may fit it -- every unit's connections within 4096
        // groups of four columns -- and units of interleaved segments (unit_neuron) may need far fewer columns
        // than units of 4096 neighbours: in a strided pattern the neurons j, j + stride, j + 2 stride, ... read
        // the same columns.  Every segment length from 4096 down to 64 is tried and the one whose largest unit
        // needs the fewest groups wins (the longer segment on a tie).
        // The rank table is set-up scratch: this stream's column -> slot table, which such a layer does not use.
        const int32_t* gather_map = nullptr;
        const uint16_t* gather_rank = nullptr;
        int seg_log2 = spdnn::kSegLog2Max, seg_stride = N;
        int widest_unit = 0;  // columns of the widest unit's window, units of 4096 neighbours
        for (int32_t u = 0; row2_ok && u < nblk / 4; ++u) {
            int x = 0, y = 0;
            for (int i = 0; i < 4; ++i)
                spdnn::win_union(x, y, hw[(size_t)l * nblk + 4 * u + i].x, hw[(size_t)l * nblk + 4 * u + i].y, N, x, y);
            widest_unit = std::max(widest_unit, y);
        }
        if (row2_ok && r2_room && widest_unit > spdnn::kUnit4) {
            const int32_t nunit = nblk / 4;
            int best_a = -1, best = spdnn::kRow2Cols / 4 + 1;
            for (int y = 0; y < kCand; ++y) {
                const int most = *std::max_element(ngr.begin() + (size_t)y * nunit, ngr.begin() + (size_t)(y + 1) * nunit);
                if (most < best) {
                    best = most;
                    best_a = spdnn::kSegLog2Max - y;
                }
            }
            // worth it if the window does not fit the tile at all, or if the tile shrinks to half the window or less
            const bool take = best_a >= 0 && (!row2 || 4 * best <= widest_unit / 2);
            if (take) {
                spdnn::row2_gather_kernel<<<nunit, spdnn::kBlk, 0, stream>>>(di, N, best_a, (N / spdnn::kUnit4) << best_a, d.r2_map,
                                                                           slot_tab, d.r2_ngroups);
                HIP_TRY(hipGetLastError());
                row2 = true;
                seg_log2 = best_a;
                seg_stride = (N / spdnn::kUnit4) << best_a;
                gather_map = d.r2_map;
                gather_rank = slot_tab;
            }
        }
        if (row2) {
            // the windows read back above are the blocks' own; pair_merge_kernel has widened them on the device to
            // common windows of block pairs, whose unions per unit are the same
            d.r2 = spdnn::Row2Weights{reinterpret_cast<const uint4*>(d.r2_codes), win_dev[l], gather_map, seg_log2, seg_stride};
            const int groups = N / spdnn::kGroup32;
            spdnn::row2_pack_kernel<<<groups, spdnn::kRow2PackThreads, 0, stream>>>(di, N, win_dev[l], gather_rank, seg_log2,
                                                                                    seg_stride, d.r2_codes);
            HIP_TRY(hipGetLastError());
            d.mode = kRow2;
            d.lds_cols = spdnn::kRow2Cols;
            std::memcpy(&d.wuni, &pair_info[1], sizeof(float));
            if (ooc)
                HIP_TRY(hipMemcpyAsync(static_cast<char*>(host_arena) + (size_t)l * blk_bytes, m->ooc_slot[l & 1], blk_bytes,
                                       hipMemcpyDeviceToHost, stream));
            if (where == SPDNN_HOST) HIP_TRY(hipStreamSynchronize(stream));  // staging is reused
            continue;
        }
        {  // Rows of up to 16384 columns that the blocks read more of than one LDS stage: whole rows in LDS, whatever the
           // weights (two-row tiles, which hold four neurons per lane for one weight and N a multiple of 4096, were
           // taken above).  The arena's wide format stays empty.
           // But one weight, pairs of blocks and windows of two stages in rows of more than two: a window takes fewer bytes
           // than the row (4 layers on 8000 rows, whole rows -> windows: 10240 neurons, 4200 columns 1.30 -> 1.02 ms, 8000
           // columns 1.30 -> 1.21; 14336 neurons, 4200 columns 1.69 -> 1.39, 6500 columns 1.68 -> 1.69, 9000 columns, three
           // stages, 1.67 -> 3.45; 6144 neurons, 5500 columns 0.80 -> 1.27.  On 100 rows windows take 0.13 ms, whole rows 0.10.)
            int widest = 4;
            for (int32_t b = 0; b < nblk; ++b) widest = std::max(widest, hw[(size_t)l * nblk + b].y);
            const int nst = stages_of(widest);
            const bool windows = wide_pair && nst == 2 && nst <= nstage_cap && d.ww.ps && N > 2 * spdnn::kCap;
            if (!d.multi && !pair && nst >= 2 && N <= spdnn::kFlatCols && !windows) {
                spdnn::flat_pack_kernel<<<nblk * spdnn::kBlk / spdnn::kGroup32, spdnn::kRow2PackThreads, 0, stream>>>(
                    di, dv, N, const_cast<uint16_t*>(d.w.rel), const_cast<float*>(d.w.val));
                HIP_TRY(hipGetLastError());
                d.mode = kFlat;
                d.lds_cols = N;
                std::memcpy(&d.wuni, &pair_info[1], sizeof(float));
                if (ooc)
                    HIP_TRY(hipMemcpyAsync(static_cast<char*>(host_arena) + (size_t)l * blk_bytes, m->ooc_slot[l & 1], blk_bytes,
                                           hipMemcpyDeviceToHost, stream));
                if (where == SPDNN_HOST) HIP_TRY(hipStreamSynchronize(stream));  // staging is reused
                continue;
            }
        }
        const int unit = whole ? nblk : pair ? 2 : 1;  // blocks that share a tile layout
        if (unit > 2)
            spdnn::balance_kernel<4><<<1, spdnn::kBalanceThreads, sizeof(spdnn::BalanceScratch<4>), stream>>>(
                di, N, win_dev[l], widest_dev, slot_tab, const_cast<uint32_t*>(d.w.qsel));
        else if (unit == 2)
            spdnn::balance_kernel<2><<<nblk / 2, spdnn::kBalanceThreads, sizeof(spdnn::BalanceScratch<2>), stream>>>(
                di, N, win_dev[l], widest_dev, slot_tab, const_cast<uint32_t*>(d.w.qsel));
        else
            spdnn::balance_kernel<1><<<nblk, spdnn::kBalanceThreads, sizeof(spdnn::BalanceScratch<1>), stream>>>(
                di, N, win_dev[l], widest_dev, slot_tab, const_cast<uint32_t*>(d.w.qsel), nrows);
        spdnn::order_pack_kernel<<<nblk * spdnn::kOrderThreads, spdnn::kOrderPackThreads, 0, stream>>>(
            di, dv, N, win_dev[l], widest_dev, slot_tab, unit, d.w.planes_log2, const_cast<uint16_t*>(d.w.rel),
            const_cast<float*>(d.w.val), nrows, lens, lens ? const_cast<uint8_t*>(d.virt.nb8) : nullptr);
        HIP_TRY(hipGetLastError());
        if (whole) {  // what the blocks (pairs of blocks) read of the row, from a multiple of 256 columns on (LayerWeights)
            bool narrow = false;
            for (int32_t b = 0; b < nblk; ++b) {
                int2& w = hw[(size_t)l * nblk + b];
                if (pair && (b & 1)) {
                    w = hw[(size_t)l * nblk + b - 1];
                    continue;
                }
                if (pair) spdnn::win_union(w.x, w.y, hw[(size_t)l * nblk + b + 1].x, hw[(size_t)l * nblk + b + 1].y, N, w.x, w.y);
                if (w.x + w.y > N) w = make_int2(0, N);  // it wraps around the row end
                w = make_int2(w.x & ~255, w.y + (w.x & 255));
                narrow = narrow || w.y < N;
            }
            if (narrow) HIP_TRY(hipMemcpyAsync(win_dev[l], &hw[(size_t)l * nblk], sizeof(int2) * nblk, hipMemcpyHostToDevice, stream));
        }
        int widest = 4;
        for (int32_t b = 0; b < nblk; ++b) widest = std::max(widest, hw[(size_t)l * nblk + b].y);
        const int nst = stages_of(widest);
        d.lds_cols = std::min(widest, spdnn::kCap);
        d.mode = pair ? kPair : nst <= 1 ? kSingle : kStaged;
        std::memcpy(&d.wuni, &pair_info[1], sizeof(float));
        // the wide format: 3 and more stages, or 2 stages when the layer can run two neurons per lane
        if (!d.multi && (nst >= 3 || (nst == 2 && wide_pair && d.ww.ps)) && nst <= nstage_cap) {
            d.ww.nstage = nst;
            spdnn::wide_pack_kernel<<<nblk, spdnn::kOrderThreads, wide_lds, stream>>>(
                di, dv, N, win_dev[l], nst, const_cast<uint2*>(d.ww.pk), const_cast<uint8_t*>(d.ww.nb8), const_cast<uint16_t*>(d.ww.spill_col),
                const_cast<float*>(d.ww.spill_val), const_cast<uint8_t*>(d.ww.spill_n), err_dev + 1 + l);
            HIP_TRY(hipGetLastError());
            d.mode = kWide;
            if (wide_pair && spdnn::wide_steps(nst) >= 16 && d.ww.ps) {
                const int S = spdnn::wide_steps(nst);
                const size_t n_out = (size_t)nblk * nst * (S / 8) * spdnn::kBlk;
                spdnn::wide_slots_kernel<<<(unsigned)((n_out + 255) / 256), 256, 0, stream>>>(
                    d.ww.pk, const_cast<uint4*>(d.ww.ps), n_out, S);
                const size_t n_sp = (size_t)nblk * spdnn::kSpill * spdnn::kBlk;
                spdnn::wide_spill16_kernel<<<(unsigned)((n_sp + 255) / 256), 256, 0, stream>>>(
                    d.ww.spill_col, d.ww.spill_val, const_cast<uint16_t*>(d.ww.sp16), n_sp);
                HIP_TRY(hipGetLastError());
                d.mode = kWidePair;
                d.pair4 = nst <= 4;
            }
        }
        if (ooc)  // the finished block goes to the host; its slot is rebuilt two passes later, after this copy
            HIP_TRY(hipMemcpyAsync(static_cast<char*>(host_arena) + (size_t)l * blk_bytes, m->ooc_slot[l & 1], blk_bytes,
                                   hipMemcpyDeviceToHost, stream));
        if (where == SPDNN_HOST) HIP_TRY(hipStreamSynchronize(stream));  // staging is reused
    }
    for (int i = 1; i < ss.n; ++i) HIP_TRY(hipStreamSynchronize(ss.s[i]));
    // error flag and the layers whose patterns did not fit the wide format
    std::vector<int> herr((size_t)P + 1, 0);
    HIP_TRY(hipMemcpyAsync(herr.data(), err_dev, sizeof(int) * (size_t)(P + 1), hipMemcpyDeviceToHost, stream));
    HIP_TRY(hipStreamSynchronize(stream));
    if (herr[0]) return fail(SPDNN_EINVAL, "a column index is outside [0, N)");
    for (int32_t l = 0; l < P; ++l)
        if ((m->layers[l].mode == kWide || m->layers[l].mode == kWidePair) && herr[1 + l]) m->layers[l].mode = kStaged;
    // flat layers: is there one weight for all connections?
    if (N > spdnn::kCap && N <= spdnn::kFlatCols) {
        std::vector<int> differ((size_t)P);
        HIP_TRY(hipMemcpyAsync(differ.data(), err_dev + 1 + 2 * P, sizeof(int) * (size_t)P, hipMemcpyDeviceToHost, stream));
        HIP_TRY(hipStreamSynchronize(stream));
        for (int32_t l = 0; l < P; ++l) m->layers[l].flat_uniform = differ[l] == 0;
    }
    // Rows of at most one LDS stage: they can stay in LDS from layer to layer (resident_kernel, which takes the layers'
    // descriptors from device memory).
    if (resident) {
        std::vector<int> differ((size_t)P);  // passes with more than one weight value
        std::vector<int> info(2 * (size_t)P);
        HIP_TRY(hipMemcpyAsync(differ.data(), err_dev + 1 + 2 * P, sizeof(int) * (size_t)P, hipMemcpyDeviceToHost, stream));
        HIP_TRY(hipMemcpyAsync(info.data(), err_dev + 1 + 3 * P, sizeof(int) * 2 * (size_t)P, hipMemcpyDeviceToHost, stream));
        HIP_TRY(hipStreamSynchronize(stream));
        std::vector<spdnn::ResidentLayer> rl((size_t)L);
        m->res_mode = parts ? spdnn::kResParts : spdnn::kResUniform;
        for (int32_t l = 0; l < L; ++l) {
            const LayerDesc& d = m->layers[first_pass[l]];
            rl[l] = spdnn::ResidentLayer{d.w.rel, d.w.val, d.w.qsel, 0.0f, d.virt.slot, d.virt.fin};
            std::memcpy(&rl[l].wuni, &info[2 * (size_t)first_pass[l] + 1], sizeof(float));
            if (!parts && differ[first_pass[l]]) m->res_mode = spdnn::kResWeights;
        }
        HIP_TRY(hipMemcpyAsync(res_layers_dev, rl.data(), sizeof(spdnn::ResidentLayer) * (size_t)L, hipMemcpyHostToDevice, stream));
        HIP_TRY(hipStreamSynchronize(stream));
        m->res_layers = res_layers_dev;
        m->res_rows = res_rows_dev;
        m->res_part_stride = (uint32_t)blk_bytes;
    }
    if (all_strided) {
        spdnn::StridedLayer* layers_dev = reinterpret_cast<spdnn::StridedLayer*>(st_val);
        HIP_TRY(hipMemcpyAsync(layers_dev, strided.data(), sizeof(spdnn::StridedLayer) * (size_t)L, hipMemcpyHostToDevice, stream));
        HIP_TRY(hipStreamSynchronize(stream));
        m->strided = layers_dev;
        m->res_rows = reinterpret_cast<int*>(layers_dev + L);
        m->strided_bias = hb[0];
        for (const spdnn::StridedLayer& sl : strided) m->strided_lanes = std::max(m->strided_lanes, spdnn::strided_lanes(sl));
        m->strided_known = std::all_of(strided.begin(), strided.end(), [&](const spdnn::StridedLayer& sl) { return spdnn::strided_known(sl, N); });
    }
    guard.m = nullptr;
    *out = m;
    return SPDNN_OK;
}


// No entry point lets an exception out (a failed host allocation in a std::vector, for example).
template <typename F>
int guarded(F f) {
    try {
        return f();
    } catch (const std::bad_alloc&) {
        return fail(SPDNN_EHIP, "out of host memory");
    } catch (...) {
        return fail(SPDNN_EHIP, "unexpected exception");
    }
}

// Argument checks shared by the inference entry points; batch == 0 is answered here (n_active = 0).
int check_infer_args(spdnn_t h, const float* Y0_dev, int32_t batch, int32_t* n_active_host,
                     const int32_t* active_rows_dev, const float* Y_final_dev) {
    if (!h) return fail(SPDNN_EINVAL, "handle is NULL");
    if (!n_active_host) return fail(SPDNN_EINVAL, "n_active_host is NULL");
    if (batch < 0) return fail(SPDNN_EINVAL, "batch < 0");
    h->prof_layers = 0;
    h->launches = h->res_launches = h->row_kernel = 0;
    if (batch == 0) {
        *n_active_host = 0;
        return SPDNN_OK;
    }
    if (!Y0_dev || !active_rows_dev) return fail(SPDNN_EINVAL, "null argument");
    if (reinterpret_cast<uintptr_t>(Y0_dev) % 16) return fail(SPDNN_EINVAL, "Y0 must be 16-byte aligned");
    if (Y_final_dev && reinterpret_cast<uintptr_t>(Y_final_dev) % 16) return fail(SPDNN_EINVAL, "Y_final must be 16-byte aligned");
    return SPDNN_OK;
}

// Address of the current device's copy of the static scratch array.  The array's name is only a
// host-side stand-in; every GPU holds its own copy at its own address, looked up once per device
// (at spdnn_create, else on the first spdnn_infer_static on that device) and kept.
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
void* g_scratch_ptr[kMaxDevices] = {};
int static_scratch(void** out) {
    int dev = 0;
    HIP_TRY(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxDevices) return fail(SPDNN_EINVAL, "device %d: only devices 0..%d are supported", dev, kMaxDevices - 1);
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void* p = nullptr;
        HIP_TRY(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
        if (!p || reinterpret_cast<uintptr_t>(p) % kAlign) return fail(SPDNN_EHIP, "static scratch array has no usable device address");
        g_scratch_ptr[dev] = p;
    }
    *out = g_scratch_ptr[dev];
    return SPDNN_OK;
}

// Is this pinned host memory, copies from which run beside kernels?
bool pinned(const void* host) {
    hipPointerAttribute_t a{};
    if (hipPointerGetAttributes(&a, host) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    return a.type == hipMemoryTypeHost;
}

constexpr int32_t kCopyBoundLayers = 48;             // spdnn_infer_host: so many layers take less time than their input's copy
constexpr size_t kPieceBytes = (size_t)16 << 20;     // ... and so much of it is cut in two, ...
constexpr size_t kPieceBytesPerLayer = 700 << 10;    // ... or so much per pass of a layer, if that is more: rows stay in LDS
constexpr size_t kPieceBytesPerLaunch = 2400 << 10;  // (the same where every layer is a launch)
// Networks of strided sums take a third of the time per layer and less for a batch: little is left behind the last byte of a
// small one, and a piece costs 10 us beside its layers.  Whole -> two pieces, 4096 and 16384 neurons, MB in the batch that is cut:
// 4 layers, 34 662 -> 675 and 662 -> 676 us, 42 820 -> 824 and 823 -> 821, 101 1882 -> 1870 (three pieces 1877); 12, 42 857 -> 844, 34
// 684 -> 689 and 681 -> 691; 24, 67 1377 -> 1328 and 1394 -> 1318; 96, 42 1117 -> 1083; 144, 50 1406 -> 1368, 34 1064 -> 1049 and 1017 ->
// 1096; 200, 50 1566 -> 1659 and 1505 -> 1536, 67 2180 -> 1830 and 2304 -> 1758.
constexpr int32_t kStridedCopyBoundLayers = 200;
constexpr size_t kStridedPieceBytes = (size_t)40 << 20, kStridedPieceBytesPerLayer = 320 << 10;
constexpr int32_t kFewLayers = 4;  // networks of so few layers are not cut into launches that keep rows in LDS

// How resident_kernel runs a network: the most groups of 64 neurons a wave owns, the most planes of 4 rows a pass
// holds, the workgroup's threads and LDS, and how many workgroups fit the GPU at once.
struct ResidentShape {
    int nb, planes, threads, lds, slots;
};
ResidentShape resident_shape(const spdnn_model* h, int32_t rows) {
    ResidentShape r;
    r.planes = 1 << spdnn::res_planes_log2(h->nblk);
    r.nb = resident_groups_per_wave(h->nblk, rows <= spdnn::kRows * h->num_cu);
    const int waves = resident_waves(h->N, r.nb);
    r.threads = 64 * waves;
    r.lds = (int)spdnn::res_tile_bytes(h->N, r.planes) + spdnn::kResMiscBytes + (h->res_mode == spdnn::kResParts ? 4 * h->N : 0);
    r.slots = h->num_cu * std::max(1, std::min(16 / waves, 160 * 1024 / r.lds));
    return r;
}

// How strided_kernel runs a network on `rows` rows: pairs of rows per pass, the workgroup's threads and LDS, and how many
// workgroups fit the GPU at once.  The kernel's registers leave a CU eight waves: two workgroups of four, one of which adds
// while the other waits at a barrier, where two pairs of rows fit the LDS; else one of eight.  Few rows: as few per
// workgroup as it takes to give every slot some.
struct StridedShape {
    int pairs, threads, lds, slots;
};
StridedShape strided_shape(const spdnn_model* h, int32_t rows) {
    StridedShape r;
    const int pair = 8 * h->N;
    const bool two = 2 * h->strided_lanes <= spdnn::kStrideThreads && 2 * (pair + spdnn::kStrideMisc) <= kLdsBytes;
    r.threads = two ? spdnn::kStrideThreads / 2 : spdnn::kStrideThreads;
    r.slots = h->num_cu * (two ? 2 : 1);
    r.pairs = std::min({16, r.threads / h->strided_lanes, (kLdsBytes / (two ? 2 : 1) - spdnn::kStrideMisc) / pair});
    r.pairs = std::max(1, std::min(r.pairs, ((rows + 1) / 2 + r.slots - 1) / r.slots));
    r.lds = r.pairs * pair + spdnn::kStrideMisc;
    return r;
}

// Few rows: few_kernel, in one launch, or, where so many layers follow that it pays to share out anew the rows that are left
// behind the first two, in two.  (How many are left is not known beforehand.  One weight, 900 to 1000 rows,
// resident_kernel -> few_kernel with 450, 510, 700 and 1000 of them left: 64 layers of 1024 neurons 155 -> 137, 147, 149 and 162 us,
// 120 of 2048 430 -> 365, 404, 403 and 453, 120 of 256 152 -> 129, 138, 138 and 145; weights of their own, 64 of 1024, 188 -> 181 at
// worst.  The second launch costs 5 us; four rows per workgroup, of about 1024 or 2048 neurons with one weight, are what loses.)
constexpr int32_t kFewSplitLayers = 64;
// Four rows per workgroup are as many as resident_kernel's smallest pass: not for more than two output blocks, where its
// second barrier weighs little (24 layers of 4096 neurons, 1000 rows: 192 -> 197 us with four, 500 rows of 12 layers with weights
// 135 -> 130 with two).  Neurons of any length: not above kFewPartsN, where it was measured to
// lose (6 layers, 7 and 500 rows, resident_kernel -> few_kernel: 16 to 64
// connections, 2200 neurons 83 -> 79 and 84 -> 80 us, 2600 87 -> 89 and 88 -> 88, 3200 96 -> 103 and 96 -> 103, 4096 112 -> 124 and
// 111 -> 124; 8 to 32 connections, 4096 neurons 81 -> 87 and 82 -> 90).
constexpr int32_t kFewPartsN = 2560;
bool few_rows(const spdnn_model* h, int32_t batch) {
    const int32_t most = h->nblk > 2 ? 2 : spdnn::kFewRows;
    return h->res_layers && !h->strided && batch <= std::min(most * h->num_cu, spdnn::kFewCount) && (h->res_mode != spdnn::kResParts || h->N <= kFewPartsN);
}
bool few_split(const spdnn_model* h, int32_t batch) { return batch > h->num_cu && h->L >= kFewSplitLayers; }

// All layers in one launch?  With rows in LDS from layer to layer, if a workgroup's share of the rows is small: they
// stay with the workgroup they started in, and a share that is packed together again as rows die is all the
// rebalancing there is.  One output block: up to kShareRows rows per CU; more blocks: what one pass holds.
bool one_launch(const spdnn_model* h, int32_t batch) {
    if (batch > 0 && h->strided) {  // what the workgroups hold at a time
        const StridedShape s = strided_shape(h, batch);
        return (batch + 2 * s.pairs - 1) / (2 * s.pairs) <= s.slots;
    }
    if (batch <= 0 || h->res_layers == nullptr) return false;
    if (few_rows(h, batch)) return !few_split(h, batch);
    const int32_t groups = (batch + spdnn::kRows - 1) / spdnn::kRows;
    const int32_t share = (groups + h->num_cu - 1) / h->num_cu * spdnn::kRows;
    return share <= (h->nblk == 1 ? spdnn::kShareRows : spdnn::kRows * (1 << spdnn::res_planes_log2(h->nblk)));
}

// How many layers, from the first on, run one by one, through the kernels they are set up for: all, two or none.  A launch that
// keeps rows in LDS brings them in and out again beside its arithmetic, not under it, which a few layers of many passes
// do not make up for (once most of the rows that die have died, the rest is fewer passes and more layers).
// Whole passes on 60 000 rows, rows in LDS -> one by one, the layers of 4096 neurons with one weight: 1 layer 1073 -> 812 us;
// half the rows dead behind the first layer 816 -> 610; 2 layers 1408 -> 1211; the first 2 of 6 1690 -> 1469; with weights
// of their own 1 layer 1136 -> 891, 2 layers 1496 -> 1411; 2048 neurons, one weight, 1 layer 536 -> 419, the first 2 of 6 873 ->
// 792, weights 562 -> 414, 1015 -> 944.  20 000 rows of 4096 neurons with weights and windows of 300 columns, 2 layers:
// 508 -> 400; 60 000 rows of 1024 neurons, 1 layer: 284 -> 221 (512 neurons on the chip: 166).  Not for three output blocks, which the CUs cannot share evenly (3072 neurons, 3 layers, 1003 -> 1347), nor for four
// where the last one is ragged and there is no pair of neurons per lane (4000 neurons, one weight, 3 layers: 1208 -> 1194).
int32_t one_by_one(const spdnn_model* h, int32_t batch) {
    if (h->strided || few_rows(h, batch) || h->N <= 512 || h->nblk == 3 || h->res_mode == spdnn::kResParts || one_launch(h, batch)) return 0;
    const ResidentShape shape = resident_shape(h, batch);
    const int32_t rows = shape.slots * shape.planes * spdnn::kRows;
    const int32_t passes = (batch + rows - 1) / rows;
    if (h->L == 1) return passes >= 2 ? 1 : 0;
    if (h->nblk == 1 || (h->nblk == 4 && h->N != spdnn::kCap)) return 0;
    bool pair = true, narrow = true;  // the first two layers: two neurons per lane; windows of at most half a row
    for (int32_t l = 0; l < 2; ++l) {
        pair = pair && h->layers[l].mode == kPair;
        narrow = narrow && 2 * h->layers[l].lds_cols <= h->N;
    }
    if (h->L <= kFewLayers) return passes >= (narrow ? 4 : pair ? (h->L == 2 ? 5 : 8) : 12) ? h->L : 0;
    return passes >= (pair ? 8 : h->nblk == 2 ? 12 : INT32_MAX) ? 2 : 0;
}

hipError_t launch_resident(spdnn_t h, const ResidentShape& r, int32_t Q, const float* Yin, float* Yout, uint8_t* flags,
                           const spdnn::RowLists& rl, const spdnn::ResidentArgs& ra) {
    const auto run = [&](auto nb, auto planes, auto mode) {
        spdnn::resident_kernel<decltype(nb)::value, decltype(planes)::value, decltype(mode)::value>
            <<<Q, r.threads, r.lds, h->stream>>>(Yin, Yout, flags, rl, ra, h->bias_dev, h->N);
    };
    const auto run_mode = [&](auto nb, auto planes) {
        if (h->res_mode == spdnn::kResUniform) run(nb, planes, std::integral_constant<int, spdnn::kResUniform>{});
        else if (h->res_mode == spdnn::kResParts) run(nb, planes, std::integral_constant<int, spdnn::kResParts>{});
        else run(nb, planes, std::integral_constant<int, spdnn::kResWeights>{});
    };
    if (r.nb == 1) run_mode(std::integral_constant<int, 1>{}, std::integral_constant<int, 4>{});
    else if (r.nb == 2) run_mode(std::integral_constant<int, 2>{}, std::integral_constant<int, 4>{});
    else run_mode(std::integral_constant<int, 4>{}, std::integral_constant<int, 2>{});
    return hipGetLastError();
}

hipError_t launch_few(spdnn_t h, const spdnn::FewArgs& fa, int32_t workgroups, const float* Yin) {
    const int threads = 64 * std::min(16, (h->N + 63) / 64);
    const auto run = [&](auto mode) {
        spdnn::few_kernel<decltype(mode)::value><<<workgroups, threads, few_lds(h->N, h->nblk), h->stream>>>(fa, Yin, h->bias_dev, h->N);
    };
    if (h->res_mode == spdnn::kResUniform) run(std::integral_constant<int, spdnn::kResUniform>{});
    else if (h->res_mode == spdnn::kResParts) run(std::integral_constant<int, spdnn::kResParts>{});
    else run(std::integral_constant<int, spdnn::kResWeights>{});
    return hipGetLastError();
}

// Layers l0 .. l1-1 through strided_kernel on `rows` rows.
hipError_t launch_strided(spdnn_t h, int32_t l0, int32_t l1, int32_t rows, const float* Yin, float* Yout, uint8_t* flags,
                          const spdnn::RowLists& rl, int* layer_rows) {
    const StridedShape r = strided_shape(h, rows);
    const spdnn::StridedArgs sa{h->strided, l0, l1, rows, r.pairs, h->strided_bias, layer_rows};
    const int grid = std::min((rows + 2 * r.pairs - 1) / (2 * r.pairs), r.slots);
    const auto run = [&](auto pairs, auto known, auto scaled) {
        spdnn::strided_kernel<decltype(pairs)::value, decltype(known)::value, decltype(scaled)::value>
            <<<grid, r.threads, r.lds, h->stream>>>(Yin, Yout, flags, rl, sa, h->N);
    };
    const auto run_pairs = [&](auto pairs, auto known) {
        spdnn::strided_scaled(h->strided_bias) ? run(pairs, known, std::true_type{}) : run(pairs, known, std::false_type{});
    };
    if (r.pairs > 1) h->strided_known ? run_pairs(std::true_type{}, std::true_type{}) : run_pairs(std::true_type{}, std::false_type{});
    else h->strided_known ? run_pairs(std::false_type{}, std::true_type{}) : run_pairs(std::false_type{}, std::false_type{});
    return hipGetLastError();
}

// One layer through fused_flat_kernel on at most `bound` rows.  The units of a row chunk go to one XCD (32 CUs, one L2), so
// that a row is fetched from memory once; no more chunks than an XCD has CUs for all their units at once.
hipError_t launch_flat(spdnn_t h, const LayerDesc& d, const float* Yin, float* Yout, uint8_t* flags, const spdnn::RowLists& rl,
                       int32_t bound) {
    const int32_t N = h->N, groups = (N + 63) / 64;
    const int rows = spdnn::flat_rows(N), slots = d.flat_uniform ? 4 : 2;
    const int32_t ncb = (groups + 16 * slots - 1) / (16 * slots), gpu = (groups + ncb - 1) / ncb;
    const int32_t Q = std::max(1, std::min(8 * std::max(1, h->num_cu / 8 / ncb), (bound + rows - 1) / rows));
    const int32_t grid = (Q + 7) / 8 * 8 * ncb;
    const auto run = [&](auto r, auto uni) {
        spdnn::fused_flat_kernel<decltype(r)::value, decltype(uni)::value><<<grid, spdnn::kBlk, spdnn::flat_lds_bytes(rows), h->stream>>>(
            Yin, Yout, flags, rl, d.w, h->bias_dev, N, ncb, ncb, Q, gpu, d.wuni);
    };
    const auto run_r = [&](auto r) {
        if (d.flat_uniform) run(r, std::true_type{});
        else run(r, std::false_type{});
    };
    if (rows == 1) run_r(std::integral_constant<int, 1>{});
    else if (rows == 2) run_r(std::integral_constant<int, 2>{});
    else if (rows == 3) run_r(std::integral_constant<int, 3>{});
    else run_r(std::integral_constant<int, 4>{});
    return hipGetLastError();
}

// The row lists of layer l's launch.  The layer's first kernel compacts the list of active rows on its way in (the flags
// layer l-1 raised -> slots and row numbers); later passes of the same layer find the lists in place.
spdnn::RowLists layer_lists(const spdnn_model* h, const WorkView& wv, int32_t l, bool first) {
    spdnn::RowLists rl;
    rl.flags_prev = first ? wv.flags[(l + 2) % 3] : nullptr;
    rl.count_prev = wv.count[(l + 1) & 1];
    rl.gid_prev = wv.gid[(l + 1) & 1];
    rl.cat = wv.cat[l & 1];
    rl.gid = wv.gid[l & 1];
    rl.count = wv.count[l & 1];
    rl.host_count = h->host_counts + l;
    rl.flags_clear = wv.flags[(l + 1) % 3];
    return rl;
}

// "Layer -1": every row of the batch is flagged alive, under its own number.
hipError_t launch_init_lists(spdnn_t h, const WorkView& wv, int32_t batch, int32_t row_offset) {
    spdnn::init_lists_kernel<<<(batch + 255) / 256, 256, 0, h->stream>>>(wv.gid[1], wv.flags[2], wv.flags[0], wv.count[1], batch,
                                                                         row_offset);
    return hipGetLastError();
}

// One launch of a layer: one pass of it, through the kernel it is set up for, on at most `bound` rows.
hipError_t launch_layer(spdnn_t h, const LayerDesc& d, const float* Yin, float* Yout, uint8_t* flags, const spdnn::RowLists& rl,
                        int32_t bound) {
    if (d.mode == kFlat) return launch_flat(h, d, Yin, Yout, flags, rl, bound);
    const int32_t N = h->N;
    hipStream_t s = h->stream;
    // launch shape: one workgroup per CU; the rows are cut into Q chunks per output block
    const int32_t rows_per_group = d.mode == kRow2 ? spdnn::kRows2 : spdnn::kRows;
    const int32_t ngroups = (bound + rows_per_group - 1) / rows_per_group;
    // kPair: the workgroups' column blocks are pairs of output blocks
    const bool two = d.mode == kPair || d.mode == kWidePair;
    const int32_t ncb = d.mode == kRow2 ? h->nblk / 4 : two ? h->nblk / 2 : h->nblk;
    // Workgroups that read the same rows go to one XCD (32 CUs, one L2).  In a wide layer every
    // column block reads whole rows: as many of them as possible share an XCD, so that a row is
    // fetched from memory once, not once per XCD.
    int32_t G = d.mode == kPair ? ((ncb % 2 == 0) ? 2 : 1) : h->G;
    if (d.multi)  // fewer neurons per workgroup: up to P times as many workgroups read the same window
        for (int32_t g : {32, 16, 8, 4, 3, 2, 1})
            if (g <= h->G * d.virt_lanes && ncb % g == 0) {
                G = g;
                break;
            }
    if (d.mode == kWide || d.mode == kWidePair || d.mode == kRow2)
        for (int32_t g : {32, 16, 8, 4, 3, 2, 1})
            if (ncb % g == 0) {
                G = g;
                break;
            }
    int32_t Q = std::max(1, h->num_cu / ncb);
    // several lanes per neuron: the launches of a layer have different numbers of workgroups with neurons,
    // rarely a divisor of the CUs; four times as many workgroups as CUs, taken up as CUs fall free
    if (d.multi) Q = (4 * h->num_cu + std::max(1, d.virt_blocks) - 1) / std::max(1, d.virt_blocks);
    Q = std::max(1, std::min(Q, ngroups));
    const int32_t units = (ncb / G) * Q;
    const int32_t grid = (units + 7) / 8 * 8 * G;
    const size_t lds = spdnn::tile_pair_bytes((d.lds_cols + 255) / 256 * 256);  // whole waves of 256 columns
    if (d.mode == kRow2)
        spdnn::fused_row2_kernel<<<grid, spdnn::kBlk, spdnn::kRow2LdsBytes, s>>>(
            Yin, Yout, flags, rl, d.r2, h->bias_dev, N, ncb, G, Q, d.wuni);
    else if (d.multi) {  // several lanes per neuron: the lanes' sums meet in LDS behind the tile pair
        spdnn::VirtInfo vi = d.virt;
        vi.part_off = (uint32_t)lds;
        if (d.mode == kStaged)
            spdnn::fused_layer_kernel<true, true><<<grid, spdnn::kBlk, lds + kVirtLds, s>>>(
                Yin, Yout, flags, rl, d.w, h->bias_dev, N, h->nblk, G, Q, vi);
        else
            spdnn::fused_layer_kernel<false, true><<<grid, spdnn::kBlk, lds + kVirtLds, s>>>(
                Yin, Yout, flags, rl, d.w, h->bias_dev, N, h->nblk, G, Q, vi);
    }
    else if (d.mode == kPair && d.relabel)
        spdnn::fused_pair_kernel<true><<<grid, spdnn::kBlk, lds, s>>>(
            Yin, Yout, flags, rl, d.w, h->bias_dev, N, ncb, G, Q, d.wuni, d.rn);
    else if (d.mode == kPair && d.w.planes_log2)
        spdnn::fused_pair_kernel<false, true><<<grid, spdnn::kBlk, lds, s>>>(
            Yin, Yout, flags, rl, d.w, h->bias_dev, N, ncb, G, Q, d.wuni);
    else if (d.mode == kPair)
        spdnn::fused_pair_kernel<false><<<grid, spdnn::kBlk, lds, s>>>(
            Yin, Yout, flags, rl, d.w, h->bias_dev, N, ncb, G, Q, d.wuni);
    else if (d.mode == kWidePair && d.pair4 && d.ww.nstage == 2)  // + the all-zero entries and the spill table
        spdnn::fused_wide_pair4_kernel<2, 32><<<grid, spdnn::kBlk, lds + spdnn::kPair4LdsExtra, s>>>(
            Yin, Yout, flags, rl, d.ww, h->bias_dev, N, ncb, G, Q, d.wuni);
    else if (d.mode == kWidePair && d.pair4)
        spdnn::fused_wide_pair4_kernel<4, 16><<<grid, spdnn::kBlk, lds + spdnn::kPair4LdsExtra, s>>>(
            Yin, Yout, flags, rl, d.ww, h->bias_dev, N, ncb, G, Q, d.wuni);
    else if (d.mode == kWidePair)
        spdnn::fused_wide_pair_kernel<<<grid, spdnn::kBlk, lds + spdnn::kPadLds, s>>>(
            Yin, Yout, flags, rl, d.ww, h->bias_dev, N, ncb, G, Q, d.wuni);
    else if (d.mode == kWide && d.ww.nstage > 8)
        spdnn::fused_wide_kernel<8><<<grid, spdnn::kBlk, lds, s>>>(
            Yin, Yout, flags, rl, d.ww, h->bias_dev, N, ncb, G, Q);
    else if (d.mode == kWide)
        spdnn::fused_wide_kernel<16><<<grid, spdnn::kBlk, lds, s>>>(
            Yin, Yout, flags, rl, d.ww, h->bias_dev, N, ncb, G, Q);
    else if (d.mode == kStaged)
        spdnn::fused_layer_kernel<true><<<grid, spdnn::kBlk, lds, s>>>(
            Yin, Yout, flags, rl, d.w, h->bias_dev, N, h->nblk, G, Q);
    else if (d.w.planes_log2)
        spdnn::fused_layer_kernel<false, false, true><<<grid, spdnn::kBlk, lds, s>>>(
            Yin, Yout, flags, rl, d.w, h->bias_dev, N, h->nblk, G, Q);
    else
        spdnn::fused_layer_kernel<false><<<grid, spdnn::kBlk, lds, s>>>(
            Yin, Yout, flags, rl, d.w, h->bias_dev, N, h->nblk, G, Q);
    return hipGetLastError();
}

// Waits until a kernel has stored a count to its slot in pinned host memory.  The slot is polled; the stream is
// asked now and then whether it has run dry, only so that a failed launch ends the wait.
int wait_count(spdnn_t h, int32_t l, int32_t* count) {
    volatile int* slot = h->host_counts + l;
    int32_t c = *slot;
    for (uint32_t spin = 1; c < 0; ++spin) {
        if ((spin & 1023u) == 0) {
            const hipError_t q = hipStreamQuery(h->stream);
            if (q == hipSuccess) {  // everything launched is done: the count has been stored
                c = *slot;
                if (c < 0) return fail(SPDNN_EHIP, "layer %d finished without reporting its active rows", l);
                break;
            }
            if (q != hipErrorNotReady) HIP_TRY(q);
        }
        c = *slot;
    }
    std::atomic_thread_fence(std::memory_order_acquire);
    *count = c;
    return SPDNN_OK;
}

// The result: the rows whose flag is set among those the last launch wrote (numbers gid_in, or without lists the whole
// batch), their numbers ascending to active_rows_dev and their values, from Y_last, to Y_final_dev.  Nothing here waits
// for the count but the host at the end: rows are numbered straight into the caller's array, and the gather takes the
// count from device memory (at most `bound` rows).  Returns with the stream drained.
// Y_last == Y_final_dev: the last launch wrote its rows there, row i of its list to row i (write_through); if all of them
// survived they are in place, else they move together by way of `spare`, the work buffer that launch read.
int finish_infer(spdnn_t h, const uint8_t* flags, const int* count_in, const int* gid_in, int32_t batch, int32_t row_offset,
                 int* count_out, int* cat_out, int32_t slot, const float* Y_last, float* spare, int32_t bound,
                 int32_t* n_active_host, int32_t* active_rows_dev, float* Y_final_dev) {
    hipStream_t s = h->stream;
    h->host_counts[slot] = -1;
    const int n4 = h->N / 4;
    const float4* from = reinterpret_cast<const float4*>(Y_last);
    float4* to = reinterpret_cast<float4*>(Y_final_dev);
    if (bound <= spdnn::kFinishRows && (size_t)bound * h->N * sizeof(float) <= spdnn::kFinishBytes &&
        (!Y_final_dev || Y_last != Y_final_dev)) {  // both in one launch
        const int per = std::max(1, (bound + spdnn::kFinishGrid - 1) / spdnn::kFinishGrid), grid = std::max(1, (bound + per - 1) / per);
        // a few long rows: a row's copy is shared by as many workgroups as have one turn of it each (one workgroup per row: 40 rows through
        // 20 layers of 65536 neurons 339 -> 337 us now, 363 without; 86 rows, 2 layers of 16384 75 -> 72, 77 without; first = two launches)
        const int parts = to ? std::max(1, std::min(n4 / (4 * spdnn::kFinishThreads), 2048 / grid)) : 1;
        spdnn::finish_rows_kernel<<<dim3(grid, parts), spdnn::kFinishThreads, 0, s>>>(flags, count_in, gid_in, batch, row_offset, per, active_rows_dev,
                                                                         h->host_counts + slot, from, n4, to);
        HIP_TRY(hipGetLastError());
    } else {
        spdnn::compact_kernel<<<spdnn::kCompactWGs, 1024, 0, s>>>(flags, nullptr, count_in, count_out, gid_in, active_rows_dev, cat_out,
                                                                  h->host_counts + slot, batch, row_offset);
        HIP_TRY(hipGetLastError());
        if (Y_final_dev && bound > 0) {
            const size_t total = (size_t)bound * n4;
            if (Y_last != Y_final_dev)
                spdnn::gather_rows_kernel<<<(int)std::min<size_t>((total + 255) / 256, 65536), 256, 0, s>>>(from, cat_out, count_out, nullptr, n4, to);
            else {
                const int g = (int)std::min<size_t>((total + 255) / 256, 2048);
                float4* by = reinterpret_cast<float4*>(spare);
                spdnn::gather_rows_kernel<<<g, 256, 0, s>>>(from, cat_out, count_out, count_in, n4, by);
                spdnn::gather_rows_kernel<<<g, 256, 0, s>>>(by, nullptr, count_out, count_in, n4, to);
            }
            HIP_TRY(hipGetLastError());
        }
    }
    HIP_TRY(hipStreamSynchronize(s));
    const int n = h->host_counts[slot];
    if (n < 0) return fail(SPDNN_EHIP, "the last layer finished without reporting its active rows");
    *n_active_host = n;
    return SPDNN_OK;
}

// Should the last launch write its rows straight to the caller's array?  Saves a pass over them (0.16 ms for 30 000 rows of
// 4096 neurons) when they all survive, costs one when they do not: only if no row died lately, not for small results,
// which the two kernels that make sure would take longer than, and not in a network of so few layers that little is known
// and the pass counts (4 layers of 65536 neurons on 4000 rows, half of them dead in the last: 1.82 -> 2.02 ms with it).
// Three layers will do up to 16384 columns (3 layers of 16384 neurons on 8000 rows: all alive 1.12 -> 0.99 ms, half of them
// dead in the last 1.03 -> 1.15).
bool write_through(const spdnn_model* h, const float* Y_final_dev, int32_t rows, bool none_died) {
    return Y_final_dev && none_died && (h->L > kFewLayers || (h->L > 2 && h->N > spdnn::kCap && h->N <= spdnn::kFlatCols)) && (size_t)rows * h->N * sizeof(float) >= ((size_t)8 << 20);
}

// infer_impl for networks whose rows stay in LDS from layer to layer (resident_kernel, strided_kernel).
int infer_resident(spdnn_t h, const float* Y0_dev, int32_t batch, const WorkView& wv, int32_t row_offset,
                   int32_t* n_active_host, int32_t* active_rows_dev, float* Y_final_dev) {
    const int32_t L = h->L;
    hipStream_t s = h->stream;
    struct DrainModel {  // nothing of this call is left running on return, whatever happens
        hipStream_t s;
        bool armed = true;
        ~DrainModel() {
            if (armed) (void)hipStreamSynchronize(s);
        }
    } drain_model{s};
    const bool one = one_launch(h, batch);
    int* layer_rows = nullptr;
    if (h->profiling) {
        layer_rows = h->res_rows;
        spdnn::clear_counters_kernel<<<(L + 256) / 256, 256, 0, s>>>(layer_rows, L + 1);
        HIP_TRY(hipGetLastError());
    }
    // Runs of layers.  In one launch the workgroups pack their shares together once, behind the first two layers, if
    // they are of several passes.  Few layers are one launch as well.  Otherwise the batch is compacted and shared out anew after two layers, where most
    // of the rows that die have died.  If fewer than a quarter died, or not many layers are left, they are one launch;
    // if not, the next run is four times as long, and so on.  (A launch costs the gap before it, 20 us, and the rows'
    // way through memory, together what two to three layers of 4096 neurons take; rows that die afterwards are the
    // kernel's own business, which stops and merges passes.)
    // With weights of their own above 2048 neurons a layer's connections are 576 KB and more: workgroups that stop at
    // different layers no longer find them in L2.  There the rest is cut in half as long as rows die (24 layers of 4096
    // neurons, 30 000 rows that die evenly: 4.54 -> 3.75 ms) and more than 12 layers are left.
    // Strided sums take a third of the time per layer: more layers are one launch.
    const int32_t last_layers = h->strided ? 64 : 32;
    const bool halves = !h->strided && h->res_mode != spdnn::kResUniform && h->nblk > 2;
    std::vector<spdnn::LayerRun> runs;
    int32_t alive = batch, before = batch;
    spdnn::RowLists rl{};    // the rows on entry to the next run (rl.count == NULL: the whole batch)
    const float* Yin = Y0_dev;
    float* Y_last = nullptr;
    int yo = 0, lo = 0;      // the work buffer and the lists that the next run writes
    int32_t k = 0;           // runs so far
    int32_t len = 2;         // layers of the next run
    int32_t l0 = 0;
    // the lists of the rows that the last run left, for the next one at layer l
    const auto compact = [&](const uint8_t* flags, const int* count_in, const int* gid_in, int32_t l) -> int {
        h->host_counts[l] = -1;
        spdnn::compact_kernel<<<spdnn::kCompactWGs, 1024, 0, s>>>(flags, nullptr, count_in, wv.count[lo], gid_in, wv.gid[lo], wv.cat[lo],
                                                                  h->host_counts + l, batch, row_offset);
        HIP_TRY(hipGetLastError());
        before = alive;
        const int rc = wait_count(h, l, &alive);
        rl.count = wv.count[lo];
        rl.gid = wv.gid[lo];
        rl.cat = wv.cat[lo];
        lo ^= 1;
        return rc;
    };
    const uint8_t* last_flags = wv.flags[0];  // of the last launch
    bool finished = false;  // the last launch has done what finish_infer does
    if (few_rows(h, batch)) {
        const bool split = few_split(h, batch);
        finished = batch == 1;  // (a workgroup with more rows would take longer than the launch it saves)
        if (finished) h->host_counts[L + 1] = -1;
        spdnn::FewArgs fa{h->res_layers, 0, split ? 2 : L, batch, h->res_part_stride, spdnn::res_planes_log2(h->nblk), layer_rows,
                          nullptr, wv.gid[0], wv.count[0], row_offset, nullptr, nullptr, finished ? active_rows_dev : nullptr, h->host_counts + L + 1};
        const int32_t workgroups = std::min(batch, h->num_cu);
        for (int32_t i = 0; i <= (split ? 1 : 0); ++i) {
            if (h->profiling) HIP_TRY(hipEventRecord(h->t0[fa.l0], s));
            Y_last = fa.Yout = finished ? Y_final_dev : wv.Y[i];
            last_flags = fa.flags = wv.flags[i];
            HIP_TRY(launch_few(h, fa, workgroups, i == 0 ? Y0_dev : wv.Y[0]));
            ++h->launches;
            ++h->res_launches;
            h->row_kernel = SPDNN_ROWS_FEW;
            if (h->profiling) HIP_TRY(hipEventRecord(h->t1[fa.l0], s));
            runs.push_back({fa.l0, fa.l1, false});
            fa.l0 = fa.l1;
            fa.l1 = L;
            fa.flags_prev = wv.flags[0];
        }
        if (split) {  // the second launch has made the list its rows are numbered by
            rl.count = wv.count[0];
            rl.gid = wv.gid[0];
        }
        yo = split ? 1 : 0;
        lo = 1;
        l0 = L;
    } else if (one_by_one(h, batch) == 2) {
        HIP_TRY(launch_init_lists(h, wv, batch, row_offset));
        for (int32_t l = 0; l < 2; ++l) {
            if (h->profiling) HIP_TRY(hipEventRecord(h->t0[l], s));
            HIP_TRY(launch_layer(h, h->layers[l], l == 0 ? Y0_dev : wv.Y[0], wv.Y[l], wv.flags[l], layer_lists(h, wv, l, true), batch));
            ++h->launches;
            if (h->profiling) HIP_TRY(hipEventRecord(h->t1[l], s));
            runs.push_back({l, l + 1, true});
        }
        const int rc = compact(wv.flags[1], wv.count[1], wv.gid[1], 2);
        if (rc != SPDNN_OK) return rc;
        Yin = wv.Y[1];
        l0 = 2;
        k = 1;
        len = 8;
    }
    for (; l0 < L && alive > 0; ++k, len *= 4) {
        if (halves && k > 0) len = (int64_t)alive * 32 > (int64_t)before * 31 || L - l0 <= 12 ? L : std::max(8, (L - l0 + 1) / 2);
        const bool rest = one || L <= kFewLayers || (!halves && k > 0 && ((int64_t)alive * 4 > (int64_t)before * 3 || L - l0 <= last_layers)) || len >= L - l0;
        const int32_t l1 = rest ? L : l0 + len;
        if (h->profiling) HIP_TRY(hipEventRecord(h->t0[l0], s));
        // (rows that lived through two or more layers mostly live on)
        Y_last = rest && write_through(h, Y_final_dev, alive, k > 0) ? Y_final_dev : wv.Y[yo];
        if (h->strided) {
            HIP_TRY(launch_strided(h, l0, l1, alive, Yin, Y_last, wv.flags[0], rl, layer_rows));
        } else {
            const ResidentShape shape = resident_shape(h, alive);
            const int32_t groups = (alive + spdnn::kRows - 1) / spdnn::kRows;
            const int32_t Q = std::min(groups, shape.slots);
            const bool several = (groups + Q - 1) / Q > shape.planes;
            const spdnn::ResidentArgs ra{h->res_layers, l0, one && several ? std::min(l0 + 2, l1) : l1, l1, L, batch, h->res_part_stride, layer_rows};
            HIP_TRY(launch_resident(h, shape, Q, Yin, Y_last, wv.flags[0], rl, ra));
        }
        ++h->launches;
        ++h->res_launches;
        h->row_kernel = h->strided ? SPDNN_ROWS_STRIDED : SPDNN_ROWS_RESIDENT;
        if (h->profiling) HIP_TRY(hipEventRecord(h->t1[l0], s));
        runs.push_back({l0, l1, false});
        l0 = l1;
        if (l1 == L) break;
        const int rc = compact(wv.flags[0], rl.count, rl.gid, l1);
        if (rc != SPDNN_OK) return rc;
        Yin = wv.Y[yo];
        yo ^= 1;
    }
    int32_t rc = SPDNN_OK;
    if (finished) {
        HIP_TRY(hipStreamSynchronize(s));
        *n_active_host = h->host_counts[L + 1];
        if (*n_active_host < 0) return fail(SPDNN_EHIP, "the last layer finished without reporting its active rows");
    } else if (alive > 0)
        rc = finish_infer(h, last_flags, rl.count, rl.gid, batch, row_offset, wv.count[lo], wv.cat[lo], L + 1,
                          Y_last, wv.Y[yo ^ 1], alive, n_active_host, active_rows_dev, Y_final_dev);
    else {
        HIP_TRY(hipStreamSynchronize(s));
        *n_active_host = 0;
    }
    if (rc != SPDNN_OK) return rc;
    drain_model.armed = false;
    if (h->profiling) {  // a launch's time is shared out among its layers by the rows they had
        std::vector<int> rows((size_t)L + 1);
        HIP_TRY(hipMemcpy(rows.data(), layer_rows, sizeof(int) * rows.size(), hipMemcpyDeviceToHost));
        rows[0] = batch;
        spdnn::take_host_counts(runs.data(), runs.size(), h->host_counts, rows.data());
        int32_t run = L;  // "launched": up to the first layer without rows
        for (int32_t l = 1; l < L; ++l)
            if (rows[l] == 0) {
                run = l + 1;
                break;
            }
        h->prof_layers = run;
        h->prof_ms.assign(run, 0.0f);
        h->prof_rows.assign(rows.begin(), rows.begin() + run);
        for (const spdnn::LayerRun& r : runs) {
            float ms = 0.0f;
            HIP_TRY(hipEventElapsedTime(&ms, h->t0[r.l0], h->t1[r.l0]));
            double sum = 0.0;
            for (int32_t l = r.l0; l < std::min(r.l1, run); ++l) sum += rows[l];
            for (int32_t l = r.l0; l < std::min(r.l1, run); ++l) h->prof_ms[l] = sum > 0 ? (float)(ms * rows[l] / sum) : 0.0f;
        }
    }
    return SPDNN_OK;
}

// All L layers on `batch` rows whose first row has the original number row_offset; wv = the carved
// work memory.  Returns with the model's stream drained, also when a HIP call fails half way.
int infer_impl(spdnn_t h, const float* Y0_dev, int32_t batch, const WorkView& wv, int32_t row_offset,
               int32_t* n_active_host, int32_t* active_rows_dev, float* Y_final_dev) {
    const int32_t L = h->L;
    if (h->strided || (h->res_layers && one_by_one(h, batch) < L))
        return infer_resident(h, Y0_dev, batch, wv, row_offset, n_active_host, active_rows_dev, Y_final_dev);
    hipStream_t s = h->stream;
    // Kernels may be queued when a later HIP call fails: nothing of this call is left running on return.
    struct DrainModel {
        hipStream_t s;
        bool armed = true;
        ~DrainModel() {
            if (armed) (void)hipStreamSynchronize(s);
        }
    } drain_model{s};

    for (int32_t l = 1; l <= L; ++l) h->host_counts[l] = -1;  // "not reported yet"
    h->host_counts[0] = batch;
    HIP_TRY(launch_init_lists(h, wv, batch, row_offset));
    int32_t bound = batch;  // upper bound of the rows active at the layer being launched
    int32_t before = -1;    // the bound one layer earlier
    int32_t run = 0;        // layers launched
    float* Y_last = nullptr;  // where the last layer launched writes
    // Out-of-core weights (Section III-B-1): pass p runs from device slot p & 1.  The copy stream fills
    // the two slots, and refills a slot with pass p + 2 as soon as the kernels of pass p are done with
    // it, so the transfer of the next layer runs under the current layer's kernel.
    const int32_t P = (int32_t)h->layers.size();
    auto ooc_fetch = [&](int32_t p) -> hipError_t {
        hipError_t e = hipMemcpyAsync(h->ooc_slot[p & 1], h->ooc_host + (size_t)p * h->ooc_block, h->ooc_block,
                                      hipMemcpyHostToDevice, h->ooc_stream);
        return e != hipSuccess ? e : hipEventRecord(h->ooc_ready[p & 1], h->ooc_stream);
    };
    // whatever happens below, the copy stream is idle again when the call returns
    struct Drain {
        hipStream_t cs;
        ~Drain() {
            if (cs) (void)hipStreamSynchronize(cs);
        }
    } drain{h->ooc_stream};
    if (h->ooc_host)
        for (int32_t p = 0; p < std::min(P, 2); ++p) HIP_TRY(ooc_fetch(p));
    for (int32_t l = 0; l < L; ++l) {
        const float* Yin = (l == 0) ? Y0_dev : wv.Y[(l - 1) & 1];
        float* Yout = wv.Y[l & 1];
        if (l == L - 1 && write_through(h, Y_final_dev, bound, bound == before)) Yout = Y_final_dev;
        Y_last = Yout;
        if (h->profiling) HIP_TRY(hipEventRecord(h->t0[l], s));
        // one launch per pass: a layer is a single pass unless some neuron has more than 32 connections
        for (int32_t p = h->first_pass[l]; p < h->first_pass[l + 1]; ++p) {
            const LayerDesc& d = h->layers[p];
            if (d.multi && d.virt_blocks == 0 && p != h->first_pass[l]) continue;  // no workgroup of the layer is left for this launch
            if (h->ooc_host) HIP_TRY(hipStreamWaitEvent(s, h->ooc_ready[p & 1], 0));
            const spdnn::RowLists rl = layer_lists(h, wv, l, p == h->first_pass[l]);
            HIP_TRY(launch_layer(h, d, Yin, Yout, wv.flags[l % 3], rl, bound));
            ++h->launches;
            if (h->ooc_host) {  // the slot is free once this kernel is done: refill it with pass p + 2
                HIP_TRY(hipEventRecord(h->ooc_freed[p & 1], s));
                if (p + 2 < P) {
                    HIP_TRY(hipStreamWaitEvent(h->ooc_stream, h->ooc_freed[p & 1], 0));
                    HIP_TRY(ooc_fetch(p + 2));
                }
            }
        }
        if (h->profiling) HIP_TRY(hipEventRecord(h->t1[l], s));
        run = l + 1;
        // Feedback with bounded lag: the number of rows active on entry to layer l+2-kLag bounds all later
        // ones.  That layer's kernel stores it to pinned host memory as it starts, which is polled here
        // (so at most kLag-1 kernels are queued behind the running one); the stream is asked now and then
        // whether it has run dry, only so that a failed launch ends the wait.  Nothing else is put between two
        // layers' kernels: an event recorded after every layer made the gap between them longer.
        if (l + 2 >= kLag) {
            int32_t c = 0;
            const int rc = wait_count(h, l + 2 - kLag, &c);
            if (rc != SPDNN_OK) return rc;
            before = bound;
            bound = c;
            if (bound == 0) break;
        }
    }
    // the rows that survive the last layer launched: the same compaction, as a kernel of its own; its count goes to
    // host_counts[run] (rows on entry to the layer that would come next)
    const int rc = finish_infer(h, wv.flags[(run + 2) % 3], wv.count[(run + 1) & 1], wv.gid[(run + 1) & 1], batch, row_offset, wv.count[run & 1],
                                wv.cat[run & 1], run, Y_last, wv.Y[run & 1], bound, n_active_host, active_rows_dev, Y_final_dev);
    if (rc != SPDNN_OK) return rc;
    drain_model.armed = false;
    if (h->profiling) {
        h->prof_layers = run;
        h->prof_ms.assign(run, 0.0f);
        h->prof_rows.assign(run, 0);
        for (int32_t l = 0; l < run; ++l) {
            h->prof_rows[l] = h->host_counts[l];
            HIP_TRY(hipEventElapsedTime(&h->prof_ms[l], h->t0[l], h->t1[l]));
        }
    }
    return SPDNN_OK;
}

}  // namespace

extern "C" {

const char* spdnn_last_error(void) { return g_err.c_str(); }

int spdnn_weights_bytes(int32_t N, int32_t L, size_t* bytes) {
    if (!bytes) return fail(SPDNN_EINVAL, "bytes is NULL");
    if (!valid_n(N) || L < 1) return fail(SPDNN_EINVAL, "need 32 <= N <= 65536, N %% 4 == 0, L >= 1");
    *bytes = arena_bytes_for(N, L, stages_of(N));
    return SPDNN_OK;
}

int spdnn_weights_bytes_for_window(int32_t N, int32_t L, int32_t widest_window, size_t* bytes) {
    if (!bytes) return fail(SPDNN_EINVAL, "bytes is NULL");
    if (!valid_n(N) || L < 1 || widest_window < 1)
        return fail(SPDNN_EINVAL, "need 32 <= N <= 65536, N %% 4 == 0, L >= 1, widest_window >= 1");
    *bytes = arena_bytes_for(N, L, stages_of(std::min(widest_window, N)));
    return SPDNN_OK;
}

int spdnn_scan_windows(int32_t N, int32_t L, const int32_t* const* idx, int32_t where, void* scratch_dev,
                       size_t scratch_bytes, void* hip_stream, int32_t* widest_window) {
    return guarded([&]() -> int {
        if (!widest_window) return fail(SPDNN_EINVAL, "widest_window is NULL");
        if (!valid_n(N) || L < 1) return fail(SPDNN_EINVAL, "need 32 <= N <= 65536, N %% 4 == 0, L >= 1");
        if (!idx || !scratch_dev) return fail(SPDNN_EINVAL, "null argument");
        if (where != SPDNN_HOST && where != SPDNN_DEVICE) return fail(SPDNN_EINVAL, "where must be SPDNN_HOST or SPDNN_DEVICE");
        const int32_t nblk = (N + spdnn::kBlk - 1) / spdnn::kBlk;
        const size_t raw = up((size_t)N * spdnn::kNnz * sizeof(int32_t));
        const size_t need = raw + up((size_t)nblk * sizeof(int2)) + up(sizeof(int));
        if (scratch_bytes < need) return fail(SPDNN_ESIZE, "scan scratch has %zu bytes, %zu needed", scratch_bytes, need);
        if (reinterpret_cast<uintptr_t>(scratch_dev) % kAlign) return fail(SPDNN_EINVAL, "scratch must be 256-byte aligned");
        hipStream_t stream = reinterpret_cast<hipStream_t>(hip_stream);
        char* base = static_cast<char*>(scratch_dev);
        int32_t* st_idx = reinterpret_cast<int32_t*>(base);
        int2* win = reinterpret_cast<int2*>(base + raw);
        int* err = reinterpret_cast<int*>(base + raw + up((size_t)nblk * sizeof(int2)));
        HIP_TRY(hipMemsetAsync(err, 0, 2 * sizeof(int), stream));  // error flag, widest window (unused here)
        std::vector<int2> hw(nblk);
        int widest = 4;
        for (int32_t l = 0; l < L; ++l) {
            if (!idx[l]) return fail(SPDNN_EINVAL, "idx[%d] is NULL", l);
            const int32_t* di = idx[l];
            if (where == SPDNN_HOST) {
                HIP_TRY(hipMemcpyAsync(st_idx, idx[l], (size_t)N * spdnn::kNnz * sizeof(int32_t), hipMemcpyHostToDevice, stream));
                di = st_idx;
            }
            spdnn::block_window_kernel<<<nblk, spdnn::kBlk, 0, stream>>>(di, N, win, err, err + 1);
            HIP_TRY(hipGetLastError());
            HIP_TRY(hipMemcpyAsync(hw.data(), win, sizeof(int2) * nblk, hipMemcpyDeviceToHost, stream));
            HIP_TRY(hipStreamSynchronize(stream));
            for (int32_t b = 0; b < nblk; ++b) widest = std::max(widest, hw[b].y);
            // layers that run two neurons per lane give blocks 2u and 2u+1 their common window
            if (N % (2 * spdnn::kBlk) == 0)
                for (int32_t b = 0; b + 1 < nblk; b += 2) {
                    int x, y;  // windows are cyclic
                    spdnn::win_union(hw[b].x, hw[b].y, hw[b + 1].x, hw[b + 1].y, N, x, y);
                    widest = std::max(widest, y);
                }
        }
        int herr = 0;
        HIP_TRY(hipMemcpy(&herr, err, sizeof(int), hipMemcpyDeviceToHost));
        if (herr) return fail(SPDNN_EINVAL, "a column index is outside [0, N)");
        *widest_window = widest;
        return SPDNN_OK;
    });
}

int spdnn_work_bytes(int32_t N, int32_t max_batch, size_t* bytes) {
    if (!bytes) return fail(SPDNN_EINVAL, "bytes is NULL");
    if (!valid_n(N) || max_batch < 0) return fail(SPDNN_EINVAL, "need 32 <= N <= 65536, N %% 4 == 0, batch >= 0");
    *bytes = carve_work(N, max_batch, nullptr, nullptr);
    return SPDNN_OK;
}

int spdnn_create(spdnn_t* out, int32_t N, int32_t L, const int32_t* const* idx, const float* const* val,
                 const float* bias, int32_t where, void* weights_arena, size_t weights_arena_bytes,
                 void* hip_stream) {
    return guarded([&]() -> int {
        if (!out) return fail(SPDNN_EINVAL, "out is NULL");
        *out = nullptr;
        if (!valid_n(N) || L < 1) return fail(SPDNN_EINVAL, "need 32 <= N <= 65536, N %% 4 == 0, L >= 1");
        if (!idx || !val || !bias || !weights_arena) return fail(SPDNN_EINVAL, "null argument");
        if (where != SPDNN_HOST && where != SPDNN_DEVICE) return fail(SPDNN_EINVAL, "where must be SPDNN_HOST or SPDNN_DEVICE");
        if (reinterpret_cast<uintptr_t>(weights_arena) % kAlign) return fail(SPDNN_EINVAL, "weights_arena must be 256-byte aligned");
        for (int32_t l = 0; l < L; ++l)
            if (!idx[l] || !val[l]) return fail(SPDNN_EINVAL, "idx[%d] or val[%d] is NULL", l, l);
        return create_impl(out, N, L, std::vector<int32_t>((size_t)L, 1), nullptr, idx, val, bias, where, weights_arena,
                           weights_arena_bytes, reinterpret_cast<hipStream_t>(hip_stream));
    });
}

int spdnn_ooc_bytes(int32_t N, int32_t L, int32_t widest_window, size_t* device_bytes, size_t* host_bytes) {
    if (!device_bytes || !host_bytes) return fail(SPDNN_EINVAL, "null argument");
    if (!valid_n(N) || L < 1 || widest_window < 1)
        return fail(SPDNN_EINVAL, "need 32 <= N <= 65536, N %% 4 == 0, L >= 1, widest_window >= 1");
    const int cap = stages_of(std::min(widest_window, N));
    *device_bytes = ooc_device_bytes_for(N, L, cap);
    *host_bytes = (size_t)L * block_bytes(N, cap);
    return SPDNN_OK;
}

int spdnn_create_ooc(spdnn_t* out, int32_t N, int32_t L, const int32_t* const* idx, const float* const* val,
                     const float* bias, int32_t where, void* device_arena, size_t device_arena_bytes,
                     void* host_arena, size_t host_arena_bytes, void* hip_stream) {
    return guarded([&]() -> int {
        if (!out) return fail(SPDNN_EINVAL, "out is NULL");
        *out = nullptr;
        if (!valid_n(N) || L < 1) return fail(SPDNN_EINVAL, "need 32 <= N <= 65536, N %% 4 == 0, L >= 1");
        if (!idx || !val || !bias || !device_arena || !host_arena) return fail(SPDNN_EINVAL, "null argument");
        if (where != SPDNN_HOST && where != SPDNN_DEVICE) return fail(SPDNN_EINVAL, "where must be SPDNN_HOST or SPDNN_DEVICE");
        if (reinterpret_cast<uintptr_t>(device_arena) % kAlign || reinterpret_cast<uintptr_t>(host_arena) % 16)
            return fail(SPDNN_EINVAL, "device_arena must be 256-byte aligned, host_arena 16-byte aligned");
        for (int32_t l = 0; l < L; ++l)
            if (!idx[l] || !val[l]) return fail(SPDNN_EINVAL, "idx[%d] or val[%d] is NULL", l, l);
        return create_impl(out, N, L, std::vector<int32_t>((size_t)L, 1), nullptr, idx, val, bias, where, device_arena,
                           device_arena_bytes, reinterpret_cast<hipStream_t>(hip_stream), host_arena, host_arena_bytes);
    });
}

int spdnn_csr_passes(int32_t N, int32_t L, const int32_t* const* ptr, const int32_t* const* idx, void* scratch_dev,
                     size_t scratch_bytes, void* hip_stream, int32_t* passes, int32_t* total, int32_t* widest_window) {
    return guarded([&]() -> int {
        if (!valid_n(N) || L < 1) return fail(SPDNN_EINVAL, "need 32 <= N <= 65536, N %% 4 == 0, L >= 1");
        if (!ptr || !scratch_dev || !total) return fail(SPDNN_EINVAL, "null argument");
        if (widest_window && !idx) return fail(SPDNN_EINVAL, "widest_window needs idx");
        std::vector<int32_t> po;
        const int rc = scan_csr(N, L, ptr, scratch_dev, scratch_bytes, reinterpret_cast<hipStream_t>(hip_stream), &po, idx,
                                widest_window);
        if (rc != SPDNN_OK) return rc;
        int64_t sum = 0;
        for (int32_t l = 0; l < L; ++l) {
            if (passes) passes[l] = po[l];
            sum += po[l];
        }
        if (sum > INT32_MAX) return fail(SPDNN_EINVAL, "too many passes");
        *total = (int32_t)sum;
        return SPDNN_OK;
    });
}

int spdnn_create_csr(spdnn_t* out, int32_t N, int32_t L, const int32_t* const* ptr, const int32_t* const* idx,
                     const float* const* val, const float* bias, void* weights_arena, size_t weights_arena_bytes,
                     void* hip_stream) {
    return guarded([&]() -> int {
        if (!out) return fail(SPDNN_EINVAL, "out is NULL");
        *out = nullptr;
        if (!valid_n(N) || L < 1) return fail(SPDNN_EINVAL, "need 32 <= N <= 65536, N %% 4 == 0, L >= 1");
        if (!ptr || !idx || !val || !bias || !weights_arena) return fail(SPDNN_EINVAL, "null argument");
        if (reinterpret_cast<uintptr_t>(weights_arena) % kAlign) return fail(SPDNN_EINVAL, "weights_arena must be 256-byte aligned");
        for (int32_t l = 0; l < L; ++l)
            if (!ptr[l] || !idx[l] || !val[l]) return fail(SPDNN_EINVAL, "ptr[%d], idx[%d] or val[%d] is NULL", l, l, l);
        // the arena's head serves as scratch for the scan; nothing else is in it yet
        hipStream_t stream = reinterpret_cast<hipStream_t>(hip_stream);
        std::vector<int32_t> passes_of;
        const int rc = scan_csr(N, L, ptr, weights_arena, weights_arena_bytes, stream, &passes_of);
        if (rc != SPDNN_OK) return rc;
        return create_impl(out, N, L, passes_of, ptr, idx, val, bias, SPDNN_DEVICE, weights_arena, weights_arena_bytes, stream);
    });
}

int spdnn_destroy(spdnn_t h) {
    return guarded([&]() -> int {
        if (!h) return SPDNN_OK;
        if (h->host_counts) (void)hipHostFree(h->host_counts);
        for (int i = 0; i < 2; ++i) {
            if (h->ooc_ready[i]) (void)hipEventDestroy(h->ooc_ready[i]);
            if (h->ooc_freed[i]) (void)hipEventDestroy(h->ooc_freed[i]);
        }
        if (h->ooc_stream) (void)hipStreamDestroy(h->ooc_stream);
        for (hipEvent_t e : h->in_ready)
            if (e) (void)hipEventDestroy(e);
        if (h->in_stream) (void)hipStreamDestroy(h->in_stream);
        for (hipEvent_t e : h->t0) (void)hipEventDestroy(e);
        for (hipEvent_t e : h->t1) (void)hipEventDestroy(e);
        delete h;
        return SPDNN_OK;
    });
}

int spdnn_set_profiling(spdnn_t h, int32_t on) {
    return guarded([&]() -> int {
        if (!h) return fail(SPDNN_EINVAL, "handle is NULL");
        if (on && h->t0.empty()) {
            h->t0.resize(h->L, nullptr);
            h->t1.resize(h->L, nullptr);
            for (int32_t l = 0; l < h->L; ++l) {
                HIP_TRY(hipEventCreate(&h->t0[l]));
                HIP_TRY(hipEventCreate(&h->t1[l]));
            }
        }
        h->profiling = on ? 1 : 0;
        return SPDNN_OK;
    });
}

int spdnn_layer_kernel(spdnn_t h, int32_t l, int32_t* kind) {
    if (!h || !kind) return fail(SPDNN_EINVAL, "null argument");
    if (l < 0 || l >= h->L) return fail(SPDNN_EINVAL, "layer %d outside [0, %d)", l, h->L);
    static_assert(kSingle == SPDNN_KERNEL_SINGLE && kStaged == SPDNN_KERNEL_STAGED && kWide == SPDNN_KERNEL_WIDE &&
                      kPair == SPDNN_KERNEL_PAIR && kWidePair == SPDNN_KERNEL_WIDE_PAIR,
                  "layer modes are the header's kernel kinds");
    const LayerDesc& d = h->layers[h->first_pass[l]];
    *kind = d.mode == kWidePair && d.pair4 ? SPDNN_KERNEL_WIDE_PAIR4
            : d.mode == kRow2              ? SPDNN_KERNEL_ROW2
            : d.mode == kFlat              ? SPDNN_KERNEL_FLAT
                                           : d.mode;
    return SPDNN_OK;
}

int spdnn_one_launch(spdnn_t h, int32_t batch, int32_t* yes) {
    if (!h || !yes) return fail(SPDNN_EINVAL, "null argument");
    if (batch < 0) return fail(SPDNN_EINVAL, "batch < 0");
    *yes = one_launch(h, batch) ? 1 : 0;
    return SPDNN_OK;
}

int spdnn_get_launches(spdnn_t h, int32_t* launches, int32_t* resident) {
    if (!h || !launches) return fail(SPDNN_EINVAL, "null argument");
    *launches = h->launches;
    if (resident) *resident = h->res_launches;
    return SPDNN_OK;
}

int spdnn_row_kernel(spdnn_t h, int32_t* kind) {
    if (!h || !kind) return fail(SPDNN_EINVAL, "null argument");
    *kind = h->row_kernel;
    return SPDNN_OK;
}

int spdnn_layer_passes(spdnn_t h, int32_t l, int32_t* passes) {
    if (!h || !passes) return fail(SPDNN_EINVAL, "null argument");
    if (l < 0 || l >= h->L) return fail(SPDNN_EINVAL, "layer %d outside [0, %d)", l, h->L);
    *passes = h->first_pass[l + 1] - h->first_pass[l];
    return SPDNN_OK;
}

int spdnn_get_profile(spdnn_t h, int32_t cap, int32_t* layers_run, int32_t* rows_in, float* fused_ms) {
    return guarded([&]() -> int {
        if (!h || !layers_run) return fail(SPDNN_EINVAL, "null argument");
        *layers_run = h->prof_layers;
        const int32_t n = std::min<int32_t>(cap, h->prof_layers);
        for (int32_t l = 0; l < n; ++l) {
            if (rows_in) rows_in[l] = h->prof_rows[l];
            if (fused_ms) fused_ms[l] = l < (int32_t)h->prof_ms.size() ? h->prof_ms[l] : 0.0f;
        }
        return SPDNN_OK;
    });
}

int spdnn_infer(spdnn_t h, const float* Y0_dev, int32_t batch, void* work_arena, size_t work_arena_bytes,
                int32_t* n_active_host, int32_t* active_rows_dev, float* Y_final_dev) {
    return guarded([&]() -> int {
        const int rc = check_infer_args(h, Y0_dev, batch, n_active_host, active_rows_dev, Y_final_dev);
        if (rc != SPDNN_OK || batch == 0) return rc;
        if (!work_arena) return fail(SPDNN_EINVAL, "null argument");
        if (reinterpret_cast<uintptr_t>(work_arena) % kAlign) return fail(SPDNN_EINVAL, "work_arena must be 256-byte aligned");
        const size_t need = carve_work(h->N, batch, nullptr, nullptr);
        if (work_arena_bytes < need) return fail(SPDNN_ESIZE, "work arena has %zu bytes, %zu needed", work_arena_bytes, need);
        WorkView wv;
        carve_work(h->N, batch, static_cast<char*>(work_arena), &wv);
        return infer_impl(h, Y0_dev, batch, wv, 0, n_active_host, active_rows_dev, Y_final_dev);
    });
}

int spdnn_infer_static(spdnn_t h, const float* Y0_dev, int32_t batch, int32_t* n_active_host,
                       int32_t* active_rows_dev, float* Y_final_dev) {
    return guarded([&]() -> int {
        const int rc = check_infer_args(h, Y0_dev, batch, n_active_host, active_rows_dev, Y_final_dev);
        if (rc != SPDNN_OK || batch == 0) return rc;
        const size_t need = carve_work(h->N, batch, nullptr, nullptr);
        if (need > kStaticScratchBytes)
            return fail(SPDNN_ESIZE,
                        "batch %d x N %d needs %zu bytes of scratch, the static scratch array holds %zu: use spdnn_infer "
                        "with a work arena",
                        batch, h->N, need, kStaticScratchBytes);
        void* ptr = nullptr;
        const int rs = static_scratch(&ptr);  // this device's copy of the array (looked up at spdnn_create)
        if (rs != SPDNN_OK) return rs;
        WorkView wv;
        carve_work(h->N, batch, static_cast<char*>(ptr), &wv);
        return infer_impl(h, Y0_dev, batch, wv, 0, n_active_host, active_rows_dev, Y_final_dev);
    });
}

int spdnn_host_work_bytes(int32_t N, int32_t rows_per_batch, size_t* bytes) {
    if (!bytes) return fail(SPDNN_EINVAL, "bytes is NULL");
    if (!valid_n(N) || rows_per_batch < 1) return fail(SPDNN_EINVAL, "need 32 <= N <= 65536, N %% 4 == 0, rows_per_batch >= 1");
    *bytes = 2 * up((size_t)rows_per_batch * N * sizeof(float)) + carve_work(N, rows_per_batch, nullptr, nullptr);
    return SPDNN_OK;
}

int spdnn_infer_host(spdnn_t h, const float* Y0_host, int32_t batch, int32_t rows_per_batch, void* work_arena,
                     size_t work_arena_bytes, int32_t* n_active_host, int32_t* active_rows_dev, float* Y_final_dev) {
    return guarded([&]() -> int {
        if (!h) return fail(SPDNN_EINVAL, "handle is NULL");
        if (!n_active_host) return fail(SPDNN_EINVAL, "n_active_host is NULL");
        if (batch < 0 || rows_per_batch < 1) return fail(SPDNN_EINVAL, "need batch >= 0 and rows_per_batch >= 1");
        h->prof_layers = 0;
        h->launches = h->res_launches = h->row_kernel = 0;
        *n_active_host = 0;
        if (batch == 0) return SPDNN_OK;
        if (!Y0_host || !work_arena || !active_rows_dev) return fail(SPDNN_EINVAL, "null argument");
        if (Y_final_dev && reinterpret_cast<uintptr_t>(Y_final_dev) % 16) return fail(SPDNN_EINVAL, "Y_final must be 16-byte aligned");
        if (reinterpret_cast<uintptr_t>(work_arena) % kAlign) return fail(SPDNN_EINVAL, "work_arena must be 256-byte aligned");
        const int32_t N = h->N;
        const int32_t step = std::min(rows_per_batch, batch);
        const size_t in_bytes = up((size_t)step * N * sizeof(float));
        const size_t need = 2 * in_bytes + carve_work(N, step, nullptr, nullptr);
        if (work_arena_bytes < need) return fail(SPDNN_ESIZE, "work arena has %zu bytes, %zu needed", work_arena_bytes, need);
        char* base = static_cast<char*>(work_arena);
        float* in[2] = {reinterpret_cast<float*>(base), reinterpret_cast<float*>(base + in_bytes)};
        WorkView wv;
        carve_work(N, step, base + 2 * in_bytes, &wv);
        if (!h->in_stream) {  // made on first use: a second stream of default priority, and one event per input buffer
            HIP_TRY(hipStreamCreateWithFlags(&h->in_stream, hipStreamNonBlocking));
            for (hipEvent_t& e : h->in_ready) HIP_TRY(hipEventCreateWithFlags(&e, hipEventDisableTiming));
        }
        // whatever happens below, the copy stream is idle again when the call returns
        struct Drain {
            hipStream_t cs;
            ~Drain() { (void)hipStreamSynchronize(cs); }
        } drain{h->in_stream};
        // The batches, and the last one in pieces of one half, a quarter, ..., a piece being copied while the one before it is
        // inferred: what is left to do when the last byte has come is a piece, not a batch (6000 rows of 4096 neurons through 24
        // layers in batches of 1500: 2110 -> 2026 us; in one batch 2319 -> 2034).  Only where copying takes longer than inferring:
        // 4 bytes per neuron and row at PCIe's 55 GB/s against 32 multiply-adds per layer, and what a layer takes however few
        // rows it has, which every piece takes again, so the line is at bytes per layer.  4096 neurons, whole -> pieces, MB per
        // layer in the batch that is cut: 1.4 (12 layers) 493 -> 447 us, 0.9 (24, three batches) 1509 -> 1471, 0.6 (36, three batches)
        // 1648 -> 1736; 2500 neurons, 1.0 (24) 726 -> 706, 0.5 (48) 929 -> 1053.  A launch per layer: 16384 neurons, 8.2 (12) 2357 ->
        // 2186, 1.6 (12) 657 -> 686; windows of 16384 columns, 1.3 (22) 980 -> 1040; 12128 neurons, 1.5 (18, seven batches) 4182 -> 4380.
        // Weights out of core go over PCIe too, with every piece again: never cut.  Nor are inputs in pageable memory, where a piece's
        // copy is over before the next call to the GPU is made and every piece takes its layers' fixed times for nothing (4096 neurons,
        // 24 layers, 6000 rows, whole -> pieces 4107 -> 4584 us; 16384, 6 layers, 2000 rows 5260 -> 5584).
        struct Piece {
            int32_t first, rows;
            float* to;
            hipEvent_t ready;
        };
        std::vector<Piece> pieces;
        const size_t passes = (size_t)h->first_pass.back();
        const bool cut = h->L <= (h->strided ? kStridedCopyBoundLayers : kCopyBoundLayers) && !h->ooc_host && pinned(Y0_host);
        const size_t cut_bytes = h->strided ? std::max(kStridedPieceBytes, kStridedPieceBytesPerLayer * passes)
                                            : std::max(kPieceBytes, (h->res_layers ? kPieceBytesPerLayer : kPieceBytesPerLaunch) * passes);
        for (int32_t k = 0, first = 0; first < batch; ++k) {
            int32_t rows = std::min(step, batch - first);
            float* to = in[k & 1];
            if (cut && first + rows == batch)
                for (int i = 2; i < kInEvents && (size_t)rows * N * sizeof(float) >= cut_bytes; ++i) {
                    const int32_t half = rows / 2 & ~7;
                    pieces.push_back(Piece{first, half, to, h->in_ready[i]});
                    first += half;
                    rows -= half;
                    to += (size_t)half * N;
                }
            pieces.push_back(Piece{first, rows, to, h->in_ready[k & 1]});
            first += rows;
        }
        auto fetch = [&](const Piece& p) -> hipError_t {  // on the copy stream
            hipError_t e = hipMemcpyAsync(p.to, Y0_host + (size_t)p.first * N, sizeof(float) * (size_t)p.rows * N, hipMemcpyHostToDevice, h->in_stream);
            return e != hipSuccess ? e : hipEventRecord(p.ready, h->in_stream);
        };
        // A batch is fetched while the one before it is inferred: the buffer it goes to was last read by the batch before that,
        // whose inference has drained the model's stream.
        size_t fetched = 0;
        const auto fetch_batch = [&]() -> hipError_t {  // the next batch: the pieces up to the next one at the start of a buffer
            do {
                const hipError_t e = fetch(pieces[fetched]);
                if (e != hipSuccess) return e;
                ++fetched;
            } while (fetched < pieces.size() && pieces[fetched].to != in[0] && pieces[fetched].to != in[1]);
            return hipSuccess;
        };
        HIP_TRY(fetch_batch());
        int32_t total = 0;
        for (size_t k = 0; k < pieces.size(); ++k) {
            const Piece& p = pieces[k];
            HIP_TRY(hipStreamWaitEvent(h->stream, p.ready, 0));
            if (k + 1 == fetched && fetched < pieces.size()) HIP_TRY(fetch_batch());
            int32_t n = 0;
            const int rc = infer_impl(h, p.to, p.rows, wv, p.first, &n, active_rows_dev + total,
                                      Y_final_dev ? Y_final_dev + (size_t)total * N : nullptr);
            if (rc != SPDNN_OK) return rc;
            total += n;
        }
        *n_active_host = total;
        return SPDNN_OK;
    });
}

}  // extern "C"
