// Networks whose layers are strided sums: neuron j of a layer reads the 32 columns (j + off + k * S) mod N, k = 0 .. 31,
// all with one weight -- the building block of the RadiX-Net topologies (Section II-A) -- and one bias for all neurons.
//
// Such a layer is a sliding sum over every orbit of "+S": along an orbit neuron t adds the inputs t .. t + 31, and
// neighbours share 31 of them.  33 neighbours' 64 inputs are cut in two halves: the sums of x[i .. 31] for every i and of
// x[32 .. i] are chains of 31 additions each, and a neuron's sum is one of the first plus one of the second -- 93 additions
// for 33 neurons, 3 per neuron instead of 32 multiply-adds, from 2 reads per neuron instead of 32, and there are no
// connections to store or fetch: a layer is {S, off, weight}.  A sum is 31 additions as before, in two runs, with weight
// and bias in one fused multiply-add at the end.  (Nothing is ever subtracted.  Five rounds of doubling, x[i] += x[i + 1],
// x[i] += x[i + 2], ... + 16, take 263 additions: 383 us where this takes 363.)  The runs are shorter than the chain was, and so is
// the error of dense rows: 0.80 to 0.93 of it, 2-norm, in the first layer, which rounds its products, 0.1 to 0.6 behind later ones.  Where one
// to four of a neuron's 32 inputs are not 0 and the weight is no power of two, the first layer's is 1.0 to 1.12 of it.
//
// Rows stay in LDS over a run of layers, two of them side by side (an entry = the two rows of a column, 8 bytes).  A lane
// owns kStrideOut neighbours of an orbit: it reads its 64 entries into registers, adds, and after a barrier writes its 33
// results over the input.  33 is odd so that lanes next to each other along an orbit of stride 1 (33 entries apart) fall
// into different bank pairs; lanes of orbits next to each other read neighbouring entries anyway.  The last lane of an
// orbit that 33 does not divide writes fewer.  An orbit of exactly 32 (S = N / 32) has one sum for all its neurons: one lane computes it once.
//
// The rows are kept as 1/32 of what they are, where no bit is lost by it (strided_scaled): ReLU and clip are then the clamp of the
// multiply-add that weight and bias take.
// Strides that are powers of two, and the row length a multiple, have code of their own (strided_known): an entry's distance from a
// lane's first is in the read's offset, and a lane that comes past the row end chooses between two addresses.  With one address
// worked out per entry and ReLU and clip instructions of their own before, pairs of rows through layers of one stride, clocks of 2.4 GHz
// per layer of 32768 neurons and rows: 4096 neurons, stride 1 8660 -> 6890, 32 8680 -> 7340, 128 4380 -> 4170, 3 (any other) 8850 -> 7920;
// 16384 neurons 7390 -> 6930, 7400 -> 7510 (the lanes past the row end), 512 4550 -> 4280, 3 7710 -> 7300.  All ten strides in one network take
// more code than the instruction cache holds: 50 layers of 16384 neurons on 2000 rows 401 -> 399 us.
//
// What bounds it: the chain of reading, adding and writing: a CU's LDS has room for the rows of 8 waves, two per SIMD, which meet at two
// barriers per layer.  A wave issues an instruction every 5 clocks, so two do not fill a SIMD; a write of 8 bytes per lane takes the LDS 6.2
// clocks where a read takes 2.5 (33 writes of 8 waves: 1640 clocks, with nothing else to do meanwhile); and the wave that comes past the row
// end has a third more instructions than the others, which wait for it.  48 layers of 16384 neurons,
// strides 1, 32 and 512 in turn, on 2000 rows of which half die: 1.95 -> 0.35 ms (two neurons per lane under new names, one launch per
// layer before: 40 us a layer, 28 for the first two now and 6 for the others, on half the rows); 24 layers of
// 4096 neurons, strides 1, 32 and 128, 60 000 rows 4.45 -> 1.50 ms (resident_kernel before) -> 1.31 with code for known strides, 48 of them on 100 rows 324 -> 133 -> 108 us.
#pragma once

namespace spdnn {

constexpr int kStrideOut = 33;                      // neurons a lane owns
constexpr int kStrideIn = kStrideOut + kNnz - 1;    // inputs they read
constexpr int kStrideThreads = 512;
constexpr int kStrideMisc = 16;  // bytes of LDS behind the rows: an entry that nobody reads, two words of flags

struct StridedLayer {
    int S, off;     // columns (j + off + k * S) mod N
    int orbits, T;  // gcd(N, S) orbits of T columns each
    int per;        // lanes per orbit: ceil(T / 33), 1 if T == 32
    float w;        // the weight of all connections
};
struct StridedArgs {
    const StridedLayer* layers;
    int l0, l1;       // layers l0 .. l1-1
    int A;            // rows, if there are no lists yet (rl.count == NULL): row i is in slot i
    int pairs;        // pairs of rows a pass holds
    float bias;
    int* layer_rows;  // NULL, or counters: [l] += rows alive on entry to layer l
};
SPDNN_HD inline int strided_lanes(const StridedLayer& d) { return d.orbits * d.per; }
// Has strided_kernel code of its own for the layer's stride?  A power of two up to 512 that divides N; and a lane's entries come past
// the row end at most once, or the orbit is one sum.  (The networks of the Sparse DNN Challenge have such strides only.)
SPDNN_HD inline bool strided_known(const StridedLayer& d, int N) {
    return d.S <= 512 && (d.S & (d.S - 1)) == 0 && N % d.S == 0 && (N / d.S >= kStrideIn || N / d.S == kNnz);
}
// Can the rows be kept as 1/32 of what they are, bit for bit?  Below 2^-121 an entry would lose its last bits.  An output is weight times sum (48
// bits at most) and a bias that is not above 0, rounded once: 0, or at least 2^-48 of the bias.  A bias of -2^-60 and more leaves no output
// below 2^-108, and what layer 0's products lose below 2^-121 is far below the last bit of a sum that gets past the bias.  (That layer's weight
// meets its inputs as it is, and the product is scaled: a weight below 2^-121 has no bits to spare.  Sums of inputs
// that are as large overflow five binary places later than unscaled ones.)  Smaller biases, 0 among them: rows as they are,
// with an instruction more per neuron and row (rows that all live: 24 layers of 4096 neurons, strides 1, 32 and 128, 60 000 rows 2195 -> 2308 us,
// 48 layers of 16384 neurons, strides 1, 32 and 512, 2000 rows 615 -> 628).
SPDNN_HD inline bool strided_scaled(float bias) { return bias <= -0x1p-60f; }

// n entries of an orbit, from column c on, every S-th, around the row end.
template <int n>
__device__ __forceinline__ void read_orbit(f32x2 (&x)[n], __attribute__((address_space(3))) char* row, uint32_t c, uint32_t S, uint32_t N) {
    using lds_f2 = __attribute__((address_space(3))) f32x2;
    const uint32_t s8 = 8u * S, back = 8u * S - 8u * N;
    if (__builtin_amdgcn_ballot_w64(c + (n - 1) * S >= N) == 0ull) {  // no lane of the wave gets to the row end
#pragma unroll
        for (int k = 0; k < n; ++k) x[k] = *(const lds_f2*)(row + (8u * c + k * s8));
    } else {
        uint32_t at = 8u * c;
#pragma unroll
        for (int k = 0; k < n; ++k) {
            x[k] = *(const lds_f2*)(row + at);
            at = min(at + s8, at + back);
        }
    }
}

// The same for a stride that is known beforehand and divides N, with what is done with the entries: an entry's distance from the first is
// part of the read, and no addition.  (It has 16 bits: every kFar entries the address moves on.)  base: of the row.
// Both ways have reads and additions in one block of code: only there does the compiler mix them.
template <int n, int S, typename Sums>
__device__ __forceinline__ void sum_stride(f32x2 (&x)[n], uint32_t base, uint32_t c, uint32_t N, Sums sums) {
    using lds_f2 = __attribute__((address_space(3))) f32x2;
    constexpr int kFar = S <= 128 ? n : 65536 / (8 * S);
    if (__builtin_amdgcn_ballot_w64(c + (n - 1) * S >= N) == 0ull) {
        uint32_t at[(n + kFar - 1) / kFar];
#pragma unroll
        for (int g = 0; g < n; g += kFar) {
            at[g / kFar] = base + 8u * c + 8u * S * g;
            if constexpr (kFar < n) asm("" : "+v"(at[g / kFar]));
        }
#pragma unroll
        for (int i = 0; i < n; ++i) {  // as they are added: from the middle on, to both sides
            const int k = i & 1 ? n / 2 + i / 2 : n / 2 - 1 - i / 2;
            x[k] = *(const lds_f2*)(at[k / kFar] + 8u * S * (k % kFar));
        }
        sums();
        asm volatile("");  // (or what the ways have in common would be put behind them)
    } else {
        const uint32_t over = (N - c + S - 1u) / S;  // the first entry past the row end
        const uint32_t gone[2] = {over < 32u ? ~0u << over : 0u, over < 32u ? ~0u : over < 64u ? ~0u << (over - 32u) : 0u};  // bit k: entry k is
        uint32_t at[(n + kFar - 1) / kFar], past[(n + kFar - 1) / kFar];
#pragma unroll
        for (int g = 0; g < n; g += kFar) {
            at[g / kFar] = base + 8u * c + 8u * S * g;
            past[g / kFar] = at[g / kFar] - 8u * N;
            asm("" : "+v"(at[g / kFar]), "+v"(past[g / kFar]));  // (or the choice would be moved in front of the sums that make an address)
        }
#pragma unroll
        for (int i = 0; i < n; ++i) {
            const int k = i & 1 ? n / 2 + i / 2 : n / 2 - 1 - i / 2;
            // A choice by bits: one by a comparison has to wait for VCC, an instruction more per entry where a wave has nothing else to do
            // (24 layers of 4096 neurons, strides 1, 32 and 128, 60 000 rows 1357 us, this way 1287).
            uint32_t mask = (uint32_t)__builtin_amdgcn_sbfe((int)gone[k / 32], k % 32, 1);
            asm("" : "+v"(mask));  // (or it would become a comparison)
            const uint32_t from = (mask & past[k / kFar]) | (~mask & at[k / kFar]);
            x[k] = *(const lds_f2*)(from + 8u * S * (k % kFar));
        }
        sums();
    }
}

// PAIRS: more than one pair of rows, the lanes shared out among them.  KNOWN: all strides are.  SCALED: rows as 1/32.
template <bool PAIRS, bool KNOWN, bool SCALED>
__global__ __launch_bounds__(kStrideThreads) void strided_kernel(const float* __restrict__ Yin, float* __restrict__ Yout,
                                                                 uint8_t* __restrict__ flags, RowLists rl, StridedArgs sa, int N) {
    extern __shared__ __align__(16) char strided_lds[];
    using lds_f2 = __attribute__((address_space(3))) f32x2;
    using lds_f4 = __attribute__((address_space(3))) f32x4;
    using lds_char = __attribute__((address_space(3))) char;
    lds_char* const tile = (lds_char*)strided_lds;
    const int tid = threadIdx.x, lane = tid & 63, nthreads = blockDim.x;
    const int np = PAIRS ? sa.pairs : 1;
    const uint32_t row_bytes = 8u * (uint32_t)N;  // of a pair
    uint32_t* live_word = reinterpret_cast<uint32_t*>(strided_lds + (size_t)np * row_bytes + 8);  // [2], raised by the layers in turn
    const uint32_t live_at = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint32_t*)live_word;
    const int A = rl.count ? __builtin_amdgcn_readfirstlane(*rl.count) : sa.A;
    const int npass = (A + 2 * np - 1) / (2 * np), n4 = N >> 2;
    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
    constexpr float kScale = SCALED ? 1.0f / kClip : 1.0f, kMost = kClip * kScale;  // of the rows in LDS
    const float bias = sa.bias * kScale;
    using clayer = const __attribute__((address_space(4))) StridedLayer;  // constant while the kernel runs: scalar loads

    for (int pass = blockIdx.x; pass < npass; pass += gridDim.x) {
        const int row0 = pass * 2 * np, nrow = min(2 * np, A - row0);
        if (tid < 2) live_word[tid] = 0u;
        // the rows; layer 0 sums inputs of any size, so they meet its weight before they are added up
        const float first_w = sa.l0 == 0 ? ((clayer*)(uintptr_t)sa.layers)->w : 1.0f;
        for (int p = 0; p < np; ++p) {
            const bool one = 2 * p < nrow, two = 2 * p + 1 < nrow;
            const int s0 = !one ? 0 : rl.count ? rl.cat[row0 + 2 * p] : row0 + 2 * p;
            const int s1 = !two ? 0 : rl.count ? rl.cat[row0 + 2 * p + 1] : row0 + 2 * p + 1;
            const f32x4* src0 = reinterpret_cast<const f32x4*>(Yin + (size_t)s0 * N);
            const f32x4* src1 = reinterpret_cast<const f32x4*>(Yin + (size_t)s1 * N);
            for (int t0 = tid; t0 < n4; t0 += 4 * nthreads) {
                f32x4 a[4], b[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int t = min(t0 + i * nthreads, n4 - 1);
                    a[i] = one ? src0[t] : zero;
                    b[i] = two ? src1[t] : zero;
                }
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int t = t0 + i * nthreads;
                    if (t < n4) {
                        a[i] = a[i] * first_w * kScale;
                        b[i] = b[i] * first_w * kScale;
                        lds_f4* to = (lds_f4*)(tile + p * row_bytes + 32u * t);
                        to[0] = f32x4{a[i].x, b[i].x, a[i].y, b[i].y};
                        to[1] = f32x4{a[i].z, b[i].z, a[i].w, b[i].w};
                    }
                }
            }
        }
        uint32_t live = 0u;
        const auto layer_at = [&](int l) -> StridedLayer {
            clayer* d = (clayer*)(uintptr_t)(sa.layers + l);
            return StridedLayer{d->S, d->off, d->orbits, d->T, d->per, d->w};
        };
        StridedLayer cur = layer_at(sa.l0);
        __syncthreads();
        // A layer of stride S (0: of any), up to where its outputs are in place.
        const auto layer = [&](int l, auto Stag, uint32_t& raised) {
            constexpr uint32_t kS = decltype(Stag)::value;
            const uint32_t S = kS ? kS : (uint32_t)cur.S, orbits = kS ? kS : (uint32_t)cur.orbits, T = (uint32_t)cur.T, per = (uint32_t)cur.per;
            const float w = l == 0 ? 1.0f : cur.w;
            const uint32_t lanes = orbits * per;
            // my pair of rows, my orbit, my place on it
            uint32_t me = (uint32_t)tid;
            asm volatile("" : "+v"(me));  // (or the places of all strides' entries would be worked out before the layers, for registers that are not there)
            const uint32_t p = PAIRS ? me / lanes : 0u;
            const uint32_t i = me - p * lanes;
            const bool mine = PAIRS ? p < (uint32_t)np : me < lanes;
            const uint32_t b = i / orbits, r = i - b * orbits;
            const uint32_t t0 = b * kStrideOut, left = T - t0;  // the last lane of an orbit has fewer neurons: `left`
            const uint32_t j0 = kS ? r + t0 * S : (r + t0 * S) % (uint32_t)N;
            uint32_t c0 = j0 + (uint32_t)cur.off;
            c0 = min(c0, c0 - (uint32_t)N);
            const uint32_t base = PAIRS ? p * row_bytes : 0u;
            const uint32_t s8 = 8u * S, back = 8u * S - row_bytes;
            const bool whole = T == (uint32_t)kNnz;  // one sum for all of an orbit
            f32x2 y[kStrideOut];
            uint32_t bits = 0u;
            if (mine) {
                float m0 = 0.0f, m1 = 0.0f;
                const auto finish = [&](f32x2 v) -> f32x2 {
                    v.x = fminf(fmaxf(__builtin_fmaf(w, v.x, bias), 0.0f), kMost);
                    v.y = fminf(fmaxf(__builtin_fmaf(w, v.y, bias), 0.0f), kMost);
                    m0 = fmaxf(m0, v.x);
                    m1 = fmaxf(m1, v.y);
                    return v;
                };
                if (whole) {
                    f32x2 v[kNnz];
                    const auto sums = [&]() {
#pragma unroll
                        for (int h = 1; h < kNnz; h *= 2)
#pragma unroll
                            for (int k = 0; k + h < kNnz; k += 2 * h) v[k] += v[k + h];
                        y[0] = finish(v[0]);
                    };
                    if constexpr (kS != 0) {
                        sum_stride<kNnz, kS>(v, base, c0 & (kS - 1u), (uint32_t)N, sums);  // (all of the orbit, whichever comes first)
                    } else {
                        read_orbit<kNnz>(v, tile + base, c0, S, (uint32_t)N);
                        sums();
                    }
                } else {
                    f32x2 x[kStrideIn];
                    const auto sums = [&]() {
#pragma unroll
                        for (int k = kNnz - 2; k >= 0; --k) x[k] += x[k + 1];  // x[k .. 31]
#pragma unroll
                        for (int k = kNnz + 1; k < kStrideIn; ++k) x[k] += x[k - 1];  // x[32 .. k]
                        y[0] = finish(x[0]);
#pragma unroll
                        for (int k = 1; k < kNnz; ++k) y[k] = finish(x[k] + x[k + kNnz - 1]);
                        y[kNnz] = finish(x[kStrideIn - 1]);
                    };
                    if constexpr (kS != 0) {
                        sum_stride<kStrideIn, kS>(x, base, c0, (uint32_t)N, sums);
                    } else {
                        read_orbit<kStrideIn>(x, tile + base, c0, S, (uint32_t)N);
                        sums();
                    }
                }
                // which rows have a positive output: the wave's first lane of every pair speaks for it
                const unsigned long long pos0 = __builtin_amdgcn_ballot_w64(m0 > 0.0f), pos1 = __builtin_amdgcn_ballot_w64(m1 > 0.0f);
                unsigned long long of_pair = ~0ull;
                bool first = lane == 0;
                if constexpr (PAIRS) {
                    const int from = max((int)(p * lanes) - (tid - lane), 0), to = min((int)((p + 1) * lanes) - (tid - lane), 64);
                    of_pair = (~0ull >> (64 - (to - from))) << from;
                    first = lane == from;
                }
                bits = (pos0 & of_pair ? 1u : 0u) | (pos1 & of_pair ? 2u : 0u);
                // (a plain LDS operation: the compiler's atomic would look for the first active lane on its own)
                if (first) asm volatile("ds_or_b32 %0, %1" ::"v"(live_at + 4u * (uint32_t)(l & 1)), "v"(bits << (2u * p)) : "memory");
            }
            cur = layer_at(min(l + 1, sa.l1 - 1));  // (here nothing else waits for it)
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            __syncthreads();  // every wave has read what it needs of the rows
            raised = live_word[l & 1];  // (on its way while the results go out)
            if (!mine) return;
            const uint32_t nowhere = (uint32_t)np * row_bytes;
            const auto put = [&](auto n, auto value) {  // outputs that stay on this side of the row end
                constexpr int far = kS == 0 || kS <= 128 ? decltype(n)::value : 65536 / (8 * (int)kS);
#pragma unroll
                for (int g = 0; g < decltype(n)::value; g += far) {
                    uint32_t at = base + 8u * j0 + g * s8;
                    if constexpr (kS != 0 && far < decltype(n)::value) asm("" : "+v"(at));
#pragma unroll
                    for (int k = g; k < g + far && k < decltype(n)::value; ++k) *(lds_f2*)(at + (k - g) * s8) = value(k);
                }
                asm volatile("");
            };
            if (whole && kS != 0) {
                put(std::integral_constant<int, kNnz>{}, [&](int) { return y[0]; });
            } else if (whole) {
                uint32_t at = 8u * j0;
#pragma unroll
                for (int k = 0; k < kNnz; ++k) {
                    *(lds_f2*)(tile + (base + at)) = y[0];
                    at = min(at + s8, at + back);
                }
            } else if (__builtin_amdgcn_ballot_w64(j0 + (kStrideOut - 1) * S >= (uint32_t)N) == 0ull) {
                put(std::integral_constant<int, kStrideOut>{}, [&](int k) { return y[k]; });
            } else if constexpr (kS != 0) {  // an orbit ends at the row end
#pragma unroll
                for (int k = 0; k < kStrideOut; ++k) *(lds_f2*)(PAIRS ? ((uint32_t)k < left ? base + 8u * j0 + k * s8 : nowhere) : min(8u * j0 + k * s8, row_bytes)) = y[k];
            } else {
                // an orbit's last lane is always among these: it comes past the row end where the orbit ends
                uint32_t at = 8u * j0;
#pragma unroll
                for (int k = 0; k < kStrideOut; ++k) {
                    *(lds_f2*)(tile + ((uint32_t)k < left ? base + at : nowhere)) = y[k];
                    at = min(at + s8, at + back);
                }
            }
        };
        for (int l = sa.l0; l < sa.l1; ++l) {
            uint32_t raised = 0u;
            if constexpr (!KNOWN) layer(l, std::integral_constant<uint32_t, 0>{}, raised);
            else switch (cur.S) {
#define SPDNN_STRIDE(S_) \
    case S_: layer(l, std::integral_constant<uint32_t, S_>{}, raised); break;
                SPDNN_STRIDE(1) SPDNN_STRIDE(2) SPDNN_STRIDE(4) SPDNN_STRIDE(8) SPDNN_STRIDE(16) SPDNN_STRIDE(32)
                SPDNN_STRIDE(64) SPDNN_STRIDE(128) SPDNN_STRIDE(256)
#undef SPDNN_STRIDE
                default: layer(l, std::integral_constant<uint32_t, 512>{}, raised);
            }
            live = __builtin_amdgcn_readfirstlane(raised);
            if (tid == 0) {
                live_word[(l + 1) & 1] = 0u;
                if (sa.layer_rows && live) atomicAdd(&sa.layer_rows[l + 1], __popc(live));
            }
            __syncthreads();
            if (!live) break;
        }
        if (tid < nrow) flags[row0 + tid] = (live >> tid) & 1u;
        if (live) {
            for (int p = 0; p < np; ++p) {
                const bool one = (live >> (2 * p)) & 1u, two = (live >> (2 * p + 1)) & 1u;
                if (!one && !two) continue;
                f32x4* dst0 = reinterpret_cast<f32x4*>(Yout + (size_t)(row0 + 2 * p) * N);
                f32x4* dst1 = reinterpret_cast<f32x4*>(Yout + (size_t)(row0 + 2 * p + 1) * N);
                for (int t = tid; t < n4; t += nthreads) {
                    const lds_f4* from = (const lds_f4*)(tile + p * row_bytes + 32u * t);
                    const f32x4 u = from[0], v = from[1];
                    if (one) dst0[t] = f32x4{u.x, u.z, v.x, v.z} * (1.0f / kScale);
                    if (two) dst1[t] = f32x4{u.y, u.w, v.y, v.w} * (1.0f / kScale);
                }
            }
        }
        __syncthreads();  // the tile and the live words are free for the next pass
    }
}

// Set-up: is the layer a strided sum?  info[0] != 0: no; info[1] .. info[3]: S, off and the weight's bits, as neuron 0 suggests.  Neuron 0's
// columns, sorted, are an arithmetic sequence on the circle if all gaps but (at most) one are equal; every other neuron has
// to read the same columns moved by its number, each exactly once, with the same weight.
__global__ __launch_bounds__(256) void strided_detect_kernel(const int32_t* __restrict__ idx, const float* __restrict__ val, int N,
                                                             int* __restrict__ info) {
    __shared__ int col[kNnz];
    __shared__ int found[2];
    const int tid = threadIdx.x;
    if (tid < kNnz) {  // rank of my column among neuron 0's
        const int c = idx[tid];
        int rank = 0;
        for (int k = 0; k < kNnz; ++k) {
            const int o = idx[k];
            rank += o < c || (o == c && k < tid);
        }
        col[rank] = c;
    }
    __syncthreads();
    if (tid == 0) {
        int S = 0, off = 0;
        if (col[0] >= 0 && col[kNnz - 1] < N) {
            const auto gap = [&](int k) { return k + 1 < kNnz ? col[k + 1] - col[k] : col[0] + N - col[kNnz - 1]; };
            // the gap that two of three neighbouring ones have in common is the stride; the sequence starts behind the odd one
            const int s = gap(0) == gap(1) ? gap(0) : gap(2);
            int odd = -1, nodd = 0;
            for (int k = 0; k < kNnz; ++k)
                if (gap(k) != s) {
                    odd = k;
                    ++nodd;
                }
            if (s > 0 && nodd <= 1) {
                S = s;
                off = nodd ? col[(odd + 1) % kNnz] : col[0];
            }
        }
        found[0] = S;
        found[1] = off;
        if (blockIdx.x == 0) {
            info[1] = S;
            info[2] = off;
            info[3] = __float_as_int(val[0]);
        }
    }
    __syncthreads();
    const int S = found[0], off = found[1];
    const int j = blockIdx.x * 256 + tid;
    if (j >= N) return;
    bool ok = S > 0;
    if (ok) {
        const float w = val[0];
        int from = j + off;
        from = from >= N ? from - N : from;
        uint32_t seen = 0u;
        for (int k = 0; k < kNnz; ++k) {
            const int c = idx[(size_t)j * kNnz + k];
            int d = c - from;
            d = d < 0 ? d + N : d;
            const int q = d / S;
            ok = ok && c >= 0 && c < N && q < kNnz && q * S == d && __float_as_uint(val[(size_t)j * kNnz + k]) == __float_as_uint(w);
            seen |= 1u << (q & 31);
        }
        ok = ok && seen == 0xffffffffu;
    }
    if (!ok) info[0] = 1;
}

}  // namespace spdnn
