// HIP kernels of libspd for gfx950 (MI355X).
//
// Scan (Sections 3.1-3.3, 4.1): every pair sets LR bits of the LDCA and, when sampled, SR bits of
// the SEAV.  Two kernels record a batch:
//   * direct:  one thread per pair, global atomicOr per bit.  Device-wide random atomics run at a
//              fixed rate on MI355X whatever the footprint, so this path serves small batches.
//   * binned:  a workgroup reads a tile of pairs, turns each pair into bit addresses and
//              counting-sorts them in LDS by sketch bucket (2^S bits); an apply kernel gives one
//              workgroup per bucket, replays the bucket's items into an LDS bitmap with LDS
//              atomicOr, and writes the bucket back with plain stores.  No global atomics on the
//              hot path.  Three item layouts: k_region writes each tile's segments into
//              fixed-capacity (chunk of tiles, bucket) regions, read by k_apply_rg (the default,
//              one pass over the pairs); k_count + k_place write one exact bucket-major stream,
//              read by k_apply_bm; k_bin writes per-tile regions, gathered by k_apply.
// End of window (Sections 3.2-3.3): k_close gives one wavefront per SEA (one RP) or part of one: hot-SE
// lists by ballot, the candidate product with Eq. 3 consistency and the SEU weight test, then the
// ULDC of each candidate (AND over LR rows, popcount by wavefront reduction).
#include <hip/hip_ext.h>

#include "spd_internal.h"

namespace spd {

typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

// A pair as the method sees it: (hip, oip) = the record, or the swapped record for a
// destination-keyed batch (uniform per batch).
__device__ __forceinline__ u32x2 keyed(u32x2 pr, uint32_t swap) { return swap ? u32x2{pr.y, pr.x} : pr; }
// Pair i of a batch, keyed.  Batch pointers come from descriptors in memory, so the compiler
// cannot tell their address space; naming it keeps these global (not flat) loads, which do not
// hold up the LDS wait counter.
typedef __attribute__((address_space(1))) const u32x2 global_u32x2;
__device__ __forceinline__ u32x2 load_pair(const u32x2 *pairs, uint64_t i, uint32_t swap) {
    return keyed(__builtin_nontemporal_load((const global_u32x2 *)pairs + i), swap);
}
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

struct BatchTable {
    BatchDesc b[kMaxGroup];
    uint32_t n;
};
// Index of the batch that tile belongs to: the last one whose first tile is <= tile.
__device__ __forceinline__ uint32_t find_batch(const BatchList &bl, uint32_t tile) {
    uint32_t lo = 0, hi = bl.n;   // b[lo].first_tile <= tile < b[hi].first_tile (b[n] = infinity)
    while (hi - lo > 1) {
        const uint32_t mid = (lo + hi) / 2;
        if (bl.b[mid].first_tile <= tile) lo = mid;
        else hi = mid;
    }
    return lo;
}
// The batch of a tile, from device memory or from the inline copies (constant indices only, so
// that the kernel-argument array is never copied to scratch memory).
__device__ __forceinline__ BatchDesc batch_of(const BatchList &bl, uint32_t tile) {
    if (bl.b) return bl.b[find_batch(bl, tile)];
    BatchDesc B = bl.inl[0];
#pragma unroll
    for (uint32_t i = 1; i < kInlineBatches; ++i)
        if (i < bl.n && bl.inl[i].first_tile <= tile) B = bl.inl[i];
    return B;
}
struct SlotTable {
    SlotPtrs s[kMaxGroup];
};
struct ApplyTable {
    ApplySlot s[kMaxGroup];
};
struct SrcTable {
    const uint32_t *p[kMaxGroup];
};
struct SrcTable16 {
    const uint16_t *p[kMaxGroup];
};

__device__ __forceinline__ void global_or(uint32_t *p, uint32_t v) {
    __hip_atomic_fetch_or(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ bool sampled(uint32_t oip, const Consts &c) {
    // lsb(H1(oip)) >= tau, with lsb(0) = 32 (Section 3.1): the low tau bits are all zero.
    return (mas_hi(oip, c.mul[0], c.add[0]) & c.tau_mask) == 0u;
}

__device__ __forceinline__ uint32_t se_bit(uint32_t oip, const Consts &c) { return mas_hi(oip, c.mul[1], c.add[1]) >> 29; }

__device__ __forceinline__ uint32_t ldc_bit(uint32_t oip, const Consts &c) {
    return top_bits(mas_hi(oip, c.mul[2], c.add[2]), c.sh_k);
}

__device__ __forceinline__ uint32_t ldc_col(uint32_t hip, uint32_t i, const Consts &c) {
    return top_bits(mas_hi(hip, c.mul[3 + i], c.add[3 + i]), c.sh_lc);
}

// Per-row SEAV constants (ISB, IBN, byte offset of the row in a SEA) copied to LDS by one thread
// with constant indices: loops over a runtime row count then read LDS instead of indexing the
// kernel-argument block, which would otherwise be copied to scratch memory.
struct RowLds {
    uint32_t v[3 * kMaxRows];
};
__device__ __forceinline__ void rows_to_lds(RowLds &rl, const Consts &c) {
    if (threadIdx.x == 0) {
#pragma unroll
        for (int k = 0; k < kMaxRows; ++k) {
            rl.v[3 * k] = c.isb[k];
            rl.v[3 * k + 1] = c.ibn[k];
            rl.v[3 * k + 2] = c.row_off[k];
        }
    }
}
__device__ __forceinline__ uint32_t seav_byte_l(uint32_t hip, uint32_t i, const RowLds &rl, const Consts &c) {
    const uint32_t rp = hip & c.rmask;
    const uint32_t lp = (uint32_t)((uint64_t)hip >> c.r);
    return rp * c.sea_bytes + rl.v[3 * i + 2] + row_index(lp, rl.v[3 * i], rl.v[3 * i + 1], c.L);
}

// ------------------------------------------------------------------------------ fill
__global__ void k_fill_u32(uint32_t *__restrict__ p, uint64_t n, uint32_t v) {
    uint64_t i = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x;
    uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    uint64_t n4 = n / 4;
    u32x4 vv = {v, v, v, v};
    for (uint64_t j = i; j < n4; j += stride) reinterpret_cast<u32x4 *>(p)[j] = vv;
    for (uint64_t j = n4 * 4 + i; j < n; j += stride) p[j] = v;
}

hipError_t launch_fill_u32(uint32_t *p, uint64_t n_words, uint32_t value, hipStream_t s) {
    if (n_words == 0) return hipSuccess;
    uint64_t blocks = (n_words / 4 + 255) / 256;
    uint32_t grid = (uint32_t)(blocks < 4096 ? (blocks ? blocks : 1) : 4096);
    hipLaunchKernelGGL(k_fill_u32, dim3(grid), dim3(256), 0, s, p, n_words, value);
    return hipGetLastError();
}

// ------------------------------------------------------------------------------ direct scan
template <bool SEAV_LDS>
__global__ __launch_bounds__(1024) void k_scan_direct(Consts c, BatchTable bt, SlotTable st, uint32_t lds_words) {
    extern __shared__ uint32_t lds[];
    if (SEAV_LDS) {
        for (uint32_t w = threadIdx.x; w < lds_words; w += blockDim.x) lds[w] = 0;
        __syncthreads();
    }
    const uint64_t gtid = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x;
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint32_t bi = 0; bi < bt.n; ++bi) {
        const BatchDesc B = bt.b[bi];
        const SlotPtrs S = st.s[B.slot];
        uint32_t *seav_w = reinterpret_cast<uint32_t *>(S.seav);
        const u32x2 *pairs = reinterpret_cast<const u32x2 *>(B.pairs);
        for (uint64_t i = gtid; i < B.n; i += stride) {
            const u32x2 pr = load_pair(pairs, i, B.swap);
            const uint32_t hip = pr.x, oip = pr.y;
            const uint32_t q = ldc_bit(oip, c);
            for (uint32_t r = 0; r < c.lr; ++r) {
                uint32_t bit = ldca_bit(r, ldc_col(hip, r, c), q, c);
                global_or(S.ldca + (bit >> 5), 1u << (bit & 31u));
            }
            if (sampled(oip, c)) {
                const uint32_t b = se_bit(oip, c);
                for (uint32_t r = 0; r < c.sr; ++r) {
                    uint32_t bit = seav_byte(hip, r, c) * 8u + b;
                    if (SEAV_LDS)
                        atomicOr(&lds[bit >> 5], 1u << (bit & 31u));
                    else
                        global_or(seav_w + (bit >> 5), 1u << (bit & 31u));
                }
            }
        }
    }
    if (SEAV_LDS) {
        // OR the workgroup's SEAV copy into the sketch; untouched words cost nothing.
        __syncthreads();
        uint32_t *seav_w = reinterpret_cast<uint32_t *>(st.s[0].seav);
        for (uint32_t w = threadIdx.x; w < lds_words; w += blockDim.x) {
            uint32_t v = lds[w];
            if (v) global_or(seav_w + w, v);
        }
    }
}

hipError_t launch_scan_direct(const Consts &c, const BatchDesc *batches, uint32_t n_batches, const SlotPtrs *slots,
                              uint32_t block, uint32_t grid, bool seav_lds, hipStream_t s) {
    BatchTable bt{};
    SlotTable st{};
    if (n_batches > (uint32_t)kMaxGroup) return hipErrorInvalidValue;
    for (uint32_t i = 0; i < n_batches; ++i) bt.b[i] = batches[i];
    bt.n = n_batches;
    for (int i = 0; i < kMaxGroup; ++i) st.s[i] = slots[i];
    if (seav_lds) {
        uint32_t words = (uint32_t)((c.seav_bytes + 3) / 4);
        hipLaunchKernelGGL(k_scan_direct<true>, dim3(grid), dim3(block), words * 4u, s, c, bt, st, words);
    } else {
        hipLaunchKernelGGL(k_scan_direct<false>, dim3(grid), dim3(block), 0, s, c, bt, st, 0u);
    }
    return hipGetLastError();
}

// ------------------------------------------------------------------------------ sliding scan
// Every bit the discrete scan would set receives the slice's value: a 16-bit stamp, or an 8-bit
// AT code.  All writers of one slice store the same value, and slices are ordered by the stream,
// so plain stores suffice.
template <typename T>
__device__ __forceinline__ T *ldca_counters(const SlotPtrs &S);
template <>
__device__ __forceinline__ uint16_t *ldca_counters<uint16_t>(const SlotPtrs &S) { return S.ldca_ts; }
template <>
__device__ __forceinline__ uint8_t *ldca_counters<uint8_t>(const SlotPtrs &S) { return S.ldca_at; }
template <typename T>
__device__ __forceinline__ T *seav_counters(const SlotPtrs &S);
template <>
__device__ __forceinline__ uint16_t *seav_counters<uint16_t>(const SlotPtrs &S) { return S.seav_ts; }
template <>
__device__ __forceinline__ uint8_t *seav_counters<uint8_t>(const SlotPtrs &S) { return S.seav_at; }

template <typename T>
__global__ __launch_bounds__(1024) void k_scan_stamp(Consts c, BatchTable bt, SlotTable st, uint32_t value) {
    const uint64_t gtid = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x;
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    const T v = (T)value;
    for (uint32_t bi = 0; bi < bt.n; ++bi) {
        const BatchDesc B = bt.b[bi];
        const SlotPtrs S = st.s[B.slot];
        T *ldca = ldca_counters<T>(S), *seav = seav_counters<T>(S);
        const u32x2 *pairs = reinterpret_cast<const u32x2 *>(B.pairs);
        for (uint64_t i = gtid; i < B.n; i += stride) {
            const u32x2 pr = load_pair(pairs, i, B.swap);
            const uint32_t hip = pr.x, oip = pr.y;
            const uint32_t q = ldc_bit(oip, c);
            for (uint32_t r = 0; r < c.lr; ++r) ldca[ldca_bit(r, ldc_col(hip, r, c), q, c)] = v;
            if (sampled(oip, c)) {
                const uint32_t b = se_bit(oip, c);
                for (uint32_t r = 0; r < c.sr; ++r) seav[(uint64_t)seav_byte(hip, r, c) * 8u + b] = v;
            }
        }
    }
}

hipError_t launch_scan_stamp(const Consts &c, const BatchDesc *batches, uint32_t n_batches, const SlotPtrs *slots,
                             uint32_t value, bool at, uint32_t block, uint32_t grid, hipStream_t s, KTiming kt) {
    BatchTable bt{};
    SlotTable st{};
    if (n_batches > (uint32_t)kMaxGroup) return hipErrorInvalidValue;
    for (uint32_t i = 0; i < n_batches; ++i) bt.b[i] = batches[i];
    bt.n = n_batches;
    for (int i = 0; i < kMaxGroup; ++i) st.s[i] = slots[i];
    if (at) hipExtLaunchKernelGGL(k_scan_stamp<uint8_t>, dim3(grid), dim3(block), 0, s, kt.start, kt.stop, 0, c, bt, st, value);
    else hipExtLaunchKernelGGL(k_scan_stamp<uint16_t>, dim3(grid), dim3(block), 0, s, kt.start, kt.stop, 0, c, bt, st, value);
    return hipGetLastError();
}

// AT pool maintenance and views.  A pool is handled 16 counters (one 16-byte vector) per lane.
struct PoolTable {
    uint8_t *p[kMaxGroup];
};
struct CPoolTable {
    const uint8_t *p[kMaxGroup];
};

// Byte k of a 16-byte vector.
__device__ __forceinline__ uint32_t byte_of(const u32x4 &v, uint32_t k) { return (v[k >> 2] >> (8 * (k & 3))) & 0xFFu; }

__global__ __launch_bounds__(256) void k_at_sweep(PoolTable pt, uint32_t n, uint64_t lo16, uint64_t hi16, uint32_t ct,
                                                  uint32_t K) {
    const uint64_t stride = (uint64_t)gridDim.x * 256;
    const uint32_t ex = (ct - K) & (kAtCodes - 1u);   // the code of slice t - K: expired, age K
    for (uint32_t k = 0; k < n; ++k) {
        u32x4 *p = reinterpret_cast<u32x4 *>(pt.p[k]);
        for (uint64_t i = lo16 + blockIdx.x * (uint64_t)256 + threadIdx.x; i < hi16; i += stride) {
            const u32x4 v = p[i];
            u32x4 o = v;
            bool changed = false;
#pragma unroll
            for (uint32_t b = 0; b < 16; ++b) {
                const uint32_t x = byte_of(v, b);
                if (!at_active(x, ct, K) && x != ex) {
                    o[b >> 2] = (o[b >> 2] & ~(0xFFu << (8 * (b & 3)))) | (ex << (8 * (b & 3)));
                    changed = true;
                }
            }
            if (changed) p[i] = o;
        }
    }
}

hipError_t launch_at_sweep(uint8_t *const *pools, uint32_t n, uint64_t lo, uint64_t hi, uint32_t ct, uint32_t K,
                           hipStream_t s) {
    if (lo % 16 || hi % 16 || hi < lo) return hipErrorInvalidValue;
    for (uint32_t k0 = 0; k0 < n; k0 += kMaxGroup) {
        PoolTable pt{};
        const uint32_t m = n - k0 < (uint32_t)kMaxGroup ? n - k0 : (uint32_t)kMaxGroup;
        for (uint32_t k = 0; k < m; ++k) pt.p[k] = pools[k0 + k];
        const uint64_t vec = (hi - lo) / 16;
        if (vec == 0) return hipSuccess;
        const uint32_t grid = (uint32_t)((vec + 255) / 256 < 2048 ? (vec + 255) / 256 : 2048);
        hipLaunchKernelGGL(k_at_sweep, dim3(grid), dim3(256), 0, s, pt, m, lo / 16, hi / 16, ct, K);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// Per counter, the most recent of the sources: the smallest age.  Every source is maintained, so
// every age read modulo 256 is the true age.
__global__ __launch_bounds__(256) void k_at_merge(uint8_t *__restrict__ dst, CPoolTable src, uint32_t n_src,
                                                  uint64_t n16, uint32_t ct) {
    const uint64_t stride = (uint64_t)gridDim.x * 256;
    for (uint64_t i = blockIdx.x * (uint64_t)256 + threadIdx.x; i < n16; i += stride) {
        u32x4 best = reinterpret_cast<const u32x4 *>(src.p[0])[i];
        for (uint32_t k = 1; k < n_src; ++k) {
            const u32x4 v = reinterpret_cast<const u32x4 *>(src.p[k])[i];
#pragma unroll
            for (uint32_t b = 0; b < 16; ++b) {
                const uint32_t x = byte_of(v, b), y = byte_of(best, b);
                if (((ct - x) & (kAtCodes - 1u)) < ((ct - y) & (kAtCodes - 1u)))
                    best[b >> 2] = (best[b >> 2] & ~(0xFFu << (8 * (b & 3)))) | (x << (8 * (b & 3)));
            }
        }
        reinterpret_cast<u32x4 *>(dst)[i] = best;
    }
}

hipError_t launch_at_merge(uint8_t *dst, const uint8_t *const *src, uint32_t n_src, uint64_t n_bytes, uint32_t ct,
                           hipStream_t s) {
    if (n_src == 0 || n_src > (uint32_t)kMaxGroup || n_bytes % 16) return hipErrorInvalidValue;
    CPoolTable t{};
    for (uint32_t k = 0; k < n_src; ++k) t.p[k] = src[k];
    const uint64_t n16 = n_bytes / 16;
    const uint32_t grid = (uint32_t)((n16 + 255) / 256 < 8192 ? (n16 + 255) / 256 : 8192);
    hipLaunchKernelGGL(k_at_merge, dim3(grid ? grid : 1), dim3(256), 0, s, dst, t, n_src, n16, ct);
    return hipGetLastError();
}

// The bits of eight counters (two words) as one byte: counter j of a at bit j, of b at bit 4 + j.
__device__ __forceinline__ uint32_t at_byte(uint32_t a, uint32_t b, const AtView &v) {
    const uint32_t p = ((at_flags4(a, v) >> 4) & 0x08080808u) | (at_flags4(b, v) & 0x80808080u);   // bits 8 j + 3 and 8 j + 7
    return (p * 0x00204081u) >> 24;   // bit 8 j + 3 moves by 21 - 7 j (no two bits meet)
}
// 32 counters (two 16-byte vectors) as one word of bits, in order.
__device__ __forceinline__ uint32_t at_word(const u32x4 &x, const u32x4 &y, const AtView &v) {
    return at_byte(x.x, x.y, v) | at_byte(x.z, x.w, v) << 8 | at_byte(y.x, y.y, v) << 16 | at_byte(y.z, y.w, v) << 24;
}

// Bit view of AT counters.
__global__ __launch_bounds__(256) void k_bit_view_at(const uint8_t *__restrict__ at, uint64_t n_words, AtView v,
                                                     uint32_t *__restrict__ out) {
    const uint64_t stride = (uint64_t)gridDim.x * 256;
    for (uint64_t w = blockIdx.x * (uint64_t)256 + threadIdx.x; w < n_words; w += stride)
        out[w] = at_word(reinterpret_cast<const u32x4 *>(at)[2 * w], reinterpret_cast<const u32x4 *>(at)[2 * w + 1], v);
}

hipError_t launch_bit_view_at(const uint8_t *at, uint64_t n_bits, uint32_t ct, uint32_t K, uint32_t *out_words,
                              hipStream_t s) {
    if (n_bits % 32) return hipErrorInvalidValue;
    const uint64_t words = n_bits / 32;
    const uint32_t grid = (uint32_t)((words + 255) / 256 < 8192 ? (words + 255) / 256 : 8192);
    hipLaunchKernelGGL(k_bit_view_at, dim3(grid ? grid : 1), dim3(256), 0, s, at, words, at_view(ct, K), out_words);
    return hipGetLastError();
}

// ------------------------------------------------------------------------------ binned scan
// Block-wide pass over the bucket counters: cl[b] = LDCA items, cs[b] = SEAV items of bucket b.
// Afterwards cl[b] = first slot of bucket b in the tile's item list, cs[b] = first SEAV slot
// (after the bucket's LDCA items), cl[nb] = total items.
template <int BLOCK>
__device__ void bucket_offsets(uint32_t *cl, uint32_t *cs, uint32_t nb, uint32_t *scratch) {
    constexpr int NW = BLOCK / 64;
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wid = tid >> 6;
    const uint32_t per = (nb + BLOCK - 1) / BLOCK;
    const uint32_t beg = tid * per < nb ? tid * per : nb;
    const uint32_t end = beg + per < nb ? beg + per : nb;
    uint32_t local = 0;
    for (uint32_t b = beg; b < end; ++b) local += cl[b] + cs[b];
    uint32_t incl = local;
    for (int o = 1; o < 64; o <<= 1) {
        uint32_t t = __shfl_up(incl, o, 64);
        if ((int)lane >= o) incl += t;
    }
    if (lane == 63u) scratch[wid] = incl;
    __syncthreads();
    if (tid == 0) {
        uint32_t run = 0;
        for (int w = 0; w < NW; ++w) {
            uint32_t t = scratch[w];
            scratch[w] = run;
            run += t;
        }
        scratch[NW] = run;
    }
    __syncthreads();
    uint32_t run = scratch[wid] + incl - local;
    for (uint32_t b = beg; b < end; ++b) {
        uint32_t l = cl[b], s = cs[b];
        cl[b] = run;
        cs[b] = run + l;
        run += l + s;
    }
    if (tid == 0) cl[nb] = scratch[NW];
    __syncthreads();
}

// Bit addresses of a tile's pairs: LDCA items are counted per bucket in cl (the returned rank is
// kept per item), sampled pairs are staged in samp; once samp is full the rest are recorded directly.
template <int LR, int PPT, int BLOCK, bool FULL>
__device__ __forceinline__ void bin_hash_pairs(const Consts &c, const RowLds &rl, const BinGeometry &g, const SlotPtrs &S,
                                               const u32x2 (&pr)[PPT], uint64_t p0, uint64_t n, uint32_t *cl,
                                               uint32_t *samp, uint32_t *misc, uint32_t (&bits)[PPT * LR],
                                               uint32_t (&rk)[(PPT * LR + 1) / 2]) {
    const uint32_t tid = threadIdx.x;
#pragma unroll
    for (int j = 0; j < PPT; ++j) {
        const bool valid = FULL || p0 + (uint64_t)j * BLOCK + tid < n;
        const uint32_t hip = pr[j].x, oip = pr[j].y;
        const uint32_t q = ldc_bit(oip, c);
#pragma unroll
        for (int r = 0; r < LR; ++r) {
            const int k = j * LR + r;
            const uint32_t bit = ldca_bit((uint32_t)r, ldc_col(hip, (uint32_t)r, c), q, c);
            const uint32_t rank = valid ? atomicAdd(&cl[bit >> g.S], 1u) : 0xFFFFu;
            bits[k] = bit;
            if (k & 1)
                rk[k / 2] |= rank << 16;
            else
                rk[k / 2] = rank;
        }
        if (valid && sampled(oip, c)) {
            const uint32_t b = se_bit(oip, c);
            uint32_t e = atomicAdd(&misc[0], 1u);
            if (e < g.scap) {
                samp[2 * e] = hip;
                samp[2 * e + 1] = b;
            } else {
                // more sampled pairs than the tile reserved: record them directly
                uint32_t *seav_w = reinterpret_cast<uint32_t *>(S.seav);
                for (uint32_t r = 0; r < c.sr; ++r) {
                    uint32_t bit = seav_byte_l(hip, r, rl, c) * 8u + b;
                    global_or(seav_w + (bit >> 5), 1u << (bit & 31u));
                }
            }
        }
    }
}

// Each tile writes its items bucket-major into its own region (item j of the tile in 64-bit word
// j / 3) plus its nb + 1 bucket offsets in meta[tile].
template <int LR, int PPT, int BLOCK>
__global__ __launch_bounds__(BLOCK) void k_bin(Consts c, BinGeometry g, BatchTable bt, SlotTable st,
                                               uint32_t *__restrict__ items, uint32_t *__restrict__ meta) {
    extern __shared__ uint32_t lds[];
    __shared__ RowLds rl;   // read after the first barrier
    rows_to_lds(rl, c);
    const uint32_t nb = g.nb;
    uint32_t *cl = lds;                  // [nb + 1] LDCA counts, then offsets
    uint32_t *cs = cl + (nb + 1);        // [nb + 1] SEAV counts, then cursors
    uint32_t *stage = lds + ((2 * (nb + 1) + 3) & ~3u);  // [cap] bucket-major items (16-byte aligned)
    uint32_t *samp = stage + g.cap;      // [2 * scap] sampled (hip, H2 bit)
    uint32_t *misc = samp + 2 * g.scap;  // [0] sampled count, [1..] scan scratch
    const uint32_t tid = threadIdx.x;
    const uint32_t tile = xcd_contiguous(blockIdx.x, gridDim.x);   // neighbouring tiles on one XCD
    uint32_t bi = 0;
    while (bi + 1 < bt.n && bt.b[bi + 1].first_tile <= tile) ++bi;
    const BatchDesc B = bt.b[bi];
    const SlotPtrs S = st.s[B.slot];
    const uint64_t p0 = (uint64_t)(tile - B.first_tile) * (uint64_t)(PPT * BLOCK);
    const uint32_t smask = (1u << g.S) - 1u;
    const uint32_t seav_base = (uint32_t)c.ldca_bits;   // SEAV bits follow the LDCA bits

    for (uint32_t i = tid; i < 2 * (nb + 1); i += BLOCK) cl[i] = 0;
    if (tid == 0) misc[0] = 0;
    // every lane loads unconditionally (past-the-end lanes re-read the last pair and are masked
    // out below), so all PPT loads of a lane are in flight together
    const u32x2 *pairs = reinterpret_cast<const u32x2 *>(B.pairs);
    const uint64_t last = B.n - 1;
    u32x2 pr[PPT];
#pragma unroll
    for (int j = 0; j < PPT; ++j) {
        const uint64_t idx = p0 + (uint64_t)j * BLOCK + tid;
        pr[j] = load_pair(pairs, idx < B.n ? idx : last, B.swap);
    }
    __syncthreads();

    // per item: its bit address, and its rank inside its bucket (16 bits, two per register;
    // 0xFFFF marks a lane past the end of the batch)
    uint32_t bits[PPT * LR], rk[(PPT * LR + 1) / 2];
    // a full tile (all but the last of a batch) needs no per-pair range test
    if (p0 + (uint64_t)(PPT * BLOCK) <= B.n)
        bin_hash_pairs<LR, PPT, BLOCK, true>(c, rl, g, S, pr, p0, B.n, cl, samp, misc, bits, rk);
    else
        bin_hash_pairs<LR, PPT, BLOCK, false>(c, rl, g, S, pr, p0, B.n, cl, samp, misc, bits, rk);
    __syncthreads();
    // a tile with more sampled pairs than it can stage records all of them directly (the decision
    // depends only on the tile's sampled count, so a counting pass can repeat it)
    uint32_t ns = misc[0];
    if (ns > g.scap) {
        uint32_t *seav_w = reinterpret_cast<uint32_t *>(S.seav);
        for (uint32_t e = tid; e < g.scap; e += BLOCK) {
            const uint32_t hip = samp[2 * e], b = samp[2 * e + 1];
            for (uint32_t r = 0; r < c.sr; ++r) {
                uint32_t bit = seav_byte_l(hip, r, rl, c) * 8u + b;
                global_or(seav_w + (bit >> 5), 1u << (bit & 31u));
            }
        }
        ns = 0;
    }
    for (uint32_t e = tid; e < ns; e += BLOCK) {
        const uint32_t hip = samp[2 * e], b = samp[2 * e + 1];
        for (uint32_t r = 0; r < c.sr; ++r) {
            uint32_t bit = seav_base + seav_byte_l(hip, r, rl, c) * 8u + b;
            atomicAdd(&cs[bit >> g.S], 1u);
        }
    }
    __syncthreads();
    bucket_offsets<BLOCK>(cl, cs, nb, misc + 1);

#pragma unroll
    for (int k = 0; k < PPT * LR; ++k) {
        const uint32_t rank = (rk[k / 2] >> (16 * (k & 1))) & 0xFFFFu;
        if (rank != 0xFFFFu) stage[cl[bits[k] >> g.S] + rank] = bits[k] & smask;
    }
    for (uint32_t e = tid; e < ns; e += BLOCK) {
        const uint32_t hip = samp[2 * e], b = samp[2 * e + 1];
        for (uint32_t r = 0; r < c.sr; ++r) {
            uint32_t bit = seav_base + seav_byte_l(hip, r, rl, c) * 8u + b;
            uint32_t pos = atomicAdd(&cs[bit >> g.S], 1u);
            stage[pos] = bit & smask;
        }
    }
    __syncthreads();
    // items are at most 21 bits (S <= 20): three per 64-bit word
    const uint32_t total = cl[nb];
    uint64_t *out = reinterpret_cast<uint64_t *>(items + (uint64_t)tile * g.region);
    const uint32_t n64 = (total + 2) / 3;
    for (uint32_t i = tid; i < n64; i += BLOCK) {
        const uint32_t j = 3 * i;
        uint64_t v = stage[j];
        if (j + 1 < total) v |= (uint64_t)stage[j + 1] << 21;
        if (j + 2 < total) v |= (uint64_t)stage[j + 2] << 42;
        out[i] = v;
    }
    uint32_t *mo = meta + (uint64_t)tile * (nb + 1);
    for (uint32_t i = tid; i <= nb; i += BLOCK) mo[i] = cl[i];
}

// The bucket counts of bin_hash_pairs without keeping the items.  NEEDQ = false: a bucket holds
// whole LDCs (at least k bits) and a row holds more than one bucket, so a bucket index is the top
// bits of LH_r alone (H3 is not needed).
template <int LR, int PPT, int BLOCK, bool FULL, bool NEEDQ>
__device__ __forceinline__ void count_hash_pairs(const Consts &c, const BinGeometry &g, const u32x2 (&pr)[PPT],
                                                 uint64_t p0, uint64_t n, uint32_t *hl, uint32_t *samp, uint32_t *misc) {
    const uint32_t tid = threadIdx.x;
#pragma unroll
    for (int j = 0; j < PPT; ++j) {
        if (!FULL && p0 + (uint64_t)j * BLOCK + tid >= n) continue;
        const uint32_t hip = pr[j].x, oip = pr[j].y;
        if (NEEDQ) {
            const uint32_t q = ldc_bit(oip, c);
#pragma unroll
            for (int r = 0; r < LR; ++r) {
                uint32_t bit = ldca_bit((uint32_t)r, ldc_col(hip, (uint32_t)r, c), q, c);
                atomicAdd(&hl[bit >> g.S], 1u);
            }
        } else {
            // bucket = (r * LC + col) >> (S - log2 k): the top nbits bits of LH_r, after r's rows
            const uint32_t nbits = c.log2lc + c.log2k - g.S;   // >= 1 on this path
#pragma unroll
            for (int r = 0; r < LR; ++r)
                atomicAdd(&hl[((uint32_t)r << nbits) + (mas_hi(hip, c.mul[3 + r], c.add[3 + r]) >> (32u - nbits))], 1u);
        }
        if (sampled(oip, c)) {   // staged; its SR items are counted by the whole workgroup later
            const uint32_t e = atomicAdd(&misc[0], 1u);
            if (e < g.scap) {
                samp[2 * e] = hip;
                samp[2 * e + 1] = se_bit(oip, c);
            }
        }
    }
}

// Exact per-tile item counts by bucket (the first pass of the bucket-major layout): the same bit
// addresses as k_bin, counted in LDS, SEAV items left out for tiles that record them directly.
template <int LR, int PPT, int BLOCK>
__global__ __launch_bounds__(BLOCK) void k_count(Consts c, BinGeometry g, BatchList bl, ClearList clr,
                                                 uint32_t *__restrict__ cnt) {
    extern __shared__ uint32_t lds[];
    __shared__ RowLds rl;   // read after the first barrier
    rows_to_lds(rl, c);
    const uint32_t nb = g.nb;
    uint32_t *hl = lds;              // [nb] LDCA items
    uint32_t *hs = hl + nb;          // [nb] SEAV items
    uint32_t *misc = hs + nb;        // [0] sampled pairs
    uint32_t *samp = misc + 1;       // [2 * scap] sampled (hip, H2 bit)
    const uint32_t tid = threadIdx.x;
    const uint32_t tile = blockIdx.x;
    const BatchDesc B = bl.b[find_batch(bl, tile)];   // descriptors in device memory
    const uint64_t p0 = (uint64_t)(tile - B.first_tile) * (uint64_t)(PPT * BLOCK);
    for (uint32_t i = tid; i < 2 * nb; i += BLOCK) hl[i] = 0;
    if (tid == 0) misc[0] = 0;
    const u32x2 *pairs = reinterpret_cast<const u32x2 *>(B.pairs);
    const uint64_t last = B.n - 1;
    u32x2 pr[PPT];
#pragma unroll
    for (int j = 0; j < PPT; ++j) {
        const uint64_t idx = p0 + (uint64_t)j * BLOCK + tid;
        pr[j] = load_pair(pairs, idx < B.n ? idx : last, B.swap);
    }
    // the SEAVs of fresh slots, spread over the whole grid (16-byte stores)
    {
        const uint64_t gt = (uint64_t)blockIdx.x * BLOCK + tid, stride = (uint64_t)gridDim.x * BLOCK;
        for (uint32_t k = 0; k < clr.n; ++k) {
            u32x4 *p4 = reinterpret_cast<u32x4 *>(clr.p[k]);
            for (uint64_t w = gt; w < clr.words[k] / 4; w += stride) p4[w] = u32x4{0u, 0u, 0u, 0u};
        }
    }
    __syncthreads();
    const bool full = p0 + (uint64_t)(PPT * BLOCK) <= B.n;
    if (g.S < c.log2k || g.S >= c.log2lc + c.log2k) {
        if (full) count_hash_pairs<LR, PPT, BLOCK, true, true>(c, g, pr, p0, B.n, hl, samp, misc);
        else count_hash_pairs<LR, PPT, BLOCK, false, true>(c, g, pr, p0, B.n, hl, samp, misc);
    } else {
        if (full) count_hash_pairs<LR, PPT, BLOCK, true, false>(c, g, pr, p0, B.n, hl, samp, misc);
        else count_hash_pairs<LR, PPT, BLOCK, false, false>(c, g, pr, p0, B.n, hl, samp, misc);
    }
    __syncthreads();
    const uint32_t ns = misc[0];
    const bool direct = ns > g.scap;
    if (!direct) {
        // one thread per (sampled pair, row)
        const uint32_t seav_base = (uint32_t)c.ldca_bits;
        for (uint32_t w = tid; w < ns * c.sr; w += BLOCK) {
            const uint32_t e = w / c.sr, r = w - e * c.sr;
            const uint32_t bit = seav_base + seav_byte_l(samp[2 * e], r, rl, c) * 8u + samp[2 * e + 1];
            atomicAdd(&hs[bit >> g.S], 1u);
        }
        __syncthreads();
    }
    uint32_t *co = cnt + (uint64_t)tile * nb;
    for (uint32_t b = tid; b < nb; b += BLOCK) co[b] = hl[b] + (direct ? 0u : hs[b]);
}

// Bit addresses of a tile's pairs placed straight into their bucket's segment of the stage: the
// cursors start at the segment bases, so the returning LDS atomic gives the final position.  All
// of a lane's LDCA bit addresses are computed first and all their atomics issued together, so the
// LDS round trips overlap; sampled pairs (about one in 2^tau) follow.
template <int LR, int PPT, int BLOCK, bool FULL>
__device__ __forceinline__ void place_hash_pairs(const Consts &c, const RowLds &rl, const BinGeometry &g, const SlotPtrs &S,
                                                 const u32x2 (&pr)[PPT], uint64_t p0, uint64_t n, uint32_t *cur,
                                                 uint32_t *stage, uint32_t *samp, uint32_t *nsamp) {
    const uint32_t tid = threadIdx.x;
    // pairs in chunks of CH: a chunk's LR * CH atomics are in flight together
    constexpr int CH = PPT < 4 ? PPT : 4;
#pragma unroll
    for (int j0 = 0; j0 < PPT; j0 += CH) {
        uint32_t bits[CH * LR], pos[CH * LR];
        uint32_t valid = 0;
#pragma unroll
        for (int jj = 0; jj < CH; ++jj) {
            const int j = j0 + jj;
            const bool v = FULL || p0 + (uint64_t)j * BLOCK + tid < n;
            valid |= (uint32_t)v << jj;
            const uint32_t hip = pr[j].x, oip = pr[j].y;
            const uint32_t q = ldc_bit(oip, c);
#pragma unroll
            for (int r = 0; r < LR; ++r) bits[jj * LR + r] = ldca_bit((uint32_t)r, ldc_col(hip, (uint32_t)r, c), q, c);
            if (v && sampled(oip, c)) {   // staged; placed by the whole workgroup later
                const uint32_t e = atomicAdd(nsamp, 1u);
                const uint32_t b = se_bit(oip, c);
                if (e < g.scap) {
                    samp[2 * e] = hip;
                    samp[2 * e + 1] = b;
                } else {
                    // only a tile whose SEAV items were left out of the counts gets here
                    uint32_t *seav_w = reinterpret_cast<uint32_t *>(S.seav);
                    for (uint32_t r = 0; r < c.sr; ++r) {
                        const uint32_t bit = seav_byte_l(hip, r, rl, c) * 8u + b;
                        global_or(seav_w + (bit >> 5), 1u << (bit & 31u));
                    }
                }
            }
        }
#pragma unroll
        for (int k = 0; k < CH * LR; ++k)
            pos[k] = (FULL || ((valid >> (k / LR)) & 1u)) ? atomicAdd(&cur[bits[k] >> g.S], 1u) : 0u;
#pragma unroll
        for (int k = 0; k < CH * LR; ++k)
            if (FULL || ((valid >> (k / LR)) & 1u)) stage[pos[k]] = bits[k];
    }
}

// Bucket-major binning (after k_count and the offset scans): a workgroup re-reads a tile, builds
// its padded segment bases from the tile's exact counts (cnt[tile]), places every item directly
// at its final position in an LDS stage, pads each segment to whole 64-bit words with copies of
// its last item, and writes segment b to global item offset off[tile][b].  A tile whose SEAV
// items were left out of the counts (more sampled pairs than the stage reserves) records them with
// global atomics instead, exactly as k_count decided.
template <int LR, int PPT, int BLOCK>
__global__ __launch_bounds__(BLOCK) void k_place(Consts c, BinGeometry g, BatchList bl, SlotTable st, ChunkTable ct,
                                                 uint64_t *__restrict__ items, const uint32_t *__restrict__ cnt,
                                                 const uint32_t *__restrict__ off, const uint32_t *__restrict__ cstart) {
    extern __shared__ uint32_t lds[];
    __shared__ RowLds rl;   // read after the first barrier
    rows_to_lds(rl, c);
    const uint32_t nb = g.nb;
    uint32_t *cur = lds;                 // [nb + 1] padded counts, then cursors, then global offsets
    uint32_t *lb = cur + (nb + 1);       // [nb + 1] segment bases in the stage; lb[nb] = padded total
    uint32_t *stage = lds + ((2 * (nb + 1) + 3) & ~3u);   // [cap]
    uint32_t *misc = stage + g.cap;      // [0..16] scan scratch, [17] sampled pairs
    uint32_t *samp = misc + 18;          // [2 * scap] sampled (hip, H2 bit)
    const uint32_t tid = threadIdx.x;
    const uint32_t tile = xcd_contiguous(blockIdx.x, gridDim.x);   // neighbouring tiles on one XCD
    const BatchDesc B = bl.b[find_batch(bl, tile)];   // descriptors in device memory
    const SlotPtrs S = st.s[B.slot];
    const uint64_t p0 = (uint64_t)(tile - B.first_tile) * (uint64_t)(PPT * BLOCK);

    // counts and global offsets of this tile (two per thread held in registers), and the pairs:
    // every load is issued before the first wait
    // this tile's offset of bucket b = its offset inside its chunk + the chunk's start
    const uint32_t chunk = ct.cbase[B.slot] + (tile - ct.lo[B.slot]) / kChunk;
    const uint32_t *ctr = cnt + (uint64_t)tile * nb;
    const uint32_t *ot = off + (uint64_t)tile * nb;
    const uint32_t *cs0 = cstart + (uint64_t)chunk * nb;
    // (the two parts of an offset are added where they are used, so no wait comes before the pairs)
    uint32_t c_pre[2] = {0u, 0u}, o_pre[2] = {0u, 0u}, s_pre[2] = {0u, 0u};
    if (tid < nb) {
        c_pre[0] = ctr[tid];
        o_pre[0] = ot[tid];
        s_pre[0] = cs0[tid];
    }
    if (tid + BLOCK < nb) {
        c_pre[1] = ctr[tid + BLOCK];
        o_pre[1] = ot[tid + BLOCK];
        s_pre[1] = cs0[tid + BLOCK];
    }
    const u32x2 *pairs = reinterpret_cast<const u32x2 *>(B.pairs);
    const uint64_t last = B.n - 1;
    u32x2 pr[PPT];
#pragma unroll
    for (int j = 0; j < PPT; ++j) {
        const uint64_t idx = p0 + (uint64_t)j * BLOCK + tid;
        pr[j] = load_pair(pairs, idx < B.n ? idx : last, B.swap);
    }
    for (uint32_t b = tid, m = 0; b < nb; b += BLOCK, ++m) {
        const uint32_t v = m == 0 ? c_pre[0] : m == 1 ? c_pre[1] : ctr[b];
        cur[b] = (v + 2) / 3 * 3;
        lb[b] = 0;
    }
    if (tid == 0) {
        cur[nb] = lb[nb] = 0;
        misc[17] = 0;
    }
    __syncthreads();
    // exclusive scan of the padded counts (lb is all zero: bucket_offsets adds cur[b] + lb[b])
    bucket_offsets<BLOCK>(cur, lb, nb, misc);
    // bucket_offsets leaves cur[b] = base, lb[b] = base + padded count (= the next base)
    for (uint32_t b = tid; b <= nb; b += BLOCK) {
        const uint32_t base = cur[b];
        lb[b] = base;
    }
    __syncthreads();
    const bool seav_direct = lb[nb] == lb[g.nb_ldca];   // no SEAV items were counted for this tile
    if (p0 + (uint64_t)(PPT * BLOCK) <= B.n)
        place_hash_pairs<LR, PPT, BLOCK, true>(c, rl, g, S, pr, p0, B.n, cur, stage, samp, misc + 17);
    else
        place_hash_pairs<LR, PPT, BLOCK, false>(c, rl, g, S, pr, p0, B.n, cur, stage, samp, misc + 17);
    __syncthreads();
    // the staged sampled pairs: one thread per (pair, row)
    {
        const uint32_t ns = misc[17] < g.scap ? misc[17] : g.scap;
        const uint32_t seav_base = (uint32_t)c.ldca_bits;
        uint32_t *seav_w = reinterpret_cast<uint32_t *>(S.seav);
        for (uint32_t w = tid; w < ns * c.sr; w += BLOCK) {
            const uint32_t e = w / c.sr, r = w - e * c.sr;
            const uint32_t byte = seav_byte_l(samp[2 * e], r, rl, c), b = samp[2 * e + 1];
            if (seav_direct) {
                const uint32_t bit = byte * 8u + b;
                global_or(seav_w + (bit >> 5), 1u << (bit & 31u));
            } else {
                const uint32_t bit = seav_base + byte * 8u + b;
                stage[atomicAdd(&cur[bit >> g.S], 1u)] = bit;
            }
        }
    }
    __syncthreads();
    // pad every segment to whole words with its last item; cur[b] becomes the distance in words
    // from the segment's place in the stage to its place in the item buffer
    for (uint32_t b = tid, m = 0; b < nb; b += BLOCK, ++m) {
        const uint32_t e = cur[b], s0 = lb[b], pe = lb[b + 1];
        if (e > s0)
            for (uint32_t p = e; p < pe; ++p) stage[p] = stage[e - 1];
        cur[b] = (m == 0 ? o_pre[0] + s_pre[0] : m == 1 ? o_pre[1] + s_pre[1] : ot[b] + cs0[b]) / 3 - s0 / 3;
    }
    __syncthreads();
    // one thread per stage word: the stage holds full bit addresses, so a word's first item names
    // its bucket; three 21-bit offsets per 64-bit word
    const uint32_t smask = (1u << g.S) - 1u;
    const uint32_t nwords = lb[nb] / 3;
    for (uint32_t w = tid; w < nwords; w += BLOCK) {
        const uint32_t s0 = stage[3 * w], s1 = stage[3 * w + 1], s2 = stage[3 * w + 2];
        items[w + cur[s0 >> g.S]] =
            (uint64_t)(s0 & smask) | ((uint64_t)(s1 & smask) << 21) | ((uint64_t)(s2 & smask) << 42);
    }
}

template <int LR, int PPT, int BLOCK>
static void launch_bin_t(int kind, const Consts &c, const BinGeometry &g, const BatchTable &bt, const BatchList &bl,
                         const SlotTable &st, const ClearList &clr, const ChunkTable &ct, const uint32_t *cstart,
                         uint32_t n_tiles, uint32_t *items, uint32_t *meta, const uint32_t *off, hipStream_t s) {
    if (kind == 0)
        hipLaunchKernelGGL((k_bin<LR, PPT, BLOCK>), dim3(n_tiles), dim3(BLOCK), g.lds_bytes, s, c, g, bt, st, items, meta);
    else if (kind == 1)
        hipLaunchKernelGGL((k_place<LR, PPT, BLOCK>), dim3(n_tiles), dim3(BLOCK), g.lds_bytes, s, c, g, bl, st, ct,
                           reinterpret_cast<uint64_t *>(items), meta, off, cstart);
    else
        hipLaunchKernelGGL((k_count<LR, PPT, BLOCK>), dim3(n_tiles), dim3(BLOCK), (2 * g.nb + 1 + 2 * g.scap) * 4u, s, c,
                           g, bl, clr, meta);
}

template <int LR>
static hipError_t launch_bin_lr(int kind, const Consts &c, const BinGeometry &g, const BatchTable &bt,
                                const BatchList &bl, const SlotTable &st, const ClearList &clr, const ChunkTable &ct,
                                const uint32_t *cstart, uint32_t n_tiles, uint32_t *items, uint32_t *meta,
                                const uint32_t *off, hipStream_t s) {
    const uint32_t ppt = g.tile_pairs / g.block;
#define SPD_BIN_CASE(B, P) \
    else if (g.block == B && ppt == P)                                                                             \
        launch_bin_t<LR, P, B>(kind, c, g, bt, bl, st, clr, ct, cstart, n_tiles, items, meta, off, s);
    if (false) {
    }
    SPD_BIN_CASE(1024, 16) SPD_BIN_CASE(1024, 8) SPD_BIN_CASE(1024, 4) SPD_BIN_CASE(512, 16) SPD_BIN_CASE(512, 8)
    SPD_BIN_CASE(512, 4) SPD_BIN_CASE(256, 16) SPD_BIN_CASE(256, 8)
#undef SPD_BIN_CASE
    else return hipErrorInvalidConfiguration;
    return hipGetLastError();
}

// kind: 0 = k_bin (tile regions; batches by value, at most kMaxGroup), 1 = k_place (bucket-major),
// 2 = k_count (both: batches in device memory, any number)
static hipError_t launch_bin_kind(int kind, const Consts &c, const BinGeometry &g, const BatchDesc *batches,
                                  uint32_t n_batches, uint32_t n_tiles, uint32_t *items, uint32_t *meta,
                                  const uint32_t *off, const SlotPtrs *slots, const ClearList *clear,
                                  const ChunkTable *chunks, const uint32_t *cstart, hipStream_t s) {
    ClearList clr{};
    if (clear) clr = *clear;
    ChunkTable ct{};
    if (chunks) ct = *chunks;
    BatchTable bt{};
    BatchList bl{};
    SlotTable st{};
    if (n_batches == 0) return hipErrorInvalidValue;
    if (kind == 0) {
        if (n_batches > (uint32_t)kMaxGroup) return hipErrorInvalidValue;
        for (uint32_t i = 0; i < n_batches; ++i) bt.b[i] = batches[i];
        bt.n = n_batches;
    } else {
        bl.b = batches;
        bl.n = n_batches;
    }
    if (slots)
        for (int i = 0; i < kMaxGroup; ++i) st.s[i] = slots[i];
    switch (c.lr) {
    case 1: return launch_bin_lr<1>(kind, c, g, bt, bl, st, clr, ct, cstart, n_tiles, items, meta, off, s);
    case 2: return launch_bin_lr<2>(kind, c, g, bt, bl, st, clr, ct, cstart, n_tiles, items, meta, off, s);
    case 3: return launch_bin_lr<3>(kind, c, g, bt, bl, st, clr, ct, cstart, n_tiles, items, meta, off, s);
    case 4: return launch_bin_lr<4>(kind, c, g, bt, bl, st, clr, ct, cstart, n_tiles, items, meta, off, s);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_bin(const Consts &c, const BinGeometry &g, const BatchDesc *batches, uint32_t n_batches,
                      uint32_t n_tiles, uint32_t *items, uint32_t *meta, const SlotPtrs *slots, hipStream_t s) {
    return launch_bin_kind(0, c, g, batches, n_batches, n_tiles, items, meta, nullptr, slots, nullptr, nullptr, nullptr, s);
}

hipError_t launch_place(const Consts &c, const BinGeometry &g, const BatchDesc *batches_dev, uint32_t n_batches,
                        uint32_t n_tiles, uint32_t *items, const uint32_t *cnt, const uint32_t *loc,
                        const uint32_t *cstart, const ChunkTable &ct, const SlotPtrs *slots, hipStream_t s) {
    return launch_bin_kind(1, c, g, batches_dev, n_batches, n_tiles, items, const_cast<uint32_t *>(cnt), loc, slots,
                           nullptr, &ct, cstart, s);
}

hipError_t launch_count(const Consts &c, const BinGeometry &g, const BatchDesc *batches_dev, uint32_t n_batches,
                        uint32_t n_tiles, uint32_t *cnt, const ClearList &clear, hipStream_t s) {
    return launch_bin_kind(2, c, g, batches_dev, n_batches, n_tiles, nullptr, cnt, nullptr, nullptr, &clear, nullptr,
                           nullptr, s);
}

// ---- region layout (one pass over the pairs)

// Inclusive prefix sum over the wavefront, and over rows of 16 lanes, in registers (DPP: no LDS round
// trip per step).
template <int CTRL, int ROWS>
__device__ __forceinline__ uint32_t dpp_add(uint32_t v) {
    return v + (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROWS, 0xF, false);
}
__device__ __forceinline__ uint32_t row_scan(uint32_t v) {
    v = dpp_add<0x111, 0xF>(v);   // row_shr 1, 2, 4, 8
    v = dpp_add<0x112, 0xF>(v);
    v = dpp_add<0x114, 0xF>(v);
    return dpp_add<0x118, 0xF>(v);
}
__device__ __forceinline__ uint32_t wave_scan(uint32_t v) {
    v = row_scan(v);
    v = dpp_add<0x142, 0xA>(v);   // lane 15 of rows 0 and 2 to rows 1 and 3
    return dpp_add<0x143, 0xC>(v);   // lane 31 to rows 2 and 3
}

// Pair tid + j * BLOCK of a tile from pair p0 of batch B, as stored; lanes past the batch's end read its
// last pair (they are masked later), so that all loads are in flight together.
template <int PPT, int BLOCK>
__device__ __forceinline__ void load_tile(const BatchDesc &B, uint64_t p0, u32x2 (&pr)[PPT]) {
    const u32x2 *pairs = reinterpret_cast<const u32x2 *>(B.pairs) + p0;
    if (p0 + (uint64_t)(PPT * BLOCK) <= B.n) {
#pragma unroll
        for (int j = 0; j < PPT; ++j) pr[j] = load_pair(pairs + j * BLOCK, threadIdx.x, 0u);
    } else {
        const uint32_t last = (uint32_t)(B.n - p0 - 1);
#pragma unroll
        for (int j = 0; j < PPT; ++j) {
            const uint32_t i = (uint32_t)(j * BLOCK) + threadIdx.x;
            pr[j] = load_pair(pairs, i < last ? i : last, 0u);
        }
    }
}

// Bit addresses of a tile's pairs: LDCA items are counted per bucket in cl and the returned rank kept
// per item; sampled pairs are staged in samp while it has room and counted in *n_samp.  H1 is tested on
// its low 24 bits first, which a 24-bit product gives.  A lane keeps its last sampled pair and stages it
// at the end, or when it meets another, so that the wavefront does not wait for an LDS counter at every
// pair that some lane samples.
template <int LR, int PPT, int BLOCK, bool FULL>
__device__ __forceinline__ void region_hash(const Consts &c, const BinGeometry &g, const u32x2 (&pr)[PPT], uint32_t left,
                                            uint32_t *cl, uint32_t *samp, uint32_t *n_samp, uint32_t (&bits)[PPT * LR],
                                            uint32_t (&rk)[(PPT * LR + 1) / 2]) {
    const uint32_t tid = threadIdx.x;
    const uint32_t low = c.tau_mask & 0xFFFFFFu;
    uint32_t s_hip = 0, s_oip = 0;
    bool has = false;
    auto stage_sample = [&]() {
        const uint32_t e = atomicAdd(n_samp, 1u);
        if (e < g.scap) {
            samp[2 * e] = s_hip;
            samp[2 * e + 1] = se_bit(s_oip, c);
        }
    };
#pragma unroll
    for (int j = 0; j < PPT; ++j) {
        const bool valid = FULL || (uint32_t)(j * BLOCK) + tid < left;
        const uint32_t hip = pr[j].x, oip = pr[j].y;
        const uint32_t q = ldc_bit(oip, c);
#pragma unroll
        for (int r = 0; r < LR; ++r) {
            const int k = j * LR + r;
            const uint32_t bit = ldca_bit((uint32_t)r, ldc_col(hip, (uint32_t)r, c), q, c);
            const uint32_t rank = valid ? atomicAdd(&cl[bit >> g.S], 1u) : 0xFFFFu;
            bits[k] = bit;
            if (k & 1)
                rk[k / 2] |= rank << 16;
            else
                rk[k / 2] = rank;
        }
        // the low 24 bits of H1 (its high product enters modulo 2^24), the others when they count
        const uint32_t h1 = (uint32_t)(((uint64_t)(uint32_t)c.mul[0] * oip + c.add[0]) >> 32) +
                            __umul24((uint32_t)(c.mul[0] >> 32), oip);
        bool hit = valid && (h1 & low) == 0u;
        if (c.tau_mask > 0xFFFFFFu) hit = hit && sampled(oip, c);
        if (__ballot(hit && has)) {
            if (hit && has) stage_sample();
        }
        s_hip = hit ? hip : s_hip;
        s_oip = hit ? oip : s_oip;
        has = has || hit;
    }
    if (has) stage_sample();
}

// A tile's items binned in LDS (ranks per bucket, then segment bases), with each bucket's segment
// padded to whole 64-bit words (copies of its last item).  Each non-empty segment takes room in its
// (chunk, bucket) region with one atomic; the atomics are issued before the items are placed in the
// stage, so their round trip overlaps that work.  The stage holds full bit addresses, so a stage word's
// first item names its bucket at write-out, and the last two places of each segment are first filled
// with an address of another bucket: those still holding it after placement are the padding.
//
// At most 80 scalar registers: with more, a SIMD holds fewer than eight wavefronts and the compute
// unit one workgroup of 1024 instead of two (64 Mi pairs: 320 instead of 229 us).
template <int LR, int PPT, int BLOCK>
__global__ __launch_bounds__(BLOCK) __attribute__((amdgpu_num_sgpr(80))) void k_region(Consts c, BinGeometry g, BatchList bl,
                                                                                       ChunkTable ct, RegionArgs ra) {
    extern __shared__ uint32_t lds[];
    __shared__ RowLds rl;   // read after the first barrier
    rows_to_lds(rl, c);
    constexpr uint32_t NW = BLOCK / 64;
    const uint32_t nb = g.nb;
    uint32_t *cl = lds;                  // [nb + 1] LDCA counts, then bases
    uint32_t *cs = cl + (nb + 1);        // [nb + 1] SEAV counts, then SEAV cursors, then distances
    uint32_t *stage = lds + ((2 * (nb + 1) + 3) & ~3u);   // [cap] full bit addresses, bucket-major
    uint32_t *samp = stage + g.cap;      // [2 * scap] sampled (hip, H2 bit)
    uint32_t *misc = samp + 2 * g.scap;  // [0] sampled count, [1] a segment is past its region, [2..17] scan
    const uint32_t tid = threadIdx.x, lane = tid & 63u;
    const uint32_t wid = __builtin_amdgcn_readfirstlane(tid >> 6);
    // each thread owns `per` consecutive buckets
    const uint32_t per = (nb + BLOCK - 1) / BLOCK;
    const uint32_t b_beg = tid * per < nb ? tid * per : nb, b_end = b_beg + per < nb ? b_beg + per : nb;

    const uint32_t tile = xcd_contiguous(blockIdx.x, gridDim.x);   // neighbouring tiles on one XCD
    const BatchDesc B = batch_of(bl, tile);
    const uint64_t p0 = (uint64_t)(tile - B.first_tile) * (uint64_t)(PPT * BLOCK);
    u32x2 pr[PPT];
    load_tile<PPT, BLOCK>(B, p0, pr);
    const uint32_t left = B.n - p0 < (uint64_t)(PPT * BLOCK) ? (uint32_t)(B.n - p0) : (uint32_t)(PPT * BLOCK);
    const bool full = left == (uint32_t)(PPT * BLOCK);
    const uint32_t slot = B.slot, t_lo = ct.lo[slot], cc = (tile - t_lo) / ct.tiles;
    const uint32_t seav_base = (uint32_t)c.ldca_bits;   // SEAV bits follow the LDCA bits
    const uint32_t smask = (1u << g.S) - 1u;
    for (uint32_t i = tid; i < 2 * (nb + 1); i += BLOCK) cl[i] = 0;
    if (tid < 2) misc[tid] = 0;
    __syncthreads();
    if (B.swap) {   // destination-keyed
#pragma unroll
        for (int j = 0; j < PPT; ++j) pr[j] = u32x2{pr[j].y, pr[j].x};
    }
    uint32_t bits[PPT * LR], rk[(PPT * LR + 1) / 2];
    if (full)
        region_hash<LR, PPT, BLOCK, true>(c, g, pr, left, cl, samp, misc, bits, rk);
    else
        region_hash<LR, PPT, BLOCK, false>(c, g, pr, left, cl, samp, misc, bits, rk);
    __syncthreads();
    // a tile with more sampled pairs than it can stage stages none: it is listed, and its pairs are
    // read again once the apply phase has written the SEAV buckets
    uint32_t ns = misc[0];
    if (ns > g.scap) {
        if (tid == 0) {
            ListedTile &t = ra.tile[t_lo + atomicAdd(&ra.list->listed[slot], 1u)];   // (one entry per tile of the slot)
            t.pairs = B.pairs + 2 * p0;
            t.n = left;
            t.swap = B.swap;
        }
        ns = 0;
    }
    for (uint32_t w = tid; w < ns * c.sr; w += BLOCK) {
        const uint32_t e = w / c.sr, r = w - e * c.sr;
        const uint32_t bit = seav_base + seav_byte_l(samp[2 * e], r, rl, c) * 8u + samp[2 * e + 1];
        atomicAdd(&cs[bit >> g.S], 1u);
    }
    __syncthreads();
    // padded counts (whole words) and their prefix sum; then, per bucket, its base, room in its
    // region (the offsets of a thread's first two buckets stay in flight) and the padding marks
    // (two named registers: an array indexed by the loop counter would live in scratch memory)
    uint32_t local = 0;
    for (uint32_t b = b_beg; b < b_end; ++b) local += (cl[b] + cs[b] + 2) / 3 * 3;
    const uint32_t incl = wave_scan(local);
    if (lane == 63u) misc[2 + wid] = incl;
    __syncthreads();
    const uint32_t wsum = lane < NW ? misc[2 + lane] : 0u, wincl = row_scan(wsum);
    uint32_t run = __builtin_amdgcn_readlane(wincl, wid) - __builtin_amdgcn_readlane(wsum, wid) + incl - local;
    const uint32_t nwords = __builtin_amdgcn_readlane(wincl, NW - 1) / 3;
    uint32_t *rcur = ra.cur + (uint64_t)(ct.cbase[slot] + cc) * nb;
    uint32_t o_pre0 = 0u, o_pre1 = 0u, n_own = 0u;
    for (uint32_t b = b_beg; b < b_end; ++b) {
        n_own = (cl[b] + cs[b] + 2) / 3;
        cl[b] = cs[b] = run;
        run += 3 * n_own;
    }
    if (tid == 0) cl[nb] = 3 * nwords;
    // (from here on a thread's buckets lie BLOCK apart, which with one bucket each changes nothing: the
    // lanes' atomics meet in few lines.  2304 buckets, 8 Mi pairs: 77.7 us -> 60.2.)
    if (per > 1) __syncthreads();
    for (uint32_t b = tid, m = 0; b < nb; b += BLOCK, ++m) {
        const uint32_t s0 = cl[b], n = per > 1 ? (cl[b + 1] - s0) / 3 : n_own;
        if (n) {
            if (m == 0) o_pre0 = atomicAdd(rcur + b, n);
            else if (m == 1) o_pre1 = atomicAdd(rcur + b, n);
            stage[s0 + 3 * n - 2] = stage[s0 + 3 * n - 1] = (b ^ 1u) << g.S;
        }
    }
    __syncthreads();
    if (full) {   // every lane's items are valid
#pragma unroll
        for (int k = 0; k < PPT * LR; ++k)
            stage[cl[bits[k] >> g.S] + ((rk[k / 2] >> (16 * (k & 1))) & 0xFFFFu)] = bits[k];
    } else {
#pragma unroll
        for (int k = 0; k < PPT * LR; ++k) {
            const uint32_t rank = (rk[k / 2] >> (16 * (k & 1))) & 0xFFFFu;
            if (rank != 0xFFFFu) stage[cl[bits[k] >> g.S] + rank] = bits[k];
        }
    }
    for (uint32_t w = tid; w < ns * c.sr; w += BLOCK) {
        const uint32_t e = w / c.sr, r = w - e * c.sr;
        const uint32_t bit = seav_base + seav_byte_l(samp[2 * e], r, rl, c) * 8u + samp[2 * e + 1];
        stage[atomicAdd(&cs[bit >> g.S], 1u)] = bit;
    }
    __syncthreads();
    // Pad every segment with its last item (the room of a thread's buckets past its first two is
    // taken here).  cs[b] becomes the distance from a stage word of bucket b to its place among the
    // chunk's regions; a segment that does not fit its region is listed under its bucket, its
    // remaining words go to the same places of the tile's part of the spill array.
    for (uint32_t b = tid, m = 0; b < nb; b += BLOCK, ++m) {
        const uint32_t s0 = cl[b], pe = cl[b + 1];
        if (pe > s0) {
            if ((stage[pe - 2] >> g.S) != b) stage[pe - 2] = stage[pe - 3];
            if ((stage[pe - 1] >> g.S) != b) stage[pe - 1] = stage[pe - 2];
            const uint32_t w0 = s0 / 3, n = (pe - s0) / 3;
            const uint32_t o = m == 0 ? o_pre0 : m == 1 ? o_pre1 : atomicAdd(rcur + b, n);
            uint32_t capw;
            const uint32_t in = region_in(ra, g.nb_ldca, slot, cc, b, &capw);
            cs[b] = in + o - w0;
            if (o + n > capw) {
                const uint32_t fit = o < capw ? capw - o : 0u;
                const uint32_t nt = ct.hi[slot] - t_lo;
                const uint32_t k = atomicAdd(ra.seg_n + slot * nb + b, 1u);   // below nt
                ra.seg[(uint64_t)t_lo * nb + (uint64_t)b * nt + k] = SpillSeg{tile * ra.tile_words + w0 + fit, n - fit};
                misc[1] = 1u;
            }
        }
    }
    __syncthreads();
    // one thread per stage word: three 21-bit offsets per 64-bit word
    uint64_t *dst = ra.items + chunk_at(ra, slot, cc);
    auto word = [&](uint32_t w, uint32_t &b) {
        const uint32_t s0 = stage[3 * w], s1 = stage[3 * w + 1], s2 = stage[3 * w + 2];
        b = s0 >> g.S;
        const uint32_t lo = (s0 & smask) | (s1 << 21), hi = ((s1 & smask) >> 11) | ((s2 & smask) << 10);
        return (uint64_t)lo | ((uint64_t)hi << 32);
    };
    if (!misc[1]) {
        for (uint32_t w = tid; w < nwords; w += BLOCK) {
            uint32_t b;
            const uint64_t v = word(w, b);
            dst[w + cs[b]] = v;
        }
    } else {
        // cl[b] becomes the first stage word past the region's room
        for (uint32_t b = tid; b < nb; b += BLOCK) {
            const uint32_t w0 = cl[b] / 3;
            uint32_t capw;
            const uint32_t o = cs[b] + w0 - region_in(ra, g.nb_ldca, slot, cc, b, &capw);
            cl[b] = w0 + (o < capw ? capw - o : 0u);
        }
        __syncthreads();
        uint64_t *spill = ra.spill_w + (uint64_t)tile * ra.tile_words;
        for (uint32_t w = tid; w < nwords; w += BLOCK) {
            uint32_t b;
            const uint64_t v = word(w, b);
            if (w < cl[b]) dst[w + cs[b]] = v;
            else spill[w] = v;
        }
    }
}

template <int LR>
static hipError_t launch_region_lr(const Consts &c, const BinGeometry &g, const BatchList &bl, const ChunkTable &ct,
                                   const RegionArgs &ra, uint32_t n_tiles, hipStream_t s, KTiming kt) {
    const uint32_t ppt = g.tile_pairs / g.block;
#define SPD_RG_CASE(B, P)                                                                                        \
    else if (g.block == B && ppt == P)                                                                         \
        hipExtLaunchKernelGGL((k_region<LR, P, B>), dim3(n_tiles), dim3(B), g.lds_bytes, s, kt.start, kt.stop, 0, c, g, \
                              bl, ct, ra);
    if (false) {
    }
    SPD_RG_CASE(1024, 16) SPD_RG_CASE(1024, 8) SPD_RG_CASE(1024, 7) SPD_RG_CASE(1024, 6) SPD_RG_CASE(1024, 5)
    SPD_RG_CASE(1024, 4) SPD_RG_CASE(1024, 2) SPD_RG_CASE(512, 16) SPD_RG_CASE(512, 8)
    SPD_RG_CASE(512, 4) SPD_RG_CASE(256, 16) SPD_RG_CASE(256, 8)
#undef SPD_RG_CASE
    else return hipErrorInvalidConfiguration;
    return hipGetLastError();
}

hipError_t launch_region(const Consts &c, const BinGeometry &g, const BatchList &bl, uint32_t n_tiles,
                         const ChunkTable &ct, const RegionArgs &ra, hipStream_t s, KTiming kt) {
    if (bl.n == 0 || n_tiles == 0 || (!bl.b && bl.n > kInlineBatches)) return hipErrorInvalidValue;
    switch (c.lr) {
    case 1: return launch_region_lr<1>(c, g, bl, ct, ra, n_tiles, s, kt);
    case 2: return launch_region_lr<2>(c, g, bl, ct, ra, n_tiles, s, kt);
    case 3: return launch_region_lr<3>(c, g, bl, ct, ra, n_tiles, s, kt);
    case 4: return launch_region_lr<4>(c, g, bl, ct, ra, n_tiles, s, kt);
    default: return hipErrorInvalidValue;
    }
}

// Zeroes every buffer of a clear list (16-byte stores over the whole grid).
__global__ __launch_bounds__(256) void k_clear(ClearList clr) {
    const uint64_t gt = (uint64_t)blockIdx.x * 256 + threadIdx.x, stride = (uint64_t)gridDim.x * 256;
    for (uint32_t k = 0; k < clr.n; ++k) {
        u32x4 *p4 = reinterpret_cast<u32x4 *>(clr.p[k]);
        for (uint64_t w = gt; w < clr.words[k] / 4; w += stride) p4[w] = u32x4{0u, 0u, 0u, 0u};
    }
}

hipError_t launch_clear(const ClearList &clear, hipStream_t s) {
    uint64_t words = 0;
    for (uint32_t k = 0; k < clear.n; ++k) {
        if (clear.words[k] % 4 || reinterpret_cast<uintptr_t>(clear.p[k]) % 16) return hipErrorInvalidValue;
        words += clear.words[k];
    }
    if (words == 0) return hipSuccess;
    // about eight 16-byte stores per lane: few waves to launch
    const uint64_t want = (words / 4 + 2047) / 2048;
    const uint32_t grid = (uint32_t)(want < 1024 ? (want ? want : 1) : 1024);
    hipLaunchKernelGGL(k_clear, dim3(grid), dim3(256), 0, s, clear);
    return hipGetLastError();
}

// Apply phase of the region layout: one workgroup per (slot, bucket) ORs the used part of the bucket's
// region in each of the slot's chunks into an LDS bitmap.
__device__ __forceinline__ void apply_word(uint32_t *bm, uint64_t v) {
#pragma unroll
    for (uint32_t f = 0; f < 3; ++f) {
        const uint32_t it = (uint32_t)(v >> (21 * f)) & 0x1FFFFFu;
        atomicOr(&bm[it >> 5], 1u << (it & 31u));
    }
}

// What does not fit a region is ordered by bucket too, and applied in LDS like the rest.  It was once
// appended word by word to one list (one counter: its atomics are serialized device-wide) and recorded
// with global atomics by a kernel of its own: 8 Mi pairs, half of them from four hosts, took 606 us of
// binning + 1930 us of that kernel, now 47 + 101 us of binning and apply; 5 Mi pairs with 60 planted
// hosts 84 + 36 us, now 28 us; and without such words the kernel's launch is saved (4 us).
//
// The listed segments of one (slot, bucket): each wavefront takes 64 at a time (one descriptor per
// lane) and reads the first 64 words of eight segments before it waits, since most segments are
// short; the rest of a long one follows in pieces of 64 * U words.
template <int BLOCK, int U>
__device__ __forceinline__ void apply_segments(const SpillSeg *__restrict__ seg, uint32_t n,
                                               const uint64_t *__restrict__ spill_w, uint32_t wid, uint32_t lane,
                                               uint32_t *bm) {
    constexpr uint32_t NW = BLOCK / 64, G = 8;
    // few segments: fewer of them per wavefront, so that every wavefront has some
    const uint32_t per = n >= 64 * NW ? 64u : (n + NW - 1) / NW;
    for (uint32_t d0 = wid * per; d0 < n; d0 += NW * per) {
        const uint32_t m = n - d0 < per ? n - d0 : per;
        const SpillSeg mine = seg[d0 + (lane < m ? lane : m - 1)];
        for (uint32_t j0 = 0; j0 < m; j0 += G) {
            uint64_t v[G];
            uint32_t len[G], st[G];
#pragma unroll
            for (uint32_t j = 0; j < G; ++j) {
                const uint32_t k = j0 + j < m ? j0 + j : m - 1;   // (a repeated segment is masked below)
                st[j] = __builtin_amdgcn_readlane(mine.start, k);
                len[j] = __builtin_amdgcn_readlane(mine.words, k);
                v[j] = spill_w[(uint64_t)st[j] + (lane < len[j] ? lane : len[j] - 1)];
            }
#pragma unroll
            for (uint32_t j = 0; j < G; ++j)
                if (j0 + j < m && lane < len[j]) apply_word(bm, v[j]);
            for (uint32_t j = 0; j < G && j0 + j < m; ++j) {
                const uint32_t s0 = __builtin_amdgcn_readlane(mine.start, j0 + j);
                const uint32_t l0 = __builtin_amdgcn_readlane(mine.words, j0 + j);
                for (uint32_t w0 = 64; w0 < l0; w0 += 64 * U) {
                    uint64_t x[U];
#pragma unroll
                    for (uint32_t k = 0; k < U; ++k) {
                        const uint32_t w = w0 + k * 64 + lane;
                        x[k] = spill_w[(uint64_t)s0 + (w < l0 ? w : l0 - 1)];
                    }
#pragma unroll
                    for (uint32_t k = 0; k < U; ++k)
                        if (w0 + k * 64 + lane < l0) apply_word(bm, x[k]);
                }
            }
        }
    }
}

// Listed tiles are read once, when the slot's SEAV buckets are in memory.  The workgroups of the SEAV's
// buckets (which come last in the grid) count them written, and with those of the LDCA buckets before them,
// where the SEAV has few, wait a little for the last; then they take tiles from a counter and record their
// sampled pairs with global atomics.  The wait is bounded, and a workgroup that gives up leaves: the one that
// counts the last bucket takes whatever tiles are left, so no workgroup depends on another that has not
// started.
// What lists a tile is one sampled peer with more than about 1.6 % of its pairs (8192 pairs, tau = 7),
// and then nearly every tile of a window is listed.  (Read again by every SEAV bucket, for the items
// of its own: 8 Mi pairs with a peer of 2 % into 72 MiB, 7.2 ms; by a launch of its own of 32
// workgroups: 0.92; so 0.20, of which 0.10 without such a peer too.)
constexpr uint32_t kListedGroups = 64;   // workgroups that share a slot's listed tiles, or its SEAV buckets if more
constexpr uint32_t kListedPolls = 32;    // of about two microseconds
constexpr uint32_t kListedWords = 128;   // LDS words that record_listed needs at least
__host__ __device__ __forceinline__ uint32_t apply_lds_words(uint32_t S) {   // and the piece counter after them
    return 1u << (S - 5) < kListedWords ? kListedWords : 1u << (S - 5);
}
// Whether this workgroup, which has stored bucket b, may take tiles.
__device__ __forceinline__ bool seav_written(uint32_t *written, uint32_t b, const BinGeometry &g, uint32_t *lds) {
    const uint32_t buckets = g.nb - g.nb_ldca;
    const bool mine = b >= g.nb_ldca;
    if (!mine && b + kListedGroups < g.nb) return false;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // this wavefront's stores are in the L2
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t n = 0;
        if (mine) {
            // one release for the workgroup: it writes the L2 back
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
            n = __hip_atomic_fetch_add(written, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1u;
        }
        for (uint32_t k = 0; n < buckets && k < kListedPolls; ++k) {
            __builtin_amdgcn_s_sleep(32);   // (2048 cycles; polls of one address follow each other)
            n = __hip_atomic_load(written, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        lds[0] = n;
    }
    __syncthreads();
    const bool all = lds[0] >= buckets;
    __syncthreads();
    return all;
}

// Takes listed tiles and records their sampled pairs in the SEAV, and in a second one if there is one: the
// sampled pairs are gathered in LDS, so that the lanes share their bits evenly and nothing waits for
// memory between them.  A heavy flow's pairs set the same bits over and over, and atomics on one address
// follow each other device-wide: a bit that the table in LDS still holds is not set again (8 Mi pairs, 30 %
// of them one flow: 2.2 ms; with the atomics alone, in a launch of their own, 55).
// The method constants are read from the kernel arguments (they are the first one) behind an opaque
// pointer, so that nothing of this is loaded on the path of a launch that lists no tile.
typedef __attribute__((address_space(4))) const Consts ArgConsts;
template <int BLOCK>
__device__ __forceinline__ void record_listed(const ListedTile *tiles, uint32_t n, uint32_t *taken, uint32_t *seav,
                                              uint32_t *seav2, uint32_t *lds, uint32_t lds_words) {
    constexpr uint32_t U = 8;   // pairs in flight per lane
    auto args = __builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(args));
    ArgConsts &c = *(ArgConsts *)args;
    // [0] tile, [1] sampled pairs gathered, then the table of bits, then the pairs (hip, H2 bit)
    const uint32_t tab_bits = 31u - __builtin_clz(lds_words) - 2u;   // a quarter of the words (at least 128)
    uint32_t *tab = lds + 2, *list = tab + (1u << tab_bits);
    const uint32_t cap = (lds_words - 2u - (1u << tab_bits)) / 2u;
    for (uint32_t i = threadIdx.x; i < (1u << tab_bits); i += BLOCK) tab[i] = ~0u;   // (no bit's address)
    auto record = [&](uint32_t hip, uint32_t b, uint32_t r) {
        const uint32_t rp = hip & c.rmask, lp = (uint32_t)((uint64_t)hip >> c.r);
        const uint32_t bit = (rp * c.sea_bytes + c.row_off[r] + row_index(lp, c.isb[r], c.ibn[r], c.L)) * 8u + b;
        uint32_t *t = tab + (bit * 0x9E3779B1u >> (32u - tab_bits));
        if (*t == bit) return;
        *t = bit;
        global_or(seav + (bit >> 5), 1u << (bit & 31u));
        if (seav2) global_or(seav2 + (bit >> 5), 1u << (bit & 31u));
    };
    for (;;) {
        if (threadIdx.x == 0) {
            lds[0] = __hip_atomic_fetch_add(taken, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            lds[1] = 0;
        }
        __syncthreads();
        const uint32_t t = __builtin_amdgcn_readfirstlane(lds[0]);
        if (t >= n) break;
        const ListedTile T = tiles[t];
        const u32x2 *pairs = reinterpret_cast<const u32x2 *>(T.pairs);
        for (uint32_t i0 = 0; i0 < T.n; i0 += U * BLOCK) {
            u32x2 pr[U];
#pragma unroll
            for (uint32_t k = 0; k < U; ++k) {
                const uint32_t i = i0 + k * BLOCK + threadIdx.x;
                pr[k] = load_pair(pairs, i < T.n ? i : T.n - 1, T.swap);
            }
#pragma unroll
            for (uint32_t k = 0; k < U; ++k) {
                const bool valid = i0 + k * BLOCK + threadIdx.x < T.n;
                if (!valid || (mas_hi(pr[k].y, c.mul[0], c.add[0]) & c.tau_mask)) continue;
                const uint32_t b = mas_hi(pr[k].y, c.mul[1], c.add[1]) >> 29;
                const uint32_t e = atomicAdd(&lds[1], 1u);
                if (e < cap) {
                    list[2 * e] = pr[k].x;
                    list[2 * e + 1] = b;
                } else {   // (buckets of fewer than 2^18 bits)
                    for (uint32_t r = 0; r < c.sr; ++r) record(pr[k].x, b, r);
                }
            }
            __syncthreads();
            const uint32_t m = (lds[1] < cap ? lds[1] : cap) * c.sr;
            for (uint32_t w = threadIdx.x; w < m; w += BLOCK) {
                const uint32_t e = w / c.sr;
                record(list[2 * e], list[2 * e + 1], w - e * c.sr);
            }
            __syncthreads();
            if (threadIdx.x == 0) lds[1] = 0;
            __syncthreads();
        }
    }
    __syncthreads();
}

// Bucket b of slot si: loaded into the LDS bitmap bm (zero for a fresh slot:
// nothing else writes the bucket's memory before it is stored), the filled part of the bucket's region in
// every chunk of the slot, then its listed segments, applied with LDS atomicOr, the counters read
// zeroed for the next launch, the bitmap stored back.  Ends with bm complete and visible to the whole
// workgroup.
// Bound by the LDS atomics of random words (about 9 items per ns and compute unit) for crowded buckets.
// The region's words come in pieces of 64 * U, which the wavefronts take from a counter as they get
// free.  (Dealt out in turn, 6 to 8 of a bucket's 37 us went by until the last wavefront had ended: 64 Mi
// pairs, 83 -> 73 us; 5 Mi, 27 -> 23.5 us.)
template <int BLOCK, int U>
__device__ __forceinline__ void apply_bucket(const BinGeometry &g, const ApplySlot &A, uint32_t si, uint32_t b,
                                             const ChunkTable &ct, const RegionArgs &ra, uint32_t *bm) {
    constexpr uint32_t PIECE = 64 * U;
    const uint32_t words = 1u << (g.S - 5);
    const uint32_t tid = threadIdx.x, lane = tid & 63u;
    const uint32_t wid = __builtin_amdgcn_readfirstlane(tid >> 6);
    uint32_t *dst = b < g.nb_ldca ? A.ldca + (uint64_t)b * words : A.seav_w + (uint64_t)(b - g.nb_ldca) * words;
    const uint32_t words4 = words / 4;
    u32x4 *bm4 = reinterpret_cast<u32x4 *>(bm), *dst4 = reinterpret_cast<u32x4 *>(dst);
    const uint32_t n_seg = ra.seg_n[si * g.nb + b];
    // the slot's chunks (at most kXcds + 1), one per lane: words filled, pieces, and pieces up to here
    const uint32_t c0 = ct.cbase[si], nch = ct.cbase[si + 1] - c0;
    uint32_t cap_c = 0;
    const uint32_t in_full = region_in(ra, g.nb_ldca, si, 0, b, &cap_c), cap_full = cap_c;
    const uint32_t in_last = region_in(ra, g.nb_ldca, si, nch - 1, b, &cap_c), cap_last = cap_c;
    uint32_t len = lane < nch ? ra.cur[(uint64_t)(c0 + lane) * g.nb + b] : 0u;
    uint32_t *next_piece = bm + words;   // (after the bitmap, which has to start on 16 bytes)
    if (tid == 0) *next_piece = 0;
    if (A.fresh) {
        for (uint32_t w = tid; w < words4; w += BLOCK) bm4[w] = u32x4{0u, 0u, 0u, 0u};
        for (uint32_t w = words4 * 4 + tid; w < words; w += BLOCK) bm[w] = 0;
    } else {
        // eight 16-byte loads of a lane in flight (word by word, each waiting for the one before, took 20
        // of a bucket's 24 us)
        for (uint32_t w = tid; w < words4; w += 8 * BLOCK) {
            u32x4 x[8];
#pragma unroll
            for (uint32_t k = 0; k < 8; ++k) x[k] = dst4[w + k * BLOCK < words4 ? w + k * BLOCK : w];
#pragma unroll
            for (uint32_t k = 0; k < 8; ++k)
                if (w + k * BLOCK < words4) bm4[w + k * BLOCK] = x[k];
        }
        for (uint32_t w = words4 * 4 + tid; w < words; w += BLOCK) bm[w] = dst[w];
    }
    if (lane < nch) {
        const uint32_t cap = lane == nch - 1 ? cap_last : cap_full;
        len = len < cap ? len : cap;
    }
    const uint32_t np = (len + PIECE - 1) / PIECE, upto = wave_scan(np);
    const uint32_t n_piece = __builtin_amdgcn_readlane(upto, 63);
    __syncthreads();
    auto take = [&]() -> uint32_t {
        uint32_t p = 0;
        if (lane == 0) p = atomicAdd(next_piece, 1u);
        return __builtin_amdgcn_readfirstlane(p);
    };
    auto fetch = [&](uint32_t p, uint64_t (&v)[U], uint32_t &left) {   // p < n_piece
        const uint32_t cc = (uint32_t)__popcll(__ballot(upto <= p));
        const uint32_t l = __builtin_amdgcn_readlane(len, cc);
        const uint32_t w0 = (p - (__builtin_amdgcn_readlane(upto, cc) - __builtin_amdgcn_readlane(np, cc))) * PIECE;
        const uint64_t *src = ra.items + chunk_at(ra, si, cc) + (cc == nch - 1 ? in_last : in_full) + w0;
        left = l - w0;
#pragma unroll
        for (uint32_t k = 0; k < U; ++k) {
            const uint32_t w = k * 64 + lane;
            v[k] = __builtin_nontemporal_load(src + (w < left ? w : left - 1));   // unconditional loads
        }
    };
    auto apply = [&](const uint64_t (&v)[U], uint32_t left) {
#pragma unroll
        for (uint32_t k = 0; k < U; ++k)
            if (k * 64 + lane < left) apply_word(bm, v[k]);
    };
    for (uint32_t p = take(); p < n_piece;) {
        uint64_t v[U];
        uint32_t left;
        fetch(p, v, left);
        p = take();
        apply(v, left);
    }
    if (n_seg) {
        const uint32_t lo = ct.lo[si], nt = ct.hi[si] - lo;
        apply_segments<BLOCK, 2 * U>(ra.seg + (uint64_t)lo * g.nb + (uint64_t)b * nt, n_seg, ra.spill_w, wid, lane, bm);
    }
    __syncthreads();
    // the counters of this (slot, bucket) start the next launch at zero, and so do its tile lists
    if (tid < nch) ra.cur[(uint64_t)(c0 + tid) * g.nb + b] = 0u;
    if (tid == 0) ra.seg_n[si * g.nb + b] = 0u;
    if (b == 0 && si == 0 && tid < kListWords) reinterpret_cast<uint32_t *>(ra.list_next)[tid] = 0u;
    for (uint32_t w = tid; w < words4; w += BLOCK) dst4[w] = bm4[w];
    for (uint32_t w = words4 * 4 + tid; w < words; w += BLOCK) dst[w] = bm[w];
}

// One workgroup per (slot, bucket).  (The first argument is read by record_listed.)  At most 80 scalar
// registers, as in k_region: small buckets leave room for two workgroups per compute unit.
template <int BLOCK, int U>
__global__ __launch_bounds__(BLOCK) __attribute__((amdgpu_num_sgpr(80))) void k_apply_rg(Consts, BinGeometry g, ApplyTable at, ChunkTable ct, RegionArgs ra) {
    extern __shared__ __align__(16) uint32_t bm[];
    const uint32_t si = blockIdx.x / g.nb, b = blockIdx.x % g.nb;
    apply_bucket<BLOCK, U>(g, at.s[si], si, b, ct, ra, bm);
    const uint32_t n = ra.list->listed[si];
    if (n && seav_written(&ra.list->written[si], b, g, bm))
        record_listed<BLOCK>(ra.tile + ct.lo[si], n, &ra.list->taken[si], at.s[si].seav_w, nullptr, bm, apply_lds_words(g.S));
}

// The same with the router OR merge fused in (Section 4.2): one workgroup per bucket applies the
// bucket of every slot of the launch in turn and keeps their OR in registers (a 2^S-bit bucket is
// 32 words per lane of 1024), then writes it to the global sketch's bucket.  The global's previous
// content is replaced.
template <int U>
__global__ __launch_bounds__(1024) void k_apply_rg_merge(Consts, BinGeometry g, ApplyTable at, uint32_t n_slots,
                                                         ChunkTable ct, RegionArgs ra, ApplySlot gs) {
    extern __shared__ __align__(16) uint32_t bm[];
    constexpr uint32_t BLOCK = 1024, PER = 32;   // words per lane of a 2^20-bit bucket
    const uint32_t words = 1u << (g.S - 5);
    const uint32_t tid = threadIdx.x, b = blockIdx.x;
    uint32_t acc[PER];
#pragma unroll
    for (uint32_t k = 0; k < PER; ++k) acc[k] = 0;
    for (uint32_t si = 0; si < n_slots; ++si) {
        apply_bucket<BLOCK, U>(g, at.s[si], si, b, ct, ra, bm);
#pragma unroll
        for (uint32_t k = 0; k < PER; ++k)
            if (k * BLOCK + tid < words) acc[k] |= bm[k * BLOCK + tid];
        __syncthreads();   // every lane has read bm before the next slot's bucket overwrites it
    }
    uint32_t *dst = b < g.nb_ldca ? gs.ldca + (uint64_t)b * words : gs.seav_w + (uint64_t)(b - g.nb_ldca) * words;
#pragma unroll
    for (uint32_t k = 0; k < PER; ++k)
        if (k * BLOCK + tid < words) dst[k * BLOCK + tid] = acc[k];
    uint32_t listed = 0;
    for (uint32_t si = 0; si < n_slots; ++si) listed |= ra.list->listed[si];
    if (!listed || !seav_written(&ra.list->written[0], b, g, bm)) return;
    for (uint32_t si = 0; si < n_slots; ++si) {
        const uint32_t n = ra.list->listed[si];
        if (n) record_listed<BLOCK>(ra.tile + ct.lo[si], n, &ra.list->taken[si], at.s[si].seav_w, gs.seav_w, bm, apply_lds_words(g.S));
    }
}

template <int U>
static void launch_apply_rg_u(const Consts &c, const BinGeometry &g, const ApplyTable &at, const ChunkTable &ct,
                              const RegionArgs &ra, dim3 grid, uint32_t lds, uint32_t block, hipStream_t s, KTiming kt) {
    if (block == 1024)
        hipExtLaunchKernelGGL((k_apply_rg<1024, U>), grid, dim3(1024), lds, s, kt.start, kt.stop, 0, c, g, at, ct, ra);
    else if (block == 512)
        hipExtLaunchKernelGGL((k_apply_rg<512, U>), grid, dim3(512), lds, s, kt.start, kt.stop, 0, c, g, at, ct, ra);
    else hipExtLaunchKernelGGL((k_apply_rg<256, U>), grid, dim3(256), lds, s, kt.start, kt.stop, 0, c, g, at, ct, ra);
}

hipError_t launch_apply_rg(const Consts &c, const BinGeometry &g, const ApplySlot *slots, uint32_t n_slots,
                           const ChunkTable &ct, const RegionArgs &ra, uint32_t block, uint32_t unroll, hipStream_t s,
                           KTiming kt) {
    ApplyTable at{};
    if (n_slots == 0 || n_slots > (uint32_t)kMaxGroup || ct.n != n_slots) return hipErrorInvalidValue;
    if (block != 1024 && block != 512 && block != 256) return hipErrorInvalidConfiguration;
    for (uint32_t i = 0; i < n_slots; ++i) {
        at.s[i] = slots[i];
        if (ct.cbase[i + 1] - ct.cbase[i] > 64u) return hipErrorInvalidValue;   // a lane per chunk
    }
    const uint32_t lds = apply_lds_words(g.S) * 4u + 16u;
    const dim3 grid(n_slots * g.nb);
    switch (unroll) {
    case 8: launch_apply_rg_u<2>(c, g, at, ct, ra, grid, lds, block, s, kt); break;
    case 16: launch_apply_rg_u<4>(c, g, at, ct, ra, grid, lds, block, s, kt); break;
    case 32: launch_apply_rg_u<8>(c, g, at, ct, ra, grid, lds, block, s, kt); break;
    default: return hipErrorInvalidConfiguration;
    }
    return hipGetLastError();
}

hipError_t launch_apply_rg_merge(const Consts &c, const BinGeometry &g, const ApplySlot *slots, uint32_t n_slots,
                                 const ChunkTable &ct, const RegionArgs &ra, const ApplySlot &global, uint32_t unroll,
                                 hipStream_t s, KTiming kt) {
    ApplyTable at{};
    if (n_slots == 0 || n_slots > (uint32_t)kMaxGroup || ct.n != n_slots || g.S > 20) return hipErrorInvalidValue;
    for (uint32_t i = 0; i < n_slots; ++i) {
        at.s[i] = slots[i];
        if (ct.cbase[i + 1] - ct.cbase[i] > 64u) return hipErrorInvalidValue;   // a lane per chunk
    }
    const uint32_t lds = apply_lds_words(g.S) * 4u + 16u;
    const dim3 grid(g.nb), block(1024);
    switch (unroll) {
    case 8: hipExtLaunchKernelGGL((k_apply_rg_merge<2>), grid, block, lds, s, kt.start, kt.stop, 0, c, g, at, n_slots, ct, ra, global); break;
    case 16: hipExtLaunchKernelGGL((k_apply_rg_merge<4>), grid, block, lds, s, kt.start, kt.stop, 0, c, g, at, n_slots, ct, ra, global); break;
    case 32: hipExtLaunchKernelGGL((k_apply_rg_merge<8>), grid, block, lds, s, kt.start, kt.stop, 0, c, g, at, n_slots, ct, ra, global); break;
    default: return hipErrorInvalidConfiguration;
    }
    return hipGetLastError();
}

// ---- offsets of the bucket-major layout
// Per slot, bucket b's items are the concatenation over the slot's tiles of each tile's segment
// (count rounded up to a multiple of 3: whole 64-bit words); slots follow each other per bucket:
// base[s * nb + b] = start of (slot s, bucket b).  Tiles are scanned in chunks of kChunk that
// never span two slots: k_colscan writes each (tile, bucket) offset inside its chunk and each
// chunk's total, k_chunkscan turns the chunk totals into chunk starts (base included), and
// k_place adds a tile's chunk start to its offsets.
__device__ __forceinline__ uint32_t slot_of_chunk(const ChunkTable &ct, uint32_t c) {
    uint32_t si = 0;
    while (si + 1 < ct.n && ct.cbase[si + 1] <= c) ++si;
    return si;
}

// grid (ceil(nb / 64), chunks), 256 threads: 64 buckets x 4 groups of 32 tiles
__global__ __launch_bounds__(256) void k_colscan(const uint32_t *__restrict__ cnt, uint32_t *__restrict__ loc,
                                                 uint32_t *__restrict__ csum, ChunkTable ct, uint32_t nb) {
    static_assert(kChunk == 128, "four groups of 32 tiles");
    __shared__ uint32_t ps[4][64];
    const uint32_t c = blockIdx.y;
    const uint32_t si = slot_of_chunk(ct, c);
    const uint32_t t0 = ct.lo[si] + (c - ct.cbase[si]) * kChunk;
    const uint32_t t1 = t0 + kChunk < ct.hi[si] ? t0 + kChunk : ct.hi[si];   // > t0
    const uint32_t col = threadIdx.x & 63u, rg = threadIdx.x >> 6;
    const uint32_t b = blockIdx.x * 64 + col;
    const bool okb = b < nb;
    const uint32_t bb = okb ? b : nb - 1;
    const uint32_t r0 = t0 + rg * 32;
    uint32_t v[32];
#pragma unroll
    for (uint32_t k = 0; k < 32; ++k) {   // unconditional (clamped) loads, all in flight together
        const uint32_t t = r0 + k < t1 ? r0 + k : t1 - 1;
        v[k] = cnt[(uint64_t)t * nb + bb];
    }
    uint32_t sum = 0;
#pragma unroll
    for (uint32_t k = 0; k < 32; ++k) {
        const uint32_t x = (r0 + k < t1) ? (v[k] + 2) / 3 * 3 : 0u;
        v[k] = sum;
        sum += x;
    }
    ps[rg][col] = sum;
    __syncthreads();
    uint32_t pre = 0;
    for (uint32_t r = 0; r < rg; ++r) pre += ps[r][col];
    if (okb) {
#pragma unroll
        for (uint32_t k = 0; k < 32; ++k)
            if (r0 + k < t1) loc[(uint64_t)(r0 + k) * nb + b] = pre + v[k];
        if (rg == 3) csum[(uint64_t)c * nb + b] = pre + sum;
    }
}

// One workgroup: chunk totals -> chunk starts (in place, base included); base[s * nb + b] and
// base[n * nb] = all items.
__global__ __launch_bounds__(1024) void k_chunkscan(uint32_t *__restrict__ csum, uint32_t *__restrict__ base,
                                                    ChunkTable ct, uint32_t nb) {
    __shared__ uint32_t wsum[17];
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wid = tid >> 6;
    const uint32_t n = ct.n * nb;
    // 1. per (slot, bucket): exclusive prefix over the slot's chunks; the total goes to base
    for (uint32_t e = tid; e < n; e += 1024) {
        const uint32_t s = e / nb, b = e - s * nb;
        uint32_t run = 0;
        for (uint32_t c0 = ct.cbase[s]; c0 < ct.cbase[s + 1]; c0 += 8) {
            uint32_t x[8];
#pragma unroll
            for (uint32_t k = 0; k < 8; ++k) x[k] = c0 + k < ct.cbase[s + 1] ? csum[(uint64_t)(c0 + k) * nb + b] : 0u;
#pragma unroll
            for (uint32_t k = 0; k < 8; ++k) {
                if (c0 + k < ct.cbase[s + 1]) csum[(uint64_t)(c0 + k) * nb + b] = run;
                run += x[k];
            }
        }
        base[e] = run;
    }
    __syncthreads();
    // 2. exclusive prefix of the (slot, bucket) totals
    uint32_t carry = 0;
    for (uint32_t i0 = 0; i0 < n; i0 += 1024) {
        const uint32_t i = i0 + tid;
        const uint32_t v = i < n ? base[i] : 0u;
        uint32_t incl = v;
        for (int o = 1; o < 64; o <<= 1) {
            uint32_t x = __shfl_up(incl, o, 64);
            if ((int)lane >= o) incl += x;
        }
        if (lane == 63u) wsum[wid] = incl;
        __syncthreads();
        if (tid == 0) {
            uint32_t run = 0;
            for (uint32_t w = 0; w < 16; ++w) {
                uint32_t x = wsum[w];
                wsum[w] = run;
                run += x;
            }
            wsum[16] = run;
        }
        __syncthreads();
        if (i < n) base[i] = carry + wsum[wid] + incl - v;
        carry += wsum[16];
        __syncthreads();
    }
    if (tid == 0) base[n] = carry;
    __syncthreads();
    // 3. chunk starts become absolute
    for (uint32_t e = tid; e < n; e += 1024) {
        const uint32_t s = e / nb, b = e - s * nb, add = base[e];
        for (uint32_t c = ct.cbase[s]; c < ct.cbase[s + 1]; ++c) csum[(uint64_t)c * nb + b] += add;
    }
}

hipError_t launch_offsets(const uint32_t *cnt, uint32_t *loc, uint32_t *csum, uint32_t *base, const ChunkTable &ct,
                          uint32_t nb, hipStream_t s) {
    if (ct.n == 0 || ct.n > (uint32_t)kMaxGroup || ct.cbase[ct.n] == 0 || ct.cbase[ct.n] > 65535u)
        return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_colscan, dim3((nb + 63) / 64, ct.cbase[ct.n]), dim3(256), 0, s, cnt, loc, csum, ct, nb);
    hipLaunchKernelGGL(k_chunkscan, dim3(1), dim3(1024), 0, s, csum, base, ct, nb);
    return hipGetLastError();
}

// Phase 2 of the bucket-major layout: one workgroup per (slot, bucket) streams the bucket's
// contiguous items (three per 64-bit word) into an LDS bitmap and writes the bucket back.
template <int BLOCK, int U>
__global__ __launch_bounds__(BLOCK) void k_apply_bm(BinGeometry g, ApplyTable at, const uint64_t *__restrict__ items,
                                                    const uint32_t *__restrict__ base) {
    // U: 8-byte loads in flight per lane
    extern __shared__ __align__(16) uint32_t bm[];
    const uint32_t words = 1u << (g.S - 5);
    const uint32_t tid = threadIdx.x;
    const uint32_t blk = blockIdx.x;
    const uint32_t si = blk / g.nb, b = blk % g.nb;
    const ApplySlot A = at.s[si];
    uint32_t *dst = b < g.nb_ldca ? A.ldca + (uint64_t)b * words : A.seav_w + (uint64_t)(b - g.nb_ldca) * words;
    if (A.fresh && b < g.nb_ldca) {
        for (uint32_t w = tid; w < words; w += BLOCK) bm[w] = 0;
    } else {
        for (uint32_t w = tid; w < words; w += BLOCK) bm[w] = dst[w];
    }
    __syncthreads();
    const uint32_t w0 = base[blk] / 3, w1 = base[blk + 1] / 3;
    for (uint32_t w = w0 + tid; w < w1; w += BLOCK * U) {
        uint64_t v[U];
#pragma unroll
        for (uint32_t u = 0; u < U; ++u) {
            const uint32_t ww = w + u * BLOCK < w1 ? w + u * BLOCK : w1 - 1;   // unconditional loads
            v[u] = __builtin_nontemporal_load(items + ww);
        }
#pragma unroll
        for (uint32_t u = 0; u < U; ++u) {
            if (w + u * BLOCK >= w1) continue;
#pragma unroll
            for (uint32_t f = 0; f < 3; ++f) {
                const uint32_t it = (uint32_t)(v[u] >> (21 * f)) & 0x1FFFFFu;
                atomicOr(&bm[it >> 5], 1u << (it & 31u));
            }
        }
    }
    __syncthreads();
    const uint32_t words4 = words / 4;
    if (words4) {
        for (uint32_t w = tid; w < words4; w += BLOCK)
            reinterpret_cast<u32x4 *>(dst)[w] = reinterpret_cast<const u32x4 *>(bm)[w];
    } else {
        for (uint32_t w = tid; w < words; w += BLOCK) dst[w] = bm[w];
    }
}

template <int U>
static void launch_apply_bm_u(const BinGeometry &g, const ApplyTable &at, dim3 grid, uint32_t lds, const uint64_t *it,
                              const uint32_t *base, uint32_t block, hipStream_t s) {
    if (block == 1024) hipLaunchKernelGGL((k_apply_bm<1024, U>), grid, dim3(1024), lds, s, g, at, it, base);
    else if (block == 512) hipLaunchKernelGGL((k_apply_bm<512, U>), grid, dim3(512), lds, s, g, at, it, base);
    else hipLaunchKernelGGL((k_apply_bm<256, U>), grid, dim3(256), lds, s, g, at, it, base);
}

hipError_t launch_apply_bm(const BinGeometry &g, const ApplySlot *slots, uint32_t n_slots, const uint32_t *items,
                           const uint32_t *base, uint32_t block, uint32_t unroll, hipStream_t s) {
    ApplyTable at{};
    if (n_slots == 0 || n_slots > (uint32_t)kMaxGroup) return hipErrorInvalidValue;
    if (block != 1024 && block != 512 && block != 256) return hipErrorInvalidConfiguration;
    for (uint32_t i = 0; i < n_slots; ++i) at.s[i] = slots[i];
    const uint32_t lds = (1u << (g.S - 5)) * 4u;
    const uint64_t *it = reinterpret_cast<const uint64_t *>(items);
    dim3 grid(n_slots * g.nb);
    switch (unroll) {
    case 8: launch_apply_bm_u<4>(g, at, grid, lds, it, base, block, s); break;
    case 16: launch_apply_bm_u<8>(g, at, grid, lds, it, base, block, s); break;
    case 32: launch_apply_bm_u<16>(g, at, grid, lds, it, base, block, s); break;
    default: return hipErrorInvalidConfiguration;
    }
    return hipGetLastError();
}

// meta[rows][cols] -> metaT[cols][rows]
__global__ __launch_bounds__(256) void k_transpose(const uint32_t *__restrict__ in, uint32_t *__restrict__ out,
                                                   uint32_t rows, uint32_t cols) {
    __shared__ uint32_t t[32][33];
    const uint32_t bx = blockIdx.y * 32, by = blockIdx.x * 32;   // bx: column block, by: row block
    const uint32_t tx = threadIdx.x & 31u, ty = threadIdx.x >> 5;   // 32 x 8
    for (uint32_t k = ty; k < 32; k += 8) {
        uint32_t r = by + k, col = bx + tx;
        if (r < rows && col < cols) t[k][tx] = in[(uint64_t)r * cols + col];
    }
    __syncthreads();
    for (uint32_t k = ty; k < 32; k += 8) {
        uint32_t col = bx + k, r = by + tx;
        if (r < rows && col < cols) out[(uint64_t)col * rows + r] = t[tx][k];
    }
}

hipError_t launch_transpose(const uint32_t *meta, uint32_t *metaT, uint32_t rows, uint32_t cols, hipStream_t s) {
    if (rows == 0 || cols == 0 || (cols + 31) / 32 > 65535u) return hipErrorInvalidValue;
    dim3 grid((rows + 31) / 32, (cols + 31) / 32);
    hipLaunchKernelGGL(k_transpose, grid, dim3(256), 0, s, meta, metaT, rows, cols);
    return hipGetLastError();
}

constexpr uint32_t kApplyChunk = 1024;

template <int BLOCK, int U>
__global__ __launch_bounds__(BLOCK) void k_apply(BinGeometry g, ApplyTable at, const uint32_t *__restrict__ items,
                                                 const uint32_t *__restrict__ metaT, uint32_t n_tiles) {
    // U: tiles per wavefront per step, i.e. U segment loads in flight per lane
    extern __shared__ uint32_t lds[];
    constexpr uint32_t NW = BLOCK / 64;
    const uint32_t words = 1u << (g.S - 5);
    uint32_t *bm = lds;
    uint32_t *mbeg = bm + words;
    uint32_t *mend = mbeg + kApplyChunk;
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wid = tid >> 6;
    const uint32_t si = blockIdx.x / g.nb, b = blockIdx.x % g.nb;
    const ApplySlot A = at.s[si];
    uint32_t *dst = b < g.nb_ldca ? A.ldca + (uint64_t)b * words : A.seav_w + (uint64_t)(b - g.nb_ldca) * words;
    // LDCA buckets of a fresh slot start from zero; SEAV buckets always start from the sketch
    // (a tile with more sampled pairs than it staged records the rest there directly)
    if (A.fresh && b < g.nb_ldca) {
        for (uint32_t w = tid; w < words; w += BLOCK) bm[w] = 0;
    } else {
        for (uint32_t w = tid; w < words; w += BLOCK) bm[w] = dst[w];
    }
    const uint64_t *items64 = reinterpret_cast<const uint64_t *>(items);
    const uint32_t region64 = g.region / 2;
    for (uint32_t t0 = A.tile_lo; t0 < A.tile_hi; t0 += kApplyChunk) {
        const uint32_t nt = A.tile_hi - t0 < kApplyChunk ? A.tile_hi - t0 : kApplyChunk;
        __syncthreads();
        for (uint32_t k = tid; k < nt; k += BLOCK) {
            mbeg[k] = metaT[(uint64_t)b * n_tiles + t0 + k];
            mend[k] = metaT[(uint64_t)(b + 1) * n_tiles + t0 + k];
        }
        __syncthreads();
        for (uint32_t k0 = wid * U; k0 < nt; k0 += NW * U) {
            uint32_t v[U];
            bool ok[U];
            // unconditional loads (lanes without an item re-read the tile's first word and are
            // masked out), so all U loads of a lane are in flight together
            uint64_t w[U];
            uint32_t f[U];
#pragma unroll
            for (uint32_t u = 0; u < U; ++u) {
                const uint32_t k = k0 + u < nt ? k0 + u : nt - 1;
                const uint32_t j = mbeg[k] + lane;
                ok[u] = (k0 + u < nt) && (j < mend[k]);
                const uint32_t jj = ok[u] ? j : 0u;
                f[u] = jj % 3;
                w[u] = items64[(uint64_t)(t0 + k) * region64 + jj / 3];
            }
#pragma unroll
            for (uint32_t u = 0; u < U; ++u) v[u] = (uint32_t)(w[u] >> (21 * f[u])) & 0x1FFFFFu;
#pragma unroll
            for (uint32_t u = 0; u < U; ++u)
                if (ok[u]) atomicOr(&bm[v[u] >> 5], 1u << (v[u] & 31u));
            // segments longer than one wavefront
            for (uint32_t u = 0; u < U; ++u) {
                const uint32_t k = k0 + u;
                if (k >= nt) break;
                const uint32_t end = mend[k];
                for (uint32_t j = mbeg[k] + 64 + lane; j < end; j += 64) {
                    const uint64_t w = items64[(uint64_t)(t0 + k) * region64 + j / 3];
                    const uint32_t it = (uint32_t)(w >> (21 * (j % 3))) & 0x1FFFFFu;
                    atomicOr(&bm[it >> 5], 1u << (it & 31u));
                }
            }
        }
    }
    __syncthreads();
    const uint32_t words4 = words / 4;
    if (words4) {
        for (uint32_t w = tid; w < words4; w += BLOCK)
            reinterpret_cast<u32x4 *>(dst)[w] = reinterpret_cast<const u32x4 *>(bm)[w];
    } else {
        for (uint32_t w = tid; w < words; w += BLOCK) dst[w] = bm[w];
    }
}

template <int U>
static hipError_t launch_apply_u(const BinGeometry &g, const ApplyTable &at, uint32_t n_slots, const uint32_t *items,
                                 const uint32_t *metaT, uint32_t n_tiles, uint32_t block, hipStream_t s) {
    uint32_t lds = ((1u << (g.S - 5)) + 2 * kApplyChunk) * 4u;
    dim3 grid(n_slots * g.nb);
    if (block == 1024) hipLaunchKernelGGL((k_apply<1024, U>), grid, dim3(1024), lds, s, g, at, items, metaT, n_tiles);
    else if (block == 512) hipLaunchKernelGGL((k_apply<512, U>), grid, dim3(512), lds, s, g, at, items, metaT, n_tiles);
    else if (block == 256) hipLaunchKernelGGL((k_apply<256, U>), grid, dim3(256), lds, s, g, at, items, metaT, n_tiles);
    else return hipErrorInvalidConfiguration;
    return hipGetLastError();
}

hipError_t launch_apply(const BinGeometry &g, const ApplySlot *slots, uint32_t n_slots, const uint32_t *items,
                        const uint32_t *metaT, uint32_t n_tiles, uint32_t block, uint32_t unroll, hipStream_t s) {
    ApplyTable at{};
    if (n_slots == 0 || n_slots > (uint32_t)kMaxGroup) return hipErrorInvalidValue;
    for (uint32_t i = 0; i < n_slots; ++i) at.s[i] = slots[i];
    switch (unroll) {
    case 8: return launch_apply_u<8>(g, at, n_slots, items, metaT, n_tiles, block, s);
    case 16: return launch_apply_u<16>(g, at, n_slots, items, metaT, n_tiles, block, s);
    case 32: return launch_apply_u<32>(g, at, n_slots, items, metaT, n_tiles, block, s);
    default: return hipErrorInvalidConfiguration;
    }
}

// ------------------------------------------------------------------------------ merge
__global__ void k_or_merge(uint32_t *__restrict__ dst, SrcTable src, uint32_t n_src, uint64_t n_words) {
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    const uint64_t n4 = n_words / 4;
    for (uint64_t i = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; i < n4; i += stride) {
        u32x4 v = {0u, 0u, 0u, 0u};
        for (uint32_t k = 0; k < n_src; ++k) v |= __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(src.p[k]) + i);
        reinterpret_cast<u32x4 *>(dst)[i] = v;
    }
    for (uint64_t i = n4 * 4 + blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; i < n_words; i += stride) {
        uint32_t v = 0;
        for (uint32_t k = 0; k < n_src; ++k) v |= src.p[k][i];
        dst[i] = v;
    }
}

hipError_t launch_or_merge(uint32_t *dst, const uint32_t *const *srcp, uint32_t n_src, uint64_t n_words, hipStream_t s) {
    SrcTable src{};
    if (n_src == 0 || n_src > (uint32_t)kMaxGroup) return hipErrorInvalidValue;
    for (uint32_t i = 0; i < n_src; ++i) src.p[i] = srcp[i];
    uint64_t blocks = (n_words / 4 + 255) / 256;
    uint32_t grid = (uint32_t)(blocks < 8192 ? (blocks ? blocks : 1) : 8192);
    hipLaunchKernelGGL(k_or_merge, dim3(grid), dim3(256), 0, s, dst, src, n_src, n_words);
    return hipGetLastError();
}

__global__ void k_max_merge_u16(uint16_t *__restrict__ dst, SrcTable16 src, uint32_t n_src, uint64_t n) {
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t i = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; i < n; i += stride) {
        uint16_t v = 0;
        for (uint32_t k = 0; k < n_src; ++k) {
            uint16_t t = src.p[k][i];
            v = t > v ? t : v;
        }
        dst[i] = v;
    }
}

hipError_t launch_max_merge_u16(uint16_t *dst, const uint16_t *const *srcp, uint32_t n_src, uint64_t n, hipStream_t s) {
    SrcTable16 src{};
    if (n_src == 0 || n_src > (uint32_t)kMaxGroup) return hipErrorInvalidValue;
    for (uint32_t i = 0; i < n_src; ++i) src.p[i] = srcp[i];
    uint64_t blocks = (n + 255) / 256;
    uint32_t grid = (uint32_t)(blocks < 8192 ? (blocks ? blocks : 1) : 8192);
    hipLaunchKernelGGL(k_max_merge_u16, dim3(grid), dim3(256), 0, s, dst, src, n_src, n);
    return hipGetLastError();
}

// Shift every stamp down by off; stamps at or below off (outside every future window) become 0.
__global__ void k_renormalize_u16(uint16_t *__restrict__ p, uint64_t n, uint16_t off) {
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t i = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; i < n; i += stride) {
        uint16_t v = p[i];
        p[i] = v > off ? (uint16_t)(v - off) : (uint16_t)0;
    }
}

hipError_t launch_renormalize_u16(uint16_t *p, uint64_t n, uint16_t off, hipStream_t s) {
    uint64_t blocks = (n + 255) / 256;
    uint32_t grid = (uint32_t)(blocks < 8192 ? (blocks ? blocks : 1) : 8192);
    hipLaunchKernelGGL(k_renormalize_u16, dim3(grid), dim3(256), 0, s, p, n, off);
    return hipGetLastError();
}

// Bit view of stamps: bit j of word w is 1 iff ts[32 w + j] >= thr.
__global__ void k_bit_view(const uint16_t *__restrict__ ts, uint64_t n_words, uint16_t thr, uint32_t *__restrict__ out) {
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t w = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; w < n_words; w += stride) {
        uint32_t v = 0;
        for (uint32_t j = 0; j < 32; ++j) v |= (ts[w * 32 + j] >= thr ? 1u : 0u) << j;
        out[w] = v;
    }
}

hipError_t launch_bit_view(const uint16_t *ts, uint64_t n_bits, uint16_t thr, uint32_t *out_words, hipStream_t s) {
    uint64_t n_words = n_bits / 32;
    uint64_t blocks = (n_words + 255) / 256;
    uint32_t grid = (uint32_t)(blocks < 8192 ? (blocks ? blocks : 1) : 8192);
    hipLaunchKernelGGL(k_bit_view, dim3(grid), dim3(256), 0, s, ts, n_words, thr, out_words);
    return hipGetLastError();
}

// ------------------------------------------------------------------------------ end of window
// What the end of window reads: bits, or the counters of a sliding window, of which 32 stand for a
// word of bits.
template <int MODE>
struct RawWord {
    u32x4 v[MODE == kCloseStamps ? 4 : 2];
};
template <>
struct RawWord<kCloseBits> {
    uint32_t v;
};
template <int MODE>
__device__ __forceinline__ RawWord<MODE> load_raw(const void *p) {
    RawWord<MODE> r;
#pragma unroll
    for (uint32_t q = 0; q < (MODE == kCloseStamps ? 4u : 2u); ++q) r.v[q] = reinterpret_cast<const u32x4 *>(p)[q];
    return r;
}
template <>
__device__ __forceinline__ RawWord<kCloseBits> load_raw<kCloseBits>(const void *p) {
    return RawWord<kCloseBits>{*reinterpret_cast<const uint32_t *>(p)};
}
// The two 16-bit stamps of a 32-bit word as bits.
__device__ __forceinline__ uint32_t ts_bits2(uint32_t w, uint32_t thr) {
    return ((w & 0xFFFFu) >= thr ? 1u : 0u) | ((w >> 16) >= thr ? 2u : 0u);
}
template <int MODE>
__device__ __forceinline__ uint32_t decode_raw(const CloseArgs &a, const RawWord<MODE> &r) {
    if constexpr (MODE == kCloseBits) {
        return r.v;
    } else if constexpr (MODE == kCloseAt) {
        return at_word(r.v[0], r.v[1], a.at);
    } else {
        uint32_t v = 0;
#pragma unroll
        for (uint32_t q = 0; q < 4; ++q) {
            const u32x4 x = r.v[q];
            v |= (ts_bits2(x.x, a.thr) | ts_bits2(x.y, a.thr) << 2 | ts_bits2(x.z, a.thr) << 4 | ts_bits2(x.w, a.thr) << 6)
                 << (8 * q);
        }
        return v;
    }
}
// 32 AT counters as one word of bits in a permuted order, counter 4 h + j at bit 8 j + h: a shift and a
// merge for every four counters.  The order is the same for all words, so it serves wherever bits are
// only compared with bits of the same place and counted: the AND of a candidate's LDCs, and the AND of
// its SEs.  (In their own order, and with an at_flags4 of 14 operations, decoding was two thirds of the
// arithmetic of the end of a sliding window, which kept the SIMDs busy for 37 of its 68 us.)
__device__ __forceinline__ uint32_t at_word_permuted(const u32x4 &x, const u32x4 &y, const AtView &v) {
    constexpr uint32_t H = 0x80808080u;
    uint32_t p = at_flags4(x.x, v);
    auto put = [&](uint32_t w) { p = ((p >> 1) & ~H) | (at_flags4(w, v) & H); };
    put(x.y); put(x.z); put(x.w); put(y.x); put(y.y); put(y.z); put(y.w);
    return p;
}
// The bits of an LDC word, or of four SEs: decoded as in decode_raw, but AT counters permuted.
template <int MODE>
__device__ __forceinline__ uint32_t decode_any_order(const CloseArgs &a, const RawWord<MODE> &r) {
    if constexpr (MODE == kCloseAt) return at_word_permuted(r.v[0], r.v[1], a.at);
    else return decode_raw<MODE>(a, r);
}
// Of such a word of four SEs: without its first d SEs (0 to 3); the weights of the SEs, one per byte; the bits of
// SE j (in any fixed order).  Permuted, SE q has bits 8 j + 2 q and 8 j + 2 q + 1 of the four bytes j.
template <int MODE>
__device__ __forceinline__ uint32_t skip_ses(uint32_t v, uint32_t d) {
    if constexpr (MODE == kCloseAt) return (v >> (2 * d)) & ((0xFFu >> (2 * d)) * 0x01010101u);
    else return v >> (8 * d);
}
template <int MODE>
__device__ __forceinline__ uint32_t se_weights(uint32_t v) {
    uint32_t t = v - ((v >> 1) & 0x55555555u);
    if constexpr (MODE == kCloseAt) {
        const uint32_t even = ((t & 0x33333333u) * 0x01010101u) >> 24;          // SE 0, and 2 in the upper half
        const uint32_t odd = (((t >> 2) & 0x33333333u) * 0x01010101u) >> 24;    // SE 1 and 3
        t = even | odd << 8;
        return (t & 0x0F0Fu) | (t & 0xF0F0u) << 12;
    } else {
        t = (t & 0x33333333u) + ((t >> 2) & 0x33333333u);
        return (t + (t >> 4)) & 0x0F0F0F0Fu;
    }
}
template <int MODE>
__device__ __forceinline__ uint32_t se_bits(uint32_t v, uint32_t j) {
    if constexpr (MODE == kCloseAt) return (((v >> (2 * j)) & 0x03030303u) * 0x01041040u) >> 24;   // byte i to bit 2 i
    else return (v >> (8 * j)) & 0xFFu;
}
// 32 bits of the SEAV from byte `byte` on; one byte of it; word `word` of the LDCA (below 2^27: a
// sketch has fewer than 2^32 bits).
template <int MODE>
__device__ __forceinline__ RawWord<MODE> load_sea(const CloseArgs &a, uint32_t byte) {
    if constexpr (MODE == kCloseBits) return load_raw<MODE>(a.seav + byte);
    else if constexpr (MODE == kCloseAt) return load_raw<MODE>(a.seav_at + byte * 8u);
    else return load_raw<MODE>(a.seav_ts + (uint64_t)byte * 8);
}
template <int MODE>
__device__ __forceinline__ uint32_t load_se(const CloseArgs &a, uint64_t byte) {
    if constexpr (MODE == kCloseBits) {
        return a.seav[byte];
    } else if constexpr (MODE == kCloseAt) {
        const uint32_t *t = reinterpret_cast<const uint32_t *>(a.seav_at + byte * 8);
        return at_byte(t[0], t[1], a.at);
    } else {
        const u32x4 x = *reinterpret_cast<const u32x4 *>(a.seav_ts + byte * 8);
        return ts_bits2(x.x, a.thr) | ts_bits2(x.y, a.thr) << 2 | ts_bits2(x.z, a.thr) << 4 | ts_bits2(x.w, a.thr) << 6;
    }
}
template <int MODE>
__device__ __forceinline__ RawWord<MODE> load_ldc(const CloseArgs &a, uint32_t word) {
    // (bits and AT counters: a 32-bit byte offset from a scalar base)
    if constexpr (MODE == kCloseBits) return load_raw<MODE>(reinterpret_cast<const uint8_t *>(a.ldca) + word * 4u);
    else if constexpr (MODE == kCloseAt) return load_raw<MODE>(a.ldca_at + word * 32u);
    else return load_raw<MODE>(a.ldca_ts + (uint64_t)word * 32);
}

// Orders LDS traffic between lanes of one wavefront (writes by some lanes, reads by others).
__device__ __forceinline__ void wave_lds_sync() {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_wave_barrier();
}

__device__ __forceinline__ uint32_t wave_sum(uint32_t v) {
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// One super point: to the device records, and the first ones straight to host-visible memory, written
// through (the workgroup waits for them before it counts itself finished).
__device__ __forceinline__ void report(const CloseArgs &a, uint32_t h, uint32_t z0) {
    const uint32_t slot = atomicAdd(&a.counters[0], 1u);
    const uint64_t v = (uint64_t)h | (uint64_t)z0 << 32;
    if (slot < a.rec_cap) reinterpret_cast<uint64_t *>(a.rec)[slot] = v;
    if (slot < a.host_recs)
        __hip_atomic_store(reinterpret_cast<uint64_t *>(a.host_out + 4) + slot, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// ULDC of candidates cand(e), e < n, of which this wavefront takes its share (share of NS): AND of
// the LR LDCs, z0 = k - popcount, reported if z0 <= z_theta.
// Bits: four candidates at a time, 16 lanes each; a lane reads 8 words of each of two LDCs before it
// waits, so one round trip to memory serves four candidates (k = 4096, LR = 2).
// Counters: an LDC word is 32 counters (64 or 32 bytes), so one candidate takes the whole wavefront:
// each lane reads two words of a row at a time; AT counters of two rows are loaded before either is
// decoded (the larger 16-bit stamps go one row at a time).
template <int MODE, typename Get>
__device__ __forceinline__ void filter_candidates(const CloseArgs &a, const Consts &c, Get cand, uint32_t n, uint32_t share,
                                                  uint32_t NS, uint32_t lane) {
    const uint32_t words = 1u << (c.log2k - 5);
    if constexpr (MODE == kCloseBits) {
        constexpr uint32_t G = 16, W = 8, RB = 2, PER = 64 / G;
        const uint32_t grp = lane / G, sub = lane % G;
        for (uint32_t e0 = share * PER; e0 < n; e0 += NS * PER) {
            const bool live = e0 + grp < n;
            const uint32_t h = cand(live ? e0 + grp : e0);
            uint32_t ones = 0;
            for (uint32_t w0 = 0; w0 < words; w0 += G * W) {
                uint32_t u[W];
#pragma unroll
                for (uint32_t k = 0; k < W; ++k) u[k] = 0xFFFFFFFFu;
                for (uint32_t r0 = 0; r0 < c.lr; r0 += RB) {
                    uint32_t v[RB][W];
#pragma unroll
                    for (uint32_t rr = 0; rr < RB; ++rr) {
                        const uint32_t r = r0 + rr < c.lr ? r0 + rr : c.lr - 1;   // a repeated row is harmless
                        const uint32_t base = ((r << c.log2lc) | ldc_col(h, r, c)) << (c.log2k - 5);
#pragma unroll
                        for (uint32_t k = 0; k < W; ++k) {
                            const uint32_t w = w0 + k * G + sub;
                            v[rr][k] = load_ldc<MODE>(a, base + (w < words ? w : words - 1)).v;
                        }
                    }
#pragma unroll
                    for (uint32_t rr = 0; rr < RB; ++rr)
#pragma unroll
                        for (uint32_t k = 0; k < W; ++k) u[k] &= v[rr][k];
                }
#pragma unroll
                for (uint32_t k = 0; k < W; ++k)
                    if (w0 + k * G + sub < words) ones += __popc(u[k]);
            }
            for (uint32_t o = G / 2; o > 0; o >>= 1) ones += __shfl_xor(ones, o, 64);
            const uint32_t z0 = (1u << c.log2k) - ones;
            if (live && sub == 0 && z0 <= c.z_theta) report(a, h, z0);
        }
    } else {
        // Counters are 8 or 16 times the bits' bytes, and the AND of the rows has no more ones than its
        // first row: a candidate whose first row alone is too empty is done (most of the false ones).
        // Two candidates' first rows of AT counters are loaded together: 55 us of the sliding window
        // below, one at a time 64, four (94 registers) 65; all rows of one at once 68.
        constexpr uint32_t C = MODE == kCloseAt ? 2 : 1, RB = MODE == kCloseAt ? 2 : 1;
        const uint32_t row_words = c.log2k - 5;
        auto row_base = [&](uint32_t h, uint32_t r) { return ((r << c.log2lc) | ldc_col(h, r, c)) << row_words; };
        for (uint32_t e = share; e < n; e += C * NS) {
            uint32_t h[C], ones[C], ua[C], ub[C];
#pragma unroll
            for (uint32_t k = 0; k < C; ++k) {
                h[k] = __builtin_amdgcn_readfirstlane(cand(e + k * NS < n ? e + k * NS : e));
                ones[k] = 0;
            }
            for (uint32_t w0 = 0; w0 < words; w0 += 128) {
                const uint32_t wa = w0 + lane < words ? w0 + lane : words - 1;
                const uint32_t wb = w0 + 64 + lane < words ? w0 + 64 + lane : words - 1;
                RawWord<MODE> x[C], y[C];
#pragma unroll
                for (uint32_t k = 0; k < C; ++k) {
                    const uint32_t base = row_base(h[k], 0);
                    x[k] = load_ldc<MODE>(a, base + wa);
                    y[k] = load_ldc<MODE>(a, base + wb);
                }
#pragma unroll
                for (uint32_t k = 0; k < C; ++k) {
                    ua[k] = w0 + lane < words ? decode_any_order<MODE>(a, x[k]) : 0u;
                    ub[k] = w0 + 64 + lane < words ? decode_any_order<MODE>(a, y[k]) : 0u;
                    ones[k] += __popc(ua[k]) + __popc(ub[k]);
                }
            }
#pragma unroll
            for (uint32_t k = 0; k < C; ++k) {
                uint32_t z0 = (1u << c.log2k) - __builtin_amdgcn_readfirstlane(wave_sum(ones[k]));
                if (z0 > c.z_theta || e + k * NS >= n) continue;
                if (c.lr > 1) {
                    // the other rows (all of them again where a row takes several rounds)
                    const bool once = words <= 128;
                    uint32_t sum = 0;
                    for (uint32_t w0 = 0; w0 < words; w0 += 128) {
                        const uint32_t wa = w0 + lane < words ? w0 + lane : words - 1;
                        const uint32_t wb = w0 + 64 + lane < words ? w0 + 64 + lane : words - 1;
                        uint32_t va = once ? ua[k] : 0xFFFFFFFFu, vb = once ? ub[k] : 0xFFFFFFFFu;
                        for (uint32_t r0 = once ? 1u : 0u; r0 < c.lr; r0 += RB) {
                            RawWord<MODE> x[RB], y[RB];
#pragma unroll
                            for (uint32_t rr = 0; rr < RB; ++rr) {
                                const uint32_t base = row_base(h[k], r0 + rr < c.lr ? r0 + rr : c.lr - 1);
                                x[rr] = load_ldc<MODE>(a, base + wa);
                                y[rr] = load_ldc<MODE>(a, base + wb);
                            }
#pragma unroll
                            for (uint32_t rr = 0; rr < RB; ++rr) {
                                va &= decode_any_order<MODE>(a, x[rr]);
                                vb &= decode_any_order<MODE>(a, y[rr]);
                            }
                        }
                        sum += (w0 + lane < words ? __popc(va) : 0u) + (w0 + 64 + lane < words ? __popc(vb) : 0u);
                    }
                    z0 = (1u << c.log2k) - wave_sum(sum);
                }
                if (lane == 0 && z0 <= c.z_theta) report(a, h[k], z0);
            }
        }
    }
}

// The same for a queue that has filled up (crowded SEAs only): one candidate at a time, little code.
template <int MODE>
__device__ __forceinline__ void filter_queue(const CloseArgs &a, const Consts &c, const uint32_t *queue, uint32_t n,
                                             uint32_t lane) {
    const uint32_t words = 1u << (c.log2k - 5);
    for (uint32_t e = 0; e < n; ++e) {
        const uint32_t h = queue[e];
        uint32_t ones = 0;
        for (uint32_t w = lane; w < words; w += 64) {
            uint32_t u = 0xFFFFFFFFu;
            for (uint32_t r = 0; r < c.lr; ++r)
                u &= decode_any_order<MODE>(a, load_ldc<MODE>(a, (((r << c.log2lc) | ldc_col(h, r, c)) << (c.log2k - 5)) + w));
            ones += __popc(u);
        }
        const uint32_t z0 = (1u << c.log2k) - wave_sum(ones);
        if (lane == 0 && z0 <= c.z_theta) report(a, h, z0);
    }
}

// One wavefront per work item, an SEA or one of its 2^parts_log2 parts.  An SEA's words go straight
// from memory to registers (those of the next item are loaded before the current one is worked on);
// hot SEs are found four at a time by a bytewise popcount and listed in LDS in the SEA's order, so that
// a row's are neighbours and every wavefront of an SEA sees the same list.
// Candidates wait in a queue per wavefront; when the workgroup's items are done, its wavefronts share
// the filtering of all of them, so that an SEA with many candidates does not hold up one wavefront.
// Bound by latency: a round trip for the SEAs, one or two per candidate filtered.
// (64 Mi pairs, 16384 SEAs, 16 700 candidates: 39.6 us and a separate kernel of 4 us that copied the
// counts and records out, now 29 us with both; 8 routers, 36 000 candidates 87 + 4 -> 51; a sliding
// window of AT counters, 20 900 candidates, 89 + 4 and 17 for a bit view of the SEAV -> 55; of stamps,
// 1024 SEAs, 67 + 4 and 5 -> 25.)
// RMAX: SR itself when it is 4, else 8 (the rows' registers).
template <int MODE, int BLOCK, int RMAX>
__device__ __forceinline__ void close_window(const Consts &c, const CloseArgs &a) {
    extern __shared__ uint32_t lds[];
    constexpr uint32_t NW = BLOCK / 64;
    constexpr uint32_t U = MODE == kCloseBits ? 8 : 2;   // words in flight per lane
    __shared__ uint32_t wave_q[NW], wave_cand[NW];   // kCloseStaticWords each
    const uint32_t sr = RMAX == 4 ? 4u : c.sr;
    const uint32_t lane = threadIdx.x & 63u, wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t per_wave = close_wave_words(c.sea_bytes, a.qcap);
    // hot SEs row after row: (the LP bits each stands for, or, of more than 24, its cell) << 8 | value
    uint32_t *list = lds + wid * per_wave;
    const bool lp24 = c.L <= 24u;
    uint32_t *queue = list + c.sea_bytes;
    const uint64_t lane_lt = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    const uint64_t lmask = (c.L == 32) ? 0xFFFFFFFFull : ((1ull << c.L) - 1ull);
    uint32_t n_cand = 0, qn = 0;
    // work items: (SEA, part); the 2^parts_log2 parts of a SEA take interleaved shares of its tuples
    // (or of its LPs), or of the candidates when the tuples are few: disjoint candidates either way
    const uint32_t P = 1u << a.parts_log2, part_mask = P - 1u;
    const uint32_t n_items = a.n_rp << a.parts_log2, step = gridDim.x * NW;   // at most 2^30
    // an SEA's words; the last one is read from the SEA's last four bytes
    const uint32_t sea_words = (c.sea_bytes + 3) / 4, last_byte = c.sea_bytes - 4;
    auto word_byte = [&](uint32_t w) { return w < sea_words ? min(4 * w, last_byte) : 0u; };
    RawWord<MODE> raw[U];
    auto fetch = [&](uint32_t wi, uint32_t w0) {
        const uint32_t sea = (wi >> a.parts_log2) * c.sea_bytes;   // below 2^29
#pragma unroll
        for (uint32_t k = 0; k < U; ++k)
            if (w0 + k * 64 < sea_words) raw[k] = load_sea<MODE>(a, sea + word_byte(w0 + k * 64 + lane));
    };
    // the candidates of a round, one per lane, to the queue, which is filtered when it is full
    auto flush = [&]() {
        wave_lds_sync();
        filter_queue<MODE>(a, c, queue, qn, lane);
        n_cand += qn;
        qn = 0;
        wave_lds_sync();
    };
    auto push = [&](uint64_t bal, uint32_t h) {
        if (bal >> lane & 1u) queue[qn + __popcll(bal & lane_lt)] = h;
        qn += (uint32_t)__popcll(bal);
        if (qn + 64 > a.qcap) flush();
    };

    uint32_t wi = blockIdx.x * NW + wid;
    if (wi < n_items) fetch(wi, 0);
    for (; wi < n_items; wi += step) {
        const uint32_t rp = wi >> a.parts_log2, part = wi & part_mask, sea = rp * c.sea_bytes;
        uint32_t n_hot = 0;
        for (uint32_t w0 = 0; w0 < sea_words; w0 += 64 * U) {
            uint32_t v[U];
#pragma unroll
            for (uint32_t k = 0; k < U; ++k) {
                const uint32_t w = w0 + k * 64 + lane;
                v[k] = 0;
                if (w0 + k * 64 < sea_words) {
                    v[k] = decode_any_order<MODE>(a, raw[k]);
                    v[k] = w < sea_words ? skip_ses<MODE>(v[k], 4 * w - word_byte(w)) : 0u;
                }
            }
            if (w0 + 64 * U < sea_words) fetch(wi, w0 + 64 * U);
            else if (wi + step < n_items) fetch(wi + step, 0);
#pragma unroll
            for (uint32_t k = 0; k < U; ++k) {
                if (w0 + k * 64 >= sea_words) continue;
                // bytes of weight >= kSeHot
                uint32_t hot = (se_weights<MODE>(v[k]) + (0x80u - kSeHot) * 0x01010101u) & 0x80808080u;
                if (!__ballot(hot != 0)) continue;
                // places by lane: a prefix sum of the lanes' counts (0 to 4), one bit at a time
                const uint32_t n = __popc(hot);
                const uint64_t b0 = __ballot(n & 1u), b1 = __ballot(n & 2u), b2 = __ballot(n & 4u);
                uint32_t pos = n_hot + (uint32_t)(__popcll(b0 & lane_lt) + 2 * __popcll(b1 & lane_lt) + 4 * __popcll(b2 & lane_lt));
                n_hot += (uint32_t)(__popcll(b0) + 2 * __popcll(b1) + 4 * __popcll(b2));
                const uint32_t byte0 = 4 * (w0 + k * 64 + lane);
                while (hot) {
                    const uint32_t j = (uint32_t)__builtin_ctz(hot) >> 3;
                    hot &= hot - 1;
                    list[pos++] = (byte0 + j) << 8 | se_bits<MODE>(v[k], j);
                }
            }
        }
        if (n_hot < sr) continue;
        wave_lds_sync();
        // the rows' parts of the list: begin[i] = entries before row i; cells become LP bits (Eq. 3).
        // Row loops run over RMAX with constant indices (guarded by the row count), so the per-row
        // arrays stay in registers and the row constants are read from the kernel arguments directly.
        uint32_t begin[RMAX];
#pragma unroll
        for (uint32_t i = 0; i < (uint32_t)RMAX; ++i) begin[i] = 0;
        for (uint32_t e0 = 0; e0 < n_hot; e0 += 64) {
            const bool in = e0 + lane < n_hot;
            const uint32_t e = list[in ? e0 + lane : e0], byte = e >> 8;
            uint32_t off = 0, isb = c.isb[0];
#pragma unroll
            for (uint32_t i = 1; i < (uint32_t)RMAX; ++i) {
                if (i >= sr) continue;
                const bool past = byte >= c.row_off[i];
                off = past ? c.row_off[i] : off;
                isb = past ? c.isb[i] : isb;
                begin[i] += (uint32_t)__popcll(__ballot(in && !past));
            }
            const uint32_t cell = byte - off;
            if (in) list[e0 + lane] = (lp24 ? row_bits_in_lp(cell, isb, c.L) : cell) << 8 | (e & 0xFFu);
        }
        uint32_t cnt[RMAX];
        uint64_t prod = 1;
#pragma unroll
        for (uint32_t i = 0; i < (uint32_t)RMAX; ++i) {
            cnt[i] = 1;
            if (i >= sr) continue;
            const bool last = i + 1 >= (uint32_t)RMAX || i + 1 >= sr;
            cnt[i] = (last ? n_hot : begin[i + 1 < (uint32_t)RMAX ? i + 1 : i]) - begin[i];
            prod = min(prod * cnt[i], 1ull << 33);   // (past every LP count)
        }
        if (prod == 0) continue;
        wave_lds_sync();
        const bool each_lp = prod > lmask;
        bool crowded = prod > 2048u;
        if (crowded && prod <= 8192u && !each_lp) {   // (short rows: too few entries for a step of their own)
            crowded = false;
#pragma unroll
            for (uint32_t i = 0; i < (uint32_t)RMAX; ++i) crowded = crowded || cnt[i] >= 16u;
        }
        if (crowded) {
            // Crowded, in two steps.  The tuples of the other rows, one per lane: those whose own bits agree
            // and whose SEs share enough bits (few: two overlaps of two bits alone leave one in 16) meet the
            // longest row's entries, one per lane.  With as many tuples as hosts in this SEA, or more, every
            // LP instead (the candidate definition), its SEs in LDS in place of the list: the upper bits of an
            // LP decide the rows that take none of the lowest six, and the 64 LPs of those that pass are
            // tested together.
            // (One lane per whole tuple or LP: windows of 64 SEAs at theta = 64, 200,000 pairs, 2.69 ms, so
            // 0.115; 256 SEAs at theta = 128, 1,000,000 pairs, 4.55 and 0.19.)
            // (The constants of the rows come from the kernel arguments behind an opaque pointer: nothing of
            // this is kept in registers by a launch without such an SEA.)
            auto args = __builtin_amdgcn_kernarg_segment_ptr();
            asm volatile("" : "+s"(args));
            ArgConsts &rc = *(ArgConsts *)args;
            auto *lp_mask = ((__attribute__((address_space(4))) const CloseArgs *)((ArgConsts *)args + 1))->lp_mask;
            uint32_t cm = cnt[0], im = 0, bm = begin[0], mask = lp_mask[0], isbm = rc.isb[0], cover = 0, total = 1;
#pragma unroll
            for (uint32_t i = 1; i < (uint32_t)RMAX; ++i)
                if (i < sr && cnt[i] > cm) cm = cnt[i], im = i, bm = begin[i], mask = lp_mask[i], isbm = rc.isb[i];
            float rcp[RMAX];
#pragma unroll
            for (uint32_t i = 0; i < (uint32_t)RMAX; ++i) {
                rcp[i] = __builtin_amdgcn_rcpf((float)cnt[i]);
                if (i >= sr || i == im) continue;
                total *= cnt[i];
                cover |= lp_mask[i];
            }
            mask &= cover;   // the bits that the longest row shares with others
            const bool small = total <= (1u << 20);
            uint8_t *se = reinterpret_cast<uint8_t *>(list);
            if (each_lp) {
                total = (uint32_t)((lmask + 1) >> 6);
                cm = 64;
#pragma nounroll
                for (uint32_t b = lane; b < c.sea_bytes; b += 64) se[b] = (uint8_t)load_se<MODE>(a, sea + b);
                wave_lds_sync();
            }
            // (shares interleaved one by one: the other rows' tuples may be few)
            for (uint64_t t0 = part; t0 < total; t0 += 64u * P) {
                uint32_t lp = 0, seu = 0xFFu, differ = 0;
                bool ok = t0 + (uint64_t)lane * P < total;
                uint32_t u = ok ? (uint32_t)t0 + lane * P : 0u;
                if (each_lp) {
                    lp = u << 6;
#pragma unroll
                    for (uint32_t i = 0; i < (uint32_t)RMAX; ++i)
                        if (i < sr && !(lp_mask[i] & 63u)) seu &= se[rc.row_off[i] + row_index(lp, rc.isb[i], rc.ibn[i], c.L)];
                } else {
                    uint32_t bits[RMAX];
#pragma unroll
                    for (uint32_t i = 0; i < (uint32_t)RMAX; ++i) {
                        bits[i] = 0;
                        if (i >= sr || i == im) continue;
                        const uint32_t q = small ? (uint32_t)(((float)u + 0.5f) * rcp[i]) : u / cnt[i];
                        const uint32_t e = list[begin[i] + u - q * cnt[i]];
                        u = q;
                        bits[i] = lp24 ? e >> 8 : row_bits_in_lp(e >> 8, rc.isb[i], c.L);
                        seu &= e;
                        lp |= bits[i];
                    }
#pragma unroll
                    for (uint32_t i = 0; i < (uint32_t)RMAX; ++i)
                        if (i < sr && i != im) differ |= (lp & lp_mask[i]) ^ bits[i];
                }
                ok = ok && __popc(seu) >= kSeHot && differ == 0;
                for (uint64_t left = __ballot(ok); left; left &= left - 1) {
                    const uint32_t l = (uint32_t)__builtin_ctzll(left);
                    const uint32_t lp1 = __builtin_amdgcn_readlane(lp, l), seu1 = __builtin_amdgcn_readlane(seu, l);
                    for (uint32_t e0 = 0; e0 < cm; e0 += 64) {
                        uint32_t lp2 = lp1 | lane, seu2 = seu1;
                        bool cand = true;
                        if (each_lp) {
#pragma unroll
                            for (uint32_t i = 0; i < (uint32_t)RMAX; ++i)
                                if (i < sr && (lp_mask[i] & 63u)) seu2 &= se[rc.row_off[i] + row_index(lp2, rc.isb[i], rc.ibn[i], c.L)];
                        } else {
                            cand = e0 + lane < cm;
                            const uint32_t e = list[bm + (cand ? e0 + lane : e0)];
                            const uint32_t b = lp24 ? e >> 8 : row_bits_in_lp(e >> 8, isbm, c.L);
                            cand = cand && ((lp1 ^ b) & mask) == 0;
                            seu2 &= e;
                            lp2 = lp1 | b;
                        }
                        const uint64_t bal = __ballot(cand && __popc(seu2) >= kSeHot);
                        if (bal) push(bal, (uint32_t)((uint64_t)lp2 << c.r | rp));
                    }
                }
            }
        } else {
            const uint32_t total = (uint32_t)prod;
            // the product CIS of the hot lists (Section 3.2), one tuple per lane: the tuple number's
            // mixed-radix digits (row 0 least significant) pick its entries.  A digit's quotient is
            // exact in single precision (below 2^20): (u + 1/2) / cnt is at least 1 / (2 cnt) from an
            // integer, and the product's relative error is below 2^-22.  (Integer divisions took three
            // quarters of this kernel: 64 Mi pairs, 16384 SEAs of one tuple on average.)  Few tuples
            // are enumerated by every part, which keeps its share of the candidates: their filtering
            // is what takes time then.
            const bool all = total <= 256u;
            const uint32_t first = all ? 0u : part * 64u, stride = all ? 64u : 64u * P;
            float rcp[RMAX];
#pragma unroll
            for (uint32_t i = 0; i < (uint32_t)RMAX; ++i) rcp[i] = __builtin_amdgcn_rcpf((float)cnt[i]);
            uint32_t found = 0;
            uint32_t u0 = first, rounds = first < total ? ((total - 1 - first) >> (all ? 6u : 6u + a.parts_log2)) + 1 : 0u;
            for (; rounds; --rounds, u0 += stride) {
                bool cand = false;
                uint32_t h = 0;
                if (lane < total - u0) {
                    uint32_t u = u0 + lane, lp = 0, seu = 0xFFu;
                    uint32_t bits[RMAX];
#pragma unroll
                    for (uint32_t i = 0; i < (uint32_t)RMAX; ++i) {
                        bits[i] = 0;
                        if (i >= sr) continue;
                        uint32_t q = 0;
                        if (i + 1 < sr) q = (uint32_t)(((float)u + 0.5f) * rcp[i]);
                        const uint32_t e = list[begin[i] + u - q * cnt[i]];
                        u = q;
                        bits[i] = lp24 ? e >> 8 : row_bits_in_lp(e >> 8, c.isb[i], c.L);
                        seu &= e;
                        lp |= bits[i];
                    }
                    // Eq. 3: the rebuilt LP must give back every row's bits (overlap bits agree)
                    uint32_t differ = 0;
#pragma unroll
                    for (uint32_t i = 0; i < (uint32_t)RMAX; ++i)
                        if (i < sr) differ |= (lp & a.lp_mask[i]) ^ bits[i];
                    cand = __popc(seu) >= kSeHot && differ == 0;
                    h = (uint32_t)(((uint64_t)lp << c.r) | rp);
                }
                uint64_t bal = __ballot(cand);
                if (!bal) continue;
                if (all && P > 1) {
                    const uint32_t j = found + (uint32_t)__popcll(bal & lane_lt);
                    found += (uint32_t)__popcll(bal);
                    cand = cand && (j & part_mask) == part;
                    bal = __ballot(cand);
                }
                push(bal, h);
            }
        }
    }
    // the candidates left in the wavefronts' queues, shared out among them
    if (lane == 0) {
        wave_q[wid] = qn;
        wave_cand[wid] = n_cand + qn;
    }
    __syncthreads();
    uint32_t left = 0, sum = 0;
#pragma unroll
    for (uint32_t w = 0; w < NW; ++w) {
        left += __builtin_amdgcn_readfirstlane(wave_q[w]);
        sum += wave_cand[w];
    }
    if (left) {
        auto get = [&](uint32_t e) {
            uint32_t w = 0;
#pragma unroll
            for (uint32_t i = 0; i + 1 < NW; ++i) {   // past the first w queues
                const bool past = w == i && e >= wave_q[i];
                e -= past ? wave_q[i] : 0u;
                w += past ? 1u : 0u;
            }
            return lds[w * per_wave + c.sea_bytes + e];
        };
        filter_candidates<MODE>(a, c, get, left, wid, NW, lane);
    }
    // Every wavefront's records have been written through to host memory before its workgroup counts
    // itself finished, so no cache has to be written back (a release per workgroup cost 11 us over
    // 1280 of them).  That rests on the hardware, not on the memory model: system-scope stores to coherent
    // host memory are write-through on this chip, and the counter waited for falls when they are
    // acknowledged.  The last workgroup publishes the counts and, last of all, the close's sequence
    // number, which the host may poll instead of waiting for the stream.
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (threadIdx.x) return;
    auto finish = [](uint64_t *p, uint64_t v, uint32_t members, uint32_t &cand) {
        const uint64_t old = __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + v;
        cand = (uint32_t)(old >> 32);
        if ((uint32_t)old != members) return false;
        *p = 0;   // for the next close (nobody else reads it in this one)
        return true;
    };
    const uint32_t grp = blockIdx.x % kCloseGroups, groups = min(gridDim.x, kCloseGroups);
    uint32_t cand;
    if (!finish(a.counts + (1 + grp) * kCloseLine, (uint64_t)sum << 32 | 1u, (gridDim.x - grp + kCloseGroups - 1) / kCloseGroups, cand))
        return;
    if (!finish(a.counts, (uint64_t)cand << 32 | 1u, groups, cand)) return;
    const uint32_t n = __hip_atomic_load(&a.counters[0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const uint32_t seq = a.counters[2] + 1u;
    a.counters[0] = 0u;
    a.counters[2] = seq;
    __hip_atomic_store(a.host_out, n, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    __hip_atomic_store(a.host_out + 1, cand, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __hip_atomic_store(a.host_out + 2, seq, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// Wavefronts per SIMD that the registers leave room for: with many small SEAs (2^20 of 64 bytes) the LDS
// leaves eight, and one wavefront less costs a tenth.  (One more in the instances for any row count spills
// to memory.)
constexpr uint32_t close_waves(int mode, int rows) {
    return rows != 4 ? (mode == kCloseStamps ? 4u : 6u) : mode == kCloseBits ? 7u : mode == kCloseAt ? 6u : 5u;
}
template <int MODE, int BLOCK, int RMAX>
__global__ __launch_bounds__(BLOCK, close_waves(MODE, RMAX)) void k_close(Consts c, CloseArgs a) { close_window<MODE, BLOCK, RMAX>(c, a); }

// Several windows at once (the serving loop closes what a scan launch has completed): one window's close
// waits for memory most of its time, so they run side by side, blockIdx.y naming the window.  16 windows
// of 4 Mi pairs: 500 us one after another (13.5 us each, and the launches between them).
template <int BLOCK, int RMAX>
__global__ __launch_bounds__(BLOCK, close_waves(kCloseBits, RMAX)) void k_close_many(Consts c, CloseArgs a, CloseTable t) {
    const CloseSlot s = t.s[blockIdx.y];
    a.seav = s.seav;
    a.ldca = s.ldca;
    a.rec = s.rec;
    a.counters = s.counters;
    a.counts += blockIdx.y * (kCloseCountBytes / 8);
    a.host_out = s.host_out;
    a.host_recs = s.host_recs;
    a.rec_cap = s.rec_cap;
    close_window<kCloseBits, BLOCK, RMAX>(c, a);
}

// The instance for a mode, a workgroup size and a row count.
typedef void (*CloseKernel)(Consts, CloseArgs);
template <int MODE, int BLOCK>
static CloseKernel close_kernel_rows(uint32_t sr) { return sr == 4 ? k_close<MODE, BLOCK, 4> : k_close<MODE, BLOCK, 8>; }
template <int MODE>
static CloseKernel close_kernel_block(uint32_t block, uint32_t sr) {
    return block == 256 ? close_kernel_rows<MODE, 256>(sr)
         : block == 128 ? close_kernel_rows<MODE, 128>(sr)
         : block == 64  ? close_kernel_rows<MODE, 64>(sr) : nullptr;
}
static CloseKernel close_kernel(int mode, uint32_t block, uint32_t sr) {
    return mode == kCloseStamps ? close_kernel_block<kCloseStamps>(block, sr)
         : mode == kCloseAt     ? close_kernel_block<kCloseAt>(block, sr)
                                : close_kernel_block<kCloseBits>(block, sr);
}

uint32_t close_blocks_per_cu(int mode, uint32_t block, uint32_t sr, uint32_t lds_bytes) {
    int n = 0;
    const CloseKernel k = close_kernel(mode, block, sr);
    const hipError_t e =
        k ? hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, reinterpret_cast<const void *>(k), (int)block, lds_bytes)
          : hipErrorInvalidValue;
    return (e == hipSuccess && n > 0) ? (uint32_t)n : 1u;
}

hipError_t launch_close(const Consts &c, const CloseArgs &a, int mode, uint32_t block, uint32_t grid, hipStream_t s) {
    const CloseKernel k = close_kernel(mode, block, c.sr);
    if (!k) return hipErrorInvalidConfiguration;
    const uint32_t lds = (block / 64) * close_wave_words(c.sea_bytes, a.qcap) * 4u;
    hipLaunchKernelGGL(k, dim3(grid), dim3(block), lds, s, c, a);
    return hipGetLastError();
}

hipError_t launch_close_many(const Consts &c, const CloseArgs &a, const CloseTable &t, uint32_t n, uint32_t block,
                             uint32_t grid, hipStream_t s) {
    if (n == 0 || n > (uint32_t)kMaxGroup) return hipErrorInvalidValue;
    const bool four = c.sr == 4;
    void (*k)(Consts, CloseArgs, CloseTable) = nullptr;
    if (block == 256) k = four ? k_close_many<256, 4> : k_close_many<256, 8>;
    else if (block == 128) k = four ? k_close_many<128, 4> : k_close_many<128, 8>;
    else if (block == 64) k = four ? k_close_many<64, 4> : k_close_many<64, 8>;
    else return hipErrorInvalidConfiguration;
    const uint32_t lds = (block / 64) * close_wave_words(c.sea_bytes, a.qcap) * 4u;
    hipLaunchKernelGGL(k, dim3(grid, n), dim3(block), lds, s, c, a, t);
    return hipGetLastError();
}

}  // namespace spd
