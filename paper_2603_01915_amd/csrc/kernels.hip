// HIP kernels for gfx950: SpMV / SpMM / transpose / decode fused with dtANS
// decoding of CSR-dtANS streams, the fix-up of rows split across lanes, the
// persistent multi-matrix launch and the plain-CSR baseline.
//
// Work mapping (Sec. II-B and IV-B of Schaetzle, Pegolotti, Pueschel, "Fast
// Entropy Decoding for Sparse MVM on GPUs", 2026, with 64-lane wavefronts):
// one wavefront decodes one encoded wave (64 lane streams) at a time.  Every
// lane holds the state of its own stream; the conditional and unconditional
// word loads of a step are coalesced by a 64-bit ballot and a lane prefix
// count (v_mbcnt), as the paper does with a warp ballot and two popcounts.
// Both coding tables live in LDS for the whole (persistent) workgroup.
//
// Workgroups are persistent (a few per CU); each wavefront takes a contiguous
// range of encoded waves, and workgroups are renumbered so that those running
// on the same XCD (dispatch is round-robin over the 8 XCDs) own neighbouring
// ranges, which keeps their x gathers in the same L2.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <mutex>
#include <type_traits>
#include <utility>
#include <vector>

#include "dtans_core.hpp"
#include "kernels.hpp"

namespace dtans {
namespace {

// How a lane holds a row: all of it; its end (the head: the row started in an
// earlier lane); its start (the tail: it continues in later lanes); or, in
// the nonzero layout, only a middle piece (started earlier, continues later).
constexpr int kComplete = 0, kHead = 1, kTail = 2, kMid = 3;
constexpr int kNumXcd = 8;
constexpr int kRingWords = 1024;  // per-wavefront LDS ring of the ring kernels (4 KiB)

__device__ __forceinline__ uint32_t lane_prefix(uint64_t mask) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32),
                                     __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

// A load from a wave-uniform address through the scalar unit (constant
// address space): the value lands in SGPRs.  Only for data no kernel of the
// library writes while it runs (the matrix's offsets).
template <typename T>
__device__ __forceinline__ T uniform_load(const T *p) {
    return *(const __attribute__((address_space(4))) T *)p;
}

// Pointers into global memory for the decoder's loads.  A pointer the kernel
// read from device memory (the per-matrix views of the multi-matrix launches)
// is generic to the compiler, which then reads through it with flat
// instructions: 64-bit addresses, and counted against the LDS wait counter
// too, so that every wait for a table lookup would also wait for the gathers
// and stream words in flight.  Loads through these pointers are global loads
// whatever the pointer's origin (every matrix and vector is a device
// allocation).
template <typename T>
using gptr = const __attribute__((address_space(1))) T *;
template <typename T>
using gmut = __attribute__((address_space(1))) T *;
// (the declared alignment is what the addresses guarantee: a load declared
// more aligned than its address lets the compiler draw wrong conclusions)
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));                // 16-byte aligned
typedef uint32_t u32x4_a8 __attribute__((ext_vector_type(4), aligned(8)));  // 16 bytes, 8-byte aligned
typedef uint64_t u64_a4 __attribute__((aligned(4)));                        // 8 bytes, 4-byte aligned
typedef uint32_t u32x4_a4 __attribute__((ext_vector_type(4), aligned(4)));  // 16 bytes, 4-byte aligned

template <typename VT> struct Bits;
template <> struct Bits<double> { typedef uint64_t T; };
template <> struct Bits<float> { typedef uint32_t T; };

template <typename VT>
__device__ __forceinline__ VT load_value(const void *p, uint64_t i) {
    return ((const VT *)p)[i];
}

// Value-table entry (device memory and LDS): the value's bits, then the slot's
// metadata b | d << 16 | escape << 31 (see dtans_core.hpp).  12 bytes for
// double: a value read is then two dword reads and the metadata a third, at
// 12 * slot, instead of a second table at another stride.
template <typename VT> struct VEntry;
template <> struct VEntry<double> {
    uint32_t lo, hi, meta;
    __device__ __forceinline__ double value() const {
        return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
    }
};
template <> struct VEntry<float> {
    uint32_t bits, meta;
    __device__ __forceinline__ float value() const { return __builtin_bit_cast(float, bits); }
};

// Both coding tables in LDS, the value table first so that every read of
// either has a constant offset below 2^16 (FP64: 48 + 32 KiB, FP32: 32 + 32).
template <typename VT> struct Tables {
    VEntry<VT> tv[kSlots];
    uint64_t td[kSlots];
};
static_assert(sizeof(VEntry<double>) == 12 && sizeof(VEntry<float>) == 8, "value entry sizes");
static_assert(sizeof(Tables<double>) == kSlots * 20 && sizeof(Tables<float>) == kSlots * 16,
              "tables are two packed arrays");

// ------------------------------------------------------------------ sinks
// A sink consumes one lane's decoded nonzeros a segment at a time:
//   segment<MULTI>(col, v, nreal, g, rowk): nonzeros k < nreal with columns
//     col[k] and values v[k]; nonzero k is number g + k in row-major order and
//     lies in row rowk[k].  MULTI is false when a lane holds a single row.
//     Every sink issues all its loads for the segment before it uses any.
//   finish_row(row, kind): row layout: the lane has seen its last nonzero of
//     `row`, which it holds whole.
//   finish_lane(row, kind, live): nonzero layout, called by every lane of the
//     wavefront together at the end of an encoded wave; `row` holds the live
//     lane's last nonzeros, `kind` how the lane holds it (kComplete, kHead,
//     kTail or kMid).
//   col_scale(params): the decoder multiplies every column delta by it, so
//     that col[k] arrives as column * col_scale modulo 2^32 (e.g. the byte
//     offset of x[column], which saves a shift per gather).
// Rows that end in the middle of a lane are finished inside segment().  Rows
// without nonzeros are a lane of their own in the row layout (finish_row with
// no segment) and never visited in the nonzero layout.

__device__ __forceinline__ uint64_t ballot(bool p) { return __builtin_amdgcn_ballot_w64(p); }

// y (k columns) = alpha * A x + beta * y.  UNIT: k = 1 with unit strides and
// n * sizeof(VT) <= 2^32.
// ACC: accumulator type.  double everywhere except FP32 SpMM with many
// columns in the nonzero-balanced layout, where a lane sums a bounded number
// of nonzeros (at most 1024; measured error ~1e-7 of |A||x| at 512) before
// its partial sums are combined in double.
// DEFER (KC <= 4): a segment's x values are loaded when it arrives and
// multiplied at the start of the next decoding step (or when the lane ends),
// so their latency overlaps one step.  1: lanes hold single rows; 2: lanes
// may cross rows, and the rows of the deferred nonzeros are kept with them.
// XLDS (single vectors): the kernel holds x in LDS (decode_x_kernel).
template <typename VT, int KC, bool UNIT, typename ACC = double, int DEFER = 0, bool XLDS = false>
struct SpmmSink {
    static constexpr bool kCoop = false;
    // paired x loads (see segment); the general-table decoder runs without them
    static constexpr bool kPairs = UNIT && KC == 1 && sizeof(VT) == 8 && !XLDS;
    static constexpr bool kPairs32 = UNIT && KC == 1 && sizeof(VT) == 4 && !XLDS;  // per-lane pairs
    static_assert(!XLDS || (UNIT && KC == 1 && !DEFER), "x in LDS: single vectors only");
    static_assert(!DEFER || KC <= 4, "deferred products keep 4*KC x values in registers");
    static constexpr int kOcc = KC <= 2 ? 8 : 4;  // waves per SIMD to allow
    struct Params {
        const VT *X;
        uint32_t ldx;
        VT *Y;
        uint32_t ldy;
        double *partial;  // [lane][head/tail][KC]
        double alpha, beta;
        // x holds at least two values, so that a read of two adjacent values
        // starting at column 0 stays inside it (the FP64 short segments and
        // the FP32 per-lane pairs in segment); 0 turns those reads off
        uint32_t pair_x = 0;
        const VT *lx = nullptr;  // XLDS: x in LDS, set by the kernel
    };
    const Params p;
    uint32_t lane;
    int32_t cur, head_row;  // row being accumulated; the lane's head row or -1
    ACC acc[KC];
    VT pv[DEFER ? 4 : 1], px[DEFER ? 4 : 1][KC];  // deferred segment
    int32_t prow[DEFER == 2 ? 4 : 1];             // its rows (DEFER 2)
    int pn;                                       // its nonzeros (0: none)
    // cur starts at the lane's first row, which holds its first nonzero
    __device__ SpmmSink(const Params &pp, int64_t l, int32_t first_row, bool first_is_head)
        : p(pp), lane((uint32_t)l), cur(first_row), head_row(first_is_head ? first_row : -1), pn(0) {
#pragma unroll
        for (int c = 0; c < KC; ++c) acc[c] = (ACC)0;
    }
    // multiply the deferred segment (its x loads were issued a step ago)
    __device__ __forceinline__ void consume() {
        if constexpr (DEFER == 1) {
            if (!ballot(pn < 4)) {
#pragma unroll
                for (int k = 0; k < 4; ++k)
#pragma unroll
                    for (int c = 0; c < KC; ++c) acc[c] = fma((ACC)pv[k], (ACC)px[k][c], acc[c]);
            } else {
#pragma unroll
                for (int k = 0; k < 4; ++k)
#pragma unroll
                    for (int c = 0; c < KC; ++c) {
                        const ACC t = fma((ACC)pv[k], (ACC)px[k][c], acc[c]);
                        acc[c] = k < pn ? t : acc[c];
                    }
            }
            pn = 0;
        } else if constexpr (DEFER == 2) {
            // rows never decrease along a lane: prow[3] == cur means no row ends
            if (!ballot(pn < 4 || prow[3] != cur)) {
#pragma unroll
                for (int k = 0; k < 4; ++k)
#pragma unroll
                    for (int c = 0; c < KC; ++c) acc[c] = fma((ACC)pv[k], (ACC)px[k][c], acc[c]);
            } else {
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    if (k < pn) {
                        if (prow[k] != cur) {
                            store(cur, cur == head_row ? kHead : kComplete);
                            cur = prow[k];
                        }
#pragma unroll
                        for (int c = 0; c < KC; ++c) acc[c] = fma((ACC)pv[k], (ACC)px[k][c], acc[c]);
                    }
            }
            pn = 0;
        }
    }
    // called once per decoding step before the step issues any loads
    __device__ __forceinline__ void pre_step() { consume(); }
    // UNIT: x spans at most 4 GiB, so columns arrive as 32-bit byte offsets
    // from the uniform base (the decoder scales the deltas; base in SGPRs)
    static __device__ __forceinline__ uint32_t col_scale(const Params &) {
        return UNIT ? (uint32_t)sizeof(VT) : 1u;
    }
    __device__ __forceinline__ auto xrow(uint32_t col) const {
        if constexpr (XLDS) return (const VT *)((const char *)p.lx + col);
        else return UNIT ? (gptr<VT>)((const char *)p.X + col) : (gptr<VT>)(p.X + (uint64_t)col * p.ldx);
    }
    __device__ __forceinline__ void store(int32_t row, int kind) {
        if (kind == kComplete) {
            const gmut<VT> y = (gmut<VT>)(UNIT ? p.Y + row : p.Y + (uint64_t)(uint32_t)row * p.ldy);
#pragma unroll
            for (int c = 0; c < KC; ++c)
                y[c] = (VT)(p.beta == 0.0 ? p.alpha * (double)acc[c]
                                          : p.alpha * (double)acc[c] + p.beta * (double)y[c]);
        } else {
            double *q = p.partial + (2 * (int64_t)lane + (kind == kTail ? 1 : 0)) * KC;
#pragma unroll
            for (int c = 0; c < KC; ++c) q[c] = (double)acc[c];
        }
#pragma unroll
        for (int c = 0; c < KC; ++c) acc[c] = (ACC)0;
    }
    template <bool MULTI, bool PAIRS = kPairs>
    __device__ __forceinline__ void segment(const uint32_t col[4], const VT v[4], int nreal,
                                            int64_t, const int32_t rowk[4]) {
        if constexpr (DEFER) {
            static_assert(MULTI == (DEFER == 2), "DEFER 1 is for single-row lanes, 2 for the others");
            {
                // every lane loads four x values (column 0 stands in for
                // nonzeros past the lane's end; their products are dropped)
                uint32_t cc[4];
#pragma unroll
                for (int k = 0; k < 4; ++k) cc[k] = col[k];
                if (ballot(nreal < 4)) {
#pragma unroll
                    for (int k = 0; k < 4; ++k) cc[k] = k < nreal ? col[k] : 0u;
                }
#pragma unroll
                for (int k = 0; k < 4; ++k)
#pragma unroll
                    for (int c = 0; c < KC; ++c) px[k][c] = xrow(cc[k])[c];
#pragma unroll
                for (int k = 0; k < 4; ++k) pv[k] = v[k];
                if constexpr (DEFER == 2) {
#pragma unroll
                    for (int k = 0; k < 4; ++k) prow[k] = rowk[k];
                }
                pn = nreal;
                return;
            }
        }
        if (KC * sizeof(VT) <= 32) {  // all four rows of X in flight at once
            VT x[4][KC];
            // common case, taken by the whole wavefront or not at all (a
            // uniform branch): no lane has a tail or a row end here
            if (!ballot(!(nreal >= 4 && (!MULTI || rowk[3] == cur)))) {
                if constexpr (PAIRS) {
                    // FP64 vector: when nonzeros k and k+1 of every lane are
                    // adjacent columns (uniform tests), one 16-byte load gives
                    // both x values.  The address unit takes such a load of a
                    // wavefront in the cycles of one 8-byte load (stencil and
                    // banded rows have runs of adjacent columns).
#pragma unroll
                    for (int k = 0; k < 4; k += 2) {
                        if (!ballot(col[k + 1] != col[k] + 8u)) {
                            // (an offset the compiler cannot share with the
                            // other branch: a shared address would be formed
                            // as a 64-bit pointer ahead of the branch, where
                            // this form keeps the base in SGPRs)
                            uint32_t o = col[k];
                            asm("" : "+v"(o));
                            const u32x4_a8 q = *(gptr<u32x4_a8>)((const char *)p.X + o);
                            x[k][0] = __builtin_bit_cast(VT, (uint64_t)q.y << 32 | q.x);
                            x[k + 1][0] = __builtin_bit_cast(VT, (uint64_t)q.w << 32 | q.z);
                        } else {
                            x[k][0] = xrow(col[k])[0];
                            x[k + 1][0] = xrow(col[k + 1])[0];
                        }
                    }
                } else if constexpr (kPairs32) {
                    // FP32 vector, pairs per lane: an 8-byte load ending at
                    // column k+1 gives x at k+1 and, in the lanes whose
                    // columns k and k+1 are adjacent, x at k too; only the
                    // other lanes load x at k on their own, so the address
                    // unit sees their cache lines only (half the lanes of a
                    // weight pruned to half its entries).  The load starts at
                    // column 0 when column k+1 is 0 (repeated columns), so it
                    // stays inside x once x holds two values.
                    // (every load is issued before any value is selected,
                    // so that no wait comes between them)
                    if (p.pair_x) {  // uniform
                        uint64_t q[2];
                        VT xs[2];
#pragma unroll
                        for (int h = 0; h < 2; ++h) {
                            const uint32_t c1 = col[2 * h + 1];
                            q[h] = *(gptr<u64_a4>)((const char *)p.X + (c1 >= 4u ? c1 - 4u : 0u));
                        }
#pragma unroll
                        for (int h = 0; h < 2; ++h) {
                            xs[h] = (VT)0;
                            if (col[2 * h] + 4u != col[2 * h + 1]) xs[h] = xrow(col[2 * h])[0];
                        }
#pragma unroll
                        for (int h = 0; h < 2; ++h) {
                            const uint32_t c1 = col[2 * h + 1];
                            const VT lo = __builtin_bit_cast(VT, (uint32_t)q[h]);
                            const VT hi = __builtin_bit_cast(VT, (uint32_t)(q[h] >> 32));
                            x[2 * h + 1][0] = c1 >= 4u ? hi : lo;
                            x[2 * h][0] = col[2 * h] + 4u == c1 ? lo : xs[h];
                        }
                    } else {
#pragma unroll
                        for (int k = 0; k < 4; ++k) x[k][0] = xrow(col[k])[0];
                    }
                } else {
#pragma unroll
                    for (int k = 0; k < 4; ++k)
#pragma unroll
                        for (int c = 0; c < KC; ++c) x[k][c] = xrow(col[k])[c];
                }
#pragma unroll
                for (int k = 0; k < 4; ++k)
#pragma unroll
                    for (int c = 0; c < KC; ++c) acc[c] = fma((ACC)v[k], (ACC)x[k][c], acc[c]);
                return;
            }
            if constexpr (!MULTI) {
                // single-row lanes: only a lane's last segment is short (or it
                // has none left); column 0 stands in for the missing nonzeros,
                // whose products are dropped by a select, with no branches
                if constexpr (PAIRS) {
                    // Pairs as in the common case when both pairs of every
                    // lane holding them are adjacent (a uniform test) and x
                    // holds at least two values.  A lane holding both
                    // nonzeros of a pair reads them at the first column; a
                    // lane holding only the first reads the 16 bytes that end
                    // at its column (or start at column 0), a lane holding
                    // neither reads columns 0 and 1: every read stays inside
                    // x.
                    if (p.pair_x && !ballot((1 < nreal && col[1] != col[0] + 8u) ||
                                            (3 < nreal && col[3] != col[2] + 8u))) {
                        bool up[2];
                        u32x4_a8 q[2];
#pragma unroll
                        for (int h = 0; h < 2; ++h) {
                            const int k = 2 * h;
                            const bool one = k < nreal, both = k + 1 < nreal;
                            up[h] = one && !both && col[k] != 0u;
                            const uint32_t off = both ? col[k] : (up[h] ? col[k] - 8u : 0u);
                            q[h] = *(gptr<u32x4_a8>)((const char *)p.X + off);
                        }
#pragma unroll
                        for (int h = 0; h < 2; ++h) {
                            const VT lo = __builtin_bit_cast(VT, (uint64_t)q[h].y << 32 | q[h].x);
                            const VT hi = __builtin_bit_cast(VT, (uint64_t)q[h].w << 32 | q[h].z);
                            x[2 * h][0] = up[h] ? hi : lo;
                            x[2 * h + 1][0] = hi;
                        }
#pragma unroll
                        for (int k = 0; k < 4; ++k) {
                            const ACC t = fma((ACC)v[k], (ACC)x[k][0], acc[0]);
                            acc[0] = k < nreal ? t : acc[0];
                        }
                        return;
                    }
                }
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const uint32_t cc = k < nreal ? col[k] : 0u;
#pragma unroll
                    for (int c = 0; c < KC; ++c) x[k][c] = xrow(cc)[c];
                }
#pragma unroll
                for (int k = 0; k < 4; ++k)
#pragma unroll
                    for (int c = 0; c < KC; ++c) {
                        const ACC t = fma((ACC)v[k], (ACC)x[k][c], acc[c]);
                        acc[c] = k < nreal ? t : acc[c];
                    }
                return;
            }
            // (every lane loads, column 0 past its end: the loads stay
            // together, with no branch between them)
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const uint32_t cc = k < nreal ? col[k] : 0u;
#pragma unroll
                for (int c = 0; c < KC; ++c) x[k][c] = xrow(cc)[c];
            }
#pragma unroll
            for (int k = 0; k < 4; ++k)
                if (k < nreal) {
                    if (MULTI && rowk[k] != cur) {
                        store(cur, cur == head_row ? kHead : kComplete);
                        cur = rowk[k];
                    }
#pragma unroll
                    for (int c = 0; c < KC; ++c) acc[c] = fma((ACC)v[k], (ACC)x[k][c], acc[c]);
                }
        } else {
            // wider rows of X: load nonzero k+1 while multiplying nonzero k
            VT xa[KC], xb[KC];
            if (nreal > 0) {
#pragma unroll
                for (int c = 0; c < KC; ++c) xa[c] = xrow(col[0])[c];
            }
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                VT *xc = (k & 1) ? xb : xa;
                VT *xn = (k & 1) ? xa : xb;
                if (k + 1 < 4 && k + 1 < nreal) {
#pragma unroll
                    for (int c = 0; c < KC; ++c) xn[c] = xrow(col[k + 1])[c];
                }
                if (k < nreal) {
                    if (MULTI && rowk[k] != cur) {
                        store(cur, cur == head_row ? kHead : kComplete);
                        cur = rowk[k];
                    }
#pragma unroll
                    for (int c = 0; c < KC; ++c) acc[c] = fma((ACC)v[k], (ACC)xc[c], acc[c]);
                }
            }
        }
    }
    __device__ __forceinline__ void finish_row(int32_t row, int kind) {
        consume();
        store(row, kind);
    }
    // Middle pieces of a row are summed across the wavefront first: a
    // segmented suffix sum over consecutive lanes holding middles of the same
    // row (rows never decrease along the lanes, so equal rows d lanes apart
    // mean the whole stretch holds that row), after which only the first
    // such lane of each stretch stores (its head slot).  The fix-up then reads
    // one partial per wavefront a row spans instead of one per lane.
    __device__ __forceinline__ void finish_lane(int32_t row, int kind, bool live) {
        consume();
        const uint32_t wl = lane & (kWave - 1);
        const bool mid = live && kind == kMid;
        const int32_t key = mid ? row : -1;
#pragma unroll
        for (int d = 1; d < kWave; d <<= 1) {
            const int32_t kd = __shfl_down(key, d);
            const bool ok = mid && wl + d < (uint32_t)kWave && kd == key;
#pragma unroll
            for (int c = 0; c < KC; ++c) {
                const ACC t = __shfl_down(acc[c], d);
                if (ok) acc[c] += t;
            }
        }
        const int32_t kp = __shfl_up(key, 1);
        if (mid) {
            if (wl == 0 || kp != key) store(row, kHead);
        } else if (live) {
            store(row, kind);
        }
    }
};

// Orders a wavefront's LDS accesses before and after it as its other lanes see
// them.  The hardware keeps a wavefront's LDS operations in order; this holds
// the compiler to it (no instruction of its own).
__device__ __forceinline__ void wave_exchange_fence() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// A 32-bit value of lane `src` (all lanes of the wavefront active)
__device__ __forceinline__ uint32_t lane_value(uint32_t v, uint32_t src) {
    return (uint32_t)__builtin_amdgcn_ds_bpermute((int)(src << 2), (int)v);
}
template <typename T>
__device__ __forceinline__ T lane_value_of(T v, uint32_t src) {
    if constexpr (sizeof(T) == 8) {
        const uint64_t b = __builtin_bit_cast(uint64_t, v);
        const uint64_t r = (uint64_t)lane_value((uint32_t)b, src) |
                           ((uint64_t)lane_value((uint32_t)(b >> 32), src) << 32);
        return __builtin_bit_cast(T, r);
    } else {
        return __builtin_bit_cast(T, lane_value(__builtin_bit_cast(uint32_t, v), src));
    }
}

// Y (KC = G * CL columns) = alpha * A X + beta * Y with G lanes per row of X.
// The 64 lanes of a wavefront form 64 / G groups; group q keeps, in G slots,
// the sums of the streams q*G .. q*G + G - 1 (slot i: stream q*G + i), each
// lane for CL = 16 / sizeof(VT) consecutive columns (one 16-byte load per
// nonzero).  A step's (column, value) pairs move from the decoding lane to
// its group with ds_bpermute, so that one load instruction reads 64 / G whole
// rows of X (the address unit takes one cache line of an instruction at a
// time: rows read one per lane cost a line per lane).  Columns arrive as byte
// offsets of rows of X (col_scale = ldx * sizeof(VT)); X and Y rows are
// 16-byte aligned.  Rows split over lanes give the same partial sums as
// SpmmSink (tail and head slots; the middle pieces of a row summed per
// wavefront into the head slot of the stretch's first stream), so the same
// fix-up finishes them.
//
// STRAIGHT: a full step of a wavefront whose streams all stay in their rows
// runs without masks, one straight run of loads and products (pruned 11008 x
// 4096 weight, FP32, k = 32: 172 -> 163 us).  Its registers spill beside those
// of the general step, which the straight one then has to make up for: it is a
// variant for long rows (see spmm_impl).
template <typename VT, int G, typename ACC = double, bool STRAIGHT = false>
struct CoopSpmmSink {
    static constexpr bool kCoop = true;
    static constexpr bool kPairs = false;
    static constexpr int CL = 16 / (int)sizeof(VT), KC = G * CL, NG = kWave / G;
    // waves per SIMD to allow: with eight slots per lane the accumulators and
    // the rows of X in flight do not fit beside the decoder in 128 registers;
    // with two or four, 168 registers avoid spills (measured faster than four
    // waves per SIMD with spills, and than two)
    static constexpr int kOcc = G >= 8 ? 2 : 3;
    static_assert(G == 2 || G == 4 || G == 8, "2, 4 or 8 lanes per row of X");
    struct Params {
        const VT *X;
        uint32_t ldx;
        VT *Y;
        uint32_t ldy;
        double *partial;  // [lane][head/tail][KC]
        double alpha, beta;
    };
    const Params p;
    uint32_t grp, part;      // group, column chunk of this lane
    int64_t wave0;           // global index of stream 0 of the wave
    ACC acc[G][CL];
    int32_t cur[G];          // row being summed in slot i (at first the stream's first row)
    int32_t head_row[G];     // the slot's first row when it began before the stream, else -1
    int32_t last;            // row of this lane's last nonzero so far (at first its first row)

    static __device__ __forceinline__ uint32_t col_scale(const Params &pp) {
        return pp.ldx * (uint32_t)sizeof(VT);
    }
    __device__ CoopSpmmSink(const Params &pp, int64_t l, int32_t first_row, bool first_is_head) : p(pp) {
        const uint32_t lane = (uint32_t)l & (kWave - 1);
        grp = lane / G;
        part = lane % G;
        wave0 = l - lane;
        last = first_row;
        const int32_t hr = first_is_head ? first_row : -1;
#pragma unroll
        for (int i = 0; i < G; ++i) {
            const uint32_t src = grp * G + i;
            cur[i] = (int32_t)lane_value((uint32_t)first_row, src);
            head_row[i] = (int32_t)lane_value((uint32_t)hr, src);
#pragma unroll
            for (int c = 0; c < CL; ++c) acc[i][c] = (ACC)0;
        }
    }
    __device__ __forceinline__ void pre_step() {}
    __device__ __forceinline__ VT *yrow(int32_t row) const {
        return p.Y + (uint64_t)(uint32_t)row * p.ldy + part * CL;
    }
    __device__ __forceinline__ double *slot(int64_t stream, int kind) const {
        return p.partial + (2 * stream + (kind == kTail ? 1 : 0)) * KC + part * CL;
    }
    // store slot i's sums for `row` (kind as for SpmmSink::store) and clear them
    __device__ __forceinline__ void store(int i, int32_t row, int kind) {
        if (kind == kComplete) {
            VT *y = yrow(row);
#pragma unroll
            for (int c = 0; c < CL; ++c)
                y[c] = (VT)(p.beta == 0.0 ? p.alpha * (double)acc[i][c]
                                          : p.alpha * (double)acc[i][c] + p.beta * (double)y[c]);
        } else {
            double *q = slot(wave0 + grp * G + i, kind);
#pragma unroll
            for (int c = 0; c < CL; ++c) q[c] = (double)acc[i][c];
        }
#pragma unroll
        for (int c = 0; c < CL; ++c) acc[i][c] = (ACC)0;
    }
    template <bool MULTI>
    __device__ __forceinline__ void segment(const uint32_t col[4], const VT v[4], int nreal, int64_t,
                                            const int32_t rowk[4]) {
        // some stream reaches a row it did not end the last step in (a
        // uniform test); otherwise the slots' rows stay as they are
        const bool moved = MULTI && ballot(nreal > 0 && rowk[nreal - 1] != last) != 0;
        if (MULTI && nreal > 0) last = rowk[nreal - 1];
        if (STRAIGHT && !ballot(nreal < 4) && !moved) {  // uniform
            constexpr int R = 4 * G;
            u32x4 xs[2];
            VT vv[2];
            auto get = [&](int r) {
                const uint32_t src = grp * G + (r >> 2);
                vv[r & 1] = lane_value_of(v[r & 3], src);
                xs[r & 1] = *(gptr<u32x4>)((const char *)p.X + (lane_value(col[r & 3], src) + part * 16));
            };
            get(0);
            get(1);
#pragma unroll
            for (int r = 0; r < R; ++r) {
                VT x[CL];
                __builtin_memcpy(x, &xs[r & 1], 16);
                const ACC vr = (ACC)vv[r & 1];
                if (r + 2 < R) get(r + 2);
#pragma unroll
                for (int c = 0; c < CL; ++c) acc[r >> 2][c] = fma(vr, (ACC)x[c], acc[r >> 2][c]);
            }
            return;
        }
        int nr[G];
#pragma unroll
        for (int i = 0; i < G; ++i) nr[i] = (int)lane_value((uint32_t)nreal, grp * G + i);
        // rounds r = 4 i + j (nonzero j of slot i's stream), each row of X
        // requested kAhead rounds before it is multiplied
        constexpr int R = 4 * G, kAhead = 2;
        uint4 xs[kAhead];
        VT vv[kAhead];
        int32_t rk[kAhead];
        auto fetch = [&](int r) {
            const int b = r % kAhead, i = r >> 2, j = r & 3;
            const uint32_t src = grp * G + i;
            const uint32_t cj = lane_value(col[j], src);
            vv[b] = lane_value_of(v[j], src);
            if (MULTI && moved) rk[b] = (int32_t)lane_value((uint32_t)rowk[j], src);
            // nonzeros past a stream's end read row 0 of X (their products are dropped)
            xs[b] = *(const uint4 *)((const char *)p.X + (j < nr[i] ? cj : 0u) + part * 16);
        };
#pragma unroll
        for (int r = 0; r < kAhead && r < R; ++r) fetch(r);
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int b = r % kAhead, i = r >> 2, j = r & 3;
            VT x[CL];
            __builtin_memcpy(x, &xs[b], 16);
            const VT vr = vv[b];
            const int32_t rr = (MULTI && moved) ? rk[b] : 0;
            if (r + kAhead < R) fetch(r + kAhead);
            if (j < nr[i]) {
                if (MULTI && moved && rr != cur[i]) {
                    store(i, cur[i], cur[i] == head_row[i] ? kHead : kComplete);
                    cur[i] = rr;
                }
#pragma unroll
                for (int c = 0; c < CL; ++c) acc[i][c] = fma((ACC)vr, (ACC)x[c], acc[i][c]);
            }
        }
    }
    // single-row streams (row layout): every lane calls this at the end of the
    // wave; `live` lanes' rows are complete
    __device__ __forceinline__ void finish_row(int32_t row, int kind) { finish_all(row, kind, true); }
    __device__ __forceinline__ void finish_lane(int32_t row, int kind, bool live) { finish_all(row, kind, live); }

    __device__ __forceinline__ void finish_all(int32_t row, int kind, bool live) {
        int32_t rw[G], key[G];
        int kd[G];
#pragma unroll
        for (int i = 0; i < G; ++i) {
            const uint32_t src = grp * G + i;
            rw[i] = (int32_t)lane_value((uint32_t)row, src);
            kd[i] = (int)lane_value((uint32_t)(live ? kind : -1), src);
            key[i] = kd[i] == kMid ? rw[i] : -1;
        }
        // non-middle pieces: complete rows to Y, heads and tails to their slots
#pragma unroll
        for (int i = 0; i < G; ++i)
            if (kd[i] >= 0 && kd[i] != kMid) store(i, rw[i], kd[i]);
        // middle pieces: suffix sums over the wave's streams in order (slots
        // of a group, then groups), keyed by row (rows never decrease along
        // the streams, so equal keys far apart mean the whole stretch holds
        // that row); the first stream of each stretch stores the total
#pragma unroll
        for (int i = G - 2; i >= 0; --i)
            if (key[i] >= 0 && key[i + 1] == key[i]) {
#pragma unroll
                for (int c = 0; c < CL; ++c) acc[i][c] += acc[i + 1][c];
            }
        const int32_t k0 = key[0];
        const int32_t kn = (int32_t)lane_value((uint32_t)k0, ((grp + 1) % NG) * G + part);
        const int32_t kprev = (int32_t)lane_value((uint32_t)key[G - 1], ((grp + NG - 1) % NG) * G + part);
        bool kok[6];  // the cross-group steps that join equal keys
#pragma unroll
        for (int t = 0, d = 1; d < NG; d <<= 1, ++t) {
            const int32_t kdn = (int32_t)lane_value((uint32_t)k0, ((grp + d) % NG) * G + part);
            kok[t] = k0 >= 0 && grp + d < (uint32_t)NG && kdn == k0;
        }
#pragma unroll
        for (int c = 0; c < CL; ++c) {
            ACC V = acc[0][c];
#pragma unroll
            for (int t = 0, d = 1; d < NG; d <<= 1, ++t) {
                const ACC u = lane_value_of(V, ((grp + d) % NG) * G + part);
                if (kok[t]) V += u;
            }
            // the next group's slot-0 total
            const ACC Vn = lane_value_of(V, ((grp + 1) % NG) * G + part);
#pragma unroll
            for (int i = 0; i < G; ++i) {
                if (key[i] < 0) continue;
                const bool first = i > 0 ? key[i - 1] != key[i] : (grp == 0 || kprev != key[i]);
                if (!first) continue;
                const bool more = key[G - 1] == key[i] && grp + 1 < (uint32_t)NG && kn == key[i];
                const ACC tot = i == 0 ? V : acc[i][c] + (more ? Vn : (ACC)0);
                slot(wave0 + grp * G + i, kHead)[c] = (double)tot;
            }
        }
    }
};

// dX (k columns) += alpha * A^T dY, scattered with atomic adds.
template <typename VT, int KC>
struct TransSink {
    static constexpr bool kCoop = false;
    static constexpr bool kPairs = false;
    static constexpr int kOcc = KC <= 2 ? 8 : 4;
    struct Params {
        const VT *dY;
        uint32_t lddy;
        VT *dX;
        uint32_t lddx;
        double alpha;
    };
    const Params p;
    int32_t cur;
    VT dy[KC];
    static __device__ __forceinline__ uint32_t col_scale(const Params &) { return 1u; }
    __device__ TransSink(const Params &pp, int64_t, int32_t first_row, bool) : p(pp), cur(-1) {
        (void)first_row;
    }
    __device__ __forceinline__ void load_row(int32_t row) {
        cur = row;
        const VT *src = p.dY + (uint64_t)(uint32_t)row * p.lddy;
#pragma unroll
        for (int c = 0; c < KC; ++c) dy[c] = (VT)(p.alpha * (double)src[c]);
    }
    template <bool MULTI>
    __device__ __forceinline__ void segment(const uint32_t col[4], const VT v[4], int nreal,
                                            int64_t, const int32_t rowk[4]) {
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (k < nreal) {
                if (rowk[k] != cur) load_row(rowk[k]);
                VT *dst = p.dX + (uint64_t)col[k] * p.lddx;
#pragma unroll
                for (int c = 0; c < KC; ++c) unsafeAtomicAdd(dst + c, v[k] * dy[c]);
            }
    }
    __device__ __forceinline__ void pre_step() {}
    __device__ __forceinline__ void finish_row(int32_t, int) {}
    __device__ __forceinline__ void finish_lane(int32_t, int, bool) {}
};

// Position of column i in a plane of the LDS block of dX: a permutation within
// every 32 columns that differs from one 32 to the next, so that lanes whose
// columns lie a multiple of 32 apart (equal lane lengths over a regular row
// walk exactly such strides) do not all hit one LDS bank pair.  Planes are
// padded to a multiple of 32 columns.
__device__ __forceinline__ uint32_t lds_slot(uint32_t i) { return i ^ ((i >> 5) & 31u); }

// dX[c0 .. c0 + cols) += A^T dY for up to KC columns of dY into a block of dX
// in LDS (trans_lds_kernel); alpha is applied when the copies are summed.
// The block is FP64 for either value type: what bounds the scatter is the
// rate of LDS atomic adds, measured at 0.33 lane operations per clock and CU
// for ds_add_f32 whatever the addresses, 2.9 (random addresses) to 6.4 (unit
// stride) for ds_add_f64.
template <typename VT, int KC>
struct TransLdsSink {
    static constexpr bool kCoop = false;
    static constexpr bool kPairs = false;
    static constexpr int kOcc = 4;
    struct Params {
        const VT *dY;     // the first column of this pass
        uint32_t lddy;
        uint32_t width;   // columns of dY in this pass, at most KC
        uint32_t c0, cols;  // columns of A (rows of dX) of this pass
        uint32_t plane;   // elements of one column's plane in the block
        double *lds;      // width planes, set by the kernel
    };
    const Params p;
    int32_t cur;
    double dy[KC];
    static __device__ __forceinline__ uint32_t col_scale(const Params &) { return 1u; }
    __device__ TransLdsSink(const Params &pp, int64_t, int32_t, bool) : p(pp), cur(-1) {}
    __device__ __forceinline__ void load_row(int32_t row) {
        cur = row;
        const VT *src = p.dY + (uint64_t)(uint32_t)row * p.lddy;
#pragma unroll
        for (int c = 0; c < KC; ++c)
            if (c < (int)p.width) dy[c] = (double)src[c];  // uniform test
    }
    __device__ __forceinline__ void add(uint32_t col, VT v) {
        const uint32_t i = col - p.c0;
        if (i < p.cols) {
            double *dst = p.lds + lds_slot(i);
#pragma unroll
            for (int c = 0; c < KC; ++c)
                if (c < (int)p.width) unsafeAtomicAdd(dst + c * p.plane, (double)v * dy[c]);
        }
    }
    template <bool MULTI>
    __device__ __forceinline__ void segment(const uint32_t col[4], const VT v[4], int nreal,
                                            int64_t, const int32_t rowk[4]) {
        // common case of the whole wavefront: four nonzeros of the row at hand
        if (!ballot(nreal < 4 || rowk[3] != cur)) {
#pragma unroll
            for (int k = 0; k < 4; ++k) add(col[k], v[k]);
            return;
        }
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (k < nreal) {
                if (rowk[k] != cur) load_row(rowk[k]);
                add(col[k], v[k]);
            }
    }
    __device__ __forceinline__ void pre_step() {}
    __device__ __forceinline__ void finish_row(int32_t, int) {}
    __device__ __forceinline__ void finish_lane(int32_t, int, bool) {}
};

// A workgroup's sums for some of y, in LDS: 64 sets of 2 blocks, a block being
// 64 consecutive elements (block b of y lives in set b mod 64).  A block is
// claimed by the first element added to it; when both blocks of a set are
// taken, elements go to y itself.  FP64 for either value type (the LDS adds
// them nine times as fast as FP32, see TransLdsSink).
struct BlockSums {
    static constexpr uint32_t kSets = 64, kWays = 2, kBlock = 64, kFree = ~0u;
    static constexpr size_t kBytes = kSets * kWays * (kBlock * sizeof(double) + sizeof(uint32_t));
    double *sum;      // kSets * kWays * kBlock
    uint32_t *owner;  // kSets * kWays: block numbers or kFree
    __device__ __forceinline__ BlockSums(void *lds)
        : sum((double *)lds), owner((uint32_t *)(sum + kSets * kWays * kBlock)) {}
    // by the whole workgroup; a barrier has to follow
    __device__ __forceinline__ void clear() const {
        for (uint32_t i = threadIdx.x; i < kSets * kWays * kBlock; i += blockDim.x) sum[i] = 0.0;
        for (uint32_t i = threadIdx.x; i < kSets * kWays; i += blockDim.x) owner[i] = kFree;
    }
    // the sum of element i, or null
    __device__ __forceinline__ double *find(uint32_t i) const {
        const uint32_t b = i / kBlock, set = b % kSets;
        const uint2 t = *(const uint2 *)(owner + set * kWays);
        int way = t.x == b ? 0 : (t.y == b ? 1 : -1);
        if (way < 0) {
            if (t.x == kFree) {
                const uint32_t o = atomicCAS(owner + set * kWays, kFree, b);
                if (o == kFree || o == b) way = 0;
            }
            if (way < 0 && t.y == kFree) {
                const uint32_t o = atomicCAS(owner + set * kWays + 1, kFree, b);
                if (o == kFree || o == b) way = 1;
            }
        }
        return way < 0 ? nullptr : sum + (set * kWays + way) * kBlock + i % kBlock;
    }
    // y += alpha * sums; frees every block.  By the whole workgroup, between
    // barriers.  (A sum of zero adds nothing.)
    __device__ __forceinline__ void flush(double *y, double alpha) const {
        const uint32_t lane = threadIdx.x & (kWave - 1), nw = blockDim.x / kWave;
        for (uint32_t s = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave); s < kSets * kWays; s += nw) {
            const uint32_t b = owner[s];
            if (b == kFree) continue;
            const double v = sum[s * kBlock + lane];
            if (v != 0.0) {
                sum[s * kBlock + lane] = 0.0;
                unsafeAtomicAdd(y + (uint64_t)b * kBlock + lane, alpha * v);
            }
            if (lane == 0) owner[s] = kFree;
        }
    }
};

// y += alpha (S + S^T) x in one decode of S (the strict triangle of a
// symmetric matrix): a nonzero (r, c, v) adds v x[c] to the sum of row r and
// v x[r] to y[c], both through BlockSums.  Pieces of a row in several lanes
// just add to the same element.  y is FP64 for either value type: each flush
// and each element without a block is an addition of its own, which in FP32
// would round y once for each of them (random matrices of order 4000 to 20000:
// error 1.4e-7 of |y|, 3.9e-8 with one rounding at the end).
template <typename VT>
struct SymSink {
    static constexpr bool kCoop = false;
    static constexpr bool kPairs = false;
    static constexpr int kOcc = 4;
    struct Params {
        const VT *x;
        double *y;
        double alpha;
        void *lds;  // set by the kernel
    };
    const Params p;
    int32_t cur;  // row of acc (-1: none yet)
    double xr, acc;
    static __device__ __forceinline__ uint32_t col_scale(const Params &) { return 1u; }
    __device__ SymSink(const Params &pp, int64_t, int32_t, bool) : p(pp), cur(-1), xr(0.0), acc(0.0) {}
    __device__ __forceinline__ void add(uint32_t i, double v) const {
        double *q = BlockSums(p.lds).find(i);
        if (q) unsafeAtomicAdd(q, v);
        else unsafeAtomicAdd(p.y + i, p.alpha * v);
    }
    __device__ __forceinline__ void to_row(int32_t row) {
        if (cur >= 0) add((uint32_t)cur, acc);
        cur = row;
        xr = (double)((gptr<VT>)p.x)[(uint32_t)row];
        acc = 0.0;
    }
    template <bool MULTI>
    __device__ __forceinline__ void segment(const uint32_t col[4], const VT v[4], int nreal, int64_t,
                                            const int32_t rowk[4]) {
        VT x[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) x[k] = ((gptr<VT>)p.x)[k < nreal ? col[k] : 0u];
        if (!MULTI && nreal > 0 && cur < 0) to_row(rowk[0]);
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (k < nreal) {
                if (MULTI && rowk[k] != cur) to_row(rowk[k]);
                add(col[k], (double)v[k] * xr);
                acc = fma((double)v[k], (double)x[k], acc);
            }
    }
    __device__ __forceinline__ void pre_step() {}
    __device__ __forceinline__ void finish_row(int32_t, int) {
        if (cur >= 0) add((uint32_t)cur, acc);
    }
    __device__ __forceinline__ void finish_lane(int32_t, int, bool) {
        if (cur >= 0) add((uint32_t)cur, acc);
    }
};

// decode to CSR: column and value bits of every nonzero in one walk (see
// decode_impl; most matrices take decode_slice_csr)
template <typename VT>
struct DecodeSink {
    static constexpr bool kCoop = false;
    static constexpr bool kPairs = false;
    static constexpr int kOcc = 8;
    struct Params {
        int32_t *col;
        typename Bits<VT>::T *vals;
    };
    const Params p;
    static __device__ __forceinline__ uint32_t col_scale(const Params &) { return 1u; }
    __device__ DecodeSink(const Params &pp, int64_t, int32_t, bool) : p(pp) {}
    template <bool MULTI>
    __device__ __forceinline__ void segment(const uint32_t col[4], const VT v[4], int nreal,
                                            int64_t g, const int32_t *) {
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (k < nreal) {
                p.col[g + k] = (int32_t)col[k];
                p.vals[g + k] = __builtin_bit_cast(typename Bits<VT>::T, v[k]);
            }
    }
    __device__ __forceinline__ void pre_step() {}
    __device__ __forceinline__ void finish_row(int32_t, int) {}
    __device__ __forceinline__ void finish_lane(int32_t, int, bool) {}
};

// Decode to CSR in two walks over a few segments at a time (decode_slice_csr):
// not a sink of decode_slice, only its parameters.  XCH: the second walk deals
// rows to groups of lanes through LDS (row layout, no escapes).
template <typename VT, bool XCH = false>
struct CsrOut {
    static constexpr uint32_t kLaneWords = 25;  // of the exchange, per lane: eight segments' words and a spare
    // waves per SIMD: the walks keep kBuf segments' words; more waves would
    // not help a kernel bound by its stores
    static constexpr int kOcc = 4;
    struct Params {
        int32_t *col;
        typename Bits<VT>::T *vals;
        uint32_t *xch = nullptr;  // XCH: this wavefront's 64 * kLaneWords words of LDS, set by the kernel
    };
    static __device__ __forceinline__ uint32_t col_scale(const Params &) { return 1u; }
};

// --------------------------------------------------------- wave decoding
// Word sources.  A decoder reads the words of its wave's stream at 32-bit
// byte offsets that are wave-uniform plus a lane prefix.
//
// GlobalWords reads them from device memory: every step's loads depend on the
// previous step's ballots, so each step waits for one memory round trip.
struct GlobalWords {
    const char *W;   // stream base of the current encoded wave
    // its length, kept in 64 bits: a narrower copy would leave half of the
    // loaded offset unused, and reusing that register before the load has
    // returned makes the wave wait for it
    uint64_t bytes;
    // the word at byte offset pos (uniform) + 4 * (lanes of mask below this one):
    // the base stays fixed in SGPRs and each lane forms its 32-bit offset with
    // one shift-add (readfirstlane keeps pos a scalar sum, which the compiler
    // would otherwise fold into the lane count)
    __device__ __forceinline__ uint32_t read(uint32_t pos, uint64_t mask) const {
        const uint32_t p = __builtin_amdgcn_readfirstlane(pos);
        return *(gptr<uint32_t>)(W + (p + 4 * lane_prefix(mask)));
    }
    // the same when every lane of the wavefront reads (prefix = lane)
    __device__ __forceinline__ uint32_t read_lanes(uint32_t pos, uint32_t lane) const {
        const uint32_t p = __builtin_amdgcn_readfirstlane(pos);
        return *(gptr<uint32_t>)(W + (p + 4 * lane));
    }
    // the word at byte offset pos (uniform) + off (per lane): escapes stored
    // in the stream
    __device__ __forceinline__ uint32_t word_at(uint32_t pos, uint32_t off) const {
        const uint32_t p = __builtin_amdgcn_readfirstlane(pos);
        return *(gptr<uint32_t>)(W + (p + off));
    }
    // Nothing in the memory system fetches a stream ahead of its reads, so
    // every step's words would come from HBM.  Once the first words are
    // requested, one load per lane touches the next 64 cache lines (128 B)
    // of the stream, which brings them into L2 while the first steps run.
    // The value is kept (retire) so that the load is not removed; loads
    // complete in order, so the steps' own waits already cover it.
    __device__ __forceinline__ uint32_t prefetch(uint32_t pos, uint32_t lane) const {
        const uint32_t o = (pos & ~127u) + 128u * (lane + 1);
        return o < bytes ? *(gptr<uint32_t>)(W + o) : 0u;
    }
    __device__ __forceinline__ void retire(uint32_t v) const { asm volatile("" ::"v"(v)); }
    __device__ __forceinline__ void step_begin() {}
    __device__ __forceinline__ void consumed(uint32_t) {}
};

// RingWords stages a contiguous run of streams (the encoded waves [a, b) of
// one wavefront are adjacent in memory) through a per-wavefront ring of kRing
// words in LDS.  Chunks of 1 KiB (one aligned 16-byte load per lane) are requested
// as soon as the ring has room and written into it at the start of the next
// step, so the words a step reads were loaded at least one step earlier and
// the decode's serial chain runs through LDS only.  Invariant: chunks are
// requested in order, at most one per step, and written one step later,
// after that step's reads; a step reads at most 768 bytes (three words per
// lane) < one chunk, so the requested end stays at least kRing*4 - 1 KiB
// ahead of the read position, and the words a step reads were requested two
// steps earlier: kRing*4 - 1 KiB >= 2 * 768 + 768 bytes suffices.  A chunk
// overwrites only words already read.  LDS operations of one wavefront
// complete in order, so no barrier is needed between chunk writes and reads.
template <int kRing>
struct RingWords {
    static constexpr uint32_t kChunk = 1024;
    // the first kMirror words of the ring are kept a second time after its
    // end, so that the at most 64 words one read instruction spans never
    // wrap: a read is a prefix count from a uniform start, as from memory
    static constexpr int kMirror = 64;
    static constexpr int kWords = kRing + kMirror;  // LDS words per wavefront
    static_assert(kRing * 4 >= (int)kChunk + 3 * 768, "ring too small for two steps of lead");
    static_assert((kRing & (kRing - 1)) == 0 && kRing % 256 == 0, "ring of whole chunks");
    uint32_t *ring;     // this wavefront's ring (kWords words)
    const char *base;   // the run's first word rounded down to 16 bytes
    uint32_t skew;      // bytes from base to the run's first word (0..12)
    uint32_t total;     // skew + bytes in the run
    uint32_t fetched;   // bytes from base requested so far (multiple of kChunk)
    uint32_t pend_at;   // offset from base of the chunk in flight
    bool has_pend;
    uint4 pend;         // this lane's 16 bytes of the chunk in flight
    uint32_t lane;

    // 16-byte aligned loads; the last one of a run passes its end by at most
    // 15 bytes, which stay inside the padded word buffer.  Lanes past the end
    // reload the run's first 16 bytes (unconditional loads keep the wait
    // counts static); what they write to the ring is never read.
    __device__ __forceinline__ uint4 load_chunk_part(uint32_t at) const {
        const uint32_t o = at + 16 * lane;
        return *(const uint4 *)(base + (o < total ? o : 0u));
    }
    __device__ __forceinline__ void write_chunk_part(uint32_t at, uint4 v) {
        const uint32_t i = ((at >> 2) + 4 * lane) & (kRing - 1);
        *(uint4 *)(ring + i) = v;
        if (i < kMirror) *(uint4 *)(ring + kRing + i) = v;
    }
    __device__ __forceinline__ void start(uint32_t *r, const uint32_t *first, uint32_t bytes,
                                          uint32_t ln) {
        ring = r;
        skew = (uint32_t)((uintptr_t)first & 15);
        base = (const char *)first - skew;
        total = skew + bytes;
        lane = ln;
        fetched = 0;
        has_pend = false;
        // fill the whole ring before the first read
#pragma unroll
        for (int c = 0; c < kRing * 4 / (int)kChunk; ++c) {
            if (fetched < total) {
                write_chunk_part(fetched, load_chunk_part(fetched));
                fetched += kChunk;
            }
        }
    }
    // pos: bytes from the run's first word (uniform, so the start address is
    // scalar work); the lane adds its prefix count
    __device__ __forceinline__ uint32_t read(uint32_t pos, uint64_t mask) const {
        const uint32_t *at = ring + (((pos + skew) >> 2) & (kRing - 1));
        return at[lane_prefix(mask)];
    }
    __device__ __forceinline__ uint32_t read_lanes(uint32_t pos, uint32_t ln) const {
        const uint32_t *at = ring + (((pos + skew) >> 2) & (kRing - 1));
        return at[ln];
    }
    // from memory (streams with escapes inside are never staged through a
    // ring: a step may read more of them than the ring holds ahead)
    __device__ __forceinline__ uint32_t word_at(uint32_t pos, uint32_t off) const {
        const uint32_t p = __builtin_amdgcn_readfirstlane(pos);
        return *(const uint32_t *)(base + (p + skew + off));
    }
    __device__ __forceinline__ uint32_t prefetch(uint32_t, uint32_t) const { return 0u; }
    __device__ __forceinline__ void retire(uint32_t) const {}
    __device__ __forceinline__ void step_begin() {
        if (has_pend) {
            write_chunk_part(pend_at, pend);
            has_pend = false;
        }
    }
    // the decoder's read position has advanced to pos (bytes from the run's
    // first word); request the next chunk once the ring has room for it
    __device__ __forceinline__ void consumed(uint32_t pos) {
        if (fetched < total && fetched + kChunk <= pos + skew + kRing * 4) {
            pend = load_chunk_part(fetched);
            pend_at = fetched;
            has_pend = true;
            fetched += kChunk;
        }
    }
};

// Read positions of a stream: words (bytes), escaped deltas and escaped values
// (counts), with the escape region bases.  A cursor restarts at every encoded
// wave for GlobalWords and runs on across a run for RingWords.
template <typename VT>
struct Cursor {
    uint32_t pos, dpos, vpos;
    const uint32_t *ED;
    const VT *EV;
    // elements of the wave's escape regions to bring into L2 when it starts
    // (0: none)
    uint32_t nd = 0, nv = 0;
};

// As GlobalWords::prefetch for the escape regions: one load per lane touches
// the first 64 cache lines of each, which would otherwise come from memory in
// the middle of the steps that use them.
template <typename VT>
__device__ __forceinline__ uint32_t prefetch_escapes(const Cursor<VT> &c, uint32_t lane) {
    uint32_t t = 0;
    if (c.nd) t = ((gptr<uint32_t>)c.ED)[min(32 * lane, c.nd - 1)];  // uniform
    if (c.nv) t ^= ((gptr<uint32_t>)c.EV)[min(32 * lane, (uint32_t)(sizeof(VT) / 4) * c.nv - 1)];
    return t;
}

// Where a lane's stream sits in the matrix: its first nonzero g0 and count
// (the row layout keeps only the row's [beg, end)); the row of that nonzero
// with the row's [beg, end).  The nonzero layout
// walks the list of nonempty rows ({row, end} pairs, a sentinel {m, nnz} at
// the end), so a lane never visits empty rows (their y is written by
// epilogue_kernel) and crosses exactly one row per nonzero that starts one;
// it keeps the next four list entries, all that one segment can cross
// (next_rows).  Finding the first entry takes two dependent loads (lane_row,
// then the list), so callers issue the first a wave ahead (lane_first_row).
struct LaneGeo {
    int32_t g0;
    int cnt;
    int32_t krow;  // layout NNZ: index of `row` in the nonempty-row list
    int32_t row, row_beg, row_end;
    int2 next[4];  // layout NNZ: the entries after krow
    // layout ROW: the row of the original matrix this lane's row is (rows
    // sorted within windows are encoded in that order) and the position of
    // its first nonzero there
    int32_t orow;
    int32_t gout;
};

template <int LAYOUT>
__device__ __forceinline__ int32_t lane_first_row(const DevMat &a, int64_t slice, uint32_t lane) {
    const int64_t l = slice * kWave + lane;
    if constexpr (LAYOUT == 1) return l < a.num_lanes ? (int32_t)l : 0;
    else return ((gptr<int32_t>)a.lane_row)[l < a.num_lanes ? l : 0];
}

// The list entries krow + 1 .. krow + 4.  Entries past the sentinel lie in the
// buffer's padding; no nonzero reaches them.
__device__ __forceinline__ void next_rows(const DevMat &a, int32_t krow, int2 next[4]) {
    const gptr<u32x4_a8> q = (gptr<u32x4_a8>)(a.nzr + (int64_t)krow + 1);
    const u32x4_a8 lo = q[0], hi = q[1];
    next[0] = make_int2((int)lo.x, (int)lo.y);
    next[1] = make_int2((int)lo.z, (int)lo.w);
    next[2] = make_int2((int)hi.x, (int)hi.y);
    next[3] = make_int2((int)hi.z, (int)hi.w);
}

template <int LAYOUT>
__device__ __forceinline__ LaneGeo lane_geo(const DevMat &a, int64_t slice, uint32_t lane,
                                            int32_t first) {
    LaneGeo q;
    const int64_t l = slice * kWave + lane;
    if constexpr (LAYOUT == 1) {
        // the row's bounds only (lanes past the last row read the last
        // row's): the count is formed where the wave starts, so that a wave
        // loading the next one's geometry does not wait for it
        const int64_t lc = l < a.num_lanes ? l : a.num_lanes - 1;
        q.row = first;
        q.row_beg = ((gptr<int32_t>)a.row_ptr)[lc];
        q.row_end = ((gptr<int32_t>)a.row_ptr)[lc + 1];
        q.orow = first;
        q.gout = q.row_beg;
        if (a.row_perm) {  // uniform
            q.orow = ((gptr<int32_t>)a.row_perm)[lc];
            q.gout = ((gptr<int32_t>)a.orig_row_ptr)[q.orow];
        }
    } else {
        // (lanes past the last one read lane 0's row and hold no nonzeros)
        const bool live = l < a.num_lanes;
        q.g0 = live ? (int32_t)(l * a.lane_nnz) : 0;
        q.cnt = live ? min(a.lane_nnz, (int32_t)a.nnz - q.g0) : 0;
        q.krow = first;
        const int2 c = a.nzr[first];
        q.row = c.x;
        q.row_end = c.y;
        q.row_beg = first > 0 ? a.nzr[first - 1].y : 0;
        next_rows(a, first, q.next);
    }
    return q;
}

// Layout NNZ: the rows of one segment, nonzeros g .. g + nreal: a nonzero at
// the end of the current row starts the next nonempty one, where the column
// restarts.  Selects over the four entries at hand, with no load in the chain
// from one nonzero to the next; the entries after the new row are requested
// at the end, for the next segment that crosses one.  (The entries were
// loaded two crossings ahead, one load per crossing, under a branch per
// nonzero: a segment in which several lanes crossed rows at different
// nonzeros waited for memory at each of them.)  cols: deltas in, columns out.
__device__ __forceinline__ void cross_rows(const DevMat &a, uint32_t scale, uint32_t g, int nreal, int32_t &row,
                                           int32_t &row_end, int32_t &krow, int2 next[4], bool &head, uint32_t &col,
                                           uint32_t cols[4], int32_t rowk[4]) {
    if (!ballot(nreal > 0 && g + (uint32_t)nreal > (uint32_t)row_end)) {  // uniform: no lane crosses a row
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            col += cols[k];
            cols[k] = col;
            rowk[k] = row;
        }
        return;
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const bool c = k < nreal && g + (uint32_t)k >= (uint32_t)row_end;
        row = c ? next[0].x : row;
        row_end = c ? next[0].y : row_end;
#pragma unroll
        for (int i = 0; i + k < 3; ++i) {
            next[i].x = c ? next[i + 1].x : next[i].x;
            next[i].y = c ? next[i + 1].y : next[i].y;
        }
        krow += c ? 1 : 0;
        head = head && !c;
        col = (c ? first_base(a.first_mode, (uint32_t)row) * scale : col) + cols[k];
        cols[k] = col;
        rowk[k] = row;
    }
    next_rows(a, krow, next);
}

// LDS byte offsets of a segment's eight slots (unpack8 of dtans_core.hpp
// with the entry sizes folded in): delta slots i1, i3, i5, i7 into the delta
// table (8-byte entries), value slots i2, i4, i6, i8 into the value table
// (E-byte entries), straight from the three words.
template <int E>
__device__ __forceinline__ void slot_offsets(uint32_t w1, uint32_t w2, uint32_t w3, uint32_t od[4],
                                             uint32_t ov[4]) {
    od[0] = (w3 << 3) & 0x7ff8u;                                  // i1 = w3[0:12]
    ov[0] = ((w3 >> 12) & 0xfffu) * E;                             // i2 = w3[12:24]
    od[1] = __builtin_amdgcn_alignbit(w2, w3, 21) & 0x7ff8u;       // i3 = w3[24:32] | w2[0:4] << 8
    ov[1] = ((w2 >> 4) & 0xfffu) * E;                              // i4 = w2[4:16]
    od[2] = (w2 >> 13) & 0x7ff8u;                                  // i5 = w2[16:28]
    ov[2] = (__builtin_amdgcn_alignbit(w1, w2, 28) & 0xfffu) * E;  // i6 = w2[28:32] | w1[0:8] << 4
    od[3] = (w1 >> 5) & 0x7ff8u;                                   // i7 = w1[8:20]
    ov[3] = (w1 >> 20) * E;                                        // i8 = w1[20:32]
}

// A segment's escaped deltas and values from their regions, in the order
// (nonzero, lane): flag bits in md and mv, nreal nonzeros in this lane.
// TOGETHER: all eight loads are issued before any of their values is used (a
// use between them made the wavefront wait for memory up to eight times a
// segment); lanes without an escape read the region's next element, or, past
// the last one, the buffer's padding.  The values on their way take twelve
// registers with FP64, which the row layout's kernels, at eight waves per
// SIMD, do not have: they spilled (band of 2,000,000 rows with escaped values:
// 56 -> 64 us), so there each load goes straight to its place.
template <typename VT, bool TOGETHER>
__device__ __forceinline__ void take_escapes(gptr<uint32_t> ED, gptr<VT> EV, uint32_t &dpos, uint32_t &vpos, int nreal,
                                             const uint32_t md[4], const uint32_t mv[4], uint32_t scale,
                                             uint32_t dl[4], VT v[4]) {
    if constexpr (!TOGETHER) {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const bool f = k < nreal && (int32_t)md[k] < 0;
            const uint64_t mk = ballot(f);
            if (f) dl[k] = ED[dpos + lane_prefix(mk)] * scale;
            dpos += (uint32_t)__popcll(mk);
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const bool f = k < nreal && (int32_t)mv[k] < 0;
            const uint64_t mk = ballot(f);
            if (f) v[k] = EV[vpos + lane_prefix(mk)];
            vpos += (uint32_t)__popcll(mk);
        }
        return;
    }
    uint32_t rd[4];
    VT rv[4];
    // (uniform branches: in most matrices few of the eight hold an escape)
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const bool f = k < nreal && (int32_t)md[k] < 0;
        const uint64_t mk = ballot(f);
        if (mk) rd[k] = ED[dpos + (f ? lane_prefix(mk) : 0u)];
        dpos += (uint32_t)__popcll(mk);
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const bool f = k < nreal && (int32_t)mv[k] < 0;
        const uint64_t mk = ballot(f);
        if (mk) rv[k] = EV[vpos + (f ? lane_prefix(mk) : 0u)];
        vpos += (uint32_t)__popcll(mk);
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        if (k < nreal && (int32_t)md[k] < 0) dl[k] = rd[k] * scale;
        if (k < nreal && (int32_t)mv[k] < 0) v[k] = rv[k];
    }
}

// Decode encoded wave `slice` (lanes slice*64 .. slice*64+63) and feed the
// nonzeros of this thread's lane to a sink constructed here.
// TF, the table format: 0 some base is 256 (the paper's M; a digit group's
// base product may reach 2^32); 1 "direct" tables (every base at most 255: a
// group's arithmetic runs on packed 16-bit halves); 2 direct tables without
// an escape symbol in either alphabet (no escape checks at all).
// A step of the whole wavefront is "full" when every lane decodes four
// nonzeros and has a next segment (no masks, every lane loads its words);
// other steps handle lanes that end, are short or have nothing left.
template <int LAYOUT, typename VT, class Sink, class Src, int TF>
__device__ __forceinline__ void decode_slice(const DevMat &a, const Tables<VT> &tb, int64_t slice,
                                             uint32_t lane, const typename Sink::Params &sp,
                                             Src &src, Cursor<VT> &cur, const LaneGeo &geo) {
    const int64_t l = slice * kWave + lane;
    const bool live = l < a.num_lanes;
    const int32_t g0 = LAYOUT == 1 ? geo.row_beg : geo.g0;
    const int cnt = LAYOUT == 1 ? (live ? geo.row_end - geo.row_beg : 0) : geo.cnt;
    int32_t row = geo.row, row_end = geo.row_end, krow = geo.krow;
    bool head = LAYOUT == 2 && geo.row_beg < g0;  // the current row began in an earlier lane
    int2 next[4];
    if constexpr (LAYOUT == 2) {
#pragma unroll
        for (int i = 0; i < 4; ++i) next[i] = geo.next[i];
    }
    // the sink sees rows and nonzero positions of the original matrix (row
    // layout: rows may be encoded in another order); the decoder's own row
    // (first deltas) is the encoded one
    const int32_t srow = LAYOUT == 1 ? geo.orow : row;
    Sink sink(sp, l, srow, head);
    const uint32_t scale = Sink::col_scale(sp);  // column deltas arrive multiplied by it
    const int S = (cnt + 3) >> 2;
    const int F = min(S - 1, cnt >> 2);  // steps j < F: four nonzeros and a next segment

    // stream offsets are 32-bit and wave-uniform (popcounts of ballots), so
    // they live in SGPRs
    uint32_t pos = cur.pos, dpos = cur.dpos, vpos = cur.vpos;
    const uint32_t *__restrict__ ED = cur.ED;
    const VT *__restrict__ EV = cur.EV;
    // A step's words: l1, l2 as loaded unless the check extracted them from
    // the state (e1, e2; then x1, x2), l3 always loaded.  The selection is
    // made at the top of the step that uses them, so that no instruction of
    // the step that loads them waits for those loads.
    uint32_t l1, l2, l3, x1 = 0, x2 = 0;
    bool e1 = false, e2 = false;
    {
        // lanes without a stream read a neighbouring word (buffers are padded)
        const uint64_t mk = ballot(S > 0);
        const uint32_t c = 4 * (uint32_t)__popcll(mk);
        l1 = src.read(pos, mk);
        l2 = src.read(pos + c, mk);
        l3 = src.read(pos + 2 * c, mk);
        pos += 3 * c;
        src.step_begin();
        src.consumed(pos);
    }
    const uint32_t pf = src.prefetch(pos, lane);
    const uint32_t pe = TF != 2 ? prefetch_escapes<VT>(cur, lane) : 0u;
    if constexpr (LAYOUT == 2) {
        // The lane's rows are waited for here, behind the requests for the
        // first words: loaded on some paths only, they would otherwise be
        // waited for in every step of the loops below, and with them whatever
        // was requested after them.
        asm volatile("" : "+v"(row), "+v"(row_end));
#pragma unroll
        for (int i = 0; i < 4; ++i) asm volatile("" : "+v"(next[i].x), "+v"(next[i].y));
    }
    uint32_t d = 0, r = 1, col = first_base(a.first_mode, (uint32_t)row) * scale;
    uint32_t g = (uint32_t)(LAYOUT == 1 ? geo.gout : g0);

    auto step = [&](auto fullc, int j) {
        constexpr bool FULL = decltype(fullc)::value;
        const bool act = FULL || j < S;
        const bool more = FULL || j + 1 < S;
        const int rem = cnt - 4 * j;
        uint32_t od[4], ov[4];
        slot_offsets<(int)sizeof(VEntry<VT>)>(e1 ? x1 : l1, e2 ? x2 : l2, l3, od, ov);
        uint32_t dl[4], md[4], mv[4];
        VT v[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const uint64_t e = *(const uint64_t *)((const char *)tb.td + od[k]);
            const VEntry<VT> ve = *(const VEntry<VT> *)((const char *)tb.tv + ov[k]);
            dl[k] = (uint32_t)e;
            md[k] = (uint32_t)(e >> 32);
            v[k] = ve.value();
            mv[k] = ve.meta;
        }
        // Escapes (their loads issued before the next words, so that waiting
        // for them does not wait for the words): flagged by bit 31 of a slot's
        // metadata.  When no active lane has a flag in any of its eight
        // entries (the common case) nothing is masked; padding symbols are
        // never escapes, so only lanes past their last segment can hold one
        // otherwise.
        if constexpr (TF != 2) {
            const uint32_t fl = md[0] | md[1] | md[2] | md[3] | mv[0] | mv[1] | mv[2] | mv[3];
            if ((FULL ? ~0ull : ballot(act)) & ballot((int32_t)fl < 0)) {  // uniform
                if (a.esc_in_stream) {
                    // raw bits in the word stream at the read position:
                    // deltas, then values (FP64 as two words, low first),
                    // each nonzero position in lane order; the step's own
                    // words follow them
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        const bool f = act && k < rem && (int32_t)md[k] < 0;
                        const uint64_t mk = ballot(f);
                        if (f) dl[k] = src.word_at(pos, 4 * lane_prefix(mk)) * scale;
                        pos += 4 * (uint32_t)__popcll(mk);
                    }
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        const bool f = act && k < rem && (int32_t)mv[k] < 0;
                        const uint64_t mk = ballot(f);
                        if (f) {
                            const uint32_t o = (uint32_t)sizeof(VT) * lane_prefix(mk);
                            if constexpr (sizeof(VT) == 8) {
                                const uint64_t bits = (uint64_t)src.word_at(pos, o + 4) << 32 | src.word_at(pos, o);
                                v[k] = __builtin_bit_cast(VT, bits);
                            } else {
                                v[k] = __builtin_bit_cast(VT, src.word_at(pos, o));
                            }
                        }
                        pos += (uint32_t)sizeof(VT) * (uint32_t)__popcll(mk);
                    }
                } else {
                    constexpr bool together = sizeof(VT) == 4 || LAYOUT == 2;
                    take_escapes<VT, together>((gptr<uint32_t>)ED, (gptr<VT>)EV, dpos, vpos,
                                               act ? min(rem, 4) : 0, md, mv, scale, dl, v);
                }
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    md[k] &= ~kMetaEscape;
                    mv[k] &= ~kMetaEscape;
                }
            }
        }
        // the two digit groups and their checks (Alg. 3), then the next
        // segment's words, in flight while this segment's x gathers are
        // served.  The loads are issued on every step, so that the wait
        // counts of the loads before them are the same on every path; lanes
        // that do not load (all of them on a wave's last step) read a
        // neighbouring word of the stream, whose value is not used.
        const uint64_t m3 = FULL ? ~0ull : ballot(more);  // lanes that load this step's words
        uint64_t m1 = 0, m2 = 0;
        if (FULL || m3) {
            uint32_t D, R;
            if constexpr (TF >= 1) {
                group_pairs(pair_rd(md[0], mv[0]), pair_rd(md[1], mv[1]), D, R);
                e1 = append_word(d, r, D, R, x1);
                group_pairs(pair_rd(md[2], mv[2]), pair_rd(md[3], mv[3]), D, R);
                e2 = append_word(d, r, D, R, x2);
            } else {
                group_general(md[0], mv[0], md[1], mv[1], D, R);
                e1 = append_and_check(d, r, D, R, x1);
                group_general(md[2], mv[2], md[3], mv[3], D, R);
                e2 = append_and_check(d, r, D, R, x2);
            }
            // masks combined on the scalar unit: a ballot of a plain compare
            // is the compare's own lane mask
            m1 = m3 & ~ballot(e1);
            m2 = m3 & ~ballot(e2);
        }
        {
            const uint32_t c1 = 4 * (uint32_t)__popcll(m1), c2 = 4 * (uint32_t)__popcll(m2);
            l1 = src.read(pos, m1);
            l2 = src.read(pos + c1, m2);
            if constexpr (FULL) {
                l3 = src.read_lanes(pos + c1 + c2, lane);
                pos += c1 + c2 + 4 * kWave;
            } else {
                l3 = src.read(pos + c1 + c2, m3);
                pos += c1 + c2 + 4 * (uint32_t)__popcll(m3);
            }
        }
        // deferred products of the previous step and the ring's pending chunk,
        // then the next chunk and this step's x loads, which the next step
        // waits for: a step waits on memory for loads issued a step earlier
        sink.pre_step();
        src.step_begin();
        src.consumed(pos);
        const int nreal = FULL ? 4 : (act ? min(rem, 4) : 0);
        uint32_t cols[4];
        int32_t rowk[4];
        if constexpr (LAYOUT == 1) {
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                col += dl[k];
                cols[k] = col;
                rowk[k] = srow;
            }
            // (the general-table decoder measured slower with paired loads)
            if constexpr (Sink::kPairs && TF == 0) sink.template segment<false, false>(cols, v, nreal, g, rowk);
            else sink.template segment<false>(cols, v, nreal, g, rowk);
        } else {
            // resolve row boundaries first: a column delta restarts at every
            // row; the sink finishes the rows left behind
#pragma unroll
            for (int k = 0; k < 4; ++k) cols[k] = dl[k];
            cross_rows(a, scale, g, nreal, row, row_end, krow, next, head, col, cols, rowk);
            sink.template segment<true>(cols, v, nreal, g, rowk);
        }
        g += 4;
    };
    // full steps while every lane of the wavefront has one (a uniform test),
    // then the rest with per-lane masks
    int j = 0;
    if (ballot(0 < F) == ~0ull) {
        do {
            step(std::true_type(), j);
            ++j;
        } while (ballot(j < F) == ~0ull);
    }
    for (; ballot(j < S) != 0; ++j) step(std::false_type(), j);
    src.retire(pf);
    if (TF != 2) src.retire(pe);
    cur.pos = pos;
    cur.dpos = dpos;
    cur.vpos = vpos;
    if constexpr (LAYOUT == 1) {
        // (a cooperative sink needs every lane of the wavefront)
        if constexpr (Sink::kCoop) sink.finish_lane(srow, kComplete, live && l < a.m);
        else if (live && l < a.m) sink.finish_row(srow, kComplete);
    } else {
        // `row` holds this lane's last nonzeros: complete when it ends here;
        // started in an earlier lane, a head when it ends here, else a
        // middle; else a tail
        const bool ends = row_end <= g0 + cnt;
        sink.finish_lane(row, head ? (ends ? kHead : kMid) : (ends ? kComplete : kTail), live);
    }
}

// Decode encoded wave `slice` to CSR.  A lane's nonzeros are consecutive in
// memory, but one segment is only 16 bytes of columns and 16 or 32 of values:
// stored segment by segment, every cache line is written in pieces too far
// apart in time for the L2 to put together (27-point stencil on 100^3, FP64:
// 0.9 to 1.0 GB written for 317 MB of CSR, 0.27 ms).  So kBuf segments are decoded in
// two walks: the first follows the stream's serial chain with the tables'
// metadata alone and keeps each segment's three words; the second looks their
// columns and values up and stores them, all within a short time (568 MB,
// 0.18 ms: still bound by what the lines' pieces cost).  Escapes
// stay in their regions until the second walk (in-stream escapes, whose
// positions the first walk would need, take decode_slice with DecodeSink).
//
// XCH: one lane's segments are 16 bytes at a row's stride from its neighbour's,
// so even together they cost an instruction 64 cache lines, most of them in
// part.  The second walk instead gives 2^lg lanes to a row, a segment each
// (the words pass through LDS, the columns by a scan over the group), so that
// an instruction stores whole rows one after the other: 0.18 -> 0.13 ms, 320 MB
// written.
template <int LAYOUT, typename VT, class Src, int TF, bool XCH>
__device__ __forceinline__ void decode_slice_csr(const DevMat &a, const Tables<VT> &tb, int64_t slice, uint32_t lane,
                                                 const typename CsrOut<VT, XCH>::Params &sp, Src &src,
                                                 Cursor<VT> &cur, const LaneGeo &geo) {
    constexpr int kBuf = 8;
    typedef typename Bits<VT>::T BT;
    const int64_t l = slice * kWave + lane;
    const bool live = l < a.num_lanes;
    const int cnt = LAYOUT == 1 ? (live ? geo.row_end - geo.row_beg : 0) : geo.cnt;
    int32_t row = geo.row, row_end = geo.row_end, krow = geo.krow;
    bool head = false;
    int2 next[4];
    if constexpr (LAYOUT == 2) {
#pragma unroll
        for (int i = 0; i < 4; ++i) next[i] = geo.next[i];
    }
    const int S = (cnt + 3) >> 2;
    uint32_t pos = cur.pos, dpos = cur.dpos, vpos = cur.vpos;
    uint32_t l1, l2, l3, x1 = 0, x2 = 0;
    bool e1 = false, e2 = false;
    {
        const uint64_t mk = ballot(S > 0);
        const uint32_t c = 4 * (uint32_t)__popcll(mk);
        l1 = src.read(pos, mk);
        l2 = src.read(pos + c, mk);
        l3 = src.read(pos + 2 * c, mk);
        pos += 3 * c;
    }
    const uint32_t pf = src.prefetch(pos, lane);
    uint32_t d = 0, r = 1, col = first_base(a.first_mode, (uint32_t)row);
    int64_t g = LAYOUT == 1 ? geo.gout : geo.g0;
    for (int j = 0; ballot(j < S) != 0; j += kBuf) {
        uint32_t w1[kBuf], w2[kBuf], w3[kBuf];
        // first walk: the words of segments j .. j + kBuf (see decode_slice
        // for the steps; past a lane's end nothing of it is used)
#pragma unroll
        for (int i = 0; i < kBuf; ++i) {
            w1[i] = e1 ? x1 : l1;
            w2[i] = e2 ? x2 : l2;
            w3[i] = l3;
            const uint64_t m3 = ballot(j + i + 1 < S);  // lanes with a next segment
            if (m3 == 0) continue;
            uint32_t od[4], ov[4], md[4], mv[4];
            slot_offsets<(int)sizeof(VEntry<VT>)>(w1[i], w2[i], w3[i], od, ov);
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                md[k] = *(const uint32_t *)((const char *)tb.td + od[k] + 4);
                mv[k] = ((const VEntry<VT> *)((const char *)tb.tv + ov[k]))->meta;
                if constexpr (TF != 2) {
                    md[k] &= ~kMetaEscape;
                    mv[k] &= ~kMetaEscape;
                }
            }
            uint32_t D, R;
            if constexpr (TF >= 1) {
                group_pairs(pair_rd(md[0], mv[0]), pair_rd(md[1], mv[1]), D, R);
                e1 = append_word(d, r, D, R, x1);
                group_pairs(pair_rd(md[2], mv[2]), pair_rd(md[3], mv[3]), D, R);
                e2 = append_word(d, r, D, R, x2);
            } else {
                group_general(md[0], mv[0], md[1], mv[1], D, R);
                e1 = append_and_check(d, r, D, R, x1);
                group_general(md[2], mv[2], md[3], mv[3], D, R);
                e2 = append_and_check(d, r, D, R, x2);
            }
            const uint64_t m1 = m3 & ~ballot(e1), m2 = m3 & ~ballot(e2);
            const uint32_t c1 = 4 * (uint32_t)__popcll(m1), c2 = 4 * (uint32_t)__popcll(m2);
            l1 = src.read(pos, m1);
            l2 = src.read(pos + c1, m2);
            l3 = src.read(pos + c1 + c2, m3);
            pos += c1 + c2 + 4 * (uint32_t)__popcll(m3);
        }
        // second walk: columns and values
        if constexpr (XCH) {
            static_assert(LAYOUT == 1 && TF == 2, "rows of one lane, no escapes");
            constexpr uint32_t kL = CsrOut<VT, XCH>::kLaneWords;
            // 2^lg lanes a row: as many as some row has segments here
            const uint32_t lg = ballot(j + 4 < S) ? 3u : ballot(j + 2 < S) ? 2u : ballot(j + 1 < S) ? 1u : 0u;
#pragma unroll
            for (int i = 0; i < kBuf; ++i) {
                if (i >= 1 << lg) break;  // uniform
                sp.xch[lane * kL + 3 * i] = w1[i];
                sp.xch[lane * kL + 3 * i + 1] = w2[i];
                sp.xch[lane * kL + 3 * i + 2] = w3[i];
            }
            wave_exchange_fence();  // the words are read by other lanes
            const uint32_t sub = lane & ((1u << lg) - 1u), grp = lane >> lg, rows = 64u >> lg;
            for (uint32_t b = 0; b < 1u << lg; ++b) {
                const uint32_t rl = b * rows + grp;  // the lane that decoded this group's row
                const int nreal = min(max((int)lane_value((uint32_t)cnt, rl) - 4 * (j + (int)sub), 0), 4);
                const uint32_t gr = lane_value((uint32_t)g, rl) + 4 * sub;
                const uint32_t *w = sp.xch + rl * kL + 3 * sub;
                uint32_t od[4], ov[4], cols[4];
                VT v[4];
                // (lanes without a segment look up whatever lies there; every
                // slot is in the tables)
                slot_offsets<(int)sizeof(VEntry<VT>)>(w[0], w[1], w[2], od, ov);
                uint32_t sum = 0, own = 0;
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    sum += *(const uint32_t *)((const char *)tb.td + od[k]);
                    cols[k] = sum;
                    own = k < nreal ? sum : own;
                    v[k] = ((const VEntry<VT> *)((const char *)tb.tv + ov[k]))->value();
                }
                uint32_t upto = own;  // deltas of the row up to this segment's end
                for (uint32_t t = 1; t < 1u << lg; t <<= 1) {
                    const uint32_t o = lane_value(upto, (lane - t) & (kWave - 1));
                    upto += sub >= t ? o : 0u;
                }
                const uint32_t before = lane_value(col, rl) + upto - own;
                if (nreal == 4) {
                    *(gmut<u32x4_a4>)(sp.col + gr) =
                        u32x4_a4{before + cols[0], before + cols[1], before + cols[2], before + cols[3]};
                    constexpr int per = 16 / (int)sizeof(VT);
#pragma unroll
                    for (int h = 0; h < 4; h += per) {
                        u32x4_a4 q;
                        __builtin_memcpy(&q, v + h, 16);
                        *(gmut<u32x4_a4>)(sp.vals + gr + h) = q;
                    }
                } else {
#pragma unroll
                    for (int k = 0; k < 3; ++k)
                        if (k < nreal) {
                            ((gmut<int32_t>)sp.col)[gr + k] = (int32_t)(before + cols[k]);
                            ((gmut<BT>)sp.vals)[gr + k] = __builtin_bit_cast(BT, v[k]);
                        }
                }
                // the row's column so far, back to its lane
                const uint32_t all = lane_value(upto, ((lane & (rows - 1u)) << lg) + (1u << lg) - 1u);
                if ((lane >> (6u - lg)) == b) col += all;
            }
            wave_exchange_fence();  // the next segments' words come over these
            g += 4 * kBuf;
            continue;
        }
#pragma unroll
        for (int i = 0; i < kBuf; ++i) {
            if (ballot(j + i < S) == 0) break;
            const int nreal = min(max(cnt - 4 * (j + i), 0), 4);
            uint32_t od[4], ov[4], dl[4], md[4], mv[4], cols[4];
            VT v[4];
            slot_offsets<(int)sizeof(VEntry<VT>)>(w1[i], w2[i], w3[i], od, ov);
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const uint64_t e = *(const uint64_t *)((const char *)tb.td + od[k]);
                const VEntry<VT> ve = *(const VEntry<VT> *)((const char *)tb.tv + ov[k]);
                dl[k] = (uint32_t)e;
                md[k] = (uint32_t)(e >> 32);
                v[k] = ve.value();
                mv[k] = ve.meta;
            }
            if constexpr (TF != 2) {
                const uint32_t fl = md[0] | md[1] | md[2] | md[3] | mv[0] | mv[1] | mv[2] | mv[3];
                if (ballot(nreal > 0) & ballot((int32_t)fl < 0)) {  // uniform
                    take_escapes<VT, true>((gptr<uint32_t>)cur.ED, (gptr<VT>)cur.EV, dpos, vpos, nreal, md, mv, 1u, dl, v);
                }
            }
            if constexpr (LAYOUT == 2) {
                int32_t rowk[4];
#pragma unroll
                for (int k = 0; k < 4; ++k) cols[k] = dl[k];
                cross_rows(a, 1u, (uint32_t)g, nreal, row, row_end, krow, next, head, col, cols, rowk);
            } else {
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    col += dl[k];
                    cols[k] = col;
                }
            }
            if (nreal == 4) {
                *(gmut<u32x4_a4>)(sp.col + g) = u32x4_a4{cols[0], cols[1], cols[2], cols[3]};
                constexpr int per = 16 / (int)sizeof(VT);
#pragma unroll
                for (int h = 0; h < 4; h += per) {
                    u32x4_a4 q;
                    __builtin_memcpy(&q, v + h, 16);
                    *(gmut<u32x4_a4>)(sp.vals + g + h) = q;
                }
            } else {
#pragma unroll
                for (int k = 0; k < 3; ++k)
                    if (k < nreal) {
                        ((gmut<int32_t>)sp.col)[g + k] = (int32_t)cols[k];
                        ((gmut<BT>)sp.vals)[g + k] = __builtin_bit_cast(BT, v[k]);
                    }
            }
            g += 4;
        }
    }
    src.retire(pf);
    cur.pos = pos;
    cur.dpos = dpos;
    cur.vpos = vpos;
}

// the decoder of a sink (or of CsrOut)
template <int LAYOUT, typename VT, class Sink, class Src, int TF>
__device__ __forceinline__ void decode_wave(const DevMat &a, const Tables<VT> &tb, int64_t slice, uint32_t lane,
                                            const typename Sink::Params &sp, Src &src, Cursor<VT> &cur,
                                            const LaneGeo &geo) {
    if constexpr (std::is_same<Sink, CsrOut<VT, false>>::value)
        decode_slice_csr<LAYOUT, VT, Src, TF, false>(a, tb, slice, lane, sp, src, cur, geo);
    else if constexpr (std::is_same<Sink, CsrOut<VT, true>>::value)
        decode_slice_csr<LAYOUT, VT, Src, TF, true>(a, tb, slice, lane, sp, src, cur, geo);
    else
        decode_slice<LAYOUT, VT, Sink, Src, TF>(a, tb, slice, lane, sp, src, cur, geo);
}

// Offsets of an encoded wave's words and escapes (uniform, scalar loads).  ESC:
// with the ends of the escape regions, for their prefetch (nonzero layout; in
// the row layout's kernels, at eight waves per SIMD, the scalars that hold
// them would spill).
template <bool ESC>
struct WaveSpan {
    uint64_t w0, w1, d0, v0, d1 = 0, v1 = 0;
    __device__ __forceinline__ WaveSpan(const DevMat &a, int64_t s)
        : w0(uniform_load(a.woff + s)), w1(uniform_load(a.woff + s + 1)), d0(uniform_load(a.doff + s)),
          v0(uniform_load(a.voff + s)) {
        if constexpr (ESC) {
            d1 = uniform_load(a.doff + s + 1);
            v1 = uniform_load(a.voff + s + 1);
        }
    }
    __device__ __forceinline__ GlobalWords words(const DevMat &a) const {
        return GlobalWords{(const char *)(a.words + w0), 4 * (w1 - w0)};
    }
    template <typename VT>
    __device__ __forceinline__ Cursor<VT> cursor(const DevMat &a) const {
        Cursor<VT> c{0, 0, 0, a.escd + d0, (const VT *)a.escv + v0, 0, 0};
        if constexpr (ESC) {
            c.nd = (uint32_t)(d1 - d0);
            c.nv = (uint32_t)(v1 - v0);
        }
        return c;
    }
};

// Both tables into LDS in 16-byte pieces, every piece of a pass loaded before
// any is stored, so that a pass costs one memory round trip (two passes for a
// 1024-thread workgroup); the column deltas are multiplied by `scale` on the
// way (the sink's col_scale).
template <typename VT>
__device__ __forceinline__ void stage_tables(const DevMat &a, Tables<VT> &tb, uint32_t scale) {
    constexpr int kV = kSlots * (int)sizeof(VEntry<VT>) / 16, kT = kSlots * 8 / 16;
    constexpr int kAll = kV + kT, kU = 4;  // pieces per thread and pass
    const gptr<u32x4> gv = (gptr<u32x4>)a.tabval, gt = (gptr<u32x4>)a.tab;
    u32x4 *lds = (u32x4 *)&tb;  // tv, then td
    const int nt = blockDim.x;
    for (int b = 0; b < kAll; b += kU * nt) {
        u32x4 t[kU];
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const int i = b + u * nt + (int)threadIdx.x;
            t[u] = u32x4{0u, 0u, 0u, 0u};
            if (i < kV) t[u] = gv[i];
            else if (i < kAll) {
                t[u] = gt[i - kV];
                t[u].x *= scale;  // two entries per piece: {delta, meta}, {delta, meta}
                t[u].z *= scale;
            }
        }
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const int i = b + u * nt + (int)threadIdx.x;
            if (i < kAll) lds[i] = t[u];
        }
    }
    __syncthreads();
}

// Wave priority from the share of a wavefront's encoded waves still ahead of
// it (3 with more than three quarters left ... 0 in the last quarter).  The
// arbiter otherwise favours the oldest wavefronts, which then finish their
// (equal) shares early and leave the younger ones to end the launch at low
// occupancy; ranking by remaining work keeps the wavefronts of a CU in step.
// (The quarter is found by comparisons, not a 64-bit division, which would
// cost a hundred scalar instructions per wave.)
__device__ __forceinline__ void set_progress_priority(int64_t remaining, int64_t total) {
    const int64_t q = (remaining - 1) * 4;  // quarter = floor(q / total)
    if (total <= 0 || q < total) __builtin_amdgcn_s_setprio(0);
    else if (q < 2 * total) __builtin_amdgcn_s_setprio(1);
    else if (q < 3 * total) __builtin_amdgcn_s_setprio(2);
    else __builtin_amdgcn_s_setprio(3);
}

// The row-layout sweep of decode_kernel over waves s0, s0 + stride, ... below
// s_end (share of them).
// stage: 0 the tables are in LDS already; 1 stage them; 2 wait for the
// workgroup (its previous matrix), then stage them (the whole workgroup
// passes the same value).
template <typename VT, class Sink, int TF>
__device__ __forceinline__ void decode_rows(const DevMat &a, Tables<VT> &tb,
                                            uint32_t lane, const typename Sink::Params &sp,
                                            int64_t s_end, int64_t s0, int64_t stride,
                                            int64_t share, int stage = 1) {
    // Row layout: the next encoded wave's lane geometry and stream bases are
    // loaded while this one decodes, so a wave starts with one memory round
    // trip (its first words) instead of two; the first wave's are requested
    // before the tables are staged.  The loads for the next wave are issued
    // on every pass (past the last wave they read this wave's again), so that
    // no branch around them makes the wait counts of later loads unknown,
    // which would turn the first wait of the wave into a wait for everything
    // in flight.
    const int64_t sf = s0 < s_end ? s0 : a.num_waves - 1;  // in bounds for idle wavefronts
    LaneGeo geo = lane_geo<1>(a, sf, lane, lane_first_row<1>(a, sf, lane));
    WaveSpan<false> span(a, sf);
    if (stage == 2) __syncthreads();
    if (stage) stage_tables<VT>(a, tb, Sink::col_scale(sp));
    int64_t k = 0;
    for (int64_t s = s0; s < s_end; s += stride, ++k) {
        const int64_t s1 = s + stride < s_end ? s + stride : s;
        const LaneGeo next = lane_geo<1>(a, s1, lane, lane_first_row<1>(a, s1, lane));
        const WaveSpan<false> span1(a, s1);
        GlobalWords src = span.words(a);
        Cursor<VT> cur = span.template cursor<VT>(a);
        set_progress_priority(share - k, share);
        decode_wave<1, VT, Sink, GlobalWords, TF>(a, tb, s, lane, sp, src, cur, geo);
        geo = next;
        span = span1;
    }
}

// The place of workgroup `block` among `grid` when the workgroups of one XCD
// (dispatch is round-robin) are numbered one after the other: first + pos, of
// the blocks on its XCD; and the first of W items that falls to workgroup i
// when they are dealt evenly in that order, floor(i W / grid).  (32-bit
// divisions: 64-bit ones cost the start of every wavefront about a hundred
// instructions each.  A grid has below 2^16 workgroups.)
struct XcdShare {
    uint32_t grid, first, pos, blocks, per, rem;
    __device__ __forceinline__ XcdShare(uint32_t grid_, uint32_t block, uint32_t W) : grid(grid_) {
        const uint32_t xcd = block % kNumXcd, q = grid / kNumXcd, r = grid % kNumXcd;
        pos = block / kNumXcd;
        blocks = q + (xcd < r ? 1u : 0u);
        first = xcd * q + min(xcd, r);
        per = W / grid;
        rem = W - per * grid;
    }
    __device__ __forceinline__ uint32_t cut(uint32_t i) const { return i * per + i * rem / grid; }
};

// The nonzero-layout sweep over waves s0, s0 + stride, ... below s_end (share
// of them), tables staged on the way.  A wave starts with a chain of loads
// (offsets and lane_row, then the row list, then the first words), so the
// first two are issued a wave ahead, and for the first wave before the tables
// are staged.  (Touching the first wave's words and escapes there as well
// measured 5 us slower on the pruned weight: the staging then waits for them.)
template <typename VT, class Sink, int TF>
__device__ __forceinline__ void decode_lanes(const DevMat &a, Tables<VT> &tb, uint32_t lane,
                                             const typename Sink::Params &sp, int64_t s_end, int64_t s0,
                                             int64_t stride, int64_t share) {
    const int64_t sf = s0 < s_end ? s0 : a.num_waves - 1;  // in bounds for idle wavefronts
    WaveSpan<(TF != 2)> span(a, sf);
    LaneGeo geo = lane_geo<2>(a, sf, lane, lane_first_row<2>(a, sf, lane));
    stage_tables<VT>(a, tb, Sink::col_scale(sp));
    int64_t k = 0;
    for (int64_t s = s0; s < s_end; s += stride, ++k) {
        const int64_t s1 = s + stride < s_end ? s + stride : s;
        const WaveSpan<(TF != 2)> span1(a, s1);
        const int32_t first1 = lane_first_row<2>(a, s1, lane);
        GlobalWords src = span.words(a);
        Cursor<VT> cur = span.template cursor<VT>(a);
        set_progress_priority(share - k, share);
        decode_wave<2, VT, Sink, GlobalWords, TF>(a, tb, s, lane, sp, src, cur, geo);
        // (on every pass: under a branch, the decoder's waits cover both paths
        // and came out a sixth slower)
        geo = lane_geo<2>(a, s1, lane, first1);
        span = span1;
    }
}

// The sweep of one persistent workgroup over its encoded waves (tables
// staged into LDS on the way).
template <int LAYOUT, typename VT, class Sink, int TF>
__device__ __forceinline__ void decode_sweep(const DevMat &a, const typename Sink::Params &sp,
                                             Tables<VT> &tb) {
    const uint32_t lane = threadIdx.x & (kWave - 1), wib = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const uint32_t wpb = blockDim.x / kWave;
    // Workgroups are dispatched round-robin over the XCDs.  The workgroups of
    // one XCD own one contiguous share of the encoded waves, and their
    // wavefronts sweep it together (wavefront i takes waves i, i + W, ...), so
    // at any time an XCD decodes a compact window of rows and its x gathers
    // stay in that XCD's L2.  The wave index is uniform (readfirstlane).
    const XcdShare sh(gridDim.x, blockIdx.x, (uint32_t)a.num_waves);
    int64_t s0 = sh.cut(sh.first) + sh.pos * wpb + wib, s_end = sh.cut(sh.first + sh.blocks);
    const int64_t stride = sh.blocks * wpb;
    if (a.num_waves <= (int64_t)gridDim.x * wpb) {
        // no more waves than wavefronts: neighbouring waves to each workgroup,
        // the same number to all (taken in order, the first workgroups would
        // be full and the last idle)
        s0 = sh.cut(sh.first + sh.pos) + wib;
        s_end = sh.cut(sh.first + sh.pos + 1);
    }
    // encoded waves of this wavefront
    const int64_t share = s0 < s_end ? (uint32_t)(s_end - 1 - s0) / (uint32_t)stride + 1 : 0;
    if constexpr (LAYOUT == 2) {
        decode_lanes<VT, Sink, TF>(a, tb, lane, sp, s_end, s0, stride, share);
    } else {
        decode_rows<VT, Sink, TF>(a, tb, lane, sp, s_end, s0, stride, share);
    }
}

// MINW: waves per SIMD the register allocation must allow (8 lets two
// 16-wave workgroups share a CU, which is what the LDS tables permit).  Below
// 4 the workgroup is capped at 4 * MINW waves, so that the compiler may give
// a wave more than 128 registers.
constexpr int decode_max_threads(int minw) { return minw >= 4 ? 1024 : 256 * minw; }
template <int LAYOUT, typename VT, class Sink, int MINW, int TF>
__global__ __launch_bounds__(decode_max_threads(MINW), MINW) void decode_kernel(DevMat a, typename Sink::Params sp) {
    __shared__ __align__(16) Tables<VT> tb;
    decode_sweep<LAYOUT, VT, Sink, TF>(a, sp, tb);
}

// decode_kernel for CsrOut<VT, true>: up to 12 waves, whose exchange takes 75
// KiB of LDS beside the tables, one workgroup a CU.
constexpr int kXchWaves = 12;
template <typename VT>
__global__ __launch_bounds__(64 * kXchWaves, 3) void csr_rows_kernel(DevMat a, typename CsrOut<VT, true>::Params sp) {
    __shared__ __align__(16) Tables<VT> tb;
    extern __shared__ __align__(16) unsigned char s_dyn[];
    typedef CsrOut<VT, true> CO;
    typename CO::Params q = sp;
    q.xch = (uint32_t *)s_dyn + threadIdx.x / kWave * (kWave * CO::kLaneWords);
    decode_sweep<1, VT, CO, 2>(a, q, tb);
}

// decode_kernel for a single vector short enough to lie in LDS beside the
// tables of every resident workgroup: the gathers, whose cache lines the
// address unit takes one at a time, then are LDS reads, and a step waits on
// memory for its words alone (pruned 11008 x 4096 weight, FP32: 38.7 us, 41.9
// with gathers from L2; two workgroups of 12 waves a CU either way, bound by
// the step chain's latency and VALU issue; the reads of x add LDS bank
// conflicts, 5.2 M cycles in all against 3.4 M for the table lookups alone).
template <typename VT, int MINW, int TF>
__global__ __launch_bounds__(decode_max_threads(MINW), MINW) void decode_x_kernel(
    DevMat a, typename SpmmSink<VT, 1, true, double, 0, true>::Params sp) {
    __shared__ __align__(16) Tables<VT> tb;
    extern __shared__ __align__(16) unsigned char s_dyn[];
    VT *lx = (VT *)s_dyn;
    const uint32_t n = (uint32_t)a.n;
    for (uint32_t i = threadIdx.x; i < n; i += blockDim.x) lx[i] = ((gptr<VT>)sp.X)[i];
    // (the barrier that ends the staging of the tables orders these stores)
    typename SpmmSink<VT, 1, true, double, 0, true>::Params q = sp;
    q.lx = lx;
    decode_sweep<2, VT, SpmmSink<VT, 1, true, double, 0, true>, TF>(a, q, tb);
}

// The passes of a transposed product with dX privatised in LDS: pass p takes
// the columns of dY from (p / blocks) * width on (width of them, the last pass
// what is left) and the columns of A from (p % blocks) * cols on.
struct TransPlan {
    int64_t n;           // columns of A
    int32_t k;           // columns of dY
    int32_t width;       // columns of dY per pass
    int32_t blocks;      // column blocks of A
    int32_t cols, plane;  // columns of A per block; the same padded to a multiple of 32
    int32_t pass0, passes;  // passes of this launch: pass0 .. pass0 + passes
    __device__ __forceinline__ int32_t first(int32_t p) const { return p / blocks * width; }
    __device__ __forceinline__ int32_t columns(int32_t p) const { return min(width, k - first(p)); }
    __device__ __forceinline__ int32_t row0(int32_t p) const { return p % blocks * cols; }
    __device__ __forceinline__ int32_t rows(int32_t p) const { return (int32_t)min((int64_t)cols, n - row0(p)); }
};

// Transposed product with dX privatised in LDS: a workgroup (one per CU)
// scatters into its own block of dX with LDS atomic adds, then writes it to
// part[blockIdx.x]; trans_reduce_kernel sums the copies.  No global atomics,
// so no contention when n is small (the tall pruned weight: every column of
// dX receives thousands of contributions).  All passes run in one launch,
// workgroup b on pass b % passes with its share of the encoded waves: the
// copies to sum are then as many per pass as it has workgroups, and the
// tables are staged once per workgroup.  Bound by decoding the streams once
// per pass and by the LDS atomic adds (see TransLdsSink): pruned 11008 x 4096
// weight, k = 16, 6 passes of up to 3 columns: 0.356 ms, 31% of it bank
// conflicts in the LDS, reduction 5 us (FP32 adds in 4 passes of 4 columns: 4 x
// 0.64 ms, reductions 4 x 12 us).
template <int LAYOUT, typename VT, int KC, int TF>
__global__ __launch_bounds__(1024, 4) void trans_lds_kernel(DevMat a,
                                                            typename TransLdsSink<VT, KC>::Params sp,
                                                            TransPlan tp, VT *part) {
    __shared__ __align__(16) Tables<VT> tb;
    extern __shared__ __align__(16) unsigned char s_dyn[];
    typename TransLdsSink<VT, KC>::Params q = sp;
    q.lds = (double *)s_dyn;
    const int32_t pb = (int32_t)(blockIdx.x % (uint32_t)tp.passes), p = tp.pass0 + pb;
    q.dY += tp.first(p);
    q.width = (uint32_t)tp.columns(p);
    q.c0 = (uint32_t)tp.row0(p);
    q.cols = (uint32_t)tp.rows(p);
    q.plane = (uint32_t)tp.plane;
    const uint32_t slots = q.width * q.plane;
    for (uint32_t i = threadIdx.x; i < slots; i += blockDim.x) q.lds[i] = 0.0;
    // (the table staging inside the sweep ends with a barrier, which also
    // orders these stores before the first scatter)
    typedef TransLdsSink<VT, KC> Sink;
    const uint32_t lane = threadIdx.x & (kWave - 1);
    const int64_t wpb = blockDim.x / kWave;
    const int64_t groups = (gridDim.x - (uint32_t)pb + tp.passes - 1) / (uint32_t)tp.passes;  // of this pass
    // encoded waves are dealt to the pass's workgroups in turn, so that all of
    // them have the same number whatever there are (dealt by the workgroup, a
    // matrix of fewer waves than wavefronts left whole workgroups idle: 4096 x
    // 1000 at 30%, FP64, row layout, k = 8: 557 -> 167 us; pruned weight, k =
    // 16: 362 -> 345 us)
    const int64_t stride = groups * wpb;
    const int64_t s0 = blockIdx.x / (uint32_t)tp.passes + __builtin_amdgcn_readfirstlane(threadIdx.x / kWave) * groups;
    const int64_t share = s0 < a.num_waves ? (uint32_t)(a.num_waves - 1 - s0) / (uint32_t)stride + 1 : 0;
    if constexpr (LAYOUT == 2) {
        decode_lanes<VT, Sink, TF>(a, tb, lane, q, a.num_waves, s0, stride, share);
    } else {
        decode_rows<VT, Sink, TF>(a, tb, lane, q, a.num_waves, s0, stride, share);
    }
    __syncthreads();
    VT *dst = part + (int64_t)blockIdx.x * tp.width * tp.plane;
    for (uint32_t i = threadIdx.x; i < slots; i += blockDim.x) {
        const uint32_t c = i / q.plane, j = i - c * q.plane;
        dst[i] = (VT)q.lds[c * q.plane + lds_slot(j)];
    }
}

// dX = alpha * (sum of the copies of its pass) + beta * dX for the columns of
// this launch's passes; grid workgroups wrote the copies.  A thread per
// element, consecutive threads on consecutive rows of dX (elements of a plane).
template <typename VT>
__global__ __launch_bounds__(256) void trans_reduce_kernel(const VT *part, TransPlan tp, int32_t grid, VT *dX,
                                                           int64_t lddx, double alpha, double beta) {
    const int32_t pb = (int32_t)blockIdx.y, p = tp.pass0 + pb;
    const int32_t i = (int32_t)(blockIdx.x * blockDim.x + threadIdx.x);
    const int32_t c = i / tp.plane, j = i - c * tp.plane;
    if (c >= tp.columns(p) || j >= tp.rows(p)) return;
    const int64_t copy = (int64_t)tp.width * tp.plane, step = (int64_t)tp.passes * copy;
    const VT *q = part + (int64_t)pb * copy + i;
    const int32_t G = (grid - pb + tp.passes - 1) / tp.passes;
    double acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};  // eight loads in flight
    int32_t b = 0;
    for (; b + 8 <= G; b += 8)
#pragma unroll
        for (int u = 0; u < 8; ++u) acc[u] += (double)q[(b + u) * step];
    for (; b < G; ++b) acc[0] += (double)q[b * step];
    const double sum = ((acc[0] + acc[1]) + (acc[2] + acc[3])) + ((acc[4] + acc[5]) + (acc[6] + acc[7]));
    VT *d = dX + (int64_t)(tp.row0(p) + j) * lddx + tp.first(p) + c;
    *d = (VT)(beta == 0.0 ? alpha * sum : alpha * sum + beta * (double)*d);
}

// The symmetric product: each workgroup (one per CU) decodes one contiguous
// run of encoded waves, a round of one wave per wavefront at a time, and adds
// its sums to y after every kRounds rounds.  Global FP64 atomic adds bound
// the product (182 G a second when coalesced), so neighbouring rows first
// meet in LDS: on the 27-point stencil kRounds = 2 leaves about 2 of 14 adds
// per row.  96^3, FP64: 37 us and 5 us to start y, against 111 us for the
// product and the transposed product with global adds after each other; a
// random graph (R-MAT scale 18), whose elements mostly find no block: 190
// against 267 us.
template <int LAYOUT, typename VT, int TF>
__global__ __launch_bounds__(1024, 4) void sym_kernel(DevMat a, typename SymSink<VT>::Params sp) {
    __shared__ __align__(16) Tables<VT> tb;
    extern __shared__ __align__(16) unsigned char s_dyn[];
    constexpr int kRounds = 2;
    typename SymSink<VT>::Params q = sp;
    q.lds = s_dyn;
    const BlockSums sums(s_dyn);
    sums.clear();  // (the barrier that ends the staging orders it)
    const uint32_t lane = threadIdx.x & (kWave - 1);
    const int64_t wpb = blockDim.x / kWave;
    // neighbouring runs on the same XCD, as in decode_sweep
    const XcdShare sh(gridDim.x, blockIdx.x, (uint32_t)a.num_waves);
    const int64_t begin = sh.cut(sh.first + sh.pos), end = sh.cut(sh.first + sh.pos + 1);
    const int64_t rounds = (end - begin + wpb - 1) / wpb;
    int64_t s = begin + __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    // row layout: the next wave's geometry and offsets are loaded while this
    // one decodes (see decode_rows)
    auto clamp = [&](int64_t i) { return i < end ? i : (end > begin ? end - 1 : (int64_t)0); };
    LaneGeo geo = lane_geo<LAYOUT>(a, clamp(s), lane, lane_first_row<LAYOUT>(a, clamp(s), lane));
    stage_tables<VT>(a, tb, 1u);
    for (int64_t i = 0; i < rounds; ++i, s += wpb) {
        if (s < end) {
            const LaneGeo next = lane_geo<LAYOUT>(a, clamp(s + wpb), lane, lane_first_row<LAYOUT>(a, clamp(s + wpb), lane));
            const WaveSpan<false> span(a, s);
            GlobalWords src = span.words(a);
            Cursor<VT> cur = span.template cursor<VT>(a);
            decode_slice<LAYOUT, VT, SymSink<VT>, GlobalWords, TF>(a, tb, s, lane, q, src, cur, geo);
            geo = next;
        }
        if (i % kRounds == kRounds - 1 || i == rounds - 1) {  // uniform over the workgroup
            __syncthreads();
            sums.flush(q.y, q.alpha);
            __syncthreads();
        }
    }
}

// Same work as decode_kernel, with every wavefront owning one contiguous run
// of encoded waves (so that its streams are adjacent in memory) and reading
// them through an LDS ring (RingWords).  The XCD shares are those of
// decode_kernel; inside a share the runs are consecutive, which keeps the
// rows an XCD works on within a window of its share.
template <int LAYOUT, typename VT, class Sink, int MINW, int TF>
__global__ __launch_bounds__(1024, MINW) void ring_kernel(DevMat a, typename Sink::Params sp) {
    __shared__ __align__(16) Tables<VT> tb;
    extern __shared__ uint32_t s_ring[];  // RingWords<kRingWords>::kWords per wavefront
    stage_tables<VT>(a, tb, Sink::col_scale(sp));
    const uint32_t lane = threadIdx.x & (kWave - 1);
    const int64_t wpb = blockDim.x / kWave;
    const int64_t wib = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int64_t G = gridDim.x, xcd = blockIdx.x % kNumXcd, pos_in_xcd = blockIdx.x / kNumXcd;
    const int64_t q = G / kNumXcd, rr = G % kNumXcd;
    const int64_t xcd_blocks = q + (xcd < rr ? 1 : 0);
    const int64_t xcd_first = xcd * q + (xcd < rr ? xcd : rr);
    const int64_t total = G * wpb;
    const int64_t s_begin = xcd_first * wpb * a.num_waves / total;
    const int64_t s_end = (xcd_first + xcd_blocks) * wpb * a.num_waves / total;
    const int64_t nw = xcd_blocks * wpb, widx = pos_in_xcd * wpb + wib;
    const int64_t sa = s_begin + widx * (s_end - s_begin) / nw;
    const int64_t sb = s_begin + (widx + 1) * (s_end - s_begin) / nw;
    if (sa >= sb) return;
    RingWords<kRingWords> src;
    const uint64_t w0 = a.woff[sa];
    src.start(s_ring + wib * RingWords<kRingWords>::kWords, a.words + w0,
              (uint32_t)(4 * (a.woff[sb] - w0)), lane);
    Cursor<VT> cur{0, 0, 0, a.escd + a.doff[sa], (const VT *)a.escv + a.voff[sa]};
    // lane geometry two stages ahead: first rows of wave s + 2 and row
    // pointers of wave s + 1 are loaded while wave s decodes
    LaneGeo geo = lane_geo<LAYOUT>(a, sa, lane, lane_first_row<LAYOUT>(a, sa, lane));
    int32_t fr1 = sa + 1 < sb ? lane_first_row<LAYOUT>(a, sa + 1, lane) : 0;
    for (int64_t s = sa; s < sb; ++s) {
        const int32_t fr2 = s + 2 < sb ? lane_first_row<LAYOUT>(a, s + 2, lane) : 0;
        const int64_t s1 = s + 1 < sb ? s + 1 : s;
        const LaneGeo next = lane_geo<LAYOUT>(a, s1, lane, s + 1 < sb ? fr1 : (LAYOUT == 2 ? geo.krow : geo.row));
        decode_slice<LAYOUT, VT, Sink, RingWords<kRingWords>, TF>(a, tb, s, lane, sp, src, cur, geo);
        geo = next;
        fr1 = fr2;
    }
}

// rows split over lanes (layout NNZ): y = alpha * (tail of the first lane +
// heads of the following lanes) + beta * y.  A row spanning at most
// kLongSplit (kLongSplitRuns) following lanes is summed by one thread
// (fixup_short); a longer one by a whole wavefront (fixup_long, rows
// listed on the host): its lanes stride over the row's partials, one running
// sum per column, then a butterfly reduction per column.
constexpr int kMaxFixupCols = 32;

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
    return v;
}

template <typename VT>
__device__ __forceinline__ void fixup_put(VT *Y, int64_t ldy, int32_t row, int c, double sum,
                                          double alpha, double beta) {
    VT *y = Y + (int64_t)row * ldy + c;
    *y = (VT)(beta == 0.0 ? alpha * sum : alpha * sum + beta * (double)*y);
}

// runs: the middle lanes' pieces were summed per wavefront (finish_lane), so
// of the lanes strictly between the first (a) and the last (b) only the one
// after the first and those starting a wavefront hold a partial; the first
// wavefront start after a + 1:
__device__ __forceinline__ int64_t first_run_start(int32_t a) { return ((int64_t)(a + 1) | (kWave - 1)) + 1; }

template <typename VT>
__device__ __forceinline__ void fixup_short(const SplitRows &sr, const double *partial, int KC, int runs, VT *Y,
                                            int64_t ldy, double alpha, double beta, int log_tpr, int64_t block) {
    // 2^log_tpr >= KC threads per split row, one column each (consecutive
    // threads read consecutive doubles of a partial slot)
    const int64_t s = (block * blockDim.x + threadIdx.x) >> log_tpr;
    const int c = (int)(threadIdx.x & ((1u << log_tpr) - 1));
    if (s >= sr.n || c >= KC) return;
    const int32_t a = sr.first[s], b = sr.last[s];
    if (b - a > (runs ? kLongSplitRuns : kLongSplit)) return;
    {
        const double *head = partial + c;  // head slot of lane l: head[2 * l * KC]
        double sum = partial[(2 * (int64_t)a + 1) * KC + c];
        if (runs) {
            sum += head[2 * (int64_t)(a + 1) * KC];
            for (int64_t l = first_run_start(a); l < b; l += kWave) sum += head[2 * l * KC];
            if (b > a + 1) sum += head[2 * (int64_t)b * KC];
        } else {
            for (int64_t l = a + 1; l <= b; ++l) sum += head[2 * l * KC];
        }
        fixup_put(Y, ldy, sr.row[s], c, sum, alpha, beta);
    }
}

template <typename VT>
__device__ __forceinline__ void fixup_long(const SplitRows &sr, const double *partial, int KC, int runs, VT *Y,
                                           int64_t ldy, double alpha, double beta, int64_t block) {
    const int64_t w = (block * blockDim.x + threadIdx.x) / kWave;
    const int lane = (int)(threadIdx.x & (kWave - 1));
    if (w >= sr.n_long) return;  // whole wavefronts
    const int64_t s = sr.longs[w];
    const int32_t a = sr.first[s], b = sr.last[s];
    double acc[kMaxFixupCols];
#pragma unroll
    for (int c = 0; c < kMaxFixupCols; ++c) acc[c] = 0.0;
    auto add = [&](const double *q) {
#pragma unroll
        for (int c = 0; c < kMaxFixupCols; ++c)
            if (c < KC) acc[c] += q[c];
    };
    if (runs) {
        // lane 0: the tail of lane a and the head of lane a + 1; lane 1: the
        // head of lane b; all lanes: the wavefront starts in between
        if (lane == 0) {
            add(partial + (2 * (int64_t)a + 1) * KC);
            add(partial + 2 * (int64_t)(a + 1) * KC);
        }
        if (lane == 1) add(partial + 2 * (int64_t)b * KC);
        for (int64_t l = first_run_start(a) + (int64_t)lane * kWave; l < b; l += (int64_t)kWave * kWave)
            add(partial + 2 * l * KC);
    } else {
        for (int64_t l = (int64_t)a + lane; l <= b; l += kWave)
            add(partial + (2 * l + (l == a ? 1 : 0)) * KC);  // tail of lane a, heads after
    }
#pragma unroll
    for (int c = 0; c < kMaxFixupCols; ++c)
        if (c < KC) {
            const double sum = wave_sum(acc[c]);
            if (lane == c) fixup_put(Y, ldy, sr.row[s], c, sum, alpha, beta);
        }
}

// What follows a product in the nonzero layouts, in one launch: the long split
// rows (they take longest, so their workgroups come first), the other split
// rows, and y = beta * y on the rows without nonzeros (never decoded).  The
// three write different rows of Y.  (A launch each cost R-MAT scale 22 25 us
// of 620, and smaller graphs as much.)
template <typename VT>
__global__ __launch_bounds__(256) void epilogue_kernel(SplitRows sr, const int32_t *empty, int64_t n_empty,
                                                       const double *partial, int KC, int runs, VT *Y, int64_t ldy,
                                                       double alpha, double beta, int log_tpr, uint32_t long_blocks,
                                                       uint32_t short_blocks) {
    if (blockIdx.x < long_blocks) {
        fixup_long<VT>(sr, partial, KC, runs, Y, ldy, alpha, beta, blockIdx.x);
    } else if (blockIdx.x < long_blocks + short_blocks) {
        fixup_short<VT>(sr, partial, KC, runs, Y, ldy, alpha, beta, log_tpr, blockIdx.x - long_blocks);
    } else {
        const int64_t i = (int64_t)(blockIdx.x - long_blocks - short_blocks) * blockDim.x + threadIdx.x;
        if (i >= n_empty * KC) return;
        VT *y = Y + (int64_t)empty[i / KC] * ldy + i % KC;
        *y = beta == 0.0 ? (VT)0 : (VT)(beta * (double)*y);
    }
}

// the epilogue for KC <= kMaxFixupCols columns of Y
template <typename VT>
hipError_t launch_epilogue(const SplitRows &sr, const int32_t *empty, int64_t n_empty, const double *partial, int KC,
                           int runs, VT *Y, int64_t ldy, double alpha, double beta, hipStream_t st) {
    if (sr.n == 0 && n_empty == 0) return hipSuccess;
    if (KC > kMaxFixupCols) return hipErrorInvalidValue;
    int lt = 0;
    while ((1 << lt) < KC) ++lt;
    const int64_t nl = sr.n ? (sr.n_long + 3) / 4 : 0, ns = ((sr.n << lt) + 255) / 256, ne = (n_empty * KC + 255) / 256;
    hipLaunchKernelGGL(epilogue_kernel<VT>, dim3((unsigned)(nl + ns + ne)), dim3(256), 0, st, sr, empty, n_empty,
                       partial, KC, runs, Y, ldy, alpha, beta, lt, (uint32_t)nl, (uint32_t)ns);
    return hipGetLastError();
}

// Y[rows, :KC] = beta * Y (beta == 0: zero)
template <typename VT>
__global__ void scale_kernel(VT *Y, int64_t rows, int KC, int64_t ldy, double beta) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= rows * KC) return;
    VT *y = Y + (i / KC) * ldy + i % KC;
    *y = beta == 0.0 ? (VT)0 : (VT)(beta * (double)*y);
}

__global__ __launch_bounds__(256) void flush_kernel(const uint4 *p, int64_t n, uint32_t *sink) {
    uint32_t acc = 0;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x) {
        const uint4 v = p[i];
        acc ^= v.x ^ v.y ^ v.z ^ v.w;
    }
    if (acc == 0x9e3779b9u) sink[0] = acc;  // keeps the loads; the buffer is zero
}

// ------------------------------------------------- multi-matrix launch
template <typename VT>
__global__ __launch_bounds__(1024, 7) void batch_kernel(BatchDev b, double alpha, double beta) {
    __shared__ __align__(16) Tables<VT> tb;
    const uint32_t lane = threadIdx.x & (kWave - 1);
    const int wib = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), wpb = blockDim.x / kWave;
    const int t0 = b.wg_task[blockIdx.x], t1 = b.wg_task[blockIdx.x + 1];
    int cur = -1;
    for (int t = t0; t < t1; ++t) {
        const BatchTask task = b.tasks[t];
        const DevMat a = b.mats[task.mat];  // uniform: scalar loads into SGPRs
        // the tables are restaged only when the matrix changes
        const int stage = task.mat == cur ? 0 : (cur < 0 ? 1 : 2);
        cur = task.mat;
        typename SpmmSink<VT, 1, true>::Params sp;
        sp.X = (const VT *)b.ptrs[2 * task.mat];
        sp.ldx = 1;
        sp.Y = (VT *)b.ptrs[2 * task.mat + 1];
        sp.ldy = 1;
        sp.partial = nullptr;
        sp.alpha = alpha;
        sp.beta = beta;
        sp.pair_x = a.n >= 2;
        // this wavefront's waves of the task: first_wave + wib, + wpb, ...
        const int64_t s0 = task.first_wave + wib, s_end = (int64_t)task.first_wave + task.num_waves;
        const int64_t share = s0 < s_end ? (s_end - 1 - s0) / wpb + 1 : 0;
        if (a.base_direct)
            decode_rows<VT, SpmmSink<VT, 1, true>, 1>(a, tb, lane, sp, s_end, s0, wpb, share, stage);
        else
            decode_rows<VT, SpmmSink<VT, 1, true>, 0>(a, tb, lane, sp, s_end, s0, wpb, share, stage);
    }
}

// The same launch for k right-hand sides: X_i is n_i x k and Y_i m_i x k, row
// major with leading dimension k; this launch takes the columns c0 .. c0 + KC
// of every matrix (the sink's chunk), each matrix decoded once per launch.
template <typename VT, class Sink, int MINW>
__global__ __launch_bounds__(decode_max_threads(MINW), MINW) void batch_spmm_kernel(BatchDev b, int c0, int k,
                                                                                     double alpha, double beta) {
    __shared__ __align__(16) Tables<VT> tb;
    const uint32_t lane = threadIdx.x & (kWave - 1);
    const int wib = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), wpb = blockDim.x / kWave;
    const int t0 = b.wg_task[blockIdx.x], t1 = b.wg_task[blockIdx.x + 1];
    int cur = -1;
    for (int t = t0; t < t1; ++t) {
        const BatchTask task = b.tasks[t];
        const DevMat a = b.mats[task.mat];
        const int stage = task.mat == cur ? 0 : (cur < 0 ? 1 : 2);
        cur = task.mat;
        typename Sink::Params sp;
        sp.X = (const VT *)b.ptrs[2 * task.mat] + c0;
        sp.ldx = (uint32_t)k;
        sp.Y = (VT *)b.ptrs[2 * task.mat + 1] + c0;
        sp.ldy = (uint32_t)k;
        sp.partial = nullptr;  // row layout: every row ends in its lane
        sp.alpha = alpha;
        sp.beta = beta;
        const int64_t s0 = task.first_wave + wib, s_end = (int64_t)task.first_wave + task.num_waves;
        const int64_t share = s0 < s_end ? (s_end - 1 - s0) / wpb + 1 : 0;
        if (a.base_direct)
            decode_rows<VT, Sink, 1>(a, tb, lane, sp, s_end, s0, wpb, share, stage);
        else
            decode_rows<VT, Sink, 0>(a, tb, lane, sp, s_end, s0, wpb, share, stage);
    }
}

// ------------------------------------------------------- plain CSR
// variant 1: G lanes per row (G a power of two <= 64), lanes of a group read
// consecutive nonzeros; butterfly reduction inside the group.
template <typename VT, int G, int KC>
__global__ __launch_bounds__(256) void csr_vector_kernel(CsrDev c, const VT *__restrict__ X,
                                                         int64_t ldx, VT *__restrict__ Y,
                                                         int64_t ldy, double alpha, double beta) {
    const int64_t tid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t nthreads = (int64_t)gridDim.x * blockDim.x;
    const int q = threadIdx.x % G;
    const VT *__restrict__ val = (const VT *)c.val;
    for (int64_t row = tid / G; row < c.m; row += nthreads / G) {
        const int32_t b = c.row_ptr[row], e = c.row_ptr[row + 1];
        double acc[KC];
#pragma unroll
        for (int k = 0; k < KC; ++k) acc[k] = 0.0;
        for (int32_t i = b + q; i < e; i += G) {
            const VT v = val[i];
            const VT *x = X + (int64_t)c.col[i] * ldx;
#pragma unroll
            for (int k = 0; k < KC; ++k) acc[k] = fma((double)v, (double)x[k], acc[k]);
        }
#pragma unroll
        for (int k = 0; k < KC; ++k) {
#pragma unroll
            for (int off = G / 2; off > 0; off >>= 1) acc[k] += __shfl_xor(acc[k], off, G);
        }
        if (q == 0) {
            VT *y = Y + row * ldy;
#pragma unroll
            for (int k = 0; k < KC; ++k)
                y[k] = (VT)(beta == 0.0 ? alpha * acc[k] : alpha * acc[k] + beta * (double)y[k]);
        }
    }
}

// variant 2: lane_nnz consecutive nonzeros per lane, rows tracked through
// row_ptr, partial sums of rows that cross lanes go to `partial`.
template <typename VT, int KC>
__global__ __launch_bounds__(256) void csr_split_kernel(CsrDev c, const VT *__restrict__ X,
                                                        int64_t ldx, VT *__restrict__ Y,
                                                        int64_t ldy, double alpha, double beta,
                                                        double *partial) {
    const int64_t l = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (l >= c.num_lanes) return;
    const VT *__restrict__ val = (const VT *)c.val;
    const int64_t g0 = l * (int64_t)c.lane_nnz;
    const int64_t gend = min(g0 + c.lane_nnz, c.nnz);
    int32_t row = c.lane_row[l];
    int32_t row_beg = c.row_ptr[row], row_end = c.row_ptr[row + 1];
    double acc[KC];
#pragma unroll
    for (int k = 0; k < KC; ++k) acc[k] = 0.0;
    auto done = [&](int kind) {
        if (kind == kComplete) {
            VT *y = Y + (int64_t)row * ldy;
#pragma unroll
            for (int k = 0; k < KC; ++k)
                y[k] = (VT)(beta == 0.0 ? alpha * acc[k] : alpha * acc[k] + beta * (double)y[k]);
        } else {
            double *q = partial + (2 * l + (kind == kTail ? 1 : 0)) * KC;
#pragma unroll
            for (int k = 0; k < KC; ++k) q[k] = acc[k];
        }
#pragma unroll
        for (int k = 0; k < KC; ++k) acc[k] = 0.0;
    };
    for (int64_t g = g0; g < gend; ++g) {
        while (g >= row_end) {
            done(row_beg < g0 ? kHead : kComplete);
            ++row;
            row_beg = row_end;
            row_end = c.row_ptr[row + 1];
        }
        const VT v = val[g];
        const VT *x = X + (int64_t)c.col[g] * ldx;
#pragma unroll
        for (int k = 0; k < KC; ++k) acc[k] = fma((double)v, (double)x[k], acc[k]);
    }
    while (row < c.m && row_end <= gend) {
        done(row_beg < g0 ? kHead : kComplete);
        ++row;
        row_beg = row_end;
        if (row < c.m) row_end = c.row_ptr[row + 1];
    }
    if (row < c.m && row_beg < gend) done(row_beg < g0 ? kHead : kTail);
}

// variant 3 (SpMV): CSR-stream.  A workgroup takes a block of consecutive
// rows holding at most kStreamNnz nonzeros, loads their column indices and
// values coalesced (four per thread, all x gathers in flight together),
// stages the products in LDS and sums each row from LDS.  A block that is a
// single row longer than that is reduced across the workgroup instead.
constexpr int kStreamNnz = 1024;
template <typename VT>
__global__ __launch_bounds__(256) void csr_stream_kernel(CsrDev c, const int32_t *__restrict__ blk,
                                                         const VT *__restrict__ x, VT *__restrict__ y,
                                                         double alpha, double beta) {
    __shared__ double prod[kStreamNnz];
    __shared__ double red[4];
    const int r0 = blk[blockIdx.x], r1 = blk[blockIdx.x + 1];
    const int32_t g0 = c.row_ptr[r0], g1 = c.row_ptr[r1];
    const VT *__restrict__ val = (const VT *)c.val;
    const int32_t *__restrict__ col = c.col;
    const int tid = threadIdx.x;
    if (g1 - g0 > kStreamNnz) {  // one long row
        double s = 0.0;
        for (int32_t base = g0; base < g1; base += 4 * 256) {
            VT v[4], xv[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int32_t i = base + u * 256 + tid;
                v[u] = i < g1 ? val[i] : (VT)0;
                xv[u] = i < g1 ? x[col[i]] : (VT)0;
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) s = fma((double)v[u], (double)xv[u], s);
        }
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off);
        if ((tid & 63) == 0) red[tid >> 6] = s;
        __syncthreads();
        if (tid == 0) {
            const double t = red[0] + red[1] + red[2] + red[3];
            y[r0] = (VT)(beta == 0.0 ? alpha * t : alpha * t + beta * (double)y[r0]);
        }
        return;
    }
    const int32_t cnt = g1 - g0;
    VT v[4], xv[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int32_t i = u * 256 + tid;
        if (i < cnt) {
            v[u] = val[g0 + i];
            xv[u] = x[col[g0 + i]];
        }
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int32_t i = u * 256 + tid;
        if (i < cnt) prod[i] = (double)v[u] * (double)xv[u];
    }
    __syncthreads();
    for (int r = r0 + tid; r < r1; r += 256) {
        const int32_t b = c.row_ptr[r] - g0, e = c.row_ptr[r + 1] - g0;
        double s = 0.0;
        for (int32_t i = b; i < e; ++i) s += prod[i];
        y[r] = (VT)(beta == 0.0 ? alpha * s : alpha * s + beta * (double)y[r]);
    }
}

// ------------------------------------------------------------ dispatch
template <class T> struct TypeBox { typedef T type; };

// the nonzero-balanced layout tracks rows and needs more registers: six waves
// per SIMD, which is what its workgroup shapes keep resident
constexpr int occ_nnz(int occ) { return occ > 6 ? 6 : occ; }

template <typename F>
hipError_t for_kc(int k, int kcmax, F f);
template <typename F>
hipError_t for_kc(int k, F f) {
    return for_kc(k, kMaxPassCols, f);
}
template <typename F>
hipError_t for_kc(int k, int kcmax, F f) {
    // split k columns into compile-time chunks of at most kcmax
    int c0 = 0;
    while (c0 < k) {
        int left = k - c0 < kcmax ? k - c0 : kcmax;
        hipError_t e;
        if (left >= 32) { e = f(std::integral_constant<int, 32>(), c0); c0 += 32; }
        else if (left >= 16) { e = f(std::integral_constant<int, 16>(), c0); c0 += 16; }
        else if (left >= 8) { e = f(std::integral_constant<int, 8>(), c0); c0 += 8; }
        else if (left >= 4) { e = f(std::integral_constant<int, 4>(), c0); c0 += 4; }
        else if (left >= 2) { e = f(std::integral_constant<int, 2>(), c0); c0 += 2; }
        else { e = f(std::integral_constant<int, 1>(), c0); c0 += 1; }
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// layout NNZ after the decode: rows split over lanes, and rows without
// nonzeros (both only write y)
template <typename VT>
hipError_t nnz_epilogue(const DevMat &a, const double *partial, int KC, VT *Y, int64_t ldy,
                        double alpha, double beta, hipStream_t st) {
    return launch_epilogue(a.split, a.empty_rows, a.n_empty, partial, KC, 1, Y, ldy, alpha, beta, st);
}

// the kernel instance for the matrix's table format
template <typename K>
K pick_bd(const DevMat &a, K direct, K general) {
    return a.base_direct ? direct : general;
}
template <typename K>
K pick_tf(const DevMat &a, K direct_noesc, K direct, K general) {
    return a.base_direct ? (a.no_escape ? direct_noesc : direct) : general;
}

// Launch of a persistent direct-read decode kernel.  Unless the caller fixed
// the shape, the workgroup size (16, 12, 8 or 4 waves: multiples of the
// CU's 4 SIMDs) is the one that keeps the most wavefronts resident according
// to the runtime's occupancy for this kernel, whose registers and LDS both
// limit it (a 12-wave workgroup of a kernel that fits 4 waves per SIMD would
// leave a CU with one workgroup, 3 waves per SIMD); cached per kernel.
struct Shape {
    int wpw, per_cu;
};
template <typename K>
Shape fit_shape(K kern, const Launch &L) {
    // the occupancy query does not know the kernel's workgroup-size bound, and
    // a fixed shape may exceed it (kernels that need more than 128 registers)
    auto max_threads = [&]() {
        hipFuncAttributes fa;
        return hipFuncGetAttributes(&fa, (const void *)kern) == hipSuccess ? fa.maxThreadsPerBlock : 1024;
    };
    if (L.fixed_shape)
        return Shape{std::min(L.waves_per_wg, max_threads() / 64), std::max(1, (L.grid + L.num_cus - 1) / L.num_cus)};
    static std::mutex mu;
    static std::vector<std::pair<const void *, Shape>> cache;
    const void *key = (const void *)kern;
    std::lock_guard<std::mutex> lock(mu);
    for (const auto &c : cache)
        if (c.first == key) return c.second;
    const int mt = max_threads();
    Shape best{L.waves_per_wg, std::max(1, (L.grid + L.num_cus - 1) / L.num_cus)};
    int best_res = 0;
    for (int w : {16, 12, 8, 4}) {
        int nb = 0;
        if (64 * w > mt) continue;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, kern, 64 * w, 0) != hipSuccess) continue;
        if (nb * w > best_res) {
            best_res = nb * w;
            best = Shape{w, nb};
        }
    }
    cache.emplace_back(key, best);
    return best;
}

// Wavefronts of the one workgroup a CU of a kernel whose LDS admits no second
// one: as many as a caller's shape keeps on a CU, `most` otherwise.
int lone_group_waves(const Launch &L, int most) {
    if (!L.fixed_shape) return most;
    return std::min(most, L.waves_per_wg * std::max(1, (L.grid + L.num_cus - 1) / L.num_cus));
}

template <typename K, typename... Args>
hipError_t launch_persistent(K kern, const DevMat &a, const Launch &L, hipStream_t st, Args... args) {
    const Shape sh = fit_shape(kern, L);
    // small matrices: four encoded waves (one per SIMD) to a workgroup, up to a
    // workgroup for every CU; its other wavefronts only help to stage the
    // tables (31 waves of a 4096 x 4096 band, FP64: 17 us on 8 CUs, 20 us on 3)
    const int64_t need = std::max((a.num_waves + sh.wpw - 1) / sh.wpw,
                                  a.num_waves <= L.max_spread ? std::min<int64_t>((a.num_waves + 3) / 4, L.num_cus) : 0);
    const int64_t grid = L.fixed_shape ? L.grid : std::min<int64_t>((int64_t)L.num_cus * sh.per_cu, need);
    hipLaunchKernelGGL(kern, dim3((unsigned)std::max<int64_t>(1, grid)), dim3(64 * sh.wpw), 0, st, args...);
    return hipGetLastError();
}

template <typename VT>
hipError_t spmm_impl(const DevMat &a, int k, const VT *X, int64_t ldx, VT *Y, int64_t ldy,
                     double alpha, double beta, double *partial, Launch L, hipStream_t st) {
    if (a.nnz == 0 || a.num_waves == 0) {
        if (a.m == 0) return hipSuccess;
        return for_kc(k, [&](auto KCc, int c0) {
            constexpr int KC = decltype(KCc)::value;
            int64_t tot = a.m * KC;
            hipLaunchKernelGGL(scale_kernel<VT>, dim3((unsigned)((tot + 255) / 256)), dim3(256), 0,
                               st, Y + c0, a.m, KC, ldy, beta);
            return hipGetLastError();
        });
    }
    auto launch_kernel = [&](auto sinkc, auto kern, int KC, int c0) -> hipError_t {
        typedef typename decltype(sinkc)::type SinkT;
        typename SinkT::Params sp;
        sp.X = X + c0;
        sp.ldx = (uint32_t)ldx;
        sp.Y = Y + c0;
        sp.ldy = (uint32_t)ldy;
        sp.partial = partial;
        sp.alpha = alpha;
        sp.beta = beta;
        hipError_t e = launch_persistent(kern, a, L, st, a, sp);
        if (e != hipSuccess || a.layout != 2) return e;
        return nnz_epilogue(a, partial, KC, Y + c0, ldy, alpha, beta, st);
    };
    auto launch = [&](auto sinkc, int KC, int c0) -> hipError_t {
        typedef typename decltype(sinkc)::type SinkT;
        return launch_kernel(sinkc,
                             a.layout == 1 ? pick_bd(a, decode_kernel<1, VT, SinkT, SinkT::kOcc, 1>,
                                                     decode_kernel<1, VT, SinkT, SinkT::kOcc, 0>)
                                           : pick_bd(a, decode_kernel<2, VT, SinkT, occ_nnz(SinkT::kOcc), 1>,
                                                     decode_kernel<2, VT, SinkT, occ_nnz(SinkT::kOcc), 0>),
                             KC, c0);
    };
    // 32 FP32 columns of a matrix with long rows, nonzero layout.  Steps
    // without row ends have to prevail and a wavefront's start and end, which
    // spill, to be a small part of its work.  Against the general step, 2^25
    // nonzeros and more: rows of 512 0.98, 1024 1.02 to 1.04, 2048 1.04 to 1.09
    // times as fast; 22 M: rows of 512 0.97, 1024 and more 1.00 to 1.06; 6 M:
    // 0.92 to 0.97, rows of 2048 1.05 or 0.95; rows of 4, 6 M: 0.67.
    const bool straight = sizeof(VT) == 4 && a.layout == 2 && a.nnz >= (1ll << 24) && a.nnz >= 1024 * a.m;
    auto launch_straight = [&](int c0) -> hipError_t {
        if constexpr (sizeof(VT) == 4) {
            typedef CoopSpmmSink<VT, 8, double, true> SinkT;
            return launch_kernel(TypeBox<SinkT>(), pick_bd(a, decode_kernel<2, VT, SinkT, occ_nnz(SinkT::kOcc), 1>,
                                                           decode_kernel<2, VT, SinkT, occ_nnz(SinkT::kOcc), 0>),
                                 32, c0);
        } else {
            return hipErrorInvalidValue;  // not reached
        }
    };
    // LDS-ring kernels: deferred products, at most 2 (FP64) / 4 (FP32) columns
    // per pass so that the deferred x values stay in registers
    auto ring = [&](auto sinkc, auto kern, int KC, int c0) -> hipError_t {
        typedef typename decltype(sinkc)::type SinkT;
        typename SinkT::Params sp;
        sp.X = X + c0;
        sp.ldx = (uint32_t)ldx;
        sp.Y = Y + c0;
        sp.ldy = (uint32_t)ldy;
        sp.partial = partial;
        sp.alpha = alpha;
        sp.beta = beta;
        const int rw = L.ring_waves_per_wg;
        const dim3 rblock(64 * rw);
        const size_t lds = (size_t)rw * RingWords<kRingWords>::kWords * 4;
        int per_cu = L.wg_per_cu;
        if (per_cu <= 0) {
            hipError_t e = hipFuncSetAttribute((const void *)kern,
                                               hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
            if (e != hipSuccess) return e;
            e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kern, (int)rblock.x, lds);
            if (e != hipSuccess) return e;
            per_cu = per_cu > 0 ? per_cu : 1;
        }
        const int64_t need = (a.num_waves + rw - 1) / rw;
        const int grid = (int)std::max<int64_t>(1, std::min<int64_t>((int64_t)L.num_cus * per_cu, need));
        hipLaunchKernelGGL(kern, dim3(grid), rblock, lds, st, a, sp);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess || a.layout != 2) return e;
        return nnz_epilogue(a, partial, KC, Y + c0, ldy, alpha, beta, st);
    };
    const bool unit = k == 1 && ldx == 1 && ldy == 1 && a.n * (int64_t)sizeof(VT) <= (1ll << 32);
    if (L.ring) {
        if (unit) {
            typedef SpmmSink<VT, 1, true, double, 1> RowSink;
            typedef SpmmSink<VT, 1, true, double, 2> NnzSink;
            if (a.layout == 1)
                return ring(TypeBox<RowSink>(), pick_bd(a, ring_kernel<1, VT, RowSink, 4, 1>,
                                                        ring_kernel<1, VT, RowSink, 4, 0>), 1, 0);
            return ring(TypeBox<NnzSink>(), pick_bd(a, ring_kernel<2, VT, NnzSink, 4, 1>,
                                                    ring_kernel<2, VT, NnzSink, 4, 0>), 1, 0);
        }
        return for_kc(k, std::is_same<VT, double>::value ? 2 : 4, [&](auto KCc, int c0) {
            constexpr int KC = decltype(KCc)::value;
            if constexpr (KC > 4 || (std::is_same<VT, double>::value && KC > 2)) {
                return hipErrorInvalidValue;  // excluded by the chunk limit
            } else {
                typedef SpmmSink<VT, KC, false, double, 1> RowSink;
                typedef SpmmSink<VT, KC, false, double, 2> NnzSink;
                if (a.layout == 1)
                    return ring(TypeBox<RowSink>(), pick_bd(a, ring_kernel<1, VT, RowSink, 4, 1>,
                                                            ring_kernel<1, VT, RowSink, 4, 0>),
                                KC, c0);
                return ring(TypeBox<NnzSink>(), pick_bd(a, ring_kernel<2, VT, NnzSink, 4, 1>,
                                                        ring_kernel<2, VT, NnzSink, 4, 0>),
                            KC, c0);
            }
        });
    }
    if (unit) {
        // single vectors also have instances without escape handling
        typedef SpmmSink<VT, 1, true> SinkT;
        typename SinkT::Params sp;
        sp.X = X;
        sp.ldx = 1;
        sp.Y = Y;
        sp.ldy = 1;
        sp.partial = partial;
        sp.alpha = alpha;
        sp.beta = beta;
        sp.pair_x = a.n >= 2;
        if constexpr (sizeof(VT) == 4) {
            // x beside the tables in every workgroup of 12 waves, two a CU
            // (80 KiB each): where it fits it was the faster one for every
            // matrix measured.  64 to 1,000,000 rows, 512 to 4096 columns, rows
            // of 8, 32 and 256, scattered or in runs of up to 64 adjacent
            // columns (where the paired gathers save most): 0.82 to 0.95 of the
            // time with gathers from 2 M nonzeros on, and none of 110 matrices
            // down to a single encoded wave slower than before.
            const size_t dyn = (size_t)a.n * sizeof(VT);
            if (a.layout == 2 && !L.fixed_shape && sizeof(Tables<VT>) + dyn <= 80 * 1024) {
                typedef SpmmSink<VT, 1, true, double, 0, true> XSink;
                typename XSink::Params sx;
                sx.X = X;
                sx.ldx = 1;
                sx.Y = Y;
                sx.ldy = 1;
                sx.partial = partial;
                sx.alpha = alpha;
                sx.beta = beta;
                auto kern = pick_tf(a, decode_x_kernel<VT, 6, 2>, decode_x_kernel<VT, 6, 1>, decode_x_kernel<VT, 6, 0>);
                const int64_t need = std::max((a.num_waves + 11) / 12, std::min<int64_t>((a.num_waves + 3) / 4, L.num_cus));
                const int64_t grid = std::min<int64_t>(2ll * L.num_cus, need);
                hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(768), dyn, st, a, sx);
                hipError_t e = hipGetLastError();
                if (e != hipSuccess) return e;
                return nnz_epilogue(a, partial, 1, Y, ldy, alpha, beta, st);
            }
        }
        constexpr int occ = SinkT::kOcc, occn = occ_nnz(SinkT::kOcc);
        hipError_t e =
            a.layout == 1
                ? launch_persistent(pick_tf(a, decode_kernel<1, VT, SinkT, occ, 2>, decode_kernel<1, VT, SinkT, occ, 1>,
                                            decode_kernel<1, VT, SinkT, occ, 0>),
                                    a, L, st, a, sp)
                : launch_persistent(pick_tf(a, decode_kernel<2, VT, SinkT, occn, 2>, decode_kernel<2, VT, SinkT, occn, 1>,
                                            decode_kernel<2, VT, SinkT, occn, 0>),
                                    a, L, st, a, sp);
        if (e != hipSuccess || a.layout != 2) return e;
        return nnz_epilogue(a, partial, 1, Y, ldy, alpha, beta, st);
    }
    // Several columns: groups of lanes share each row of X (CoopSpmmSink) when
    // its rows can be read as aligned 16-byte pieces at 32-bit byte offsets;
    // chunks of 32 / 16 / 8 FP32 or 16 / 8 / 4 FP64 columns, the rest as below.
    const bool coop = (uintptr_t)X % 16 == 0 && (ldx * (int64_t)sizeof(VT)) % 16 == 0 &&
                      a.n * ldx * (int64_t)sizeof(VT) <= (1ll << 32);
    if (coop) {
        constexpr int CLv = 16 / (int)sizeof(VT);
        int c0 = 0;
        hipError_t e = hipSuccess;
        while (e == hipSuccess && k - c0 >= 2 * CLv) {
            const int left = k - c0;
            if (left >= 8 * CLv) {
                e = straight ? launch_straight(c0) : launch(TypeBox<CoopSpmmSink<VT, 8>>(), 8 * CLv, c0);
                c0 += 8 * CLv;
            } else if (left >= 4 * CLv) {
                e = launch(TypeBox<CoopSpmmSink<VT, 4>>(), 4 * CLv, c0);
                c0 += 4 * CLv;
            } else {
                e = launch(TypeBox<CoopSpmmSink<VT, 2>>(), 2 * CLv, c0);
                c0 += 2 * CLv;
            }
        }
        if (e != hipSuccess || c0 == k) return e;
        X += c0;
        Y += c0;
        k -= c0;
    }
    // widest column chunk that fits the registers without spilling; FP32
    // accumulators only while a lane's sum has at most 32 terms, so that the
    // worst-case rounding error, (T - 1) 2^-24 |A||x|, stays below 2e-6 |A||x|
    const bool f32acc = std::is_same<VT, float>::value && a.layout == 2 && a.lane_nnz <= 32;
    const int kcmax = std::is_same<VT, double>::value ? 8 : 16;
    return for_kc(k, kcmax, [&](auto KCc, int c0) {
        constexpr int KC = decltype(KCc)::value;
        if constexpr (std::is_same<VT, float>::value && KC >= 8 && KC <= 16) {
            if (f32acc) return launch(TypeBox<SpmmSink<VT, KC, false, float>>(), KC, c0);
        }
        if constexpr (KC > 16 || (std::is_same<VT, double>::value && KC > 8)) {
            return hipErrorInvalidValue;  // excluded by kcmax
        } else {
            return launch(TypeBox<SpmmSink<VT, KC, false>>(), KC, c0);
        }
    });
}

// The LDS block of the transposed product: columns of A per block, padded to
// a multiple of 32, and columns of dY a pass can hold (kMaxTransCols at
// most).  Up to two column blocks (each decodes the streams again, against
// scattered global atomics at 21 G lane operations a second); plane 0: dX
// does not fit.
constexpr int kMaxTransCols = 8;
struct TransBlock {
    int32_t blocks = 0, cols = 0, plane = 0, width = 0;
};
template <typename VT>
TransBlock trans_block(const DevMat &a) {
    const int64_t room = (160 * 1024 - (int64_t)sizeof(Tables<VT>)) / (int64_t)sizeof(double);
    TransBlock t;
    for (int b = 1; b <= 2; ++b) {
        const int64_t cols = (a.n + b - 1) / b, plane = (cols + 31) / 32 * 32;
        if (plane == 0 || plane > room) continue;
        t.blocks = b;
        t.cols = (int32_t)cols;
        t.plane = (int32_t)plane;
        t.width = (int32_t)std::min<int64_t>(kMaxTransCols, room / plane);
        break;
    }
    return t;
}

template <typename VT>
hipError_t spmm_t_impl(const DevMat &a, int k, const VT *dY, int64_t lddy, VT *dX, int64_t lddx,
                       double alpha, double beta, Launch L, void *work, size_t work_bytes,
                       hipStream_t st) {
    if (a.n == 0) return hipSuccess;
    const TransBlock tb = trans_block<VT>(a);
    const int64_t G = L.num_cus;
    if (tb.plane > 0 && a.nnz > 0 && a.num_waves > 0 &&
        work_bytes >= (size_t)G * (size_t)tb.plane * (size_t)tb.width * sizeof(VT)) {
        VT *part = (VT *)work;
        // passes of equal width; a launch runs at most kPasses of them side by
        // side, each on its share of the CUs.  A pass of a small matrix gets a
        // workgroup for every four waves: more would only add copies to sum
        // (157 waves, k = 1: 12 us, 15 with a workgroup for two, 18 for one).
        const int kPasses = (int)std::min<int64_t>(32, G);
        const int chunks = (k + tb.width - 1) / tb.width;
        TransPlan tp;
        tp.n = a.n;
        tp.k = k;
        tp.width = (k + chunks - 1) / chunks;
        tp.blocks = tb.blocks;
        tp.cols = tb.cols;
        tp.plane = tb.plane;
        const int total = ((k + tp.width - 1) / tp.width) * tp.blocks;
        const size_t dyn = (size_t)tp.width * tp.plane * sizeof(double);
        for (tp.pass0 = 0; tp.pass0 < total; tp.pass0 += kPasses) {
            tp.passes = std::min(kPasses, total - tp.pass0);
            const int grid = (int)std::min<int64_t>(G, (int64_t)tp.passes * ((a.num_waves + 3) / 4));
            auto run = [&](auto KCc) -> hipError_t {
                constexpr int KC = decltype(KCc)::value;
                typename TransLdsSink<VT, KC>::Params sp{};
                sp.dY = dY;
                sp.lddy = (uint32_t)lddy;
                auto kern = a.layout == 1 ? pick_bd(a, trans_lds_kernel<1, VT, KC, 1>, trans_lds_kernel<1, VT, KC, 0>)
                                          : pick_bd(a, trans_lds_kernel<2, VT, KC, 1>, trans_lds_kernel<2, VT, KC, 0>);
                hipError_t e = hipFuncSetAttribute((const void *)kern,
                                                   hipFuncAttributeMaxDynamicSharedMemorySize, (int)dyn);
                if (e != hipSuccess) return e;
                hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(1024), dyn, st, a, sp, tp, part);
                return hipGetLastError();
            };
            hipError_t e = tp.width <= 1   ? run(std::integral_constant<int, 1>())
                           : tp.width <= 2 ? run(std::integral_constant<int, 2>())
                           : tp.width <= 3 ? run(std::integral_constant<int, 3>())
                           : tp.width <= 4 ? run(std::integral_constant<int, 4>())
                           : tp.width <= 6 ? run(std::integral_constant<int, 6>())
                                           : run(std::integral_constant<int, 8>());
            if (e != hipSuccess) return e;
            hipLaunchKernelGGL(trans_reduce_kernel<VT>,
                               dim3((unsigned)((tp.width * tp.plane + 255) / 256), (unsigned)tp.passes), dim3(256),
                               0, st, (const VT *)part, tp, grid, dX, lddx, alpha, beta);
            e = hipGetLastError();
            if (e != hipSuccess) return e;
        }
        return hipSuccess;
    }
    // The scatter is bound by global atomic adds, which more CUs at work only
    // make contend: it spreads over them up to four waves a CU (157 waves, FP64:
    // 27 us, 59 in full workgroups) and runs in full workgroups past that (1563
    // waves, 60 a row, FP64: 281 us, 308 on all CUs; FP32, 40 a row: 236, 293).
    L.max_spread = 4 * L.num_cus;
    return for_kc(k, [&](auto KCc, int c0) {
        constexpr int KC = decltype(KCc)::value;
        const int64_t tot = a.n * KC;
        hipLaunchKernelGGL(scale_kernel<VT>, dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, st,
                           dX + c0, a.n, KC, lddx, beta);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess || a.nnz == 0 || a.num_waves == 0) return e;
        typename TransSink<VT, KC>::Params sp;
        sp.dY = dY + c0;
        sp.lddy = (uint32_t)lddy;
        sp.dX = dX + c0;
        sp.lddx = (uint32_t)lddx;
        sp.alpha = alpha;
        typedef TransSink<VT, KC> TS;
        if (a.layout == 1)
            return launch_persistent(pick_bd(a, decode_kernel<1, VT, TS, TS::kOcc, 1>,
                                             decode_kernel<1, VT, TS, TS::kOcc, 0>),
                                     a, L, st, a, sp);
        return launch_persistent(pick_bd(a, decode_kernel<2, VT, TS, occ_nnz(TS::kOcc), 1>,
                                         decode_kernel<2, VT, TS, occ_nnz(TS::kOcc), 0>),
                                 a, L, st, a, sp);
    });
}

template <typename VT>
hipError_t sym_impl(const DevMat &a, const VT *x, double *y, double alpha, Launch L, hipStream_t st) {
    if (a.nnz == 0 || a.num_waves == 0) return hipSuccess;
    const typename SymSink<VT>::Params sp{x, y, alpha, nullptr};
    auto kern = a.layout == 1 ? pick_tf(a, sym_kernel<1, VT, 2>, sym_kernel<1, VT, 1>, sym_kernel<1, VT, 0>)
                              : pick_tf(a, sym_kernel<2, VT, 2>, sym_kernel<2, VT, 1>, sym_kernel<2, VT, 0>);
    hipError_t e = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize,
                                       (int)BlockSums::kBytes);
    if (e != hipSuccess) return e;
    // small matrices: four waves a workgroup at least, so that fewer tables
    // are staged
    const int64_t grid =
        L.fixed_shape ? std::min(L.grid, L.num_cus) : std::min<int64_t>(L.num_cus, (a.num_waves + 3) / 4);
    hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(64 * lone_group_waves(L, 16)), BlockSums::kBytes, st, a, sp);
    return hipGetLastError();
}

template <typename VT>
hipError_t decode_impl(const DevMat &a, int32_t *col, void *vals, Launch L, hipStream_t st) {
    if (a.nnz == 0 || a.num_waves == 0) return hipSuccess;
    typedef typename Bits<VT>::T BT;
    // one walk for escapes inside the stream, and for rows so unequal that few
    // lanes decode most of the time
    if ((a.esc_in_stream && !a.no_escape) || L.one_walk) {
        typedef DecodeSink<VT> DS;
        const typename DS::Params sp{col, (BT *)vals};
        if (a.layout == 1)
            return launch_persistent(pick_bd(a, decode_kernel<1, VT, DS, DS::kOcc, 1>, decode_kernel<1, VT, DS, DS::kOcc, 0>),
                                     a, L, st, a, sp);
        return launch_persistent(pick_bd(a, decode_kernel<2, VT, DS, occ_nnz(DS::kOcc), 1>,
                                         decode_kernel<2, VT, DS, occ_nnz(DS::kOcc), 0>),
                                 a, L, st, a, sp);
    }
    // Rows by groups of lanes: what it saves is the stores' cache lines, what it
    // costs is a longer walk.  So from four waves a CU on (rows of 60, FP64:
    // 4096 waves 75 -> 60 us, 1024 waves 28 -> 24, 512 waves 21 us either way,
    // 64 waves 17 -> 19; FP32: 67 -> 55, 25 -> 23, 17 -> 20, 14 -> 18) and where
    // the values of a mean row fill a line's half (15625 waves, FP64: rows of 8
    // 36 -> 30 us, of 4 19 -> 21; FP32: of 16 51 -> 41, of 8 24 -> 26).
    if (a.layout == 1 && a.base_direct && a.no_escape && a.num_waves >= 4 * L.num_cus &&
        a.nnz * (int64_t)sizeof(VT) >= 64 * a.m) {
        typedef CsrOut<VT, true> CX;
        const typename CX::Params sx{col, (BT *)vals, nullptr};
        const int waves = lone_group_waves(L, kXchWaves);
        const size_t dyn = (size_t)waves * kWave * CX::kLaneWords * 4;
        hipError_t e = hipFuncSetAttribute((const void *)csr_rows_kernel<VT>,
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)dyn);
        if (e != hipSuccess) return e;
        const int64_t grid = L.fixed_shape ? std::min(L.grid, L.num_cus) : L.num_cus;
        hipLaunchKernelGGL(csr_rows_kernel<VT>, dim3((unsigned)grid), dim3(64 * waves), dyn, st, a, sx);
        return hipGetLastError();
    }
    typedef CsrOut<VT> CO;
    const typename CO::Params sp{col, (BT *)vals, nullptr};
    constexpr int occ = CO::kOcc;
    if (a.layout == 1)
        return launch_persistent(pick_tf(a, decode_kernel<1, VT, CO, occ, 2>, decode_kernel<1, VT, CO, occ, 1>,
                                         decode_kernel<1, VT, CO, occ, 0>),
                                 a, L, st, a, sp);
    return launch_persistent(pick_tf(a, decode_kernel<2, VT, CO, occ, 2>, decode_kernel<2, VT, CO, occ, 1>,
                                     decode_kernel<2, VT, CO, occ, 0>),
                             a, L, st, a, sp);
}

template <typename VT>
hipError_t csr_impl(const CsrDev &c, int k, const VT *X, int64_t ldx, VT *Y, int64_t ldy,
                    double alpha, double beta, double *partial, int num_cus, hipStream_t st) {
    if (c.m == 0) return hipSuccess;
    return for_kc(k, [&](auto KCc, int c0) {
        constexpr int KC = decltype(KCc)::value;
        if (c.nnz == 0) {
            const int64_t tot = c.m * KC;
            hipLaunchKernelGGL(scale_kernel<VT>, dim3((unsigned)((tot + 255) / 256)), dim3(256), 0,
                               st, Y + c0, c.m, KC, ldy, beta);
            return hipGetLastError();
        }
        if (c.variant == 3 && KC == 1 && ldx == 1 && ldy == 1) {
            hipLaunchKernelGGL(csr_stream_kernel<VT>, dim3((unsigned)c.nblk), dim3(256), 0, st, c,
                               c.blk, X + c0, Y + c0, alpha, beta);
            return hipGetLastError();
        }
        if (c.variant == 2) {
            hipLaunchKernelGGL((csr_split_kernel<VT, KC>), dim3((unsigned)((c.num_lanes + 255) / 256)),
                               dim3(256), 0, st, c, X + c0, ldx, Y + c0, ldy, alpha, beta, partial);
            hipError_t e = hipGetLastError();
            if (e != hipSuccess) return e;
            return launch_epilogue(c.split, (const int32_t *)nullptr, 0, partial, KC, 0, Y + c0, ldy, alpha, beta, st);
        }
        const int64_t rows_per_block = 256 / c.group;
        int64_t blocks = (c.m + rows_per_block - 1) / rows_per_block;
        blocks = blocks < (int64_t)num_cus * 8 ? blocks : (int64_t)num_cus * 8;
#define DTANS_CSR_G(GG)                                                                         \
    case GG:                                                                                    \
        hipLaunchKernelGGL((csr_vector_kernel<VT, GG, KC>), dim3((unsigned)blocks), dim3(256), 0, \
                           st, c, X + c0, ldx, Y + c0, ldy, alpha, beta);                      \
        break;
        switch (c.group) {
            DTANS_CSR_G(1)
            DTANS_CSR_G(2)
            DTANS_CSR_G(4)
            DTANS_CSR_G(8)
            DTANS_CSR_G(16)
            DTANS_CSR_G(32)
            DTANS_CSR_G(64)
            default:
                return hipErrorInvalidValue;
        }
#undef DTANS_CSR_G
        return hipGetLastError();
    });
}

}  // namespace

hipError_t launch_spmm(const DevMat &a, bool f64, int k, const void *X, int64_t ldx, void *Y,
                       int64_t ldy, double alpha, double beta, double *partial, Launch L,
                       hipStream_t st) {
    if (f64)
        return spmm_impl<double>(a, k, (const double *)X, ldx, (double *)Y, ldy, alpha, beta,
                                 partial, L, st);
    return spmm_impl<float>(a, k, (const float *)X, ldx, (float *)Y, ldy, alpha, beta, partial, L,
                            st);
}

size_t spmm_scratch_bytes(const DevMat &a, int k) {
    if (a.layout != 2 || a.nnz == 0) return 0;
    return (size_t)(2 * a.num_lanes * (int64_t)std::min(k, kMaxPassCols) + 1) * sizeof(double);
}

size_t spmm_t_work_bytes(const DevMat &a, bool f64, int num_cus) {
    const TransBlock t = f64 ? trans_block<double>(a) : trans_block<float>(a);
    return (size_t)num_cus * (size_t)t.plane * (size_t)t.width * (f64 ? 8 : 4);
}

hipError_t launch_spmm_t(const DevMat &a, bool f64, int k, const void *dY, int64_t lddy, void *dX,
                         int64_t lddx, double alpha, double beta, Launch L, void *work,
                         size_t work_bytes, hipStream_t st) {
    if (f64)
        return spmm_t_impl<double>(a, k, (const double *)dY, lddy, (double *)dX, lddx, alpha, beta,
                                   L, work, work_bytes, st);
    return spmm_t_impl<float>(a, k, (const float *)dY, lddy, (float *)dX, lddx, alpha, beta, L,
                              work, work_bytes, st);
}

hipError_t launch_sym(const DevMat &a, bool f64, const void *x, double *y, double alpha, Launch L, hipStream_t st) {
    return f64 ? sym_impl<double>(a, (const double *)x, y, alpha, L, st)
               : sym_impl<float>(a, (const float *)x, y, alpha, L, st);
}

hipError_t launch_decode(const DevMat &a, bool f64, int32_t *col, void *vals, Launch L,
                         hipStream_t st) {
    return f64 ? decode_impl<double>(a, col, vals, L, st) : decode_impl<float>(a, col, vals, L, st);
}

// copies the x / y pointers of one call from the launch arguments into the
// batch's device pointer table (stream-ordered with the batch kernel)
__global__ void batch_ptrs_kernel(BatchPtrs p, int count, void **table) {
    const int i = threadIdx.x;
    if (i < count) {
        table[2 * i] = (void *)p.xs[i];
        table[2 * i + 1] = p.ys[i];
    }
}

hipError_t launch_batch(const BatchDev &b, const BatchPtrs &ptrs, int count, bool f64, double alpha,
                        double beta, Launch L, hipStream_t st) {
    hipLaunchKernelGGL(batch_ptrs_kernel, dim3(1), dim3(kMaxBatch), 0, st, ptrs, count,
                       (void **)b.ptrs);
    hipError_t e0 = hipGetLastError();
    if (e0 != hipSuccess) return e0;
    const dim3 block(64 * L.waves_per_wg);
    if (f64)
        hipLaunchKernelGGL(batch_kernel<double>, dim3(L.grid), block, 0, st, b, alpha, beta);
    else
        hipLaunchKernelGGL(batch_kernel<float>, dim3(L.grid), block, 0, st, b, alpha, beta);
    return hipGetLastError();
}

template <typename VT>
hipError_t batch_spmm_impl(const BatchDev &b, int k, bool aligned, double alpha, double beta, Launch L,
                           hipStream_t st) {
    auto go = [&](auto kern, int c0) -> hipError_t {
        // the task lists hold for any workgroup size; the kernel may allow fewer
        // waves per workgroup than the plan (more registers per wave)
        hipFuncAttributes fa;
        int wpw = L.waves_per_wg;
        if (hipFuncGetAttributes(&fa, (const void *)kern) == hipSuccess)
            wpw = std::max(1, std::min(wpw, fa.maxThreadsPerBlock / 64));
        hipLaunchKernelGGL(kern, dim3(L.grid), dim3(64 * wpw), 0, st, b, c0, k, alpha, beta);
        return hipGetLastError();
    };
    constexpr int CL = 16 / (int)sizeof(VT);
    int c0 = 0;
    hipError_t e = hipSuccess;
    // lane groups sharing each row of X (16-byte pieces), then single columns
    while (aligned && e == hipSuccess && k - c0 >= 2 * CL) {
        if (k - c0 >= 8 * CL) {
            typedef CoopSpmmSink<VT, 8> S;
            e = go(batch_spmm_kernel<VT, S, S::kOcc>, c0);
            c0 += 8 * CL;
        } else if (k - c0 >= 4 * CL) {
            typedef CoopSpmmSink<VT, 4> S;
            e = go(batch_spmm_kernel<VT, S, S::kOcc>, c0);
            c0 += 4 * CL;
        } else {
            typedef CoopSpmmSink<VT, 2> S;
            e = go(batch_spmm_kernel<VT, S, S::kOcc>, c0);
            c0 += 2 * CL;
        }
    }
    while (e == hipSuccess && c0 < k) {
        if (k - c0 >= 4) {
            typedef SpmmSink<VT, 4, false> S;
            e = go(batch_spmm_kernel<VT, S, S::kOcc>, c0);
            c0 += 4;
        } else if (k - c0 >= 2) {
            typedef SpmmSink<VT, 2, false> S;
            e = go(batch_spmm_kernel<VT, S, S::kOcc>, c0);
            c0 += 2;
        } else {
            typedef SpmmSink<VT, 1, false> S;
            e = go(batch_spmm_kernel<VT, S, S::kOcc>, c0);
            c0 += 1;
        }
    }
    return e;
}

hipError_t launch_batch_spmm(const BatchDev &b, const BatchPtrs &ptrs, int count, bool f64, int k,
                             bool aligned, double alpha, double beta, Launch L, hipStream_t st) {
    hipLaunchKernelGGL(batch_ptrs_kernel, dim3(1), dim3(kMaxBatch), 0, st, ptrs, count,
                       (void **)b.ptrs);
    hipError_t e0 = hipGetLastError();
    if (e0 != hipSuccess) return e0;
    return f64 ? batch_spmm_impl<double>(b, k, aligned, alpha, beta, L, st)
               : batch_spmm_impl<float>(b, k, aligned, alpha, beta, L, st);
}

hipError_t launch_flush(const void *buf, int64_t bytes, uint32_t *sink, hipStream_t st) {
    if (bytes % 16) return hipErrorInvalidValue;
    hipLaunchKernelGGL(flush_kernel, dim3(2048), dim3(256), 0, st, (const uint4 *)buf, bytes / 16, sink);
    return hipGetLastError();
}

hipError_t launch_csr(const CsrDev &c, bool f64, int k, const void *X, int64_t ldx, void *Y,
                      int64_t ldy, double alpha, double beta, double *partial, int num_cus,
                      hipStream_t st) {
    if (f64)
        return csr_impl<double>(c, k, (const double *)X, ldx, (double *)Y, ldy, alpha, beta, partial,
                                num_cus, st);
    return csr_impl<float>(c, k, (const float *)X, ldx, (float *)Y, ldy, alpha, beta, partial,
                           num_cus, st);
}

// Scratch for callers that cannot allocate device memory (dtans_spmm_noalloc):
// a file-scope array that every GPU the library runs on holds from the first
// use until the process ends.  On the host its name is only a stand-in
// symbol, so host code never passes it to a kernel, a memset or a copy: it
// looks up the device address of each GPU's own copy once, with that device
// current, and passes that address instead.
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

hipError_t static_scratch(void **ptr) {
    constexpr int kMaxDevices = 64;
    static std::mutex mu;
    static void *addr[kMaxDevices] = {};
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(mu);
    if (!addr[dev]) {
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (!p) return hipErrorInvalidSymbol;
        addr[dev] = p;
    }
    *ptr = addr[dev];
    return hipSuccess;
}

}  // namespace dtans
