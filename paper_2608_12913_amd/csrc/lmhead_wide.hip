// LM-head projection for more rows than the streaming kernel's 128 (bf16; route.h has the
// small vocabularies that stay with that one), with the same epilogues (Alg. 1 "parallel
// model evaluation", the per-tile pieces of Eq. (1); with the plausibility mask of Sec. 2.1
// or, at theta = 0, the untruncated target).
//
// Tile.  A workgroup owns 256 tokens x TR = 32*RB rows; its 8 waves form a 4 x 2 grid
// of 64 tokens x 16*RB rows (4 x RB blocks of v_mfma_f32_16x16x32_bf16).  K is walked in
// 128-byte chunks of every row, two k-steps each.  Weights (whole chunks) and hidden
// states (half chunks, one k-step) load straight into two rings of LDS stages
// (global_load_lds) while earlier ones are multiplied.  TR is chosen per problem
// (wide_row_blocks in route.h).
//
// Two waves share a SIMD, one of each row half (wave w and w + 4), and take turns: a
// k-step is a slot of LDS reads and a slot of MFMAs, and the second half of the waves
// runs one slot behind the first.  Every slot ends with a workgroup barrier, so while
// one wave of a SIMD multiplies, the other one reads its fragments.  Without the offset
// both waves read, wait and multiply in step and the matrix cores idle during the reads.
//
// The first half of the waves loads the weights, the second the hidden states.  A wave's
// loads complete in issue order, so one that loads both cannot leave the weights (from
// HBM) in flight for longer than the hidden states (from L2).
//
// What bounds it, measured on the 2048-row batch of 4096/2048-wide heads over 128,256
// tokens (LM head alone; 4 waves of 128 x 128 before): 3.16 -> 2.64 ms, 1.02 -> 1.22
// PFLOP/s epilogues included (a library matrix product of the expert head alone reaches 1.24
// to 1.31 on such cards and inputs, 1.59 on zeros: the clock falls under load).  Timing
// copies: without the loads 1.89 ms, without the MFMAs 2.20, every load an L2 hit 2.58.
// 285 rows: 0.69 -> 0.43 ms, 651 rows: 1.37 -> 1.14 ms.  Measured and not kept: the lines
// of a later chunk pulled into L2 by one of the workgroups that share them (+6%), K walks
// started at another chunk per XCD or per tile (+1 to +7%).
#include "dcd_internal.h"

namespace dcd {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

constexpr int NT = 512;               // threads per workgroup (8 waves)
constexpr int TT = kTileTokens;       // tokens per tile (the partials' tile)
constexpr int CB = 128;               // bytes of every row per K-chunk
constexpr int LPR = CB / 16;          // lanes per row in a load instruction
constexpr int RPI = kWaveSize / LPR;  // rows per load instruction
constexpr int TW = 4;                 // waves along the tokens (two along the rows)
constexpr int BV = TT / TW / 16;      // 16-token blocks per wave
constexpr int WT = 16 * BV;           // tokens per wave (64)
constexpr int KS = CB / 64;           // MFMA k-steps per chunk
constexpr uint32_t KSTEP = 64;        // bytes of a row in one k-step
constexpr int WL = TT / RPI / TW;     // weight load instructions per loading wave and chunk
constexpr int HRPI = 16;              // rows of a hidden-state load instruction (64 bytes each)
constexpr int WSTAGE = TT * CB;       // bytes of a weight stage
static_assert(TT == 256 && BV == 4 && WL == 8 && LPR == RPI, "tile geometry");

template <int RB>
struct Geo {
    static constexpr int TR = 32 * RB;                  // rows per workgroup
    static constexpr int WR = 16 * RB;                  // rows per wave
    static constexpr int HI = TR / HRPI;                // hidden-state load instructions per k-step
    static constexpr int HL = (HI + TW - 1) / TW;       // of one loading wave
    static constexpr int HSTAGE = TR * (int)KSTEP;      // bytes of a hidden-state stage
    static constexpr int NW = RB <= 4 ? 4 : 3;          // weight stages
    static constexpr int NH = RB > 4 && RB <= 7 ? 4 : 3;  // hidden-state stages
    static constexpr int RING = NW * WSTAGE + NH * HSTAGE;
};

typedef __attribute__((address_space(3))) void *lds_ptr;

// Waits until at most N of this wave's vector memory operations are outstanding
// (loads complete in issue order; the compiler does not track loads that write LDS).
template <int N>
__device__ __forceinline__ void wait_loads() {
    static_assert(N < 64, "vmcnt is 6 bits");
    __builtin_amdgcn_s_waitcnt(0x0F70 | (N & 15) | (N >> 4) << 14);
}

// Ends a slot: the wave's LDS reads have returned (lgkmcnt) before it arrives.  Unlike
// __syncthreads() it leaves direct-to-LDS loads in flight.
__device__ __forceinline__ void slot_end() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
}

// A uniform address the compiler may not take apart again: the loads then use the scalar
// base with a 32-bit lane offset, instead of a hoisted 64-bit address per load and lane.
__device__ __forceinline__ const char *uniform_base(const char *p) {
    asm("" : "+s"(p));
    return p;
}

// A 32-bit lane offset, kept as such (widened at the load, not hoisted as 64 bits).
__device__ __forceinline__ uint32_t lane_offset(uint32_t o) {
    asm("" : "+v"(o));
    return o;
}

// The wave's index in a scalar register.
__device__ __forceinline__ int wave_id() {
    int w = __builtin_amdgcn_readfirstlane(threadIdx.x / kWaveSize);
    asm("" : "+s"(w));
    return w;
}

__device__ __forceinline__ float wave_max16_32(float x) {
    x = fmaxf(x, __shfl_xor(x, 16));
    return fmaxf(x, __shfl_xor(x, 32));
}
__device__ __forceinline__ float wave_sum16_32(float x) {
    x += __shfl_xor(x, 16);
    return x + __shfl_xor(x, 32);
}

// Per-thread load addresses of one model.  A weight load instruction fills 8 rows x 128
// bytes (1 KB) of a stage, lane l landing at byte 16 l: row l/8, slot l%8, which holds
// column (l%8) ^ (row%8).  A hidden-state one fills 16 rows x 64 bytes: row l/4, slot l%4,
// column (l%4) ^ (-(row/4) mod 4).  ds_read_b128 serves lanes {0-3, 12-15, 20-27} of
// each half wave together and the other 16 after them; either layout puts such a group
// in 16 distinct bank groups (with (l%4) ^ (row/4%4) 39% of the LDS cycles were conflicts).
// Wave w < 4 loads weight rows 64w .. 64w+63, wave 4+w the hidden-state row groups
// w, w+4, ... of 16 rows (past the last one: the last one again, so that every wave counts
// the same loads).  Address = uniform row base (scalar registers) + a 32-bit lane offset.
// Rows past the vocabulary or past row R are clamped to the last one (their results are
// discarded).  G: the wave's half.  ONE: the problem has one row tile, so each weight byte
// is read once (non-temporal loads, and each vocabulary tile starts its K walk at a chunk
// of its own, for the HBM channels).
template <int RB, int G, bool ONE>
struct Stream {
    using Q = Geo<RB>;
    static constexpr int L = G == 0 ? WL : Q::HL;  // load instructions per stage
    static constexpr int AUX = ONE && G == 0 ? 2 : 0;  // non-temporal
    const char *row;          // first row of the operand this wave loads
    uint32_t rowbytes;
    int nch, rot;             // K chunks, and the chunk the walk starts with
    uint32_t off[L];          // lane offsets
    uint32_t dst;             // LDS byte offset of the first instruction in a stage
    uint32_t colb;            // byte column of the lane's slot
    int last;                 // LDS byte step of the last hidden-state instruction
    // the lane's LDS byte offsets of its first weight and hidden-state fragment in a stage
    // (k-step 1 of a weight chunk: the same with KSTEP flipped, the swizzle being an
    // exclusive or)
    uint32_t wl, hl;

    __device__ __forceinline__ void init(const void *h, const void *w, int d, int R, int V, int row0, int tile0,
                                         int tile, int wave) {
        const int lane = threadIdx.x % kWaveSize, wv = wave % TW;
        rowbytes = (uint32_t)d * 2;
        nch = (int)((rowbytes + CB - 1) / CB);
        rot = rowbytes % CB ? nch - 1 : ONE ? (int)((7u * (uint32_t)tile) % (uint32_t)nch) : 0;
        if constexpr (G == 0) {
            const int r = lane / LPR, wlast = V - 1 - tile0;
            colb = (uint32_t)((lane % LPR) ^ r) * 16;
            row = (const char *)w + (size_t)tile0 * rowbytes;
            dst = (uint32_t)(WL * RPI * wv * CB);
#pragma unroll
            for (int q = 0; q < L; ++q)
                off[q] = (uint32_t)min(WL * RPI * wv + RPI * q + r, wlast) * rowbytes + col_in_row();
        } else {
            const int r = lane / 4, hlast = R - 1 - row0;
            colb = (uint32_t)((lane % 4) ^ (-(r / 4) & 3)) * 16;
            row = (const char *)h + (size_t)row0 * rowbytes;
            dst = (uint32_t)(HRPI * wv * KSTEP);
            last = (min(TW * (L - 1) + wv, Q::HI - 1) - wv) * HRPI * (int)KSTEP;
#pragma unroll
            for (int k = 0; k < L; ++k)
                off[k] = (uint32_t)min(HRPI * min(wv + TW * k, Q::HI - 1) + r, hlast) * rowbytes + col_in_row();
        }
        const int n = lane % 16, g = lane / 16;
        wl = (uint32_t)((wv * WT + n) * CB + (g ^ (n % LPR)) * 16);
        hl = (uint32_t)((G * Q::WR + n) * (int)KSTEP + (g ^ (-(n / 4) & 3)) * 16);
    }

    // the lane's column, inside the row also where a row is shorter than a chunk
    __device__ __forceinline__ uint32_t col_in_row() const { return min(colb, rowbytes - 16); }

    // chunk c of the walk -> byte offset of its columns
    __device__ __forceinline__ uint32_t koff(int c) const {
        return (uint32_t)(c + rot < nch ? c + rot : c + rot - nch) * CB;
    }

    // One stage's loads of this wave: uniform source and LDS destination.
    struct Request {
        const char *base;
        char *at;
        uint32_t shift;  // of the lane's column (the sum with off[] is never negative)
    };

    // Stage i of the walk (weights: chunk i; hidden states: k-step i) into the ring's byte
    // `to`; past the last one, the last chunk again (never read).  first: the walk's first
    // chunk, the only one that may reach past the row end (a row that ends inside a chunk
    // has its walk start there): a lane past the end then re-reads the row's last 16 bytes
    // (finite values), and the hidden-state slots there are zeroed after arrival (zero_tail).
    __device__ __forceinline__ Request request(char *lds, uint32_t to, int i, bool first = false) const {
        uint32_t k0, shift = 0;
        if constexpr (G == 0) {
            k0 = koff(first ? i : min(i, nch - 1));
        } else {
            const int c = i >> 1;
            k0 = c < nch ? koff(c) + (uint32_t)(i & 1) * KSTEP : koff(nch - 1);
        }
        if (first) {
            const uint32_t end = rowbytes - 16, col = min(k0 + colb, end);
            k0 = min(k0, end);  // (k0 may lie past the row end: the first chunk's second k-step)
            shift = col - k0 - col_in_row();
        }
        return Request{uniform_base(row + k0), lds + to + dst, shift};
    }
    __device__ __forceinline__ void load(const Request &r, int q) const {
        const int step = G == 0 ? q * RPI * CB : q + 1 < L ? q * TW * HRPI * (int)KSTEP : last;
        __builtin_amdgcn_global_load_lds(r.base + lane_offset(off[q] + r.shift), (lds_ptr)(r.at + step), 16, 0, AUX);
    }
    __device__ __forceinline__ void load_all(const Request &r) const {
#pragma unroll
        for (int q = 0; q < L; ++q) load(r, q);
    }

    // After this wave's hidden-state loads of the walk's k-step s (0 or 1) landed at `to`:
    // its slots past the row end become zero, so the re-read weights there multiply zeros.
    __device__ __forceinline__ void zero_tail(char *lds, uint32_t to, int s) const {
        if constexpr (G == 1) {
            if (koff(0) + (uint32_t)s * KSTEP + colb < rowbytes) return;
            const int lane = threadIdx.x % kWaveSize;
            char *at = lds + to + dst + lane * 16;
#pragma unroll
            for (int q = 0; q < L; ++q)
                *reinterpret_cast<u32x4 *>(at + (q + 1 < L ? q * TW * HRPI * (int)KSTEP : last)) =
                    u32x4{0u, 0u, 0u, 0u};
        }
    }
};

// The fragments of one k-step: A = weights (tokens as M), B = hidden states (rows as N);
// lane l supplies row l%16 of a block and K columns 8*(l/16).. of the k-step.
//
// The reads are one asm block that ends with their own wait.  Written as plain loads, the
// compiler takes some of them for readers of the direct-to-LDS loads in flight and waits
// for those (vmcnt(0)) in every chunk; which loads a slot must have waited for is known
// here and stated with wait_loads.
#define DCD_W4                                                                       \
    "ds_read_b128 %[a0], %[w]\n ds_read_b128 %[a1], %[w] offset:2048\n"              \
    "ds_read_b128 %[a2], %[w] offset:4096\n ds_read_b128 %[a3], %[w] offset:6144\n"
#define DCD_H4                                                                       \
    "ds_read_b128 %[b0], %[h]\n ds_read_b128 %[b1], %[h] offset:1024\n"              \
    "ds_read_b128 %[b2], %[h] offset:2048\n ds_read_b128 %[b3], %[h] offset:3072\n"
#define DCD_H5 DCD_H4 "ds_read_b128 %[b4], %[h] offset:4096\n"
#define DCD_H6 DCD_H5 "ds_read_b128 %[b5], %[h] offset:5120\n"
#define DCD_H7 DCD_H6 "ds_read_b128 %[b6], %[h] offset:6144\n"
#define DCD_H8 DCD_H7 "ds_read_b128 %[b7], %[h] offset:7168\n"
#define DCD_H9 DCD_H8 "ds_read_b128 %[b8], %[h] offset:8192\n"
#define DCD_WAIT "s_waitcnt lgkmcnt(0)"
#define DCD_O4                                                                                 \
    [a0] "=&v"(a[0]), [a1] "=&v"(a[1]), [a2] "=&v"(a[2]), [a3] "=&v"(a[3]), [b0] "=&v"(b[0]), \
        [b1] "=&v"(b[1]), [b2] "=&v"(b[2]), [b3] "=&v"(b[3])
#define DCD_O5 DCD_O4, [b4] "=&v"(b[4])
#define DCD_O6 DCD_O5, [b5] "=&v"(b[5])
#define DCD_O7 DCD_O6, [b6] "=&v"(b[6])
#define DCD_O8 DCD_O7, [b7] "=&v"(b[7])
#define DCD_O9 DCD_O8, [b8] "=&v"(b[8])
#define DCD_READ(n) asm volatile(DCD_W4 DCD_H##n DCD_WAIT : DCD_O##n : [w] "v"(w), [h] "v"(h) : "memory")
static_assert(16 * CB == 2048 && 16 * KSTEP == 1024, "block strides of the fragment reads");

template <int RB>
struct Frags {
    u32x4 a[BV], b[RB];

    // w, h: LDS byte addresses of the lane's first fragments
    __device__ __forceinline__ void read(uint32_t w, uint32_t h) {
        static_assert(RB >= 4 && RB <= 9, "row blocks per wave");
        if constexpr (RB == 4) DCD_READ(4);
        if constexpr (RB == 5) DCD_READ(5);
        if constexpr (RB == 6) DCD_READ(6);
        if constexpr (RB == 7) DCD_READ(7);
        if constexpr (RB == 8) DCD_READ(8);
        if constexpr (RB == 9) DCD_READ(9);
    }

    // The MFMAs of the k-step, with loads LO .. HI-1 of a request spread over them: issued
    // together they hold up the wave (and with it the slot) behind the CU's address unit.
    template <int LO, int HI, class S>
    __device__ __forceinline__ void multiply(f32x4 (&acc)[BV][RB], const S &st,
                                             const typename S::Request &r) const {
        __builtin_amdgcn_s_setprio(1);
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
#pragma unroll
            for (int q = LO; q < HI; ++q)
                if ((q - LO) * RB / (HI - LO) == rb) {
                    st.load(r, q);
                    __builtin_amdgcn_sched_barrier(0);
                }
#pragma unroll
            for (int vb = 0; vb < BV; ++vb)
                acc[vb][rb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a[vb]),
                                                                      __builtin_bit_cast(bf16x8, b[rb]),
                                                                      acc[vb][rb], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        }
        __builtin_amdgcn_s_setprio(0);
        __builtin_amdgcn_sched_barrier(0);
    }
};

// One pass over a model's K chunks.
//
// Slots: the first half of the waves (G = 0) reads k-step q in slot 2q and multiplies it in
// slot 2q+1; the second half one slot later.  Every read of k-step q has returned by the
// end of slot 2q+1 (each read block waits for its own).  So from slot 2q+2 on, its hidden-
// state stage may be filled again, and its weight stage if q is a chunk's second k-step.
//   G = 0 requests weight chunk c+NW-1 in slots 4c+1 and 4c+3 (its multiply slots), into the
//     stage of chunk c-1, and has waited for chunk c+1 by the end of slot 4c+3.
//   G = 1 requests k-step q+NH-1 in slot 2q (its multiply slot of k-step q-1), into the
//     stage of k-step q-1, and has waited for k-step q+1 by the end of slot 2q+1.
// Requests past the walk's end repeat its last chunk, so the loop has no branches (with
// branches the compiler splits the accumulators' live ranges and spills) and the waits
// count the same loads in every round.
//
// start_pass requests the first stages; on return of run_pass no load is in flight and
// every wave is done with the rings.
template <int RB, int G, bool ONE>
__device__ __forceinline__ void start_pass(const Stream<RB, G, ONE> &st, char *lds) {
    using Q = Geo<RB>;
    if constexpr (G == 0) {
        st.load_all(st.request(lds, 0, 0, true));
#pragma unroll
        for (int i = 1; i < Q::NW - 1; ++i) st.load_all(st.request(lds, i * WSTAGE, i));
    } else {
        char *ring = lds + Q::NW * WSTAGE;
        st.load_all(st.request(ring, 0, 0, true));
        st.load_all(st.request(ring, Q::HSTAGE, 1, true));
#pragma unroll
        for (int i = 2; i < Q::NH - 1; ++i) st.load_all(st.request(ring, i * Q::HSTAGE, i));
    }
}

template <int RB, int G, bool ONE>
__device__ __forceinline__ void run_pass(const Stream<RB, G, ONE> &st, char *lds, f32x4 (&acc)[BV][RB]) {
    using Q = Geo<RB>;
    constexpr uint32_t WRING = Q::NW * WSTAGE, HRING = Q::NH * Q::HSTAGE;
    const uint32_t base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const char *)lds;
    const uint32_t wl = base + st.wl, hl = base + WRING + st.hl;
    char *hring = lds + WRING;
#pragma unroll
    for (int vb = 0; vb < BV; ++vb)
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) acc[vb][rb] = f32x4{0.f, 0.f, 0.f, 0.f};
    wait_loads<0>();
    st.zero_tail(hring, 0, 0);
    st.zero_tail(hring, Q::HSTAGE, 1);
    slot_end();
    // ring positions (bytes): the stages being read, and those to be filled next
    uint32_t wcur = 0, hcur = 0, wnew = (Q::NW - 1) * WSTAGE, hnew = (Q::NH - 1) * Q::HSTAGE;
    auto next = [](uint32_t x, uint32_t stage, uint32_t ring) { return x + stage == ring ? 0u : x + stage; };
    Frags<RB> f;
    if constexpr (G == 0) {
        for (int c = 0; c < st.nch; ++c) {
            f.read(wl + wcur, hl + hcur);
            slot_end();
            const auto r = st.request(lds, wnew, c + Q::NW - 1);
            f.template multiply<0, WL / 2>(acc, st, r);
            slot_end();
            hcur = next(hcur, Q::HSTAGE, HRING);
            f.read((wl ^ KSTEP) + wcur, hl + hcur);
            slot_end();
            f.template multiply<WL / 2, WL>(acc, st, r);
            wait_loads<(Q::NW - 2) * WL>();
            slot_end();
            hcur = next(hcur, Q::HSTAGE, HRING);
            wcur = next(wcur, WSTAGE, WRING);
            wnew = next(wnew, WSTAGE, WRING);
        }
        slot_end();
    } else {
        st.load_all(st.request(hring, hnew, Q::NH - 1));
        hnew = next(hnew, Q::HSTAGE, HRING);
        slot_end();
        for (int c = 0; c < st.nch; ++c) {
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                f.read((s ? wl ^ KSTEP : wl) + wcur, hl + hcur);
                wait_loads<(Q::NH - 2) * Q::HL>();
                slot_end();
                f.template multiply<0, Q::HL>(acc, st, st.request(hring, hnew, 2 * c + s + Q::NH));
                slot_end();
                hcur = next(hcur, Q::HSTAGE, HRING);
                hnew = next(hnew, Q::HSTAGE, HRING);
            }
            wcur = next(wcur, WSTAGE, WRING);
        }
    }
    wait_loads<0>();  // the requests past the last chunk
    slot_end();
}

// acc -> logits divided by T, in place (-inf past the vocabulary), and per row the wave's
// max and sum of exp, left in pairs[wt][row of the workgroup].
template <int RB>
__device__ __forceinline__ void wave_softmax(f32x4 (&acc)[BV][RB], const float *bias, float inv_T, int tok0, int V,
                                             int wt, int wr, float2 *pairs) {
    constexpr float kLog2e = 1.4426950408889634f;
    const int lane = threadIdx.x % kWaveSize, n = lane % 16, g = lane / 16;
    f32x4 b[BV];
#pragma unroll
    for (int vb = 0; vb < BV; ++vb) b[vb] = *reinterpret_cast<const f32x4 *>(bias + wt * WT + 16 * vb + 4 * g);
    const bool ragged = tok0 + WT > V;  // wave-uniform
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
        float m = -INFINITY;
#pragma unroll
        for (int vb = 0; vb < BV; ++vb)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                float z = fmaf(acc[vb][rb][j], inv_T, b[vb][j]);
                if (ragged && tok0 + 16 * vb + 4 * g + j >= V) z = -INFINITY;
                acc[vb][rb][j] = z;
                m = fmaxf(m, z);
            }
        m = wave_max16_32(m);
        const float ml = m * kLog2e;
        float s = 0.f;
#pragma unroll
        for (int vb = 0; vb < BV; ++vb)
#pragma unroll
            for (int j = 0; j < 4; ++j) s += __builtin_amdgcn_exp2f(fmaf(acc[vb][rb][j], kLog2e, -ml));
        if (m == -INFINITY) s = 0.f;  // nothing finite in this wave row
        s = wave_sum16_32(s);
        if (g == 0) pairs[wt * Geo<RB>::TR + wr * Geo<RB>::WR + rb * 16 + n] = float2{m, s};
    }
}

// The tile's (max, sum of exp) of row r from the four token waves' pairs, in their order.
template <int RB>
__device__ __forceinline__ float2 merge_pairs(const float2 *pairs, int r) {
    float m = -INFINITY;
#pragma unroll
    for (int w = 0; w < TW; ++w) m = fmaxf(m, pairs[w * Geo<RB>::TR + r].x);
    float s = 0.f;
    if (m != -INFINITY) {
#pragma unroll
        for (int w = 0; w < TW; ++w) {
            const float2 p = pairs[w * Geo<RB>::TR + r];
            if (p.x != -INFINITY) s += p.y * __expf(p.x - m);
        }
    }
    return float2{m, s};
}

__device__ __forceinline__ YStat ystat_shfl_xor(const YStat &x, int m) {
    return YStat{__shfl_xor(x.y1, m), __shfl_xor(x.i1, m), __shfl_xor(x.y2, m), __shfl_xor(x.ys, m),
                 __shfl_xor(x.zp1, m), __shfl_xor(x.zq1, m), __shfl_xor(x.a, m), __shfl_xor(x.ip, m)};
}

// LDS beside the rings.  Epilogue scratch (pairs, candidate words and counts) reuses the
// last weight stage, which the amateur pass fills only once every wave has entered it;
// the y statistics, after the last pass, the whole weight ring.
template <int RB>
struct Misc {
    float bias_p[TT], bias_q[TT];
    float2 park[Geo<RB>::TR];  // the expert's (max, sum of exp) per row during the amateur pass
    float thr[Geo<RB>::TR];    // per row: candidate threshold, then whether the tile is kept
};

template <int RB, bool FULL, int G, bool ONE>
__device__ __forceinline__ void wide_tile(const Plan &P, const Inputs &in, int tile, int row0, char *lds,
                                          Misc<RB> &ms) {
    using Q = Geo<RB>;
    constexpr int TR = Q::TR;
    constexpr float kLog2e = 1.4426950408889634f;
    const int tid = threadIdx.x, lane = tid % kWaveSize;
    const int wave = wave_id(), wt = wave % TW, wr = G;
    const int n = lane % 16, g = lane / 16;
    const int tile0 = tile * TT;
    const int tok0 = tile0 + wt * WT;          // first token of the wave
    const int wrow0 = row0 + wr * Q::WR;       // first row of the wave
    const int myrow = row0 + tid;              // threads below TR: the row they merge
    const bool owner = tid < TR && myrow < P.R;

    char *scratch = lds + (Q::NW - 1) * WSTAGE;
    float2 *pairs = reinterpret_cast<float2 *>(scratch);                               // [TW][TR]
    uint32_t *twords = reinterpret_cast<uint32_t *>(scratch + TW * TR * sizeof(float2));  // [TR][words]
    int *tcnt = reinterpret_cast<int *>(twords + TR * kWordsPerTile);                  // [TR]
    YStat *ys = reinterpret_cast<YStat *>(lds);                                        // [TW][TR]
    static_assert(TW * TR * sizeof(YStat) <= (size_t)(Q::NW - 1) * WSTAGE, "y statistics fit beside the pairs");
    static_assert(TW * TR * sizeof(float2) + TR * (kWordsPerTile + 1) * 4 <= (size_t)WSTAGE, "scratch fits a stage");

    if (tid < TT) {
        const int t = tile0 + tid;
        ms.bias_p[tid] = (t < P.V && in.bp) ? in.bp[t] * P.inv_T : 0.f;
    } else {
        const int t = tile0 + tid - TT;
        ms.bias_q[tid - TT] = (t < P.V && in.bq) ? in.bq[t] * P.inv_T : 0.f;
    }

    f32x4 acc[BV][RB];
    // untruncated target: few row blocks keep the expert logits in registers across the
    // amateur pass, the others park them in the dense y rows
    constexpr bool kKeepZp = FULL && RB <= 4;
    f32x4 zpk[kKeepZp ? BV : 1][kKeepZp ? RB : 1];
    uint32_t flags[(RB + 1) / 2];  // 16 bits per row block, bit vb*4 + j: tile-local candidate

    // ---- expert head
    Stream<RB, G, ONE> st;
    st.init(in.hp, in.wp, P.dp, P.R, P.V, row0, tile0, tile, wave);
    start_pass(st, lds);
    run_pass(st, lds, acc);
    // the amateur head's first stages load during the expert epilogue
    st.init(in.hq, in.wq, P.dq, P.R, P.V, row0, tile0, tile, wave);
    start_pass(st, lds);
    bool pruning = false;
    uint32_t f[RB];
    if constexpr (!FULL) {
        // the row bounds of this call are cleared by workgroup 0 (long done by now)
        pruning = await_call_state(P.ctl);
        float bnd = -INFINITY;
        if (owner && pruning) bnd = read_bound(P.bound, P.R, myrow);
        wave_softmax<RB>(acc, ms.bias_p, P.inv_T, tok0, P.V, wt, wr, pairs);
        __syncthreads();
        if (tid < TR) {
            const float2 p = merge_pairs<RB>(pairs, tid);
            ms.park[tid] = p;
            // a tile whose expert max is below the row bound + ln(theta) holds no mask member
            ms.thr[tid] = owner && p.x >= bnd + P.log_theta ? p.x + P.log_theta : NAN;  // (no z >= NaN)
            if (owner && pruning) raise_bound(P.bound, P.R, myrow, p.x);
        }
        __syncthreads();
        // tile-local candidates: z_p within ln(theta) of the tile max.  Their expert
        // logits are stored now; most tiles are pruned before (or by) the amateur epilogue
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
            const float thr = ms.thr[wr * Q::WR + rb * 16 + n];
            uint32_t b = 0;
#pragma unroll
            for (int vb = 0; vb < BV; ++vb)
#pragma unroll
                for (int j = 0; j < 4; ++j) b |= acc[vb][rb][j] >= thr ? 1u << (vb * 4 + j) : 0u;
            // thr is -inf where the tile max is (a row of -inf): tokens past the vocabulary
            // compare equal then and are taken out
            if (tok0 + WT > P.V) {
#pragma unroll
                for (int vb = 0; vb < BV; ++vb)
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        if (tok0 + 16 * vb + 4 * g + j >= P.V) b &= ~(1u << (vb * 4 + j));
            }
            f[rb] = b;
            if (__builtin_amdgcn_ballot_w64(b != 0)) {  // wave-uniform
                float2 *crow = P.cand + (size_t)(wrow0 + rb * 16 + n) * P.V + tok0 + 4 * g;
#pragma unroll
                for (int vb = 0; vb < BV; ++vb)
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        if (b & 1u << (vb * 4 + j)) crow[16 * vb + j].x = acc[vb][rb][j];
            }
        }
#pragma unroll
        for (int rb = 0; rb < RB; rb += 2) flags[rb / 2] = f[rb] | (rb + 1 < RB ? f[rb + 1] << 16 : 0u);
    } else {
        wave_softmax<RB>(acc, ms.bias_p, P.inv_T, tok0, P.V, wt, wr, pairs);
        __syncthreads();
        if (tid < TR) ms.park[tid] = merge_pairs<RB>(pairs, tid);
        if constexpr (kKeepZp) {
#pragma unroll
            for (int vb = 0; vb < BV; ++vb)
#pragma unroll
                for (int rb = 0; rb < RB; ++rb) zpk[vb][rb] = acc[vb][rb];
        } else {
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) {
                const int row = wrow0 + rb * 16 + n;
                if (row >= P.R) continue;
                float *dst = P.y_full + (size_t)row * P.zstride + tok0 + 4 * g;
#pragma unroll
                for (int vb = 0; vb < BV; ++vb) *reinterpret_cast<f32x4 *>(dst + 16 * vb) = acc[vb][rb];
            }
        }
    }

    // ---- amateur head
    run_pass(st, lds, acc);
    if constexpr (!FULL) {
        float bnd = -INFINITY;
        if (owner && pruning) bnd = read_bound(P.bound, P.R, myrow);
        for (int i = tid; i < TR * (kWordsPerTile + 1); i += NT) twords[i] = 0;  // and tcnt
        wave_softmax<RB>(acc, ms.bias_q, P.inv_T, tok0, P.V, wt, wr, pairs);
        __syncthreads();
        if (tid < TR) {
            const float2 p = ms.park[tid], q = merge_pairs<RB>(pairs, tid);
            ms.thr[tid] = p.x >= bnd + P.log_theta ? 1.f : 0.f;
            if (owner) P.partials[(size_t)myrow * P.ntiles + tile] = float4{p.x, p.y, q.x, q.y};
        }
        __syncthreads();
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
            const int rloc = wr * Q::WR + rb * 16 + n;
            uint32_t b = (flags[rb / 2] >> (rb % 2 * 16)) & 0xffffu;
            if (!__builtin_amdgcn_ballot_w64(b != 0)) continue;  // wave-uniform skip
            b = ms.thr[rloc] != 0.f ? b : 0u;
            float2 *crow = P.cand + (size_t)(row0 + rloc) * P.V + tok0 + 4 * g;
#pragma unroll
            for (int vb = 0; vb < BV; ++vb) {
                const uint32_t bv = (b >> (4 * vb)) & 15u;
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if (bv & 1u << j) crow[16 * vb + j].y = acc[vb][rb][j];
                if (bv) {
                    const int t = wt * WT + 16 * vb + 4 * g;  // the lane's first token of the block
                    atomicOr(&twords[rloc * kWordsPerTile + t / 32], bv << (t % 32));
                }
            }
            if (b) atomicAdd(&tcnt[rloc], __popc(b));
        }
        __syncthreads();
        // per (row, tile): the candidate count, and the bitmap words where it is nonzero
        for (int i = tid; i < TR * kWordsPerTile; i += NT) {
            const int r = i / kWordsPerTile, row = row0 + r;
            if (row < P.R && tcnt[r] > 0)
                P.bits[(size_t)row * P.wstride + tile * kWordsPerTile + i % kWordsPerTile] = twords[i];
        }
        if (owner) P.tcount[(size_t)myrow * P.ntiles + tile] = tcnt[tid];
    } else {
        // the lane's dense y row of row block rb, where its parked expert logits are: read
        // one row block ahead (the y stores in between keep the compiler from it; 2048 rows,
        // whole steps: 3113 -> 3097 us with 4096/2048-wide heads, proposals of 1024/512 1859 -> 1832)
        auto yrow_of = [&](int rb) {
            return P.y_full + (size_t)min(wrow0 + rb * 16 + n, P.R - 1) * P.zstride + tok0 + 4 * g;
        };
        f32x4 zn[BV];
        auto fetch_zp = [&](int rb) {
            const float *src = yrow_of(rb);
#pragma unroll
            for (int vb = 0; vb < BV; ++vb) zn[vb] = *reinterpret_cast<const f32x4 *>(src + 16 * vb);
            __builtin_amdgcn_sched_barrier(0);
        };
        if constexpr (!kKeepZp) fetch_zp(0);
        wave_softmax<RB>(acc, ms.bias_q, P.inv_T, tok0, P.V, wt, wr, pairs);
        const float s1f = 1.f + P.s;
        // per row: statistics of y over the lane's tokens (ascending, so a strict
        // comparison keeps the lowest id on ties), merged over the wave's lanes of that
        // row and then over the token waves in order
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
            const int rloc = wr * Q::WR + rb * 16 + n, row = row0 + rloc;
            float *yrow = yrow_of(rb);
            const float pmax = ms.park[rloc].x;
            f32x4 zp[BV];
#pragma unroll
            for (int vb = 0; vb < BV; ++vb) {
                if constexpr (kKeepZp)
                    zp[vb] = zpk[vb][rb];
                else
                    zp[vb] = zn[vb];
            }
            if constexpr (!kKeepZp)
                if (rb + 1 < RB) fetch_zp(rb + 1);
            YStat st{-INFINITY, -1, -INFINITY, 0.f, 0.f, 0.f, 0.f, -1};
            f32x4 y[BV];
#pragma unroll
            for (int vb = 0; vb < BV; ++vb)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int t = tok0 + 16 * vb + 4 * g + j;
                    const bool ok = t < P.V;
                    const float p = zp[vb][j], q = acc[vb][rb][j];
                    y[vb][j] = ok ? s1f * p - P.s * q : -INFINITY;
                    st.a += ok ? __builtin_amdgcn_exp2f((p - pmax) * kLog2e) * (p - q) : 0.f;
                    st.ip = (ok && st.ip < 0 && p == pmax) ? t : st.ip;
                    if (ok && y[vb][j] > st.y1) {
                        st.y2 = st.y1;
                        st.y1 = y[vb][j];
                        st.i1 = t;
                        st.zp1 = p;
                        st.zq1 = q;
                    } else if (ok) {
                        st.y2 = fmaxf(st.y2, y[vb][j]);
                    }
                }
            if (P.store_y && row < P.R) {
#pragma unroll
                for (int vb = 0; vb < BV; ++vb) *reinterpret_cast<f32x4 *>(yrow + 16 * vb) = y[vb];
            }
            if (st.i1 >= 0) {
                const float ml = st.y1 * kLog2e;
#pragma unroll
                for (int vb = 0; vb < BV; ++vb)
#pragma unroll
                    for (int j = 0; j < 4; ++j) st.ys += __builtin_amdgcn_exp2f(fmaf(y[vb][j], kLog2e, -ml));
            }
            st = ystat_merge(st, ystat_shfl_xor(st, 16));
            st = ystat_merge(st, ystat_shfl_xor(st, 32));
            if (g == 0) ys[wt * TR + rloc] = st;
        }
        __syncthreads();
        if (owner) {
            const float2 p = ms.park[tid], q = merge_pairs<RB>(pairs, tid);
            YStat st = ys[tid];
#pragma unroll
            for (int w = 1; w < TW; ++w) st = ystat_merge(st, ys[w * TR + tid]);
            float4 *dst = P.ypart + ((size_t)myrow * P.ntiles + tile) * 2;
            dst[0] = float4{st.y1, st.ys, st.y2, st.a};
            dst[1] = float4{__int_as_float(st.i1), st.zp1, st.zq1, __int_as_float(st.ip)};
            P.partials[(size_t)myrow * P.ntiles + tile] = float4{p.x, p.y, q.x, q.y};
        }
    }
}

template <int RB, bool FULL, bool ONE>
__global__ __launch_bounds__(NT, 1) void lmhead_wide_kernel(Plan P, Inputs in) {
#ifdef __HIP_DEVICE_COMPILE__  // the host pass does not know the asm constraints
    using Q = Geo<RB>;
    __shared__ __align__(256) char lds[Q::RING];  // (the k-step flip needs 128)
    __shared__ __align__(16) Misc<RB> ms;
    // workgroup 0 clears this call's row bounds and sequence counters first
    if (blockIdx.x == 0) clear_call_state(P.ctl, P.bound, kBoundCopies * P.R, P.seqdone, 2 * P.B);
    // workgroup -> (vocabulary tile, row tile); the row tiles of one vocabulary tile
    // are dispatched back to back on the same XCD (workgroup id modulo 8), so the
    // tile's weights are read from HBM once and from that XCD's L2 otherwise
    const int nrt = (P.R + Q::TR - 1) / Q::TR;
    const int id = blockIdx.x, xcd = id % 8, local = id / 8;
    const int tile = (local / nrt) * 8 + xcd;
    if (tile >= P.ntiles) return;
    const int row0 = (local % nrt) * Q::TR;
    if (wave_id() < TW)
        wide_tile<RB, FULL, 0, ONE>(P, in, tile, row0, lds, ms);
    else
        wide_tile<RB, FULL, 1, ONE>(P, in, tile, row0, lds, ms);
#endif
}

template <int RB, bool FULL>
hipError_t launch_rb_full(const Plan &p, const Inputs &in, hipStream_t st) {
    const int nrt = (p.R + Geo<RB>::TR - 1) / Geo<RB>::TR;
    const int groups = ((p.ntiles + 7) / 8) * 8 * nrt;
    if constexpr (RB > kStreamRowsLarge / 32) {  // (fewer rows than one tile of those: the streaming kernel)
        if (nrt == 1) {
            hipLaunchKernelGGL((lmhead_wide_kernel<RB, FULL, true>), dim3(groups), dim3(NT), 0, st, p, in);
            return hipGetLastError();
        }
    }
    hipLaunchKernelGGL((lmhead_wide_kernel<RB, FULL, false>), dim3(groups), dim3(NT), 0, st, p, in);
    return hipGetLastError();
}

template <int RB>
hipError_t launch_rb(const Plan &p, const Inputs &in, hipStream_t st) {
    return p.full ? launch_rb_full<RB, true>(p, in, st) : launch_rb_full<RB, false>(p, in, st);
}

}  // namespace

// The row shapes are compiled in three translation units of two shapes each
// (lmhead_wide45.hip and lmhead_wide67.hip include this file).
#ifndef DCD_WIDE_LO
#define DCD_WIDE_LO 8
#define DCD_WIDE_LAUNCH launch_lmhead_wide89
#endif
hipError_t DCD_WIDE_LAUNCH(const Plan &p, const Inputs &in, int rb, hipStream_t st) {
    return rb == DCD_WIDE_LO ? launch_rb<DCD_WIDE_LO>(p, in, st) : launch_rb<DCD_WIDE_LO + 1>(p, in, st);
}

#if DCD_WIDE_LO == 8
hipError_t launch_lmhead_wide(const Plan &p, const Inputs &in, hipStream_t st) {
    const int rb = p.wide;
    if (rb < 6) return launch_lmhead_wide45(p, in, rb, st);
    return rb < 8 ? launch_lmhead_wide67(p, in, rb, st) : launch_lmhead_wide89(p, in, rb, st);
}
#endif

}  // namespace dcd
