// Persistent kernel for groups of workgroups that fit one XCD: the recurrence of one (layer, direction, block of
// 16 sequences) never leaves the L2 of the XCD its workgroups run on.
//
// Decomposition and arithmetic are those of wavefront_ll.hip (paper Section 2.2: one group of workgroups per
// (layer, direction) of the unrolled grid; a workgroup owns RT * 4 hidden units of one block of up to 16 sequences;
// W_hh in the registers of four h waves that split K, W_ih in those of four x waves that work a step ahead).  What
// bounds a step at these sizes is the exchange of h between the workgroups, and its cost is a matter of where the
// data meets (this kernel, us per step, one bf16 layer of 128 / 256 / 512 units, 16 sequences; rnn_model_set_device_scope):
//     device-scope stores (written through to memory), device-scope loads     1.05 / 1.41 / 2.24
//     plain stores (they stay in the XCD's L2), loads that bypass the L1       0.76 / 0.94 / 1.09
// The second line needs every workgroup of a group on one XCD.  The dispatcher deals consecutive workgroups to the
// XCDs in turn, so the launch numbers its groups by blockIdx % 8; nothing relies on that: every workgroup publishes
// the XCC it really runs on before the first step (while its weights travel), and a group that finds itself on more
// than one uses device-scope stores instead.
// A bf16 layer of 640 to 1024 units needs more workgroups than an XCD has compute units: its group is laid over two, always with
// device-scope stores.  What that still gains over tagged words (half the bytes, MFMA fragments straight from the load) stands at
// the rule that chooses it; 16 sequences through a layer of 1024 units take 1.7 us a step, one 1.4 (tagged words 4 and 1.9).
// Layers of 1280 to 2048 units are laid over all eight, 8 units a workgroup (160 to 256 of them, one layer in a launch): every
// workgroup brings in the whole state, 16 sequences x 3 KiB at 1536 units, 9.4 MiB a step over the chip, 93 % of the requests found in
// the L2s, and a step takes 1.5 (one sequence) to 1.9 us (16; tagged words 2.9 to 6.8).  At 2048 units the state of more than eight
// sequences comes in two halves, one after the other: its fragments do not all fit the registers beside the weights (2.3 us).
// What such a group waits for most is a poll that came too early (see PAUSE_MORE).
//
// Layout of the exchanged state: 16-byte chunks (8 bf16 or 4 fp32 units of one sequence), chunk-major, the sequences of
// the block side by side (room for 4, 8 or 16, so that a workgroup's chunks do not share a half line with another's).  A lane's MFMA B
// fragment is one chunk, so a load instruction of a wave brings a whole K block of 16 sequences from 8 consecutive cache lines straight
// into the registers the matrix instruction reads: no tags, no staging through LDS.  Whether a chunk has been written is told from the
// data: a slot is filled with the bit pattern of all ones (two bf16 NaNs; one fp32 NaN) several steps before it is used, no published
// value has that pattern (a NaN is published with another one), and what is stored at once (8 bytes in bf16, 4 in fp32) is checked at
// once.  Order: a wave marks slot s + AHEAD in step s; before it publishes slot s it has waited for loads issued after it had marked slot
// s + 1, and memory operations of a wave complete in order, so whoever has seen slot s finds slot s + 1 marked or written.  The first
// AHEAD slots are marked before the group's start words are published.
//
// For layers in the same launch the layer below hands its state to the layer above through a second sequence with
// device-scope stores (the two may run on different XCDs); the x waves do that, and write the layer output, from
// LDS, so that no store other than the state itself stands before the next poll of an h wave.
// Every wait is bounded (poll budget, shared status word), so the grid always drains.
//
// What a step costs, for 512 units and 16 sequences (clocks of 2.4 GHz, each with its stamp of some 40; the slots of the state used in
// turn): from the tile's sums to the request of the next state 590 (gather, store, mark, tile to the x waves, loop), the state 620 (880
// with a slot for every step; the same there with one load instead of four and without the loads of the x waves, so that it is a round
// trip and no queue), products 290, partial sums to LDS 120, barrier 190, sum 225, gates 330.  Asking sooner behind the publication makes
// polls fail (20 to 90 %, 600 clocks each): 5 to 45 % longer.  Multiplying what has come while the rest travels: 0 to 33 % longer, since
// vain products hold up the next poll.  Words in LDS instead of the barrier: 0 to 12 % longer; input asked for behind the state instead
// of behind the barrier: 3 to 15 %.  Whole forward passes, on tagged words -> here: 2-layer LSTM of 512 units, both directions, batch 64,
// 256 steps 1.29 -> 0.55 ms; 2-layer GRU of 512 units at batch 8 183 -> 112 us for 100 steps; 12 fp32 layers of 64 units 159 -> 103 us; 2
// fp32 layers of 512 units at batch 64 1.15 -> 0.63 ms; GRU with the reset gate before the product (one launch per cell part without it)
// 1719 -> 98 us.
#include "wf_traits.h"

#include <type_traits>

// The variants are compiled in several translation units so that the build runs in parallel: this file is part 0 (bf16,
// and the public functions); wavefront_xcd_b.hip and so on include it with other values.
//   RNN_XR_DT    0 = bf16, 1 = fp32
//   RNN_XR_KIND  0 = LSTM and GRU with the plain cell, 1 = with the peephole and clipping terms, 2 = the GRU that applies the
//                reset gate before the candidate's recurrent product (always with the clipping term)
//   RNN_XR_APART (bf16, groups on an XCD each) 1 = the sums of the two products apart (see there)
#ifndef RNN_XR_DT
#define RNN_XR_DT 0
#endif
#ifndef RNN_XR_KIND
#define RNN_XR_KIND 0
#endif
#ifndef RNN_XR_APART
#define RNN_XR_APART 0
#endif
//   RNN_XR_WIDE  1 = groups on two XCDs, 2 = on all of them
#ifndef RNN_XR_WIDE
#define RNN_XR_WIDE 0
#endif

namespace rnn {
namespace {

constexpr int AHEAD = XCD_AHEAD;                // steps between marking a slot of the state and publishing it
constexpr int AHEAD_UP = 8;                     // the same for the sequence handed to the layer above: an x wave of the first layer has up
                                                // to three steps of loads in flight (two buffers and the lead), so that what it marked in a
                                                // step is known to be done that much later: before the slot in front of it is published
constexpr uint32_t UNWRITTEN = 0xFFFFFFFFu;
enum { X_PLAIN, X_BELOW, X_PROJECTED };          // where an x wave's input comes from: a finished tensor, the layer below, a projection
constexpr int CELL_GRU_RB = 2;                  // GRU, reset gate before the candidate's recurrent product

struct XRBf16 : TraitsBf16 {
    static constexpr int EPC = 8;               // elements per 16-byte chunk
    static constexpr int MPL = 1;               // matrix instructions per loaded chunk
    static constexpr int MMA_CLOCKS = 16;       // clocks one of them keeps the matrix unit busy
    static constexpr int PUB_LANES = 16;        // lanes that store a tile: one per sequence, 4 units each
    typedef uint64_t pub_t;
    static __device__ inline frag part(const u32x4& v, int) { return __builtin_bit_cast(frag, v); }
    // running maximum of the words that tell whether a chunk has been written (8 bytes are stored at once)
    static __device__ inline uint32_t seen(uint32_t m, const u32x4& v) { return max(m, max(v[0], v[2])); }
    static __device__ inline u32x4 pack(const float* f) {
        u32x4 r;
#pragma unroll
        for (int i = 0; i < 4; ++i) r[i] = (uint32_t)f32_to_bf16(f[2 * i]) | ((uint32_t)f32_to_bf16(f[2 * i + 1]) << 16);
        return r;
    }
    // the tile's values of one sequence: lanes n, n + 16, n + 32, n + 48 hold units 0..3 of sequence n; valid in lanes < 16
    static __device__ inline void gather(elem state, elem outv, pub_t& s, pub_t& o) {
        uint32_t v0, v1, v2, v3;
        gather_rows((uint32_t)state | ((uint32_t)outv << 16), v0, v1, v2, v3);
        const uint32_t lo = min((v0 & 0xFFFFu) | (v1 << 16), UNWRITTEN - 1), hi = min((v2 & 0xFFFFu) | (v3 << 16), UNWRITTEN - 1);
        s = (uint64_t)lo | ((uint64_t)hi << 32);
        o = (uint64_t)((v0 >> 16) | (v1 & 0xFFFF0000u)) | ((uint64_t)((v2 >> 16) | (v3 & 0xFFFF0000u)) << 32);
    }
    static __device__ inline pub_t mark() { return ~0ull; }
    // byte offset inside a slot of what this lane stores of the tile whose first unit is unit0
    static __device__ inline uint32_t pub_off(int unit0, int Bs, int lane) {
        return ((uint32_t)(unit0 >> 3) * Bs + (lane & 15)) * 16u + ((unit0 >> 2) & 1) * 8u;
    }
    static __device__ inline int pub_unit(int) { return 0; }     // first unit inside the tile of what a lane stores
    typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;
    template <int AUX>
    static __device__ inline void store(__amdgpu_buffer_rsrc_t r, pub_t v, uint32_t voff, uint32_t soff) {
        __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, v), r, voff, soff, AUX);
    }
};

struct XRF32 : TraitsF32 {
    static constexpr int EPC = 4;
    static constexpr int MPL = 4;
    static constexpr int MMA_CLOCKS = 32;
    static constexpr int PUB_LANES = 64;        // every lane stores its own unit
    typedef uint32_t pub_t;
    // K order inside a chunk block: matrix instruction j takes unit 4 * (lane / 16) + j of the 16 (weights likewise)
    static __device__ inline frag part(const u32x4& v, int j) { return __uint_as_float(v[j]); }
    static __device__ inline uint32_t seen(uint32_t m, const u32x4& v) { return max(max(m, max(v[0], v[1])), max(v[2], v[3])); }
    static __device__ inline u32x4 pack(const float* f) {
        return u32x4{__float_as_uint(f[0]), __float_as_uint(f[1]), __float_as_uint(f[2]), __float_as_uint(f[3])};
    }
    static __device__ inline void gather(elem state, elem outv, pub_t& s, pub_t& o) {
        s = min(__float_as_uint(state), UNWRITTEN - 1);
        o = __float_as_uint(outv);
    }
    static __device__ inline pub_t mark() { return UNWRITTEN; }
    static __device__ inline uint32_t pub_off(int unit0, int Bs, int lane) {
        return ((uint32_t)(unit0 >> 2) * Bs + (lane & 15)) * 16u + (lane >> 4) * 4u;
    }
    static __device__ inline int pub_unit(int lane) { return lane >> 4; }
    template <int AUX>
    static __device__ inline void store(__amdgpu_buffer_rsrc_t r, pub_t v, uint32_t voff, uint32_t soff) {
        __builtin_amdgcn_raw_buffer_store_b32(v, r, voff, soff, AUX);
    }
};

// A word in LDS that waves watch without a barrier.  (Through the LDS address space: a volatile access by a generic pointer
// is a flat one, which waits for every memory operation the wave has in flight.)
typedef volatile __attribute__((address_space(3))) unsigned lds_word;
__device__ inline void lds_put(unsigned* p, unsigned v) { *(lds_word*)p = v; }
__device__ inline unsigned lds_get(unsigned* p) { return *(lds_word*)p; }
typedef volatile __attribute__((address_space(3))) u32x4 lds_chunk;

// Buffer descriptor over `bytes` bytes at p (wave-uniform; said so, which keeps it in scalar registers).
__device__ inline __amdgpu_buffer_rsrc_t uniform_rsrc(const void* p, uint32_t bytes) {
    const uint64_t b = reinterpret_cast<uint64_t>(p);
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)b), hi = __builtin_amdgcn_readfirstlane((uint32_t)(b >> 32));
    return __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void*>(((uint64_t)hi << 32) | lo), 0,
                                             __builtin_amdgcn_readfirstlane((int)bytes), 0x00020000);
}

// K block b of those that a load brought, SEQS sequences of each, in lanes 0 .. SEQS - 1 of every 16.
template <int SEQS>
__device__ inline u32x4 rotate(const u32x4& v, int b) {
    if (b == 0) return v;
    u32x4 r;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
#define ROTATE_BY(k) case k: r[i] = __builtin_amdgcn_mov_dpp(v[i], 0x120 + 16 - k, 0xF, 0xF, true); break;   // row_ror
        switch (b * SEQS) {
            ROTATE_BY(2) ROTATE_BY(4) ROTATE_BY(6) ROTATE_BY(8) ROTATE_BY(10) ROTATE_BY(12) ROTATE_BY(14)
            default: __builtin_unreachable();
        }
#undef ROTATE_BY
    }
    return r;
}

// cell_update with what the compiler makes of it in the tag-in-data kernel spelled out: which of the two products of the new state is
// rounded by itself.  (With peepholes it makes the same of both kernels.)
template <int CELL, bool EXT>
__device__ inline float cell_update_tagged(const float a[SLOTS], float h_prev, float& c, const CellExt& ext) {
    if constexpr (CELL == CELL_LSTM) {
        if constexpr (EXT) return cell_update_ext<CELL>(a, h_prev, c, ext);
        c = __builtin_fmaf(sigmoid_f(a[1]), c, __fmul_rn(sigmoid_f(a[0]), tanh_f(a[2])));
        return sigmoid_f(a[3]) * tanh_f(c);
    } else {
        auto limit = [&](float v) { return EXT ? limit_to(v, ext.lim) : v; };
        const float r = sigmoid_f(limit(a[0])), z = sigmoid_f(limit(a[1])), n = tanh_f(limit(__builtin_fmaf(r, a[3], a[2])));
        return __builtin_fmaf(z, h_prev, __fmul_rn(1.0f - z, n));
    }
}

// LN / XLN: 16-byte chunks a lane loads per wave of the state / of the layer input (a wave's quarter of H is 4 * EPC * LN
// units; K blocks of the input are dealt to the waves in turn, and those beyond its width get zero weights).  The first layer
// of a launch may have its input product done by a projection launch (p.gx): its x waves then only bring that in.
// PK: K blocks that a load of the state brings (see packed_blocks).
template <class TR, int CELL, int RT, int LN, int XLN, bool EXT, bool APART, int PK>
__global__ __launch_bounds__(512) void wavefront_xcd_kernel(WavefrontXcdArgs p) {
    constexpr bool RB = CELL == CELL_GRU_RB;
    constexpr int GATES = RB ? CELL_GRU : CELL;
    typedef typename TR::elem elem;
    typedef typename TR::frag frag;
    typedef typename TR::pub_t pub_t;
    constexpr int EPC = TR::EPC, MPL = TR::MPL;
    constexpr int NW = 8;
    constexpr int NOWN = 1;                          // tiles finished by one wave (arrays of one and loops over them: with scalars
                                                     // the compiler contracts and orders the gate phase otherwise, and 2 GRU
                                                     // layers of 256 units, reset gate first, take 110 us for 64 steps instead of 104)
    static_assert(RT <= 4, "one tile per wave");
    // Layers of 640 to 1536 units sum in the order of the tag-in-data kernel, which ran them before (up to 1024 units it still does on few
    // steps): the same results, to the bit, on inputs H or H / 2 wide and behind a projection.  At 1280 and 1536 units that order is also
    // shorter than one of its own, each workgroup from another K block on (48 steps, us: 2 layers of 1280, batch 8 214 -> 206, 1 on 1032
    // values, batch 16 117 -> 106; 2 of 1536, batch 16 255 -> 240); up to 1024 units it costs up to 4 % (64 steps: 1, 2 and 4 layers of
    // 768, batch 4, 92.0 -> 94.5, 97.1 -> 101, 114 -> 120, of 1024 105 -> 106, 111 -> 111, 119 -> 123; batch 16, 2 of 1024 118 -> 116).
    // At 2048 units it does not fit the registers.
    constexpr bool TAGGED_ORDER = RNN_XR_WIDE && LN <= 12;
    // ... the i-th block of four chunks of wave w: of an input KX wide a quarter of the blocks, not every fourth; none from there on
    auto quarter_block = [](int i, int w, int KX) -> int {
        const int mine = XLN == LN ? LN : (KX + 16 * EPC - 1) / (16 * EPC);
        return i < mine ? w * mine + i : 4 * mine;
    };
    // A wave numbers the tiles from its own on, so that (RT = 4) it keeps its own tile's partial sum as acc[0].
    constexpr bool KEEP = RT == 4;
    constexpr int OTHERS = KEEP ? 3 : 4;             // partial sums of a tile that go through LDS
    constexpr int PART = OTHERS * RT * 64;           // f32x4 entries of one set of them
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
    f32x4* red = reinterpret_cast<f32x4*>(smem_raw);              // [2][RT tiles][OTHERS waves][64 lanes]
    constexpr int XPART = 4 * RT * 64;
    f32x4* xacc = red + 2 * PART;                                 // [2][4][RT][64]: x wave w to h wave w
    pub_t* pub = reinterpret_cast<pub_t*>(xacc + 2 * XPART);      // [RT][PUB_LANES]
    unsigned* done = reinterpret_cast<unsigned*>(pub + RT * TR::PUB_LANES);   // [4] steps whose tile h wave w has handed over
    unsigned* ready = done + 4;                                   // [4] steps whose input part x wave w has handed over
    unsigned* placed = ready + 4;                                 // 1: the whole group runs on one XCD
    constexpr int TURN = 4 * (16 + 2);                            // u32x4 entries to turn one load of rows in: [4 chunks][16 rows + 2]
    u32x4* turn = reinterpret_cast<u32x4*>(smem_raw + (((size_t)(2 * PART + 2 * XPART) * sizeof(f32x4) +
                                                        (size_t)RT * TR::PUB_LANES * sizeof(pub_t) + 9 * sizeof(unsigned) + 15) & ~(size_t)15));   // [4 x waves][XLN][TURN]

    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int w = wv & 3;                            // K quarter
    const int n = lane & 15, q = lane >> 4;
    auto tile_of = [&](int j) -> int { return KEEP ? (w + j) & 3 : j; };   // this wave's j-th tile

    // workgroup b runs on XCD b % 8: gpx groups of nrb workgroups on each, or on each pair of neighbouring XCDs, or on all eight (as
    // much of a group on each; consecutive row blocks, which write neighbouring chunks, stay together)
    const int spread = p.span == 8 ? 3 : p.span == 2 ? 1 : 0;
    const int here = p.nrb >> spread;                             // workgroups of a group on one XCD
    const int gi = (int)(blockIdx.x >> 3) / here;
    const int rb = (int)(blockIdx.x >> 3) - gi * here + (int)(blockIdx.x & (p.span - 1)) * here;
    const int g = ((int)(blockIdx.x & 7) >> spread) * p.gpx + gi; // (cb, d, ll), the layers of a column block side by side
    if (g >= p.LP * p.D * p.ncb) return;
    const int ll = g % p.LP, d = (g / p.LP) % p.D, cb = g / (p.LP * p.D);
    const int l = p.l0 + ll, ld = ll * p.D + d;
    const bool fused = RNN_XR_WIDE < 2 && ll > 0;    // (launches of groups on all XCDs hold one layer)
    const bool project = ll == 0 && p.gx != nullptr;
    const bool last = ll == p.LP - 1;                // writes the layer output; the others hand their state to the layer above
    const int H = p.H, T = p.T, B = p.B;
    const int Bs = p.stride;                         // sequences side by side in a chunk row
    const int ncol = min(16, B - cb * 16);
    const int nc = min(n, ncol - 1);                 // columns beyond the block repeat its last sequence and are never stored
    const bool valid = n < ncol;
    const int col = cb * 16 + nc;
    const uint32_t epoch = p.epoch;
    const uint32_t slot_bytes = (uint32_t)(H / EPC) * Bs * 16u;
    const int ring = p.ring;                         // slots of a state sequence: a power of two, or more than T
    const size_t seq_bytes = (size_t)min(ring, T) * slot_bytes;
    char* hbase = static_cast<char*>(p.hseq) + (size_t)g * (RB ? 2 : 1) * seq_bytes;
    const __amdgpu_buffer_rsrc_t hrs = uniform_rsrc(hbase, (uint32_t)seq_bytes);
    const __amdgpu_buffer_rsrc_t rrs = uniform_rsrc(hbase + (RB ? seq_bytes : 0), (uint32_t)seq_bytes);   // r * h
    // sequences between layers: [cb][ll < LP - 1][T]
    const size_t xseq_bytes = (size_t)T * slot_bytes;
    char* xbase = static_cast<char*>(p.xseq) + ((size_t)cb * (p.LP - 1) + ll) * xseq_bytes;
    const __amdgpu_buffer_rsrc_t urs = uniform_rsrc(xbase, last ? 0u : (uint32_t)xseq_bytes);             // up, to the layer above
    const __amdgpu_buffer_rsrc_t brs = uniform_rsrc(xbase - xseq_bytes, fused ? (uint32_t)xseq_bytes : 0u);   // from the layer below
    const int rmask = ring - 1;
    auto slot_of = [&](int s) -> uint32_t { return (uint32_t)(ring > T ? s : (s & rmask)) * slot_bytes; };
    bool aborted = false;
    auto give_up = [&](unsigned spins) {
        if (ld_dev_u32(p.status) != 0u || spins >= p.spin_limit) {
            st_dev_u32(p.status, 1u);
            aborted = true;
        }
    };

    // ---- start: mark the first slots, say where this workgroup runs ------------------------------
    const bool shake = T > 1 || p.LP > 1 || RB || p.in_place;   // else: a single step of a single layer exchanges nothing
    if (tid < 8) done[tid] = 0u;                     // (and ready)
    if (shake && wv == NW - 1) {
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) {
            const uint32_t off = TR::pub_off((rb * RT + rt) * 4, Bs, lane);
            if (valid && lane < TR::PUB_LANES)
                for (int s = 0; s < AHEAD_UP && s < T; ++s) {
                    if (s < AHEAD) TR::template store<16>(hrs, TR::mark(), off, slot_of(s));
                    if (RB && s < AHEAD) TR::template store<16>(rrs, TR::mark(), off, slot_of(s));
                    if (!last) TR::template store<16>(urs, TR::mark(), off, (uint32_t)s * slot_bytes);
                }
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    }
    auto start_word = [&]() {                        // last wave
        // XCC_ID: hardware register 20, bits 3:0
        const uint32_t xcc = __builtin_amdgcn_s_getreg(20 | (0 << 6) | (3 << 11));
        if (lane == 0) st_dev_u64(p.flagv + (size_t)g * p.nrb + rb, ((uint64_t)epoch << 32) | xcc);
    };
    if (shake && wv == NW - 1 && !p.in_place) start_word();
    auto start_wait = [&]() {                        // last wave: everybody this workgroup exchanges data with has started
        // Every workgroup reads the h0 of all units.  Where an output takes its place, a start word says as well that this has
        // been read (otherwise the exchange orders it: whoever writes hT has seen the states of step 0).
        if (p.in_place) {
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            __syncthreads();
            if (wv == NW - 1) start_word();
        }
        bool same = true;
        if (shake && wv == NW - 1) {
            for (int other = fused ? 1 : 0; other >= 0; --other) {
                const uint64_t* row = p.flagv + (size_t)(g - other) * p.nrb;
                uint64_t mine = 0;
                unsigned spins = 0;
                for (;;) {
                    bool ok = true;
                    for (int i = 0; i < p.nrb; i += 64) {
                        mine = ld_dev_u64(row + min(i + lane, p.nrb - 1));
                        ok = ok && (uint32_t)(mine >> 32) == epoch;
                    }
                    if (__all(ok) || aborted) break;
                    if ((++spins & 63u) == 0u || spins == 8u) give_up(spins);
                }
                if (other == 0) same = __all((uint32_t)mine == (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)mine));
            }
        }
        if (wv == NW - 1 && lane == 0) lds_put(placed, same && p.nrb <= 64 && !p.device_scope ? 1u : 0u);
        __syncthreads();
    };

    if (wv >= 4) {
        __builtin_amdgcn_s_setprio(1);
        // ---- x waves: the input product, one step ahead of the h waves ------------------------------
        const int KX = fused ? H : p.I;              // width of this layer's input
        constexpr int NBUF = XLN <= 8 ? 2 : 1;       // steps of x in flight (a plain x comes from HBM; the widest steps are long)
        // Rows of the caller's tensor: a load whose four neighbouring lanes lie in four rows takes the address unit four times
        // as long as one whose neighbours share 64 bytes (64 against 16 clocks, measured), and h waves wait behind it.  So lanes
        // bring 64 bytes of a row together, and the wave turns them into fragments through LDS.
        const bool rows = !fused && !project && !p.x_blocked && ncol > 2;
        u32x4* const my_turn = turn + w * XLN * TURN;
        frag wx[RT][XLN * MPL];
        uint32_t xoff[XLN];                          // byte offset of this lane's chunk inside a step of x, or inside its row (rows of a
                                                     // batch-first x can lie 4 GiB apart: the row is in the 64-bit address)
        if (project) {
#pragma unroll
            for (int i = 0; i < XLN; ++i) xoff[i] = 0u;
        } else {
            // W_ih of all directions is one matrix [D * 4H, KX]; direction d owns rows d * 4H ...
            const elem* wih = static_cast<const elem*>(p.wih[ld]) + (size_t)d * SLOTS * H * KX;
#pragma unroll
            for (int i = 0; i < XLN; ++i) {
                const int chunk = (TAGGED_ORDER ? quarter_block(i, w, KX) : i * 4 + w) * 4 + q;
                const bool in = chunk * EPC < KX;    // beyond the input: zero weights, and any chunk that exists
                const int k = in ? chunk * EPC : 0;
                if (fused || p.x_blocked) xoff[i] = ((uint32_t)(k / EPC) * Bs + nc) * 16u;
                else if (!rows) xoff[i] = (uint32_t)k * (uint32_t)sizeof(elem);
                else {                               // lane 4 * r + c brings chunk c of row r
                    const int rc = (TAGGED_ORDER ? quarter_block(i, w, KX) : i * 4 + w) * 4 + (lane & 3);
                    xoff[i] = rc * EPC < KX ? rc * 16u : 0u;
                }
#pragma unroll
                for (int rt = 0; rt < RT; ++rt) {
                    const size_t row = (size_t)(rb * RT + tile_of(rt)) * 16 + n;
                    u32x4 v = *reinterpret_cast<const u32x4*>(wih + row * KX + k);
                    if (!in) v = u32x4{0, 0, 0, 0};
#pragma unroll
                    for (int j = 0; j < MPL; ++j) wx[rt][i * MPL + j] = TR::part(v, j);
                }
            }
        }
        // a step of a finished input: rows of the caller's tensor, or a slot of a sequence in the layout of the state; (project) the
        // four slot values of this lane's pair of tile w
        const size_t xstep = project ? (size_t)p.x_t * p.D * H * SLOTS * sizeof(float)
                             : p.x_blocked ? (size_t)(KX / EPC) * Bs * 16 : (size_t)p.x_t * KX * sizeof(elem);
        const char* xsrc = project ? reinterpret_cast<const char*>(p.gx + (((size_t)col * p.x_b * p.D + d) * H + min((rb * RT + w) * 4 + q, H - 1)) * SLOTS)
                           : static_cast<const char*>(p.xin) + (p.x_blocked ? (size_t)cb * T * xstep
                                                                           : (size_t)(rows ? cb * 16 + min(lane >> 2, ncol - 1) : col) * p.x_b * KX * sizeof(elem));
        u32x4 xb[NBUF][XLN];
        // The s-th step in this direction's order.  No branch stands between the loads and their use: where two ways of loading
        // meet, the compiler copies what they loaded, and waits for it there and then (an x from HBM then stops the x wave for its
        // whole latency in every step: 657 us instead of 615 for 2 layers of 512 units, both directions, batch 64, 256 steps).
        constexpr int XBELOW = XLN < LN ? XLN : LN;  // (layers above the first: as many loads as their H takes)
        constexpr int XPACKED = (XBELOW + PK - 1) / PK;   // ... several K blocks each, as the h waves bring the state
        if (PK > 1 && fused) {
#pragma unroll
            for (int i = 0; i < XPACKED; ++i) {
                const int block = min(i * PK + n / (16 / PK), XBELOW - 1);
                xoff[i] = ((uint32_t)((TAGGED_ORDER ? w * LN + block : block * 4 + w) * 4 + q) * Bs + min(n & (16 / PK - 1), ncol - 1)) * 16u;
            }
        }
        auto request_below = [&](int s, u32x4 (&v)[XLN]) {
            const uint32_t at = (uint32_t)min(s, T - 1) * slot_bytes;
#pragma unroll
            for (int i = 0; i < XPACKED; ++i) v[i] = __builtin_amdgcn_raw_buffer_load_b128(brs, xoff[i], at, 16);
        };
        auto request = [&](auto from, int s, u32x4 (&v)[XLN]) {
            const int sc = min(s, T - 1);
            const char* src = xsrc + (size_t)(d ? T - 1 - sc : sc) * xstep;
            if constexpr (decltype(from)::value == X_PROJECTED) v[0] = *reinterpret_cast<const u32x4*>(src);
            else {
#pragma unroll
                for (int i = 0; i < XLN; ++i) v[i] = *reinterpret_cast<const u32x4*>(src + xoff[i]);
            }
        };
        // layer output of the workgroup's tiles, or their state for the layer above
        elem* out = static_cast<elem*>(p.out);
        auto gates_done = [&](int s) {
            while (lds_get(done + w) < (unsigned)(s + 1)) __builtin_amdgcn_s_sleep(1);   // (every h wave takes every step, whatever became of its waits)
            asm volatile("" ::: "memory");
        };
        auto forward = [&](int s) {
            if (w >= RT) return;                     // x wave w takes the tile that h wave w finished
            gates_done(s);
            if (valid && lane < TR::PUB_LANES) {
                const pub_t v = pub[w * TR::PUB_LANES + lane];
                const int unit0 = (rb * RT + w) * 4;
                const int t = d ? T - 1 - s : s;
                if (!last) {
                    const uint32_t off = TR::pub_off(unit0, Bs, lane);
                    TR::template store<16>(urs, v, off, (uint32_t)s * slot_bytes);
                    if (s + AHEAD_UP < T) TR::template store<16>(urs, TR::mark(), off, (uint32_t)(s + AHEAD_UP) * slot_bytes);
                } else if (p.y_blocked) {
                    *reinterpret_cast<pub_t*>(reinterpret_cast<char*>(out) + ((size_t)cb * T + t) * p.D * slot_bytes +
                                              (size_t)d * slot_bytes + TR::pub_off(unit0, Bs, lane)) = v;
                } else if (unit0 < p.out_units) {
                    *reinterpret_cast<pub_t*>(out + ((size_t)t * p.y_t + (size_t)col * p.y_b) * (p.D * p.out_units) +
                                              (size_t)d * p.out_units + unit0 + TR::pub_unit(lane)) = v;
                }
            }
            asm volatile("" ::: "memory");
        };
        start_wait();
        // Between barriers s - 1 and s an x wave asks for the input of a later step (at once: the h waves are in their gates then,
        // and the address unit, which the state of the next step waits for, is free) and produces the input part of step
        // sx = s + lead.
        // With lead = 1 the part is there a step before h wave w picks it up, as the start of its accumulators, while its state
        // fragments travel; the product then waits until h wave w, on the same SIMD, is through its gates, whose vector
        // instructions otherwise queue behind matrix instructions one by one (2 layers of 512 units, both directions: a gate phase, sum
        // and publication with it, of 1078 clocks instead of 860).  A product of a few instructions, or of an input wider than the state,
        // which would come too late, does not wait in a launch of one layer (128 units, 48 steps, 16 groups or more: 51 us with the wait,
        // 45 without; with layers above, 2 of 128 units, 47 with it and 52 without).  A layer above another is a step later for it, so
        // deep stacks on few steps take lead = 0 there (p.lead): then the layer output of step s - 1 leaves behind the product, or before
        // it where that is long.  With the reset gate first, r * h goes round the group behind the barrier: a first layer whose input is
        // wider than its state, by more than four chunks a wave, asks before the barrier and multiplies in the step itself (1 layer of
        // 512 units on 848 values, 33 sequences, 20 steps: 54.7 us, 58.4 the other way).  Up to four chunks the product is short and
        // better done ahead (48 steps, late -> ahead: 2 layers of 64 to 256 units on 136 to 504 values, one sequence, 10 to 15 % shorter,
        // 16 sequences 0 to 12 %; 1 layer 1 to 4 %, but 2 % longer at 256 units, 40 sequences; fp32, on 136 and 224 values, 2 layers, one
        // sequence 8 to 15 % shorter, 16 sequences 3 to 5 % longer).
        constexpr bool LATE = RB && XLN > LN && XLN > 4;
        // In a launch of several fp32 layers of 256 units or more, on few steps, the first layer does without as well (p.lead_first): its
        // first barrier would wait for two long products, and every layer above with it (2 layers of 512 units, 16 sequences, us with
        // the lead -> without it: 3 steps 39.0 -> 34.3, 8 steps 64.3 -> 59.6, 16 steps 104 -> 99.5, 32 steps 169 -> 180; of 296 units, 3
        // steps 36.9 -> 32.0).  Short products lose by it from the first steps on (16 steps, 2 layers of 128 fp32 units 20.6 -> 22.4, of
        // 256 bf16 units 19.3 -> 21.2), and inputs wider than the state come too late (6 layers of 384 bf16 units on 1024 values, 100
        // steps, 137 -> 166).
        constexpr bool CHOICE = MPL > 1 && LN >= 4 && XLN == LN;
        const int lead = fused ? p.lead : LATE ? 0 : CHOICE ? p.lead_first : 1;
        constexpr int PRODUCT = XLN * MPL * RT * TR::MMA_CLOCKS;
        constexpr bool OUT_FIRST = PRODUCT > 512;
        const bool wait_gates = lead && w < RT && ((PRODUCT > 128 && XLN <= LN) || p.LP > 1);
        auto produce = [&](auto from, int sx, u32x4 (&cur)[XLN]) {
            constexpr int FROM = decltype(from)::value;
            constexpr bool BELOW = FROM == X_BELOW, PROJECTED = FROM == X_PROJECTED;
            constexpr int XL = PROJECTED ? 1 : BELOW ? XPACKED : XLN;
            const int s = sx - lead;                 // between barriers s - 1 and s
            bool sent = s <= 0 || s >= T;
            if (!lead && OUT_FIRST && !sent) { forward(s - 1); sent = true; }
            if (sx < T) {
                if constexpr (BELOW) {
                    unsigned spins = 0;
                    for (;;) {
                        uint32_t m = 0;
#pragma unroll
                        for (int i = 0; i < XL; ++i) m = TR::seen(m, cur[i]);
                        if (!__any(m == UNWRITTEN) || aborted) break;
                        if (!lead && !sent) { forward(s - 1); sent = true; }   // nothing to multiply yet
                        if ((++spins & 63u) == 0u || spins == 8u) give_up(spins);
                        request_below(sx, cur);
                        asm volatile("" ::: "memory");
                    }
                }
                // chunks beyond the input: zero like their weights (0 * infinity is no zero)
                if (!project && !(BELOW && PK > 1) && XL * 16 * EPC > KX) {
#pragma unroll
                    for (int i = 0; i < XL; ++i) {
                        const int chunk = (TAGGED_ORDER ? quarter_block(i, w, KX) : i * 4 + w) * 4;
                        if ((chunk + 4) * EPC > KX && (chunk + (rows ? lane & 3 : q)) * EPC >= KX) cur[i] = u32x4{0, 0, 0, 0};
                    }
                }
                if (!BELOW && rows) {                    // (no barrier: LDS operations of a wave keep their order)
#pragma unroll
                    for (int i = 0; i < XL; ++i) my_turn[i * TURN + (lane & 3) * 18 + (lane >> 2)] = cur[i];
                    asm volatile("" ::: "memory");
#pragma unroll
                    for (int i = 0; i < XL; ++i) cur[i] = my_turn[i * TURN + q * 18 + n];
                }
                if (wait_gates && !sent) gates_done(s - 1);
                f32x4 acc[RT];
#pragma unroll
                for (int rt = 0; rt < RT; ++rt) acc[rt] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
                if (!BELOW && project) {
                    if (KEEP) acc[0] = __builtin_bit_cast(f32x4, cur[0]);
                    else {
#pragma unroll
                        for (int rt = 0; rt < RT; ++rt)
                            if (rt == w) acc[rt] = __builtin_bit_cast(f32x4, cur[0]);
                    }
                } else {
#pragma unroll
                    for (int i = 0; i < (BELOW ? XBELOW : XL); ++i) {
                        const u32x4 v = BELOW && PK > 1 ? rotate<16 / PK>(cur[i / PK], i % PK) : cur[i];
#pragma unroll
                        for (int j = 0; j < MPL; ++j)
#pragma unroll
                            for (int rt = 0; rt < RT; ++rt) acc[rt] = TR::mfma(wx[rt][i * MPL + j], TR::part(v, j), acc[rt]);
                    }
                    // Results of a matrix instruction may be read a number of wait states after it was issued; the compiler
                    // counts them inside a block, but was seen not to where two branches join before the read (fp32, RT = 1).
#pragma unroll
                    for (int rt = 0; rt < RT; ++rt) asm volatile("" : "+v"(acc[rt]));
                    asm volatile("s_nop 7\n\ts_nop 7\n\ts_nop 3" : "+v"(acc[RT - 1]));
                }
#pragma unroll
                for (int rt = 0; rt < RT; ++rt) xacc[(sx & 1) * XPART + (w * RT + rt) * 64 + lane] = acc[rt];
                asm volatile("" ::: "memory");           // (LDS operations of a wave keep their order)
                if (lane == 0) lds_put(ready + w, (unsigned)(sx + 1));
            }
            if (!sent) forward(s - 1);
            if (!(LATE && !BELOW) && s >= 0 && s < T) {
                __syncthreads();
                if (RB) __syncthreads();
            }
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (BELOW) request_below(sx + 1, cur);
            else request(from, sx + NBUF, cur);
            __builtin_amdgcn_sched_barrier(0);
            if (LATE && !BELOW && s >= 0 && s < T) {
                __syncthreads();
                __syncthreads();
            }
        };
        // A projection is one load a step: in a loop of its own in the variants of three chunk loads and of more than four (64 steps,
        // us, as many loads of the same chunk as the layers above take -> one: 4 layers of 768 units, batch 8 and 16 169 -> 142 and
        // 198 -> 154, of 1024 190 -> 163 and 215 -> 204, of 640 158 -> 133 and 184 -> 149; 2 of 384, batch 1, 8 and 16 75 -> 77.5,
        // 82.8 -> 80 and 90 -> 79; but with four loads, 4 layers of 512 units at batch 1 and 8, 82 -> 83 and 90 -> 92; fp32 the same).
        // Launches of one layer take one or two loads for it as it is.
        constexpr bool OWN_LOOP = MPL == 1 && LN <= 8 && XLN >= LN && (XLN == 3 || XLN > 4);
        if (fused) {
            request_below(0, xb[0]);
            for (int sx = 0; sx < T + lead; ++sx) produce(std::integral_constant<int, X_BELOW>(), sx, xb[0]);
        } else if (OWN_LOOP && project) {
            constexpr std::integral_constant<int, OWN_LOOP ? X_PROJECTED : X_PLAIN> FROM{};
#pragma unroll
            for (int b = 0; b < NBUF; ++b) {
                request(FROM, b, xb[b]);
                __builtin_amdgcn_sched_barrier(0);
            }
            for (int s0 = 0; s0 < T + lead; s0 += NBUF)
#pragma unroll
                for (int b = 0; b < NBUF; ++b) produce(FROM, s0 + b, xb[b]);
        } else {
            constexpr std::integral_constant<int, X_PLAIN> FROM{};
#pragma unroll
            for (int b = 0; b < NBUF; ++b) {
                request(FROM, b, xb[b]);
                __builtin_amdgcn_sched_barrier(0);   // (in this order: the loop's waits count on it)
            }
            // (A whole number of rounds, beyond the last step where need be: a way round a step, or out of the loop between steps,
            // would make the compiler wait for the newest loads at the head of the loop.)
            for (int s0 = 0; s0 < T + lead; s0 += NBUF)
#pragma unroll
                for (int b = 0; b < NBUF; ++b) produce(FROM, s0 + b, xb[b]);
        }
        forward(T - 1);
        return;
    }

    // ---- h waves -------------------------------------------------------------------------------------
    __builtin_amdgcn_s_setprio(3);                   // the dependency chain runs through these
    const int rot = TAGGED_ORDER ? 0 : rb % LN;      // workgroups start at different K blocks: spreads them over the L2 channels
    frag wh[RT][LN * MPL];
    {
        const elem* whh = static_cast<const elem*>(p.whh[ld]);
#pragma unroll
        for (int i = 0; i < LN; ++i) {
            const int ir = i + rot >= LN ? i + rot - LN : i + rot;
            const int k = ((w * LN + ir) * 4 + q) * EPC;
#pragma unroll
            for (int rt = 0; rt < RT; ++rt) {
                const size_t row = (size_t)(rb * RT + tile_of(rt)) * 16 + n;
                const u32x4 v = *reinterpret_cast<const u32x4*>(whh + row * H + k);
#pragma unroll
                for (int j = 0; j < MPL; ++j) wh[rt][i * MPL + j] = TR::part(v, j);
            }
        }
    }
    constexpr int LOADS = (LN + PK - 1) / PK;
    constexpr int HL = LOADS > 12 ? LOADS / 2 : LOADS;   // loads of the state before the step, HL at a time (16 do not fit the
                                                     // registers beside 32 K blocks of weights)
    // With PK > 1 a lane brings sequence n % SEQS of K block i * PK + n / SEQS (in the order of wh) in load i.
    constexpr int SEQS = 16 / PK;
    const int own_seq = PK == 1 ? nc : min(n & (SEQS - 1), ncol - 1);
    auto block_of = [&](int i) -> int {
        const int b = PK == 1 ? i : min(i * PK + n / SEQS, LN - 1);
        return b + rot >= LN ? b + rot - LN : b + rot;
    };
    uint32_t hoff[PK == 1 ? 1 : LOADS];              // byte offset inside a slot (PK = 1: without the K block)
#pragma unroll
    for (int i = 0; i < (PK == 1 ? 1 : LOADS); ++i)
        hoff[i] = ((uint32_t)((w * LN + (PK == 1 ? 0 : block_of(i))) * 4 + q) * Bs + own_seq) * 16u;

    float c_reg[NOWN], h_reg[NOWN];
    f32x4 bias_reg[NOWN];
    CellExt ext_reg[EXT ? NOWN : 1];
    const int len = valid ? (p.lengths ? min(max(p.lengths[col], 0), T) : T) : 0;
    const int Hu = p.out_units_state;                // width of the caller's state tensors
    const size_t state_row = (size_t)(l * p.D + d) * p.state_b + col;
#pragma unroll
    for (int o = 0; o < NOWN; ++o) {
        const int unit = min((rb * RT + w + 4 * o) * 4 + q, H - 1);
        c_reg[o] = h_reg[o] = 0.0f;
        bias_reg[o] = *reinterpret_cast<const f32x4*>(p.bias[ld] + (size_t)unit * SLOTS);
        if constexpr (EXT) ext_reg[o] = load_cell_ext(GATES == CELL_LSTM ? p.peep[ld] : nullptr, H, unit, p.clip);
        if (valid && unit < Hu) {
            if (p.h0) h_reg[o] = p.h0[state_row * Hu + unit];
            if (p.c0) c_reg[o] = p.c0[state_row * Hu + unit];
        }
    }
    u32x4 hv[HL];                                    // B fragments of the state before the step, or PK of them each
    u32x4* const h0_rest = turn + 4 * XLN * TURN + (w * 64 + lane) * (LOADS - HL);   // the other half of h0, read with the first: an
                                                                                     // output may take its place
    const size_t own_row = PK == 1 ? state_row : (size_t)(l * p.D + d) * p.state_b + cb * 16 + own_seq;
#pragma unroll
    for (int i = 0; i < LOADS; ++i) {                // step 0: the caller's h0
        const int k = ((w * LN + block_of(i)) * 4 + q) * EPC;
        float f[EPC];
#pragma unroll
        for (int e = 0; e < EPC; ++e) f[e] = 0.0f;
        if (p.h0 && k < Hu) {
#pragma unroll
            for (int e = 0; e < EPC; ++e) f[e] = p.h0[own_row * Hu + k + e];
        }
        if (i < HL) hv[i < HL ? i : 0] = TR::pack(f);
        else h0_rest[i - HL] = TR::pack(f);
    }
    start_wait();
    const bool local = __builtin_amdgcn_readfirstlane((int)lds_get(placed)) != 0;

    auto ask = [&](__amdgpu_buffer_rsrc_t rs, int s, int first) {   // request HL loads of slot s
#pragma unroll
        for (int i = 0; i < HL; ++i) {
            if constexpr (PK == 1)
                hv[i] = __builtin_amdgcn_raw_buffer_load_b128(rs, hoff[0], slot_of(s) + (uint32_t)(block_of(first + i) * 64) * Bs, 16);
            else hv[i] = __builtin_amdgcn_raw_buffer_load_b128(rs, hoff[first + i], slot_of(s), 16);
        }
    };
    // Groups on several XCDs: a wave waits before its first request of a step.  A request that finds a chunk unwritten costs a whole
    // round trip through memory, and its answers delay the stores everybody waits for, so it is better sent late than too early; how late
    // depends on the shape, the step and the wave (those without a tile of their own ask first and were sent back in four steps of five),
    // so every wave finds out for itself: longer after a step that sent it back, a little shorter after every other (in balance it is
    // sent back once in 33 steps; in 25 at 640 and 768 units).  64 steps, us, without -> with it: 2 layers of 1024 units, batch 5 / 8 /
    // 16 147 / 154 / 175 -> 112 / 116 / 116, of 768, batch 8 / 16 125 / 140 -> 100 / 101, one of 1536, batch 1 / 16 147 / 167 -> 110 /
    // 123, of 2048 183 / 204 -> 149 / 162.  Other choices (sixteenths more, sixteenths less, at first): 16, 1, 10 up to 3 % longer, 48,
    // 1, 8 the same, 96, 1, 0 and the best constant of each shape 1 to 10 % longer.  Within one XCD the loop as it is is late enough
    // (retries in 0 to 30 % of the steps, 600 clocks each); there such pauses made 12 narrow layers 2 to 13 % longer and little shorter.
    // Sixteenths of a round of the loop, about 40 clocks.  (640 and 768 units, their fewer workgroups sooner through: 32, 1, 8 -> 24, 1,
    // 5, 64 steps, us, one layer, batch 1 and 8 85.1 and 90.1 -> 82.1 and 85.8, 87.1 and 91.3 -> 82.8 and 87.3; four, batch 2 and 12 111
    // and 117 -> 112 and 107, 106 and 118 -> 107 and 112.  Of 1024 units one layer gains 3 % by it, several lose 2 to 7, wider ones 0 to
    // 3.)
    constexpr int PAUSE_MORE = LN <= 6 ? 24 : 32, PAUSE_LESS = 1, PAUSE_FIRST = (LN <= 6 ? 5 : 8) * 16, PAUSE_MOST = 64 * 16;
    int pause = PAUSE_FIRST;
    unsigned in_vain = 0;                            // requests of the last fetch that found a chunk unwritten
    auto hold_back = [&]() {
        for (int i = __builtin_amdgcn_readfirstlane(pause) >> 4; i > 0; --i) asm volatile("s_nop 7");
    };
    // The chunks of slot s from `first` on in hv, waiting until all of them have been written; `meanwhile` runs while the first
    // request travels.
    auto fetch = [&](__amdgpu_buffer_rsrc_t rs, int s, int first, auto meanwhile) {
        unsigned spins = 0;
        for (;;) {
            ask(rs, s, first);
            if (spins == 0u) meanwhile();
            uint32_t m = 0;
#pragma unroll
            for (int i = 0; i < HL; ++i) m = TR::seen(m, hv[i]);
            if (!__any(m == UNWRITTEN) || aborted) break;
            if ((++spins & 63u) == 0u || spins == 8u) give_up(spins);
            asm volatile("" ::: "memory");
        }
        asm volatile("" ::: "memory");
        if (RNN_XR_WIDE) in_vain = spins;
    };
    // partial products of this wave's K quarter (of the loads from `first` on) added to acc
    auto multiply = [&](f32x4 (&acc)[RT], auto first) {
#pragma unroll
        for (int i = 0; i < HL * PK; ++i) {
            if (PK > 1 && first * PK + i >= LN) break;
            const u32x4 v = PK == 1 ? hv[i] : rotate<SEQS>(hv[i / PK], i % PK);
#pragma unroll
            for (int j = 0; j < MPL; ++j)
#pragma unroll
                for (int rt = 0; rt < RT; ++rt) acc[rt] = TR::mfma(wh[rt][(first * PK + i) * MPL + j], TR::part(v, j), acc[rt]);
        }
    };
    // all tiles but the wave's own go to LDS
    auto hand_over = [&](const f32x4 (&acc)[RT], int buf) {
#pragma unroll
        for (int rt = KEEP ? 1 : 0; rt < RT; ++rt)
            red[buf * PART + (tile_of(rt) * OTHERS + (KEEP ? rt - 1 : w)) * 64 + lane] = acc[rt];
    };
    // after the barrier: the sum of tile w over the four K quarters
    auto total = [&](const f32x4 (&acc)[RT], int buf) -> f32x4 {
        const int rt = min(w, RT - 1);
        f32x4 part[OTHERS];
#pragma unroll
        for (int k = 0; k < OTHERS; ++k) {
            // (quarters 0 and 1, 2 and 3 belong together: entry k is that of wave w - 1 - k, so for an even w the quarter beside it is
            // the last entry, for an odd one the first)
            const int entry = TAGGED_ORDER && KEEP && (w & 1) == 0 ? OTHERS - 1 - k : k;
            part[k] = red[buf * PART + (rt * OTHERS + entry) * 64 + lane];
        }
        __builtin_amdgcn_sched_barrier(0);           // (one LDS round trip)
        if constexpr (TAGGED_ORDER && KEEP) return (acc[0] + part[0]) + (part[1] + part[2]);
        if constexpr (TAGGED_ORDER) return (part[0] + part[1]) + (part[2] + part[OTHERS - 1]);
        return ((KEEP ? acc[0] : part[OTHERS - 1]) + part[0]) + (part[1] + part[2]);
    };
    auto publish = [&](__amdgpu_buffer_rsrc_t rs, pub_t v, int unit0, int s) {   // slot s of this lane's share; mark slot s + AHEAD
        if (valid && lane < TR::PUB_LANES) {
            const uint32_t off = TR::pub_off(unit0, Bs, lane);
            if (local) {
                TR::template store<0>(rs, v, off, slot_of(s));
                if (s + AHEAD < T) TR::template store<0>(rs, TR::mark(), off, slot_of(s + AHEAD));
            } else {
                TR::template store<16>(rs, v, off, slot_of(s));
                if (s + AHEAD < T) TR::template store<16>(rs, TR::mark(), off, slot_of(s + AHEAD));
            }
        }
    };
    for (int s = 0; s < T; ++s) {
        const int t = d ? T - 1 - s : s;
        // The recurrent product starts from the input part.  Not so in fp32, where one chain of sums as long as both products loses
        // precision (2 layers of 512 units, distance of hT from 64 bits 4.7e-7 against 3.6e-7), nor in layers of 640 units and more,
        // whose chains are the longest (cT after one step, 1536 units on 1536 values 1.92e-7 against 1.35e-7, 2048 on 2048 2.17e-7
        // against 1.45e-7; tagged words 1.37e-7 and 1.46e-7, and no time lost: 64 steps of 2 such layers 0 to 2 % shorter), nor in
        // passes that take a batch over from launches of larger tiles, which sum apart as well (p.apart; both directions of 512 units,
        // 72 sequences: larger tiles 1.29e-7, one chain 1.35e-7, apart 1.13e-7; 256 units, 136 sequences 1.14e-7, 1.18e-7, 1.08e-7.
        // Everywhere up to 512 units it would make calls 0 to 4 % longer): there (APART) the wave that finishes a tile sums the tile's
        // input part, and the bias, for itself meanwhile.
        f32x4 acc[RT], from_x;
        if constexpr (APART) from_x = TAGGED_ORDER ? f32x4{0.0f, 0.0f, 0.0f, 0.0f} : bias_reg[0];
        auto input_part = [&]() {                    // (every x wave takes every step, whatever became of its waits)
            if constexpr (APART) {
#pragma unroll
                for (int rt = 0; rt < RT; ++rt) acc[rt] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
                if (w < RT) {
                    // the words first, the sums behind them in one LDS round trip (operations of a wave keep their order)
                    u32x4 at;
                    f32x4 part[4];
                    do {
                        at = *(lds_chunk*)ready;
#pragma unroll
                        for (int k = 0; k < 4; ++k)
                            part[k] = __builtin_bit_cast(f32x4, (u32x4)*(lds_chunk*)&xacc[(s & 1) * XPART + (k * RT + (KEEP ? (w - k) & 3 : w)) * 64 + lane]);
                    } while (min(min(at[0], at[1]), min(at[2], at[3])) < (unsigned)(s + 1));
                    from_x += (part[0] + part[1]) + (part[2] + part[3]);
                }
            } else {
                while (lds_get(ready + w) < (unsigned)(s + 1)) {}
                asm volatile("" ::: "memory");
#pragma unroll
                for (int rt = 0; rt < RT; ++rt) acc[rt] = xacc[(s & 1) * XPART + (w * RT + rt) * 64 + lane];
            }
        };
        if (w >= RT && s > 0)                        // (no use in asking before the workgroup's own tiles are out)
            while (lds_get(done + (w & (RT - 1))) < (unsigned)s) __builtin_amdgcn_s_sleep(1);
        constexpr std::integral_constant<int, 0> FRONT{};
        if (s > 0) {
            if (RNN_XR_WIDE) hold_back();
            fetch(hrs, s - 1, FRONT, input_part);
            if (RNN_XR_WIDE) pause = in_vain ? min(pause + PAUSE_MORE, PAUSE_MOST) : max(pause - PAUSE_LESS, 0);
        } else input_part();
        multiply(acc, FRONT);
        if constexpr (HL < LOADS) {
            constexpr std::integral_constant<int, HL> REST{};
            if (s > 0) fetch(hrs, s - 1, REST, [] {});
            else {
#pragma unroll
                for (int i = 0; i < HL; ++i) hv[i] = h0_rest[i];
            }
            multiply(acc, REST);
        }
        hand_over(acc, RB ? 0 : (s & 1));
        __syncthreads();
        f32x4 pre[NOWN];
#pragma unroll
        for (int o = 0; o < NOWN; ++o) {
            pre[o] = total(acc, RB ? 0 : (s & 1));
            if constexpr (APART) pre[o] += from_x;
            if constexpr (!APART || TAGGED_ORDER) pre[o] += bias_reg[o];
        }
        float zg[RB ? NOWN : 1], nx[RB ? NOWN : 1];
        if constexpr (RB) {
            // r * h goes round the group before the candidate's recurrent product
#pragma unroll
            for (int o = 0; o < NOWN; ++o) {
                if (w + 4 * o < RT) {
                    const float r = sigmoid_f(limit_to(pre[o][0], ext_reg[o].lim));
                    zg[o] = sigmoid_f(limit_to(pre[o][1], ext_reg[o].lim));
                    nx[o] = pre[o][2];
                    float unused;
                    pub_t sv, ov;
                    TR::gather(TR::store_val(r * h_reg[o], unused), TR::zero(), sv, ov);
                    publish(rrs, sv, (rb * RT + w + 4 * o) * 4, s);
                }
            }
            static_assert(HL == LOADS, "the reset gate first: no variant of more than 512 units");
            fetch(rrs, s, FRONT, [] {});
#pragma unroll
            for (int rt = 0; rt < RT; ++rt) acc[rt] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
            multiply(acc, FRONT);
            hand_over(acc, 1);
            __syncthreads();
            pre[0][3] = total(acc, 1)[3] + bias_reg[0][3];
        }
#pragma unroll
        for (int o = 0; o < NOWN; ++o) {
            const int rt = w + 4 * o;
            if (rt < RT) {                           // uniform per wave
                const bool active = valid && t < len;
                float c_new = c_reg[o];
                float hn;
                if constexpr (RB) {
                    const float nn = tanh_f(limit_to(nx[o] + pre[o][3], ext_reg[o].lim));
                    hn = (1.0f - zg[o]) * nn + zg[o] * h_reg[o];
                } else {
                    const float a[SLOTS] = {pre[o][0], pre[o][1], pre[o][2], pre[o][3]};
                    if constexpr (TAGGED_ORDER) hn = cell_update_tagged<GATES, EXT>(a, h_reg[o], c_new, ext_reg[0]);
                    else if constexpr (EXT) hn = cell_update_ext<GATES>(a, h_reg[o], c_new, ext_reg[o]);
                    else hn = cell_update<GATES>(a, h_reg[o], c_new);
                }
                if (active) {
                    float kept;
                    (void)TR::store_val(hn, kept);
                    c_reg[o] = c_new;
                    h_reg[o] = kept;
                }
                float unused;
                const elem state_v = TR::store_val(h_reg[o], unused);   // held value when inactive
                const elem out_v = active ? state_v : TR::zero();
                const int unit0 = (rb * RT + rt) * 4;
                pub_t sv, ov;
                TR::gather(state_v, out_v, sv, ov);
                if (s + 1 < T) publish(hrs, sv, unit0, s);
                if (lane < TR::PUB_LANES) pub[rt * TR::PUB_LANES + lane] = last ? ov : sv;
                asm volatile("" ::: "memory");       // (LDS operations of a wave keep their order)
                if (lane == 0) lds_put(done + w, (unsigned)(s + 1));
            }
        }
        if (p.ticks && tid == 0 && rb == 0 && cb == 0) p.ticks[(size_t)ld * T + s] = wall_clock64();
    }

#pragma unroll
    for (int o = 0; o < NOWN; ++o) {
        const int unit = (rb * RT + w + 4 * o) * 4 + q;
        if (w + 4 * o < RT && valid && unit < Hu) {
            if (p.hT) p.hT[state_row * Hu + unit] = h_reg[o];
            if (p.cT && GATES == CELL_LSTM) p.cT[state_row * Hu + unit] = c_reg[o];
        }
    }
}

// Forces one workgroup per compute unit: more than half of the 160 KiB.
constexpr size_t MIN_LDS = 84 * 1024;

constexpr bool apart(int MPL) { return MPL > 1 || RNN_XR_WIDE || RNN_XR_APART; }

template <class TR, int CELL, int RT, int LN, int XLN, bool EXT, int PK>
hipError_t launch_variant(const WavefrontXcdArgs& a, hipStream_t stream) {
    const size_t need = (size_t)((RT == 4 ? 6 : 8) + 8) * RT * 64 * sizeof(f32x4) + (size_t)RT * TR::PUB_LANES * sizeof(typename TR::pub_t) +
                        9 * sizeof(unsigned) + 16 + (size_t)4 * XLN * 4 * 18 * 16 + (LN > 12 ? (size_t)4 * 64 * (LN / 2) * 16 : 0);
    const size_t smem = need < MIN_LDS ? MIN_LDS : need;
    auto kern = wavefront_xcd_kernel<TR, CELL, RT, LN, XLN, EXT, apart(TR::MPL), PK>;
    static bool configured = false;
    if (!configured) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
        if (e != hipSuccess) return e;
        configured = true;
    }
    kern<<<dim3(8 * a.gpx * (a.nrb / a.span)), dim3(512), smem, stream>>>(a);
    return hipGetLastError();
}

// K blocks that a load brings, in the groups on several XCDs that have variants for it.  With eight sequences or fewer a load
// instruction's lanes for the sequences that are not there bring those of the next K blocks instead, two, four or eight of them, and the
// fragments are turned into place by rotating lanes (v_mov_dpp; no sum changes).  A wave then asks for its share of the state in one to
// six loads instead of five to sixteen, so that a request takes less of the address unit and a vain one is back sooner.  64 steps, us, one
// block a load -> this, one layer on an input as wide, batch 1 / 4 / 8:
//     768 units   89.1 / 90.6 / 92.5 -> 83.9 / 85.0 / 87.6        1024   103 / 105 / 106 -> 92.5 / 96.8 / 101
//     1280        101 / 103 / 103 -> 93.4 / 98.4 / 97.5           1536   109 / 111 / 111 -> 98.4 / 109 / 109
//     2048        135 / 140 -> 110 / 137; on 80 values 118 / 117 / 120 -> 98.7 / 97.9 / 104, 3 layers, batch 8 402 -> 372
// One launch is left out: from 8 steps on, a layer of 2048 units that reads rows as wide (not the chunks of a layer below), five to eight
// sequences, whose state in one request of eight loads instead of two takes longer: 64 steps, batch 5 and 8 135 -> 140 and 141, GRU 135 ->
// 140, 16 steps 46.9 -> 47.7 (6 steps 28.0 -> 28.1, 2 steps 19.6 -> 19.1; other widths of such rows gain, 1536 values 166 -> 164, 2000
// 163 -> 161).
// Groups on one XCD wait for the round trip and not for the loads: 512 units, batch 1 and 8 67.0 -> 68.4 and 68.2 -> 68.2, four layers
// 78 -> 81 and 80 -> 84.
int packed_blocks(const WavefrontXcdArgs& a, int LN) {
    if (LN > 12 && a.B > 4 && a.T >= 8 && !a.gx && !a.x_blocked && a.I == a.H) return 1;
    return a.B <= 2 ? 8 : a.B <= 4 ? 4 : a.B <= 8 ? 2 : 1;
}

template <class TR, int CELL, int RT, int LN, int XLN, bool EXT>
hipError_t launch_packed(const WavefrontXcdArgs& a, hipStream_t stream) {
#if RNN_XR_WIDE
    switch (packed_blocks(a, LN)) {
        case 8: return launch_variant<TR, CELL, RT, LN, XLN, EXT, 8>(a, stream);
        case 4: return launch_variant<TR, CELL, RT, LN, XLN, EXT, 4>(a, stream);
        case 2: return launch_variant<TR, CELL, RT, LN, XLN, EXT, 2>(a, stream);
        default: break;
    }
#endif
    return launch_variant<TR, CELL, RT, LN, XLN, EXT, 1>(a, stream);
}

template <class TR, int RT, int LN, int XLN>
hipError_t launch_cell(const WavefrontXcdArgs& a, hipStream_t stream) {
#if RNN_XR_KIND == 2
    return launch_packed<TR, CELL_GRU_RB, RT, LN, XLN, true>(a, stream);
#else
    if (a.cell == CELL_LSTM) return launch_packed<TR, CELL_LSTM, RT, LN, XLN, RNN_XR_KIND == 1>(a, stream);
    return launch_packed<TR, CELL_GRU, RT, LN, XLN, RNN_XR_KIND == 1>(a, stream);
#endif
}

// (RT, LN) that are compiled: a group of at most 32 workgroups, H = LN * 128 (bf16) or LN * 64 (fp32) units
#define RNN_XR_SHAPES_0(X) X(1, 1) X(2, 1) X(2, 2) X(4, 1) X(4, 2) X(4, 3) X(4, 4)
#define RNN_XR_SHAPES_1(X) X(1, 1) X(1, 2) X(2, 1) X(2, 2) X(2, 4) X(4, 1) X(4, 2) X(4, 4) X(4, 8)

// ... and, in bf16, of 40, 48 or 64 workgroups on two XCDs (1024 units are as many as the registers hold: 32 K blocks of four
// tiles are 128 registers of weights in a wave).  Translation units of their own (RNN_XR_WIDE = 1).  Layers of 1280, 1536 and 2048
// units in groups of 160, 192 and 256 workgroups of 8 units on all XCDs (RNN_XR_WIDE = 2).
#define RNN_XR_SHAPES_WIDE(X) X(4, 5) X(4, 6) X(4, 8)
#define RNN_XR_SHAPES_CHIP(X) X(2, 10) X(2, 12) X(2, 16)

#if RNN_XR_DT == 0
typedef XRBf16 TRHere;
#if RNN_XR_WIDE == 2
#define RNN_XR_SHAPES_HERE(X) RNN_XR_SHAPES_CHIP(X)
#elif RNN_XR_WIDE
#define RNN_XR_SHAPES_HERE(X) RNN_XR_SHAPES_WIDE(X)
#else
#define RNN_XR_SHAPES_HERE(X) RNN_XR_SHAPES_0(X)
#endif
#else
typedef XRF32 TRHere;
#define RNN_XR_SHAPES_HERE(X) RNN_XR_SHAPES_1(X)
#endif

template <int RT, int LN>
hipError_t launch_shape(const WavefrontXcdArgs& a, hipStream_t stream) {
    if constexpr (LN > 8) {
        if (a.xln == 2) return launch_cell<TRHere, RT, LN, 2>(a, stream);
        if (a.xln == 8) return launch_cell<TRHere, RT, LN, 8>(a, stream);
        if (a.xln == LN) return launch_cell<TRHere, RT, LN, LN>(a, stream);
        return hipErrorInvalidValue;
    } else
    switch (a.xln) {
        case 1: return launch_cell<TRHere, RT, LN, 1>(a, stream);
        case 2: return launch_cell<TRHere, RT, LN, 2>(a, stream);
        case 4: return launch_cell<TRHere, RT, LN, 4>(a, stream);
        case 8: return launch_cell<TRHere, RT, LN, 8>(a, stream);
        case 3: if constexpr (LN == 3) return launch_cell<TRHere, RT, LN, 3>(a, stream); else break;
        case 6: if constexpr (LN == 3 || LN == 5 || LN == 6) return launch_cell<TRHere, RT, LN, 6>(a, stream); else break;
        default: break;
    }
    return hipErrorInvalidValue;
}

hipError_t launch_here(const WavefrontXcdArgs& a, hipStream_t stream, int LN) {
#define X(rt, ln) if (a.RT == rt && LN == ln) return launch_shape<rt, ln>(a, stream);
    RNN_XR_SHAPES_HERE(X)
#undef X
    return hipErrorInvalidValue;
}

}  // namespace

#define RNN_XR_FN2(dt, kind, wide, apart) launch_wavefront_xcd_dt##dt##_kind##kind##_wide##wide##_apart##apart
#define RNN_XR_FN(dt, kind, wide, apart) RNN_XR_FN2(dt, kind, wide, apart)
hipError_t RNN_XR_FN(RNN_XR_DT, RNN_XR_KIND, RNN_XR_WIDE, RNN_XR_APART)(const WavefrontXcdArgs& a, hipStream_t stream, int LN) { return launch_here(a, stream, LN); }

#if RNN_XR_DT == 0 && RNN_XR_KIND == 0 && !RNN_XR_WIDE && !RNN_XR_APART
hipError_t launch_wavefront_xcd_dt0_kind1_wide0_apart0(const WavefrontXcdArgs& a, hipStream_t stream, int LN);
hipError_t launch_wavefront_xcd_dt0_kind2_wide0_apart0(const WavefrontXcdArgs& a, hipStream_t stream, int LN);
hipError_t launch_wavefront_xcd_dt1_kind0_wide0_apart0(const WavefrontXcdArgs& a, hipStream_t stream, int LN);
hipError_t launch_wavefront_xcd_dt1_kind1_wide0_apart0(const WavefrontXcdArgs& a, hipStream_t stream, int LN);
hipError_t launch_wavefront_xcd_dt1_kind2_wide0_apart0(const WavefrontXcdArgs& a, hipStream_t stream, int LN);
hipError_t launch_wavefront_xcd_dt0_kind0_wide1_apart0(const WavefrontXcdArgs& a, hipStream_t stream, int LN);
hipError_t launch_wavefront_xcd_dt0_kind1_wide1_apart0(const WavefrontXcdArgs& a, hipStream_t stream, int LN);
hipError_t launch_wavefront_xcd_dt0_kind0_wide2_apart0(const WavefrontXcdArgs& a, hipStream_t stream, int LN);
hipError_t launch_wavefront_xcd_dt0_kind1_wide2_apart0(const WavefrontXcdArgs& a, hipStream_t stream, int LN);
hipError_t launch_wavefront_xcd_dt0_kind0_wide0_apart1(const WavefrontXcdArgs& a, hipStream_t stream, int LN);
hipError_t launch_wavefront_xcd_dt0_kind1_wide0_apart1(const WavefrontXcdArgs& a, hipStream_t stream, int LN);

namespace {
int state_chunks(int dtype, int H) {             // LN, or 0 when H is no multiple of a wave's load
    const int unit = dtype == DT_BF16 ? 128 : 64;
    return H % unit == 0 ? H / unit : 0;
}
}  // namespace

bool wavefront_xcd_variant_exists(int dtype, int RT, int H) {
    const int LN = state_chunks(dtype, H);
#define X(rt, ln) if (RT == rt && LN == ln) return true;
    if (dtype == DT_BF16) { RNN_XR_SHAPES_0(X) }
    else { RNN_XR_SHAPES_1(X) }
#undef X
    return false;
}

bool wavefront_xcd_wide_exists(int dtype, int RT, int H, bool reset_before) {
    const int LN = state_chunks(dtype, H);
    if (dtype != DT_BF16 || reset_before) return false;
#define X(rt, ln) if (RT == rt && LN == ln) return true;
    RNN_XR_SHAPES_WIDE(X)
#undef X
    return false;
}

bool wavefront_xcd_chip_exists(int dtype, int RT, int H, bool reset_before) {
    const int LN = state_chunks(dtype, H);
    if (dtype != DT_BF16 || reset_before) return false;
#define X(rt, ln) if (RT == rt && LN == ln) return true;
    RNN_XR_SHAPES_CHIP(X)
#undef X
    return false;
}

int wavefront_xcd_input_chunks(int dtype, int H, int width, bool several_layers) {
    const int LN = state_chunks(dtype, H), epc = dtype == DT_BF16 ? 8 : 4;
    if (width % epc != 0) return 0;
    int need = ((width + 4 * epc - 1) / (4 * epc) + 3) / 4;
    if (LN > 8) return several_layers || need > LN ? 0 : need <= 2 ? 2 : need <= 8 ? 8 : LN;
    if (several_layers && need < LN) need = LN;
    static const int have[] = {1, 2, 3, 4, 6, 8};
    for (int v : have)
        if (v >= need && (LN == 3 || v != 3) && (LN == 3 || LN == 5 || LN == 6 || v != 6)) return v;
    return 0;
}

size_t wavefront_xcd_slot_bytes(int dtype, int stride, int H) {
    return (size_t)H * stride * (dtype == DT_BF16 ? 2 : 4);
}

hipError_t launch_wavefront_xcd(const WavefrontXcdArgs& a, hipStream_t stream) {
    const int LN = state_chunks(a.dtype, a.H);
    if (LN == 0 || a.LP < 1 || a.LP > WF_MAX_LAYERS || (a.D != 1 && a.D != 2) || (a.LP > 1 && a.D != 1)) return hipErrorInvalidValue;
    if ((a.span != 1 && a.span != 2 && a.span != 8) || a.nrb % a.span != 0) return hipErrorInvalidValue;
    if (a.nrb * a.RT * 4 != a.H || a.nrb > 32 * a.span || a.ncb != (a.B + 15) / 16 || a.gpx * (8 / a.span) < a.LP * a.D * a.ncb)
        return hipErrorInvalidValue;
    // with a projection the x waves of the first layer multiply nothing: they bring in the four values of their pair (one chunk)
    if ((a.gx == nullptr && a.xin == nullptr) || a.xln == 0 ||
        wavefront_xcd_input_chunks(a.dtype, a.H, a.gx ? 8 : a.I, a.LP > 1) != a.xln) return hipErrorInvalidValue;
    if (a.ring <= a.T && ((a.ring & (a.ring - 1)) != 0 || a.ring < 2 * XCD_AHEAD)) return hipErrorInvalidValue;
    if (a.stride < (a.B < 16 ? a.B : 16) || a.stride > 16) return hipErrorInvalidValue;
    if ((size_t)a.T * wavefront_xcd_slot_bytes(a.dtype, a.stride, a.H) >= ((size_t)1 << 31)) return hipErrorInvalidValue;
    const int kind = a.reset_before ? 2 : a.ext ? 1 : 0;
    if (a.reset_before && a.cell != CELL_GRU) return hipErrorInvalidValue;
    if (a.span == 2) {
        if (!wavefront_xcd_wide_exists(a.dtype, a.RT, a.H, a.reset_before != 0)) return hipErrorInvalidValue;
        return kind == 0 ? launch_wavefront_xcd_dt0_kind0_wide1_apart0(a, stream, LN) : launch_wavefront_xcd_dt0_kind1_wide1_apart0(a, stream, LN);
    }
    if (a.span == 8) {
        if (!wavefront_xcd_chip_exists(a.dtype, a.RT, a.H, a.reset_before != 0)) return hipErrorInvalidValue;
        return kind == 0 ? launch_wavefront_xcd_dt0_kind0_wide2_apart0(a, stream, LN) : launch_wavefront_xcd_dt0_kind1_wide2_apart0(a, stream, LN);
    }
    if (a.dtype == DT_BF16 && a.apart && kind < 2)
        return kind == 0 ? launch_wavefront_xcd_dt0_kind0_wide0_apart1(a, stream, LN) : launch_wavefront_xcd_dt0_kind1_wide0_apart1(a, stream, LN);
    if (a.dtype == DT_BF16)
        return kind == 0 ? launch_here(a, stream, LN) : kind == 1 ? launch_wavefront_xcd_dt0_kind1_wide0_apart0(a, stream, LN)
                                                                  : launch_wavefront_xcd_dt0_kind2_wide0_apart0(a, stream, LN);
    return kind == 0 ? launch_wavefront_xcd_dt1_kind0_wide0_apart0(a, stream, LN) : kind == 1 ? launch_wavefront_xcd_dt1_kind1_wide0_apart0(a, stream, LN)
                                                                                       : launch_wavefront_xcd_dt1_kind2_wide0_apart0(a, stream, LN);
}
#endif  // RNN_XR_DT == 0 && RNN_XR_KIND == 0 && !RNN_XR_WIDE && !RNN_XR_APART

}  // namespace rnn
