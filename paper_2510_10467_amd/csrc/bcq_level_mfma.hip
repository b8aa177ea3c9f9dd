// Large batches, the level form of the dequantising kernel: W_p is rebuilt by LOOKING UP its values instead of summing
// them.  Inside a scale group a row has only 2^p different weights, the levels z + sum_i (+-alpha_i); a lane forms those of
// its row once per group (the same fp32 sums in the same order, rounded once to binary16, that the other form makes for
// every weight) and keeps them in four registers, the low bytes and the high bytes of eight levels.  The p plane
// words of 32 columns become 32 codes of p bits in two byte transposes, and a V_PERM_B32 with four codes as its selector
// delivers one byte of four weights.  At p = 3 that is 65 vector instructions per 32 columns (bit transpose 13, byte transpose 8,
// selectors 12, look-ups 32); with the forming of the levels and the addresses the counters say 2.5 / 2.8 / 3.5 per weight
// at p = 2 / 3 / 4, where the sums take 6.8 at p = 4, and an LDS read per weight besides the operands.
//   p <= 3            2^p <= 8 levels, one pair of registers per byte
//   p = 4             the levels come in pairs +-l: eight of them are kept, the codes of planes 0..2 are complemented where
//                     plane 3 is -1 and the sign goes onto the high byte
//   p = 4, offsets    sixteen levels, two look-ups per byte and a select
//
// The product runs on v_mfma_f32_32x32x16_f16: a wave owns one tile of 32 rows and QT tiles of 32 requests.  Against 16 x 16
// tiles an instruction needs half as many operand reads from LDS per operation, and it leaves the SIMD's issue slots free for
// half of its 32 cycles, which is where the look-ups go.  The two lane halves hold the two 128-column groups of a pair
// of groups (a permutation of K which the activations follow), so that a lane sees one group and one set of levels:
//   step of 16 columns = columns c .. c+7 of group 2G (lanes 0-31) and of group 2G+1 (lanes 32-63).
// A stage is 64 columns (word w of both groups).  Its activations are staged in LDS, by loads that write LDS directly, three
// stages ahead in a ring of four tiles; at the barrier that ends a stage the tile AFTER the next one has landed (what this
// stage asked for stays under way: the wait is for all but the last XU loads), so the operands of the next stage's first
// step are read before the barrier and nothing waits behind it.  The eight 16-byte parts of a request sit XOR-permuted by the
// request number, so that the operand reads of sixteen requests use all banks.  The weights of a step are made during
// the step before it, a few look-ups after each matrix instruction (left to itself the compiler reads two operands, waits
// for them and issues two matrix instructions).
//
// A workgroup is TEAMS teams of WR x WQ waves; the teams take alternate pairs of groups with tiles of their own and meet at
// the end (short matrices: rows alone do not fill the chip).
//
// Per-request precision (level_byclass_kernel): the same body per precision in one launch, each workgroup on the requests of its precision; a
// weight is rebuilt once per precision and tile of requests by look-ups of that precision instead of by sums: 8192 x 8192 with 200
// requests at precisions from {2, 3, 4} 119 -> 63 us (on 128 x 96: a third of 200 requests fills two tiles of 64 badly, one of 128 half).
//
// What bounds it: on a full chip the matrix instructions with the look-ups between them (matrix pipe busy for 66 / 63 / 57 % of the
// cycles at p = 2 / 3 / 4) and the clock, which random operands hold at 1.7 to 1.8 GHz (with activations of zero the same cycles
// pass at 2.2 to 2.3); the library's plain fp16 product of 8192^3 reaches 1210 TFLOP/s (1750 with zeros).  Smaller tiles were bound
// by neither: leaving out the look-ups, three quarters of the matrix instructions or the operand reads changed nothing, while leaving out the
// fetch of words and scales took a quarter off (4096 x 14336 with 500 requests at p = 4 on tiles of 128 x 256: 240 -> 164 us), because
// every row, plane and pair of groups asked for a line of its own, twice (see fetch_block and load_window).  That halved (196 us there):
// 28672 x 8192 with 2048 requests at p = 3 937 -> 887 us = 1085 TFLOP/s, the linear layers of a Llama-3-8B block with 500 requests
// at p = 4 326 -> 301, 8192 x 8192 in groups of 64 with 96 requests 37.4 -> 34.4.  What the fetch still costs there is 30 us,
// the barriers about 10.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "bcq_internal.hpp"

namespace bcq {
namespace {

typedef _Float16 v8h __attribute__((ext_vector_type(8)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int kMaxP = 4;
constexpr int kRowBytes = 128;              // LDS row of one request: the 64 columns of a stage
constexpr int kRing = 4;                    // stages in LDS
// vector instructions placed between two matrix instructions
template <int QT> constexpr int kBetween = QT >= 8 ? 4 : QT >= 4 ? 6 : 12;

struct LevelParams {
    const unsigned char *planes, *scales, *offsets, *x;
    _Float16 *y;
    uint32_t plane_stride, row_stride;      // bytes between planes (m n / 8) and plane rows (n / 8)
    uint32_t scale_plane_stride, scale_row_stride;      // bytes between scale planes (m n / group * 2) and rows
    uint32_t x_stride;                      // bytes between requests: n * 2
    uint32_t m;
    int batch, npairs;                      // npairs: pairs of 128-column groups
    int gshift;                             // scale groups of 64 (-1), 128 (0) or 256 (+1) columns
    // per-request precision: a scale / offset set per precision, nullptr where there is none
    const unsigned char *scale_sets[kMaxP + 1], *offset_sets[kMaxP + 1];
    const int32_t *p_req;
    int p_max;
    uint32_t class_order;                   // byte y: the precision served by the workgroups with blockIdx.y = y
    // several matrices in one launch (nmat > 1): matrix k owns the workgroup rows mat_blk0[k] .. mat_blk0[k+1]-1
    int nmat;
    const unsigned char *mat_planes[BCQ_MAX_MULTI];
    const unsigned char *mat_scales[BCQ_MAX_MULTI];
    _Float16 *mat_y[BCQ_MAX_MULTI];
    uint32_t mat_m[BCQ_MAX_MULTI];
    uint32_t mat_blk0[BCQ_MAX_MULTI];
};

// a where the mask bit is set, b elsewhere
__device__ __forceinline__ uint32_t pick_bits(uint32_t mask, uint32_t a, uint32_t b) { return (a & mask) | (b & ~mask); }

// The levels of one row and group, low and high bytes apart: byte c of lo[0] is the low byte of level c, of lo[1] of level 4 + c.
template <int P, bool OFFSET>
struct Levels {
    static constexpr bool kSigned = P == 4 && !OFFSET;      // eight of the sixteen, those with plane 3 at +1
    static constexpr int NQ = P <= 2 ? 1 : P == 3 || kSigned ? 2 : 4;       // quadruples of levels
    uint32_t lo[NQ], hi[NQ];

    // alpha[i], z: binary16 bits
    __device__ __forceinline__ void form(const uint32_t (&alpha)[P], uint32_t z)
    {
        constexpr int NL = 4 * NQ;
        float a[P];
#pragma unroll
        for (int i = 0; i < P; ++i) a[i] = (float)__builtin_bit_cast(_Float16, (unsigned short)alpha[i]);
        float v[NL];
        v[0] = OFFSET ? (float)__builtin_bit_cast(_Float16, (unsigned short)z) : 0.f;
        // level of code c: bit i set means +alpha_i; plane 0 first, as the planes are summed
        int have = 1;
#pragma unroll
        for (int i = 0; i < P; ++i) {
            if (kSigned && i == 3) {
#pragma unroll
                for (int c = 0; c < 8; ++c) v[c] = v[c] + a[3];
            } else {
#pragma unroll
                for (int c = 0; c < NL / 2; ++c)
                    if (c < have) {
                        v[(have + c) % NL] = v[c] + a[i];
                        v[c] = v[c] - a[i];
                    }
                have *= 2;
            }
        }
#pragma unroll
        for (int k = 0; k < NQ; ++k) {
            uint32_t h[4];
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const float f = 4 * k + c < (kSigned ? 8 : 1 << P) ? v[4 * k + c] : 0.f;
                h[c] = __builtin_bit_cast(unsigned short, (_Float16)f);      // the single rounding of W_p to binary16
            }
            const uint32_t h01 = h[0] | (h[1] << 16), h23 = h[2] | (h[3] << 16);
            lo[k] = __builtin_amdgcn_perm(h23, h01, 0x06040200u);
            hi[k] = __builtin_amdgcn_perm(h23, h01, 0x07050301u);
        }
    }

    // bytes of the codes of four columns (one code per byte; bits above the code are garbage) -> two dwords of two weights
    __device__ __forceinline__ void weights(uint32_t codes, uint32_t sign, uint32_t &d0, uint32_t &d1) const
    {
        constexpr uint32_t mask = P == 1 ? 0x01010101u : P == 2 ? 0x03030303u : 0x07070707u;
        const uint32_t sel = codes & mask;
        uint32_t l, h;
        if constexpr (NQ == 1) {
            l = __builtin_amdgcn_perm(0u, lo[0], sel);
            h = __builtin_amdgcn_perm(0u, hi[0], sel);
        } else {
            l = __builtin_amdgcn_perm(lo[1], lo[0], sel);
            h = __builtin_amdgcn_perm(hi[1], hi[0], sel);
        }
        if constexpr (NQ == 4) {
            const uint32_t one = (codes >> 3) & 0x01010101u, upper = (one << 8) - one;        // 0xff in the bytes of codes 8..15
            l = pick_bits(upper, __builtin_amdgcn_perm(lo[3], lo[2], sel), l);
            h = pick_bits(upper, __builtin_amdgcn_perm(hi[3], hi[2], sel), h);
        }
        if constexpr (kSigned) h ^= sign & 0x80808080u;
        d0 = __builtin_amdgcn_perm(h, l, 0x05010400u);
        d1 = __builtin_amdgcn_perm(h, l, 0x07030602u);
    }
};

// 32 columns of P planes -> codes: byte c of out[t] holds the code of column 8t + c in its low nibble and that of column
// 8t + 4 + c in its high nibble (bit i: plane i; bits of planes that are not there are garbage)
template <int P, bool SIGNED>
__device__ __forceinline__ void transpose_codes(const uint32_t (&w)[P], uint32_t (&out)[4])
{
    uint32_t t[4];
    if constexpr (P == 1) {
#pragma unroll
        for (int c = 0; c < 4; ++c) t[c] = w[0] >> c;
    } else {
        uint32_t w0 = w[0], w1 = w[1];
        if constexpr (SIGNED) {
            w0 = ~(w0 ^ w[3]);
            w1 = ~(w1 ^ w[3]);
        }
        const uint32_t a01 = pick_bits(0x55555555u, w0, w1 << 1), b01 = pick_bits(0x55555555u, w0 >> 1, w1);
        if constexpr (P == 2) {
            t[0] = a01;
            t[1] = b01;
            t[2] = a01 >> 2;
            t[3] = b01 >> 2;
        } else {
            uint32_t a23, b23;
            if constexpr (P == 3) {
                a23 = w[2];
                b23 = w[2] >> 1;
            } else {
                const uint32_t w2 = SIGNED ? ~(w[2] ^ w[3]) : w[2], w3 = SIGNED ? ~w[3] : w[3];
                a23 = pick_bits(0x55555555u, w2, w3 << 1);
                b23 = pick_bits(0x55555555u, w2 >> 1, w3);
            }
            t[0] = pick_bits(0x33333333u, a01, a23 << 2);
            t[2] = pick_bits(0x33333333u, a01 >> 2, a23);
            t[1] = pick_bits(0x33333333u, b01, b23 << 2);
            t[3] = pick_bits(0x33333333u, b01 >> 2, b23);
        }
    }
    const uint32_t p01 = __builtin_amdgcn_perm(t[1], t[0], 0x05010400u), q01 = __builtin_amdgcn_perm(t[1], t[0], 0x07030602u);
    const uint32_t p23 = __builtin_amdgcn_perm(t[3], t[2], 0x05010400u), q23 = __builtin_amdgcn_perm(t[3], t[2], 0x07030602u);
    out[0] = __builtin_amdgcn_perm(p23, p01, 0x05040100u);
    out[1] = __builtin_amdgcn_perm(p23, p01, 0x07060302u);
    out[2] = __builtin_amdgcn_perm(q23, q01, 0x05040100u);
    out[3] = __builtin_amdgcn_perm(q23, q01, 0x07060302u);
}

// QT tiles of 32 requests per wave (and one of 32 rows), WR x WQ waves per team.  BLOCKS_FROM: from so many planes on plane words come for two
// pairs of groups at a time (see fetch_block), kNever: for one.
constexpr int kNever = kMaxP + 1;
template <int QT_, int WR_, int WQ_, int TEAMS_, int BLOCKS_FROM_>
struct Shape {
    static constexpr int QT = QT_, WR = WR_, WQ = WQ_, TEAMS = TEAMS_, BLOCKS_FROM = BLOCKS_FROM_;
    static constexpr int ROWS = 32 * WR, REQS = 32 * QT * WQ;
    static constexpr int SW = WR * WQ;                              // waves of a team
    static constexpr int THREADS = 64 * SW * TEAMS;
    static constexpr int TILE = REQS * kRowBytes;                   // one stage's activations
    static constexpr int XU = TILE / 1024 / SW;                     // loads of 1 KiB per wave and stage
    static constexpr int TILES = TEAMS * kRing * TILE;
    static_assert(XU * 1024 * SW == TILE && XU >= 1, "tile does not split over the team");
    static_assert((TEAMS - 1) * SW * QT * 4096 <= TILES, "accumulator exchange must fit in the tiles");
};

// LDS of a kernel: the tiles, then what it takes for plane words to change lanes, then the scales of a window of columns.
template <int P, typename S, bool OFFSET>
struct Lds {
    static constexpr bool COALESCE = P >= S::BLOCKS_FROM && !(OFFSET && P == 4);        // (there it would leave no room for the scales)
    static constexpr int WAVES = S::TEAMS * S::SW;
    static constexpr int HANDOVER = COALESCE ? 2048 : 0;            // per wave
    static constexpr int SCALES_AT = S::TILES + WAVES * HANDOVER;
    // two workgroups share a CU
    static constexpr bool PAIRED = S::QT == 2 && S::WR == 4;
    static constexpr int limit = PAIRED ? 80 * 1024 : 160 * 1024;
    // Offsets are kept like another plane's scales, except where a fifth plane would leave room for one workgroup on a CU instead of two: there
    // every lane reads its own from memory (128 x 64, p = 4, groups of 128, 400 workgroups: 1024 columns 24.9 -> 20.8 us, 4096 72.1 -> 64.5).
    static constexpr bool Z_DIRECT = OFFSET && PAIRED && SCALES_AT + S::ROWS * (P + 1) * 16 * S::TEAMS > limit;
    static constexpr int PLANES = P + (OFFSET && !Z_DIRECT ? 1 : 0);
    // bytes of a row's scales of one plane in LDS; at least those of two rounds in groups of 64
    static constexpr int WINDOW = SCALES_AT + S::ROWS * PLANES * 64 <= limit ? 64 : SCALES_AT + S::ROWS * PLANES * 32 <= limit || S::TEAMS > 1 ? 32 : 16;
    static constexpr int BYTES = SCALES_AT + S::ROWS * PLANES * WINDOW;
    static_assert(BYTES <= limit, "must fit in LDS, twice where two workgroups share it");
    static_assert(WINDOW >= 16 * S::TEAMS, "a window holds the scales of two rounds in groups of 64");
};

// A window of scales in LDS: every row has 2^row_log2 bytes in a plane's part of it, the scales of `pairs` pairs of groups (a power of two).
struct ScaleWindow {
    int row_log2, pairs;
};

// window: Lds::WINDOW.  Rows start at multiples of two bytes (groups of 256 columns) or four; loads of four bytes fetch them from the multiple of four
// below, and a window is half of what it could be where that would cut something off: where rows or planes of scales start at odd multiples of two
// and a row does not fit as a whole (half everywhere in groups of 256: 64 x 128, 6912 columns, p = 3 41.3 us, so 40.8).  On narrow matrices a row's place holds
// just the row, so that a load brings more of them: a workgroup starts with these loads (200 workgroups of 64 x 128, 256 columns, p = 4 with
// offsets: 80 loads 9.4 us, 5 loads 8.4).
__host__ __device__ inline ScaleWindow scale_window(int window, uint32_t scale_row_stride, int gshift, int npairs)
{
    const uint32_t row_bytes = scale_row_stride + (gshift > 0 && (npairs & 1) ? 2u : 0u);       // and what lies before an odd start
    const int row_log2 = 32 - __builtin_clz((row_bytes < (uint32_t)window ? row_bytes : (uint32_t)window) - 1);
    const bool cut = gshift > 0 && (npairs & 1) && row_bytes > (uint32_t)window;
    return {row_log2, window / (gshift < 0 ? 8 : gshift == 0 || cut ? 4 : 2)};
}

// the workgroup's rows (block rowblk of the matrix) and requests b0 .. b0 + nreq - 1
// BYCLASS (per-request precision): the requests of precision P of rank b0 .. b0 + S::REQS - 1 among them instead; every wave ranks the batch
// itself, the numbers pass through LDS before the tiles need it and wait in registers until the results are stored.
template <int P, typename S, bool OFFSET, bool BYCLASS = false>
__device__ __forceinline__ void level_body(const LevelParams &a, const int b0, int nreq, const uint32_t rowblk)
{
    constexpr int QT = S::QT, TEAMS = S::TEAMS, XU = S::XU, SW = S::SW;
    constexpr int UT = QT < 4 ? QT : 4;       // request tiles whose operands are held at a time
    constexpr int NC = QT / UT;
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    using L = Levels<P, OFFSET>;

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int team = wave / SW, tw = wave % SW, wr = tw % S::WR, wq = tw / S::WR;
    const int r32 = lane & 31, half = lane >> 5;
    unsigned char *xt = lds + team * kRing * S::TILE;
    const uint32_t row0 = rowblk * S::ROWS + wr * 32;

    uint32_t *const req_of = reinterpret_cast<uint32_t *>(lds);
    constexpr int NL = (S::REQS + 63) / 64;
    uint32_t listed[NL];
    if constexpr (BYCLASS) {
        nreq = rank_requests<S::REQS>(a.p_req, a.batch, a.p_max, P, b0, req_of);
        if (nreq <= 0) return;                // (every wave of the workgroup: none has reached a barrier yet)
        __syncthreads();
#pragma unroll
        for (int k = 0; k < NL; ++k) listed[k] = req_of[min(64 * k + lane, nreq - 1)];
    }

    // rows and requests past the end repeat the last one (their results are not stored)
    const uint32_t my_row = min(row0 + r32, a.m - 1);
    uint32_t w_off = my_row * a.row_stride + half * 16;
    const uint32_t s_pair = a.gshift > 0 ? 2u : a.gshift < 0 ? 8u : 4u;      // bytes of a row's scales per pair of groups
    // Load i of a stage brings the 1 KiB of requests 8i .. 8i+7; lane l delivers part (l & 7) ^ (request / 2 & 7) of request
    // 8i + (l >> 3).  Parts 0-3 are columns 32w .. of the pair's first group, 4-7 of its second.
    uint32_t xs_src[XU];
#pragma unroll
    for (int k = 0; k < XU; ++k) {
        const int req = 8 * (k * SW + tw) + (lane >> 3);
        const int part = (lane & 7) ^ ((req >> 1) & 7);
        const uint32_t source = BYCLASS ? req_of[min(req, nreq - 1)] : (uint32_t)(b0 + min(req, nreq - 1));
        xs_src[k] = source * a.x_stride + (part >> 2) * 256 + (part & 3) * 16;
    }
    if constexpr (BYCLASS) __syncthreads();   // the list has been read: its place belongs to the tiles
    // (buffer loads: the compiler counts loads of the global kind that write LDS among the LDS reads under way as well, and
    // then waits for all of those reads wherever it needs one)
    const auto x_rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<unsigned char *>(a.x), 0, (int)((uint32_t)a.batch * a.x_stride), 0x00020000);
    auto stage_unit = [&](int pair, int w, int k) {
        __builtin_amdgcn_raw_ptr_buffer_load_lds(x_rsrc, (__attribute__((address_space(3))) void *)(xt + w * S::TILE + (k * SW + tw) * 1024), 16,
                                                 (int)xs_src[k], pair * 512 + w * 64, 0, 0);
    };
    // What a fetch of plane words or scales costs is not its bytes but the lines it asks for, one per row: 16 bytes of the words and
    // two of the scales of every row and plane, one pair of groups at a time, made 64 requests per load and moved a whole line
    // into the CU for each, as much again as the activations.  So
    //   scales       come for a window of columns at a time, straight into LDS, shared by the waves of the rows (128 x 256, 4096 x
    //                14336 with 500 requests: 240 us with, 192 without the fetch of every pair's scales)
    //   plane words  come for two pairs at a time, four neighbouring lanes on 64 bytes of a row (lane l: rows l / 4 and 16 + l / 4,
    //                part l % 4), which the memory pipe takes as one request, and change lanes in LDS (COALESCE: another 10 %, of
    //                which the LDS takes 4 back), where it pays (see visit_shape)
    using M = Lds<P, S, OFFSET>;
    constexpr bool COALESCE = M::COALESCE;
    constexpr int WINDOW = M::WINDOW;
    u32x4 word[P], later_word[P], word_n[P][COALESCE ? 2 : 1];
    uint32_t sc[P], zc = 0;                 // scales and offset of the next pair: low half first, high half columns 64 .. (groups of 64)
#pragma unroll
    for (int i = 0; i < P; ++i) sc[i] = 0;
    uint32_t z_word = 0;
    const uint32_t z_off = my_row * a.scale_row_stride + (a.gshift > 0 ? 0u : a.gshift < 0 ? half * 4u : half * 2u);
    uint32_t wq_off[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) wq_off[j] = min(row0 + 16 * j + (lane >> 2), a.m - 1) * a.row_stride;
    unsigned char *handover = lds + S::TILES + wave * M::HANDOVER;
    // row r, part c at 64 r + 16 (c ^ (r / 4 & 3)): the 16 rows that a read takes at a time use all banks
    unsigned char *put_at = handover + (lane >> 2) * 64 + (((lane & 3) ^ ((lane >> 4) & 3)) * 16);
    const unsigned char *get_at = handover + r32 * 64;
    const int get_swz = (r32 >> 2) & 3;

    const int rounds = (a.npairs + TEAMS - 1) / TEAMS;
    const int last = a.npairs - 1;
    // The teams take pairs in turn, or blocks of two neighbouring ones, of which what is left after whole rounds of blocks goes out as single pairs
    // if there are no more of them than teams: with COALESCE, and with per-request precision on two teams, where few workgroups are under way
    // at a time and a team finds the line of its second pair in the caches (128 x 64, 40 calls: 1.4 % on average, 4608 x 10752 with 67
    // requests 84.9 -> 81.9 us).
    constexpr bool IN_BLOCKS = COALESCE || (BYCLASS && TEAMS == 2);
    auto pair_of = [&](int it) {
        return IN_BLOCKS ? (it >> 1) * (2 * TEAMS) + (it & 1) + (it == rounds - 1 && !(it & 1) ? team : 2 * team) : it * TEAMS + team;
    };

    const auto s_rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<unsigned char *>(a.scales), 0, (int)(((uint32_t)P * a.scale_plane_stride + 3) & ~3u), 0x00020000);
    const auto z_rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<unsigned char *>(OFFSET ? a.offsets : a.scales), 0, (int)((a.scale_plane_stride + 3) & ~3u), 0x00020000);
    auto fetch_direct = [&](int pair) {     // 16 bytes of the lane's own row
        asm volatile("" : "+v"(w_off));     // lane offsets stay 32 bits wide, in the load's own addressing mode
#pragma unroll
        for (int i = 0; i < P; ++i)
            word_n[i][0] = *reinterpret_cast<const u32x4 *>(a.planes + (size_t)i * a.plane_stride + (uint32_t)pair * 32 + w_off);
        // and the dword of the pair's offset
        if constexpr (M::Z_DIRECT) z_word = __builtin_amdgcn_raw_buffer_load_b32(z_rsrc, (int)((z_off + (uint32_t)pair * s_pair) & ~3u), 0, 0);
    };
    auto fetch_block = [&](int pair) {      // the pair and its neighbour
        // (past the end of a row: its last part, for a pair that is not there)
        const uint32_t col = min((uint32_t)pair * 32 + (lane & 3) * 16, a.row_stride - 16);
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            uint32_t off = wq_off[j] + col;
            asm volatile("" : "+v"(off));
#pragma unroll
            for (int i = 0; i < P; ++i) word_n[i][COALESCE ? j : 0] = *reinterpret_cast<const u32x4 *>(a.planes + (size_t)i * a.plane_stride + off);
        }
    };
    // Window w of the scales of all the workgroup's rows, four bytes per lane.  (Past the end of a row the next one follows; past the end of the set
    // at most the two bytes that fill its last dword are read.  None of it is used.)
    unsigned char *const scales_lds = lds + M::SCALES_AT;
    const uint32_t wg_row0 = rowblk * S::ROWS;
    const ScaleWindow sw = scale_window(WINDOW, a.scale_row_stride, a.gshift, a.npairs);
    const int wpairs = sw.pairs;
    auto load_window = [&](int w) {
        constexpr int kRowsLog2 = __builtin_ctz(S::ROWS);
        static_assert(S::ROWS == 1 << kRowsLog2 && S::ROWS >= 64, "a load covers rows of one plane");
        const int per_row = sw.row_log2 - 2, per_plane = kRowsLog2 + sw.row_log2 - 8;       // lanes of a row, loads of a plane: their logarithms
        const uint32_t col = (uint32_t)(w * wpairs) * s_pair;
#pragma unroll 1
        for (int j = wave; j < M::PLANES << per_plane; j += M::WAVES) {
            const int plane = j >> per_plane, part = j & ((1 << per_plane) - 1);
            const uint32_t row = (part << (6 - per_row)) + (lane >> per_row);
            const bool z = OFFSET && !M::Z_DIRECT && plane == P;
            const uint32_t at = min(wg_row0 + row, a.m - 1) * a.scale_row_stride + col + (z ? 0u : (uint32_t)plane * a.scale_plane_stride);
            __builtin_amdgcn_raw_ptr_buffer_load_lds(z ? z_rsrc : s_rsrc,
                                                     (__attribute__((address_space(3))) void *)(scales_lds + plane * (S::ROWS * WINDOW) + part * 256), 4,
                                                     (int)((at & ~3u) + (lane & ((1 << per_row) - 1)) * 4), 0, 0, 0);
        }
    };
    const unsigned char *sc_lane = scales_lds + ((row0 - wg_row0 + r32) << sw.row_log2) + (a.gshift > 0 ? 0 : a.gshift < 0 ? half * 4 : half * 2);
    const uint32_t sc_row = my_row * a.scale_row_stride;
    auto read_scales = [&](int pair) {      // of a pair in the window that is there
        const unsigned char *at = sc_lane + (pair & (wpairs - 1)) * (int)s_pair;
#pragma unroll
        for (int i = 0; i < M::PLANES; ++i) {
            const unsigned char *from = at + i * (S::ROWS * WINDOW);
            uint32_t v;
            if (a.gshift < 0) v = *reinterpret_cast<const uint32_t *>(from);
            else if (a.gshift == 0) v = *reinterpret_cast<const unsigned short *>(from);
            else v = *reinterpret_cast<const unsigned short *>(from + ((sc_row + (i < P ? (uint32_t)i * a.scale_plane_stride : 0u)) & 2));
            if (i < P) sc[i < P ? i : 0] = v;
            else zc = v;
        }
        if constexpr (M::Z_DIRECT) {
            const uint32_t at = z_off + (uint32_t)pair * s_pair;
            zc = a.gshift < 0 ? z_word : (z_word >> (8 * (at & 2))) & 0xffffu;
        }
    };

    // operand reads: request 32 (wq QT + q) + r32, part 4 half + s
    const unsigned char *xa_lane = xt + (wq * QT * 32 + r32) * kRowBytes;
    const uint32_t xa_off = (uint32_t)(((4 * half) ^ ((r32 >> 1) & 7)) * 16);
    auto operand = [&](int t, int u) {          // step t of a pair
        return *reinterpret_cast<const v8h *>(xa_lane + (t >> 2) * S::TILE + u * (32 * kRowBytes) + (xa_off ^ (uint32_t)(16 * (t & 3))));
    };

    v16f acc[QT];
#pragma unroll
    for (int q = 0; q < QT; ++q)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[q][e] = 0.f;

    L lev;
    uint32_t codes[4], later[P], later_z = 0;
    auto begin_pair = [&]() {                   // the scales of the current pair become levels
        uint32_t first[P];
#pragma unroll
        for (int i = 0; i < P; ++i) {
            first[i] = sc[i] & 0xffffu;
            later[i] = sc[i] >> 16;
        }
        later_z = zc >> 16;
        lev.form(first, zc & 0xffffu);
    };
    auto begin_block = [&]() {                  // the words that came for the next two pairs (COALESCE: through LDS to the lanes that use them)
#pragma unroll
        for (int i = 0; i < P; ++i) {
            if constexpr (COALESCE) {
                *reinterpret_cast<u32x4 *>(put_at) = word_n[i][0];
                *reinterpret_cast<u32x4 *>(put_at + 1024) = word_n[i][COALESCE ? 1 : 0];
                word[i] = *reinterpret_cast<const u32x4 *>(get_at + ((half ^ get_swz) * 16));
                later_word[i] = *reinterpret_cast<const u32x4 *>(get_at + (((2 + half) ^ get_swz) * 16));
            } else {
                word[i] = word_n[i][0];
            }
        }
        begin_pair();
    };
    auto second_pair = [&]() {
#pragma unroll
        for (int i = 0; i < P; ++i) word[i] = COALESCE ? later_word[i] : word_n[i][0];
        begin_pair();
    };
    auto make = [&](int t) {                    // weights of step t of a pair
        if (t == 8 && a.gshift < 0) lev.form(later, later_z);       // groups of 64: columns 64 .. of both groups
        if ((t & 3) == 0) {
            uint32_t w[P];
#pragma unroll
            for (int i = 0; i < P; ++i) w[i] = word[i][t >> 2];
            transpose_codes<P, L::kSigned>(w, codes);
        }
        const uint32_t c = codes[t & 3];
        uint32_t d0, d1, d2, d3;
        lev.weights(c, c << 4, d0, d1);
        lev.weights(c >> 4, c, d2, d3);
        return __builtin_bit_cast(v8h, u32x4{d0, d1, d2, d3});
    };

    if (pair_of(0) <= last) {
        if constexpr (COALESCE) fetch_block(pair_of(0));
        else fetch_direct(pair_of(0));
#pragma unroll
        for (int w = 0; w < kRing - 1; ++w)
#pragma unroll
            for (int k = 0; k < XU; ++k) stage_unit(pair_of(0), w, k);
    }
    load_window(0);
    asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier" ::: "memory");
    v8h wb, xa[UT];
    if (pair_of(0) <= last) {
        read_scales(pair_of(0));
        begin_block();
        wb = make(0);
#pragma unroll
        for (int u = 0; u < UT; ++u) xa[u] = operand(0, u);
    }
    // One pair of groups.  SECOND: of its block.
    auto run_pair = [&](auto second, int it) {
        constexpr bool SECOND = decltype(second)::value;
        const int pair = pair_of(it);
        if (pair > last) {                      // a team without a pair of its own in the last round meets the barriers
            asm volatile("s_barrier\n\ts_barrier\n\ts_barrier\n\ts_barrier" ::: "memory");
            return;
        }
        const int npair = min(pair_of(it + 1), last);               // (past the end: something that is there, for nothing)
        constexpr int FETCHED = COALESCE ? (SECOND ? 0 : 2 * P) : P + (M::Z_DIRECT ? 1 : 0);        // loads of the words that come next
        // the next pair opens a window: nobody needs the old one any more
        const int nstart = ((it + 1) >> 1) * (2 * TEAMS);
        if (SECOND && (nstart & (wpairs - 1)) == 0 && nstart <= last) load_window(nstart / wpairs);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int t = 0; t < 16; ++t) {
            v8h wn, xn[UT];
#pragma unroll
            for (int k = 0; k < XU; ++k)
                if (k * 4 / XU == (t & 3)) stage_unit(t < 4 ? pair : npair, ((t >> 2) + kRing - 1) & (kRing - 1), k);
            if (t == 13) read_scales(npair);
            if (t == 15) {
                if constexpr (SECOND) begin_block();
                else second_pair();
            }
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                const int tn = c + 1 < NC ? t : (t + 1) & 15, cn = c + 1 < NC ? c + 1 : 0;
#pragma unroll
                for (int u = 0; u < UT; ++u) xn[u] = operand(tn, UT * cn + u);
                if (c == 0) wn = make((t + 1) & 15);
#pragma unroll
                for (int u = 0; u < UT; ++u)
                    acc[UT * c + u] = __builtin_amdgcn_mfma_f32_32x32x16_f16(xa[u], wb, acc[UT * c + u], 0, 0, 0);
#pragma unroll
                for (int u = 0; u < UT; ++u) xa[u] = xn[u];
            }
            wb = wn;
            // the order of a step: the next operands first, then matrix instructions with look-ups between them
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                __builtin_amdgcn_sched_group_barrier(0x100, UT, 0);
#pragma unroll
                for (int u = 0; u < UT; ++u) {
                    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                    __builtin_amdgcn_sched_group_barrier(0x002, kBetween<QT>, 0);
                }
            }
            __builtin_amdgcn_sched_barrier(0);
            if (t == 3) {
                // behind this stage's loads, so that two barriers can leave them under way
                if constexpr (!COALESCE) fetch_direct(npair);
                else if constexpr (!SECOND) fetch_block(min(pair_of(it + 2), last));
                __builtin_amdgcn_sched_barrier(0);
            }
            // what the step before the last barrier asked for has landed; what this stage asked for is still under way
            if ((t & 3) == 3) {
                if (t <= 7) asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(XU + FETCHED) : "memory");
                else asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(XU) : "memory");
            }
        }
    };
    for (int it = 0; it < rounds; it += 2) {
        run_pair(std::false_type{}, it);
        if (it + 1 < rounds) run_pair(std::true_type{}, it + 1);
    }

    if constexpr (TEAMS > 1) {
        // the other teams hand their accumulators over through the tiles, once no load into them is under way
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        v4f *xchg = reinterpret_cast<v4f *>(lds);
        constexpr int NV = QT * 4;            // 16-byte vectors per lane
        if (team > 0) {
#pragma unroll
            for (int q = 0; q < QT; ++q)
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    xchg[(((team - 1) * SW + tw) * NV + q * 4 + e) * 64 + lane] =
                        v4f{acc[q][4 * e], acc[q][4 * e + 1], acc[q][4 * e + 2], acc[q][4 * e + 3]};
        }
        __syncthreads();
        if (team > 0) return;
#pragma unroll
        for (int k = 1; k < TEAMS; ++k)
#pragma unroll
            for (int q = 0; q < QT; ++q)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const v4f v = xchg[(((k - 1) * SW + tw) * NV + q * 4 + e) * 64 + lane];
#pragma unroll
                    for (int i = 0; i < 4; ++i) acc[q][4 * e + i] += v[i];
                }
    }

    // the list back into LDS, a copy per wave, where the scales were (the last barrier is behind all their readers)
    uint32_t *const out_req = reinterpret_cast<uint32_t *>(scales_lds) + wave * (64 * NL);
    if constexpr (BYCLASS) {
        static_assert(M::WAVES * 256 * NL <= S::ROWS * M::PLANES * WINDOW, "the list must fit");
#pragma unroll
        for (int k = 0; k < NL; ++k) out_req[64 * k + lane] = listed[k];
    }
    // element e of a tile: request 8 (e / 4) + 4 half + e % 4 of row r32
    const uint32_t row = row0 + r32;
    if (row < a.m) {
#pragma unroll
        for (int q = 0; q < QT; ++q)
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const int r = 32 * (wq * QT + q) + 8 * (e / 4) + 4 * half + (e % 4);
                if (r < nreq) a.y[(size_t)(BYCLASS ? out_req[r] : (uint32_t)(b0 + r)) * a.m + row] = (_Float16)acc[q][e];
            }
    }
}

template <int P, typename S, bool OFFSET>
__global__ __launch_bounds__(S::THREADS) void level_mfma_kernel(LevelParams a)
{
    uint32_t wg = blockIdx.x;
    if (a.nmat > 1) {
        // which matrix this row of workgroups belongs to, picked by comparison (no indexing of the arguments)
        static_assert(BCQ_MAX_MULTI == 4, "the selection below is written for four matrices");
        const bool g1 = wg >= a.mat_blk0[1], g2 = wg >= a.mat_blk0[2], g3 = wg >= a.mat_blk0[3];
        a.planes = g3 ? a.mat_planes[3] : g2 ? a.mat_planes[2] : g1 ? a.mat_planes[1] : a.mat_planes[0];
        a.scales = g3 ? a.mat_scales[3] : g2 ? a.mat_scales[2] : g1 ? a.mat_scales[1] : a.mat_scales[0];
        a.y = g3 ? a.mat_y[3] : g2 ? a.mat_y[2] : g1 ? a.mat_y[1] : a.mat_y[0];
        a.m = g3 ? a.mat_m[3] : g2 ? a.mat_m[2] : g1 ? a.mat_m[1] : a.mat_m[0];
        wg -= g3 ? a.mat_blk0[3] : g2 ? a.mat_blk0[2] : g1 ? a.mat_blk0[1] : 0u;
        a.plane_stride = a.m * a.row_stride;
        a.scale_plane_stride = a.m * a.scale_row_stride;
    }
    const int b0 = (int)blockIdx.y * S::REQS;
    level_body<P, S, OFFSET>(a, b0, min(S::REQS, a.batch - b0), wg);
}

// Per-request precision: byte blockIdx.y of class_order is the precision that a workgroup serves, blockIdx.z its tile of ranks (the slowest
// dimension, so that the tiles that hold the work go first, as in the summing form's kernel).
template <int Q, typename S>
__device__ __forceinline__ void serve_precision(LevelParams a)
{
    if (!a.scale_sets[Q]) {
        // no scale set for this precision: its requests get zeros
        extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
        uint32_t *req_of = reinterpret_cast<uint32_t *>(lds);
        const int nreq = rank_requests<S::REQS>(a.p_req, a.batch, a.p_max, Q, (int)blockIdx.z * S::REQS, req_of);
        if (nreq <= 0) return;
        __syncthreads();
        for (int i = threadIdx.x; i < nreq * S::ROWS; i += S::THREADS) {
            const uint32_t row = blockIdx.x * S::ROWS + (uint32_t)(i % S::ROWS);
            if (row < a.m) a.y[(size_t)req_of[i / S::ROWS] * a.m + row] = (_Float16)0.f;
        }
        return;
    }
    a.scales = a.scale_sets[Q];
    a.offsets = a.offset_sets[Q];
    if (a.offsets) level_body<Q, S, true, true>(a, (int)blockIdx.z * S::REQS, 0, blockIdx.x);
    else level_body<Q, S, false, true>(a, (int)blockIdx.z * S::REQS, 0, blockIdx.x);
}

template <typename S>
__global__ __launch_bounds__(S::THREADS) void level_byclass_kernel(LevelParams a)
{
    switch ((a.class_order >> (8 * blockIdx.y)) & 0xffu) {
    case 1: serve_precision<1, S>(a); break;
    case 2: serve_precision<2, S>(a); break;
    case 3: serve_precision<3, S>(a); break;
    default: serve_precision<4, S>(a); break;
    }
}

template <typename S>
hipError_t launch_byclass(const LevelParams &pr, hipStream_t stream)
{
    auto kernel = level_byclass_kernel<S>;
    constexpr int kWith = Lds<4, S, true>::BYTES > Lds<3, S, true>::BYTES ? Lds<4, S, true>::BYTES : Lds<3, S, true>::BYTES;
    constexpr int kWithout = Lds<4, S, false>::BYTES > Lds<3, S, false>::BYTES ? Lds<4, S, false>::BYTES : Lds<3, S, false>::BYTES;
    constexpr int kTwo = Lds<2, S, true>::BYTES > Lds<2, S, false>::BYTES ? Lds<2, S, true>::BYTES : Lds<2, S, false>::BYTES;
    constexpr int kOne = Lds<1, S, true>::BYTES > Lds<1, S, false>::BYTES ? Lds<1, S, true>::BYTES : Lds<1, S, false>::BYTES;
    constexpr int kMost = kWith > kWithout ? kWith : kWithout, kLess = kTwo > kOne ? kTwo : kOne;
    constexpr int kLds = kMost > kLess ? kMost : kLess;
    if (hipError_t e = allow_dynamic_lds(reinterpret_cast<const void *>(kernel), kLds)) return e;
    hipLaunchKernelGGL(kernel, dim3((pr.m + S::ROWS - 1) / S::ROWS, (unsigned)pr.p_max, (unsigned)((pr.batch + S::REQS - 1) / S::REQS)), dim3(S::THREADS),
                       kLds, stream, pr);
    return hipGetLastError();
}

// what visit_shape hands its function: the kernel of a product
template <int P_, typename S_, bool OFFSET_>
struct Kernel {
    static constexpr int P = P_;
    using S = S_;
    static constexpr bool OFFSET = OFFSET_;
};

template <int P, typename S, bool OFFSET>
hipError_t launch(LevelParams pr, hipStream_t stream)
{
    auto kernel = level_mfma_kernel<P, S, OFFSET>;
    constexpr int kLds = Lds<P, S, OFFSET>::BYTES;
    if (hipError_t e = allow_dynamic_lds(reinterpret_cast<const void *>(kernel), kLds)) return e;
    uint32_t wgs = (pr.m + S::ROWS - 1) / S::ROWS;
    if (pr.nmat > 1) {
        // every matrix gets whole workgroups
        wgs = 0;
        for (int k = 0; k < BCQ_MAX_MULTI; ++k) {
            pr.mat_blk0[k] = wgs;
            if (k < pr.nmat) wgs += (pr.mat_m[k] + S::ROWS - 1) / S::ROWS;
        }
        for (int k = pr.nmat; k < BCQ_MAX_MULTI; ++k) pr.mat_blk0[k] = wgs;      // never reached
    }
    hipLaunchKernelGGL(kernel, dim3(wgs, (unsigned)((pr.batch + S::REQS - 1) / S::REQS)), dim3(S::THREADS), kLds, stream, pr);
    return hipGetLastError();
}

template <typename S, typename F>
hipError_t visit(int p, bool offset, F f)
{
    switch (p) {
    case 1: return offset ? f(Kernel<1, S, true>{}) : f(Kernel<1, S, false>{});
    case 2: return offset ? f(Kernel<2, S, true>{}) : f(Kernel<2, S, false>{});
    case 3: return offset ? f(Kernel<3, S, true>{}) : f(Kernel<3, S, false>{});
    default: return offset ? f(Kernel<4, S, true>{}) : f(Kernel<4, S, false>{});
    }
}

// (four planes with offsets have no room for words of two pairs)
template <typename S, typename F>
hipError_t visit_wide(int p, bool offset, F f)
{
    switch (p) {
    case 1: return offset ? f(Kernel<1, S, true>{}) : f(Kernel<1, S, false>{});
    case 2: return offset ? f(Kernel<2, S, true>{}) : f(Kernel<2, S, false>{});
    case 3: return offset ? f(Kernel<3, S, true>{}) : f(Kernel<3, S, false>{});
    default: return offset ? hipErrorInvalidValue : f(Kernel<4, S, false>{});
    }
}

// f(the kernel that a product at one precision runs with on a shape).  Words for two pairs of groups at a time against one (200 workgroups, 1536 /
// 3840 / 14336 columns in groups of 128, microseconds):
//   128 x 128, p = 4   21.8 / 43.8 / 132    against  21.8 / 44.2 / 137: from three planes on
//              p = 2   17.1 / 34.7 / 108    against  16.6 / 34.0 / 108: not at one and two
//   64 x 128,  p = 4   14.9 / 27.9 / 83.0   against  14.1 / 27.6 / 83.4: beyond 5120 columns
//              p = 3   13.6 / 25.2 / 74.1   against  12.9 / 24.5 / 76.6
//   64 x 64,   p = 4   11.1 / 19.8 / 56.9   against  10.3 / 19.4 / 57.2: the same
//              p = 2   9.2 / 15.2 / 41.6    against  8.6 / 14.2 / 45
// A workgroup starts with both pairs of its first block, and of five pairs two teams get two and one team one: that is what narrow matrices lose.
// (256 x 256 has no registers for it, 128 x 64 no LDS with two workgroups on a CU.)
constexpr int64_t kBlocksBeyond = 5120;         // columns; 64 rows

template <typename F>
hipError_t visit_shape(int shape, int p, bool offset, int64_t n, F f)
{
    const bool wide = n > kBlocksBeyond && !(offset && p == 4);
    switch (shape) {
    case 0: return visit<Shape<8, 8, 1, 1, kNever>>(p, offset, f);
    case 1: return visit<Shape<4, 4, 2, 1, 3>>(p, offset, f);
    case 2: return visit<Shape<4, 4, 1, 2, 3>>(p, offset, f);
    case 3: return wide ? visit_wide<Shape<4, 2, 1, 2, 1>>(p, offset, f) : visit<Shape<4, 2, 1, 2, kNever>>(p, offset, f);
    case 4: return visit<Shape<2, 4, 1, 2, kNever>>(p, offset, f);
    case 5: return wide ? visit_wide<Shape<2, 2, 1, 4, 1>>(p, offset, f) : visit<Shape<2, 2, 1, 4, kNever>>(p, offset, f);
    default: return hipErrorInvalidValue;
    }
}

// Shapes and what a grid of each costs: microseconds per 128 columns with 256 and with at most 128 workgroups on the chip (n = 4096),
// p = 4 and p = 2.  A call costs its rounds of workgroups over the 256 CUs; a round that fills half of the chip is quicker by up to
// a third, because with random operands the full one is held back by power (256 x 256, p = 2, per pair of groups: 7.6 us on 256
// CUs, 5.6 on 128, and 5.3 on 256 with activations of zero).  full_p4z, half_p4z: sixteen levels (p = 4 with offsets), which take two look-ups
// per byte; they stand where the summing form was last measured to be level (5289 x 11520 with 955 requests), although the form has
// become about a tenth faster since: of 69 products drawn at p = 4 with offsets it takes 26, and the choice is 2.6 % behind the better of the two forms.  start_us is the part of a round that does not shrink with the width: the
// first three stages of activations have to arrive, the results to leave, the launch itself (4096 x 256 with 500 requests at
// p = 4 on 128 x 128: 8.5 us, where an eighth of the columns' share of 4096 x 4096 would be 3).
// The LDS of 128 x 64 (72 to 80 KiB, and at most 126 registers) lets two of those workgroups share a CU, that of the others
// one.  Large tiles rebuild a weight for more requests, small ones keep the CUs busy on short matrices and batches.
struct LevelShape {
    int rows, reqs;
    float full_p4, full_p2, half_p4, half_p2, start_us, full_p4z, half_p4z;
};
constexpr LevelShape kLevelShapes[kLevelShapeCount] = {{256, 256, 4.30f, 3.86f, 3.28f, 2.53f, 8.2f, 4.95f, 3.56f}, {128, 256, 2.71f, 2.40f, 2.11f, 1.65f, 5.9f, 3.30f, 2.85f},
                                       {128, 128, 1.46f, 1.29f, 1.22f, 0.97f, 6.4f, 1.78f, 1.57f}, {64, 128, 0.96f, 0.90f, 0.82f, 0.71f, 6.7f, 1.18f, 1.01f},
                                       {128, 64, 0.98f, 0.76f, 0.89f, 0.63f, 4.0f, 1.22f, 1.10f},  {64, 64, 0.63f, 0.53f, 0.57f, 0.44f, 5.3f, 0.76f, 0.74f}};
// 128 x 96, for the requests of one precision of a batch
constexpr LevelShape kLevel96 = {128, 96, 1.25f, 1.08f, 1.08f, 0.82f, 6.2f, 1.55f, 1.38f};

}  // namespace

// whole pairs of 128-column groups; 32-bit byte offsets are the caller's condition (dequant_mfma_supports)
bool level_mfma_supports(const GemmArgs &a) { return a.uniform_p >= 1 && a.uniform_p <= kMaxP && a.n % 256 == 0; }

namespace {

// What a product is expected to take on a shape; times > 0: that many products of this size in one launch, one per precision.
float shape_us(const LevelShape &c, const GemmArgs &a, int times)
{
    const int p = a.uniform_p;
    const bool classes = times > 0;
    const float wgs = (float)((a.m + c.rows - 1) / c.rows) * (float)((a.batch + c.reqs - 1) / c.reqs) * (float)(classes ? times : 1);
    const bool sixteen = p == 4 && a.offsets[p];
    const float full = sixteen ? c.full_p4z : p >= 3 ? c.full_p4 : c.full_p2, half = sixteen ? c.half_p4z : p >= 3 ? c.half_p4 : c.half_p2;
    const float rounds = __builtin_floorf(wgs / 256.f), rest = wgs / 256.f - rounds;
    float all = 32.f * (rounds * full + (rest == 0.f ? 0.f : rest <= 0.5f ? half : half + (full - half) * (2.f * rest - 1.f)));
    float start = c.start_us * __builtin_ceilf(wgs / 256.f);
    if (classes) {
        // Per-request precision: every precision at the price of the deepest comes out a seventh too high, and a workgroup ranks the
        // batch before anything else.
        const float rank_us = 2.5f;
        all *= 0.87f;
        start = (c.start_us + rank_us) * __builtin_ceilf(wgs / 256.f);
        return large_batch_us(all > start ? all : start, start, a.n) + (a.n < 4096 ? 0.f : rank_us);
    }
    // Two workgroups on a CU (4096 columns, p = 4: 256 of them take 36.9 us, 320 59.0, 512 64.0) on longer rows lose it again:
    // a lane reads 16 bytes of a row at a time, and the lines of that many rows do not stay in L2 from one read to the next
    // (21248 x 8192 with 587 requests at p = 4: 1.7 times what 4096 columns would let one expect).
    if (c.rows == 128 && c.reqs == 64 && wgs > 256.f && a.n <= 4096) all *= 0.85f;
    return large_batch_us(all, start, a.n);
}

}  // namespace

int level_mfma_cheapest(const GemmArgs &a, float &us)
{
    int best = -1;
    for (int k = 0; k < kLevelShapeCount; ++k) {
        const float all = shape_us(kLevelShapes[k], a, 0);
        if (best < 0 || all < us) {
            best = k;
            us = all;
        }
    }
    // At p <= 2 the summing form takes about 1.05 times the time its prices say.
    if (a.uniform_p <= 2) us *= 0.95f;
    return best;
}

int level_mfma_cheapest_classes(const GemmArgs &a, int nsets, float &us)
{
    int best = -1;
    for (int k = 1; k <= kLevelShapeCount; ++k) {
        const float all = shape_us(k < kLevelShapeCount ? kLevelShapes[k] : kLevel96, a, nsets);
        if (best < 0 || all < us) {
            best = k;
            us = all;
        }
    }
    if (a.n < 3072) us *= 1.15f;        // (drawn calls took 0.99 to 1.28 times the estimate there, 0.79 to 1.09 times beyond)
    return best;
}

namespace {

LevelParams level_params(const GemmArgs &a)
{
    LevelParams pr{};
    pr.planes = reinterpret_cast<const unsigned char *>(a.planes);
    pr.x = reinterpret_cast<const unsigned char *>(a.x);
    pr.y = a.y;
    pr.plane_stride = (uint32_t)(a.m * (a.n / 8));
    pr.row_stride = (uint32_t)(a.n / 8);
    pr.scale_plane_stride = (uint32_t)(a.m * (a.n / a.group) * 2);
    pr.scale_row_stride = (uint32_t)((a.n / a.group) * 2);
    pr.gshift = a.group == 256 ? 1 : a.group == 64 ? -1 : 0;
    pr.x_stride = (uint32_t)(a.n * 2);
    pr.m = (uint32_t)a.m;
    pr.batch = a.batch;
    pr.npairs = (int)(a.n / 256);
    return pr;
}

}  // namespace

hipError_t level_mfma_launch_classes(const GemmArgs &a, uint32_t class_order, int shape, hipStream_t stream)
{
    LevelParams pr = level_params(a);
    for (int q = 1; q <= kMaxP; ++q) {
        pr.scale_sets[q] = reinterpret_cast<const unsigned char *>(a.scales[q]);
        pr.offset_sets[q] = a.scales[q] ? reinterpret_cast<const unsigned char *>(a.offsets[q]) : nullptr;
    }
    pr.p_req = a.p_req;
    pr.p_max = a.p_max;
    pr.class_order = class_order;
    switch (shape) {
    case 1: return launch_byclass<Shape<4, 4, 2, 1, 3>>(pr, stream);
    case 2: return launch_byclass<Shape<4, 4, 1, 2, 3>>(pr, stream);
    case 3: return launch_byclass<Shape<4, 2, 1, 2, kNever>>(pr, stream);
    case 4: return launch_byclass<Shape<2, 4, 1, 2, kNever>>(pr, stream);
    case 5: return launch_byclass<Shape<2, 2, 1, 4, kNever>>(pr, stream);
    case 6: return launch_byclass<Shape<3, 4, 1, 2, 3>>(pr, stream);
    default: return hipErrorInvalidValue;
    }
}

hipError_t level_mfma_launch(const GemmArgs &a, int shape, hipStream_t stream, const GemmArgs *mats, int count)
{
    LevelParams pr = level_params(a);
    pr.scales = reinterpret_cast<const unsigned char *>(a.scales[a.uniform_p]);
    const bool offset = a.offsets[a.uniform_p] != nullptr;
    pr.offsets = reinterpret_cast<const unsigned char *>(a.offsets[a.uniform_p]);
    if (mats && count > 1) {
        pr.nmat = count;
        for (int k = 0; k < count; ++k) {
            pr.mat_planes[k] = reinterpret_cast<const unsigned char *>(mats[k].planes);
            pr.mat_scales[k] = reinterpret_cast<const unsigned char *>(mats[k].scales[a.uniform_p]);
            pr.mat_y[k] = mats[k].y;
            pr.mat_m[k] = (uint32_t)mats[k].m;
        }
    }
    return visit_shape(shape, a.uniform_p, offset, a.n, [&](auto k) {
        using K = decltype(k);
        return launch<K::P, typename K::S, K::OFFSET>(pr, stream);
    });
}

LevelLayout level_mfma_layout(const GemmArgs &a, int shape)
{
    const LevelParams pr = level_params(a);
    LevelLayout out{};
    (void)visit_shape(shape, a.uniform_p, a.offsets[a.uniform_p] != nullptr, a.n, [&](auto k) {
        using M = Lds<decltype(k)::P, typename decltype(k)::S, decltype(k)::OFFSET>;
        const ScaleWindow w = scale_window(M::WINDOW, pr.scale_row_stride, pr.gshift, pr.npairs);
        out = {M::BYTES, 256 * w.pairs, M::PLANES * (decltype(k)::S::ROWS << w.row_log2) / 256, M::COALESCE ? 512 : 256};
        return hipSuccess;
    });
    return out;
}

}  // namespace bcq
