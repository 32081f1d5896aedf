// A whole Gauss-Seidel half-sweep (eight colours) in one launch, for the
// levels where a launch per colour is bound by latency.
//
// A workgroup owns a tile of the level -- whole x-lines, n cells in y and m
// in z (a cell is two grid lines) -- and relaxes the eight colours of its
// tile one after the other in LDS, with a workgroup barrier in place of the
// kernel boundary.  A colour of the tile needs the new values of earlier
// colours in its neighbours, so each colour is relaxed on the tile plus the
// halo that the later colours reach: the chain of colours moves at most three
// cells in y and one in z (see sweep_args), never across workgroups.  Halo rows
// are relaxed by every workgroup that needs them, from the same old values
// with the same operations, so all copies agree and the result equals the
// colour launches bit for bit; the sweep reads its old values from one
// vector and writes the new ones to another, because a neighbouring
// workgroup may still need the old ones.  No workgroup waits for another.
//
// What bounds it: latency.  A colour launch on a small level is two dependent
// memory round trips (the row's entries, then its neighbours) and a kernel
// boundary, 3-6 us whatever the row count; here the entries of the next
// colour's rows, which depend on no z, are loaded while the current colour
// is relaxed, the neighbours come from LDS, and a colour takes 0.6-0.8 us
// (the issue of its instructions: finding the row, 26 loads, 26 LDS reads
// and 26 dependent FMAs).  The price is the halo: 1.3 to 3 times the rows on
// levels near cubes, up to 6 times where a line fills the LDS (sweep_pays).
// Measured, FP32 forward, the eight launches with their gaps against this
// one: 64^3 level 45 -> 12 us from zero with the restriction, 13.6 us with
// the prolongation; 32^3 36 -> 10; 16^3 27 -> 8.  Solves of 16^3
// (symmetric) 6.5 -> 3.4 ms, 48 x 40 x 32 9.9 -> 5.4 ms, 128^3 63 -> 52 ms.
// Where a tile's rows take one lane each, the waves split (SPLIT): while one
// half relaxes its colour the other finds and loads the next, which took
// solves of 16^3 from 3.2 to 2.8 ms, of 48 x 40 x 32 in binary16 from 5.1 to
// 4.4 ms and a batch of 3 x 40x48x56 from 7.8 to 6.9 ms.  Slower variants:
// columns loaded and mapped to LDS cells (18 us on every size), scalar loads
// of each position's constants (+0.4 us a colour), split waves with several
// row chunks each (+20 %: the registers spill).
//
// The tile's z lies in LDS with the same strides for every colour, each line
// followed by a zero cell and the lines outside the grid zero, so a
// neighbour's cell is the row's own plus an offset that depends on the
// colour and the slot only (the colour-blocked order puts every neighbour at
// a fixed offset; the padded slots fall on the zeros).  The rows' values come
// from the stored matrix.
#include "ell_device.hpp"

#include <algorithm>
#include <map>
#include <memory>
#include <stdexcept>
#include <type_traits>

namespace hpgmx {

// Threads of a workgroup at most: a row and the next one take up to 128 VGPRs
// (four waves per SIMD), in FP64 up to 256 (two).
template <typename V> constexpr int sweep_threads() { return sizeof(V) == 8 ? 512 : 1024; }
constexpr int kCus = 256;
constexpr size_t kSweepLds = 144 * 1024;  // bytes of z a workgroup may hold (of the CU's 160 KiB)

// A launch's tiles.  Boxes are in cells, relative to the tile's first cell,
// and not clipped to the grid.
struct SweepArgs {
    // per sweep position (8: the restriction) the rows worked on and the
    // neighbours read: jlo + 8, jn, klo + 8, kn in 4, 5, 4, 5 bits, then bit
    // f - 1 for the slots to colour c ^ f
    unsigned pos[9];
    int off[8];            // first row of each colour
    int nx1, ny1, nz1;     // extents + 1
    int n, m, tj;          // cells per tile in y and z, tiles in y
    int remap, forward;
    int first, tail;       // first sweep position; 0, or the restriction after the sweep: 1 from the slots to
                           // colours relaxed after colour 4, 2 r - A z
    unsigned bytes;        // of the off-diagonal values
    int sx, pj, pk;        // cells per line (the zero included), lines per plane and planes held per colour
    int hj, hk;            // the held box's first line and plane
    int coff[8], cnx1, cny1;  // the coarse level (restriction, prolongation)
};
__host__ __device__ inline unsigned pack_pos(int jlo, int jn, int klo, int kn, unsigned flips)
{
    return (unsigned)(jlo + 8) | (unsigned)jn << 4 | (unsigned)(klo + 8) << 9 | (unsigned)kn << 13 | flips << 18;
}

namespace {

__device__ __forceinline__ void lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// t / d for 0 <= t < 2^20 and 1 <= d, with rd the hardware's 1 / d: (t + 1/2) / d
// is at least 1/(2d) away from an integer, and the product's relative error
// (below 2^-21) is smaller than that for these t.
__device__ __forceinline__ int small_div(int t, float rd) { return (int)(((float)t + 0.5f) * rd); }
__device__ __forceinline__ float recip(int d) { return __builtin_amdgcn_rcpf((float)d); }

// The off-diagonal values through a buffer resource: a load takes a 32-bit
// offset per lane, the slot's place in a scalar register and an immediate,
// with no address arithmetic of its own, and a lane past the end reads 0.
// 16-bit values stay in a register each until they are used: two to a
// register, a load would wait for the one before it.
template <typename V> struct SlotLoads {
    using Raw = std::conditional_t<sizeof(V) == 2, unsigned, V>;
    static __device__ __forceinline__ V value(Raw w)
    {
        if constexpr (sizeof(V) == 2) return __builtin_bit_cast(V, (unsigned short)w);
        else return w;
    }
    static constexpr int kStride = (int)sizeof(V) << kDefaultEllChunkLog2;  // bytes from slot to slot
    __amdgpu_buffer_rsrc_t rsrc;
    __device__ __forceinline__ SlotLoads(const V *v, unsigned bytes)
        : rsrc(__builtin_amdgcn_make_buffer_rsrc(const_cast<V *>(v), 0, (int)bytes, 0x00027000)) {}
    __device__ __forceinline__ Raw at(int s, unsigned off) const
    {
        const int imm = s * kStride % 4096, base = s * kStride - imm;
        if constexpr (sizeof(V) == 8) {
            typedef unsigned u2 __attribute__((ext_vector_type(2)));
            const u2 w = __builtin_amdgcn_raw_buffer_load_b64(rsrc, (int)(off + imm), base, 0);
            return __builtin_bit_cast(V, w);
        } else if constexpr (sizeof(V) == 4) {
            return __builtin_bit_cast(V, __builtin_amdgcn_raw_buffer_load_b32(rsrc, (int)(off + imm), base, 0));
        } else {
            return (unsigned short)__builtin_amdgcn_raw_buffer_load_b16(rsrc, (int)(off + imm), base, 0);
        }
    }
};

// Internal index of coarse point (I, J, K).
__device__ __forceinline__ int coarse_index(const SweepArgs &P, int I, int J, int K)
{
    const int c = colour_of(I, J, K);
    int o[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        o[q] = P.coff[q];
        asm("" : "+s"(o[q]));  // select among eight registers, not among addresses to load from
    }
    int off = o[0];
#pragma unroll
    for (int q = 1; q < 8; ++q) off = c == q ? o[q] : off;
    const int bx = (P.cnx1 - (I & 1)) >> 1, by = (P.cny1 - (J & 1)) >> 1;
    return off + (I >> 1) + bx * ((J >> 1) + by * (K >> 1));
}

__host__ __device__ constexpr int slot_flip(int s)
{
    const int t = s < 13 ? s : s + 1;
    return ((t % 3 - 1) & 1) | (((t / 3) % 3 - 1) & 1) << 1 | ((t / 9 - 1) & 1) << 2;
}

// Right-hand sides per lane of a batch of K.  Two share the row's loads and
// read their neighbours together: 30 steps at 8 x 48^3 in FP32 7619 -> 6654
// us, 4 x 64^3 6468 -> 6022, FP64 4 x 48^3 6961 -> 6463, and 1-4 % more at
// 16^3; four lost to two at 8 x 32^3 and by 20 % in FP64.
template <int K> constexpr int kSweepR = K >= 2 ? 2 : 1;

// One row's entries, loaded ahead of its relaxation.
template <typename V, typename S, int R> struct SweepRow {
    typename SlotLoads<V>::Raw a[kSlots];
    Pack<S, R> r;
    V d;
    int cell;         // its own, times K, plus the right-hand side
    int ii, jj, kk;   // in its colour block
    bool act;
};

}  // namespace

// K interleaved right-hand sides, R per lane (K / R lanes share a row).
// SPLIT: a tile whose rows take one lane each at every position.  Half of the
// waves relax the even positions, the others the odd ones, and each half
// finds and loads its next rows while the other relaxes.
template <typename V, typename S, int K, int R, bool SPLIT>
__global__ __launch_bounds__(sweep_threads<V>()) void k_sweep(const SweepArgs P, const V *__restrict__ offv,
                                                         const V *__restrict__ diag, const S *__restrict__ r,
                                                         const S *__restrict__ zin, const S *__restrict__ zc,
                                                         S *__restrict__ zout, S *__restrict__ rc)
{
    using T = typename VecT<V>::T;
    using Row = SweepRow<V, S, R>;
    constexpr int L = K / R;
    constexpr unsigned kChunk = 1u << kDefaultEllChunkLog2;
    extern __shared__ __align__(16) unsigned char smem[];
    S *zs = reinterpret_cast<S *>(smem);
    const int tid = threadIdx.x, nt = blockDim.x;
    const int ng = SPLIT ? nt / 2 : nt;  // lanes that work on a position
    const int group = SPLIT ? __builtin_amdgcn_readfirstlane(tid >= ng ? 1 : 0) : 0, gid = tid - group * ng;
    const int rhs = K > 1 ? tid % L * R : 0;
    const int tile = (int)xcd_tile(blockIdx.x, gridDim.x, P.remap);
    const int kt = tile / P.tj, K0 = kt * P.m, J0 = (tile - kt * P.tj) * P.n;
    const int plane = P.sx * P.pj, block = plane * P.pk;  // cells
    const int bxe = P.nx1 >> 1;                           // the longer of the two line lengths
    const float rbx = recip(bxe);
    auto colour = [&](int pos) { return pos == 8 ? 4 : P.forward ? pos : 7 - pos; };
    auto ext_x = [&](int c) { return (P.nx1 - (c & 1)) >> 1; };
    auto ext_y = [&](int c) { return (P.ny1 - ((c >> 1) & 1)) >> 1; };
    auto ext_z = [&](int c) { return (P.nz1 - (((c >> 2) & 1) ^ 1)) >> 1; };

    // lane q holds position q's word, lane 16 + c colour c's first row: read
    // from there, not from the arguments, whose scalar loads each position
    // would wait for
    const int lane = tid & 63;
    int table = 0;
#pragma unroll
    for (int q = 0; q < 9; ++q) table = lane == q ? (int)P.pos[q] : table;
#pragma unroll
    for (int c = 0; c < 8; ++c) table = lane == 16 + c ? P.off[c] : table;
    auto word = [&](int pos) { return (unsigned)__builtin_amdgcn_readlane(table, pos); };
    const SlotLoads<V> slots(offv, P.bytes);

    // loads this lane's row of chunk `chunk` of position pos
    auto fetch = [&](int pos, int chunk, Row &E) {
        const unsigned q = word(pos);
        const int c = colour(pos), jn = q >> 4 & 31, jlo = (int)(q & 15) - 8, klo = (int)(q >> 9 & 15) - 8;
        const int kn = q >> 13 & 31;
        const int t = (SPLIT ? gid : chunk * nt + tid) / L;
        const int line = small_div(t, rbx), ii = t - __mul24(line, bxe);
        const int kq = small_div(line, recip(jn)), jr = jlo + (line - __mul24(kq, jn)), kr = klo + kq;
        const int jj = J0 + jr, kk = K0 + kr;
        const int bx = ext_x(c), by = ext_y(c);
        E.act = (kq < kn) & (ii < bx) & ((unsigned)jj < (unsigned)by) & ((unsigned)kk < (unsigned)ext_z(c));
        E.cell = (1 + c * block + ii + __mul24(P.sx, (jr - P.hj) + __mul24(P.pj, kr - P.hk))) * K + rhs;
        E.ii = ii; E.jj = jj; E.kk = kk;
        const int p = E.act ? (int)word(16 + c) + ii + __mul24(bx, jj + __mul24(by, kk)) : 0;
        E.r = ldp<S, R>(r + ((i64)p * K + rhs));
        E.d = diag[p];
        const unsigned e = E.act ? ((unsigned)__mul24(p / (int)kChunk, kSlots * kChunk) + (unsigned)p % kChunk) *
                                       (unsigned)sizeof(V)
                                 : 0x80000000u;  // past the end
#pragma unroll
        for (int f = 1; f < 8; ++f) {
            if (q >> (17 + f) & 1u) {
#pragma unroll
                for (int s = 0; s < kSlots; ++s)
                    if (slot_flip(s) == f) E.a[s] = slots.at(s, e);
            } else {  // not read: adds 0
#pragma unroll
                for (int s = 0; s < kSlots; ++s)
                    if (slot_flip(s) == f) E.a[s] = 0;
            }
        }
    };

    // sum over the slots of a z, the z gathered from LDS, in slot order
    auto row_sum = [&](int pos, const Row &E, T (&acc)[R]) {
        const int c = colour(pos);
        // cell of the neighbour minus the row's own: an even line's (or
        // plane's) neighbours are the odd ones of the cell before and of its
        // own, an odd one's the even ones of its own cell and of the one after
        const bool xo = c & 1, yo = c & 2, zo = !(c & 4);  // colours 0-3 lie on the odd planes
        const int fx = (xo ? -block : block) + (xo ? 0 : -1), fy = yo ? -2 * block : 2 * block,
                  fz = (c & 4) ? -4 * block : 4 * block;
        const int dy[3] = {fy - (yo ? 0 : P.sx), 0, fy + (yo ? P.sx : 0)};
        const int dz[3] = {fz - (zo ? 0 : plane), 0, fz + (zo ? plane : 0)};
        Pack<S, R> xv[kSlots];
#pragma unroll
        for (int g = 0; g < 9; ++g) {  // lines dk, dj
            const int at = E.cell + (dz[g / 3] + dy[g % 3]) * K;
            const S *x = zs + (at + fx * K);
            const int s = 3 * g - (g > 4 ? 1 : 0);  // slot of di = -1
            xv[s] = ldp<S, R>(x);
            if (g != 4) xv[s + 1] = ldp<S, R>(zs + at);
            xv[g == 4 ? s + 1 : s + 2] = ldp<S, R>(x + K);
        }
#pragma unroll
        for (int i = 0; i < R; ++i) acc[i] = (T)0;
#pragma unroll
        for (int s = 0; s < kSlots; ++s)
#pragma unroll
            for (int i = 0; i < R; ++i) acc[i] = madd(to_t<T>(SlotLoads<V>::value(E.a[s])), to_t<T>(xv[s].v[i]), acc[i]);
    };

    // The restriction after a sweep from zero leaves out slots whose z is not
    // zero (at the other positions such cells still hold zero): row_sum adds 0
    // times it, which is not 0 where it is infinite or not a number.  A sum
    // that is not a number is formed again from the position's slots alone, in
    // the same order.
    auto skip_not_finite = [&](const Row &E, T (&acc)[R]) {
        bool bad = false;
#pragma unroll
        for (int i = 0; i < R; ++i) bad = bad || acc[i] != acc[i];
        if (!bad) return;
        const unsigned q = word(8);
        const int p = (int)word(16 + 4) + E.ii + ext_x(4) * (E.jj + ext_y(4) * E.kk);
#pragma unroll
        for (int i = 0; i < R; ++i) acc[i] = (T)0;
#pragma unroll 1
        for (int s = 0; s < kSlots; ++s) {
            if (!(q >> (17 + slot_flip(s)) & 1u)) continue;
            const int t = s < 13 ? s : s + 1, di = t % 3 - 1, dj = (t / 3) % 3 - 1, dk = t / 9 - 1;
            // colour 4 lies on even lines and planes
            const int at = E.cell + ((di ? block + (di < 0 ? -1 : 0) : 0) + (dj ? 2 * block - (dj < 0 ? P.sx : 0) : 0) +
                                     (dk ? -4 * block - (dk < 0 ? plane : 0) : 0)) * K;
            const T a = to_t<T>(offv[(i64)(p / (int)kChunk) * (kSlots * kChunk) + s * kChunk + p % (int)kChunk]);
#pragma unroll
            for (int i = 0; i < R; ++i) acc[i] = madd(a, to_t<T>(zs[at + i]), acc[i]);
        }
    };

    const int last = P.tail ? 8 : 7;
    auto chunks = [&](int pos) {
        const unsigned q = word(pos);
        return (bxe * (int)(q >> 4 & 31) * (int)(q >> 13 & 31) * L + nt - 1) / nt;
    };

    // (the second half of split waves loads its first rows in the loop below:
    // here they would compete with the z that everyone waits for, 48 x 40 x 32
    // binary16 solve 4023 against 4077 us)
    Row A;
    if (group == 0) fetch(P.first, 0, A);

    // z: the old values, or zero
    if (zin) {
        if (tid < K) zs[tid] = from_t<S>((T)0);
        const float rsx = recip(P.sx), rpj = recip(P.pj);
        for (int e = tid; e < block * K; e += nt) {
            const int t = e / K, j = e % K, line = small_div(t, rsx), ii = t - line * P.sx;
            const int kq = small_div(line, rpj), jj = J0 + P.hj + (line - kq * P.pj), kk = K0 + P.hk + kq;
            S v[8], w = from_t<S>((T)0);
#pragma unroll
            for (int c = 0; c < 8; ++c) {
                const int bx = ext_x(c), by = ext_y(c);
                v[c] = from_t<S>((T)0);
                if (ii < bx && (unsigned)jj < (unsigned)by && (unsigned)kk < (unsigned)ext_z(c)) {
                    v[c] = zin[(i64)(P.off[c] + ii + bx * (jj + by * kk)) * K + j];
                    if (c == 4 && zc) w = zc[(i64)coarse_index(P, ii, jj, kk) * K + j];
                }
            }
            sched_fence();
            if (zc) v[4] = from_t<S>(to_t<T>(v[4]) + to_t<T>(w));
#pragma unroll
            for (int c = 0; c < 8; ++c) zs[(1 + c * block + t) * K + j] = v[c];
        }
    } else {
        const int words = ((1 + 8 * block) * K * (int)sizeof(S) + 15) / 16;
        for (int e = tid; e < words; e += nt) reinterpret_cast<uint4 *>(smem)[e] = uint4{0, 0, 0, 0};
    }
    lds_barrier();

    auto relax = [&](int pos, const Row &E) {
        if (E.act) {
            T acc[R];
            Pack<S, R> out;
            row_sum(pos, E, acc);
            if (pos < 8) {
#pragma unroll
                for (int i = 0; i < R; ++i) out.v[i] = from_t<S>((to_t<T>(E.r.v[i]) - acc[i]) / to_t<T>(E.d));
                stp<S, R>(zs + E.cell, out);
            } else {  // the colour-4 block is the coarse level in its natural order
                if (P.tail == 1) skip_not_finite(E, acc);
                const Pack<S, R> own = ldp<S, R>(zs + E.cell);
#pragma unroll
                for (int i = 0; i < R; ++i)
                    out.v[i] = from_t<S>(P.tail == 1 ? -acc[i]
                                                     : to_t<T>(E.r.v[i]) - (to_t<T>(E.d) * to_t<T>(own.v[i]) + acc[i]));
                stp<S, R>(rc + ((i64)coarse_index(P, E.ii, E.jj, E.kk) * K + rhs), out);
            }
        }
    };
    if constexpr (SPLIT) {
        for (int pos = P.first;; ++pos) {
            if (((pos - P.first) & 1) == group) relax(pos, A);
            else if (pos < last) fetch(pos + 1, 0, A);
            if (pos == last) break;
            lds_barrier();
        }
    } else {
        Row B;
        int pos = P.first, chunk = 0, nchunks = chunks(pos);
        // one chunk of rows: E holds its entries, F takes those of the next one
        auto step = [&](Row &E, Row &F) -> bool {
            int npos = pos, nchunk = chunk + 1;
            if (nchunk == nchunks) {
                npos = pos + 1;
                nchunk = 0;
            }
            // E was loaded during the chunk before: wait for it before the next
            // loads go out, not behind them
            __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0)
            sched_fence();
            if (npos <= last) fetch(npos, nchunk, F);
            sched_fence();
            relax(pos, E);
            if (npos > last) return true;
            if (npos != pos) {
                lds_barrier();
                nchunks = chunks(npos);
            }
            pos = npos;
            chunk = nchunk;
            return false;
        };
        while (!step(A, B) && !step(B, A)) {}
    }
    if (!P.tail) lds_barrier();

    // the tile's own rows
    const float rn = recip(P.n);
    for (int e = tid; e < bxe * P.n * P.m * K; e += nt) {
        const int t = e / K, j = e % K, line = small_div(t, rbx), ii = t - line * bxe;
        const int kq = small_div(line, rn), jq = line - kq * P.n, jj = J0 + jq, kk = K0 + kq;
        const int cell = 1 + ii + P.sx * ((jq - P.hj) + P.pj * (kq - P.hk));
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            const int bx = ext_x(c), by = ext_y(c);
            if (ii < bx && jj < by && kk < ext_z(c))
                zout[(i64)(P.off[c] + ii + bx * (jj + by * kk)) * K + j] = zs[(cell + c * block) * K + j];
        }
    }
}

namespace {

struct Box {  // [jlo, jhi) x [klo, khi) in cells
    int jlo, jhi, klo, khi;
    void add(const Box &b)
    {
        jlo = std::min(jlo, b.jlo); jhi = std::max(jhi, b.jhi);
        klo = std::min(klo, b.klo); khi = std::max(khi, b.khi);
    }
};

// The colour-(c ^ f) cells next to the colour-c cells of b: an even line's
// neighbours are the odd lines of the cell before and of its own, an odd
// line's the even lines of its own cell and of the one after.
Box reach(const Box &b, int c, int f)
{
    Box o = b;
    if (f & 2) { if (c & 2) ++o.jhi; else --o.jlo; }
    if (f & 4) { if (c & 4) --o.klo; else ++o.khi; }  // colours 4-7 lie on the even planes
    return o;
}

// Fills P for tiles of n x m cells; returns the LDS cells a workgroup needs.
i64 sweep_args(SweepArgs &P, const Geom &g, const Geom *gc, int n, int m, bool forward, bool zero, bool skip_first,
               int tail)
{
    const Box own{0, n, 0, m};
    Box need[8];
    auto pos = [&](int c) { return forward ? c : 7 - c; };
    auto flips = [&](unsigned mask) {
        unsigned b = 0;
        for (int s = 0; s < kSlots; ++s)
            if (mask >> s & 1u) b |= 1u << (slot_flip(s) - 1);
        return b;
    };
    const unsigned tailmask = tail == 1 ? kAllSlots & ~zero_guess_mask(4, forward) : kAllSlots;
    for (Box &b : need) b = own;
    if (tail)
        for (int f = 1; f < 8; ++f)
            if (flips(tailmask) >> (f - 1) & 1u) need[4 ^ f].add(reach(own, 4, f));
    // a row relaxed at a position needs the new values of every earlier colour next to it
    for (int q = 7; q >= 0; --q) {
        const int c = forward ? q : 7 - q;
        for (int f = 1; f < 8; ++f)
            if (pos(c ^ f) < q) need[c ^ f].add(reach(need[c], c, f));
    }
    // held: these, and what a row next to them reads (zeros, in a sweep from zero)
    Box held = own;
    for (int c = 0; c < 8; ++c) {
        held.add(need[c]);
        for (int f = 1; f < 8; ++f) held.add(reach(need[c], c, f));
    }
    for (int q = 0; q < 9; ++q) {
        const int c = q == 8 ? 4 : forward ? q : 7 - q;
        const Box &b = q == 8 ? own : need[c];
        P.pos[q] = pack_pos(b.jlo, b.jhi - b.jlo, b.klo, b.khi - b.klo,
                            flips(q == 8 ? tailmask : zero ? zero_guess_mask(c, forward) : kAllSlots));
    }
    for (int c = 0; c < 8; ++c) P.off[c] = (int)g.off[c];
    P.nx1 = g.nx + 1; P.ny1 = g.ny + 1; P.nz1 = g.nz + 1;
    P.n = n; P.m = m;
    P.tj = ((g.ny + 1) / 2 + n - 1) / n;
    P.forward = forward;
    P.first = skip_first ? 1 : 0;
    P.tail = tail;
    P.sx = (g.nx + 1) / 2 + 1;
    P.hj = held.jlo; P.pj = held.jhi - held.jlo;
    P.hk = held.klo; P.pk = held.khi - held.klo;
    if (gc) {
        for (int c = 0; c < 8; ++c) P.coff[c] = (int)gc->off[c];
        P.cnx1 = gc->nx + 1; P.cny1 = gc->ny + 1;
    }
    return 1 + (i64)8 * P.sx * P.pj * P.pk;
}

int sweep_tiles(const Geom &g, int n, int m)
{
    return (((g.ny + 1) / 2 + n - 1) / n) * (((g.nz + 1) / 2 + m - 1) / m);
}

// Lanes at work at position q, of the arguments P for tiles of one cell, when
// the tiles have n x m cells (every box grows with its tile).
i64 sweep_lanes(const SweepArgs &P, int q, int n, int m, int L)
{
    return (i64)(P.nx1 >> 1) * ((P.pos[q] >> 4 & 31) - 1 + n) * ((P.pos[q] >> 13 & 31) - 1 + m) * L;
}

// The tile whose workgroups, taken one per CU, have the least to work through
// one after the other: row chunks, which take a sixth less time where the
// waves can split (k_sweep); of equal ones the smallest.
struct Tile {
    int n = 1, m = 1;
    size_t lds = 0;  // bytes of a workgroup (0: no tile fits)
    i64 cost = 0;    // sixths of a row chunk
};
Tile choose_tile(const Geom &g, const SweepArgs &P, int K, int L, int threads, size_t vb)
{
    Tile t;
    for (int mm = 1; mm <= 8; ++mm)
        for (int nn = 1; nn <= 8; ++nn) {
            const i64 cells = 1 + (i64)8 * P.sx * (P.pj - 1 + nn) * (P.pk - 1 + mm);
            const size_t b = ((size_t)cells * K * vb + 15) / 16 * 16;
            if (b > kSweepLds) break;
            i64 items = 0, most = 0;
            for (int q = P.first; q < 8; ++q) {
                const i64 lanes = sweep_lanes(P, q, nn, mm, L);
                items += (lanes + threads - 1) / threads;
                most = std::max(most, lanes);
            }
            const i64 cost = (sweep_tiles(g, nn, mm) + kCus - 1) / kCus * items * (most <= threads / 2 ? 5 : 6);
            if (t.lds == 0 || cost < t.cost) t = Tile{nn, mm, b, cost};
        }
    return t;
}

template <typename V, typename S, int K, bool SPLIT>
void sweep_launch(const V *v, const V *d, const SweepArgs &P, int tiles, int threads, size_t lds, const void *r,
                  const void *zin, const void *zc, void *zout, void *rc, hipStream_t s)
{
    // the most any launch takes, not this one's: the setting is the kernel's,
    // shared by every handle and thread of the process
    if (lds > 64 * 1024 && hipFuncSetAttribute(reinterpret_cast<const void *>(&k_sweep<V, S, K, kSweepR<K>, SPLIT>),
                                               hipFuncAttributeMaxDynamicSharedMemorySize, (int)kSweepLds) != hipSuccess)
        throw std::runtime_error("launch_sweep: the device refuses the workgroup's LDS");
    hipLaunchKernelGGL((k_sweep<V, S, K, kSweepR<K>, SPLIT>), dim3(tiles), dim3(threads), lds, s, P, v, d, (const S *)r, (const S *)zin,
                       (const S *)zc, (S *)zout, (S *)rc);
}

}  // namespace

// One form of a level's sweep, ready to launch.  Working it out takes the host
// 4-6 us, as long as the launch itself and longer than the launch leaves it on
// a small level, so it is kept (16^3 symmetric solve from the host 2.78 ->
// 2.49 ms).
struct SweepPlan {
    SweepArgs P{};
    int tiles = 0, threads = 0;
    bool split = false;
    size_t lds = 0;
};
struct SweepPlans {
    std::map<unsigned, SweepPlan> form;
    std::map<unsigned, bool> possible, pays;
};

static SweepPlans &plans_of(const Matrix &A)
{
    if (!A.sweeps) A.sweeps = std::make_shared<SweepPlans>();
    return *A.sweeps;
}

// A tile of one cell fits the LDS in every form of the launch: either
// direction, from zero or from old values, with the restriction (which
// reaches further than the sweep alone).
static bool fits_lds(const Matrix &A, int K, Prec p)
{
    for (int form = 0; form < 4; ++form) {
        SweepArgs P;
        const bool zero = form & 2;
        const i64 cells = sweep_args(P, A.g, nullptr, 1, 1, form & 1, zero, false, zero ? 1 : 2);
        if (cells * K * (i64)vec_bytes(p) > (i64)kSweepLds - 16) return false;
    }
    return true;
}

static bool sweep_possible(const Matrix &A, int K, Prec p)
{
    if (A.clog2 != kDefaultEllChunkLog2 || A.g.N * K > (1 << 22)) return false;
    auto &known = plans_of(A).possible;
    const unsigned key = (unsigned)K << 4 | (unsigned)p;
    const auto it = known.find(key);
    return it != known.end() ? it->second : known.emplace(key, fits_lds(A, K, p)).first->second;
}

static int most_threads(Prec p) { return p == P64 ? sweep_threads<double>() : sweep_threads<float>(); }
static int lanes_per_row(int K) { return K / (K == 8 ? kSweepR<8> : K == 4 ? kSweepR<4> : K == 2 ? kSweepR<2> : 1); }

// The work of a half-sweep of `kind` in tiles: choose_tile's cost, on average
// over the launches that a V-cycle makes on a level, or a sweep by itself.
static double sweep_cost(const Matrix &A, int K, Prec p, int kind, bool cycle)
{
    auto cost = [&](bool forward, bool zero, bool skip_first, int tail) {
        SweepArgs one{};
        sweep_args(one, A.g, nullptr, 1, 1, forward, zero, skip_first, tail);
        return (double)choose_tile(A.g, one, K, lanes_per_row(K), most_threads(p), vec_bytes(p)).cost;
    };
    if (kind == HPGMX_GS_SYMMETRIC) {
        const double sweep = cost(true, false, false, 0) + cost(false, false, true, 0);
        return cycle ? (cost(true, true, false, 0) + cost(false, false, true, 2) + sweep) / 4.0 : sweep / 2.0;
    }
    const bool forward = kind == HPGMX_GS_FORWARD;
    const double sweep = cost(forward, false, false, 0);
    return cycle ? (cost(forward, true, false, 1) + sweep) / 2.0 : sweep;
}

// Small levels gain the launches' latency in tiles; larger ones still gain,
// because a tile's matrix entries are its values alone and its neighbours
// come from LDS, until the halo rows cost more.  How many halo rows a tile
// has depends on the x-lines: it keeps them whole, so long lines leave room
// for few cells in y and z.  So the line is drawn by the work of the tiles
// (sweep_cost) against what the colour launches cost, a part for the launches
// and a part per row.  30-step solves with two levels, level 0 in tiles
// against colour launches, with the cost in brackets (forward sweeps unless
// named):
//   FP32            256x128x120 -6 % (252)      360x100x100 +4 % (336)
//                   440x96x96 +22 % (588)       440x40x40 backward -8 % (126)
//                   440x64x64 +5 % (252)        400x100x104 +9 % (420)
//   FP64            112^3 -5 % (180)            160x96x96 +1 % (222)
//                   200x60x60 -9 % (156), symmetric +2 % (168)
//                   220x80x88 +32 % (462)
//   binary16        256x128x120 -7 % (252)      320x112x112 +2 % (336)
//   bfloat16 hier.  512x100x80 -3 % (258)       640x80x80 +3 % (324)
//                   600x60x60 -8 % (162)        900x16x16 +8 % (126)
//   batches, FP32   4 x 100x64x64 -8 % (108), symmetric +6 % (117)
//                   8 x 48^3 -11 % (90)         2 x 220x48x48 +13 % (150)
//   batches, FP64   2 x 80^3 -8 % (132)         8 x 24x64x64 symmetric +1 % (117)
// A sweep by itself has no restriction, and no SpMV after it that the colour
// launches take a part of; but for FP64 and batches tiles pay further then:
// FP32 440x96x96 -2 % (420), 420x140x70 -13 % (384); bfloat16 hierarchy
// 640x80x80 -23 % (312), 900x16x16 +6 % (108); FP64 149x101x83 -15 % (192),
// 200x88x88 +4 % (252); batches FP32 4 x 110x48x48 +9 % (120).
// The most rows (times right-hand sides) come from cubes: FP32 160^3 19852 us
// in colour launches and 18595 in tiles (4 levels); FP64 112^3 14003 and
// 13589, but 128^3 17882 and 18273; batches FP32 2 x 96^3 8957 and 7434, but
// 4 x 96^3 12312 and 14287; FP64 2 x 80^3 9388 and 8639, but 2 x 96^3 13636
// and 13944.
bool sweep_pays(const Matrix &A, int K, Prec p, int kind, bool cycle)
{
    const i64 rows = A.g.N * K, most = K == 1 ? (p == P64 ? 3 << 19 : 1 << 22) : (p == P64 ? 9 << 17 : 7 << 18);
    if (rows > most || !sweep_possible(A, K, p)) return false;
    auto &known = plans_of(A).pays;
    const unsigned key = (unsigned)K << 6 | (unsigned)p << 3 | (unsigned)kind << 1 | (unsigned)cycle;
    const auto it = known.find(key);
    if (it != known.end()) return it->second;
    // what eight colour launches cost: for the launches, and per 10^6 rows
    double launches, per_row;
    if (K > 1) launches = p == P64 ? 65.0 : 80.0, per_row = p == P64 ? 66.0 : 20.0;
    else if (p == P64) launches = 122.0, per_row = 58.0;
    else if (mg16(p)) launches = 75.0, per_row = cycle ? 54.0 : 60.0;
    else launches = 120.0, per_row = cycle ? 53.0 : 75.0;
    const bool pays = sweep_cost(A, K, p, kind, cycle) <= launches + per_row * 1e-6 * (double)rows;
    return known.emplace(key, pays).first->second;
}

static SweepPlan make_plan(const Matrix &A, Prec p, int K, const Geom *gc, bool forward, bool zero, bool skip_first,
                           int tail)
{
    const Geom &g = A.g;
    SweepPlan o;
    SweepArgs one{};
    sweep_args(one, g, gc, 1, 1, forward, zero, skip_first, tail);
    const int most = most_threads(p), L = lanes_per_row(K);
    const Tile t = choose_tile(g, one, K, L, most, vec_bytes(p));
    if (t.lds == 0) throw std::runtime_error("launch_sweep: no tile fits the LDS");
    const int n = t.n, m = t.m;
    o.lds = t.lds;
    sweep_args(o.P, g, gc, n, m, forward, zero, skip_first, tail);
    o.P.remap = tile_remap(A);
    o.P.bytes = (unsigned)(ell_entries(g.N, A.clog2) * (i64)(p == P64 ? 8 : p == P32 ? 4 : 2));
    i64 lanes = 64;
    for (int q = o.P.first; q < 8; ++q) lanes = std::max(lanes, sweep_lanes(one, q, n, m, L));
    o.split = lanes <= most / 2;  // both halves of the waves fit
    o.threads = (int)std::min<i64>(most, (lanes + 63) / 64 * 64 * (o.split ? 2 : 1));
    o.tiles = sweep_tiles(g, n, m);
    return o;
}

// gc is the level below A in every call, so it is no part of the key.
void launch_sweep(const Matrix &A, Prec p, int K, bool forward, bool skip_first, const void *r, const void *zin,
                  const Geom *gc, const void *zc, void *zout, void *rc, hipStream_t s)
{
    if (!sweep_possible(A, K, p)) throw std::runtime_error("launch_sweep: level too large");
    const bool zero = zin == nullptr;
    const int tail = !rc ? 0 : zero ? 1 : 2;
    const unsigned key = (unsigned)K << 9 | (unsigned)p << 5 | (unsigned)tail << 3 | (unsigned)forward << 2 |
                         (unsigned)zero << 1 | (unsigned)skip_first;
    auto &plans = plans_of(A).form;
    auto it = plans.find(key);
    if (it == plans.end()) it = plans.emplace(key, make_plan(A, p, K, gc, forward, zero, skip_first, tail)).first;
    const SweepArgs &P = it->second.P;
    const int tiles = it->second.tiles, threads = it->second.threads;
    const bool split = it->second.split;
    const size_t lds = it->second.lds;
    auto go2 = [&](auto kc, auto *v, auto *d, auto sv) {
        using V = std::remove_const_t<std::remove_pointer_t<decltype(v)>>;
        using S = decltype(sv);
        constexpr int KK = decltype(kc)::value;
        if (split) sweep_launch<V, S, KK, true>(v, d, P, tiles, threads, lds, r, zin, zc, zout, rc, s);
        else sweep_launch<V, S, KK, false>(v, d, P, tiles, threads, lds, r, zin, zc, zout, rc, s);
    };
    auto go = [&](auto *v, auto *d, auto sv) {
        using S = decltype(sv);
        if (K == 1) go2(std::integral_constant<int, 1>{}, v, d, S{});
        else if constexpr (!std::is_same<S, __half>::value && !std::is_same<S, bf16>::value) {
            if (K == 2) go2(std::integral_constant<int, 2>{}, v, d, S{});
            else if (K == 4) go2(std::integral_constant<int, 4>{}, v, d, S{});
            else if (K == 8) go2(std::integral_constant<int, 8>{}, v, d, S{});
            else throw std::runtime_error("launch_sweep: unsupported batch width");
        } else throw std::runtime_error("launch_sweep: no batches of the 16-bit hierarchy");
    };
    switch (p) {
    case P64: go(A.v64, A.d64, double{}); break;
    case P32: go(A.v32, A.d32, float{}); break;
    case P16: go(A.v16, A.d16, float{}); break;
    case PB16: go(A.vb16, A.db16, float{}); break;
    case P16V: go(A.v16, A.d16, __half{}); break;
    case PB16V: go(A.vb16, A.db16, bf16{}); break;
    }
    HPGMX_LAUNCH_CHECK();
}

}  // namespace hpgmx
