// Many sweeps of a small level in one launch.
// Included by hnv_kernels.hip only (after its slices and row updates).
#pragma once

namespace hnv {

// A sweep is linear in every column: column c of the new rows depends on
// column c of the old ones alone.  So a workgroup that holds one 4-byte word
// (a column in FP32, two in BF16) of every row of a level in LDS can run any
// number of sweeps without another workgroup: a workgroup per word of a row,
// one launch, and a barrier of the workgroup where the general path has the end
// of a launch.  Levels whose words, neighbour lists (16-bit) and work items fit
// in a compute unit's 160 KB take it (resident_fits): such a level's general
// sweep is bound by the launch and its chain of dependent loads from L2.  Here
// the instructions of one compute unit bound it (a wavefront's takes four
// cycles), so a slice is as narrow as LDS accesses are (with 16
// bytes of a row, a quarter of the workgroups, launches of ten sweeps took twice
// as long: 94 us instead of 47 at the time), lists start at multiples of four, four
// neighbours to an access, and residuals are left to another kernel.
//
// Every row is summed as k_gather sums it, so both give the same bits.  A
// wavefront-tier row, of which k_gather's four wavefronts take a quarter each,
// Q = 64 / G neighbours at a time, takes four lanes with Q sums each, or, when
// long, 4 Q lanes (4 Q lanes for every such row: 47 us where this takes 31).  For
// the residuals every sweep leaves its rows' words in memory, in item order, and
// k_resident_blocks forms the per-block partials of a general sweep from them.
//
// Measured, FP32, d = 32, 2,000 nodes / 1,000 hyperedges and three coarser
// levels, 10 sweeps each with residuals: 225 -> 152 us.  A sweep of the finest level takes 2.0
// us where a launch each takes 4.5, after about 8 us of loads; random LDS words
// (bank conflicts) are most of it.
constexpr int kResidentThreads = 1024;

struct ResidentArgs {
    DevSide side[2];
    int32_t n_nodes, n_edges;
    int32_t sweeps;
    int32_t edge_first, fused;
    int32_t off_e[2], off_idx[2], off_wn, off_items, off_mix, off_wide;   // LDS offsets past the node rows (bytes)
    int64_t ld;
    float omega;
    const float *r;
    const int32_t *rowmap;
    const void *src;
    void *dst;
    uint32_t *trace;          // [sweeps + 1][words][rows] the rows' words before and after each sweep, or null
};

// One word of a row: its columns as floats and back (as Slice has them).
template <typename T>
struct Word;
template <>
struct Word<float> {
    static constexpr int N = 1;
    static HNV_DEV void unpack(uint32_t w, float (&v)[1]) { v[0] = __uint_as_float(w); }
    static HNV_DEV uint32_t pack(const float (&v)[1]) { return __float_as_uint(v[0]); }
};
template <>
struct Word<bf16_t> {
    static constexpr int N = 2;
    static HNV_DEV void unpack(uint32_t w, float (&v)[2])
    {
        v[0] = bf_lo(w);
        v[1] = bf_hi(w);
    }
    static HNV_DEV uint32_t pack(const float (&v)[2]) { return to_bf16(v[0]) | (to_bf16(v[1]) << 16); }
};

template <typename T, bool SCALE>
HNV_DEV void add_word(float (&acc)[Word<T>::N], float s, uint32_t w)
{
    float v[Word<T>::N];
    Word<T>::unpack(w, v);
#pragma unroll
    for (int i = 0; i < Word<T>::N; ++i)
        acc[i] = SCALE ? fmaf(s, v[i], acc[i]) : acc[i] + v[i];
}

// Where a side-local row's list starts in LDS: a multiple of 4 entries, apart
// from the next row's by at least its length rounded up to 4.
HNV_DEV int list_start(int start, int row) { return (start + 3 * row) & ~3; }

HNV_DEV uint32_t word_at(const unsigned char *rows, uint32_t off) { return *reinterpret_cast<const uint32_t *>(rows + off); }

// A list of `len` neighbours added in order (lists are byte offsets of rows).
template <typename T, bool SCALE>
HNV_DEV void add_list(const unsigned char *rows, const uint16_t *list, const float *wn, int len, float (&acc)[Word<T>::N])
{
    for (int j = 0; j < len; j += 8) {
        const bool more = len - j > 4;
        uint32_t x[8];
        float4 s[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            if (h == 0 || more) {
                const uint2 o = *reinterpret_cast<const uint2 *>(list + j + 4 * h);
                if (SCALE)
                    s[h] = *reinterpret_cast<const float4 *>(wn + j + 4 * h);
                x[4 * h] = word_at(rows, o.x & 0xffffu);
                x[4 * h + 1] = word_at(rows, o.x >> 16);
                x[4 * h + 2] = word_at(rows, o.y & 0xffffu);
                x[4 * h + 3] = word_at(rows, o.y >> 16);
            }
        }
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            if (h == 1 && !more)
                break;
            const int n = len - j - 4 * h;
            add_word<T, SCALE>(acc, s[h].x, x[4 * h]);
            if (n > 1)
                add_word<T, SCALE>(acc, s[h].y, x[4 * h + 1]);
            if (n > 2)
                add_word<T, SCALE>(acc, s[h].z, x[4 * h + 2]);
            if (n > 3)
                add_word<T, SCALE>(acc, s[h].w, x[4 * h + 3]);
        }
    }
}

// The neighbours first, first + step, .. below len of a list, in order.
template <typename T, bool SCALE>
HNV_DEV void add_strided(const unsigned char *rows, const uint16_t *list, const float *wn, int first, int step, int len,
                         float (&acc)[Word<T>::N])
{
    for (int j = first; j < len; j += kUnroll * step) {
        uint32_t x[kUnroll];
        float s[kUnroll];
#pragma unroll
        for (int k = 0; k < kUnroll; ++k) {
            const int q = j + k * step < len ? j + k * step : j;
            s[k] = SCALE ? wn[q] : 1.0f;
            x[k] = word_at(rows, list[q]);
        }
#pragma unroll
        for (int k = 0; k < kUnroll; ++k)
            if (j + k * step < len)
                add_word<T, SCALE>(acc, s[k], x[k]);
    }
}

// What Q lanes' add_strided sums (first = 0 .. Q-1, step Q) and a butterfly over
// them come to, by one lane.
template <typename T, int Q, bool SCALE>
HNV_DEV void add_interleaved(const unsigned char *rows, const uint16_t *list, const float *wn, int len,
                             float (&acc)[Word<T>::N])
{
    constexpr int N = Word<T>::N;
    float v[Q][N];
#pragma unroll
    for (int q = 0; q < Q; ++q)
        zero(v[q]);
    for (int j = 0; j < len; j += Q) {
        uint32_t x[Q];
        float s[Q];
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const int at = j + q < len ? j + q : j;
            s[q] = SCALE ? wn[at] : 1.0f;
            x[q] = word_at(rows, list[at]);
        }
#pragma unroll
        for (int q = 0; q < Q; ++q)
            if (j + q < len)
                add_word<T, SCALE>(v[q], s[q], x[q]);
    }
#pragma unroll
    for (int off = 1; off < Q; off <<= 1)
#pragma unroll
        for (int q = 0; q < Q; q += 2 * off)
#pragma unroll
            for (int i = 0; i < N; ++i)
                v[q][i] += v[q + off][i];
#pragma unroll
    for (int i = 0; i < N; ++i)
        acc[i] = v[0][i];
}

// The value of lane L of the lane's four.
template <int L>
HNV_DEV float of_quad(float x)
{
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), 0x55 * L, 0xf, 0xf, true));
}

// Wavefront-tier rows longer than this take 4 Q lanes, others four: a lane of
// four has a chain of a quarter of the row.
constexpr int kWideRow = 256;

// A work item in LDS: its row (byte offset), where its list starts, its length.
using ResidentItem = ushort4;

// One side's rows of one sweep.  Rows (the neighbours', the side's old and new
// ones, which may be the same), lists and items are in LDS; `trace`: where the
// items' new words go in memory, or null.
template <typename T, int G, bool SCALE>
HNV_DEV void resident_side(const unsigned char *nb_rows, const unsigned char *own_rows, unsigned char *new_rows,
                           const uint16_t *idx, const float *wn, const ResidentItem *items, const float *mix,
                           int n_chunks, int n_wide, int n_small, float keep, uint32_t *__restrict__ trace)
{
    using W = Word<T>;
    constexpr int Q = kWave / G;
    const int lane = threadIdx.x % kWave;
    auto pad = [](int lanes) { return (lanes + kWave - 1) & ~(kWave - 1); };
    const int end_wide = pad(n_wide * 4 * Q);
    const int end_chunk = end_wide + pad((n_chunks - n_wide) * 4);
    const int end_small = end_chunk + pad(n_small);
    // (a wavefront's 64 lanes lie in one range)
    for (int t = threadIdx.x; t < end_small; t += kResidentThreads) {
        float acc[W::N];
        zero(acc);
        int item;
        bool writer;   // whether the lane finishes the item's row
        ResidentItem it = make_ushort4(0, 0, 0, 0);
        uint32_t own = 0;   // (own and m are read ahead of the neighbours)
        float m = 0.0f;
        if (t >= end_chunk) {
            item = n_chunks + (t - end_chunk);
            writer = item < n_chunks + n_small;
            if (writer) {
                it = items[item];
                own = word_at(own_rows, it.x);
                m = mix[item];
                add_list<T, SCALE>(nb_rows, idx + it.y, wn + it.y, it.z, acc);
            }
        } else {
            const bool wide = t < end_wide;
            const int lanes = wide ? 4 * Q : 4, u = wide ? t : t - end_wide;
            item = wide ? u / (4 * Q) : n_wide + u / 4;
            const bool valid = item < (wide ? n_wide : n_chunks);
            if (valid) {
                it = items[item];
                own = word_at(own_rows, it.x);
                m = mix[item];
            }
            const int per = (it.z + 3) / 4, w = (wide ? u / Q : u) % 4;   // the quarter w
            const int start = it.y + w * per, len = max(0, min(per, (int)it.z - w * per));
            if (wide) {
                add_strided<T, SCALE>(nb_rows, idx + start, wn + start, u % Q, Q, len, acc);
#pragma unroll
                for (int off = 1; off < Q; off <<= 1)
#pragma unroll
                    for (int i = 0; i < W::N; ++i)
                        acc[i] += __shfl_xor(acc[i], off, kWave);
                const int base = lane & ~(4 * Q - 1);
#pragma unroll
                for (int i = 0; i < W::N; ++i) {
                    float sum = __shfl(acc[i], base, kWave);
                    for (int w1 = 1; w1 < 4; ++w1)
                        sum += __shfl(acc[i], base + w1 * Q, kWave);
                    acc[i] = sum;
                }
            } else {
                add_interleaved<T, Q, SCALE>(nb_rows, idx + start, wn + start, len, acc);
#pragma unroll
                for (int i = 0; i < W::N; ++i)
                    acc[i] = ((of_quad<0>(acc[i]) + of_quad<1>(acc[i])) + of_quad<2>(acc[i])) + of_quad<3>(acc[i]);
            }
            writer = valid && u % lanes == 0;
        }
        if (writer) {
            uint32_t w = own;
            if (it.z > 0) {
                float z[W::N], o[W::N];
                W::unpack(w, z);
#pragma unroll
                for (int i = 0; i < W::N; ++i)
                    o[i] = fmaf(m, acc[i], keep * z[i]);
                w = W::pack(o);
            }
            *reinterpret_cast<uint32_t *>(new_rows + it.x) = w;
            if (trace)
                trace[item] = w;
        }
    }
}

template <typename T, int G>
__global__ __launch_bounds__(kResidentThreads) void k_resident(ResidentArgs a)
{
    static_assert(kWavesPerBlock == 4 && 4 * (kWave / G) <= kWave, "a row's quarters, in one wavefront");
    __shared__ __align__(16) unsigned char lds[kResidentLds];
    const uint32_t *src = static_cast<const uint32_t *>(a.src) + blockIdx.x;   // this workgroup's word of row 0
    uint32_t *dst = static_cast<uint32_t *>(a.dst) + blockIdx.x;
    const int64_t ld = a.ld / Word<T>::N;   // words per row
    const int nV = a.n_nodes, nE = a.n_edges, rows = nV + nE, tid = threadIdx.x;
    unsigned char *e_old = lds + a.off_e[0], *e_new = lds + a.off_e[1];
    uint16_t *idx0 = reinterpret_cast<uint16_t *>(lds + a.off_idx[0]);
    uint16_t *idx1 = reinterpret_cast<uint16_t *>(lds + a.off_idx[1]);
    float *wn = reinterpret_cast<float *>(lds + a.off_wn);
    ResidentItem *items = reinterpret_cast<ResidentItem *>(lds + a.off_items);
    float *mix = reinterpret_cast<float *>(lds + a.off_mix);
    int *n_wide = reinterpret_cast<int *>(lds + a.off_wide);   // leading items that take 4 Q lanes, per side
    if (tid < 2)
        n_wide[tid] = 0;
    __syncthreads();
    for (int u = tid; u < rows; u += kResidentThreads) {
        const uint32_t x = src[(a.fused ? a.rowmap[u] : u) * ld];
        *reinterpret_cast<uint32_t *>(u < nV ? lds + 4 * u : e_old + 4 * (u - nV)) = x;
    }
    // the items and lists; a lane-group row's by a thread, four neighbours at
    // a time (the first four lie beside the item), others by a wavefront
    for (int s = 0; s < 2; ++s) {
        const DevSide &D = a.side[s];
        const int at = s == 0 ? 0 : nE, base = s == 0 ? 0 : nV;
        uint16_t *idx = s == 0 ? idx0 : idx1;
        for (int i = tid; i < D.n_chunks + D.n_small; i += kResidentThreads) {
            const Item it = i < D.n_chunks ? D.chunks[i] : D.small[i - D.n_chunks];
            const int p = list_start(it.start, it.row);
            items[at + i] = make_ushort4((unsigned short)(4 * it.row), (unsigned short)p, (unsigned short)it.len, 0);
            mix[at + i] = it.len > 0 ? a.omega * a.r[D.row_base + it.row] : 0.0f;
            if (i < D.n_chunks) {
                if (it.len > kWideRow)
                    atomicMax(&n_wide[s], i + 1);
                continue;
            }
            for (int j = 0; j < it.len; j += 4) {
                int id[4];
                const InlineIds first = j == 0 ? D.small_ids[i - D.n_chunks] : InlineIds{};
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    id[k] = j + k >= it.len ? base : j == 0 ? first.id[k] : D.idx[it.start + j + k];
                    if (D.wn && j + k < it.len)
                        wn[p + j + k] = D.wn[it.start + j + k];
                }
                uint2 o;
                o.x = (uint32_t)(4 * (id[0] - base)) | ((uint32_t)(4 * (id[1] - base)) << 16);
                o.y = (uint32_t)(4 * (id[2] - base)) | ((uint32_t)(4 * (id[3] - base)) << 16);
                *reinterpret_cast<uint2 *>(idx + p + j) = o;
            }
        }
        for (int i = tid / kWave; i < D.n_chunks; i += kResidentThreads / kWave) {
            const Item it = D.chunks[i];
            const int p = list_start(it.start, it.row);
            for (int j = tid % kWave; j < it.len; j += kWave) {
                idx[p + j] = (uint16_t)(4 * (D.idx[it.start + j] - base));
                if (D.wn)
                    wn[p + j] = D.wn[it.start + j];
            }
        }
    }
    __syncthreads();
    const int64_t per_sweep = (int64_t)gridDim.x * rows;
    uint32_t *trace = a.trace ? a.trace + (int64_t)blockIdx.x * rows : nullptr;
    if (trace) {
        for (int i = tid; i < rows; i += kResidentThreads)
            trace[i] = word_at(i < nE ? e_old : lds, items[i].x);
        trace += per_sweep;
    }
    const float keep = 1.0f - a.omega;
    const int wide0 = __builtin_amdgcn_readfirstlane(n_wide[0]), wide1 = __builtin_amdgcn_readfirstlane(n_wide[1]);
    for (int k = 0; k < a.sweeps; ++k) {
        resident_side<T, G, false>(lds, e_old, e_new, idx0, wn, items, mix, a.side[0].n_chunks, wide0,
                                   a.side[0].n_small, keep, trace);
        __syncthreads();
        const unsigned char *e = a.edge_first ? e_new : e_old;   // the hyperedge rows that the node rows read
        uint32_t *trace1 = trace ? trace + nE : nullptr;
        if (a.side[1].wn)
            resident_side<T, G, true>(e, lds, lds, idx1, wn, items + nE, mix + nE, a.side[1].n_chunks, wide1,
                                      a.side[1].n_small, keep, trace1);
        else
            resident_side<T, G, false>(e, lds, lds, idx1, wn, items + nE, mix + nE, a.side[1].n_chunks, wide1,
                                       a.side[1].n_small, keep, trace1);
        __syncthreads();
        unsigned char *t = e_old;
        e_old = e_new;
        e_new = t;
        if (trace)
            trace += per_sweep;
    }
    for (int u = tid; u < rows; u += kResidentThreads)
        dst[u * ld] = word_at(u < nV ? lds : e_old, 4 * (u < nV ? u : u - nV));
}

// The blocks of a general sweep of one column panel in launch order: per
// segment its blocks, its first item in the trace, its items, and whether they
// are the lane-group tier's (else a block has one item: see resident_fits).
struct ResidentSegments {
    int32_t blocks[4], first[4], items[4], small[4];
};

// The residual partial of each block (blockIdx.x) of each sweep (blockIdx.y)
// from the rows' words before and after it: every lane forms what it would in
// k_gather, and the block adds them in the same order.
template <typename T, int EPL, int G>
__global__ __launch_bounds__(kBlock) void k_resident_blocks(const uint32_t *__restrict__ trace, int rows, int words,
                                                            int dp, ResidentSegments sg, double *__restrict__ part,
                                                            int64_t part_stride)
{
    constexpr int Q = kWave / G, NW = EPL / Word<T>::N;
    int b = blockIdx.x, s = 0;
    while (b >= sg.blocks[s])
        b -= sg.blocks[s++];
    const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave, g = lane / G, gl = lane % G;
    const int item = sg.small[s] ? b * (kBlock / G) + wave * Q + g : b;
    const bool has = item < sg.items[s] && (sg.small[s] || (g == 0 && wave == 0));
    double r2 = 0.0;
    if (has && gl * EPL < dp) {
        const uint32_t *before = trace + ((int64_t)blockIdx.y * words + gl * NW) * rows + sg.first[s] + item;
        const uint32_t *after = before + (int64_t)words * rows;
#pragma unroll
        for (int k = 0; k < NW; ++k) {
            float z[Word<T>::N], o[Word<T>::N];
            Word<T>::unpack(before[(int64_t)k * rows], z);
            Word<T>::unpack(after[(int64_t)k * rows], o);
#pragma unroll
            for (int i = 0; i < Word<T>::N; ++i) {
                const double dd = (double)o[i] - (double)z[i];
                r2 = fma(dd, dd, r2);
            }
        }
    }
    const double sum = block_wave_sums(r2);
    if (threadIdx.x == 0)
        part[(int64_t)blockIdx.y * part_stride + blockIdx.x] = sum;
}

}  // namespace hnv
