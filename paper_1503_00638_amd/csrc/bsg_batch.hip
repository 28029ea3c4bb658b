// Batched compression / decompression of many independent chunks (each its
// own stream of the format in bsg.h) in a handful of launches: one
// persistent kernel per class of chunks walks every block of every chunk of
// that class (chunks are independent units, like the blocks inside them,
// Section 4.2 of Masui et al.), then a scan of the block sizes and one pack
// pass (payload, offsets, header, capacity verdict, raw tail).  Common element
// sizes of few blocks share a class: a launch per element size ran one after
// the other, 220 us instead of 89 to compress 16 chunks of up to 1 MiB and 112
// instead of 41 to decompress them.  An element size with many blocks, or with
// no other to share with, has a class and a decoder of its own (kOwnMinBlocks).
// Nothing is allocated and nothing is synchronised with the host, so the whole
// sequence can be captured into a hipGraph.
#include <algorithm>
#include <cstring>
#include <map>
#include <numeric>
#include <vector>

#include "bsg_lz4_dev.hpp"

namespace bsg {

namespace {

constexpr int kMaxClasses = kSideEvents; // (one encode event per class)
// a batch of at least this many blocks splits its classes over two streams
constexpr int64_t kBatchSideMinBlocks = 16384;
// In a batch of that many blocks and kPartMinBatch bytes a class ends when it
// holds kPartMinBlocks and an eighth of the batch and leaves a quarter of that
// for the next one, so that its scan and pack run beside the next one's encode.
// (A class more costs 5 launches and a last round that does not fill the card:
// 10,000 blocks of 8 KiB, 4-byte elements, in two classes 142 us, in one 109;
// 20,000 of 2 KiB 120 and 81.)
constexpr int kMaxParts = 8;
constexpr int64_t kPartMinBlocks = 8192;
constexpr int64_t kPartMinBatch = 128ll << 20;
// Elements of 1, 2, 4, 8 bytes and those without a register path ("keys" of one
// instance block size) share a class where two keys or more have few blocks.  A
// key of at least kOwnMinBlocks and a single one are classes of their own, which
// their own decoders take: in 8 KiB blocks the mixed decoder's 128 registers
// leave 16 workgroups per CU, where those for 1, 2 and 4 bytes (91) and for no
// register path (58) have the 18 that LDS allows and the one for 8 takes 109.
// With several keys of few blocks the end of one more launch costs more than
// that gives.
// 37 GiB in 4096 chunks of 2, 4 and 8 bytes (1.5 M blocks and more each):
// decompress 33.6 ms, 34.7 as one mixed class.  0.78 GB in 256 chunks (about
// 32,000 blocks each): 659 us mixed, 707 in classes of their own; 8000 blocks,
// one sixteenth of them of another size: 45 mixed, 56.  100,000 blocks of 4 KiB
// and 3-byte elements alone: 494 us mixed, 424 in their own class.
constexpr int64_t kOwnMinBlocks = 65536;
constexpr int kKeysPerSize = 8; // mixed, no register path, 1, 2, 4, 8, 12, 16
// (a mixed class stands for two keys or more)
static_assert(kMaxClasses >= (kKeysPerSize - 1) * 4 + kMaxParts, "classes of a batch");

struct BatchHeader {
    int32_t count, n_classes;
    int64_t total_blocks, slot_total;
};

// Consecutive chunks (in table order) whose blocks one launch takes: same
// element class (kKeyClass) and instance block size.
struct BatchClass {
    int32_t ec, maxb, first_chunk, n_chunks;
    int64_t first_block, n_blocks;
};

struct BatchChunk {
    const uint8_t *in;
    uint8_t *out;
    int64_t n, in_nbytes, out_capacity;
    int64_t nb, n_full, last, tail, n_blocks;
    int64_t block_start; // global index of the chunk's first block
    int64_t slot_start;  // byte offset of its first slot in the slot area
    int64_t slot_bytes;
    int32_t E, orig;     // element size, index in the caller's array
};

// Element class of a key; place of an element class in it.
constexpr int kKeyClass[kKeysPerSize] = {kMixed, 0, 1, 2, 4, 8, 12, 16};

int key_of(int ec)
{
    int i = 1;
    while (kKeyClass[i] != ec) ++i;
    return i;
}

constexpr int64_t table_bytes(int64_t count)
{
    return (int64_t)sizeof(BatchHeader) + kMaxClasses * (int64_t)sizeof(BatchClass) +
           count * (int64_t)sizeof(BatchChunk);
}

struct TableView {
    const BatchHeader *h;
    const BatchClass *cls;
    const BatchChunk *ch;
    __host__ __device__ explicit TableView(const void *t)
        : h(reinterpret_cast<const BatchHeader *>(t)),
          cls(reinterpret_cast<const BatchClass *>(reinterpret_cast<const uint8_t *>(t) +
                                                    sizeof(BatchHeader))),
          ch(reinterpret_cast<const BatchChunk *>(reinterpret_cast<const uint8_t *>(t) +
                                                  sizeof(BatchHeader) +
                                                  kMaxClasses * sizeof(BatchClass)))
    {
    }
};

// The chunk (in table order, within [lo, hi]) that owns global block g: the
// last one whose first block is <= g.  A chunk without blocks shares its
// first-block index with the chunk after it, which the search prefers, so it
// is never chosen.
__device__ __forceinline__ int find_chunk(const BatchChunk *ch, int lo, int hi, int64_t g)
{
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (ch[mid].block_start <= g)
            lo = mid;
        else
            hi = mid - 1;
    }
    return lo;
}

// The blocks of a class that one workgroup of a persistent launch takes, in
// increasing order: every gridDim.x-th block from blockIdx.x
// (BSG_SCHED_STRIDED), or one contiguous range of ceil(n / gridDim.x) blocks
// (BSG_SCHED_RANGES).  Either way every block is taken by exactly one
// workgroup, so the output does not depend on the schedule.
struct BlockWalk {
    int64_t first, end, step;
    __device__ BlockWalk(const BatchClass &C, int schedule)
    {
        const int64_t n = C.n_blocks;
        if (schedule == BSG_SCHED_RANGES) {
            const int64_t per = (n + gridDim.x - 1) / gridDim.x;
            const int64_t lo = (int64_t)blockIdx.x * per < n ? (int64_t)blockIdx.x * per : n;
            first = C.first_block + lo;
            end = C.first_block + (lo + per < n ? lo + per : n);
            step = 1;
        } else {
            first = C.first_block + blockIdx.x;
            end = C.first_block + n;
            step = gridDim.x;
        }
    }
};

// The chunk owning block g, given the chunk c of an earlier block of the
// same walk (blocks only grow): under the range schedule the walk steps
// through the table, one read per block; under the strided one it searches
// the rest of the table.
__device__ __forceinline__ int next_chunk(const BatchChunk *ch, int c, int last, int64_t g,
                                          int64_t step)
{
    if (step == 1) {
        while (c < last && ch[c + 1].block_start <= g) ++c;
        return c;
    }
    return find_chunk(ch, c, last, g);
}

template <int MAXB, int EC>
__global__ __launch_bounds__(64) void k_batch_encode(const uint8_t *__restrict__ table, BatchClass C,
                                                     uint8_t *__restrict__ slots,
                                                     int32_t *__restrict__ sizes, int schedule)
{
    __shared__ EncLds<MAXB> L;
    const TableView T(table);
    const RoundParams none{};
    const BlockWalk W(C, schedule);
    const int last = C.first_chunk + C.n_chunks - 1;
    int c = W.first < W.end ? find_chunk(T.ch, C.first_chunk, last, W.first) : C.first_chunk;
    for (int64_t g = W.first; g < W.end; g += W.step) {
        c = next_chunk(T.ch, c, last, g, W.step);
        const BatchChunk &ch = T.ch[c];
        const int64_t local = g - ch.block_start;
        const int64_t elems = local < ch.n_full ? ch.nb : ch.last;
        const int sz = encode_one<MAXB, EC, kRoundNone>(ch.in + local * ch.nb * ch.E, elems, ch.E, none, 0,
                                                   slots + ch.slot_start + local * ch.slot_bytes, L);
        if (threadIdx.x == 0) sizes[g] = sz;
    }
}

// As dec_waves_per_eu, but 4 for 4 KiB blocks of 8-byte elements, whose
// registers beside the block walk's do not fit 5 without spills, and 3 for
// 16-byte elements (one register more, 169, leaves 2: 100,000 blocks 766 us, 975).
template <int MAXB, int EC> constexpr int bdec_waves_per_eu()
{
    constexpr int n = dec_waves_per_eu<MAXB, EC>();
    return EC == 16 && MAXB <= kSmallBlock ? 3 : EC == 8 && n > 4 ? 4 : n;
}

template <int MAXB, int EC>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(bdec_waves_per_eu<MAXB, EC>()))) void k_batch_decode(const uint8_t *__restrict__ table, BatchClass C,
                                                     int32_t *__restrict__ status, int schedule)
{
    __shared__ DecLds<MAXB> L;
    const TableView T(table);
    const BlockWalk W(C, schedule);
    const int last = C.first_chunk + C.n_chunks - 1;
    int c = W.first < W.end ? find_chunk(T.ch, C.first_chunk, last, W.first) : C.first_chunk;
    for (int64_t g = W.first; g < W.end; g += W.step) {
        c = next_chunk(T.ch, c, last, g, W.step);
        const BatchChunk &ch = T.ch[c];
        const int64_t local = g - ch.block_start;
        const int64_t elems = local < ch.n_full ? ch.nb : ch.last;
        const int64_t table_end = kHeaderBytes + 8 * (ch.n_blocks + 1);
        const int64_t payload_len = ch.in_nbytes - table_end - ch.tail * ch.E;
        bool ok = payload_len >= 0;
        if (ok) {
            uint8_t *dst = ch.out + local * ch.nb * ch.E;
            ok = decode_one<MAXB, EC>(ch.in + table_end, payload_len,
                                      reinterpret_cast<const uint64_t *>(ch.in + kHeaderBytes),
                                      local, elems, ch.E, ch.in + ch.in_nbytes, dst,
                                      ((uintptr_t)ch.out % 16) == 0, L);
        }
        if (!ok && threadIdx.x == 0) atomicCAS(&status[ch.orig], 0, BSG_ECORRUPT);
    }
}

// One wavefront per chunk: header check and raw tail of each stream.
__global__ __launch_bounds__(64) void k_batch_dec_tail(const uint8_t *__restrict__ table,
                                                       int32_t *__restrict__ status)
{
    const TableView T(table);
    const BatchChunk &ch = T.ch[blockIdx.x];
    const int64_t table_end = kHeaderBytes + 8 * (ch.n_blocks + 1);
    const int64_t tail_bytes = ch.tail * ch.E;
    const int64_t payload_len = ch.in_nbytes - table_end - tail_bytes;
    if (payload_len < 0 || !header_ok(ch.in, payload_len, ch.n, ch.E, ch.nb, ch.n_blocks)) {
        if (threadIdx.x == 0) atomicCAS(&status[ch.orig], 0, BSG_ECORRUPT);
        return;
    }
    uint8_t *dst = ch.out + (ch.n - ch.tail) * ch.E;
    for (int64_t i = threadIdx.x; i < tail_bytes; i += kWave) dst[i] = ch.in[table_end + payload_len + i];
}

// ---- prefix of the block sizes, one class at a time ------------------------
// prefix[g] = bytes of the batch's blocks before g.  One wavefront per
// 1024-block tile of a class and no LDS: the encoders beside these kernels
// hold all of it (see the single-stream scan).  Tile k holds blocks b0 +
// k kTile ..; lane l its blocks 64 i + l.
__device__ __forceinline__ void load_btile(const int32_t *__restrict__ sizes, int64_t b0, int64_t n,
                                           int64_t tile, int lane, int (&v)[kTile / kWave])
{
#pragma unroll
    for (int i = 0; i < kTile / kWave; ++i) {
        const int64_t k = tile * kTile + i * kWave + lane;
        v[i] = k < n ? sizes[b0 + k] : 0;
    }
}

__global__ __launch_bounds__(64) void k_btile_sum(const int32_t *__restrict__ sizes, int64_t b0,
                                                  int64_t n, int64_t *__restrict__ tile_sum)
{
    int v[kTile / kWave], sum = 0, total;
    load_btile(sizes, b0, n, blockIdx.x, threadIdx.x, v);
#pragma unroll
    for (int i = 0; i < kTile / kWave; ++i) sum += v[i];
    wave_excl_scan(sum, total); // a tile's bytes stay below 2^27
    if (threadIdx.x == 0) tile_sum[blockIdx.x] = total;
}

// prefix[b0 + 1 .. b0 + n], after prefix[b0] (the end of the class before;
// the first class writes it) and the sums of the class's tiles before.
__global__ __launch_bounds__(64) void k_bprefix(const int32_t *__restrict__ sizes, int64_t b0,
                                                int64_t n, int first,
                                                const int64_t *__restrict__ tile_sum,
                                                int64_t *__restrict__ prefix)
{
    const int lane = threadIdx.x;
    const int64_t tile = blockIdx.x;
    int v[kTile / kWave];
    load_btile(sizes, b0, n, tile, lane, v);
    int64_t before = 0;
#pragma unroll 4
    for (int64_t k = lane; k < tile; k += kWave) before += tile_sum[k];
    int64_t base = wave_sum_i64(before);
    if (!first)
        base += prefix[b0];
    else if (tile == 0 && lane == 0)
        prefix[b0] = 0;
#pragma unroll
    for (int i = 0; i < kTile / kWave; ++i) {
        const int64_t k = tile * kTile + i * kWave + lane;
        int total;
        const int at = wave_excl_scan(v[i], total);
        if (k < n) prefix[b0 + k + 1] = base + at + v[i];
        base += total;
    }
}

// The first `grid` workgroups take the class's blocks: a block's offset into
// its chunk's stream, and its LZ4 bytes from its slot to their place.  The
// ones after them take a chunk each: stream length and capacity verdict,
// header, end of the offset table and raw tail.  Nothing is written to a
// chunk whose stream does not fit.
__global__ __launch_bounds__(64) void k_batch_pack(const uint8_t *__restrict__ table, BatchClass C,
                                                   int64_t grid, const uint8_t *__restrict__ slots,
                                                   const int32_t *__restrict__ sizes,
                                                   const int64_t *__restrict__ prefix,
                                                   int64_t *__restrict__ d_nbytes)
{
    const TableView T(table);
    const int last = C.first_chunk + C.n_chunks - 1;
    const int lane = threadIdx.x;
    if (blockIdx.x >= grid) {
        const BatchChunk &ch = T.ch[C.first_chunk + (int)(blockIdx.x - grid)];
        const int64_t pay = prefix[ch.block_start + ch.n_blocks] - prefix[ch.block_start];
        const int64_t table_end = kHeaderBytes + 8 * (ch.n_blocks + 1);
        const int64_t tail_bytes = ch.tail * ch.E;
        const int64_t total = table_end + pay + tail_bytes;
        const bool fits = total <= ch.out_capacity;
        if (lane == 0) d_nbytes[ch.orig] = fits ? total : (int64_t)BSG_ECAPACITY;
        if (!fits) return;
        if (lane == 0) {
            bsg_header *h = reinterpret_cast<bsg_header *>(ch.out);
            h->magic = BSG_MAGIC;
            h->elem_size = (uint32_t)ch.E;
            h->n = (uint64_t)ch.n;
            h->block_elems = (uint32_t)ch.nb;
            h->n_blocks = (uint32_t)ch.n_blocks;
            reinterpret_cast<uint64_t *>(ch.out + kHeaderBytes)[ch.n_blocks] = (uint64_t)pay;
        }
        const uint8_t *tsrc = ch.in + (ch.n - ch.tail) * ch.E;
        uint8_t *tdst = ch.out + table_end + pay;
        for (int64_t i = lane; i < tail_bytes; i += kWave) tdst[i] = tsrc[i];
        return;
    }
    for (int64_t g = C.first_block + blockIdx.x; g < C.first_block + C.n_blocks; g += grid) {
        const int c = find_chunk(T.ch, C.first_chunk, last, g);
        const BatchChunk &ch = T.ch[c];
        const int64_t base = prefix[ch.block_start], at = prefix[g] - base;
        const int64_t table_end = kHeaderBytes + 8 * (ch.n_blocks + 1);
        if (table_end + (prefix[ch.block_start + ch.n_blocks] - base) + ch.tail * ch.E >
            ch.out_capacity)
            continue;
        const int64_t local = g - ch.block_start;
        if (lane == 0) reinterpret_cast<uint64_t *>(ch.out + kHeaderBytes)[local] = (uint64_t)at;
        copy_slot(ch.out + table_end + at, slots + ch.slot_start + local * ch.slot_bytes, sizes[g],
                  lane);
    }
}

int cu_count()
{
    int dev = 0, n = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 256;
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0)
        return 256;
    return n;
}

// Workgroups per CU where the caller leaves them open (more than can reside:
// each then takes a few blocks, and the hardware dispatcher balances them).
// 256 chunks, 0.78 GB: encode 1300 us at 16, 1156 at 32, 1136 at 64, 1184 at
// 128 and above; decode 797 at 16 and 32, 717 at 64, 711 from 128 on.
constexpr int kEncodeWavesPerCu = 64;
constexpr int kDecodeWavesPerCu = 256;

// The decoders' preset.  Of one element size up to about 100 blocks per CU whole
// rounds of as many workgroups as reside beat a workgroup per block, whose last
// ones start late: 8 KiB blocks of 4-byte elements 16,400 blocks 68 us at 16 per
// CU and 78 at 256, 20,000 82 and 93, 26,000 128 and 124, 100,000 484 and 436; 4
// KiB ones 32,000 71 us at 20 and 82 at 256, 45,000 109 and 112.  Blocks without
// a register path differ more in time (8 KiB: 10,000 109 and 114, 13,000 145 and
// 138; 4 KiB: 256 at every count), as do those of a mixed class (8000 of 4 and 3
// bytes 99 and 79).  The 168 registers of 16-byte elements leave 12 (100,000
// blocks 734 us at 12, 766 at 256).
int decode_waves(const BatchClass &C, int cus)
{
    const int64_t per_cu = C.n_blocks / cus;
    switch (C.maxb <= kSmallBlock ? C.ec : kMixed) {
    case 0: return C.maxb == kSmallBlock && per_cu < 48 ? 16 : kDecodeWavesPerCu;
    case 1:
    case 2:
    case 4:
        if (C.maxb == kTinyBlock) return per_cu < 144 ? 20 : kDecodeWavesPerCu;
        [[fallthrough]];
    case 8: return per_cu < 96 ? 16 : kDecodeWavesPerCu;
    case 16: return 12;
    default: return kDecodeWavesPerCu;
    }
}

// The caller's workgroups per CU or the preset, and no more than blocks.
unsigned persistent_grid(int64_t n_blocks, int waves_per_cu, int preset, int cus)
{
    const int64_t g = (int64_t)cus * (waves_per_cu > 0 ? waves_per_cu : preset);
    return (unsigned)(n_blocks < g ? n_blocks : g);
}

template <int MAXB, int EC>
hipError_t launch_benc(const uint8_t *d_table, const BatchClass &C, int wpc, int sched,
                       uint8_t *slots, int32_t *sizes, hipStream_t s)
{
    hipLaunchKernelGGL((k_batch_encode<MAXB, EC>), dim3(persistent_grid(C.n_blocks, wpc, kEncodeWavesPerCu, cu_count())),
                       dim3(kWave), 0, s, d_table, C, slots, sizes, sched);
    return hipGetLastError();
}

template <int MAXB, int EC>
hipError_t launch_bdec(const uint8_t *d_table, const BatchClass &C, int wpc, int sched,
                       int32_t *status, hipStream_t s)
{
    const int cus = cu_count();
    hipLaunchKernelGGL((k_batch_decode<MAXB, EC>),
                       dim3(persistent_grid(C.n_blocks, wpc, decode_waves(C, cus), cus)),
                       dim3(kWave), 0, s, d_table, C, status, sched);
    return hipGetLastError();
}

hipError_t benc_dispatch(const uint8_t *t, const BatchClass &C, int wpc, int sched, uint8_t *slots,
                         int32_t *sizes, hipStream_t s)
{
    return for_block_size(C.maxb, [&](auto maxb) {
        switch (C.ec) {
        case 12: return launch_benc<maxb.value, 12>(t, C, wpc, sched, slots, sizes, s);
        case 16: return launch_benc<maxb.value, 16>(t, C, wpc, sched, slots, sizes, s);
        default: return launch_benc<maxb.value, kMixed>(t, C, wpc, sched, slots, sizes, s);
        }
    });
}

hipError_t bdec_dispatch(const uint8_t *t, const BatchClass &C, int wpc, int sched, int32_t *status,
                         hipStream_t s)
{
    return for_block_size(C.maxb, [&](auto maxb) {
        switch (C.ec) {
        case 0: return launch_bdec<maxb.value, 0>(t, C, wpc, sched, status, s);
        case 1: return launch_bdec<maxb.value, 1>(t, C, wpc, sched, status, s);
        case 2: return launch_bdec<maxb.value, 2>(t, C, wpc, sched, status, s);
        case 4: return launch_bdec<maxb.value, 4>(t, C, wpc, sched, status, s);
        case 8: return launch_bdec<maxb.value, 8>(t, C, wpc, sched, status, s);
        case 12: return launch_bdec<maxb.value, 12>(t, C, wpc, sched, status, s);
        case 16: return launch_bdec<maxb.value, 16>(t, C, wpc, sched, status, s);
        default: return launch_bdec<maxb.value, kMixed>(t, C, wpc, sched, status, s);
        }
    });
}

struct WsLayout {
    int64_t slots, sizes, prefix, tiles, total;
};

WsLayout ws_layout(const BatchHeader &h)
{
    auto up = [](int64_t x) { return (x + 255) / 256 * 256; };
    const int64_t n_tiles = (h.total_blocks + kTile - 1) / kTile;
    WsLayout w;
    w.slots = 0;
    w.sizes = up(h.slot_total);
    w.prefix = w.sizes + up(4 * h.total_blocks);
    w.tiles = w.prefix + up(8 * (h.total_blocks + 1 + kTile));
    w.total = w.tiles + up(8 * (n_tiles + 1)) + 256; // (more than is used: sizes stay as they were)
    return w;
}

inline int hip_status(hipError_t e) { return e == hipSuccess ? BSG_OK : BSG_EHIP; }

} // namespace
} // namespace bsg

using namespace bsg;

extern "C" {

int64_t bsg_batch_table_bytes(int32_t count)
{
    return count < 0 ? BSG_EINVAL : table_bytes(count);
}

int bsg_batch_build_table(const bsg_chunk *chunks, int32_t count, void *host_table,
                          int64_t host_table_bytes)
{
    if (count < 0 || (count > 0 && !chunks) || !host_table ||
        host_table_bytes < table_bytes(count))
        return BSG_EINVAL;
    std::vector<BatchChunk> rows(count);
    std::vector<int> key(count);
    std::map<int, int64_t> blocks; // by key
    for (int i = 0; i < count; ++i) {
        const bsg_chunk &c = chunks[i];
        Layout L;
        if (!make_layout(c.n, c.elem_size, c.block_size, &L)) return BSG_EINVAL;
        if (L.block_bytes() > BSG_MAX_BLOCK_BYTES) return BSG_EINVAL;
        BatchChunk &r = rows[i];
        std::memset(&r, 0, sizeof(r));
        r.in = static_cast<const uint8_t *>(c.in);
        r.out = static_cast<uint8_t *>(c.out);
        r.n = c.n;
        r.in_nbytes = c.in_nbytes;
        r.out_capacity = c.out_capacity;
        r.nb = L.nb;
        r.n_full = L.n_full;
        r.last = L.last;
        r.tail = L.tail;
        r.n_blocks = L.n_blocks;
        r.slot_bytes = (lz4_bound(L.block_bytes()) + 15) / 16 * 16;
        r.E = (int32_t)c.elem_size;
        r.orig = i;
        // class key: the instance's block size and element class
        key[i] = for_block_size(L.block_bytes(), [](auto m) { return m.value; }) * kKeysPerSize +
                 key_of(element_class(c.elem_size));
        blocks[key[i]] += r.n_blocks;
    }
    // keys of few blocks share a class, two or more of one instance block size
    const auto few = [&](int k) {
        return kKeyClass[k % kKeysPerSize] <= 8 && blocks[k] < kOwnMinBlocks;
    };
    std::map<int, int> shared; // number of those by size
    for (const auto &[k, n] : blocks)
        if (few(k) && n > 0) ++shared[k / kKeysPerSize];
    for (int &k : key)
        if (few(k) && shared[k / kKeysPerSize] > 1) k -= k % kKeysPerSize;
    std::vector<int> order(count);
    std::iota(order.begin(), order.end(), 0);
    std::stable_sort(order.begin(), order.end(), [&](int a, int b) { return key[a] < key[b]; });
    uint8_t *t = static_cast<uint8_t *>(host_table);
    std::memset(t, 0, (size_t)table_bytes(count));
    BatchHeader &h = *reinterpret_cast<BatchHeader *>(t);
    BatchClass *cls = reinterpret_cast<BatchClass *>(t + sizeof(BatchHeader));
    BatchChunk *ch = reinterpret_cast<BatchChunk *>(t + sizeof(BatchHeader) +
                                                    kMaxClasses * sizeof(BatchClass));
    int64_t blk = 0, slot = 0, all = 0, bytes = 0;
    int nc = 0;
    std::map<int, int64_t> left; // blocks of a class key still to come
    for (int i = 0; i < count; ++i) {
        all += rows[i].n_blocks;
        bytes += rows[i].n_blocks * rows[i].nb * rows[i].E;
        left[key[i]] += rows[i].n_blocks;
    }
    const bool split = all >= kBatchSideMinBlocks && bytes >= kPartMinBatch;
    const int64_t part = std::max(kPartMinBlocks, all / kMaxParts + 1);
    for (int k = 0; k < count; ++k) {
        BatchChunk r = rows[order[k]];
        const int kk = key[order[k]];
        if (k == 0 || kk != key[order[k - 1]] ||
            (split && cls[nc - 1].n_blocks >= part && left[kk] >= part / 4)) {
            BatchClass &C = cls[nc++]; // at most 7 x 4 keys and kMaxParts more
            C.ec = kKeyClass[kk % kKeysPerSize];
            C.maxb = kk / kKeysPerSize;
            C.first_chunk = k;
            C.first_block = blk;
        }
        BatchClass &C = cls[nc - 1];
        C.n_chunks = k - C.first_chunk + 1;
        r.block_start = blk;
        r.slot_start = slot;
        blk += r.n_blocks;
        slot += r.n_blocks * r.slot_bytes;
        left[kk] -= r.n_blocks;
        C.n_blocks = blk - C.first_block;
        ch[k] = r;
    }
    h.count = count;
    h.n_classes = nc;
    h.total_blocks = blk;
    h.slot_total = slot;
    return BSG_OK;
}

int64_t bsg_batch_workspace_size(const void *host_table)
{
    if (!host_table) return BSG_EINVAL;
    return ws_layout(*reinterpret_cast<const BatchHeader *>(host_table)).total;
}

int bsg_batch_compress(const void *host_table, const void *d_table, int64_t *d_nbytes,
                       void *workspace, int64_t workspace_bytes, int32_t waves_per_cu,
                       int32_t schedule, void *stream)
{
    if (!host_table || !d_table || !d_nbytes || !workspace) return BSG_EINVAL;
    if (schedule != BSG_SCHED_STRIDED && schedule != BSG_SCHED_RANGES) return BSG_EINVAL;
    if ((uintptr_t)workspace % 256 || (uintptr_t)d_table % 16 || (uintptr_t)d_nbytes % 8)
        return BSG_EINVAL;
    const TableView T(host_table);
    const BatchHeader &h = *T.h;
    const WsLayout w = ws_layout(h);
    if (workspace_bytes < w.total) return BSG_ECAPACITY;
    for (int i = 0; i < h.count; ++i)
        if ((T.ch[i].n > 0 && !T.ch[i].in) || !T.ch[i].out || (uintptr_t)T.ch[i].out % 8)
            return BSG_EINVAL;
    if (h.count == 0) return BSG_OK;
    hipStream_t s = static_cast<hipStream_t>(stream);
    const uint8_t *t = static_cast<const uint8_t *>(d_table);
    uint8_t *ws = static_cast<uint8_t *>(workspace);
    uint8_t *slots = ws + w.slots;
    int32_t *sizes = reinterpret_cast<int32_t *>(ws + w.sizes);
    int64_t *prefix = reinterpret_cast<int64_t *>(ws + w.prefix);
    int64_t *tiles = reinterpret_cast<int64_t *>(ws + w.tiles);
    // Class by class: the encode on the caller's stream or (every other
    // class) the library's encode stream; then on the pack stream the
    // class's scan (after the bytes of the classes before) and pack, which run
    // beside the next classes' encodes.
    int nonempty = 0;
    for (int c = 0; c < h.n_classes; ++c) nonempty += T.cls[c].n_blocks > 0;
    std::unique_lock<std::mutex> lock;
    SideStreams *g = nullptr;
    if (nonempty >= 2 && h.total_blocks >= kBatchSideMinBlocks &&
        side_streams_begin(s, lock, &g) != hipSuccess)
        return BSG_EHIP;
    hipStream_t ps = g ? g->pack : s;
    int i = 0, last_enc = -1;
    for (int c = 0; c < h.n_classes; ++c) {
        const BatchClass &C = T.cls[c];
        if (C.n_blocks > 0) {
            hipStream_t es = (g && (i & 1)) ? g->enc : s;
            const hipError_t e =
                benc_dispatch(t, C, waves_per_cu, schedule, slots, sizes, es);
            if (e != hipSuccess) return BSG_EHIP;
            if (g) {
                if (hipEventRecord(g->done[i], es) != hipSuccess ||
                    hipStreamWaitEvent(ps, g->done[i], 0) != hipSuccess)
                    return BSG_EHIP;
                if (i & 1) last_enc = i;
            }
            ++i;
        }
        const unsigned nt = (unsigned)std::max<int64_t>((C.n_blocks + kTile - 1) / kTile, 1);
        hipLaunchKernelGGL(k_btile_sum, dim3(nt), dim3(kWave), 0, ps, sizes, C.first_block,
                           C.n_blocks, tiles);
        hipLaunchKernelGGL(k_bprefix, dim3(nt), dim3(kWave), 0, ps, sizes, C.first_block, C.n_blocks,
                           c == 0 ? 1 : 0, tiles, prefix);
        const int64_t grid = persistent_grid(C.n_blocks, waves_per_cu, kDecodeWavesPerCu, cu_count());
        hipLaunchKernelGGL(k_batch_pack, dim3((unsigned)(grid + C.n_chunks)), dim3(kWave), 0, ps, t,
                           C, grid, slots, sizes, prefix, d_nbytes);
        if (hipGetLastError() != hipSuccess) return BSG_EHIP;
    }
    if (g && side_streams_end(g, s, last_enc) != hipSuccess) return BSG_EHIP;
    return BSG_OK;
}

int bsg_batch_decompress(const void *host_table, const void *d_table, int32_t *d_status,
                         int32_t waves_per_cu, int32_t schedule, void *stream)
{
    if (!host_table || !d_table || !d_status || (uintptr_t)d_table % 16 || (uintptr_t)d_status % 4)
        return BSG_EINVAL;
    if (schedule != BSG_SCHED_STRIDED && schedule != BSG_SCHED_RANGES) return BSG_EINVAL;
    const TableView T(host_table);
    const BatchHeader &h = *T.h;
    for (int i = 0; i < h.count; ++i)
        if (!T.ch[i].in || (uintptr_t)T.ch[i].in % 8 || (T.ch[i].n > 0 && !T.ch[i].out))
            return BSG_EINVAL;
    if (h.count == 0) return BSG_OK;
    hipStream_t s = static_cast<hipStream_t>(stream);
    const uint8_t *t = static_cast<const uint8_t *>(d_table);
    hipError_t e = hipSuccess;
    for (int c = 0; c < h.n_classes && e == hipSuccess;) {
        BatchClass C = T.cls[c]; // with the classes after it that were split off it
        for (++c; c < h.n_classes && T.cls[c].ec == C.ec && T.cls[c].maxb == C.maxb; ++c) {
            C.n_chunks += T.cls[c].n_chunks;
            C.n_blocks += T.cls[c].n_blocks;
        }
        if (C.n_blocks == 0) continue;
        e = bdec_dispatch(t, C, waves_per_cu, schedule, d_status, s);
    }
    if (e != hipSuccess) return BSG_EHIP;
    hipLaunchKernelGGL(k_batch_dec_tail, dim3((unsigned)h.count), dim3(kWave), 0, s, t, d_status);
    return hip_status(hipGetLastError());
}

} // extern "C"
