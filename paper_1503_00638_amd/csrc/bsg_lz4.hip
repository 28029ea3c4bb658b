// Stage 2b: per-block LZ4 after the bit transpose (Section 4.2 of Masui et
// al.: each block is transposed and compressed while it is still on chip;
// blocks are independent).  On gfx950 a block lives in LDS and one
// wavefront owns it.
//
// Compression = k_encode (transpose into LDS [+ fused rounding], LDS hash
// table, greedy parse, write to a bound-sized slot) -> k_tile_sum ->
// k_offsets (both left out for small inputs) -> k_pack (copy slots to their
// final place, raw tail).  A large input is encoded in
// segments on two streams while a third stream scans and packs each
// finished segment, so the copy out of the slots runs under the encoding
// of the next segments (the encoder is bound by instruction issue, the
// copy by HBM).
// Decompression = k_decode (stage the LZ4 block in LDS, decode into LDS,
// inverse transpose on the way out to HBM).
#include "bsg_lz4_dev.hpp"

namespace bsg {

namespace {

struct EncArgs {
    const uint8_t *in; // first element of the buffer
    int64_t nb, E, n_full, last;
    uint8_t *slots;
    int64_t slot_bytes;
    int32_t *sizes;
    int64_t block0; // index of the first block of this launch
};

template <int MAXB, int EC, int RM>
__global__ __launch_bounds__(64) void k_encode(EncArgs a, RoundParams rp)
{
    __shared__ EncLds<MAXB> L;
    const int64_t b = a.block0 + blockIdx.x;
    const int64_t elems = b < a.n_full ? a.nb : a.last;
    const int64_t first = b * a.nb;
    const int sz = encode_one<MAXB, EC, RM>(a.in + first * a.E, elems, a.E, rp, first,
                                               a.slots + b * a.slot_bytes, L);
    if (threadIdx.x == 0) a.sizes[b] = sz;
}

struct PackArgs {
    const uint8_t *slots;
    int64_t slot_bytes;
    const int32_t *sizes;
    int64_t *tile_sum;
    int64_t n_blocks, b0; // the launch's first block (a multiple of kTile)
    int last;             // it goes to the end: header, verdict, raw tail
    int64_t fixed_bytes, cap;
    int64_t *d_nbytes;
    uint8_t *out;
    uint32_t magic;
    int64_t n, E, nb;
    const uint8_t *tail_src;
    int64_t tail_bytes, tail_first_elem;
    int round_tail;
};

__device__ __forceinline__ uint64_t *offsets_of(const PackArgs &a)
{
    return reinterpret_cast<uint64_t *>(a.out + kHeaderBytes);
}

// Stream total, capacity verdict, header and the end of the offset table
// (one thread).
__device__ __forceinline__ void finish_stream(const PackArgs &a, int64_t payload)
{
    const int64_t total = a.fixed_bytes + payload;
    *a.d_nbytes = total <= a.cap ? total : (int64_t)BSG_ECAPACITY;
    bsg_header *h = reinterpret_cast<bsg_header *>(a.out);
    h->magic = a.magic;
    h->elem_size = (uint32_t)a.E;
    h->n = (uint64_t)a.n;
    h->block_elems = (uint32_t)a.nb;
    h->n_blocks = (uint32_t)a.n_blocks;
    offsets_of(a)[a.n_blocks] = (uint64_t)payload;
}

// The two scan kernels take one wavefront per 1024-block tile and no LDS:
// the encoders beside them hold all of it (16 x 10 KiB per CU), and a
// workgroup that needs some waits until a CU's encoder ends and no other
// takes its place (a one-workgroup scan waited 1.3 ms; the packs then ran
// after the encoding instead of beside it).
//
// Sizes of tile t: lane l holds blocks 4 l .. 4 l + 3 of each of its 4 strips
// (0 past the last block; the array is padded to 256 bytes).
constexpr int kStrip = 4 * kWave;
__device__ __forceinline__ void load_tile(const PackArgs &a, int64_t tile, int lane,
                                          int (&v)[kTile / kStrip][4])
{
#pragma unroll
    for (int s = 0; s < kTile / kStrip; ++s) {
        const int64_t k = tile * kTile + s * kStrip + 4 * lane;
        const int4 x = *reinterpret_cast<const int4 *>(a.sizes + (k < a.n_blocks ? k : 0));
        v[s][0] = k < a.n_blocks ? x.x : 0;
        v[s][1] = k + 1 < a.n_blocks ? x.y : 0;
        v[s][2] = k + 2 < a.n_blocks ? x.z : 0;
        v[s][3] = k + 3 < a.n_blocks ? x.w : 0;
    }
}

__global__ __launch_bounds__(64) void k_tile_sum(PackArgs a)
{
    const int64_t tile = a.b0 / kTile + blockIdx.x;
    int v[kTile / kStrip][4], sum = 0, total;
    load_tile(a, tile, threadIdx.x, v);
#pragma unroll
    for (int s = 0; s < kTile / kStrip; ++s) sum += v[s][0] + v[s][1] + v[s][2] + v[s][3];
    wave_excl_scan(sum, total); // a tile's bytes stay below 2^27
    if (threadIdx.x == 0) a.tile_sum[tile] = total;
}

// Offsets of a tile's blocks, after the sums of all tiles before it.
__global__ __launch_bounds__(64) void k_offsets(PackArgs a)
{
    const int64_t tile = a.b0 / kTile + blockIdx.x;
    const int lane = threadIdx.x;
    int v[kTile / kStrip][4];
    load_tile(a, tile, lane, v);
    int64_t before = 0;
#pragma unroll 4
    for (int64_t k = lane; k < tile; k += kWave) before += a.tile_sum[k];
    int64_t base = wave_sum_i64(before);
    uint64_t *off = offsets_of(a);
#pragma unroll
    for (int s = 0; s < kTile / kStrip; ++s) {
        const int64_t k = tile * kTile + s * kStrip + 4 * lane;
        int total;
        int64_t o = base + wave_excl_scan(v[s][0] + v[s][1] + v[s][2] + v[s][3], total);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            if (k + q < a.n_blocks) off[k + q] = (uint64_t)o;
            o += v[s][q];
        }
        base += total;
    }
    if (a.last && blockIdx.x + 1 == gridDim.x && lane == 0) finish_stream(a, base);
}

// (Each launch moves next to nothing: its 5 us are the launch and two memory
// round trips, so fewer launches are all that helps.  Before, four scan and
// pack launches followed the encode: 53.5 -> 47.0 us for a call of 36 blocks,
// 112 -> 104 us at 2094 blocks, 150 -> 146 us at 15,600.)
//
// Copy the LZ4 bytes of blocks b0, b0 + 1, ... from their slots to the
// payload, one wavefront per block; in the last launch the wavefront past
// the last block copies the raw tail.  Nothing is written past the output's
// capacity: a block whose bytes would end past it is skipped (the stream
// then does not fit and the call reports so), and the tail is written only
// when the stream fits.
// SELF: the whole stream in one launch, no scan before it: each
// wavefront adds up the sizes of the blocks before its own, and the last one
// writes the header and the verdict too.
template <bool SELF>
__global__ __launch_bounds__(64) void k_pack(PackArgs a, RoundParams rp)
{
    const int64_t b = a.b0 + blockIdx.x;
    const int lane = threadIdx.x;
    uint64_t *off = offsets_of(a);
    uint8_t *payload = a.out + kHeaderBytes + 8 * (a.n_blocks + 1);
    const int sz = b < a.n_blocks ? a.sizes[b] : 0;
    int64_t ob;
    if constexpr (SELF) {
        const uint4 *before = reinterpret_cast<const uint4 *>(a.sizes);
        const int n1 = (int)b, n4 = n1 / 4;
        uint32_t sum = 4 * n4 + lane < n1 ? a.sizes[4 * n4 + lane] : 0;
#pragma unroll 8
        for (int k = lane; k < n4; k += kWave) {
            const uint4 v = before[k];
            sum += v.x + v.y + v.z + v.w;
        }
        int total;
        wave_excl_scan((int)sum, total);
        ob = total;
        if (lane == 0 && b < a.n_blocks) off[b] = (uint64_t)ob;
        if (lane == 0 && b == a.n_blocks) finish_stream(a, ob);
    } else {
        ob = (int64_t)off[b];
    }
    if (b < a.n_blocks) {
        if (a.fixed_bytes + ob + sz <= a.cap)
            copy_slot(payload + ob, a.slots + b * a.slot_bytes, sz, lane);
        return;
    }
    if (a.fixed_bytes + ob > a.cap) return;
    uint8_t *dst = payload + ob;
    if (a.round_tail) { // the raw tail of the fused path is rounded too (float32 elements)
        for (int64_t k = lane; k < a.tail_bytes / 4; k += kWave) {
            uint32_t x = 0;
            for (int q = 0; q < 4; ++q) x |= (uint32_t)a.tail_src[4 * k + q] << (8 * q);
            x = round_element(x, a.tail_first_elem + k, rp);
            for (int q = 0; q < 4; ++q) dst[4 * k + q] = (uint8_t)(x >> (8 * q));
        }
        return;
    }
    for (int64_t i = lane; i < a.tail_bytes; i += kWave) dst[i] = a.tail_src[i];
}

struct DecArgs {
    const uint8_t *in;
    int64_t in_nbytes;
    uint8_t *out;
    int64_t n, E, nb, n_full, last, n_blocks, tail;
    int32_t *status;
    int fast_out; // out is 16-byte aligned
    uint32_t magic; // the stream's filter: bit transpose or byte shuffle
};

template <int MAXB, int EC>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(dec_waves_per_eu<MAXB, EC>()))) void k_decode(DecArgs a)
{
    __shared__ DecLds<MAXB> L;
    const int lane = threadIdx.x;
    const int64_t b = blockIdx.x;
    const int64_t table_end = kHeaderBytes + 8 * (a.n_blocks + 1);
    const int64_t tail_bytes = a.tail * a.E;
    const int64_t payload_len = a.in_nbytes - table_end - tail_bytes; // >= 0 (host-checked)
    const uint8_t *payload = a.in + table_end;
    if (b == a.n_blocks) { // header check and raw tail
        if (!header_ok(a.in, payload_len, a.n, a.E, a.nb, a.n_blocks, a.magic)) {
            fail(a.status);
            return;
        }
        uint8_t *dst = a.out + (a.n - a.tail) * a.E;
        for (int64_t i = lane; i < tail_bytes; i += kWave) dst[i] = payload[payload_len + i];
        return;
    }
    const int64_t elems = b < a.n_full ? a.nb : a.last;
    const uint64_t *off = reinterpret_cast<const uint64_t *>(a.in + kHeaderBytes);
    if (!decode_one<MAXB, EC>(payload, payload_len, off, b, elems, a.E, a.in + a.in_nbytes,
                              a.out + b * a.nb * a.E, a.fast_out != 0, L))
        fail(a.status);
}

template <int MAXB, int EC, int RM>
hipError_t encode_launch(const EncArgs &ea, int64_t nblocks, const RoundParams &rp,
                         hipStream_t s)
{
    if (nblocks == 0) return hipSuccess;
    hipLaunchKernelGGL((k_encode<MAXB, EC, RM>), dim3((unsigned)nblocks), dim3(kWave), 0, s, ea,
                       rp);
    return hipGetLastError();
}

template <int MAXB>
hipError_t encode_dispatch(const EncArgs &ea, int64_t nblocks, const RoundParams *rp, int ec,
                           hipStream_t s)
{
    const RoundParams none{};
    if (rp) {
        if (ec != 4) return encode_launch<MAXB, 0, kRoundPlain>(ea, nblocks, *rp, s);
        return rp->fscale ? encode_launch<MAXB, 4, kRoundScaled>(ea, nblocks, *rp, s)
                          : encode_launch<MAXB, 4, kRoundPlain>(ea, nblocks, *rp, s);
    }
    switch (ec) {
    case kByteShuffle: return encode_launch<MAXB, kByteShuffle, kRoundNone>(ea, nblocks, none, s);
    case 1: return encode_launch<MAXB, 1, kRoundNone>(ea, nblocks, none, s);
    case 2: return encode_launch<MAXB, 2, kRoundNone>(ea, nblocks, none, s);
    case 4: return encode_launch<MAXB, 4, kRoundNone>(ea, nblocks, none, s);
    case 8: return encode_launch<MAXB, 8, kRoundNone>(ea, nblocks, none, s);
    case 12: return encode_launch<MAXB, 12, kRoundNone>(ea, nblocks, none, s);
    case 16: return encode_launch<MAXB, 16, kRoundNone>(ea, nblocks, none, s);
    default: return encode_launch<MAXB, 0, kRoundNone>(ea, nblocks, none, s);
    }
}

// VGPRs of an encoder instance (from its kernel attributes, read once).
template <int MAXB, int EC, int RM> int encoder_vgprs()
{
    static const int regs = [] {
        hipFuncAttributes a{};
        return hipFuncGetAttributes(&a, reinterpret_cast<const void *>(&k_encode<MAXB, EC, RM>)) ==
                       hipSuccess
                   ? a.numRegs
                   : 1 << 20;
    }();
    return regs;
}

// The VGPRs of the instance encode_dispatch picks.
template <int MAXB> int encoder_vgprs_for(const RoundParams *rp, int ec)
{
    if (rp) {
        if (ec != 4) return encoder_vgprs<MAXB, 0, kRoundPlain>();
        return rp->fscale ? encoder_vgprs<MAXB, 4, kRoundScaled>()
                          : encoder_vgprs<MAXB, 4, kRoundPlain>();
    }
    switch (ec) {
    case kByteShuffle: return encoder_vgprs<MAXB, kByteShuffle, kRoundNone>();
    case 1: return encoder_vgprs<MAXB, 1, kRoundNone>();
    case 2: return encoder_vgprs<MAXB, 2, kRoundNone>();
    case 4: return encoder_vgprs<MAXB, 4, kRoundNone>();
    case 8: return encoder_vgprs<MAXB, 8, kRoundNone>();
    case 12: return encoder_vgprs<MAXB, 12, kRoundNone>();
    case 16: return encoder_vgprs<MAXB, 16, kRoundNone>();
    default: return encoder_vgprs<MAXB, 0, kRoundNone>();
    }
}

template <int MAXB, int EC>
hipError_t decode_launch(const DecArgs &a, hipStream_t s)
{
    hipLaunchKernelGGL((k_decode<MAXB, EC>), dim3((unsigned)(a.n_blocks + 1)), dim3(kWave), 0, s, a);
    return hipGetLastError();
}

template <int MAXB>
hipError_t decode_dispatch(const DecArgs &a, int ec, hipStream_t s)
{
    switch (ec) {
    case kByteShuffle: return decode_launch<MAXB, kByteShuffle>(a, s);
    case 1: return decode_launch<MAXB, 1>(a, s);
    case 2: return decode_launch<MAXB, 2>(a, s);
    case 4: return decode_launch<MAXB, 4>(a, s);
    case 8: return decode_launch<MAXB, 8>(a, s);
    case 12: return decode_launch<MAXB, 12>(a, s);
    case 16: return decode_launch<MAXB, 16>(a, s);
    default: return decode_launch<MAXB, 0>(a, s);
    }
}

} // namespace

int64_t compress_workspace(const Layout &L)
{
    const int64_t slot = (lz4_bound(L.block_bytes()) + 15) / 16 * 16;
    const int64_t n_tiles = (L.n_blocks + kTile - 1) / kTile;
    int64_t ws = L.n_blocks * slot;
    ws = (ws + 255) / 256 * 256 + ((L.n_blocks * 4 + 255) / 256) * 256;
    ws += ((n_tiles * 8 + 255) / 256) * 256;
    ws += 256; // (unused; callers' sizes and the no-allocation limit stay as they were)
    return ws;
}

// Up to this many blocks the pack's wavefronts add up the sizes before their
// own block (at most 16 KiB each, from L2, all loads in flight); above it the
// two scan launches cost less than the reading, which grows with the square
// of the count.
constexpr int64_t kSelfMaxBlocks = 4096;

constexpr int kMaxSeg = 16;             // segments of a large input
static_assert(kMaxSeg <= kSideEvents, "an event per segment");
// ... of at least this many blocks and bytes: each costs 5 launches and an
// event on two streams, 14 us where its blocks are small (140,000 blocks of 512
// bytes, 8-byte elements, 496 us in 16 segments, 300 in one; of 2048 bytes 562 in
// 16, 478 in 4, 463 in one; of 4096 bytes 708 in 16, 660 in 8, 672 in one).
constexpr int64_t kSegMinBlocks = 8192;
constexpr int64_t kSegMinBytes = 64ll << 20;
// Segments pay only when the encoder leaves registers for the pack waves
// beside its 4 resident waves per SIMD (LDS allows 16 per CU): at 112 VGPRs
// or fewer.  An encoder that fills the register file (125 VGPRs for 8-byte
// elements) lost 14 % to them, one at 84 gained 4 %.
constexpr int kSegMaxVgprs = 112;

namespace {
constexpr int kMaxSideDevices = 64;
std::mutex side_mu;
SideStreams side_dev[kMaxSideDevices]; // guarded by side_mu
} // namespace

hipError_t side_streams_begin(hipStream_t s, std::unique_lock<std::mutex> &lock,
                              SideStreams **out)
{
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxSideDevices) return hipErrorInvalidDevice;
    lock = std::unique_lock<std::mutex>(side_mu);
    SideStreams &g = side_dev[dev];
    if (!g.made) {
        g.made = true;
        bool ok = hipStreamCreateWithFlags(&g.enc, hipStreamNonBlocking) == hipSuccess &&
                  hipStreamCreateWithFlags(&g.pack, hipStreamNonBlocking) == hipSuccess &&
                  hipEventCreateWithFlags(&g.fork, hipEventDisableTiming) == hipSuccess &&
                  hipEventCreateWithFlags(&g.join, hipEventDisableTiming) == hipSuccess;
        for (int i = 0; ok && i < kSideEvents; ++i)
            ok = hipEventCreateWithFlags(&g.done[i], hipEventDisableTiming) == hipSuccess;
        g.ok = ok;
    }
    if (!g.ok) return hipErrorOutOfMemory;
    if ((e = hipEventRecord(g.fork, s)) != hipSuccess ||
        (e = hipStreamWaitEvent(g.enc, g.fork, 0)) != hipSuccess ||
        (e = hipStreamWaitEvent(g.pack, g.fork, 0)) != hipSuccess)
        return e;
    *out = &g;
    return hipSuccess;
}

// (the encode stream is also joined directly, so that a stream capture sees
// it joined)
hipError_t side_streams_end(SideStreams *g, hipStream_t s, int last_enc)
{
    hipError_t e;
    if ((e = hipEventRecord(g->join, g->pack)) != hipSuccess ||
        (e = hipStreamWaitEvent(s, g->join, 0)) != hipSuccess)
        return e;
    if (last_enc >= 0 && (e = hipStreamWaitEvent(s, g->done[last_enc], 0)) != hipSuccess) return e;
    return hipSuccess;
}

hipError_t launch_compress(const uint8_t *in, uint8_t *out, const Layout &L, int64_t cap,
                           int64_t *d_nbytes, void *ws, int64_t ws_bytes, const RoundParams *rp,
                           hipStream_t s, int filter, bool may_segment)
{
    (void)ws_bytes;
    const int64_t slot = (lz4_bound(L.block_bytes()) + 15) / 16 * 16;
    const int64_t n_tiles = (L.n_blocks + kTile - 1) / kTile;
    uint8_t *w = static_cast<uint8_t *>(ws);
    uint8_t *slots = w;
    int64_t pos = (L.n_blocks * slot + 255) / 256 * 256;
    int32_t *sizes = reinterpret_cast<int32_t *>(w + pos);
    pos += ((L.n_blocks * 4 + 255) / 256) * 256;
    int64_t *tile_sum = reinterpret_cast<int64_t *>(w + pos);

    RoundParams none{};
    const int ec = filter == BSG_FILTER_BYTE ? kByteShuffle : element_class(L.E);
    PackArgs pa{};
    pa.slots = slots;
    pa.slot_bytes = slot;
    pa.sizes = sizes;
    pa.n_blocks = L.n_blocks;
    pa.tile_sum = tile_sum;
    pa.fixed_bytes = kHeaderBytes + 8 * (L.n_blocks + 1) + L.tail * L.E;
    pa.cap = cap;
    pa.d_nbytes = d_nbytes;
    pa.out = out;
    pa.magic = filter == BSG_FILTER_BYTE ? BSG_MAGIC_BYTE : BSG_MAGIC;
    pa.n = L.n;
    pa.E = L.E;
    pa.nb = L.nb;
    pa.tail_src = in + (L.n - L.tail) * L.E;
    pa.tail_bytes = L.tail * L.E;
    pa.tail_first_elem = L.n - L.tail;
    pa.round_tail = rp ? 1 : 0;

    // segments of whole tiles
    int nseg = (int)std::min<int64_t>({kMaxSeg, L.n_blocks / kSegMinBlocks,
                                       L.n_blocks * L.block_bytes() / kSegMinBytes});
    if (nseg > 1 && may_segment) {
        const int regs = for_block_size(
            L.block_bytes(), [&](auto maxb) { return encoder_vgprs_for<maxb.value>(rp, ec); });
        if (regs > kSegMaxVgprs) nseg = 1;
    }
    if (nseg < 1 || !may_segment) nseg = 1;
    std::unique_lock<std::mutex> lock;
    SideStreams *g = nullptr;
    hipError_t e;
    if (nseg > 1 && (e = side_streams_begin(s, lock, &g)) != hipSuccess) return e;
    hipStream_t ps = g ? g->pack : s;
    for (int i = 0; i < nseg; ++i) {
        const int64_t t0 = n_tiles * i / nseg, t1 = n_tiles * (i + 1) / nseg;
        const int64_t b0 = t0 * kTile, b1 = std::min(t1 * kTile, L.n_blocks);
        const bool last = i == nseg - 1;
        hipStream_t es = (g && (i & 1)) ? g->enc : s;
        EncArgs ea{in, L.nb, L.E, L.n_full, L.last, slots, slot, sizes, b0};
        e = for_block_size(L.block_bytes(), [&](auto maxb) {
            return encode_dispatch<maxb.value>(ea, b1 - b0, rp, ec, es);
        });
        if (e != hipSuccess) return e;
        if (g && ((e = hipEventRecord(g->done[i], es)) != hipSuccess ||
                  (e = hipStreamWaitEvent(ps, g->done[i], 0)) != hipSuccess))
            return e;
        pa.b0 = b0;
        pa.last = last ? 1 : 0;
        const unsigned npack = (unsigned)(b1 - b0 + (last ? 1 : 0));
        if (L.n_blocks <= kSelfMaxBlocks) {
            hipLaunchKernelGGL((k_pack<true>), dim3(npack), dim3(kWave), 0, ps, pa,
                               rp ? *rp : none);
        } else {
            const unsigned nt = (unsigned)(t1 - t0);
            hipLaunchKernelGGL(k_tile_sum, dim3(nt), dim3(kWave), 0, ps, pa);
            if ((e = hipGetLastError()) != hipSuccess) return e;
            hipLaunchKernelGGL(k_offsets, dim3(nt), dim3(kWave), 0, ps, pa);
            if ((e = hipGetLastError()) != hipSuccess) return e;
            hipLaunchKernelGGL((k_pack<false>), dim3(npack), dim3(kWave), 0, ps, pa,
                               rp ? *rp : none);
        }
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    // (odd segments went to the encode stream)
    if (g) return side_streams_end(g, s, (nseg & 1) ? nseg - 2 : nseg - 1);
    return hipSuccess;
}

hipError_t launch_decompress(const uint8_t *in, int64_t in_nbytes, uint8_t *out, const Layout &L,
                             int32_t *d_status, hipStream_t s, int filter)
{
    DecArgs a{in,     in_nbytes,  out,    L.n,        L.E,    L.nb, L.n_full,
              L.last, L.n_blocks, L.tail, d_status, ((uintptr_t)out % 16) == 0,
              filter == BSG_FILTER_BYTE ? BSG_MAGIC_BYTE : BSG_MAGIC};
    const int ec = filter == BSG_FILTER_BYTE ? kByteShuffle : element_class(L.E);
    return for_block_size(L.block_bytes(),
                          [&](auto maxb) { return decode_dispatch<maxb.value>(a, ec, s); });
}

} // namespace bsg
