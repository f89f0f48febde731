// msz_encode.hip -- lossless encoding of the edits (Sec. 6.3): the edited
// vertices' indices, sorted, as a gap sequence, and their edit values, each
// stream entropy-coded with a canonical Huffman code, on the GPU.
//
// Stream format (all little-endian; declared with the entry points in msz.h):
//   header (kEncHeader bytes): magic "MSZE", version, n, m, chunk count,
//       edits per chunk, then the code lengths of the 32 gap symbols and of
//       the 512 value symbols (one byte each), zero padding;
//   chunk table: per chunk {uint32 word offset into the bit stream, int32
//       index of the chunk's first edit};
//   bit stream: uint32 words; chunk c starts at its own word.
// Within a chunk the edits follow in index order.  An edit is
//   [gap, for all but the chunk's first edit]  Huffman code of the bucket
//       b = floor(log2(d)) of d = index - previous index (d >= 1), then the b
//       low bits of d (d - 2^b);
//   [value]  Huffman code of the 9 high bits of the float32 edit (sign and
//       exponent), then its 23 mantissa bits.
// Every field is emitted most significant bit first; emitted bit j of a chunk
// is bit (j % 32) of the chunk's word (j / 32).  Huffman codes are canonical
// (symbols ordered by code length, then by symbol) and at most kEncMaxLen bits
// long: the lengths come from the standard two-smallest-merge construction
// (ties broken by node age), and while a length exceeds the limit every count
// is halved (rounding up) and the code rebuilt.
// An edit is a vertex whose edit value is not +0 (the loop only lowers values,
// so every edited vertex has a negative edit).
#include <algorithm>
#include <cstring>
#include <queue>
#include <utility>
#include <vector>

#include "msz_internal.h"

namespace msz {

constexpr int kEncGapSyms = 32, kEncValSyms = 512, kEncMaxLen = 20;
constexpr int kEncChunk = 256;         // edits per chunk (one decoding thread each)
constexpr int kEncBlock = 4096;        // dense entries per compaction block (256 threads x 16)
constexpr int kEncHeader = 576;        // header bytes (24 fixed + 544 code lengths, padded)
constexpr unsigned kEncMagic = 0x455A534Du;  // "MSZE"
constexpr unsigned kEncVersion = 1u;

struct EncCode {  // canonical code of one symbol: the code in its low `len` bits
    unsigned code;
    int len;
};

// ------------------------------------------------------------- kernels ---

__device__ __forceinline__ int gap_bucket(unsigned d) { return 31 - __clz(d); }

// The dense entries of a block: thread t holds the four 4-entry groups
// 4 (t + 256 k) .. + 3 of the block, k = 0..3 (one coalesced 16-byte load
// each; entries past n read as 0).
struct EncGroups {
    uint4 v[4];
    __device__ __forceinline__ EncGroups(const unsigned* __restrict__ bits, long long n) {
        const long long base = static_cast<long long>(blockIdx.x) * kEncBlock;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const long long i = base + 4 * (threadIdx.x + 256 * k);
            if (i + 3 < n) {
                v[k] = *reinterpret_cast<const uint4*>(bits + i);
            } else {
                v[k].x = i < n ? bits[i] : 0u;
                v[k].y = i + 1 < n ? bits[i + 1] : 0u;
                v[k].z = i + 2 < n ? bits[i + 2] : 0u;
                v[k].w = 0u;
            }
        }
    }
    __device__ __forceinline__ unsigned count(int k) const {
        return (v[k].x != 0u) + (v[k].y != 0u) + (v[k].z != 0u) + (v[k].w != 0u);
    }
};

// Inclusive prefix sum of x over a wave.
__device__ __forceinline__ unsigned wave_inclusive(unsigned x) {
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const unsigned y = __shfl_up(x, o);
        if (lane >= o) x += y;
    }
    return x;
}

// Non-zero edit counts of each block of kEncBlock dense entries.  Streams the
// field once, as the compaction below does (3600x2400: 8 us and 12 us, where
// one 4-byte load per entry, 64 bytes apart over a wave, took 26 each).
__global__ void __launch_bounds__(256) k_enc_count(const unsigned* __restrict__ bits, long long n,
                                                   unsigned* __restrict__ counts) {
    __shared__ unsigned part[4];
    const EncGroups g(bits, n);
    unsigned c = g.count(0) + g.count(1) + g.count(2) + g.count(3);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) c += __shfl_xor(c, o);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = c;
    __syncthreads();
    if (threadIdx.x == 0) counts[blockIdx.x] = part[0] + part[1] + part[2] + part[3];
}

// In-place exclusive prefix sum of v[0..len) with the total in v[len] (one
// block of 1024 threads walking 8192-element pieces, 8 per thread; v is
// 16-byte aligned).
__global__ void __launch_bounds__(1024) k_enc_scan(unsigned* v, int len) {
    __shared__ unsigned waves[16];
    const int wave = threadIdx.x >> 6;
    unsigned carry = 0;
    for (int p = 0; p < len; p += 8192) {
        const int i = p + 8 * threadIdx.x;
        unsigned x[8], sum = 0;
#pragma unroll
        for (int k = 0; k < 8; ++k) x[k] = i + k < len ? v[i + k] : 0u;
#pragma unroll
        for (int k = 0; k < 8; ++k) sum += x[k];
        const unsigned incl = wave_inclusive(sum);
        if ((threadIdx.x & 63) == 63) waves[wave] = incl;
        __syncthreads();
        unsigned at = carry + incl - sum;
#pragma unroll
        for (int w = 0; w < 16; ++w) {
            const unsigned t = waves[w];
            at += w < wave ? t : 0u;
            carry += t;
        }
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            if (i + k < len) v[i + k] = at;
            at += x[k];
        }
        __syncthreads();  // waves is rewritten by the next piece
    }
    if (threadIdx.x == 0) v[len] = carry;
}

// Block-local exclusive scan of 256 thread values (returns the thread's
// offset).  s: four words; the caller does not reuse it without a barrier.
__device__ __forceinline__ unsigned block_exclusive(unsigned x, unsigned* s) {
    const unsigned incl = wave_inclusive(x);
    const int wave = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 63) s[wave] = incl;
    __syncthreads();
    unsigned r = incl - x;
#pragma unroll
    for (int w = 0; w < 4; ++w) r += w < wave ? s[w] : 0u;
    return r;
}

// The edits of each dense block, in index order, at the block's offset.
__global__ void __launch_bounds__(256) k_enc_compact(const unsigned* __restrict__ bits, long long n,
                                                     const unsigned* __restrict__ offsets, int* __restrict__ idx,
                                                     unsigned* __restrict__ val) {
    __shared__ unsigned s[4][4];  // edits per group row k and wave
    const EncGroups g(bits, n);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    unsigned c[4], at[4];
    // prefix sums over the wave, two group rows per word (at most 256 each)
    const unsigned p01 = g.count(0) | (g.count(1) << 16), p23 = g.count(2) | (g.count(3) << 16);
    const unsigned i01 = wave_inclusive(p01), i23 = wave_inclusive(p23);
    c[0] = p01 & 0xFFFFu, c[1] = p01 >> 16, c[2] = p23 & 0xFFFFu, c[3] = p23 >> 16;
    at[0] = (i01 & 0xFFFFu) - c[0], at[1] = (i01 >> 16) - c[1];
    at[2] = (i23 & 0xFFFFu) - c[2], at[3] = (i23 >> 16) - c[3];
    if (lane == 63) {
#pragma unroll
        for (int k = 0; k < 4; ++k) s[k][wave] = at[k] + c[k];
    }
    __syncthreads();
    unsigned o = offsets[blockIdx.x];
    const long long base = static_cast<long long>(blockIdx.x) * kEncBlock;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        unsigned row = 0, q = o + at[k];
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            q += w < wave ? s[k][w] : 0u;
            row += s[k][w];
        }
        o += row;
        const int i = static_cast<int>(base + 4 * (threadIdx.x + 256 * k));
        const unsigned b[4] = {g.v[k].x, g.v[k].y, g.v[k].z, g.v[k].w};
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (b[j] != 0u) {
                idx[q] = i + j;
                val[q] = b[j];
                ++q;
            }
    }
}

// Adds 1 to h[sym] for every active lane of the wave (sym < 0: none): the
// lanes of one symbol add together, so that the few symbols most edits share
// do not queue on one LDS address.
__device__ __forceinline__ void wave_count(unsigned* h, int sym) {
    unsigned long long todo = __ballot(sym >= 0);
    while (todo) {
        const int s = __shfl(sym, __ffsll(static_cast<long long>(todo)) - 1);
        const unsigned long long same = __ballot(sym == s);
        if ((threadIdx.x & 63) == __ffsll(static_cast<long long>(same)) - 1) atomicAdd(h + s, static_cast<unsigned>(__popcll(same)));
        todo &= ~same;
    }
}

// Symbol counts: gap buckets (all but each chunk's first edit) and value symbols.
__global__ void __launch_bounds__(256) k_enc_hist(const int* __restrict__ idx, const unsigned* __restrict__ val,
                                                  int m, unsigned* __restrict__ ghist, unsigned* __restrict__ vhist) {
    __shared__ unsigned g[kEncGapSyms], h[kEncValSyms];
    for (int i = threadIdx.x; i < kEncValSyms; i += blockDim.x) h[i] = 0u;
    if (threadIdx.x < kEncGapSyms) g[threadIdx.x] = 0u;
    __syncthreads();
    constexpr int PER = 4;  // edits per thread and round, their loads in flight together
    for (int base = blockIdx.x * 256 * PER; base < m; base += gridDim.x * 256 * PER) {
        int gs[PER], vs[PER];
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            const int k = base + 256 * q + static_cast<int>(threadIdx.x), kc = min(k, m - 1);
            const unsigned d = static_cast<unsigned>(idx[kc] - idx[max(kc - 1, 0)]), v = val[kc];
            gs[q] = k < m && k % kEncChunk != 0 ? gap_bucket(d) : -1;
            vs[q] = k < m ? static_cast<int>(v >> 23) : -1;
        }
#pragma unroll
        for (int q = 0; q < PER; ++q) wave_count(g, gs[q]), wave_count(h, vs[q]);
    }
    __syncthreads();
    for (int i = threadIdx.x; i < kEncValSyms; i += blockDim.x)
        if (h[i]) atomicAdd(vhist + i, h[i]);
    if (threadIdx.x < kEncGapSyms && g[threadIdx.x]) atomicAdd(ghist + threadIdx.x, g[threadIdx.x]);
}

struct EncTables {
    EncCode gap[kEncGapSyms];
    EncCode val[kEncValSyms];
};

__device__ __forceinline__ int edit_bits(const EncTables& T, const int* idx, const unsigned* val, int k) {
    int nb = T.val[val[k] >> 23].len + 23;
    if (k % kEncChunk != 0) {
        const int b = gap_bucket(static_cast<unsigned>(idx[k] - idx[k - 1]));
        nb += T.gap[b].len + b;
    }
    return nb;
}

// One block per chunk, one thread per edit: the chunk's length in words.
static_assert(kEncChunk == 256, "a chunk is one block of 256 threads");
__global__ void __launch_bounds__(256) k_enc_sizes(const EncTables* __restrict__ T, const int* __restrict__ idx,
                                                   const unsigned* __restrict__ val, int m,
                                                   unsigned* __restrict__ chunk_words) {
    __shared__ unsigned s[4];
    const int k = blockIdx.x * kEncChunk + threadIdx.x;
    const unsigned nb = k < m ? static_cast<unsigned>(edit_bits(*T, idx, val, k)) : 0u;
    const unsigned o = block_exclusive(nb, s);
    if (threadIdx.x == 255) chunk_words[blockIdx.x] = (o + nb + 31) >> 5;
}

// Appends `w` bits of v (most significant first) at bit position pos of a
// 128-bit buffer whose bit j is emitted j-th.
__device__ __forceinline__ void put_bits(unsigned long long (&buf)[2], int& pos, unsigned v, int w) {
    if (w == 0) return;
    const unsigned long long r = static_cast<unsigned long long>(__builtin_bitreverse32(v) >> (32 - w));
    if (pos < 64) {
        buf[0] |= r << pos;
        if (pos + w > 64) buf[1] |= r >> (64 - pos);
    } else {
        buf[1] |= r << (pos - 64);
    }
    pos += w;
}

// One block per chunk: the chunk's bits, put together in LDS (neighbouring
// edits share words, so each ORs its bits in), then written with its table
// entry (word offset, index of the first edit).  chunk_word0: the word
// offsets of the chunks, the total after the last.
__global__ void __launch_bounds__(256) k_enc_write(const EncTables* __restrict__ T, const int* __restrict__ idx,
                                                   const unsigned* __restrict__ val, int m,
                                                   const unsigned* __restrict__ chunk_word0,
                                                   unsigned* __restrict__ table, unsigned* __restrict__ stream) {
    constexpr int kMaxWords = (kEncChunk * (2 * kEncMaxLen + 30 + 23) + 31) / 32;
    __shared__ unsigned words[kMaxWords + 4];  // an edit's buffer spans four words
    __shared__ unsigned s[4];
    const int c = blockIdx.x, k = c * kEncChunk + threadIdx.x;
    const unsigned w0 = chunk_word0[c];
    const int nw = static_cast<int>(chunk_word0[c + 1] - w0);
    for (int i = threadIdx.x; i < nw + 4; i += 256) words[i] = 0u;
    unsigned long long buf[2] = {0ull, 0ull};
    int pos = 0;
    if (k < m) {
        if (threadIdx.x != 0) {
            const unsigned d = static_cast<unsigned>(idx[k] - idx[k - 1]);
            const int b = gap_bucket(d);
            put_bits(buf, pos, T->gap[b].code, T->gap[b].len);
            put_bits(buf, pos, d - (1u << b), b);
        }
        const unsigned v = val[k];
        put_bits(buf, pos, T->val[v >> 23].code, T->val[v >> 23].len);
        put_bits(buf, pos, v & 0x7FFFFFu, 23);
    }
    const unsigned start = block_exclusive(static_cast<unsigned>(pos), s);  // words is zeroed past its barrier
    if (k < m) {
        const unsigned sh = start & 31u;
        unsigned* w = words + (start >> 5);
        // the buffer shifted by sh: at most 31 + 93 bits, four words
        const unsigned long long lo = buf[0] << sh;
        const unsigned long long mid = sh ? (buf[0] >> (64 - sh)) | (buf[1] << sh) : buf[1];
        const unsigned out[4] = {static_cast<unsigned>(lo), static_cast<unsigned>(lo >> 32),
                                 static_cast<unsigned>(mid), static_cast<unsigned>(mid >> 32)};
#pragma unroll
        for (int q = 0; q < 4; ++q)
            if (out[q]) atomicOr(w + q, out[q]);
    }
    __syncthreads();
    for (int i = threadIdx.x; i < nw; i += 256) stream[w0 + i] = words[i];
    if (threadIdx.x == 0) {
        table[2 * c] = w0;
        table[2 * c + 1] = static_cast<unsigned>(idx[k]);
    }
}

// Canonical decoding tables: for each length L, the first code, the number
// of codes, and the offset of its symbols in the symbol list; and for the
// next kDecFast bits the symbol of a code no longer than that (its length in
// bits 9..12, 0 when the code is longer).
constexpr int kDecFast = 10;
struct DecTable {
    int first[kEncMaxLen + 1], count[kEncMaxLen + 1], offset[kEncMaxLen + 1];
    int sym[kEncValSyms];
    uint16_t fast[1 << kDecFast];
};
struct __align__(16) DecTables {
    DecTable gap, val;
};

// Reads one chunk's bits in stream order (bit j of the chunk is bit j % 32 of
// its word j / 32).  The lanes of a wave decode different chunks and use up
// words at different times, but a wave waits for all of its loads at once: a
// lane that loaded words when it ran out made the wave wait a memory round
// trip per edit.  So every lane has a ring of kRingWords words in LDS, which
// the whole wave tops up every kRefillEdits edits with loads issued one
// refill earlier.  At least 32 bits wait in buf when a field is taken, so a
// field of up to 30 bits or a code of up to 20 is taken with shifts and one
// bit reversal (fields are emitted most significant bit first).  Bits past the
// chunk's last word read as zeros; the read is then over (more bits taken
// than the chunk has).
constexpr int kDecThreads = 64;   // one wave
constexpr int kRingWords = 64, kRefillWords = 16, kRefillEdits = 4;
// A refill period uses at most 4 edits of 93 bits: 12 words.  The ring holds
// two refills when decoding starts, and from then on each refill adds 16
// words or finds more than 48 - 12 in the ring.
static_assert(kRefillEdits * 93 <= 32 * 12 && 12 < kRefillWords && kRingWords >= 4 * kRefillWords, "the ring never runs dry");

struct BitReader {
    struct __align__(4) Words4 {
        unsigned v[4];
    };
    const unsigned* w;
    unsigned* ring;          // this lane's words, kDecThreads apart
    unsigned next, limit;    // next word to load, end of the stream
    unsigned wr, rd;         // words put into the ring and taken from it
    unsigned p[kRefillWords];
    bool pending;            // p holds loaded words
    unsigned long long buf;  // the next `have` bits, the next one in bit 0
    int have;
    unsigned nw;             // the ring's next word
    __device__ __forceinline__ void init(const unsigned* words, unsigned w0, unsigned stream_words, unsigned* lane_ring) {
        w = words;
        ring = lane_ring;
        next = w0;
        limit = stream_words;
        wr = rd = 0;
        pending = false;
        buf = 0ull;
        have = 0;
        refill();
        refill();
        refill();
        nw = ring[0];
        rd = 1;
    }
    // the loaded words into the ring, the next ones on their way (zeros past
    // the end of the stream; the loads stay below it)
    __device__ __forceinline__ void refill() {
        if (pending) {
#pragma unroll
            for (int k = 0; k < kRefillWords; ++k) ring[((wr + k) % kRingWords) * kDecThreads] = p[k];
            wr += kRefillWords;
        }
        pending = wr + kRefillWords - rd < kRingWords;
        if (!pending) return;
        if (limit - next >= kRefillWords) {  // next <= limit
#pragma unroll
            for (int q = 0; q < kRefillWords / 4; ++q) {
                const Words4 v = *reinterpret_cast<const Words4*>(w + next + 4 * q);
#pragma unroll
                for (int k = 0; k < 4; ++k) p[4 * q + k] = v.v[k];
            }
            next += kRefillWords;
        } else {
#pragma unroll
            for (int k = 0; k < kRefillWords; ++k) p[k] = next < limit ? w[next++] : 0u;
        }
    }
    __device__ __forceinline__ void fill(int n) {  // n <= 32 bits at least
        if (have < n) {
            buf |= static_cast<unsigned long long>(nw) << have;
            have += 32;
            nw = ring[(rd % kRingWords) * kDecThreads];
            ++rd;
        }
    }
    __device__ __forceinline__ void skip(int n) {
        buf >>= n;
        have -= n;
    }
    // bits taken so far
    __device__ __forceinline__ long long taken() const { return 32ll * (rd - 1) - have; }
    // the next n <= 30 bits as a number (first bit most significant)
    __device__ __forceinline__ unsigned bits(int n) {
        fill(n);
        const unsigned v = __brev(static_cast<unsigned>(buf)) >> 1 >> (31 - n);  // n may be 0
        skip(n);
        return v;
    }
};

// -1 on a malformed stream.
__device__ __forceinline__ int decode_symbol(const DecTable& t, BitReader& r) {
    r.fill(kEncMaxLen);
    const unsigned peek = __brev(static_cast<unsigned>(r.buf));  // the next 20 bits at least, first one on top
    const unsigned hit = t.fast[peek >> (32 - kDecFast)];
    if (hit >> 9) {
        r.skip(static_cast<int>(hit >> 9));
        return static_cast<int>(hit & 511u);
    }
    for (int len = kDecFast + 1; len <= kEncMaxLen; ++len) {
        const int rel = static_cast<int>(peek >> (32 - len)) - t.first[len];
        if (rel >= 0 && rel < t.count[len]) {
            r.skip(len);
            return t.sym[t.offset[len] + rel];
        }
    }
    return -1;
}

// One thread per chunk: decodes its edits and writes them into the dense
// (zeroed) output.  Malformed input (a bad code, an index outside [0, n), a
// read past the chunk) sets *bad.  The code tables are staged in LDS.  Bound
// by the chain from one field's position to the next (a chunk's edits follow
// one another): a symbol is one table read on it, where a search over the code
// lengths took two LDS reads per length.  136 us for 804,000 edits in 3,142
// chunks, where that search and loads on demand took 541.
__global__ void __launch_bounds__(kDecThreads) k_dec_chunks(const DecTables* __restrict__ Tg, const unsigned* __restrict__ table,
                                                   const unsigned* __restrict__ stream, unsigned stream_words,
                                                   int nchunks, int m, int n, unsigned* __restrict__ out,
                                                   unsigned* __restrict__ bad) {
    __shared__ DecTables T_s;
    static_assert(sizeof(DecTables) % 16 == 0, "tables copied 16 bytes at a time");
    constexpr int NT = static_cast<int>(sizeof(DecTables) / 16);
#pragma unroll
    for (int k = 0; k < (NT + kDecThreads - 1) / kDecThreads; ++k) {
        const int i = threadIdx.x + kDecThreads * k;
        if (i < NT) reinterpret_cast<uint4*>(&T_s)[i] = reinterpret_cast<const uint4*>(Tg)[i];
    }
    __syncthreads();
    const DecTables* T = &T_s;
    __shared__ unsigned ring[kRingWords * kDecThreads];
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= nchunks) return;
    const unsigned w0 = table[2 * c];
    const unsigned wend = c + 1 < nchunks ? table[2 * (c + 1)] : stream_words;
    if (w0 > wend || wend > stream_words) {
        atomicOr(bad, 1u);
        return;
    }
    BitReader r;
    r.init(stream, w0, stream_words, ring + threadIdx.x);
    const int k_end = min(m, (c + 1) * kEncChunk);
    int i = static_cast<int>(table[2 * c + 1]);  // in [0, n), n < 2^31, at every step
    for (int k = c * kEncChunk; k < k_end; ++k) {
        if (k % kRefillEdits == 0) r.refill();
        r.fill(32);
        if (k != c * kEncChunk) {
            const int b = decode_symbol(T->gap, r);
            if (b < 0 || b > 30) {
                atomicOr(bad, 1u);
                return;
            }
            const int d = static_cast<int>((1u << b) + r.bits(b));  // below 2^31
            if (i < 0 || d > n - 1 - i) {
                atomicOr(bad, 1u);
                return;
            }
            i += d;
        }
        const int e = decode_symbol(T->val, r);
        const unsigned mant = r.bits(23);
        if (e < 0 || i < 0 || i >= n) {
            atomicOr(bad, 1u);
            return;
        }
        out[i] = (static_cast<unsigned>(e) << 23) | mant;
    }
    if (r.taken() > 32ll * (wend - w0)) atomicOr(bad, 1u);
}

// p is 4-byte aligned (a stream starts where the chunk table ends).
__global__ void __launch_bounds__(256) k_enc_fill(unsigned* p, long long nw, unsigned v) {
    for (long long i = blockIdx.x * 256LL + threadIdx.x; i < nw; i += static_cast<long long>(gridDim.x) * 256)
        p[i] = v;
}

// ------------------------------------------------------------ host side ---

// Code lengths of a Huffman code for the counts (0 for absent symbols): the
// two lightest nodes merge first, ties going to the older node (leaves are
// older than internal nodes and ordered by symbol); while the longest code
// exceeds kEncMaxLen every count is halved, rounding up, and the code rebuilt.
std::vector<int> huffman_lengths(std::vector<unsigned long long> f) {
    const int ns = static_cast<int>(f.size());
    std::vector<int> len(ns, 0);
    int present = 0, last = -1;
    for (int s = 0; s < ns; ++s)
        if (f[s]) ++present, last = s;
    if (present == 0) return len;
    if (present == 1) {
        len[last] = 1;
        return len;
    }
    for (;;) {
        typedef std::pair<unsigned long long, int> Node;  // (weight, id): leaves 0..ns-1, then merges
        std::priority_queue<Node, std::vector<Node>, std::greater<Node>> q;
        std::vector<int> parent(2 * ns, -1);
        for (int s = 0; s < ns; ++s)
            if (f[s]) q.push(Node(f[s], s));
        int next = ns;
        while (q.size() > 1) {
            const Node a = q.top();
            q.pop();
            const Node b = q.top();
            q.pop();
            parent[a.second] = next;
            parent[b.second] = next;
            q.push(Node(a.first + b.first, next));
            ++next;
        }
        int longest = 0;
        for (int s = 0; s < ns; ++s) {
            if (!f[s]) continue;
            int d = 0;
            for (int x = s; parent[x] >= 0; x = parent[x]) ++d;
            len[s] = d;
            longest = std::max(longest, d);
        }
        if (longest <= kEncMaxLen) return len;
        for (unsigned long long& x : f)
            if (x) x = (x + 1) >> 1;
    }
}

// Canonical codes from code lengths (symbols ordered by length, then symbol).
void canonical_codes(const std::vector<int>& len, EncCode* out) {
    const int ns = static_cast<int>(len.size());
    std::vector<int> order;
    for (int s = 0; s < ns; ++s)
        if (len[s]) order.push_back(s);
    std::sort(order.begin(), order.end(), [&](int a, int b) { return len[a] != len[b] ? len[a] < len[b] : a < b; });
    unsigned code = 0;
    int prev = order.empty() ? 0 : len[order[0]];
    for (int s = 0; s < ns; ++s) out[s] = EncCode{0u, 0};
    for (size_t k = 0; k < order.size(); ++k) {
        const int s = order[k];
        code <<= (len[s] - prev);
        prev = len[s];
        out[s] = EncCode{code, len[s]};
        ++code;
    }
}

void decode_table(const uint8_t* len, int ns, DecTable& t) {
    std::memset(&t, 0, sizeof(t));
    std::vector<int> order;
    for (int s = 0; s < ns; ++s)
        if (len[s]) order.push_back(s);
    std::sort(order.begin(), order.end(), [&](int a, int b) { return len[a] != len[b] ? len[a] < len[b] : a < b; });
    for (size_t k = 0; k < order.size(); ++k) t.sym[k] = order[k];
    unsigned code = 0;
    int pos = 0;
    for (int L = 1; L <= kEncMaxLen; ++L) {
        int cnt = 0;
        for (int s = 0; s < ns; ++s) cnt += len[s] == L;
        t.first[L] = static_cast<int>(code);
        t.count[L] = cnt;
        t.offset[L] = pos;
        pos += cnt;
        code = (code + cnt) << 1;
    }
    // the shortest matching length wins, as in the search it stands for (the
    // lengths of a malformed header may describe overlapping codes)
    for (int L = 1; L <= kDecFast; ++L) {
        const long long end = std::min<long long>(static_cast<long long>(t.first[L]) + t.count[L], 1ll << L);
        for (long long c = t.first[L]; c < end; ++c)
            for (int e = static_cast<int>(c) << (kDecFast - L); e < static_cast<int>(c + 1) << (kDecFast - L); ++e)
                if (!t.fast[e])
                    t.fast[e] = static_cast<uint16_t>(t.sym[t.offset[L] + (c - t.first[L])] | (L << 9));
    }
}

// Pinned host words of the calling thread for the counts read back (a call
// waits for each copy before it returns).
unsigned* enc_host_words() {
    thread_local unsigned* p = nullptr;
    if (!p) {
        void* q = nullptr;
        if (hipHostMalloc(&q, 4 * (kEncGapSyms + kEncValSyms), hipHostMallocDefault) != hipSuccess) {
            (void)hipGetLastError();  // said by the result
            return nullptr;
        }
        p = static_cast<unsigned*>(q);
    }
    return p;
}

size_t enc_bound(long long n, long long m) {
    const long long chunks = (m + kEncChunk - 1) / kEncChunk;
    const long long edit_bits_max = kEncMaxLen + 30 + kEncMaxLen + 23;
    return static_cast<size_t>(kEncHeader + 8 * chunks + 4 * (chunks + (m * edit_bits_max + 31) / 32));
}

}  // namespace msz

using namespace msz;

extern "C" {

size_t msz_edits_bound(int64_t n) {
    if (n < 0 || n >= (int64_t(1) << 31)) return 0;
    return enc_bound(n, n);
}

int msz_encode_edits(const float* edits, int64_t n, void* out, size_t capacity, size_t* out_bytes,
                     msz_edit_stats* st, void* stream) {
    if (!edits || !out || !out_bytes || n < 0 || n >= (int64_t(1) << 31)) return MSZ_EINVAL;
    if ((reinterpret_cast<uintptr_t>(edits) & 15u) || (reinterpret_cast<uintptr_t>(out) & 15u)) return MSZ_EINVAL;
    hipStream_t s = static_cast<hipStream_t>(stream);
    const unsigned* bits = reinterpret_cast<const unsigned*>(edits);
    const int nblocks = static_cast<int>((n + kEncBlock - 1) / kEncBlock);
    // scratch in two parts: the block offsets (+ total), then, once the number
    // of edits is known, indices, values, chunk words (+ total), histograms
    // and tables
    Scratch first, rest;
    if (int rc = first.get(nullptr, 0, 4 * (static_cast<size_t>(nblocks) + 1), s)) return rc;
    auto fail = [&](int rc) {
        (void)hipStreamSynchronize(s);
        return rc;
    };
    unsigned* off = static_cast<unsigned*>(first.p);
    unsigned* host = enc_host_words();
    if (!host) return MSZ_ENOMEM;
    unsigned m = 0;
    if (nblocks > 0) {
        hipLaunchKernelGGL(k_enc_count, dim3(nblocks), dim3(256), 0, s, bits, static_cast<long long>(n), off);
        hipLaunchKernelGGL(k_enc_scan, dim3(1), dim3(1024), 0, s, off, nblocks);
        if (hipMemcpyAsync(host, off + nblocks, 4, hipMemcpyDeviceToHost, s) != hipSuccess ||
            hipStreamSynchronize(s) != hipSuccess)
            return fail(MSZ_EDEVICE);
        m = host[0];
    }
    // word offsets are 32-bit: the stream of m edits (at most 93 bits each) must fit
    if (static_cast<unsigned long long>(m) * 93ull / 32ull + static_cast<unsigned long long>(m) / kEncChunk + 2 >
        0xFFFFFFFFull)
        return fail(MSZ_EINVAL);
    const int nchunks = static_cast<int>((m + kEncChunk - 1) / kEncChunk);
    size_t o = 0;
    auto take = [&](size_t b) {
        const size_t r = o;
        o += (b + 255) & ~size_t(255);
        return r;
    };
    const size_t room = m;
    const size_t o_idx = take(4 * room), o_val = take(4 * room),
                 o_cw = take(4 * (room / kEncChunk + 2)), o_hist = take(4 * (kEncGapSyms + kEncValSyms)),
                 o_tab = take(sizeof(EncTables));
    if (m > 0)
        if (int rc = rest.get(nullptr, 0, o, s)) return fail(rc);
    char* scratch = static_cast<char*>(rest.p);
    int* idx = reinterpret_cast<int*>(scratch + o_idx);
    unsigned* val = reinterpret_cast<unsigned*>(scratch + o_val);
    unsigned* cw = reinterpret_cast<unsigned*>(scratch + o_cw);
    unsigned* hist = reinterpret_cast<unsigned*>(scratch + o_hist);
    EncTables* tab = reinterpret_cast<EncTables*>(scratch + o_tab);
    std::vector<unsigned> h(kEncGapSyms + kEncValSyms, 0u);
    if (m > 0) {
        hipLaunchKernelGGL(k_enc_compact, dim3(nblocks), dim3(256), 0, s, bits, static_cast<long long>(n), off, idx,
                           val);
        hipLaunchKernelGGL(k_enc_fill, dim3(1), dim3(256), 0, s, hist, static_cast<long long>(kEncGapSyms + kEncValSyms),
                           0u);
        // few blocks: each adds its counts to the same few global words
        const int hb = std::min(512, static_cast<int>((m + 1023) / 1024));
        hipLaunchKernelGGL(k_enc_hist, dim3(hb), dim3(256), 0, s, idx, val, static_cast<int>(m), hist,
                           hist + kEncGapSyms);
        if (hipMemcpyAsync(host, hist, 4 * h.size(), hipMemcpyDeviceToHost, s) != hipSuccess ||
            hipStreamSynchronize(s) != hipSuccess)
            return fail(MSZ_EDEVICE);
        std::memcpy(h.data(), host, 4 * h.size());
    }
    std::vector<unsigned long long> fg(h.begin(), h.begin() + kEncGapSyms), fv(h.begin() + kEncGapSyms, h.end());
    const std::vector<int> lg = huffman_lengths(fg), lv = huffman_lengths(fv);
    EncTables ht;
    canonical_codes(lg, ht.gap);
    canonical_codes(lv, ht.val);
    unsigned words = 0;
    if (m > 0) {
        if (hipMemcpyAsync(tab, &ht, sizeof(ht), hipMemcpyHostToDevice, s) != hipSuccess) return fail(MSZ_EDEVICE);
        hipLaunchKernelGGL(k_enc_sizes, dim3(nchunks), dim3(256), 0, s, tab, idx, val, static_cast<int>(m), cw);
        hipLaunchKernelGGL(k_enc_scan, dim3(1), dim3(1024), 0, s, cw, nchunks);
        if (hipMemcpyAsync(host, cw + nchunks, 4, hipMemcpyDeviceToHost, s) != hipSuccess ||
            hipStreamSynchronize(s) != hipSuccess)
            return fail(MSZ_EDEVICE);
        words = host[0];
    }
    const size_t bytes = static_cast<size_t>(kEncHeader) + 8ull * nchunks + 4ull * words;
    *out_bytes = bytes;
    if (bytes > capacity) return fail(MSZ_EINVAL);
    std::vector<uint8_t> head(kEncHeader, 0);
    const unsigned fixed[6] = {kEncMagic, kEncVersion, static_cast<unsigned>(n), m, static_cast<unsigned>(nchunks),
                               static_cast<unsigned>(kEncChunk)};
    std::memcpy(head.data(), fixed, sizeof(fixed));
    for (int i = 0; i < kEncGapSyms; ++i) head[24 + i] = static_cast<uint8_t>(lg[i]);
    for (int i = 0; i < kEncValSyms; ++i) head[24 + kEncGapSyms + i] = static_cast<uint8_t>(lv[i]);
    char* ob = static_cast<char*>(out);
    if (hipMemcpyAsync(ob, head.data(), kEncHeader, hipMemcpyHostToDevice, s) != hipSuccess) return fail(MSZ_EDEVICE);
    if (m > 0) {
        unsigned* table = reinterpret_cast<unsigned*>(ob + kEncHeader);
        unsigned* sw = reinterpret_cast<unsigned*>(ob + kEncHeader + 8ull * nchunks);
        hipLaunchKernelGGL(k_enc_write, dim3(nchunks), dim3(256), 0, s, tab, idx, val, static_cast<int>(m), cw, table, sw);
    }
    if (hipGetLastError() != hipSuccess) return fail(MSZ_EDEVICE);
    if (st) {
        st->n = n;
        st->n_edits = m;
        st->bytes = static_cast<int64_t>(bytes);
        st->index_bits = 0;
        st->value_bits = 0;
        // split of the stream bits by field, from the symbol counts and code lengths
        for (int b = 0; b < kEncGapSyms; ++b) st->index_bits += static_cast<int64_t>(h[b]) * (lg[b] + b);
        for (int e = 0; e < kEncValSyms; ++e) st->value_bits += static_cast<int64_t>(h[kEncGapSyms + e]) * (lv[e] + 23);
    }
    if (hipStreamSynchronize(s) != hipSuccess) return MSZ_EDEVICE;
    return MSZ_OK;
}

int msz_decode_edits(const void* in, size_t in_bytes, float* edits_out, int64_t n, void* stream) {
    if (!in || !edits_out || n < 0 || n >= (int64_t(1) << 31) || in_bytes < static_cast<size_t>(kEncHeader))
        return MSZ_EINVAL;
    if ((reinterpret_cast<uintptr_t>(in) & 15u) || (reinterpret_cast<uintptr_t>(edits_out) & 15u)) return MSZ_EINVAL;
    hipStream_t s = static_cast<hipStream_t>(stream);
    std::vector<uint8_t> head(kEncHeader);
    if (hipMemcpyAsync(head.data(), in, kEncHeader, hipMemcpyDeviceToHost, s) != hipSuccess ||
        hipStreamSynchronize(s) != hipSuccess)
        return MSZ_EDEVICE;
    unsigned fixed[6];
    std::memcpy(fixed, head.data(), sizeof(fixed));
    const unsigned m = fixed[3], nchunks = fixed[4];
    if (fixed[0] != kEncMagic || fixed[1] != kEncVersion || fixed[2] != static_cast<unsigned>(n) ||
        fixed[5] != static_cast<unsigned>(kEncChunk) || nchunks != (m + kEncChunk - 1) / kEncChunk || m > fixed[2])
        return MSZ_EINVAL;
    if (in_bytes < static_cast<size_t>(kEncHeader) + 8ull * nchunks) return MSZ_EINVAL;
    const size_t stream_words = (in_bytes - kEncHeader - 8ull * nchunks) / 4;
    DecTables dt;
    for (int i = 0; i < kEncGapSyms + kEncValSyms; ++i)
        if (head[24 + i] > kEncMaxLen) return MSZ_EINVAL;
    decode_table(head.data() + 24, kEncGapSyms, dt.gap);
    decode_table(head.data() + 24 + kEncGapSyms, kEncValSyms, dt.val);
    Scratch ws;
    if (int rc = ws.get(nullptr, 0, 512 + sizeof(DecTables), s)) return rc;
    unsigned* host = enc_host_words();
    if (!host) return MSZ_ENOMEM;
    char* scratch = static_cast<char*>(ws.p);
    unsigned* bad = reinterpret_cast<unsigned*>(scratch);
    DecTables* tp = reinterpret_cast<DecTables*>(scratch + 256);
    unsigned* outw = reinterpret_cast<unsigned*>(edits_out);
    hipLaunchKernelGGL(k_enc_fill, dim3(1), dim3(256), 0, s, bad, 1LL, 0u);
    hipLaunchKernelGGL(k_enc_fill, dim3(std::max(1, std::min(4096, static_cast<int>((n + 255) / 256)))), dim3(256), 0, s,
                       outw, static_cast<long long>(n), 0u);
    int rc = MSZ_OK;
    if (hipMemcpyAsync(tp, &dt, sizeof(dt), hipMemcpyHostToDevice, s) != hipSuccess) rc = MSZ_EDEVICE;
    if (rc == MSZ_OK && nchunks > 0) {
        const char* ib = static_cast<const char*>(in);
        hipLaunchKernelGGL(k_dec_chunks, dim3((nchunks + kDecThreads - 1) / kDecThreads), dim3(kDecThreads), 0, s, tp,
                           reinterpret_cast<const unsigned*>(ib + kEncHeader),
                           reinterpret_cast<const unsigned*>(ib + kEncHeader + 8ull * nchunks),
                           static_cast<unsigned>(stream_words), static_cast<int>(nchunks), static_cast<int>(m),
                           static_cast<int>(n), outw, bad);
        if (hipGetLastError() != hipSuccess) rc = MSZ_EDEVICE;
    }
    if (rc == MSZ_OK && (hipMemcpyAsync(host, bad, 4, hipMemcpyDeviceToHost, s) != hipSuccess)) rc = MSZ_EDEVICE;
    if (hipStreamSynchronize(s) != hipSuccess) rc = MSZ_EDEVICE;
    if (rc == MSZ_OK && host[0]) rc = MSZ_EINVAL;
    return rc;
}

}  // extern "C"
