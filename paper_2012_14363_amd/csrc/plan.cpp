#include "plan.hpp"

#include <algorithm>
#include <initializer_list>
#include <limits>
#include <cstdio>

#include "status.hpp"

namespace tp {

namespace {

constexpr int64_t kPageBytes = 4096;  // rows at least this far apart each need their own address translation
constexpr int64_t kLineBytes = 128;   // memory line: what a partial write is read-modify-written in
constexpr int64_t kSoloRows = int64_t{1} << 20, kSoloBytes = int64_t{8} << 20;  // batch requests worth their own launch
constexpr int64_t kManyRows = 128, kManyBytes = int64_t{1} << 20;   // requests whose memory traffic, not latency, decides
constexpr int64_t kFillBytes = int64_t{4} << 20;  // more than 1024 workgroups of one 16-byte word per thread: four for each CU
constexpr int64_t kKeepBytes = int64_t{64} << 20; // a quarter of the Infinity Cache
constexpr int64_t kStagedRows = int64_t{1} << 19;  // fewer rows do not repay the extra passes (2^18: 15.0 against 14.5 us; 2^19: 22 against 26)
// Workgroups of a staged launch: a multiple of the eight XCDs.  Measured on 64 MiB of rows at 512-byte pitch, us for
// 96 / 128 / 160 / 192 / 224 / 256 / 320 workgroups: 1-byte rows 1766 / 1779 / 1777 / 1750 / 1779 / 1784 / 2097, 2-byte rows
// 894 / 902 / 892 / 882 / 906 / 971 / -, 8-byte rows 244 / 249 / 243 / 241 / 246 / 259 / -: a flat optimum from 168 to 208.
constexpr uint32_t kStagedGrid = 192;
const FastDiv kDivideByOne = make_fastdiv(1);
constexpr uint32_t kPrefetchGridFactor = 8;        // the read-only pass takes that many times more

struct Dim {
    int64_t count;
    int64_t stride;
};

// The dimensions of a request, innermost first: a StridedBlock's and the object count.  Planning runs on every
// call, so it works in place: no allocations, and launches are filled in where they are kept.
class Dims {
public:
    Dims() = default;
    Dims(std::initializer_list<Dim> init) {
        for (const Dim& d : init) push_back(d);
    }
    void push_back(const Dim& d) { d_[n_++] = d; }
    void pop_back() { --n_; }
    size_t size() const { return n_; }
    Dim& operator[](size_t i) { return d_[i]; }
    const Dim& operator[](size_t i) const { return d_[i]; }
    Dim& back() { return d_[n_ - 1]; }
    const Dim& back() const { return d_[n_ - 1]; }

private:
    size_t n_ = 0;
    Dim d_[kMaxDims + 1];
};

int ceil_log2(uint64_t v) { return v <= 1 ? 0 : 64 - __builtin_clzll(v - 1); }

// Thread-tile shape for runs of n0 words (Sec. 3.3 maps X to the run and fills the
// block with further rows; here the block is flat and the split is a power of two).
// Runs longer than the workgroup are cut into chunks of 256 * ux words; of ux = 1, 2, 4 the one
// that pads the run least wins (1025 words: five chunks of 256 rather than two of 1024), the
// larger on a tie since its row arithmetic is scalar.
// `ur_short`: rows per thread (1 or 4) where a run fits the workgroup.
struct TileShape {
    uint32_t bx_log2;
    int ux, ur;
};

TileShape choose_tile(uint32_t n0, int ur_short) {
    if (n0 <= static_cast<uint32_t>(kBlockThreads)) return {static_cast<uint32_t>(ceil_log2(n0)), 1, ur_short};
    TileShape t{8, 1, 4};
    uint64_t best = ~uint64_t{0};
    for (int ux : {4, 2, 1}) {
        const uint64_t chunk = static_cast<uint64_t>(kBlockThreads) * ux;   // a power of two
        const uint64_t padded = (n0 + chunk - 1) & ~(chunk - 1);
        if (padded < best) {
            best = padded;
            t.ux = ux;
        }
    }
    // One row per thread asked for: one word too, unless chunks of 256 would leave a quarter of their lanes idle and
    // wider ones no more of them (313 words: 25 us in single words, 21 in tiles of two words by two rows).
    if (ur_short == 1 && (t.ux == 1 || n0 * 4 >= best * 3)) t.ux = t.ur = 1;
    else t.ur = 4 / t.ux;
    return t;
}

// Chunks along a run of n0 words, and row chunks over `rows` (the tile's edges are powers of two).
uint64_t chunks_along(const TileShape& t, uint64_t n0) {
    const uint32_t log2 = t.bx_log2 + static_cast<uint32_t>(t.ux >> 1);   // ux 1, 2, 4
    return (n0 + (uint64_t{1} << log2) - 1) >> log2;
}
uint64_t row_chunks(const TileShape& t, uint64_t rows) {
    const uint32_t log2 = 8 - t.bx_log2 + static_cast<uint32_t>(t.ur >> 1);
    return (rows + (uint64_t{1} << log2) - 1) >> log2;
}
static_assert(kBlockThreads == 1 << 8, "row_chunks");

struct Splitter {
    const PlanInput& in;
    int word_log2;
    int64_t row_pitch;  // bytes of a full run in the packed stream
    std::vector<Launch>* out;
    int ur_short = 4;   // rows per thread in tiles for runs that fit the workgroup
    int nt = 3;         // streaming hints of the launches
    uint32_t grid = 0;  // workgroups per launch (0 = one per tile)
    int64_t chunk_rows = 0;  // > 0: no launch of more rows (staged unpack)

    int64_t word() const { return int64_t{1} << word_log2; }
    // Words that cover a run of `bytes` (>= one word): the last one may overlap its neighbour.
    uint32_t words(int64_t bytes) const { return static_cast<uint32_t>((bytes + word() - 1) >> word_log2); }

    // One launch over dims[0..nd): dims[0].count bytes per run.
    void add(const Dims& dims, const char* typed, char* packed) {
        out->emplace_back();
        Launch& l = out->back();
        l.word_log2 = word_log2;
        KParams& p = l.p;
        p.strided = typed;
        p.packed = packed;
        p.row_pitch = row_pitch;
        p.n0 = words(dims[0].count);
        p.tail_back = static_cast<uint32_t>((static_cast<int64_t>(p.n0) << word_log2) - dims[0].count);
        uint64_t rows = 1;
        p.nrd = 0;
        for (size_t d = 1; d < dims.size(); ++d) {
            if (dims[d].count == 1) continue;
            p.rcount[p.nrd] = static_cast<uint32_t>(dims[d].count);
            p.rstride[p.nrd] = dims[d].stride;
            p.rdiv[p.nrd] = make_fastdiv(p.rcount[p.nrd]);
            ++p.nrd;
            rows *= static_cast<uint64_t>(dims[d].count);
        }
        p.nrows = static_cast<uint32_t>(rows);
        const TileShape t = choose_tile(p.n0, ur_short);
        p.bx_log2 = t.bx_log2;
        l.ux = t.ux;
        l.ur = t.ur;
        l.nt = nt;
        p.nxc = static_cast<uint32_t>(chunks_along(t, p.n0));
        p.xc_div = make_fastdiv(p.nxc);
        l.nblocks = static_cast<uint32_t>(row_chunks(t, rows) * p.nxc);
        if (grid) l.grid = std::min(grid, l.nblocks);
        else if (l.nblocks > kMaxGrid) l.grid = kMaxGrid;   // more tiles than a grid may have workgroups
    }

    // Largest row count for which block ids stay below 2^30 with runs of n0 words.
    int64_t row_limit(int64_t n0) const {
        const TileShape t = choose_tile(static_cast<uint32_t>(n0), ur_short);
        const int64_t nxc = static_cast<int64_t>(chunks_along(t, static_cast<uint64_t>(n0)));
        const int64_t by_blocks = ((int64_t{1} << 30) / nxc) * (kBlockThreads >> t.bx_log2) * t.ur;
        const int64_t limit = std::min(in.max_rows_per_launch, by_blocks);
        return std::max<int64_t>(1, chunk_rows > 0 ? std::min(limit, chunk_rows) : limit);
    }

    // Rows: split the outermost dimension until a launch's row count fits.
    void split_rows(const Dims& dims, const char* typed, char* packed) {
        int64_t rows = 1;
        for (size_t d = 1; d < dims.size(); ++d) rows *= dims[d].count;
        const uint32_t n0 = words(dims[0].count);
        // (the first comparison spares nearly every call the limit's division)
        const bool few = rows <= (int64_t{1} << 20) && n0 <= static_cast<uint32_t>(kBlockThreads) && rows <= in.max_rows_per_launch &&
                         chunk_rows == 0;
        const int64_t limit = few ? rows : row_limit(n0);
        if (rows <= limit) {
            add(dims, typed, packed);
            return;
        }
        const Dim top = dims.back();
        const int64_t inner_rows = rows / top.count;
        const int64_t chunk = std::max<int64_t>(1, limit / inner_rows);
        for (int64_t i = 0; i < top.count; i += chunk) {
            const int64_t k = std::min(chunk, top.count - i);
            Dims sub = dims;
            if (inner_rows > limit) sub.pop_back(); else sub.back().count = k;
            split_rows(sub, typed + i * top.stride, packed + i * inner_rows * row_pitch);
        }
    }

    // Runs longer than the per-launch word limit are cut into pieces along dimension 0.  A piece
    // is a run of its own and needs at least one word, so a last piece shorter than that starts
    // early instead and overlaps the piece before it (same bytes written twice).
    void split_runs(const Dims& dims, const char* typed, char* packed) {
        const int64_t piece = in.max_words_per_run << word_log2;
        const int64_t total = dims[0].count;
        for (int64_t off = 0; off < total; off += piece) {
            int64_t at = off, len = std::min(piece, total - off);
            if (len < word()) {
                at = total - word();
                len = word();
            }
            if (len == total) {
                split_rows(dims, typed, packed);
                return;
            }
            Dims sub = dims;
            sub[0].count = len;
            split_rows(sub, typed + at, packed + at);
        }
    }
};

// The transposing kernel (plan.hpp: XParams) applies when the elements are short runs (a few
// words of the widest power of two dividing their length) and some outer row dimension A steps
// by exactly one element while the innermost row dimension B strides over at least two.  Returns false (and leaves `out` alone) when it does not apply or the launch would not
// fit one grid.
bool plan_xpose(const PlanInput& in, const Dims& dims, const char* typed, std::vector<Launch>* out) {
    if (!in.allow_xpose || dims.size() < 3) return false;
    const int64_t run = dims[0].count;
    if (run > 64) return false;
    const int word_log2 = std::min({4, in.max_word_log2, __builtin_ctzll(static_cast<uint64_t>(run))});
    const int64_t ew = run >> word_log2;
    // Edge of a square tile, in elements: one-word elements use the power of two the kernel's
    // constant-parameter variant is built for; elements of several words take the largest edge
    // whose rows fit the workgroup (256 words) and whose tile fits LDS.
    const int64_t lds_words = xpose_lds_words(word_log2);
    int64_t square = xpose_fast_words(word_log2);
    if (ew > 1) {
        square = kBlockThreads / ew;
        while (square > 0 && square * (square * ew + 32) > lds_words) --square;
    }
    if (square < 12) return false;
    // tests that lower the split limits mean the row-by-row kernel
    if (in.max_rows_per_launch != (int64_t{1} << 30) || in.max_words_per_run != (int64_t{1} << 30)) return false;
    const Dim& b = dims[1];
    size_t a = 0;
    for (size_t d = 2; d < dims.size() && a == 0; ++d)
        if (dims[d].stride == run && dims[d].count >= 2) a = d;
    if (a == 0) return false;
    // A dimension of very few elements (records of two or three fields): the row-by-row kernel's
    // re-reads mostly hit in cache, and tiles that thin give a workgroup little to do.  Measured on
    // 4 Mi records of 8-byte fields, row by row against transposing, pack / unpack in us: three fields
    // 72 / 120 against 84 / 87, four fields 110 / 224 against 86 / 89, eight 376 / 876 against 108 / 111.
    const int64_t thin = std::min(dims[a].count, b.count);
    if (thin < (in.unpack ? 3 : 4)) return false;
    // Walking B row by row uses one element of every |stride| bytes and comes back for the rest
    // on later rows: worth transposing from an amplification of two, given enough elements.
    const int64_t bstep = b.stride < 0 ? -b.stride : b.stride;
    if (bstep < 2 * run || dims[a].count * b.count < 1024) return false;

    // Tile shape: square where both dimensions are long; a dimension shorter than half an edge is
    // covered whole and the other edge grows (as far as LDS reaches), so that a workgroup still
    // has tens of KiB to move.
    int64_t te_a = std::min<int64_t>(square, dims[a].count), te_b = std::min<int64_t>(square, b.count);
    // LDS row pitch in words: at least a tile row, and such that lanes walking down a tile
    // column fall into distinct banks (32 of them): any odd pitch for one-word elements, a pitch
    // congruent to ew modulo 32 for elements of ew words.
    auto pitch_for = [ew](int64_t edge_a) {
        uint32_t pitch = static_cast<uint32_t>(edge_a * ew);
        if (ew == 1) return pitch | 1u;
        while (pitch % 32 != static_cast<uint32_t>(ew % 32)) ++pitch;
        return pitch;
    };
    uint32_t pitch = pitch_for(te_a);
    constexpr int64_t kLongEdge = 1024;  // elements along the grown edge of a thin tile, at most
    // a grown edge beyond one chunk of lanes is a whole number of chunks
    auto whole_chunks = [ew](int64_t edge) {
        const int64_t chunk = kBlockThreads / ew;
        return edge > chunk ? edge / chunk * chunk : edge;
    };
    if (te_a * 2 <= square) te_b = whole_chunks(std::min({b.count, kLongEdge, lds_words / pitch}));
    else if (te_b * 2 <= square) {
        te_a = whole_chunks(std::min({dims[a].count, kLongEdge, (lds_words / te_b - 32) / ew}));
        if (te_a < 1) return false;
        pitch = pitch_for(te_a);
    }
    if (te_b * pitch > lds_words) return false;

    Launch l;
    l.kind = kXpose;
    l.word_log2 = word_log2;
    l.nt = 3;
    XParams& x = l.x;
    x.strided = typed;
    x.packed = in.packed;
    x.ca = static_cast<uint32_t>(dims[a].count);
    x.cb = static_cast<uint32_t>(b.count);
    x.ew = static_cast<uint32_t>(ew);
    x.te_a = static_cast<uint32_t>(te_a);
    x.te_b = static_cast<uint32_t>(te_b);
    x.fa_log2 = static_cast<uint32_t>(std::min(8, ceil_log2(static_cast<uint64_t>(te_a * ew))));
    x.fb_log2 = static_cast<uint32_t>(std::min(8, ceil_log2(static_cast<uint64_t>(te_b * ew))));
    x.pitch = pitch;
    x.tb_stride = b.stride;
    x.tiles_a = static_cast<uint32_t>((dims[a].count + te_a - 1) / te_a);
    x.tiles_b = static_cast<uint32_t>((b.count + te_b - 1) / te_b);
    x.tiles_a_div = make_fastdiv(x.tiles_a);
    x.tiles_b_div = make_fastdiv(x.tiles_b);
    // packed bytes per step of row dimension d: one element times the counts nested inside it
    int64_t pstride = run;
    uint64_t blocks = static_cast<uint64_t>(x.tiles_a) * x.tiles_b;
    for (size_t d = 1; d < dims.size(); ++d) {
        if (d == a) {
            x.pa_stride = pstride;
        } else if (d != 1 && dims[d].count != 1) {
            x.ocount[x.nod] = static_cast<uint32_t>(dims[d].count);
            x.odiv[x.nod] = make_fastdiv(x.ocount[x.nod]);
            x.otstride[x.nod] = dims[d].stride;
            x.opstride[x.nod] = pstride;
            ++x.nod;
            blocks *= static_cast<uint64_t>(dims[d].count);
            if (blocks > kMaxGrid) return false;
        }
        pstride *= dims[d].count;
    }
    if (blocks > kMaxGrid) return false;   // one tile per workgroup
    l.nblocks = static_cast<uint32_t>(blocks);
    // Sources that stay in the Infinity Cache, as for the row-by-row launches (plan_launches): 4096 x 4096 float32 by
    // columns, 64 MiB, 31.0 -> 24.4 us together with the unchecked whole tiles.
    int64_t footprint = pstride;
    if (!in.unpack) {
        const int64_t strip = dims[a].count * run;
        footprint = pstride / strip * std::min(bstep, (strip + kLineBytes - 1) / kLineBytes * kLineBytes);
    }
    l.keep = in.nt < 0 && !(in.unpack && in.packed_on_host) && footprint <= kKeepBytes;
    out->push_back(l);
    return true;
}

// Staged unpack of tiny rows.  Partially written memory lines retire about 1.5 times faster when
// (a) the lines written at one time are exactly 512 bytes apart and (b) no read from HBM falls
// between the writes (measured with one-byte rows: 37 G rows/s against 19 to 25 G at any other
// spacing from 64 to 4096 bytes, and against 22 G with the source streamed from HBM; 64 MiB of
// one-byte rows at 512-byte pitch unpack in 1.8 ms instead of 2.7).  For rows of one word each at a
// pitch of 512 bytes, or of 256 or 128 taken in 2 or 4 passes over every 2nd or 4th row, the
// launch is therefore cut into chunks of `stage_bytes` packed bytes, and every chunk becomes a
// read-only pass that brings its packed bytes into L2 followed by the store passes, all with the
// same few workgroups taking the same tiles: workgroup ids map to XCDs round-robin, so a tile's
// bytes wait in the L2 its stores will ask.  Returns false where this does not apply.
bool plan_staged(const PlanInput& in, const Dims& all_dims, const char* typed, std::vector<Launch>* out) {
    Dims dims = {all_dims[0]};
    for (size_t d = 1; d < all_dims.size(); ++d)
        if (all_dims[d].count != 1) dims.push_back(all_dims[d]);   // a dimension of one row is none
    if (dims.size() < 2) return false;
    const int64_t run = dims[0].count, pitch = dims[1].stride;
    int64_t rows = 1;
    for (size_t d = 1; d < dims.size(); ++d) rows *= dims[d].count;
    const int64_t step = pitch < 0 ? -pitch : pitch;
    if (run > 16 || (run & (run - 1)) != 0 || (int64_t{1} << in.max_word_log2) < run) return false;
    if (step != 128 && step != 256 && step != 512) return false;
    if (dims.size() > 2 && step != 512) return false;   // passes over every 2nd or 4th row: one row dimension only
    // rows in the last of the four lines of their 512-byte block do not reach the fast rate (measured: a
    // column of 8-byte elements at byte 384 or beyond of 512-byte matrix rows unpacks as without staging)
    if (step == 512 && in.stage != 1 && (reinterpret_cast<uintptr_t>(typed) & 511u) >= 384u) return false;
    if (in.stage != 1 && rows < kStagedRows) return false;
    if (in.max_rows_per_launch != (int64_t{1} << 30) || in.max_words_per_run != (int64_t{1} << 30)) return false;
    const int64_t passes = 512 / step;
    // the passes give up the locality of neighbouring rows, which costs more the more of each line the
    // rows fill: measured to pay for 1- to 16-byte rows at 512-byte pitch, up to 4 bytes at 256, 1 byte at 128
    if (run * passes * passes > 16) return false;
    const int64_t tile_rows = int64_t{kBlockThreads} * passes;  // rows of all passes that share one tile index
    // tile_rows * run bytes per tile: a power of two, at least 256
    int64_t chunk_rows = std::max<int64_t>(in.stage_bytes / run, 1) / tile_rows * tile_rows;
    if (chunk_rows == 0) chunk_rows = tile_rows;
    const uint32_t grid = in.stage_grid > 0 ? static_cast<uint32_t>(in.stage_grid) : kStagedGrid;
    int word_log2 = 0;
    while ((int64_t{1} << word_log2) < run) ++word_log2;
    auto add_prefetch = [&](const char* base, int64_t nrows) {
        if (nrows * run < 16) return;   // the read-only pass loads 16-byte words
        Launch l;
        l.kind = kPrefetch;
        l.f.base = base;
        l.f.bytes = static_cast<uint64_t>(nrows * run);
        l.f.tile_bytes = static_cast<uint32_t>(tile_rows * run);
        l.f.ntiles = static_cast<uint32_t>((nrows + tile_rows - 1) / tile_rows);
        l.nblocks = l.f.ntiles;
        // more workgroups than the store passes have (the read is over sooner), still a multiple of the
        // eight XCDs, so tile t lands on XCD t mod 8 here as there
        l.grid = std::min(grid * kPrefetchGridFactor, l.nblocks);
        out->push_back(l);
    };
    if (dims.size() > 2) {
        // several row dimensions (512-byte pitch, one pass): the splitter cuts the outer dimensions into
        // launches of at most a chunk's rows, consecutive in the packed stream; each gets its pass in front
        std::vector<Launch> cut;
        Splitter s{in, word_log2, run, &cut, 1, in.nt >= 0 ? in.nt : 6, grid, chunk_rows};
        s.split_rows(dims, typed, in.packed);
        for (const Launch& l : cut) {
            add_prefetch(l.p.packed, static_cast<int64_t>(l.p.nrows));
            out->push_back(l);
        }
        return true;
    }
    for (int64_t lo = 0; lo < rows; lo += chunk_rows) {
        const int64_t n = std::min(chunk_rows, rows - lo);
        add_prefetch(in.packed + lo * run, n);
        for (int64_t p = 0; p < passes && p < n; ++p) {
            // rows lo + p, lo + p + passes, ...: `passes` rows apart on both sides
            Splitter s{in, word_log2, run * passes, out, 1, in.nt >= 0 ? in.nt : 6, grid};
            const Dims sub = {{run, 1}, {(n - p + passes - 1) / passes, pitch * passes}};
            s.add(sub, typed + (lo + p) * pitch, in.packed + (lo + p) * run);
        }
    }
    return true;
}

}  // namespace

int plan_launches(const PlanInput& in, std::vector<Launch>* out) {
    out->clear();
    const StridedBlock& sb = in.block;
    if (in.count == 0 || sb.counts[0] == 0) return kSuccess;

    Dims dims;
    for (int d = 0; d < sb.ndims; ++d) dims.push_back({sb.counts[d], sb.strides[d]});
    // The object count is one more outer dimension of stride `extent` (Sec. 3.3 handles it
    // with the grid's Z dimension); fold or flatten it away when objects abut.
    if (in.count > 1) {
        Dim& top = dims.back();
        const int64_t top_span = dims.size() == 1 ? top.count : top.count * top.stride;
        if (in.extent == top_span) top.count *= in.count;
        else dims.push_back({in.count, in.extent});
    }
    if (dims.size() - 1 > static_cast<size_t>(kMaxDims)) return kErrRange;

    // Word width.  Words may sit at any address and need not divide the run (KParams: ragged
    // words, unaligned accesses), so the choice is free of both; measurements decide it.
    // Reading the typed side (pack): 16 bytes wherever a run holds that much - equal to narrower
    // words on runs they divide, up to 20 % faster on the others, and 2-4 times faster than the
    // bytes that natural alignment would force at odd addresses or run lengths.
    // Writing the typed side (unpack): a row that is not made of whole aligned 128-byte lines ends
    // in partially written lines, which the memory system read-modify-writes, and how the row's
    // stores are issued then matters: see the write-through rule below.  Where that rule does not
    // apply, the earlier one holds.  It was measured with plain streaming stores and four rows per
    // thread on 60 MiB of rows at 128- to 8192-byte pitch (4 / 8 / 16-byte words, us): 100-byte rows
    // 34 / 44 / 49, 200: 33 / 40 / 40, 1000: 29 / 33 / 35, but 1040: 34 / 27 / 27, 2056: 30 / 27 / 32,
    // 4100: 27 / 26 / 25: 4-byte words up to 1 KiB and 8-byte words beyond.  Rows of whole aligned
    // lines keep 16.
    const char* typed = in.typed + sb.start;
    if (plan_xpose(in, dims, typed, out)) return kSuccess;
    const int64_t run = dims[0].count;
    int word_log2 = std::min({4, in.max_word_log2, 63 - __builtin_clzll(static_cast<uint64_t>(run))});
    int ur_short = 4, nt = 3;
    // Do the typed rows consist of whole aligned 128-byte memory lines?  How far apart are rows that follow
    // one another in the packed stream (the innermost row dimension), and how close do rows come
    // that are written far apart in time (the outer row dimensions)?
    bool partial_rows = false;
    uint64_t bits = static_cast<uint64_t>(run) | reinterpret_cast<uintptr_t>(typed);
    int64_t inner_pitch = 0, outer_pitch = std::numeric_limits<int64_t>::max();
    // Does a dimension step back into what the ones inside it have walked over (interleaved or overlapping rows)?
    bool revisits = false;
    int64_t reach = run;
    if (dims.size() > 1) {
        for (size_t d = 1; d < dims.size(); ++d) {
            const int64_t step = dims[d].stride < 0 ? -dims[d].stride : dims[d].stride;
            bits |= static_cast<uint64_t>(step);
            if (dims[d].count == 1) continue;
            if (inner_pitch == 0) inner_pitch = step;
            else outer_pitch = std::min(outer_pitch, step);
            if (step < reach) revisits = true;
            reach = std::max(reach, step * dims[d].count);
        }
        partial_rows = (bits & static_cast<uint64_t>(kLineBytes - 1)) != 0;
    }
    // A request of a batch call keeps a plan the batched kernel can run unless it is large enough
    // for a launch of its own to pay (a launch costs about 5 us on the stream).
    int64_t rows = 1;
    for (size_t d = 1; d < dims.size(); ++d) rows *= dims[d].count;
    const int64_t bytes = rows * run;
    const bool own_launch = !in.batched || rows >= kSoloRows || bytes >= kSoloBytes;
    const bool tuned = !in.batched && !in.packed_on_host && in.unpack_rule == 1;
    const bool through = in.unpack && !in.packed_on_host && in.unpack_rule == 1 && in.narrow_partial_rows && partial_rows &&
                         inner_pitch < kPageBytes && outer_pitch >= kLineBytes && own_launch;
    if (through && in.stage != 0 && plan_staged(in, dims, typed, out)) return kSuccess;
    if (in.unpack && tuned && in.narrow_partial_rows && partial_rows && outer_pitch >= kLineBytes && rows >= kManyRows &&
        bytes >= kManyBytes) {
        // Many rows that end in partially written memory lines.  Measured on 4, 16, 24, 56 and 64 MiB of rows of 1 to 65536
        // bytes at pitches from one byte above the run to 12 KiB, with every word, one and four rows per thread, and
        // streaming (`nt`) or written-through (`sc1 nt`) stores.  Pairs joined by "and" are 16 MiB unless said
        // otherwise, with sources from the Infinity Cache and from HBM behind a kernel that filled it with other data.
        //   Do rows lie so far apart that L2 has little to merge: 64 bytes, or, beyond 4 MiB, eight times the run (1 at 17
        // bytes, written through 111 and 114, streaming 129 and 138; 3 at 39: 85 and 89, 97 and 102; but 4 MiB of 2 at 16
        // 16.0 and 17.2, 12.0 and 17.8)?
        const bool apart = inner_pitch >= kLineBytes / 2 || (inner_pitch >= 8 * run && bytes > kFillBytes);
        //   Stores: written through L2 at once where a line holds at most two rows and rows are short (128-byte
        // pitch, 64 MiB: 12-byte rows 139 us against 195 streaming, 24: 72 / 100, 48: 41 / 53; 1-KiB pitch,
        // 256-byte rows 39.6 / 42.6).  Streaming where neighbouring rows share their lines, so that L2 can merge
        // them (12-byte rows at 13: 46 / 132, 24 at 25: 40 / 71, 64 at 67: 35 / 38), and for rows beyond 1 KiB
        // (2408 bytes at 4096: 24.8 / 27.3); but for rows of half a line and more only beyond 4 MiB, since what L2 still
        // holds when a kernel ends is written then (4 MiB, written through / streaming: 96 at 112 6.0 / 6.7, 128 at 129
        // 5.9 / 6.7, 1500 at 1501 5.8 / 6.6) and rows fit the workgroup, one word to a thread.
        const bool streams = bytes > kFillBytes || run < kLineBytes / 2;
        const bool shared_lines = !apart || (inner_pitch >= kLineBytes / 2 && inner_pitch < kLineBytes * 3 / 2 && inner_pitch - run < 32 && streams);
        //   One row per thread, except where rows are so close (or, short ones, so far apart: one address
        // translation each) that four are the better (24 at 25: 40 / 47; 24 at 4096: 13.1 / 16.5).
        ur_short = (run <= 32 && !apart) || (run < 64 && inner_pitch >= kPageBytes) ? 4 : 1;
        nt = ur_short == 1 && !shared_lines && (run <= 1024 || (!streams && run <= kBlockThreads * 16)) ? 7 : 3;
        //   Word.  Rows of at least a line: 16 bytes (200 at 216, words of 8 and of 16: 12.2 and 15.4, 9.3 and 13.3; 192 at 228:
        // 12.8 and 15.4, 9.5 and 13.7), or 8 for rows of at most two lines at odd addresses and 384 bytes or more apart
        // (128 at 768: 14.0 and 20.3, 16.5 and 22.8; 56 MiB, 200 at 384: 21.2 and 39.0, 24.6 and 43.8).
        //   Shorter rows: 5 to 8 lanes on a row where a line holds parts of two rows (words of 1, 2 and 4 bytes: 8 at 128
        // 52 and 57, 78 and 80, 77 and 82; 16 at 128 43 and 47, 28 and 33, 38 and 43; words of 4 and 8: 48 at 160 18.4 and 22.2,
        // 17.1 and 22.6), 9 to 16 beyond (24 at 256, words of 2 and 4: 20.3 and 30.4, 23.6 and 30.4; 100 at 512, 4, 8 and 16: 11.6
        // and 17.5, 9.9 and 16.5, 13.0 and 18.7) and 8 on whole aligned 64-byte blocks (64 at 512, words of 4 / 8 / 16: 43.6 /
        // 30.3 / 32.7).  No less than 4 bytes for rows closer than that (12 at 13, words of 1 and 4: 13.4 and 20.2, 12.6 and 15.8)
        // and for those so far apart that their translations decide (4 MiB, 16 at 1024: 14.0 and 16.5, 14.7 and 15.4).
        const int64_t two_rows = run <= 32 ? 2 * kLineBytes : kLineBytes * 3 / 2;
        const int64_t lanes = (bits & 63) == 0 || (inner_pitch < two_rows && (apart || run > 32)) ? 8 : 16;
        int by_lanes = ceil_log2(static_cast<uint64_t>((run + lanes - 1) / lanes));
        if (run >= kLineBytes) by_lanes = (bits & 15) != 0 && inner_pitch >= 3 * kLineBytes && run <= 2 * kLineBytes ? 3 : 4;
        else if (run >= 4 && (!apart || (run >= 16 && inner_pitch >= 1024))) by_lanes = std::max(2, by_lanes);
        word_log2 = std::min(word_log2, by_lanes);
    } else if (through) {
        // Fewer rows than that, closer than a page, that share no line with rows of another outer index: written through
        // L2 at once as well, one row per thread, a row spread over 8 to 15 lanes (32 MiB of rows at 512-byte pitch,
        // against four rows per thread and streaming stores in 4-byte words, us: 12-byte rows 130 -> 112, 48: 39 -> 32,
        // 100: 31 -> 23, 200: 20.4 -> 18.7).
        nt = 7;
        ur_short = 1;
        const int eighth_log2 = run >= 16 ? 63 - __builtin_clzll(static_cast<uint64_t>(run / 8)) : 0;
        word_log2 = std::min(word_log2, eighth_log2);
    } else {
        if (in.unpack && in.narrow_partial_rows && partial_rows) word_log2 = std::min(word_log2, run <= 1024 ? 2 : 3);
        // Reading mapped host memory across PCIe (zero-copy unpack): 16-byte loads were measured
        // slower than 8- or 4-byte ones (4 MiB: 115 us against 87; 64 MiB: 1270 against 1180), writes
        // to it do not care.
        if (in.unpack && in.packed_on_host) word_log2 = std::min(word_log2, 3);
        // Runs of at most 32 bytes: every run costs a whole 128-byte line whatever the word, and a
        // wavefront whose lanes share rows touches fewer lines per instruction.  Measured: gathers run
        // 5-13 % faster with four (or more) lanes per row than with one wide word per row, so cap the
        // word at a quarter of the run, and at 4 bytes.
        if (dims.size() > 1 && run <= 32) {
            const int quarter_log2 = run >= 4 ? 63 - __builtin_clzll(static_cast<uint64_t>(run / 4)) : 0;
            word_log2 = std::min(word_log2, std::min(2, quarter_log2));
        }
        // One word per thread, and so more and shorter workgroups, once there are enough of them to fill the
        // chip several times over: for long runs (64 MiB, us, against four words per thread: dense 24.2 -> 23.7, 1000 bytes at
        // 1024: 25.1 -> 23.8, 2408 at 4096: 28.3 -> 24.3, 9000 at 12288: 27.2 -> 24.5), and when packing from
        // rows far apart (100 at 512: 27.9 -> 26.3), short ones where their distance is a power of two from 512 bytes on (12 at
        // 512: 46 -> 42, 32 at 512: 52 -> 47; but 20 at 1000: 30.3 -> 31.5, 64 MiB of 8 at 1536: 195 -> 219); short rows
        // close together want the four (24 at 64: 39 / 55).
        if (tuned && bytes > kFillBytes && !revisits) {
            const bool apart = inner_pitch >= 2 * kLineBytes && inner_pitch >= 2 * run;
            if (run >= 512 || in.unpack || (apart && (run >= 64 || (inner_pitch >= 512 && inner_pitch < kPageBytes && (inner_pitch & (inner_pitch - 1)) == 0)))) ur_short = 1;
            // whole-line rows written through as well: 128 at 512 24.8 -> 23.8, 512 at 1024 24.6 -> 24.0
            if (in.unpack && !partial_rows && dims.size() > 1 && run <= 512) nt = 7;
        }
    }
    // Loads without the streaming hint leave the source in the Infinity Cache, where the next reader finds it: worth it
    // while the source is a small part of its 256 MiB.  By what ran before, plain against streaming loads (time ratio over 13 shapes
    // of rows of half their pitch or more, pack / unpack): source just written on a cache full of other data, 16 MiB 0.91 / 0.88, 56 MiB
    // 0.81 / 0.78; read again unchanged 0.99 / 0.97, 0.92 / 0.89; from HBM, the cache full of clean lines 1.00 / 0.99, 1.01 / 1.00; from
    // HBM, the cache full of lines other kernels wrote, which what is kept has to push out, 1.26 / 1.20, 1.28 / 1.33.  What is
    // packed has usually just been computed, and what is unpacked received.
    bool keep = false;
    if (in.nt < 0 && !(in.unpack && in.packed_on_host)) {
        int64_t footprint = bytes;   // of the source, in whole memory lines
        if (!in.unpack && dims.size() > 1)
            footprint = inner_pitch < kLineBytes ? rows * std::max(inner_pitch, run)
                                                 : rows * ((run + kLineBytes - 1) / kLineBytes * kLineBytes);
        // sparse rows at wide, even distances share few of the cache's sets: 12 at 2048, 64 MB of lines: 13.5 -> 15.1
        const bool sparse = !in.unpack && inner_pitch >= 512 && run < kLineBytes;
        // memory that the same request comes back to is worth keeping whatever its size (300 nested objects whose boxes
        // overlap: 201 -> 186)
        keep = footprint <= (sparse ? kKeepBytes / 2 : kKeepBytes) || (revisits && !in.unpack);
    }
    if (in.nt >= 0) nt = in.nt;
    if (in.max_ur == 1 || in.max_ur == 4) ur_short = in.max_ur;
    Splitter s{in, word_log2, run, out, ur_short, nt, in.grid > 0 ? static_cast<uint32_t>(in.grid) : 0u};
    s.split_runs(dims, typed, in.packed);
    for (Launch& l : *out) l.keep = keep;
    return kSuccess;
}

bool batchable(const Launch& l) {
    // the batched kernel carries the three four-words-per-thread tiles and plain streaming hints
    return l.kind == kTile && l.p.nrd <= static_cast<uint32_t>(kBatchRowDims) && l.nblocks > 0 && l.ux * l.ur == 4 &&
           (l.nt & 4) == 0 && l.grid == 0;
}

bool runs_compact(const Launch& l, bool unpack) {
    if (l.kind != kTile || l.grid != 0 || l.p.nrd > static_cast<uint32_t>(kBatchRowDims)) return false;
    const int nt = l.hints();
    return nt == 2 || nt == 3 || (unpack && nt >= 6 && l.ux == 1 && l.ur == 1);   // written through: planned with one word per thread alone
}

BatchDesc compact(const Launch& l) {
    BatchDesc d;
    const KParams& p = l.p;
    d.strided = p.strided;
    d.packed = p.packed;
    d.row_pitch = p.row_pitch;
    d.n0 = p.n0;
    d.nrows = p.nrows;
    d.nxc = p.nxc;
    d.xc_mul = p.xc_div.mul;
    const uint32_t tile = (l.ux == 1 ? 0u : l.ux == 2 ? 1u : 2u) | (p.tail_back << 4);
    d.shape = p.bx_log2 | static_cast<uint32_t>(l.word_log2) << 8 | tile << 16 | (p.nrd == 0 ? 1u : p.nrd) << 24;
    d.shifts = p.xc_div.shift << 24;
    for (int k = 0; k < kBatchRowDims; ++k) {
        const bool used = static_cast<uint32_t>(k) < p.nrd;
        d.rstride[k] = used ? p.rstride[k] : 0;
        d.rcount[k] = used ? p.rcount[k] : 1;
        d.rmul[k] = used ? p.rdiv[k].mul : kDivideByOne.mul;
        d.shifts |= (used ? p.rdiv[k].shift : kDivideByOne.shift) << (8 * k);
    }
    return d;
}

bool BatchBuilder::add(const Launch& l) {
    // one tile per workgroup: a batch has at most as many tiles as a grid may have workgroups
    const bool fits = n_ < static_cast<uint32_t>(kBatchMax) && total_ + l.nblocks <= kMaxGrid;
    if (!fits) return false;
    if (n_ == 0) keep_ = true;
    keep_ = keep_ && l.keep;
    desc_[n_] = compact(l);
    nblocks_[n_] = l.nblocks;
    total_ += l.nblocks;
    ++n_;
    return true;
}

void BatchBuilder::finish(BatchParams* out) {
    // Largest first: workgroups are handed out in index order, so the big descriptors start
    // while the whole chip is free and the small ones fill in behind them.  Each descriptor
    // carries its own addresses, so the order inside a launch is free.
    uint8_t order[kBatchMax];
    for (uint32_t i = 0; i < n_; ++i) {
        uint32_t at = i;
        for (; at > 0 && nblocks_[order[at - 1]] < nblocks_[i]; --at) order[at] = order[at - 1];
        order[at] = static_cast<uint8_t>(i);
    }
    out->n = n_;
    out->keep = keep_;
    out->nblocks = 0;
    for (uint32_t i = 0; i < n_; ++i) {
        out->d[i] = desc_[order[i]];
        out->nblocks += nblocks_[order[i]];
        out->block_end[i] = out->nblocks;
    }
    n_ = 0;
    total_ = 0;
}

std::string describe(const std::vector<BatchParams>& batches) {
    std::string text;
    char line[128];
    for (const BatchParams& b : batches) {
        std::snprintf(line, sizeof line, "batch descriptors=%u blocks=%u\n", b.n, b.nblocks);
        text += line;
    }
    return text;
}

std::string describe(const std::vector<Launch>& launches) {
    std::string text;
    char line[256];
    for (const Launch& l : launches) {
        if (l.kind == kXpose) {
            std::snprintf(line, sizeof line, "xpose W=%d words=%u tile=%ux%u a=%u b=%u outer=%u blocks=%u\n", 1 << l.word_log2,
                          l.x.ew, l.x.te_a, l.x.te_b, l.x.ca, l.x.cb, l.x.nod, l.nblocks);
            text += line;
            continue;
        }
        if (l.kind == kPrefetch) {
            std::snprintf(line, sizeof line, "prefetch bytes=%llu tile=%u blocks=%u grid=%u\n",
                          static_cast<unsigned long long>(l.f.bytes), l.f.tile_bytes, l.nblocks, l.grid ? l.grid : l.nblocks);
            text += line;
            continue;
        }
        std::snprintf(line, sizeof line, "tile W=%d ux=%d ur=%d nt=%d bx=%u n0=%u back=%u rows=%u nrd=%u blocks=%u",
                      1 << l.word_log2, l.ux, l.ur, l.nt, 1u << l.p.bx_log2, l.p.n0, l.p.tail_back, l.p.nrows, l.p.nrd, l.nblocks);
        text += line;
        if (l.grid) {
            std::snprintf(line, sizeof line, " grid=%u", l.grid);
            text += line;
        }
        if (l.keep) text += " keep";
        text += "\n";
    }
    return text;
}

}  // namespace tp
