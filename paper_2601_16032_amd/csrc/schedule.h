// Work decode shared by the host launcher and the kernel: which workgroup takes which query tile,
// in which round, and in which direction it then walks the K/V tiles.
//
// The paper launches G persistent workgroups that stride over a linear (batch, head, tile) index
// (Sec. 2.2, Alg. 2) and flips the K/V scan direction on every other local iteration (Sec. 4,
// Alg. 4).  The reuse it relies on happens among workgroups that share one L2 (Sec. 3.4).  On
// MI355X that sharing domain is one XCD: the hardware places workgroup `wg` on XCD `wg % 8`, so the
// linear index is decoded per domain:
//
//   * a head's query tiles are split into `parts` interleaved subsets (parts = 8 / gcd(B*H, 8), so
//     1 when B*H is a multiple of 8); chunk c = head*parts + part runs on domain c % 8, and the
//     chunks of one domain run one after another;
//   * inside a chunk the `slots` workgroups of the domain take its tiles in rounds of `slots`
//     consecutive tiles, so all of them stream the same head's K/V at the same time;
//   * a workgroup's odd local iterations (rounds counted across the chunks of its domain) hand
//     the tiles out in reverse slot order, which evens out the causal cost (tile i costs i+1 K/V
//     tiles) inside a head with an even number of rounds and over two heads otherwise; causal
//     chunks start from their longest tile;
//   * the scan direction of a round is the parity of the round index inside its chunk: this is
//     Alg. 4's local-iteration parity restarted at every chunk.  Consecutive rounds of one chunk
//     walk the same K/V, which is where reversing the direction shortens the reuse distance; the
//     first round of a new chunk meets cold K/V whichever way it walks, and walks forward so that
//     causal tiles all start from key 0 together.  Taking the round index rather than a per-
//     workgroup count keeps the whole domain walking one way when a workgroup sits a round out;
//   * a direct launch has one workgroup per tile, numbered chunk after chunk.  Under the causal mask they start in
//     another order than that of their numbers, the longest of several chunks first (start_longest_first).  Where it stands in for
//     a persistent launch of several rounds per chunk (direct_instead), every tile is walked in the direction it has there, so that
//     the workgroups that follow on a domain's first ones turn around as its rounds do (turn_after).
#pragma once

#if defined(__HIPCC__)
#define SAW_HD __host__ __device__ inline
#else
#define SAW_HD inline
#endif

namespace sawattn {

constexpr int kTileQ = 128;      // query rows per workgroup tile (twice that in the wide variant)
constexpr int kTileKV = 64;      // key/value rows per streamed tile
constexpr int kThreads = 256;    // 4 wavefronts of 32 query rows each (64 in the wide variant)
constexpr int kDomains = 8;      // XCDs
constexpr int kMaxSlots = 96;    // largest number of workgroups per domain for any tile shape

SAW_HD int gcd_i(int a, int b) { while (b) { int t = a % b; a = b; b = t; } return a; }
SAW_HD int ceil_div_i(long long a, long long b) { return (int)((a + b - 1) / b); }

// Rows per wavefront when the caller leaves the choice open: the wide variant (64 rows, 256-row
// workgroup tiles) for head dimension 128 (either input type) once the steady state dominates, i.e.
// every resident workgroup of a domain gets at least one full-length tile of a head (nearly two under the
// causal mask, where a tile walks half the keys on average), and only if the rounds of 32 tiles are well
// filled: a last round with a few tiles costs this kernel a full round, while the workgroups of 128-row tiles run faster when
// they have their compute unit to themselves.  The lines were drawn against the 32x32x16 kernels of both tile shapes.  As both
// run now (16x16x32 here, default_shared_kernel there), by 256-row tiles per head and XCD, binary16 / bfloat16, 8 heads, change of
// the rate in %: plain 32: +8 / +14, 36: -9 / -1, 40: -9 / 0, 48: -4 / +5, 56: +9 / +14, 64: +10 / +15, 72: -2 / +3, 80: +2 / +10,
// 88: +10 / +14, 96: +10 / +16; causal 48: -4 / -1, 56: +7 / +10, 64: +10 / +14, 72: +4 / +7, 80: +4 / +7, 88: +5 / +9, 96: +6 / +10.
SAW_HD int default_rows_per_wavefront(int heads, int N, int d, bool causal, bool bf16) {
    (void)bf16;
    if (d != 128) return 32;
    const int parts = kDomains / gcd_i(heads, kDomains);
    const int wide_tiles = (N + 2 * kTileQ - 1) / (2 * kTileQ);
    const int q = (wide_tiles + parts - 1) / parts;          // tiles of a head on one XCD
    if (q < (causal ? 56 : 32)) return 32;
    const int rounds = (q + 31) / 32;
    // filled to at least 4/5 over all rounds (3/4 under the mask)
    return (causal ? 4 * q >= 3 * 32 * rounds : 5 * q >= 4 * 32 * rounds) ? 64 : 32;
}

// Workgroups per domain that are resident together: 32 CUs per XCD x workgroups per CU.  A head
// dimension of 64 leaves room for three (168 VGPRs per wavefront, 32 KiB LDS per workgroup), 128 for
// two; the wide variant (256-row tiles, up to 512 registers per wavefront, 128 KiB LDS) runs one.
// With 64-row tiles (the two halves of a scan at once, twice the LDS) two fit at d = 64 and one at d = 128.
SAW_HD int resident_slots(int d, int tile_q = kTileQ) {
    if (tile_q > kTileQ) return 32;
    if (tile_q < kTileQ) return d == 64 ? 64 : 32;
    return d == 64 ? 96 : 64;
}

// Small problems: when the 128-row query tiles of the whole problem occupy at most half of the 256 compute units,
// the launch takes as long as one wavefront needs to walk all K/V tiles of a head.  Then a workgroup takes 64 rows
// instead and walks the two halves of the scan at once, two wavefronts each.  At d = 64, where two such workgroups
// fit a compute unit (512 on the chip), it goes on paying for somewhat larger problems, most under the causal mask,
// where the longest tile of a head sets the pace and is the one cut in two.  Limits, in 128-row tiles of the whole problem:
// d = 128: 128 (beyond, the 64-row workgroups, one per compute unit, no longer run all at once: up to 1.5x slower at 256);
// d = 64: 384 plain, 512 causal, and beyond 128 only for N >= 2048: a scan of 16 tiles or fewer is too short for its halves to
// pay for the merge (N = 512: 25 % slower).  They were drawn against the 32x32x16 kernel (gains of 3-10 % there, none at 768).
// Time against 128-row tiles as they run now (default_shared_kernel), binary16 and bfloat16, 1 to 16 heads: d = 128, 128 tiles: -9 to -33 %;
// d = 64, plain, 128 tiles: -28 to -42 %, 256: -11 to -2 %, 384: +1 to +12 %; causal, 128: -30 to -46 %, 256: -20 to -37 %, 384:
// -15 to -27 %, 512: -11 to -3 %.
// 1 = one scan per workgroup, 2 = two halves.
SAW_HD int default_kv_halves(int heads, int N, int d, bool causal, bool bf16) {
    (void)bf16;
    const long long tiles = (long long)heads * ((N + kTileQ - 1) / kTileQ);
    const int limit = d == 64 && N >= 2048 ? (causal ? 512 : 384) : 128;
    return tiles <= limit ? 2 : 1;
}

// Besides that default, the launch variants the paper describes are kept selectable so that they
// can be measured against it: the literal global stride of Alg. 2 (workgroup k takes the linear
// indices k, k+G, ... with the tile index fastest, direction = parity of its own iteration count,
// Alg. 4 as printed), fewer resident workgroups per domain (Sec. 3.4), and the direct launch of
// Alg. 3 with one workgroup per one or two consecutive query tiles, where the second tile is
// walked backward (the step-2 alternation of Sec. 4.3).
enum { kLaunchPersistent = 0, kLaunchGrid = 1 };

// How the tiles touched once per query tile pass the L2 when the caller leaves it open: O always as whole non-temporal
// lines; Q as well where K and V of a head take at least half the 4 MiB L2 of an XCD -- below that no scan order has
// anything to lose to the Q tiles, and direct loads hide their latency behind the first K/V fetch.
SAW_HD int default_qo_streaming(int N, int d) {
    return (unsigned long long)N * (unsigned)d * 4u >= (2u << 20) ? 3 : 1;
}

// Launch when the caller leaves the choice open.  The persistent hand-out gives one head at a time to the
// workgroups of an XCD, which is what keeps a long head's K/V in one L2; a head with fewer query tiles than the
// XCD holds workgroups then leaves compute units idle, and with several such heads per XCD one after the other
// the launch takes several times longer than it has to (B*H = 128, N = 512, d = 64: 140 us against 17 us).  There
// the direct launch of Alg. 3 with one tile per workgroup is taken: the hardware dispatcher runs the tiles of all
// heads of an XCD side by side, still head by head in workgroup order.  Under the causal mask the persistent
// hand-out has something the dispatcher has not -- it pairs a long tile with a short one per workgroup -- and keeps
// the launch unless the heads are short enough to run two abreast (measured: from half the resident count down),
// or, with only two heads per XCD, unless all their tiles find a compute unit of their own.
SAW_HD int default_launch(int heads, int N, int d, bool causal, int tile_q) {
    const int parts = kDomains / gcd_i(heads, kDomains);
    const int q_tiles = (N + tile_q - 1) / tile_q;
    const int per_part = (q_tiles + parts - 1) / parts;
    const long long chunks = ((long long)heads * parts) / kDomains;
    const int resident = tile_q > kTileQ ? 32 : (tile_q < kTileQ ? (d == 64 ? 64 : 32) : (d == 64 ? 96 : 64));
    if (per_part >= resident || chunks < 2) return kLaunchPersistent;
    if (!causal) return kLaunchGrid;
    if (chunks >= 3) return 2 * per_part <= resident ? kLaunchGrid : kLaunchPersistent;
    return 2 * per_part <= 32 ? kLaunchGrid : kLaunchPersistent;
}
enum { kDecodeDomain = 0, kDecodeLinear = 1 };

// The imbalance of a persistent hand-out: K/V tiles of its busiest workgroup over what an even share would be (the longest tile of a chunk, if that
// is more).  `n` tiles per chunk, under the causal mask of 1 .. n parts, otherwise of one; rounds as in decode_work.  Whether it is at least
// num / den, in whole numbers: whole loads give simple fractions, 1 x 131072, d = 64, without a mask exactly 3/2.  (Below 2^62: n * chunks
// is at most 2^28, n at most 2^24.)
SAW_HD bool imbalance_at_least(int num, int den, int n, long long chunks, int resident, bool causal) {
    const int slots = n < resident ? n : resident, rounds = (n + slots - 1) / slots;
    long long most = 0;
    for (int slot = 0; slot < slots; ++slot) {
        long long in_chunk[2] = {0, 0};               // the rounds of a chunk that begins with an even / odd one
        for (int first = 0; first < 2; ++first)
            for (int r = 0; r < rounds; ++r) {
                const int u = r * slots + ((r + first) & 1 ? slots - 1 - slot : slot);
                if (u < n) in_chunk[first] += causal ? n - u : 1;
            }
        const long long all = rounds % 2 == 0 ? chunks * in_chunk[0] : (chunks + 1) / 2 * in_chunk[0] + chunks / 2 * in_chunk[1];
        if (all > most) most = all;
    }
    const long long longest = causal ? n : 1, total = (causal ? n * (n + 1ll) / 2 : n) * chunks;
    return most * resident * den >= num * (total > longest * resident ? total : longest * resident);
}

// Whether a launch that default_launch leaves persistent is faster as a direct one (under the mask with its longest workgroups first): the
// dispatcher evens out what a fixed hand-out leaves uneven.  The scan directions stay those of the rounds (turn_after), but their
// workgroups no longer keep step.  Change of the time from persistent to direct, n tiles per chunk on C chunks per XCD:
//   * causal, one round per chunk.  An odd number of rounds leaves somebody with an unpaired one: -6 to -38 % at C = 3, 5, -4 to
//     -37 % at 7 and more.  With an even number all workgroups have the same, but n of them fill the compute units evenly only where
//     n is a multiple of 32: d = 128, n = 34 to 56: -35 to -3 %, 60: -2 to -1 %, 64: +1 to +2 %; d = 64, n = 34 to 52: -22 to 0 %,
//     60: -6 to +2 %, 64: -6 to +1 %, 72 to 88: -22 to -6 %, 96: -4 to -2 %;
//   * several rounds per chunk, by the imbalance above.  Causal, d = 64: 1.1 to 1.2: -3 to -6 %, 1.3 to 1.8: -3 to -16 %; d = 128: 1.17: -3 %,
//     1.3 to 1.8: -1 to -17 %.  No mask, two chunks and more: 1.3 and 1.5: -6 to -9 %, 1.7 and more: -18 to -27 % (40 heads x 8320, d =
//     128, bfloat16: 2002 -> 1466 us); one chunk, d = 64: 1.1 and 1.3: -1 to -2 %, 1.42 to 1.47: -1 % in two rounds, +2 % in three
//     (8 heads x 25920: 1427 -> 1449 us), 1.5 and more: -5 to -9 %; d = 128: 1.75 and more: -5 %, else 0.
//     Below that the persistent launch stays, although at d = 64 under the mask it is 2 to 9 % slower: its workgroups keep step;
//   * 64-row tiles: causal, one round per chunk, C = 3 and more, odd: -16 to -21 %; C = 2, n = 47: -10 %, 61: +2 %.
SAW_HD bool direct_instead(int heads, int N, int d, bool causal, int tile_q) {
    if (tile_q > kTileQ) return false;
    const int parts = kDomains / gcd_i(heads, kDomains);
    const int q_tiles = (N + tile_q - 1) / tile_q;
    const int n = (q_tiles + parts - 1) / parts, resident = resident_slots(d, tile_q);
    const long long chunks = ((long long)heads * parts) / kDomains;
    if (n <= resident) {
        if (!causal || chunks < 2) return false;
        if (tile_q < kTileQ) return chunks == 2 ? n > 32 && n < 56 : chunks % 2 != 0;
        if (d == 128) return chunks == 2 ? n > 32 && n < 64 : n <= 60 || (chunks % 2 != 0 && chunks < 7);
        if (chunks == 2) return (n > 32 && n <= 48) || (n > 64 && n < 96);
        return chunks % 2 != 0 || n % 32 != 0;
    }
    if (tile_q < kTileQ) return false;
    if (d == 128 && chunks == 1) return false;
    if (chunks == 1 && !causal) return imbalance_at_least(3, 2, n, chunks, resident, causal);
    return d == 128 && causal ? imbalance_at_least(23, 20, n, chunks, resident, causal) : imbalance_at_least(11, 10, n, chunks, resident, causal);
}

struct Schedule {
    int heads;              // B*H
    int tile_q;             // query rows per workgroup tile: kTileQ, or 2*kTileQ in the wide variant
    int q_tiles;            // ceil(N / tile_q)
    int kv_tiles;           // ceil(N / kTileKV)
    int launch;             // kLaunchPersistent | kLaunchGrid
    int decode;             // kDecodeDomain | kDecodeLinear
    int parts;              // interleaved subsets per head (domain decode; 1 for linear decode)
    int slots;              // workgroups per domain = grid / kDomains
    int chunks_per_domain;  // heads*parts / kDomains (domain decode)
    int rounds_per_chunk;   // persistent, domain decode: ceil(ceil(q_tiles/parts) / slots)
    int units_per_chunk;    // grid launch, domain decode: workgroups per chunk
    int tiles_per_wg;       // grid launch: consecutive tiles per workgroup (1 otherwise)
    int grid;               // workgroups launched (a multiple of kDomains)
    int local_iters;        // local iterations every workgroup runs through (some may be idle)
    int sync_heads;         // persistent, domain decode: the workgroups of a domain wait for each other between heads
    int sync_rounds;        // ... and after every round as well (a study of Sec. 3.4's lockstep; costs time)
    unsigned turn;          // direct launch, domain decode: 2^32 over the tiles of a chunk after which the scan direction turns, rounded up
                            // (0: all walk forward)
    int chunks_abreast;     // direct launch: chunks whose workgroups start together, longest first (1: in the order of their numbers)
    int qo_streaming;       // 1: O tiles leave through LDS as whole non-temporal lines; 2: Q tiles arrive that way; 3: both; 4: neither
};

struct Work {
    int head;        // b*H + h
    int tile;        // query tile index inside the head, -1: nothing to do in this iteration
    bool backward;   // walk the K/V tiles from the last visible one down to 0
    bool sync_after; // persistent domain decode: last round of a head that is not the domain's last
};


// max_slots in 1..resident_slots(d), tiles_per_wg in {1, 2}; the caller has validated them.
SAW_HD Schedule make_schedule(int heads, int N, bool causal, int launch, int decode, int max_slots, int tiles_per_wg,
                              int tile_q = kTileQ, bool align_rounds = false) {
    Schedule s;
    s.heads = heads;
    s.qo_streaming = 0;     // the caller's choice: not part of who computes what
    s.tile_q = tile_q;
    s.q_tiles = (N + tile_q - 1) / tile_q;
    s.kv_tiles = (N + kTileKV - 1) / kTileKV;
    s.launch = launch;
    s.decode = decode;
    s.tiles_per_wg = launch == kLaunchGrid ? tiles_per_wg : 1;
    s.parts = decode == kDecodeDomain ? kDomains / gcd_i(heads, kDomains) : 1;
    const int per_part = (s.q_tiles + s.parts - 1) / s.parts;     // tiles in the largest part
    s.chunks_per_domain = (int)(((long long)heads * s.parts) / kDomains);
    s.rounds_per_chunk = 0;
    s.units_per_chunk = 0;
    s.sync_heads = 0;
    s.sync_rounds = 0;
    s.turn = 0;             // turn_after
    s.chunks_abreast = 1;   // start_longest_first
    const long long total = (long long)heads * s.q_tiles;
    if (launch == kLaunchPersistent) {
        if (decode == kDecodeDomain) {
            s.slots = per_part < max_slots ? per_part : max_slots;
            s.rounds_per_chunk = (per_part + s.slots - 1) / s.slots;
            s.local_iters = s.chunks_per_domain * s.rounds_per_chunk;
            // Waiting for the domain between heads pays only if its workgroups finish a head together:
            // every slot gets a tile in every round, and causal tiles pair up long with short.
            const bool even_load = s.q_tiles % (s.parts * s.slots) == 0 && (!causal || s.rounds_per_chunk % 2 == 0);
            s.sync_heads = even_load && s.chunks_per_domain > 1;
            s.sync_rounds = align_rounds && s.local_iters > 1;
        } else {
            const int want = ceil_div_i(total, kDomains);
            s.slots = want < max_slots ? want : max_slots;
            s.local_iters = ceil_div_i(total, (long long)kDomains * s.slots);
        }
    } else {
        if (decode == kDecodeDomain) {
            s.units_per_chunk = (per_part + s.tiles_per_wg - 1) / s.tiles_per_wg;
            s.slots = s.chunks_per_domain * s.units_per_chunk;
        } else {
            s.slots = ceil_div_i(ceil_div_i(total, s.tiles_per_wg), kDomains);
        }
        s.local_iters = s.tiles_per_wg;
    }
    s.grid = kDomains * s.slots;
    return s;
}

// A direct launch in place of a persistent one of `tiles` workgroups per domain: tile u of a chunk, which round u / tiles would take, is walked in
// that round's direction.  The workgroups start in the order of u, as places come free, so those of a round still follow on the one before over
// the same K/V, and turning around finds in the L2 what that left there.  L2 misses, cyclic -> sawtooth (TCC_MISS, millions): 1 x 131072,
// d = 64, plain 7.5 -> 7.2 (persistent 7.5 -> 7.3); 8 x 32768, d = 64, causal 1.8 -> 1.5 (1.9 -> 1.7); 2 x 131072, d = 64, causal 71 -> 42
// (55 -> 8.7: there the workgroups drift apart, which the persistent launch's pairs of a long and a short tile prevent).  Times of the two
// orders: alike, within 1.4 %.
// (The quotient as a product: exact for r <= 96 up to u = 2^27, and a chunk has at most 2^24 tiles.  A division and its branch cost every
// direct launch 0.1 to 0.2 us, this at most 0.07: 42 x 1000, d = 64, causal: 17.14 -> 17.35 against 17.21 us.)
SAW_HD void turn_after(Schedule& s, int tiles) { s.turn = (unsigned)((0x100000000ull + tiles - 1) / tiles); }

// Direct launches under the causal mask: which workgroups start first.  The hardware starts them in the order of their block numbers and
// a new one wherever one has finished.  In the order of their own numbers, chunk after chunk, the last chunk's longest
// workgroups start when most of the work is done and finish alone: 4 chunks of 32 tiles on 64 places take 49 steps of the longest
// tile's 32 where 33 would do.  So the workgroups of several chunks start together, longest first, and the short ones
// fill up the end.  Not of all chunks: those of one chunk then start far apart and share less of its K and V in the
// L2.  Time against chunk after chunk, abreast as many chunks as make 1, 3/2, 2, 3, 4 loads of the XCD, and all of them: 128 heads x 4096, d = 128:
// -2.4, -4.7, -4.7, -4.4, -3.9, -2.0 %; 48 x 4096, d = 64: -15, -20, -20, -21, -21, -21 %; 126 x 3500, d = 128: +0.9, -0.3,
// +0.8, +7, +10, +10 %.  At 3/2 loads, over 155 launches that were direct before: -38 to +1 %, -11 % in the mean (32 x 4096, d =
// 128: 151 -> 130 us; 64 x 2048, d = 64: 52.7 -> 43 us).  Who computes what, and the recorded schedule, stay as they are.
// Not at d = 128 with 3 or 5 workgroups to a chunk and 55 chunks and more: what so few share when they start together counts for more there than the
// end.  45 to 54 chunks: 3 to a chunk -7 to +6 % (-1 % in the mean), 5 to a chunk -4 to +1 % (-1.5 %); 55 and more: 3 to a chunk -5 to +13 %
// (+6 %), 5 to a chunk -5 to +6 % (+1.6 %).  More to a chunk gain up to some 10 loads of the XCD and are even from there on, 6 to 10 loads: 7, 9, 11 ..
// -6 to +5 % (-1.5 %), 6, 10, 14 .. -8 to +4 % (-3 %); 10 and more: odd -4 to +9 % (+0.6 %), 6, 10, 14 .. -8 to +3 % (-1 %).  Multiples
// of 4 gain whatever the loads (-23 to +1 %), as workgroups of one length would meet on the compute units otherwise, and so do 2 to a chunk
// (-21 to +2 %).  d = 64: below 6 loads -35 to +2 %, 10 and more: odd -5 to +3 % (+0.4 %), even -12 to +1 % (-2.4 %).
SAW_HD void start_longest_first(Schedule& s, int d, bool causal) {
    if (!causal || s.launch != kLaunchGrid || s.decode != kDecodeDomain || s.tiles_per_wg != 1 || s.tile_q > kTileQ) return;
    const int n = s.units_per_chunk, resident = resident_slots(d, s.tile_q);
    if (n < 2 || (d == 128 && n % 2 && n < 7 && s.chunks_per_domain >= 55)) return;
    const int least = (3 * resident + 2 * n - 1) / (2 * n);
    const int groups = s.chunks_per_domain / least;
    s.chunks_abreast = groups > 1 ? (s.chunks_per_domain + groups - 1) / groups : s.chunks_per_domain;
}

// The schedule of a launch with query tiles of `tile_q` rows.  What is left open (launch -1; max_slots, tiles_per_wg 0) is chosen here: the
// persistent launch, or for short heads and uneven rounds the direct one with a tile each.  A direct launch that the caller names is that
// of Alg. 3: started in the order of the workgroups' numbers, every first tile walked forward.
SAW_HD Schedule launch_schedule(int heads, int N, int d, bool causal, int tile_q, int launch = -1, int decode = kDecodeDomain, int max_slots = 0,
                                int tiles_per_wg = 0, bool align_rounds = false) {
    const bool open = launch < 0;
    bool instead = false;
    if (open) {
        launch = kLaunchPersistent;
        if (decode == kDecodeDomain && max_slots == 0) {
            launch = default_launch(heads, N, d, causal, tile_q);
            instead = launch == kLaunchPersistent && tiles_per_wg < 2 && !align_rounds && direct_instead(heads, N, d, causal, tile_q);
            if (instead) launch = kLaunchGrid;
        }
        if (launch == kLaunchGrid && tiles_per_wg == 0) tiles_per_wg = 1;
    }
    if (tiles_per_wg == 0) tiles_per_wg = 2;
    if (max_slots == 0) max_slots = resident_slots(d, tile_q);
    Schedule s = make_schedule(heads, N, causal, launch, decode, max_slots, tiles_per_wg, tile_q, align_rounds);
    if (instead && tile_q == kTileQ) turn_after(s, max_slots);      // (with 64-row tiles only for a single round)
    if (open) start_longest_first(s, d, causal);
    return s;
}

// The workgroup that the hardware's block `block` is.
SAW_HD int workgroup_of_block(const Schedule& s, int block) {
    if (s.chunks_abreast <= 1) return block;
    int at = block / kDomains, first = 0, abreast = s.chunks_abreast;      // place in the group, its first chunk, its chunks
    if (abreast < s.chunks_per_domain) {
        const int group = at / (abreast * s.units_per_chunk);
        first = group * abreast;
        at -= first * s.units_per_chunk;
        if (s.chunks_per_domain - first < abreast) abreast = s.chunks_per_domain - first;
    }
    const int u = at / abreast;
    return ((first + at - u * abreast) * s.units_per_chunk + u) * kDomains + block % kDomains;
}

// Workgroups of a chunk (domain decode) or of a head (linear decode) in a direct launch, tiles of a chunk otherwise.
SAW_HD int per_chunk(const Schedule& s) {
    if (s.decode == kDecodeLinear) return ceil_div_i(s.q_tiles, s.tiles_per_wg);
    return s.launch == kLaunchGrid ? s.units_per_chunk : ceil_div_i(s.q_tiles, s.parts);
}

// Which kernel computes 128-row tiles: the one with 16x16x32 MFMAs (attn_fwd_shared_kernel) where workgroups share the
// compute units, the one with 32x32x16 MFMAs where a workgroup has one to itself.  The smaller MFMA switches less
// current per multiply-add, which is worth more clock once the chip is at its power limit, but takes twice the issue
// slots; a wavefront alone on its SIMD is bound by those.  What follows is the change of the time from 32x32 to 16x16
// over 1358 launches (profiles/shared_kernel_rules.txt).  With 32 workgroups per XCD and fewer 0 to +32 % (1 x 20000, d =
// 128, 20 workgroups: 244 -> 321 us).  From 33 on -12 to +2 % at d = 64, where three share a compute unit (132 heads x 256:
// 9.4 -> 8.9 us; 1 x 131072, causal: 2520 -> 2310 us).  At d = 128 it loses where workgroups run alone for a good part of the
// launch:
//   * without a mask, where the last workgroups have a compute unit each (1 to 32 left over by whole loads of 64 per XCD).
//     bfloat16: one load and up to 32 more +7.5 % in the mean (24 x 4096: 204 -> 238 us), two and three loads +3 %, a second
//     round of a persistent launch 0 to +2 %, from four loads on 0.  Binary16: one load and up to 32 more +1.8 % (3 x 28077:
//     1212 -> 1318 us), then -1 to -3 %.  (One tile per head and XCD, one load and more: -10 to +3 %.)  Elsewhere -3 % in the
//     mean for bfloat16 and -7 % for binary16;
//   * under the mask, a persistent launch of a single round, as long as its longest tile: +2 to +16 %; two rounds of which
//     the second is less than 1/8 full: +1.5 to +5 %;
//   * under the mask, few compute units shared and workgroups of unequal length: direct launches of 33 to 47 workgroups per
//     XCD, 3 and more to a chunk: -2 to +18 % (+3.7 % in the mean; 48 and more: -7 to +3 %), persistent ones of three
//     rounds of 33 and 35: +8 and +4 %.  (With the lengths evened out by a second round 33 to 39 workgroups gain 4 to 9 %, and
//     33 to 47 with one or two short tiles to a chunk gain 2 to 11 %.)
//   * under the mask, a direct launch of more workgroups than fit at once, with 2, 4 or 8 of them to a chunk: those of a
//     compute unit are then equally long and make room all together.  89 of 106 of these lose, up to 10 % (2.7 % in the
//     mean); with 16 and 32 to a chunk -9 to +4 % (-0.6 %), with 1 -7 to +3 % (-1.4 %), with others -7 to +4 % (-1.3 %).
// Direct launches whose longest workgroups start first (start_longest_first; the last two lines hold for those in the order of their
// numbers: named by a variant, or the few that start_longest_first leaves out), d = 128: up to 47 workgroups per XCD +4 to +12 %; 48 to 64, 8 and more to a chunk: +2 to +4 %, fewer: -7 to +2 %; more than fit:
// -14 to +2 % (the better of the two with and without precedence).
SAW_HD bool default_shared_kernel(const Schedule& s, int d, bool causal, bool bf16) {
    if (s.slots <= 32) return false;
    if (d == 64) return true;
    const int n = per_chunk(s), resident = resident_slots(d);
    if (s.chunks_abreast > 1) return s.slots >= 48 && (s.slots > resident || n < 8);
    if (!causal) {
        const int wgs = s.launch == kLaunchGrid ? s.slots : n;     // (persistent: what the last round of a chunk leaves)
        if (wgs <= resident || (wgs - 1) % resident >= 32) return true;
        if (s.launch == kLaunchGrid && wgs < 2 * resident) return n == 1;
        return !bf16 || wgs > 4 * resident;
    }
    if (s.launch == kLaunchPersistent) {
        if (s.local_iters == 1) return false;
        if (s.decode == kDecodeLinear) return true;
        if (s.rounds_per_chunk == 1) return s.local_iters != 3 || s.slots >= 40;
        return s.rounds_per_chunk > 2 || 8 * (n - s.slots) >= s.slots;
    }
    if (s.slots <= resident) return s.slots >= 48 || n <= 2;
    return n == 1 || n >= 16 || 32 % n != 0;
}

// Whether that kernel gives the wavefronts in their second product precedence on their SIMD (scan_tiles).  By
// itself the hardware prefers the oldest wavefront, so of the workgroups that share a compute unit one runs ahead and
// the other finishes alone, without anybody to share the units with.  With precedence by phase they advance alike, which
// is better where they also have equally much to do (12 heads x 5000, d = 128, bfloat16: 156 -> 151 us) and worse where the
// launch waits for the one with the most.  Measured under the causal mask, without -> with precedence:
//   * persistent, one round per chunk: an even number of rounds gives every workgroup the same length, -9 to -1 %; an odd
//     number leaves the longest one 1/rounds above the mean: d = 128, 3 and 5 rounds: +2 to +11 %, 7 and 9: 0 to +4 %, more:
//     -3 to 0 %; d = 64, one round: +5 to +12 %, three: -1 to +5 % up to 64 workgroups per XCD, -6 to -2 % above, five and
//     more: -6 to -1 %;
//   * persistent, two rounds per chunk, the second to a share f: the longest one is 2/(1+f) of the mean.  d = 128 (f up to
//     0.7; longer heads run 256-row tiles): +2 to +10 %; d = 64: f below 1/4: 0 to +8 %, above: -5 to -1 %.  Three rounds
//     and more: -5 to +1 %;
//   * direct launch, all workgroups at once: -6 to +1 % (one of 86: +5 %).
//   * direct launch of more than fit.  d = 64: -5 to +2 % (-0.9 % in the mean) from twice as many on; fewer: -5 to +1 % (-1.4
//     %) where a head is spread over 4 or 8 XCDs, two tiles and more to a chunk, -4 to +10 % (+2.2 %) otherwise (64 heads x
//     2048: 54 against 59 us, 40 x 3968: 104 against 114 us).  d = 128: -7 to +7 % (+0.7 %); -10 to +2 % (-2.6 %) for 4/3 to
//     twice as many, a head over 4 or 8 XCDs and five tiles and more to a chunk (5 x 23936: 844 -> 793 us);
//   * direct launch, longest workgroups first (the two lines above hold for the order of their numbers, as a variant names it).  d = 64, all at once: 8 and more to
//     a chunk, or up to 64 per XCD: 0 to +9 %, else -5 to 0 %; more than fit: -5 to +2 %, but +2 to +8 % for up to twice as many of
//     16 and more to a chunk, a head on one XCD.  d = 128, all at once: +1 to +5 %; up to 1.6 times as many as fit: 2 or 3 to a
//     chunk -5 to +2 %, more 0 to +6 %; 1.6 to 2.2 times: -10 to -1 % (32 x 4096: 137 -> 130 us); more: -8 to +3 % up to 32 to a
//     chunk, -3 to +4 % above.
SAW_HD bool default_phase_priority(const Schedule& s, int d, bool causal) {
    if (!causal) return true;
    const int rounds = s.local_iters, resident = resident_slots(d), n = per_chunk(s);
    if (s.chunks_abreast > 1) {
        if (d == 64) return s.slots <= resident ? n < 8 && s.slots > 64 : s.slots > 2 * resident || n < 16 || s.parts > 1;
        if (s.slots <= resident) return false;
        if (10ll * s.slots < 16 * resident) return n <= 3;
        return 10ll * s.slots <= 22 * resident || n <= 32;
    }
    if (s.launch == kLaunchGrid) {
        if (s.slots <= resident) return true;
        if (d == 64) return s.slots >= 2 * resident || (s.parts >= 4 && n > 1);
        return s.parts >= 4 && n >= 5 && 3 * s.slots >= 4 * resident && s.slots < 2 * resident;
    }
    if (s.decode == kDecodeLinear) return rounds > 1 && s.slots % 32 == 0;
    if (s.rounds_per_chunk == 1)
        return rounds % 2 == 0 || (d == 64 ? rounds >= 5 || (rounds == 3 && s.slots > 64) : rounds > 10);
    return s.rounds_per_chunk > 2 || (d == 64 && 4 * (n - s.slots) >= s.slots);
}

// a / b for a >= 0, b > 0.  On the GPU a division is some 40 dependent scalar and vector instructions, and the part of it
// that depends on b alone would be computed ahead of the loop over the tiles, also where no quotient is needed: most
// workgroups only ever see the first chunk (a < b).  With LATE nothing is computed ahead, because with short sequences
// the time up to the first fetch counts: 0.2 to 0.3 us of a kernel's duration (kernel trace, a launch at a time: one head of
// 256 rows, d = 64: 6.64 -> 6.36 us; 8 heads x 2048: 18.68 -> 18.36 us; 128 x 512, d = 128: 22.3 -> 22.1 us.  Calls in a row hide
// most of it: 8 x 2048 takes 16.3 us either way).  The kernel with 256-row tiles, whose scans are long, keeps the plain
// division: the change moves its registers and costs it time (128 heads x 32768, bfloat16, causal: 30.9 -> 31.4 ms).
template <bool LATE, typename T>
SAW_HD T quotient(T a, T b) {
    if constexpr (LATE) {
        if (a < b) return 0;
#ifdef __HIP_DEVICE_COMPILE__
        asm volatile("" : "+s"(b));
#endif
    }
    return a / b;
}

// What workgroup `wg` does in its local iteration `it` (0 <= it < local_iters).  TURNS false: for kernels whose tiles no launch with `turn` has.
template <bool LATE = false, bool TURNS = true>
SAW_HD Work decode_work(const Schedule& s, int wg, int it, bool causal, bool sawtooth) {
    Work w;
    w.head = 0;
    w.tile = -1;
    w.backward = false;
    w.sync_after = false;
    if (s.decode == kDecodeLinear) {
        // Alg. 2 / Alg. 3 as printed: one linear index over (head, tile), tile fastest.
        const long long k = s.launch == kLaunchPersistent ? (long long)wg + (long long)it * s.grid
                                                          : (long long)wg * s.tiles_per_wg + it;
        if (k < (long long)s.heads * s.q_tiles) {
            // (k is below 2^32 here: at most 2^31 tiles of 128 rows; a 64-bit division is several times longer)
            w.head = LATE ? (int)quotient<LATE>((unsigned)k, (unsigned)s.q_tiles) : (int)(k / s.q_tiles);
            w.tile = (int)(k - (long long)w.head * s.q_tiles);
        }
        w.backward = sawtooth && (it & 1);
        return w;
    }
    const int domain = wg % kDomains, slot = wg / kDomains;
    int cs, u;
    if (s.launch == kLaunchPersistent) {
        cs = quotient<LATE>(it, s.rounds_per_chunk);
        const int r = it - cs * s.rounds_per_chunk;
        u = r * s.slots + ((it & 1) ? s.slots - 1 - slot : slot);
        w.backward = sawtooth && (r & 1);
        w.sync_after = (s.sync_heads && r + 1 == s.rounds_per_chunk && cs + 1 < s.chunks_per_domain) ||
                       (s.sync_rounds && it + 1 < s.local_iters);
    } else {
        cs = quotient<LATE>(slot, s.units_per_chunk);
        u = (slot - cs * s.units_per_chunk) * s.tiles_per_wg + it;
        const int run = TURNS ? (int)((unsigned long long)(unsigned)u * s.turn >> 32) : 0;
        w.backward = sawtooth && ((it | run) & 1);
    }
    const int c = cs * kDomains + domain;
    const int part = c % s.parts;
    w.head = c / s.parts;
    const int in_part = (s.q_tiles - part + s.parts - 1) / s.parts;
    if (u < in_part) w.tile = part + s.parts * (causal ? in_part - 1 - u : u);
    return w;
}

// K/V tiles visible to query tile t.
SAW_HD int visible_kv_tiles(const Schedule& s, int t, int N, bool causal) {
    if (!causal) return s.kv_tiles;
    long long last_row = (long long)(t + 1) * s.tile_q;
    if (last_row > N) last_row = N;
    return (int)((last_row + kTileKV - 1) / kTileKV);
}

}  // namespace sawattn
