// The body of the decoders' kernels (pcc.hip), included into each: Net, MINBLOCKS, ROWS and the kernel's parameters
// are in scope.  (As a function inlined into the kernels the compiler allots their registers differently: with two
// workgroups per compute unit the paper's shape then spills none instead of 2, 30-160-160-128-60 27 instead of 29, seven mixtures 45 instead of
// 44; with one the paper's network takes 5,298 us in 512x512 instead of 5,271, other times are the same within 0.4 %.)
    using Lay = Layout<Net>;
    using D = DecLds<Net, ROWS>;
    constexpr int PK = D::kPartK, LP = D::kLanes;
    constexpr int K = Net::K, HS = Lay::kHeadSlots, RC = Net::kRingCols, KB0 = Net::kb(0);
    constexpr int kDelay = Net::kDelay, kMaxReach = D::kMaxReach;
    extern __shared__ __align__(16) uint8_t lds[];
    float2* lut = reinterpret_cast<float2*>(lds + D::kLutOff);
    uint8_t* act0 = lds + D::kAct0Off;
    uint8_t* act1 = lds + D::kAct1Off;
    float* headout = reinterpret_cast<float*>(lds + D::kHeadOff);
    float* cpbuf = reinterpret_cast<float*>(lds + D::kCpOff);
    uint16_t* ring = reinterpret_cast<uint16_t*>(lds + D::kRingOff);
    int* misc = reinterpret_cast<int*>(lds + D::kMiscOff);            // [0] ticket, [1] abort
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    // a scalar where a branch on it pays (two workgroups per CU); measured slower as a scalar otherwise
    const int wave = MINBLOCKS > 1 ? __builtin_amdgcn_readfirstlane(tid >> 6) : tid >> 6;
    const int wave_s = __builtin_amdgcn_readfirstlane(tid >> 6);     // for branches that whole waves take
    // network role: pixel nl of the tile, k-slot group g
    const int g = lane >> 4, nl = lane & 15;
    const bf16x4_bits_t minus_one = minus_identity(lane);
    // search role: pixel q of the band, lane j of its LP lanes, which is edge e and takes part `part` of the components
    const int q = LP == 16 ? 4 * wave + (lane >> 4) : 2 * wave + (lane >> 5), j = LP == 16 ? lane & 15 : lane & 31, part = LP == 16 ? 0 : (lane >> 4) & 1;
    SearchLane sl;
    sl.e = LP == 16 ? j : lane & 15; sl.shift = LP == 16 ? lane & 48 : lane & 32; sl.base4 = LP == 16 ? 4 * (lane & 48) : 4 * ((lane & 32) + 16);
    sl.edge1 = (float)(32 * sl.e - 1) * (1.0f / 512.0f);
    sl.edge2 = (float)(2 * sl.e - 1) * (1.0f / 512.0f);
    const bool no_sums = D::kParts > 1 && part == 0;
    sl.e1 = no_sums ? __builtin_inff() : sl.e == 0 ? -__builtin_inff() : (float)(16 * sl.e);
    sl.e2 = no_sums ? __builtin_inff() : sl.e == 0 ? -__builtin_inff() : (float)sl.e;
    sl.table = (uint32_t)(sl.e >> 2) * kLutCopyBytes;

    {
        const float2* src = reinterpret_cast<const float2*>(model + Lay::kLutOff);
        for (int i = tid; i < kLutEntries + 1; i += kDecThreads) {
            if constexpr (D::kTable == Table::kSpread) *reinterpret_cast<float2*>(lds + D::kLutOff + spread_at((uint32_t)i)) = src[i];
            else for (int c = 0; c < kLutCopies; ++c) *reinterpret_cast<float2*>(lds + D::kLutOff + c * kLutCopyBytes + 8 * i) = src[i];
        }
    }
    if constexpr (D::kParts * PK > K) {      // the component that the second part has too few: looked up, never summed
        for (int i = tid; i < ROWS * 3 * D::kCpStride; i += kDecThreads) cpbuf[i] = 0.0f;
    }
    if constexpr (MINBLOCKS > 1) {
        auto stage = [&](int dst_off, int src_off, int bytes) {
            for (int i = tid * 16; i < bytes; i += kDecThreads * 16)
                *reinterpret_cast<u32x4_t*>(lds + dst_off + i) = *reinterpret_cast<const u32x4_t*>(model + src_off + i);
        };
        if constexpr (D::kBiasInLds) stage(D::kBiasOff, Lay::kWeightBytes, D::kBiasBytes);
        if constexpr (D::kFirstInLds) stage(D::kFirstOff, Lay::w_off(0), D::kFirstBytes);
        if constexpr (D::kHeadInLds) stage(D::kHeadWOff, Lay::w_off(Net::kLayers - 1), D::kHeadBytes);
    }
    // this wave's weights stay in registers (all that is not staged above), for every band the workgroup decodes
    WaveNet<Net, (MINBLOCKS > 1), 0> net;
    net.load(model, lds, lane, wave);
    constexpr bool kFilled = MINBLOCKS == 1 && (D::kParts > 1 ? Net::kKeepAwake : Net::kKeepAwakeWide);
    using KeepAwake = Awake<kFilled>;
    KeepAwake awake;
    const float lut_scale = *reinterpret_cast<const float*>(model + Lay::kLutScaleOff);
    const int total_bands = n * nbands;

    // network role: this lane's first-layer inputs are runs of four consecutive ring values
    // (ring row, offset within the row's window that starts at column c-2); a run the
    // network does not use reads as zero
    uint32_t run_at[KB0][2];         // LDS offset of the run for a window at slot 0
    bool run_odd[KB0][2];            // does the run start at an odd element of the window?
    bool run_used[KB0][2];
#pragma unroll
    for (int kbi = 0; kbi < KB0; ++kbi) {
#pragma unroll
        for (int half = 0; half < 2; ++half) {
            int dr = 0, off = 0;
            run_used[kbi][half] = Net::run_desc(kbi, g, half, dr, off);
            run_at[kbi][half] = D::kRingOff + 2u * (((ROWS == 16 ? nl : nl & (ROWS - 1)) + 2 + dr) * D::kRingRowElems + off);
            run_odd[kbi][half] = has_odd_runs<Net>() && (off & 1) != 0;
        }
    }

    // The grid has at most as many workgroups as the chip holds at once, with one per unit also no more than bands can
    // run at a time (choose_decode), and a workgroup decodes band after band:
    // it takes a ticket, decodes that band, takes the next.  A band only ever waits for the band above it (same
    // image), which has a smaller ticket.  Tickets come from a counter, in the order they are asked for, so every
    // ticket below a held one is held by some workgroup or finished.  With two workgroups per compute unit a
    // workgroup's first ticket is its index in the grid instead (the later ones come from the counter): the two
    // workgroups that share a unit are those of index k and k + (number of units), but they ask the counter within
    // microseconds of each other and get neighbouring tickets, so that bands which become runnable at the same time
    // share units while other units hold two workgroups that both wait (measured: 24 images of 768x512 8.2 ms; with
    // the index, the bands on a unit become runnable hundreds of steps apart, 7.3 ms).  Every ticket below a held
    // one is then still held by a workgroup that has been started, or finished: the dispatcher starts workgroups
    // in the order of their index (per die; dies run ahead of each other), and the whole grid fits the chip.
    // Should that ever not hold (a chip shared with another job's resident kernels), the bounded wait for the band
    // above ends the call with an error, not a hang.  With one workgroup per unit the counter stays: the workgroup
    // that is ready first then takes the band that can run first (a single image of 768x512: 5.52 against 5.58 ms
    // by index).  (Leaving the bands beyond the
    // resident ones to the hardware's dispatcher costs up to a third: it deals workgroups to dies and shader
    // engines in strict rotation, and waits for a place in the engine whose turn it is while others are free.)
    // Tickets are numbered band-major (band 0 of every image, then band 1 of every image, ...): the order in
    // which bands become runnable, so a workgroup holds a band that can run rather than one that waits for
    // hundreds of steps, and all images advance together.
    constexpr bool kIndexTickets = MINBLOCKS > 1;
    bool first_band = true;
    for (;;) {
    __syncthreads();                                   // the previous band's last reads of the ring and of misc
    if (tid == 0) {
        const bool stop = __hip_atomic_load(&status[kStAbort], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0;
        misc[0] = stop ? total_bands
                       : (kIndexTickets && first_band) ? (int)blockIdx.x
                       : (kIndexTickets ? (int)gridDim.x : 0) + atomicAdd(&status[kStTicket], 1);
        misc[1] = 0;
    }
    for (int i = tid; i < (ROWS + 2) * D::kRingRowElems; i += kDecThreads) ring[i] = 0;
    __syncthreads();
    const int ticket = __builtin_amdgcn_readfirstlane(misc[0]);
    first_band = false;
    if (ticket >= total_bands) break;
    const int band = ticket / n, im = ticket - band * n;

    const int r0 = band * ROWS;
    const uint64_t rows_total = (uint64_t)n * H;
    const uint64_t table = (uint64_t)kStreamHeader + 8ull * (rows_total + 1);
    const uint64_t payload_bytes = nbytes - table;   // host guarantees nbytes >= table

    if (ticket == 0 && tid == 0) {
        const uint32_t* hdr = reinterpret_cast<const uint32_t*>(stream);
        const uint64_t last = reinterpret_cast<const uint64_t*>(stream + kStreamHeader)[rows_total];
        if (hdr[0] != kStreamMagic || hdr[1] != kStreamVersion || hdr[2] != (uint32_t)n || hdr[3] != (uint32_t)H ||
            hdr[4] != (uint32_t)W || hdr[5] != model_tag<Net>() || hdr[6] != dist || last != payload_bytes)
            set_error(status, PCC_E_STREAM);
    }

    // search role: row of this lane's pixel and its stream reader (the same in all LP lanes of the pixel)
    const int qrow = r0 + q;
    const bool qrow_ok = qrow < H;
    RowReader rd;
    rd.x = rd.y = kRansL; rd.w[0] = rd.w[1] = rd.w[2] = 0; rd.at = 0; rd.nwords = rd.pos = 0; rd.bad = false;
    // The wave's window of the stream starts at its first row's payload: loads address it with 32-bit offsets and read
    // zero behind the stream's end.
    uint64_t window = 0;
    {
        uint64_t a = 0, b = 0;
        if (qrow_ok) {
            const uint64_t* offs = reinterpret_cast<const uint64_t*>(stream + kStreamHeader);
            const uint64_t rowg = (uint64_t)im * H + qrow;
            a = offs[rowg]; b = offs[rowg + 1];
            if (a > b || b > payload_bytes || (b - a) < 16 || ((b - a) & 3) != 0 || (a & 3) != 0 ||
                (b - a) > 4ull * slab_words(W))
                rd.bad = true;
        }
        const uint64_t first = rd.bad ? 0 : a;
        window = (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)first) |
                 ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(first >> 32)) << 32);
        // (rows follow each other in the stream, at most slab_words each: a row that is not within reach is damage)
        if (qrow_ok && !rd.bad && (a < window || a - window > (1u << 30))) rd.bad = true;
        if (qrow_ok && !rd.bad) {
            const uint32_t* payload = reinterpret_cast<const uint32_t*>(stream + table + a);
            rd.x = (uint64_t)payload[0] | ((uint64_t)payload[1] << 32);
            rd.y = (uint64_t)payload[2] | ((uint64_t)payload[3] << 32);
            rd.at = (uint32_t)(a - window) + 16u;
            rd.nwords = (uint32_t)((b - a) / 4) - 4u;
            if (rd.x < kRansL || (rd.x >> 63)) { rd.bad = true; rd.x = kRansL; }
            if (rd.y < kRansL || (rd.y >> 63)) { rd.bad = true; rd.y = kRansL; }
        }
        // The states trade places at every step's bookkeeping, the row's first pixel comes kDelay q + 1 of them on.
        if (((kDelay * q + 1) & 1) != 0) { const uint64_t x = rd.x; rd.x = rd.y; rd.y = x; }
    }
    const uint64_t window_bytes = payload_bytes - window;
    const auto words = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(stream + table + window), 0,
                                                         (int)(uint32_t)(window_bytes < 0xFFFFFFFFull ? window_bytes : 0xFFFFFFFFull),
                                                         0x00020000 /* untyped dwords */);

    uint8_t* out_img = img_out + (size_t)im * H * W * 3;
    const uint32_t* mail_in = mailbox + ((size_t)im * nbands + (band > 0 ? band - 1 : 0)) * 2 * (size_t)W;
    uint32_t* mail_out = mailbox + ((size_t)im * nbands + band) * 2 * (size_t)W;

    const int last_row = min(r0 + ROWS - 1, H - 1);
    const int t_begin = kDelay * r0, t_end = kDelay * last_row + W - 1;
    // The first eight lanes of the fetch wave bring in the rows above the band: even lanes row r0-2 -> ring row 0, odd
    // lanes row r0-1 -> ring row 1, each pair to one of a pixel's four places.  That wave has a round without an out-block in one of the layers (DecLds::kIdleLayer)
    // and does the fetch there, off the path that all four waves share.
    const bool fetcher = band > 0 && tid >= D::kFetchWave * 64 && tid < D::kFetchWave * 64 + 8;
    const uint32_t* mail_row = mail_in + (size_t)(tid & 1) * W;
    // Columns right of the band's first row's column that the fetched row must be known to: row r0-2 is
    // read by the band's first row only; row r0-1 by the first row and, one delay later, by the second.
    const int ahead = (tid & 1) ? (Net::kReach1 > Net::kReach2 - kDelay ? Net::kReach1 : Net::kReach2 - kDelay)
                                : Net::kReach2;
    uint32_t pf = 0;                              // mailbox word for the next column, requested a step early

    // offset, in elements, of place i (0..3) that a pixel's values are written to: two slots in each of the two copies
    auto ring_place = [](int i) { return (i & 1) * 3 * RC + (i >> 1) * D::kRingCopyElems; };
    // bf16 of the three channels of pixel word px into one place of column cc of a ring row
    auto ring_put = [&](int rrow, int cc, int place, uint32_t px) {
        uint16_t* d = ring + rrow * D::kRingRowElems + ring_place(place) + (cc & (RC - 1)) * 3;
        d[0] = (uint16_t)byte_to_bf16(px & 0xFFu);
        d[1] = (uint16_t)byte_to_bf16((px >> 8) & 0xFFu);
        d[2] = (uint16_t)byte_to_bf16((px >> 16) & 0xFFu);
    };
    // Bring columns 0 .. ahead of the two rows above the band into the ring, then keep
    // one column ahead: the step at t needs column (t - t_begin) + ahead.
    // wait_word: the published word of column cc (`have` if that already is one); clears ok on abort.
    auto wait_word = [&](int cc, uint32_t have, bool& ok) -> uint32_t {
        uint32_t v = have, spins = 0;
        while (!(v & kMailTag)) {
            v = __hip_atomic_load(mail_row + cc, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (v & kMailTag) break;
            ++spins;
            if (spins > spin_limit) { set_error(status, PCC_E_INTERNAL); ok = false; break; }
            if ((spins & 63u) == 0u &&
                __hip_atomic_load(&status[kStAbort], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0) {
                ok = false;
                break;
            }
            __builtin_amdgcn_s_sleep(1);
        }
        return v;
    };
    auto give_up = [&]() {
        __hip_atomic_store(&status[kStAbort], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        misc[1] = 1;
    };
    if (fetcher) {
        bool ok = true;
        for (int cc = 0; cc <= ahead; ++cc) {
            if (ok && cc < W) {
                const uint32_t v = wait_word(cc, 0u, ok);
                if (ok) ring_put(tid & 1, cc, (tid >> 1) & 3, v);
            }
        }
        // Start one column further behind the band above than the data requires: the word requested a
        // step ahead has then been published when it is asked for, and is not waited for at the step's end.
        if (ok && W > ahead + 1) pf = wait_word(ahead + 1, 0u, ok);
        if (!ok) give_up();
    }
    lds_barrier();

    // Per step: the word of column (t - t_begin) + ahead + 1, requested in the step before, goes to the ring for the
    // next step's gather, and the column after it is requested; columns right of the image read as zero.  The fetch
    // wave does this where it has no out-block to compute, in layer kIdleLayer (or at the step's end if there is no such
    // layer): the check of the word that has arrived (fetch_check), then the ring write, which lies behind the barrier
    // that follows this step's gather and before the one that ends the step (fetch_put).  Where the first layer has such a
    // round too, the request (fetch_request) is issued at the very end of the step, after the pixel has been
    // published: the later a word is asked for, the closer the band can follow the band above (a word asked for
    // before it is published is asked for again, which holds the fetch wave up), and the load is back when layer
    // kIdleLayer of the next step checks it.  The request always loads (the row's last word again beyond the image): no
    // branch, the value is not used then.
    uint32_t fetched = 0;
    constexpr bool kLateRequest = D::kIdleInFirstLayer;
    auto fetch_check = [&](int t) __attribute__((always_inline)) {
        if (fetcher) {
            const int cc = t - t_begin + ahead + 1;
            uint32_t v = cc < W ? pf : 0u;
            if (cc < W && !(v & kMailTag)) {            // seldom: the band above is less than a step ahead
                bool ok = true;
                v = wait_word(cc, v, ok);
                if (!ok) give_up();
            }
            fetched = v;
        }
    };
    auto fetch_put = [&](int t) __attribute__((always_inline)) {
        if (fetcher) {
            const int cc = t - t_begin + ahead + 1;
            if (cc < W + kMaxReach) ring_put(tid & 1, cc, (tid >> 1) & 3, fetched);
            if constexpr (!kLateRequest) pf = __hip_atomic_load(mail_row + min(cc + 1, W - 1), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    };
    auto fetch_request = [&](int t) __attribute__((always_inline)) {
        if (fetcher) {
            const int cc = t - t_begin + ahead + 1;
            pf = __hip_atomic_load(mail_row + min(cc + 1, W - 1), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    };
    // The pixels decoded in step t_done go from the ring (which holds a pixel for kRingCols steps, as three bf16 of
    // its bytes) to the image: by the first ROWS lanes of the storing wave, a lane per row of the band, a step later,
    // where that wave has no out-block to compute, instead of by the lanes that decoded them at the end of their
    // step, where all four waves would wait for it.  In two halves: the ring read (in the first layer if that has such a
    // round), then the stores.  The image is
    // addressed as a buffer: lanes and columns without a pixel store beyond its end, which the hardware drops.
    uint16_t held[3] = {0, 0, 0};
    const auto image = __builtin_amdgcn_make_buffer_rsrc(out_img, 0, 3 * H * W, 0x00020000 /* untyped */);
    const uint16_t* held_at = ring + ((lane & (ROWS - 1)) + 2) * D::kRingRowElems;
    const uint32_t store_end = lane < ROWS && r0 + lane < H ? (uint32_t)W : 0u;
    auto store_read = [&](int t_done) __attribute__((always_inline)) {
        const int cc = t_done - kDelay * (r0 + lane);
        const uint16_t* e = held_at + (cc & (RC - 1)) * 3;
#pragma unroll
        for (int ch = 0; ch < 3; ++ch) held[ch] = e[ch];
    };
    auto store_write = [&](int t_done) __attribute__((always_inline)) {
        const int cc = t_done - kDelay * (r0 + lane);
        uint32_t at = 3u * (uint32_t)((r0 + lane) * W + cc);
        asm volatile("" : "+v"(at));        // scheduling only: no branch round its computation
        at = (uint32_t)cc < store_end ? at : 0xFFFFFFF0u;
        const uint32_t x0 = (uint32_t)__uint_as_float((uint32_t)held[0] << 16), x1 = (uint32_t)__uint_as_float((uint32_t)held[1] << 16),
                       x2 = (uint32_t)__uint_as_float((uint32_t)held[2] << 16);
        __builtin_amdgcn_raw_buffer_store_b16((short)(x0 | (x1 << 8)), image, (int)at, 0, 0);
        __builtin_amdgcn_raw_buffer_store_b8((char)x2, image, (int)at, 2, 0);
    };
    constexpr bool kStoreInIdle = D::kIdleSlack > 0;
    int t = t_begin;
    // The bookkeeping of a step's pixel that the symbols themselves do not wait for: the pops of G and B, the words the
    // next pixel may read, and where that pixel goes in the ring.  It is done a step later, in the shadow of the matrix
    // instructions of the second layer and the head (settle); R's pop has to be done before B's search and is done during G's.
    // Two VALU instructions issue for free beside an MFMA of 16 cycles; done at the end of the step, as all three pops
    // once were, this was 500 of its 7,250 cycles.
    Found found_g = {0, 0, 0, 1, 0}, found_b = {0, 0, 0, 1, 0};
    uint32_t active = 0, settle_active = 0;            // does this step's / the last step's pixel exist?  (masks)
    float slot1_x = 0.0f, slot1_y = 0.0f;
    uint16_t* ring_elem = nullptr;                     // where this lane writes the pixel: [channel]
    uint32_t mail_px = 0;
    const uint32_t row_end = qrow_ok ? (uint32_t)W : 0u, ring_end = qrow_ok && j < 4 ? (uint32_t)(W + kMaxReach) : 0u;
    const uint32_t ring_at = D::kRingOff + 2u * ((q + 2) * D::kRingRowElems + ring_place(j & 3));
    // where a step's gather reads: the window's offset for runs that start at an even element of it and at an odd one
    uint32_t window_at[2];
    auto gather_window = [&](int at) __attribute__((always_inline)) {
        const uint32_t slot = (uint32_t)(at - kDelay * (r0 + (ROWS == 16 ? nl : nl & (ROWS - 1))) - 2) & (RC - 1);
        const uint32_t second = (slot & 1u) * (2u * D::kRingCopyElems);
        window_at[0] = 6u * slot + second;
        window_at[1] = 6u * slot + 2u * D::kRingCopyElems - second;
    };
    gather_window(t);
    const float* coupling_base = headout + q * D::kHeadStride + (D::kParts > 1 ? 3 * PK * part : 0);
    // The lane picks come first, in two stages, each where the next wait for LDS is one of the network's own.
    Interval settle_g = {0, 0, 0}, settle_b = {0, 0, 0};
    auto settle_pick = [&]() __attribute__((always_inline)) {
        interval_pick(found_g, sl, settle_g);
        interval_pick(found_b, sl, settle_b);
    };
    auto settle_pick_upper = [&]() __attribute__((always_inline)) {
        interval_pick_upper(found_g, sl, settle_g);
        interval_pick_upper(found_b, sl, settle_b);
    };
    auto settle_pops = [&]() __attribute__((always_inline)) {
        uint32_t start, freq;
        interval_of(found_g, settle_g, start, freq);
        reader_pop(rd, rd.y, start, freq, settle_active);
        interval_of(found_b, settle_b, start, freq);
        reader_pop(rd, rd.x, start, freq, settle_active);
        asm volatile("" : "+v"(rd.x), "+v"(rd.y), "+v"(rd.pos));     // scheduling only: done here
        const uint64_t x = rd.x;       // the next pixel's first symbol is on the state of this one's second
        rd.x = rd.y;
        rd.y = x;
    };
    // Has this band given up?  The fetch wave says so where it checks the row above: in layer kIdleLayer, and then all waves
    // read the flag during B's search, behind that layer's barrier; or, where no layer leaves it time, at the step's end,
    // and then they read it in the next step's head, in front of that layer's barrier (in the gather it cost 1 % of the
    // step).  A barrier lies between write and read either way, so that all waves leave after the same step.
    constexpr bool kStopInSearch = D::kIdleSlack > 0;
    int stop = 0;
    auto settle = [&](auto layer) __attribute__((always_inline)) {
        constexpr int L = decltype(layer)::value;
        if constexpr (L == 0) settle_pick_upper();
        if constexpr (L == 1) {
            settle_pops();
            typedef uint32_t u32x3_t __attribute__((ext_vector_type(3)));
            const u32x3_t next = __builtin_bit_cast(u32x3_t, __builtin_amdgcn_raw_buffer_load_b96(words, (int)(rd.at + 4u * rd.pos), 0, 0));
            rd.w[0] = next.x; rd.w[1] = next.y; rd.w[2] = next.z;
        }
        if constexpr (L == Net::kLayers - 1) {
            if constexpr (!kStopInSearch) stop = misc[1];
            slot1_x = (float)(((uint32_t)rd.x & 0xFFFFu) + 1u);
            slot1_y = (float)(((uint32_t)rd.y & 0xFFFFu) + 1u);
            const int c = t - kDelay * qrow;
            active = mask_of((uint32_t)c < row_end);
            // Lanes 0 to 3 of a pixel write its four places; the columns right of the image are written as zeros when
            // their turn comes; all other lanes write where nobody reads.
            const bool writes = (uint32_t)c < ring_end;
            uint32_t elem = ring_at + 6u * (uint32_t)(c & (RC - 1));
            asm volatile("" : "+v"(elem));         // scheduling only: no branch round its computation
            elem = writes ? elem : (uint32_t)(D::kSinkOff + 4 * lane);
            gather_window(t + 1);
            // scheduling only: done here
            asm volatile("" : "+v"(slot1_x), "+v"(slot1_y), "+v"(elem), "+v"(window_at[0]), "+v"(window_at[1]));
            ring_elem = reinterpret_cast<uint16_t*>(lds + elem);
        }
    };
    // the last step's pixel of the band's last two rows, for the band below
    auto mail = [&](int t_done) __attribute__((always_inline)) {
        if (j == 0 && q >= ROWS - 2 && settle_active != 0)
            __hip_atomic_store(mail_out + (size_t)(q - (ROWS - 2)) * W + (t_done - kDelay * qrow), mail_px, __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
    };

    PhaseClock clk;
    clk.reset();
    // The steps, for a wave of a given role.  Each role has a loop of its own: a taken branch costs up to a hundred cycles
    // where four waves take it together (they all fetch from its target), so the loop has none but its own end.
    auto steps = [&](auto role) __attribute__((always_inline)) {
    using Role = decltype(role);
    auto idle = [&](auto layer) __attribute__((always_inline)) {
        constexpr int L = decltype(layer)::value;
        if constexpr (D::kIdleInFirstLayer && L == 0) {
            if constexpr (Role::kStores) store_read(t - 1);
        } else {
            if constexpr (Role::kFetches) { fetch_check(t); fetch_put(t); }
            if constexpr (Role::kStores) {
                if constexpr (!D::kIdleInFirstLayer) store_read(t - 1);
                store_write(t - 1);
            }
        }
    };
    // Gather C_ij from the ring (zeros stand for pixels outside the image), for the step's tile of 16 pixels; every wave
    // builds the full tile.  A run is four consecutive bf16 values of a ring row: two dwords, which are the operand's
    // registers as they stand.
    uint32_t v[KB0][4];
    auto gather = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int kbi = 0; kbi < KB0; ++kbi) {
#pragma unroll
            for (int half = 0; half < 2; ++half) {
                const uint32_t* run = reinterpret_cast<const uint32_t*>(lds + run_at[kbi][half] + window_at[run_odd[kbi][half] ? 1 : 0]);
                v[kbi][2 * half] = run[0];
                v[kbi][2 * half + 1] = run[1];
            }
        }
        asm volatile("" ::: "memory");
        settle_pick();
        __builtin_amdgcn_sched_barrier(0);      // scheduling only: all of these are asked for before any is waited for
    };
    do {
        clk.mark(kPhTop);
        gather();

        u32x4_t in1[KB0][2];
        {
            if constexpr (Role::kStores) mail(t - 1);
            // one batch of LDS reads
            static_assert(KB0 == 1 || KB0 == 2, "the scheduling barrier below lists the reads explicitly");
            if constexpr (KB0 == 1)
                asm volatile("" : "+v"(v[0][0]), "+v"(v[0][1]), "+v"(v[0][2]), "+v"(v[0][3]));
            else
                asm volatile("" : "+v"(v[0][0]), "+v"(v[0][1]), "+v"(v[0][2]), "+v"(v[0][3]), "+v"(v[KB0 - 1][0]),
                                  "+v"(v[KB0 - 1][1]), "+v"(v[KB0 - 1][2]), "+v"(v[KB0 - 1][3]));
#pragma unroll
            for (int kbi = 0; kbi < KB0; ++kbi) {
                const uint32_t m0 = run_used[kbi][0] ? 0xFFFFFFFFu : 0u, m1 = run_used[kbi][1] ? 0xFFFFFFFFu : 0u;
                in1[kbi][0].x = v[kbi][0] & m0;
                in1[kbi][0].y = v[kbi][1] & m0;
                in1[kbi][0].z = v[kbi][2] & m1;
                in1[kbi][0].w = v[kbi][3] & m1;
                in1[kbi][1] = in1[kbi][0];   // unused (layer-1 inputs are exact)
            }
        }

        clk.mark(kPhGather);
        // ---- network, layers meeting in LDS
        net.template run<ActLds<ROWS>, Role::kOwnsLast>(in1, lane, wave, minus_one, act0, act1, headout, idle, settle, awake, clk);

        // ---- mixtures: lane jj < 3K of pixel q prepares component jj % K of channel jj / K
        auto prepare = [&](int jj) __attribute__((always_inline)) {
            const int ch = jj / K, k = jj - K * ch;
            const float* hc = headout + q * D::kHeadStride + ch * HS;
            float pk, mk, ak;
            if constexpr (K >= 5) {
                // only this component's sigma and weight are computed (measured faster for K = 5, slower for K = 3)
                // the channel's logits (for the softmax sum) and this component's own three values
                constexpr int NV = (K + 3) / 4;
                f32x4_t lv[NV];
#pragma unroll
                for (int i = 0; i < NV; ++i) lv[i] = reinterpret_cast<const f32x4_t*>(hc)[i];
                float logit_k = hc[k], mu_k = hc[K + k], ls_k = hc[2 * K + k];
                awake.template keep<KeepAwake::kBehindHeadReads>();
                // scheduling only: all reads are issued before the first is used (whole vectors, so that the registers of
                // the padding are not wanted for the next read's address)
                asm volatile("" : "+v"(lv[0]), "+v"(lv[NV - 1]), "+v"(logit_k), "+v"(mu_k), "+v"(ls_k));
                float logits[K];
#pragma unroll
                for (int i = 0; i < K; ++i) {
                    const f32x4_t v = lv[i >> 2];
                    logits[i] = (i & 3) == 0 ? v.x : (i & 3) == 1 ? v.y : (i & 3) == 2 ? v.z : v.w;
                }
                channel_setup_one<K>(logits, logit_k, mu_k, ls_k, lut_scale, pk, mk, ak);
            } else {
                float raw[3 * K];
                lds_read_floats<3 * K>(hc, raw);
                ChanParams<K> all;
                channel_setup<K>(raw, lut_scale, all);
                pk = all.pi[0]; mk = all.mu[0]; ak = all.a[0];
#pragma unroll
                for (int kk = 1; kk < K; ++kk) if (k == kk) { pk = all.pi[kk]; mk = all.mu[kk]; ak = all.a[kk]; }
            }
            float* dst = jj < 3 * K ? cpbuf + (q * 3 + ch) * D::kCpStride + (D::kParts > 1 ? k / PK * D::kPartStride + k % PK : k)
                                    : reinterpret_cast<float*>(lds + D::kSinkOff + 4 * lane);
            dst[0] = pk; dst[PK] = mk; dst[2 * PK] = ak;
        };
        if constexpr (3 * K <= LP) {
            prepare(j);        // (lanes without a component prepare what nobody reads: no branch)
        } else {
            prepare(j);
            prepare(j + LP);
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");

        // What the three searches need, channel by channel: R's mixture now, G's and B's (with their coupling
        // coefficients) while the search before them waits for its last table reads.  Requested all at once, the reads
        // of the four waves keep LDS busy for hundreds of cycles in front of R's first table reads.
        ChanParams<PK> cpr, cpg, cpb;
        float alpha[PK], beta[PK], gamma[PK];
        // (with two workgroups per unit the address is made again in every step, and every wave makes mail_px: 29 spilled registers, not 41)
        const float* coupling_at = MINBLOCKS > 1 ? headout + q * D::kHeadStride : coupling_base;
        // `tail` receives the last vector read, padding included: the caller keeps it in use until the values are
        // consumed (register allocation only: a padding register that is free at once is handed to the next read,
        // which then has to wait for this one)
        auto load_cp = [&](int ch, ChanParams<PK>& cp, f32x4_t& tail) __attribute__((always_inline)) {
            constexpr int NV = (3 * PK + 3) / 4;
            const f32x4_t* src = reinterpret_cast<const f32x4_t*>(cpbuf + (q * 3 + ch) * D::kCpStride + (D::kParts > 1 ? part * D::kPartStride : 0));
            f32x4_t vv[NV];
#pragma unroll
            for (int i = 0; i < NV; ++i) vv[i] = src[i];
            tail = vv[NV - 1];
            auto at = [&](int i) { const f32x4_t w = vv[i >> 2]; return (i & 3) == 0 ? w.x : (i & 3) == 1 ? w.y : (i & 3) == 2 ? w.z : w.w; };
#pragma unroll
            for (int k = 0; k < PK; ++k) { cp.pi[k] = at(k); cp.mu[k] = at(PK + k); cp.a[k] = at(2 * PK + k); }
        };
        f32x4_t tail_r, tail_g, tail_b;
        // coupling coefficients: canonical head outputs 9K.. (alpha), 10K.. (beta), 11K.. (gamma), wherever the head's
        // (group, register) layout put them; for a component that the lane's part does not have it is the padding behind them
        auto coupling = [&](auto first, auto kc) __attribute__((always_inline)) {
            using Head = std::conditional_t<(MINBLOCKS > 1 && Net::kSharedByCoefficient), SharedHead<Net>, Net>;
            constexpr int c = decltype(first)::value, k = decltype(kc)::value, mine = head_slot<Net, Head>(c + k);
            static_assert(D::kParts == 1 || head_slot<Net, Head>(c + K - 1) == mine + 3 * (K - 1 - k), "one distance between the parts");
            static_assert(D::kParts == 1 || head_slot<Net, Head>(c) + 3 * (D::kParts * PK - 1) < D::kHeadStride, "the padding is there");
            return coupling_at[mine];
        };
        auto load_g = [&]() __attribute__((always_inline)) {
            load_cp(1, cpg, tail_g);
            static_for<0, PK>([&](auto kc) { alpha[decltype(kc)::value] = coupling(std::integral_constant<int, 9 * K>{}, kc); });
        };
        auto load_b = [&]() __attribute__((always_inline)) {
            load_cp(2, cpb, tail_b);
            static_for<0, PK>([&](auto kc) {
                constexpr int k = decltype(kc)::value;
                beta[k] = coupling(std::integral_constant<int, 10 * K>{}, kc);
                gamma[k] = coupling(std::integral_constant<int, 11 * K>{}, kc);
            });
        };
        auto load_nothing = [&]() __attribute__((always_inline)) {};
        auto load_stop = [&]() __attribute__((always_inline)) { if constexpr (kStopInSearch) stop = misc[1]; };
        load_cp(0, cpr, tail_r);
        asm volatile("" ::: "memory");
        awake.template keep<KeepAwake::kBehindMixtureReads>();

        clk.mark(kPhMixture);
        uint32_t start, freq;
        Found found_r;
        // R
        const int sr = group_search<K, PK>(cpr, slot1_x, lut, sl, found_r, load_nothing, load_g);
        float rhat = (float)sr;
        ring_elem[0] = bf16_bits(rhat) & active;
        Interval iv_r;
        interval_pick(found_r, sl, iv_r);
        rhat = rhat * (1.0f / 256.0f);
        clk.mark(kPhR);
        // G given R; meanwhile R's pop, whose state B is coded on
        asm volatile("" : "+v"(rhat) : "v"(tail_r), "v"(tail_g));    // (tied to a value known only now: stays here)
        couple_green<PK>(cpg, alpha, rhat);
        auto pick_r_upper = [&]() __attribute__((always_inline)) { interval_pick_upper(found_r, sl, iv_r); };
        auto pop_r = [&]() __attribute__((always_inline)) {
            load_b();
            interval_of(found_r, iv_r, start, freq);
            reader_pop(rd, rd.x, start, freq, active);
            asm volatile("" : "+v"(rd.x), "+v"(rd.w[0]), "+v"(rd.w[1]), "+v"(rd.pos));     // scheduling only: done here
        };
        const int sg = group_search<K, PK>(cpg, slot1_y, lut, sl, found_g, pick_r_upper, pop_r);
        float ghat = (float)sg;
        ring_elem[1] = bf16_bits(ghat) & active;
        ghat = ghat * (1.0f / 256.0f);
        clk.mark(kPhG);
        // B given R, G
        asm volatile("" : "+v"(ghat) : "v"(tail_b));
        couple_blue<PK>(cpb, beta, gamma, rhat, ghat);
        const int sb = group_search<K, PK>(cpb, (float)(((uint32_t)rd.x & 0xFFFFu) + 1u), lut, sl, found_b, load_stop, load_nothing);
        ring_elem[2] = bf16_bits((float)sb) & active;
        clk.mark(kPhB);

        // ---- publish
        // Made where it is stored.  Not where every wave makes it: two workgroups per unit (spilled registers, above), and bands of 16 rows
        // without fills of the waits, in whose place it is (us, 8 and 12 images of 768x512 and one of 4096x2160: diagonal 3,492, 4,536, 16,398, by
        // every wave 3,444, 4,480, 16,192; 64 filters 5,031, 5,038, 22,578 and 4,943, 4,980, 22,273; with fills 1 % less to 1 % more).
        constexpr bool kMailEverywhere = MINBLOCKS > 1 || (D::kParts == 1 && !kFilled);
        if constexpr (kMailEverywhere || Role::kStores) mail_px = (uint32_t)sr | ((uint32_t)sg << 8) | ((uint32_t)sb << 16) | kMailTag;
        settle_active = active;
        asm volatile("" : "+v"(found_b.c2), "+v"(mail_px), "+v"(settle_active));   // scheduling only: while the ring is written
        if constexpr (!kStoreInIdle) {
            if (j == 0 && active != 0) {
                uint8_t* o = out_img + ((size_t)qrow * W + (t - kDelay * qrow)) * 3;
                o[0] = (uint8_t)sr; o[1] = (uint8_t)sg; o[2] = (uint8_t)sb;
            }
        }
        if constexpr (kLateRequest && Role::kFetches) fetch_request(t);
        clk.mark(kPhPublish);
        // ---- rows above the band, where no layer leaves the fetch wave spare time for it
        if constexpr (D::kIdleSlack == 0 && Role::kFetches) { fetch_check(t); fetch_put(t); }
        clk.mark(kPhFetch);
        lds_barrier();
        clk.mark(kPhBarrier);
        ++t;
    } while (((int)(t <= t_end) & (int)(__builtin_amdgcn_readfirstlane(stop) == 0)) != 0);
    };
    if constexpr (D::kFetchWave == D::kStoreWave) {
        if (wave_s != D::kStoreWave) steps(StepRole<false, false, true>());
        else steps(StepRole<true, true, D::kStoreWave < D::kFirstIdleWave>());
    } else {
        if (wave_s < D::kFetchWave) steps(StepRole<false, false, true>());
        else if (wave_s == D::kFetchWave) steps(StepRole<true, false, false>());
        else steps(StepRole<false, true, false>());
    }
    awake.used();
#ifdef PCC_PHASE_TIMING
    if (ticket == min(kPhaseTicket, total_bands - 1) && lane == 0) {
        for (int i = 0; i < kPhCount; ++i) phase_cycles[wave][i] = clk.acc[i];
        phase_cycles[wave][kPhCount] = (unsigned long long)(t_end - t_begin + 1);
    }
#endif
    if constexpr (kStoreInIdle) if (wave_s == D::kStoreWave) { store_read(t_end); store_write(t_end); }      // the last step's pixels (the loop ended behind a barrier)
    if (misc[1] != 0) break;    // uniform: the last step's barriers lie behind any write.  The call has failed; no further bands.
    if (wave_s == D::kStoreWave) mail(t_end);
    settle_pick();
    settle_pick_upper();
    settle_pops();
    // every row's states are back where the coder started and its words are used up, neither more nor fewer
    if (j == 0 && qrow_ok && (rd.bad || rd.x != kRansL || rd.y != kRansL || rd.pos != rd.nwords)) set_error(status, PCC_E_STREAM);
    }
