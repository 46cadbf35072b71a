// One output tile of pgk_gemm_f32_terms.h, as the statements of a function: included inside the kernels there, not a header of its own.  What
// they expect: Cfg, VIEW, TIMED and INSIDE, the arguments p and out_mode, and lds_a, lds_b (operands) and rs_buf (row sums of the wave
// columns, then the tile's column biases, then its row biases) in LDS.
// INSIDE (of a convolution's input): every position that the tile reads lies inside the rows, and a thread's two columns side by side.
    constexpr int BM = Cfg::BM, BN = Cfg::BN, BK = Cfg::BK;
    constexpr int TM16 = Cfg::TM16, TN16 = Cfg::TN16, A_KV = Cfg::A_KV, A_CH = 2, B_CH = 2;
    constexpr bool BT = Cfg::BT;
    constexpr int BIAS_N = Cfg::BIAS_N;
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / Cfg::WGN, wn = wave % Cfg::WGN;
    // phase stamp k of this workgroup: (cycles, 100 MHz ticks); see pgk_probe_gemm_phases
    auto stamp = [&](int k) __attribute__((always_inline)) {
        if constexpr (TIMED) {
            __builtin_amdgcn_sched_barrier(0);
            const unsigned long long cyc = __builtin_readcyclecounter();
            const unsigned long long tick = __builtin_amdgcn_s_memrealtime();
            if (wave == 0) {
                unsigned long long* at = p.stamps + (size_t)blockIdx.x * kStampWords + 2 * k;
                at[0] = cyc;
                at[1] = tick;
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    stamp(0);
    if constexpr (TIMED) {
        if (wave == 0) {
            p.stamps[(size_t)blockIdx.x * kStampWords + 12] = (unsigned long long)__builtin_amdgcn_s_getreg(63492);   // HW_ID, 32 bits
            p.stamps[(size_t)blockIdx.x * kStampWords + 13] = (unsigned long long)__builtin_amdgcn_s_getreg(63508);   // XCC_ID, 32 bits
        }
    }

    // ---- which tile, batch entry and K slice this workgroup owns
    const unsigned int tiles = (unsigned int)p.tiles_m * (unsigned int)p.tiles_n;
    const unsigned int logical = xcd_remap(blockIdx.x, gridDim.x);
    const unsigned int z = logical / tiles;
    int tm, tn;
    tile_coords(logical - z * tiles, p.tiles_m, p.tiles_n, p.group_m, tm, tn);
    const int b = (int)(z / (unsigned int)p.splits);
    const int sp = (int)(z - (unsigned int)b * (unsigned int)p.splits);
    const int k_begin = sp * p.k_slice;
    const int k_end = (k_begin + p.k_slice < p.K) ? (k_begin + p.k_slice) : p.K;
    const int KT = (k_end - k_begin + BK - 1) / BK;
    const int k_last = (k_end - k_begin) - (KT - 1) * BK;        // k values of the last step that exist
    // (see the same variable in pgk_gemm_mfma_kernel.h: skinny products start their K loops apart)
    const int k_rot = (VIEW == VIEW_GEMM && p.k_rotate && k_last == BK)
                          ? (int)((unsigned int)(p.batch > 1 ? b : tm + tn) % (unsigned int)KT) : 0;

    const unsigned char* const Ag = (const unsigned char*)p.A +
        ((size_t)b * (size_t)p.a_batch_stride + (size_t)tm * BM * p.K + (size_t)k_begin) * 4;
    const unsigned char* b_src = (const unsigned char*)p.B;
    int ldb = p.ldb;
    long long b_batch_stride = p.b_batch_stride;
    long long b_col0 = (long long)tn * BN;
    if constexpr (VIEW == VIEW_CONV) {
        b_col0 += p.b_col_shift;
#pragma unroll
        for (int e = 0; e < 3; ++e) {
            if (p.edge_B[e] && p.edge_tn[e] == tn) {
                b_src = (const unsigned char*)p.edge_B[e];
                ldb = p.edge_ldb;
                b_batch_stride = p.edge_batch_stride;
                b_col0 = 0;
            }
        }
    }
    const unsigned char* const Bg = b_src +
        (BT ? ((long long)b * b_batch_stride + b_col0 * ldb + (long long)k_begin) * 4
            : ((long long)b * b_batch_stride + (long long)k_begin * ldb + b_col0) * 4);
    const size_t a_step = (size_t)BK * 4;
    const size_t b_step = BT ? (size_t)BK * 4 : (size_t)BK * ldb * 4;
    // one past the last byte of A and of B: what a partial last step, or a row's last columns, would
    // read behind the array the buffer resource's size check cuts off (a convolution's copies and
    // strips hold every column its tiles read, as they are laid out for that)
    const unsigned char* const A_end = (const unsigned char*)p.A +
        ((size_t)(p.batch - 1) * (size_t)p.a_batch_stride + (size_t)p.M * p.K) * 4;
    const unsigned char* const B_end = (const unsigned char*)p.B +
        ((size_t)(p.batch - 1) * (size_t)p.b_batch_stride + (size_t)(BT ? p.N : p.K) * p.ldb) * 4;
    auto records = [](const unsigned char* base, const unsigned char* end) __attribute__((always_inline)) -> int {
        const size_t left = (size_t)(end - base);
        return left < 0xffffffffull ? (int)(unsigned int)left : (int)0xffffffffu;
    };

    const int m_rem = (p.M - tm * BM) < BM ? (p.M - tm * BM) : BM;
    const int n_rem = (p.N - tn * BN) < BN ? (p.N - tn * BN) : BN;

    constexpr bool BIAS_PER_ROW = VIEW != VIEW_GEMM;
    float bias_pre = 0.0f;
    if (p.bias && out_mode == 0) {
        if constexpr (BIAS_PER_ROW) { if (tid < m_rem) bias_pre = p.bias[(size_t)tm * BM + tid]; }
        else if (tid < n_rem) bias_pre = p.bias[(size_t)tn * BN + tid];
    }

    // ---- what this thread copies: of a transposed B the eight k values of chunk tid % 4 of
    // two neighbouring rows, of A the same or (fewer rows) a half or a quarter of a chunk; of a plain B the eight k rows
    // 8 wave .. of two neighbouring columns.  Rows and columns past the edge re-read the last ones.
    constexpr int A_PER_ROW = BK / A_KV;                          // threads per row of A
    const int my_row = 2 * (tid >> 2), my_chunk = tid & 3;
    const int a_row = 2 * (tid / A_PER_ROW), a_k0 = (tid % A_PER_ROW) * A_KV;
    // (a convolution's weights: the rows past the last one lie behind the end of A and read as zero)
    unsigned int voff_a[A_CH], voff_b[BT || VIEW == VIEW_INPUT ? B_CH : 1];
#pragma unroll
    for (int t = 0; t < A_CH; ++t) {
        const int r = a_row + t;
        voff_a[t] = (unsigned int)(VIEW == VIEW_INPUT || r < m_rem ? r : m_rem - 1) * (unsigned int)p.K * 4u + (unsigned int)a_k0 * 4u;
    }
    if constexpr (BT) {
#pragma unroll
        for (int t = 0; t < B_CH; ++t) {
            const int r = my_row + t;
            voff_b[t] = (unsigned int)(r < n_rem ? r : n_rem - 1) * (unsigned int)ldb * 4u + (unsigned int)my_chunk * 32u;
        }
    } else if constexpr (VIEW == VIEW_INPUT) {
#pragma unroll
        for (int t = 0; t < B_CH; ++t) {
            const int c = 2 * lane + t;
            voff_b[t] = (((unsigned int)tn * BN + (unsigned int)(c < n_rem ? c : n_rem - 1)) * (unsigned int)p.conv_stride -
                         (INSIDE ? 0u : (unsigned int)p.conv_pad)) * 4u;
        }
    } else {
        const int c = 2 * lane, last = (n_rem - 1) / 2 * 2;
        voff_b[0] = (unsigned int)(8 * wave) * (unsigned int)ldb * 4u + (unsigned int)(c < n_rem ? c : last) * 4u;
    }
    const unsigned int b_row_bytes = (unsigned int)ldb * 4u;
    // ... and where it goes in LDS (see "LDS layout")
    auto frag_pos = [](int row, int g) __attribute__((always_inline)) {
        return (row >> 4) * 1024 + g * 256 + (((((row & 15) >> 1) + 8 * (row & 1)) ^ (6 * g & 7)) * 16);
    };
    // (the odd row of a pair lies kOddRow bytes behind the even one, whose index has that bit clear)
    constexpr int kOddRow = 128;
    const int wpos_a = frag_pos(a_row, a_k0 >> 3) + (a_k0 & 7) * 2;
    const int wpos_b = BT ? frag_pos(my_row, my_chunk) : frag_pos(2 * lane, wave);

    // ---- global -> registers, one step: ra[t] = k values of a row of A, rb[t] = of a column of B.
    // Where the next step starts is running state, as in pgk_gemm_mfma_kernel.h.
    float ra[A_CH][A_KV], rb[B_CH][8];
    size_t a_off = 0, b_off = 0;
    int next_step = 0, b_row_step = 0, b_taps_done = 0;
    long long tap_of_lane = 0;
    if constexpr (VIEW == VIEW_CONV) {
        const __attribute__((address_space(4))) long long* const tap_table =
            (const __attribute__((address_space(4))) long long*)((const __attribute__((address_space(4))) char*)
                __builtin_amdgcn_kernarg_segment_ptr() + offsetof(GemmArgs, b_tap_off));
        tap_of_lane = tap_table[lane & 31];
    }
    auto tap_entry = [&](int t) __attribute__((always_inline)) -> long long {
        const unsigned int lo = (unsigned int)__builtin_amdgcn_readlane((int)(unsigned int)(unsigned long long)tap_of_lane, t);
        const unsigned int hi = (unsigned int)__builtin_amdgcn_readlane((int)(unsigned int)((unsigned long long)tap_of_lane >> 32), t);
        return (long long)(((unsigned long long)hi << 32) | lo);
    };
    const long long b_tap_jump = VIEW == VIEW_CONV ? (long long)p.b_tap_step * 4 - (long long)p.b_tiles_per_tap * (long long)b_step : 0;
    // A convolution's input: lane e (of eight, and again in the other lanes) follows the wave's k row e of the step that is being
    // loaded: its tap, and where it starts in x, in bytes, without the padding.  What a load needs of it comes from readlane.
    const unsigned int in_row_bytes = (unsigned int)p.conv_len * 4u, in_dil = (unsigned int)p.conv_dil * 4u;
    const int in_taps = VIEW == VIEW_INPUT ? p.conv_kw : 1;
    const int in_step_ch = __builtin_amdgcn_readfirstlane(BK / in_taps), in_step_tap = BK - in_step_ch * in_taps;
    const unsigned int in_step_off = (unsigned int)in_step_ch * in_row_bytes + (unsigned int)in_step_tap * in_dil;
    const unsigned int in_next_ch = in_row_bytes - (unsigned int)in_taps * in_dil;
    // (the padding is taken off here, or off the lanes' positions)
    const unsigned char* const in_base = (const unsigned char*)p.B + ((long long)b * p.b_batch_stride - (INSIDE ? p.conv_pad : 0)) * 4;
    int in_tap = 0;
    unsigned int in_off = 0;
    auto rewind = [&]() __attribute__((always_inline)) {
        if constexpr (VIEW == VIEW_INPUT) {
            // (a step before the first one)
            const int ch = (8 * wave + (lane & 7)) / in_taps;
            in_tap = 8 * wave + (lane & 7) - ch * in_taps;
            in_off = (unsigned int)ch * in_row_bytes + (unsigned int)in_tap * in_dil - in_step_off;
            in_tap -= in_step_tap;
        }
        a_off = (size_t)k_rot * a_step;
        b_off = VIEW == VIEW_CONV ? (p.b_use_tap_table ? (size_t)p.b_tap_off[0] : 0) : (size_t)k_rot * b_step;
        next_step = k_rot;
        b_row_step = b_taps_done = 0;
    };
    const unsigned char *abase = Ag, *bbase = Bg;
    unsigned int voff_row = 0;
    auto load_begin = [&]() __attribute__((always_inline)) {      // fixes where the step starts and moves on
        if constexpr (!BT) voff_row = voff_b[0];
        abase = Ag + a_off;
        bbase = Bg + b_off;
        a_off += a_step;
        b_off += b_step;
        if constexpr (VIEW == VIEW_INPUT) {
            in_tap += in_step_tap;
            in_off += in_step_off;
            const bool over = in_tap >= in_taps;
            in_tap -= over ? in_taps : 0;
            in_off += over ? in_next_ch : 0u;
            // (rows past the last one, which clear_k_tail takes out: the first one instead)
            const bool there = next_step * BK + 8 * wave + (lane & 7) < p.K;
            in_tap = there ? in_tap : 0;
            in_off = there ? in_off : 0u;
            ++next_step;
        } else if constexpr (VIEW == VIEW_GEMM) {
            if (++next_step == KT) { next_step = 0; a_off = 0; b_off = 0; }
        } else {
            const bool new_tap = ++b_row_step == p.b_tiles_per_tap;
            b_row_step = new_tap ? 0 : b_row_step;
            b_taps_done += new_tap ? 1 : 0;
            // (the last advance comes after the final step: the index is kept inside the table)
            const long long from_table = tap_entry(b_taps_done < 32 ? b_taps_done : 31);
            const long long stepped = (long long)b_off + b_tap_jump;
            b_off = new_tap ? (size_t)(p.b_use_tap_table ? from_table : stepped) : b_off;
        }
    };
    auto four = [](auto rs, unsigned int off, float* x) __attribute__((always_inline)) {
        const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(rs, off, 0, 0);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const unsigned int w = v[e];
            x[e] = __builtin_bit_cast(float, w);
        }
    };
    // this thread's part of row t of A
    auto load_a = [&](int t) __attribute__((always_inline)) {
        auto rs = __builtin_amdgcn_make_buffer_rsrc((void*)abase, 0, records(abase, A_end), 0x00020000);
        unsigned int at = voff_a[VIEW == VIEW_INPUT ? 0 : t];
        if (VIEW == VIEW_INPUT && t == 1) {
            // (a register of its own would be one too many for three waves per SIMD)
            asm volatile("" : "+v"(at));
            at += (unsigned int)p.K * 4u;
        }
        if constexpr (A_KV == 2) {
            const u32x2 v = __builtin_amdgcn_raw_buffer_load_b64(rs, at, 0, 0);
            const unsigned int w0 = v[0], w1 = v[1];
            ra[t][0] = __builtin_bit_cast(float, w0);
            ra[t][1] = __builtin_bit_cast(float, w1);
        } else {
            four(rs, at, ra[t]);
            if constexpr (A_KV == 8) four(rs, at + 16, ra[t] + 4);
        }
    };
    // part q (of 4 B_CH) of B: of a transposed B half a chunk every other time, of a plain B the
    // k rows that part q completes when the parts are split in order (see `split`)
    auto load_b = [&](auto q_tag) __attribute__((always_inline)) {
        constexpr int q = decltype(q_tag)::value;
        if constexpr (VIEW == VIEW_INPUT) {
            if constexpr (q % 2 == 0) return;
#pragma unroll
            for (int e = q - 1; e <= q; ++e) {
                const unsigned int off = (unsigned int)__builtin_amdgcn_readlane((int)in_off, e);
                if constexpr (INSIDE) {
                    auto all = __builtin_amdgcn_make_buffer_rsrc((void*)in_base, 0, (int)0xffffffffu, 0x00020000);
                    const u32x2 v = __builtin_amdgcn_raw_buffer_load_b64(all, voff_b[0], off, 0);
                    const unsigned int w0 = v[0], w1 = v[1];
                    rb[0][e] = __builtin_bit_cast(float, w0);
                    rb[1][e] = __builtin_bit_cast(float, w1);
                } else {
                    // a resource per row, outside of which all is zero
                    const unsigned int tap = (unsigned int)__builtin_amdgcn_readlane(in_tap, e) * in_dil;
                    auto row = __builtin_amdgcn_make_buffer_rsrc((void*)(in_base + (off - tap)), 0, (int)in_row_bytes, 0x00020000);
#pragma unroll
                    for (int t = 0; t < B_CH; ++t) {
                        const unsigned int w = __builtin_amdgcn_raw_buffer_load_b32(row, voff_b[t] + tap, 0, 0);
                        rb[t][e] = __builtin_bit_cast(float, w);
                    }
                }
            }
            return;
        }
        auto rs = __builtin_amdgcn_make_buffer_rsrc((void*)bbase, 0, VIEW == VIEW_CONV ? (int)0xffffffffu : records(bbase, B_end), 0x00020000);
        if constexpr (BT) {
            if constexpr (q % 2 == 1) four(rs, voff_b[q / 4] + 16u * (q / 2 % 2), rb[q / 4] + 4 * (q / 2 % 2));
        } else if constexpr (q % 2 == 1) {
#pragma unroll
            for (int e = q - 1; e <= q; ++e) {
                const u32x2 v = __builtin_amdgcn_raw_buffer_load_b64(rs, voff_row, 0, 0);
                // (a running offset: eight of them kept in registers are eight too many)
                voff_row += b_row_bytes;
                asm volatile("" : "+v"(voff_row));
                const unsigned int w0 = v[0], w1 = v[1];
                rb[0][e] = __builtin_bit_cast(float, w0);
                rb[1][e] = __builtin_bit_cast(float, w1);
            }
        }
    };
    auto load_step = [&]() __attribute__((always_inline)) {
        load_begin();
#pragma unroll
        for (int t = 0; t < A_CH; ++t) load_a(t);
        static_for<0, 4 * B_CH>(load_b);
    };
    // k values of a partial last step that do not exist: whatever was read in their place (the start
    // of the next row; a NaN there must not reach this one) counts as zero
    auto clear_k_tail = [&]() __attribute__((always_inline)) {
        const int ka = k_last - a_k0, kb = k_last - 8 * (BT ? my_chunk : wave);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
#pragma unroll
            for (int t = 0; t < A_CH; ++t) { if (e < A_KV) ra[t][e] = e < ka ? ra[t][e] : 0.0f; }
#pragma unroll
            for (int t = 0; t < B_CH; ++t) rb[t][e] = e < kb ? rb[t][e] : 0.0f;
        }
    };
    // columns past the edge that are loaded all the same -- the neighbour of an odd row's last column, in a
    // convolution every position past the row's end -- hold other rows' values: zero, so that these do not
    // decide how this tile is computed
    const bool edge_cols = !BT && VIEW != VIEW_INPUT && (VIEW == VIEW_CONV ? n_rem < BN : n_rem % 2 != 0);
    auto clear_edge_cols = [&]() __attribute__((always_inline)) {
        const int left = n_rem - 2 * lane;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            rb[0][e] = left > 0 ? rb[0][e] : 0.0f;
            rb[1][e] = left > 1 ? rb[1][e] : 0.0f;
        }
    };
    auto meet = [&]() __attribute__((always_inline)) {
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
    };

    // ---- the step in registers, split.  Part n is a pair of k values: of A's chunks one after the other,
    // then of B's (of column pairs both columns at one k); OPS operations of two or three
    // instructions each take it apart.
    unsigned int lost = 0u;                       // what the values leave after two terms, or-ed together
    // the packed terms (of whole chunks as vectors: as single registers the loop had four waits more)
    typename std::conditional<A_KV == 8, u32x4, unsigned int[A_KV / 2]>::type pa[A_CH][3];
    u32x4 pb[B_CH][3];
    constexpr int A_PAIRS = A_KV / 2, A_PARTS = A_CH * A_PAIRS, PARTS = A_PARTS + 4 * B_CH, OPS = 5;
    auto bits = [](float x) __attribute__((always_inline)) { return __builtin_bit_cast(unsigned int, x); };
    auto value = [](unsigned int u) __attribute__((always_inline)) { return __builtin_bit_cast(float, u); };
    float t0 = 0.0f, t1 = 0.0f;
    auto split = [&](auto n_tag, auto op_tag) __attribute__((always_inline)) {
        constexpr int n = decltype(n_tag)::value, op = decltype(op_tag)::value, nb = n - A_PARTS;
        constexpr bool of_a = nb < 0;
        constexpr int t = of_a ? n / A_PAIRS : BT ? nb / 4 : nb % 2, q = of_a ? n % A_PAIRS : BT ? nb % 4 : nb / 2;
        float* x;
        if constexpr (of_a) x = &ra[t][2 * q]; else x = &rb[t][2 * q];
        auto put = [&](int plane, unsigned int w) __attribute__((always_inline)) {
            if constexpr (of_a) pa[t][plane][q] = w; else pb[t][plane][q] = w;
        };
        if constexpr (op == 0) {
            // odd rows and columns enter with their sign turned (see "Rounding"; left to the compiler, the
            // conversion's operands are turned by instructions of their own)
            unsigned int h;
            if constexpr (t == 1) {
                asm("v_cvt_pk_bf16_f32 %0, -%1, -%2" : "=v"(h) : "v"(x[0]), "v"(x[1]));
                x[0] = -x[0];
                x[1] = -x[1];
            } else {
                h = pack_bf16x2(x[0], x[1]);
            }
            put(0, h);
            t0 = value(h << 16);
            t1 = value(h & 0xffff0000u);
        } else if constexpr (op == 1) {
            x[0] -= t0;
            x[1] -= t1;
        } else if constexpr (op == 2) {
            const unsigned int m = pack_bf16x2(x[0], x[1]);
            put(1, m);
            t0 = value(m << 16);
            t1 = value(m & 0xffff0000u);
        } else if constexpr (op == 3) {
            x[0] -= t0;
            x[1] -= t1;
        } else {
            put(2, __builtin_amdgcn_perm(bits(x[1]), bits(x[0]), 0x07060302u));       // the upper halves: all there is
            lost |= bits(x[0]) | bits(x[1]);
            asm volatile("" : "+v"(lost));        // (here and now: put off to the end of the step, all remainders stay live)
        }
    };
    auto write_step = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int q = 0; q < 3; ++q) {
#pragma unroll
            for (int t = 0; t < A_CH; ++t) {
                unsigned char* const to = lds_a + q * Cfg::A_PLANE + wpos_a + kOddRow * t;
                if constexpr (A_KV == 8) *(__attribute__((address_space(3))) u32x4*)PGK_LDS(to) = pa[t][q];
                else if constexpr (A_KV == 4) *(__attribute__((address_space(3))) u32x2*)PGK_LDS(to) = u32x2{pa[t][q][0], pa[t][q][1]};
                else *(__attribute__((address_space(3))) unsigned int*)PGK_LDS(to) = pa[t][q][0];
            }
#pragma unroll
            for (int t = 0; t < B_CH; ++t) *(__attribute__((address_space(3))) u32x4*)PGK_LDS(lds_b + q * Cfg::B_PLANE + wpos_b + kOddRow * t) = pb[t][q];
        }
    };

    const int l16 = lane & 15, grp = lane >> 4;
    // this lane's 16 bytes of a fragment
    const int rpos = frag_pos(l16, grp);
    const unsigned char* const as = lds_a + wm * TM16 * 1024 + rpos;
    const unsigned char* const bs = lds_b + wn * TN16 * 1024 + rpos;

    f32x4 acc[TM16][TN16];
    auto clear_acc = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < TM16; ++i)
#pragma unroll
            for (int j = 0; j < TN16; ++j) acc[i][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    };
    clear_acc();

    // ---- one step, in LDS; the step in registers (`next`) is split, the one after it (`ahead`) loaded.
    // The instruction order is written out and pinned, slot by slot: one matrix instruction, then
    // the operand fetches, the splitting and the loads that belong to the slot.
    constexpr int PER_J = 6 * TM16, SLOTS = PER_J * TN16;
    auto step = [&](auto next_tag, auto ahead_tag) __attribute__((always_inline)) {
        constexpr bool NEXT = decltype(next_tag)::value != 0, AHEAD = decltype(ahead_tag)::value != 0;
        // two column blocks' fragments in turn; with fewer rows and three waves per SIMD only of term 0, the others into the same
        // place once it is free (two places each take seven registers more than there are)
        constexpr bool TWO = BM == 128;
        bf16x8 fa[3][TM16], fb[TWO ? 6 : 4];
        f32x4 sum[TM16];            // of this step's products of one column block (see "Rounding")
        if constexpr (NEXT && !BT) { if (edge_cols) clear_edge_cols(); }
        auto fetch_a = [&](int q, int i) __attribute__((always_inline)) { fa[q][i] = *(const __attribute__((address_space(3))) bf16x8*)PGK_LDS(as + q * Cfg::A_PLANE + i * 1024); };
        auto slot_b = [](int j, int q) constexpr { return TWO ? 3 * (j & 1) + q : q == 0 ? 2 + (j & 1) : q - 1; };
        auto fetch_b = [&](int j, int q) __attribute__((always_inline)) { fb[slot_b(j, q)] = *(const __attribute__((address_space(3))) bf16x8*)PGK_LDS(bs + q * Cfg::B_PLANE + j * 1024); };
        // (term of A, term of B) of the six products, the small ones first
        constexpr int QA[6] = {0, 2, 1, 0, 1, 0}, QB[6] = {2, 0, 1, 1, 0, 0};
        // the fragments of the first column block, in the order they are needed
#pragma unroll
        for (int u = 0; u < 3; ++u) {
            fetch_b(0, QB[u]);
#pragma unroll
            for (int i = 0; i < TM16; ++i) fetch_a(QA[u], i);
        }
        if constexpr (AHEAD) load_begin();
        // (a wave that multiplies goes before one that writes or starts: 694 -> 680 us on 4096^3)
        __builtin_amdgcn_s_setprio(2);
        __builtin_amdgcn_sched_barrier(0);
        // the operations of the parts, in order, spread over the slots FIRST to LAST - 1
        constexpr int TOTAL = OPS * PARTS, FIRST = SLOTS / 12, LAST = SLOTS - SLOTS / 24;
        auto ops_before = [](int m) constexpr { return m <= FIRST ? 0 : m >= LAST ? TOTAL : (m - FIRST) * TOTAL / (LAST - FIRST); };
        static_for<0, SLOTS>([&](auto m_tag) __attribute__((always_inline)) {
            constexpr int m = decltype(m_tag)::value;
            constexpr int j = m / PER_J, u = (m / TM16) % 6, i = m % TM16;
            // the small products' sum is complete before the large ones, theirs a column block later
            if constexpr (u == 5) acc[i][j] += sum[i];
            if constexpr (u == 0 && j > 0) acc[i][j - 1] += sum[i];
            sum[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[slot_b(j, QB[u])], fa[QA[u]][i],
                                                             u == 0 || u == 5 ? f32x4{0.0f, 0.0f, 0.0f, 0.0f} : sum[i], 0, 0, 0);
            // the next column block's fragments (term 2 is free behind the first product, term 1 behind the fourth)
            if constexpr (j + 1 < TN16) {
                constexpr int at = m % PER_J - TM16;
                if constexpr (TWO) { if constexpr (at >= 0 && at < 3) fetch_b(j + 1, QB[at]); }
                else if constexpr (at == 0) fetch_b(j + 1, 2);
                else if constexpr (at == 1) fetch_b(j + 1, 0);
                else if constexpr (at == 3 * TM16) fetch_b(j + 1, 1);
            }
            if constexpr (NEXT) {
                static_for<ops_before(m), ops_before(m + 1)>([&](auto o_tag) __attribute__((always_inline)) {
                    constexpr int o = decltype(o_tag)::value, part = o / OPS;
                    split(IC<part>{}, IC<o % OPS>{});
                    // a part's registers are free once it is split: what is to fill them next
                    if constexpr (AHEAD && o % OPS == OPS - 1) {
                        if constexpr (part < A_PARTS) { if constexpr (part % A_PAIRS == A_PAIRS - 1) load_a(part / A_PAIRS); }
                        else load_b(IC<part - A_PARTS>{});
                    }
                });
            }
            __builtin_amdgcn_sched_barrier(0);
        });
#pragma unroll
        for (int i = 0; i < TM16; ++i) acc[i][TN16 - 1] += sum[i];
    };
    auto to_next = [&]() __attribute__((always_inline)) {
        __builtin_amdgcn_s_setprio(0);
        meet();            // every wave has fetched its operands
        write_step();
        meet();            // the next step is in LDS
    };

    // prologue: step 0 in LDS, step 1 in registers
    rewind();
    load_step();
    if (KT == 1 && k_last < BK) clear_k_tail();
    if constexpr (!BT) { if (edge_cols) clear_edge_cols(); }
    static_for<0, OPS * PARTS>([&](auto o) __attribute__((always_inline)) { split(IC<decltype(o)::value / OPS>{}, IC<decltype(o)::value % OPS>{}); });
    write_step();
    float* const bias_lds = rs_buf + Cfg::WGN * BM;
    float* const bias_lds_row = bias_lds + BIAS_N;
    auto write_biases = [&]() __attribute__((always_inline)) {
        if (tid < BIAS_N) {
            bias_lds[tid] = BIAS_PER_ROW ? 0.0f : bias_pre;
            if constexpr (BIAS_PER_ROW) bias_lds_row[tid] = bias_pre;
        }
    };
    // (now, with three waves per SIMD: a register held through the loop is one too many)
    if constexpr (BM < 128) write_biases();
    if (KT > 1) load_step();
    meet();
    stamp(1);
    for (int kt = 0; kt + 2 < KT; ++kt) {
        step(IC<1>{}, IC<1>{});
        to_next();
    }
    if (KT > 1) {
        if (k_last < BK) clear_k_tail();
        step(IC<1>{}, IC<0>{});
        to_next();
    }
    step(IC<0>{}, IC<0>{});
    __builtin_amdgcn_s_setprio(0);

    // ---- did the terms hold everything?  (see "Range")
    {
        float zero = 0.0f;            // 0 x anything finite; NaN otherwise
        int smallest = 0;
#pragma unroll
        for (int i = 0; i < TM16; ++i)
#pragma unroll
            for (int j = 0; j < TN16; ++j)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    zero = __builtin_fmaf(acc[i][j][e], 0.0f, zero);
                    const int exponent = __builtin_amdgcn_frexp_expf(acc[i][j][e]);       // (0 for zero)
                    smallest = exponent < smallest ? exponent : smallest;
                }
        const int bad = (lost & 0xffffu) != 0u || zero != 0.0f || smallest < -118;
        if (__syncthreads_or(bad)) {
            // the same tile with the fp32 matrix instruction.  LDS: sixteen rows x four k values of
            // fp32 are 256 bytes, row r of k chunk c at 256 c + 16 r (BM x 32 floats fit the three planes).
            clear_acc();
            rewind();
            for (int kt = 0; kt < KT; ++kt) {
                load_step();
                if (kt + 1 == KT && k_last < BK) clear_k_tail();
                meet();
                auto put = [](unsigned char* base, int row, int c, const float* x) __attribute__((always_inline)) {
                    *(f32x4*)(base + (row >> 4) * 2048 + c * 256 + (row & 15) * 16) = f32x4{x[0], x[1], x[2], x[3]};
                };
#pragma unroll
                for (int t = 0; t < A_CH; ++t) {
                    if constexpr (A_KV >= 4) {
#pragma unroll
                        for (int h = 0; h < A_KV / 4; ++h) put(lds_a, a_row + t, a_k0 / 4 + h, &ra[t][4 * h]);
                    } else {
                        const int row = a_row + t;
                        *(float2*)(lds_a + (row >> 4) * 2048 + (a_k0 >> 2) * 256 + (row & 15) * 16 + (a_k0 & 3) * 4) = float2{ra[t][0], ra[t][1]};
                    }
                }
#pragma unroll
                for (int h = 0; h < 2; ++h) {
#pragma unroll
                    for (int t = 0; t < B_CH; ++t) {
                        if constexpr (BT) put(lds_b, my_row + t, 2 * my_chunk + h, &rb[t][4 * h]);
                        else put(lds_b, 2 * lane + t, 2 * wave + h, &rb[t][4 * h]);
                    }
                }
                meet();
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    f32x4 xa[TM16], xb[TN16];
                    const int at = (4 * h + grp) * 256 + l16 * 16;
#pragma unroll
                    for (int i = 0; i < TM16; ++i) xa[i] = *(const f32x4*)(lds_a + (wm * TM16 + i) * 2048 + at);
#pragma unroll
                    for (int j = 0; j < TN16; ++j) xb[j] = *(const f32x4*)(lds_b + (wn * TN16 + j) * 2048 + at);
#pragma unroll
                    for (int e = 0; e < 4; ++e)
#pragma unroll
                        for (int i = 0; i < TM16; ++i)
#pragma unroll
                            for (int j = 0; j < TN16; ++j)
                                acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(xb[j][e], xa[i][e], acc[i][j], 0, 0, 0);
                }
            }
            meet();
            // as the epilogue expects them
#pragma unroll
            for (int i = 0; i < TM16; ++i)
#pragma unroll
                for (int j = 0; j < TN16; ++j)
#pragma unroll
                    for (int e = 0; e < 4; ++e) acc[i][j][e] = ((l16 ^ e) & 1) ? -acc[i][j][e] : acc[i][j][e];
        }
    }
    stamp(2);          // end of the main loop (every wave is past its operand reads)

    // ---- epilogue
    unsigned char* const piece = (wave < 2 ? lds_a : lds_b) + (wave & 1) * Cfg::PIECE_BYTES;
    if (out_mode == 1) {
        // split-K pass 1: the partial products of this slice
        unsigned char* w = (unsigned char*)(p.ws + ((size_t)b * p.splits + sp) * (size_t)p.M * (size_t)p.N +
                                            (size_t)tm * BM * (size_t)p.N + (size_t)tn * BN);
        epilogue_terms<ACT_NONE, EPI_PLAIN, Cfg, false, false>(acc, nullptr, nullptr, w, (size_t)p.N * 4, m_rem, n_rem, wm, wn, lane, piece, nullptr);
        return;
    }
    float* const rs_lds = p.rs_part ? rs_buf : nullptr;
    if constexpr (BM == 128) write_biases();
    __syncthreads();
    stamp(3);
    unsigned char* c_tile = (unsigned char*)p.C + ((size_t)b * p.M * p.N + (size_t)tm * BM * (size_t)p.N + (size_t)tn * BN) * 4;
    auto run_epilogue = [&](auto kind) __attribute__((always_inline)) {
        constexpr int KIND = decltype(kind)::value;
        const float* br = KIND == EPI_ROWBIAS ? bias_lds_row : nullptr;
        switch (p.act) {
        case ACT_RELU: epilogue_terms<ACT_RELU, KIND, Cfg, true, true>(acc, bias_lds, br, c_tile, (size_t)p.N * 4, m_rem, n_rem, wm, wn, lane, piece, rs_lds); break;
        case ACT_GELU_TANH: epilogue_terms<ACT_GELU_TANH, KIND, Cfg, true, true>(acc, bias_lds, br, c_tile, (size_t)p.N * 4, m_rem, n_rem, wm, wn, lane, piece, rs_lds); break;
        case ACT_SILU: epilogue_terms<ACT_SILU, KIND, Cfg, true, true>(acc, bias_lds, br, c_tile, (size_t)p.N * 4, m_rem, n_rem, wm, wn, lane, piece, rs_lds); break;
        default: epilogue_terms<ACT_NONE, KIND, Cfg, true, true>(acc, bias_lds, br, c_tile, (size_t)p.N * 4, m_rem, n_rem, wm, wn, lane, piece, rs_lds); break;
        }
    };
    if constexpr (BIAS_PER_ROW) {
        if (p.bias) run_epilogue(IC<EPI_ROWBIAS>{});
        else run_epilogue(IC<EPI_PLAIN>{});
    } else {
        if (!rs_lds) run_epilogue(IC<EPI_PLAIN>{});
        else if (n_rem == BN) run_epilogue(IC<EPI_ROWSUM>{});
        else run_epilogue(IC<EPI_ROWSUM_MASKED>{});
    }
    if (p.rs_part) {
        __syncthreads();
        if (tid < m_rem) {
            // the wave columns' partial row sums, in order
            float sum = rs_buf[tid];
#pragma unroll
            for (int w = 1; w < Cfg::WGN; ++w) sum += rs_buf[w * BM + tid];
            p.rs_part[((size_t)b * p.tiles_n + tn) * (size_t)p.M + (size_t)tm * BM + tid] = sum;
        }
    }
    stamp(4);
    if constexpr (TIMED) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        stamp(5);
    }
