// Expert FFN kernels on 4-row weight tiles (v_mfma_f32_4x4x4_16b_bf16 and
// v_mfma_f32_4x4x1_16b_f32).  Included by expert_ffn.hip.
//
// What bounds them is the stream of weight bytes, so the layout follows the
// loads: one 16-byte load per lane reads four rows x 256 contiguous bytes
// (lane = 4 * chunk + row), and that is the operand layout of the
// 16-block 4x4 MFMA as it stands: block c multiplies the 4 rows' chunk c
// with chunk c of four tokens, and the 16 blocks' partial products add up
// once, after the last step.  No LDS transpose, no unpacking, no barrier
// while the weights stream, and a step costs a slot's own tokens (one
// operand load per four of them), not a padded batch.
//
// Every step's products start from zero and are added to the running sums
// afterwards: a sum is a chain of (steps) + (elements of a chunk) additions
// per lane and a tree over 16 blocks, as short as a 64-lane dot product's.
// The rows of a 4x4 result depend on one token each, so operand lanes without
// a token may hold any token's values; only routed rows are added.

template <bool BF>
__device__ __forceinline__ f32x4 mma44(const uint4& x, const uint4& w, f32x4 d) {
    typedef short s16x4 __attribute__((ext_vector_type(4)));
    typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
    if constexpr (BF) {
        d = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(__builtin_bit_cast(s16x4, u32x2{x.x, x.y}),
                                                   __builtin_bit_cast(s16x4, u32x2{w.x, w.y}), d, 0, 0, 0);
        d = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(__builtin_bit_cast(s16x4, u32x2{x.z, x.w}),
                                                   __builtin_bit_cast(s16x4, u32x2{w.z, w.w}), d, 0, 0, 0);
    } else {
        d = __builtin_amdgcn_mfma_f32_4x4x1f32(__uint_as_float(x.x), __uint_as_float(w.x), d, 0, 0, 0);
        d = __builtin_amdgcn_mfma_f32_4x4x1f32(__uint_as_float(x.y), __uint_as_float(w.y), d, 0, 0, 0);
        d = __builtin_amdgcn_mfma_f32_4x4x1f32(__uint_as_float(x.z), __uint_as_float(w.z), d, 0, 0, 0);
        d = __builtin_amdgcn_mfma_f32_4x4x1f32(__uint_as_float(x.w), __uint_as_float(w.w), d, 0, 0, 0);
    }
    return d;
}

// The 16 blocks' sums of one 4x4 tile: lane l gets the total of token
// (l >> 2) & 3 and weight row l & 3 (the same in all four 16-lane rows).
__device__ __forceinline__ float tile_total(const f32x4& d) {
    const int i = (threadIdx.x >> 2) & 3;
    float v[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        float t = d[r];
        t += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(t), 0x124, 0xf, 0xf, false));  // row_ror:4
        t += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(t), 0x128, 0xf, 0xf, false));  // row_ror:8
        v[r] = t;
    }
    float s = i == 0 ? v[0] : i == 1 ? v[1] : i == 2 ? v[2] : v[3];
    s += __shfl_xor(s, 16, 64);
    s += __shfl_xor(s, 32, 64);
    return s;
}

__device__ __forceinline__ int uni(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ const char* uni(const char* p) {
    const uint64_t u = reinterpret_cast<uint64_t>(p);
    const uint32_t lo = uint32_t(uni(int(uint32_t(u)))), hi = uint32_t(uni(int(uint32_t(u >> 32))));
    return reinterpret_cast<const char*>((uint64_t(hi) << 32) | lo);
}

// One slot of the plan: its blob, its tokens (bit mask, and listed in
// ascending order) and their gate weights.  nt = 0: no such slot.
struct SlotRec {
    const char* blob;
    uint32_t tok;
    int32_t nt;
    uint8_t token[kMaxB];
    float w[kMaxB];
};

// The slot plan in global memory, `cap` records: selected routed experts
// ascending, then shared experts.  Built by the router's tail launch (decode
// path) or by a workgroup of the gate/up launch for the down launch.
struct SlotList {
    int32_t n_routed, n_slots, pad[2];
    SlotRec rec[kMaxSlots];
};

__device__ void publish_b1_slot(const FfnArgs& a, int j, const char* blob) {
    a.slots->rec[j].blob = blob;
    a.slots->rec[j].tok = 1u;
}
__device__ void publish_b1_counts(const FfnArgs& a, int n_routed) {
    a.slots->n_routed = n_routed;
    a.slots->n_slots = n_routed + a.n_shared;
}

// One workgroup of T threads: build the plan of a selection in LDS (idx, w
// [B][K]; entries outside [0, E) are ignored, a repeated expert counts once,
// with its first entry's weight).
template <int T>
__device__ void publish_plan(const FfnArgs& a, const int32_t* idx, const float* w) {
    __shared__ uint32_t words[8], tok[kMaxSlots];
    const int tid = threadIdx.x, BK = a.B * a.K;
    if (tid < 8) words[tid] = 0u;
    for (int i = tid; i < a.cap; i += T) tok[i] = 0u;
    __syncthreads();
    for (int t = tid; t < BK; t += T) {
        const int e = idx[t];
        if (e >= 0 && e < a.E) atomicOr(&words[e >> 5], 1u << (e & 31));
    }
    __syncthreads();
    int total = 0;
#pragma unroll
    for (int q = 0; q < 8; ++q) total += __popc(words[q]);
    auto rank_of = [&](int e) {
        int r = __popc(words[e >> 5] & ((1u << (e & 31)) - 1u));
        for (int q = 0; q < (e >> 5); ++q) r += __popc(words[q]);
        return r;
    };
    for (int t = tid; t < BK; t += T) {
        const int e = idx[t];
        if (e >= 0 && e < a.E) atomicOr(&tok[rank_of(e)], 1u << (t / a.K));
    }
    __syncthreads();
    SlotRec* rec = a.slots->rec;
    for (int t = tid; t < BK; t += T) {
        const int e = idx[t], b = t / a.K;
        bool first = e >= 0 && e < a.E;
        for (int k = b * a.K; k < t; ++k) first = first && idx[k] != e;
        if (!first) continue;
        const int r = rank_of(e), at = __popc(tok[r] & ((1u << b) - 1u));
        rec[r].token[at] = uint8_t(b);
        rec[r].w[at] = w[t];
        if (at == 0) {
            rec[r].blob = routed_blob(a, e);
            rec[r].tok = tok[r];
            rec[r].nt = __popc(tok[r]);
        }
    }
    for (int r = total + tid; r < a.cap; r += T) {
        const bool shared = r < total + a.n_shared;
        if (shared) {
            rec[r].blob = reinterpret_cast<const char*>(a.sptr[r - total]);
            rec[r].tok = (1u << a.B) - 1u;
            for (int b = 0; b < a.B; ++b) {
                rec[r].token[b] = uint8_t(b);
                rec[r].w[b] = 1.f;
            }
        }
        rec[r].nt = shared ? a.B : 0;
    }
    if (tid == 0) {
        a.slots->n_routed = total;
        a.slots->n_slots = total + a.n_shared;
    }
}

// The slots as the down kernels read them, copied to LDS (records past
// n_slots are not used).  Ends with a barrier.
struct SlotTable {
    const char* blob[kMaxSlots];
    uint32_t tok[kMaxSlots];
    int n_routed, n_slots;
};

__device__ __forceinline__ void load_slots(const FfnArgs& a, SlotTable& p) {
    for (int s = threadIdx.x; s < a.cap; s += int(blockDim.x)) {
        p.blob[s] = a.slots->rec[s].blob;
        p.tok[s] = a.slots->rec[s].tok;
    }
    if (threadIdx.x == 0) {
        p.n_routed = a.slots->n_routed;
        p.n_slots = a.slots->n_slots;
    }
    __syncthreads();
}

// The router's tail and the plan in one workgroup, a wave per batch row.
__global__ __launch_bounds__(1024) void route_plan_kernel(gating::RouteArgs r, FfnArgs a) {
    __shared__ int32_t sel[kMaxB * kMaxK];
    __shared__ float w[kMaxB * kMaxK];
    const int lane = threadIdx.x & 63, b = threadIdx.x >> 6;
    if (b < r.B) {
        int e;
        float wt;
        gating::route_row(r.zbuf + size_t(b) * r.E, r.E, r.K, r.renorm, sel + b * r.K, w + b * r.K, e, wt);
        if (lane < r.K) {
            r.idx[b * r.K + lane] = e;
            r.w[b * r.K + lane] = wt;
        }
    }
    __syncthreads();
    publish_plan<1024>(a, sel, w);
}

// The selection of a wave: entry t = 64 * i + lane of [B][K] (-1: none).
struct Sel {
    int v[4];
    float w[4];
};

// Entries the plan ignores (outside [0, E)) become -1.
__device__ __forceinline__ Sel load_sel(const FfnArgs& a, const int32_t* idx, const float* w) {
    const int lane = threadIdx.x & 63, BK = a.B * a.K;
    Sel s;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int t = 64 * i + lane;
        const int e = t < BK ? idx[t] : -1;
        s.v[i] = e >= 0 && e < a.E ? e : -1;
        s.w[i] = t < BK ? w[t] : 0.f;
    }
    return s;
}

// The distinct selected experts as a bit mask, by one wave through 8 words of
// LDS of its own (a wave's LDS accesses complete in order: no barrier).
__device__ __forceinline__ void selected_mask(const Sel& s, uint32_t* words, uint32_t (&m)[8]) {
    const int lane = threadIdx.x & 63;
    if (lane < 8) words[lane] = 0u;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int i = 0; i < 4; ++i)
        if (s.v[i] >= 0) atomicOr(&words[s.v[i] >> 5], 1u << (s.v[i] & 31));
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int q = 0; q < 8; ++q) m[q] = uint32_t(uni(int(words[q])));
}

// A weight chunk.  Weights are read once, past the caches.  Not so (SHARED)
// behind a capped cache, whose overflow experts stay in host memory, for rows
// that are not whole 128-byte lines: their 256-byte segments share lines with
// the next step's, and read past the caches those lines come over the host link
// twice (a token of 3 layers E 10 top-4 H 1816 I 1384 fp32, batch 2: 4326 us,
// 3960 through the caches).  In HBM such rows gain 2 to 15% a token that way, but
// a pass over caches full of written lines lost 45% (FFN E 60 top-4 + 1 H 2056
// I 1000, batch 6: 64 us and 100), and whole lines lose always (Qwen3-30B shapes
// at batch 8, 4 layers: 352 and 390).
template <bool SHARED>
__device__ __forceinline__ uint4 ld_weight(const char* p) {
    if constexpr (SHARED) return ld_cached(p);
    else return ld_stream(p);
}

// One wave's rows of a slot: what the stream below needs.
struct UpTile {
    const char* x;                   // [B][H]
    const char* wg;                  // the first row in W_gate; W_up's lies `up` bytes on
    size_t up, rowb;
    int nt;                          // tokens of the slot
    int rot;                         // first step (the steps run around)
    size_t act;                      // element of token 0's activation of the first row
};

// Stream the tile's weights for up to 4 * TG tokens, U steps of 256 bytes per
// row in flight, and store the activations.  The loop has no branch around a
// load: behind one, every wait would be for all loads in flight.  So lanes
// without a token load the first token's row, and the columns' remainder is a
// step of its own ahead of the loop.  The full steps start at `rot` and run
// around, so that waves that start together do not all read the same column
// of rows a power of two apart (the same memory channels).
template <bool BF, int TG, int TGX, int U, bool SK, bool SHARED>
__device__ __forceinline__ void up_stream(const FfnArgs& a, const UpTile& z, const int (&mytok)[TGX],
                                          const float (&myw)[TGX], float (&red)[SK ? kWaves : 1][2][TGX][16]) {
    const int lane = threadIdx.x & 63, wave = uni(threadIdx.x >> 6), c = lane >> 2, nt = z.nt;
    const uint32_t woff = uint32_t(lane & 3) * uint32_t(z.rowb) + uint32_t(c) * 16u;
    uint32_t xoff[TG];
#pragma unroll
    for (int tg = 0; tg < TG; ++tg) xoff[tg] = uint32_t(mytok[tg]) * uint32_t(z.rowb) + uint32_t(c) * 16u;
    const char* wu = z.wg + z.up;
    const int full = int(z.rowb >> 8), rem = int(z.rowb & 255) >> 4;
    const int s0 = SK ? full * wave / kWaves : 0;
    const int n = SK ? full * (wave + 1) / kWaves - s0 : full;
    int at = n > 0 ? s0 + z.rot % n : 0;         // next step to load

    struct Step { uint4 g, u, x[TG]; };
    auto load = [&](Step& st) {
        const size_t o = size_t(at) << 8;
        at = at + 1 == s0 + n ? s0 : at + 1;
#pragma unroll
        for (int tg = 0; tg < TG; ++tg) st.x[tg] = ld_cached(z.x + o + xoff[tg]);
        st.g = ld_weight<SHARED>(z.wg + o + woff);
        st.u = ld_weight<SHARED>(wu + o + woff);
    };
    const f32x4 fz = f32x4{0.f, 0.f, 0.f, 0.f};
    f32x4 accg[TG], accu[TG];
#pragma unroll
    for (int tg = 0; tg < TG; ++tg) accg[tg] = accu[tg] = fz;
    auto compute = [&](const Step& st) {
#pragma unroll
        for (int tg = 0; tg < TG; ++tg) {
            accg[tg] += mma44<BF>(st.x[tg], st.g, fz);
            accu[tg] += mma44<BF>(st.x[tg], st.u, fz);
        }
    };
    Step st[U];
    if (rem != 0 && (!SK || wave == 0)) {
        const size_t o = size_t(full) << 8;
        const uint4 zero = make_uint4(0u, 0u, 0u, 0u);
        const bool in = c < rem;
#pragma unroll
        for (int tg = 0; tg < TG; ++tg) st[0].x[tg] = in ? ld_cached(z.x + o + xoff[tg]) : zero;
        st[0].g = in ? ld_weight<SHARED>(z.wg + o + woff) : zero;
        st[0].u = in ? ld_weight<SHARED>(wu + o + woff) : zero;
        compute(st[0]);
    }
    if (n >= U) {
#pragma unroll
        for (int u = 0; u < U; ++u) load(st[u]);
        int t = U;
        for (; t + U <= n; t += U)
#pragma unroll
            for (int u = 0; u < U; ++u) {
                compute(st[u]);
                load(st[u]);
            }
#pragma unroll
        for (int u = 0; u < U; ++u) compute(st[u]);
        // fewer than U steps left
        const int left = n - t;
#pragma unroll
        for (int u = 0; u < U - 1; ++u)
            if (u < left) load(st[u]);
#pragma unroll
        for (int u = 0; u < U - 1; ++u)
            if (u < left) compute(st[u]);
    } else {
#pragma unroll
        for (int u = 0; u < U - 1; ++u)
            if (u < n) load(st[u]);
#pragma unroll
        for (int u = 0; u < U - 1; ++u)
            if (u < n) compute(st[u]);
    }

    // totals: lane (.., token (l >> 2) & 3, row l & 3); token ids and weights of
    // a lane's token sit in lane (l >> 2) & 3
    const int g = (lane >> 2) & 3;
    float gs[TG], us[TG];
#pragma unroll
    for (int tg = 0; tg < TG; ++tg) {
        gs[tg] = tile_total(accg[tg]);
        us[tg] = tile_total(accu[tg]);
    }
    if constexpr (SK) {
#pragma unroll
        for (int tg = 0; tg < TG; ++tg)
            if (lane < 16) {
                red[wave][0][tg][lane] = gs[tg];
                red[wave][1][tg][lane] = us[tg];
            }
        __syncthreads();
    }
#pragma unroll
    for (int tg = 0; tg < TG; ++tg) {
        if (SK && wave != tg) continue;          // wave w finishes token group w
        const int tk = __shfl(mytok[tg], g, 64);
        const float wt = __shfl(myw[tg], g, 64);
        if (lane >= 16 || 4 * tg + g >= nt) continue;
        float gv = gs[tg], uv = us[tg];
        if constexpr (SK) {
            gv = uv = 0.f;
#pragma unroll
            for (int w = 0; w < kWaves; ++w) {
                gv += red[w][0][tg][lane];
                uv += red[w][1][tg][lane];
            }
        }
        store_act(a.act, a.act16, z.act + size_t(tk) * a.I + (lane & 3), wt * silu(gv) * uv);
    }
}

constexpr int kUpTileSteps = 2;       // steps in flight per wave (gate/up)

// gate/up: one wave = four rows of W_gate and the same rows of W_up of one
// slot (SK: the workgroup's four waves share the rows and split the columns).
// Slots with more than four tokens take the stream for up to 4 * TG of them,
// with fewer steps in flight (their registers are what the others pay for).
// The plan comes from the router's tail where there is one: each round of
// workgroups pays this kernel's prologue, and one record read is the shortest.
// Otherwise every wave finds its slot from the selection, and workgroup 0 only
// publishes the plan (and the selection it routed).
template <bool BF, int TG, bool SK, bool SHARED>
__global__ __launch_bounds__(kThreads, TG == 4 ? 4 : TG == 2 ? 6 : 7) void ffn_up_tile(FfnArgs a, int bps) {
    __shared__ uint32_t words[kWaves][8];
    __shared__ int32_t s_idx[kMaxB * kMaxK];
    __shared__ float s_w[kMaxB * kMaxK];
    __shared__ float red[SK ? kWaves : 1][2][TG][16];
    const int lane = threadIdx.x & 63, wave = uni(threadIdx.x >> 6);
    const int kinv = 65536 / a.K + 1;     // t / K = t * kinv >> 16 for t < 256
    // without a plan made beforehand, workgroup 0 publishes it (for the down launch)
    const bool pub = !a.ready && blockIdx.x == 0;
    const int blk = int(blockIdx.x) - (a.ready ? 0 : 1);
    const int j = blk / bps;
    const int i0 = SK ? (blk - j * bps) * 4 : ((blk - j * bps) * kWaves + wave) * 4;
    // the slot's blob and tokens: lane l holds token number 4 tg + (l & 3) of them
    const char* blob;
    int nt = 0, mytok[TG];
    float myw[TG];
#pragma unroll
    for (int tg = 0; tg < TG; ++tg) { mytok[tg] = 0; myw[tg] = 0.f; }
    if (a.ready) {
        const SlotRec& r = a.slots->rec[j];
        nt = r.nt;
        blob = r.blob;
#pragma unroll
        for (int tg = 0; tg < TG; ++tg) {
            mytok[tg] = r.token[4 * tg + (lane & 3)];
            myw[tg] = r.w[4 * tg + (lane & 3)];
        }
        if (nt == 0) return;
    } else {
        Sel sel;
        if (a.logits) {
            for (int b = wave; b < a.B; b += kWaves) {
                int ek;
                float wt;
                gating::route_row(a.logits + size_t(b) * a.E, a.E, a.K, a.renorm, s_idx + b * a.K, s_w + b * a.K, ek, wt);
                if (pub && lane < a.K) {
                    const_cast<int32_t*>(a.idx)[b * a.K + lane] = ek;
                    const_cast<float*>(a.w)[b * a.K + lane] = wt;
                }
            }
            __syncthreads();
            sel = load_sel(a, s_idx, s_w);
        } else {
            sel = load_sel(a, a.idx, a.w);
        }
        if (pub) {
            if (!a.logits) {
                for (int t = threadIdx.x; t < a.B * a.K; t += kThreads) {
                    s_idx[t] = a.idx[t];
                    s_w[t] = a.w[t];
                }
                __syncthreads();
            }
            publish_plan<kThreads>(a, s_idx, s_w);
            return;
        }
        uint32_t m[8];
        selected_mask(sel, words[wave], m);
        // slot j: the j-th selected expert, or a shared one
        int n_routed = 0, e = -1;
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int c = __popc(m[q]);
            if (j >= n_routed && j < n_routed + c) {
                uint32_t x = m[q];
                for (int k = n_routed; k < j; ++k) x &= x - 1u;
                e = 32 * q + __ffs(x) - 1;
            }
            n_routed += c;
        }
        if (j >= n_routed + a.n_shared) return;
        // the slot's tokens: lane l holds token number 4 tg + (l & 3) of them
        if (e >= 0) {
            unsigned tm = 0;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                unsigned long long hit = __ballot(sel.v[i] == e);
                while (hit) {
                    const int l = __ffsll(hit) - 1;
                    hit &= hit - 1ull;
                    const int b = ((64 * i + l) * kinv) >> 16;   // / K
                    if ((tm >> b) & 1u) continue;         // a repeated expert counts once, by its first entry
                    tm |= 1u << b;
                    const float wb = lane_f(sel.w[i], l);
#pragma unroll
                    for (int tg = 0; tg < TG; ++tg)
                        if (nt == 4 * tg + (lane & 3)) { mytok[tg] = b; myw[tg] = wb; }
                    ++nt;
                }
            }
        } else {
            nt = a.B;
#pragma unroll
            for (int tg = 0; tg < TG; ++tg) {
                mytok[tg] = min(4 * tg + (lane & 3), a.B - 1);
                myw[tg] = 1.f;
            }
        }
        blob = e >= 0 ? routed_blob(a, e) : reinterpret_cast<const char*>(a.sptr[j - n_routed]);
    }
    if (!SK && i0 >= a.I) return;    // I is a multiple of 4
    nt = uni(nt);
    // lanes without a token of their own load the first one's row
    const int first = uni(mytok[0]);
#pragma unroll
    for (int tg = 0; tg < TG; ++tg)
        if (4 * tg + (lane & 3) >= nt) mytok[tg] = first;
    UpTile z;
    z.rowb = size_t(a.H) * (BF ? 2 : 4);
    z.x = reinterpret_cast<const char*>(a.x);
    z.wg = uni(blob) + size_t(i0) * z.rowb;
    z.up = size_t(a.I) * z.rowb;
    z.nt = nt;
    z.rot = SK ? blk : blk * kWaves + wave;
    z.act = size_t(j) * a.B * a.I + i0;
    if (TG > 1 && z.nt > 4) up_stream<BF, TG, TG, 1, SK, SHARED>(a, z, mytok, myw, red);
    else up_stream<BF, 1, TG, kUpTileSteps, SK, SHARED>(a, z, mytok, myw, red);
}

// down: one workgroup = 4 * RQ output rows; its waves split the (slot, step)
// pairs of all slots evenly and stream them without a break at a slot's end, U
// steps in flight per wave.
// Workgroups start one step apart and run around the pairs (rows a power of
// two apart read different memory channels).
template <bool BF, int RQ, int TG, int W, bool REM, bool SHARED>
__global__ __launch_bounds__(64 * W, (W == 16 ? 4 : TG == 4 ? 2 : TG * RQ == 4 ? 3 : 4)) void ffn_down_tile(FfnArgs a) {
    constexpr int U = W == 16 && TG == 1 ? 4 : 3;
    __shared__ SlotTable p;
    __shared__ float red[W][RQ][TG][16];
    const int lane = threadIdx.x & 63, wave = uni(threadIdx.x >> 6);
    load_slots(a, p);
    const int n_slots = uni(p.n_slots);
    if (blockIdx.x == 0 && threadIdx.x == 0 && a.n_experts)
        atomicAdd(a.n_experts, (unsigned long long)p.n_routed);
    constexpr int esz = BF ? 2 : 4;
    const int h0 = blockIdx.x * 4 * RQ;      // H is a multiple of 4 * RQ
    const size_t rowb = size_t(a.I) * esz;
    const int c = lane >> 2;
    const size_t quad = 4 * rowb;
    const size_t wbase = 2 * size_t(a.I) * a.H * esz + size_t(h0) * rowb;
    const int spr = int((rowb + 255) >> 8);
    const long long T = (long long)n_slots * spr;
    const int t0 = uni(int(T * wave / W)), n = uni(int(T * (wave + 1) / W)) - t0;

    // A step's loads: branch-free (behind a branch every wait would be for all
    // loads in flight).  Lanes of unrouted tokens read a routed token's row:
    // their result rows are not added.  Lanes past a row's end read its last
    // chunk and are cleared (REM) when the step is summed.
    struct Step { uint4 w[RQ], x[TG]; uint32_t tm; int k; };
    const int last = (int(rowb) >> 4) - 1;
    const int first = T > 0 ? int((t0 + (long long)blockIdx.x) % T) : 0;
    int j = first / spr, k = first % spr;    // next step to load
    auto load = [&](Step& st) {
        const uint32_t tm = uint32_t(uni(int(p.tok[j])));
        const char* wp = uni(p.blob[j]) + wbase;
        const int ch = REM ? min(16 * k + c, last) : 16 * k + c;
        const char* ap = reinterpret_cast<const char*>(a.act) + size_t(j) * a.B * rowb;
        st.tm = tm;
        st.k = k;
#pragma unroll
        for (int tg = 0; tg < TG; ++tg) {
            const uint32_t m4 = (tm >> (4 * tg)) & 15u;
            const uint32_t b = (m4 >> (lane & 3)) & 1u ? 4 * tg + (lane & 3) : __ffs(m4 ? m4 << (4 * tg) : tm) - 1;
            const uint32_t ao = b * uint32_t(rowb) + uint32_t(ch) * 16u;
            st.x[tg] = ld_cached(ap + ao);
        }
        const uint32_t wo = uint32_t(lane & 3) * uint32_t(rowb) + uint32_t(ch) * 16u;
#pragma unroll
        for (int q = 0; q < RQ; ++q) st.w[q] = ld_weight<SHARED>(wp + q * quad + wo);
        const bool wrap = k + 1 == spr;
        k = wrap ? 0 : k + 1;
        j = wrap ? (j + 1 == n_slots ? 0 : j + 1) : j;
    };
    const f32x4 fz = f32x4{0.f, 0.f, 0.f, 0.f};
    f32x4 acc[RQ][TG];
#pragma unroll
    for (int q = 0; q < RQ; ++q)
#pragma unroll
        for (int tg = 0; tg < TG; ++tg) acc[q][tg] = fz;
    auto compute = [&](Step& st) {
        if constexpr (REM) {
            const bool in = 16 * st.k + c <= last;
            auto keep = [&](uint4& v) {
                v.x = in ? v.x : 0u; v.y = in ? v.y : 0u; v.z = in ? v.z : 0u; v.w = in ? v.w : 0u;
            };
#pragma unroll
            for (int q = 0; q < RQ; ++q) keep(st.w[q]);
#pragma unroll
            for (int tg = 0; tg < TG; ++tg) keep(st.x[tg]);
        }
#pragma unroll
        for (int tg = 0; tg < TG; ++tg) {
            const uint32_t m4 = (st.tm >> (4 * tg)) & 15u;
            if (TG > 1 && !m4) continue;
            f32x4 d[RQ];
#pragma unroll
            for (int q = 0; q < RQ; ++q) d[q] = mma44<BF>(st.x[tg], st.w[q], fz);
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if ((m4 >> i) & 1u)
#pragma unroll
                    for (int q = 0; q < RQ; ++q) acc[q][tg][i] += d[q][i];
        }
    };
    Step st[U];
    if (n >= U) {
#pragma unroll
        for (int u = 0; u < U; ++u) load(st[u]);
        int t = U;
        for (; t + U <= n; t += U)
#pragma unroll
            for (int u = 0; u < U; ++u) {
                compute(st[u]);
                load(st[u]);
            }
        // the last full round: its loads go on while fewer than U steps are left
        const int left = n - t;
        if (left) {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                compute(st[u]);
                if (u < left) load(st[u]);
            }
#pragma unroll
            for (int u = 0; u < U - 1; ++u)
                if (u < left) compute(st[u]);
        } else {
#pragma unroll
            for (int u = 0; u < U; ++u) compute(st[u]);
        }
    } else {
#pragma unroll
        for (int u = 0; u < U - 1; ++u)
            if (u < n) load(st[u]);
#pragma unroll
        for (int u = 0; u < U - 1; ++u)
            if (u < n) compute(st[u]);
    }
#pragma unroll
    for (int tg = 0; tg < TG; ++tg)
#pragma unroll
        for (int q = 0; q < RQ; ++q) {
            const float v = tile_total(acc[q][tg]);
            if (lane < 16) red[wave][q][tg][lane] = v;
        }
    __syncthreads();
    for (int i = threadIdx.x; i < RQ * TG * 16; i += 64 * W) {
        const int q = i / (TG * 16), tg = (i / 16) % TG, l = i & 15;
        const int b = 4 * tg + (l >> 2);
        if (b >= a.B) continue;
        float s = 0.f;
#pragma unroll
        for (int w = 0; w < W; ++w) s += red[w][q][tg][l];
        a.y[size_t(b) * a.H + h0 + 4 * q + (l & 3)] = s;
    }
}
