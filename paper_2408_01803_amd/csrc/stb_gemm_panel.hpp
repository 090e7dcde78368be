// Prefill products of many tokens (included by stb_gemm.hip).
//
// The fused kernels of stb_gemm.hip expand every weight once per 128 tokens, and the expansion's vector instructions take
// the issue slots that the matrix instructions need.  From a few hundred tokens on it is cheaper to expand once, to memory:
//   gemm_prepare_kernel   the packed planes -> A', fp16 (exactly the operands of the fused kernels, negated), in the order
//                         in which a wavefront of the product reads them, with the residual term of the salient columns
//                         (Eq. 4) as further columns of A'; and those columns of X, gathered, as further columns of X
//   gemm_panel_kernel     Y = X' A'^T over k + n_salient_pad columns: nothing but loads, LDS reads and matrix instructions
//   gemm_square_kernel    the same for 2:4 layers in larger tiles, where its estimated time is less (panel_plan)
// A'  [row group of 128][chunk of 32 columns][row tile][lane = 16 g + i][8]: row i of the tile, columns 8 g .. of the chunk
//     2:4 layers: per 128 columns [stage of 64 columns][row tile][lane = 16 g + i][8 kept weights of columns 16 g ..], twice,
//     then [row tile][lane] index words (16 bits a stage); the residual columns follow in the form above
// X   is read as it is (row-major); xsal [T][n_salient_pad] holds the gathered columns.
// A residual weight t * alpha_r and a main weight are separate fp16 terms: two exact products, as in the fused kernels.
namespace {

constexpr int PN_BUFS = 4;                      // X stages of 64 columns in LDS

constexpr int PN_PAIR24 = 18432;                // 2:4: 128 columns of a row group: two stages of 8 KB and 2 KB of index words

struct PanelShape {
    bool sparse;                                // 2:4 layers: kept weights only, multiplied by the sparse instruction
    int kc;                                     // chunks of 32 columns, residual columns included
    int sp;                                     // residual columns (n_salient_pad)
    int64_t main_bytes, group_bytes;            // of a row group: without and with the residual columns
    int64_t a_bytes;
};

inline PanelShape panel_shape(const stb_layout_t* L) {
    PanelShape s;
    s.sparse = L->cfg.N == 2 && L->cfg.M == 4;
    s.sp = L->n_salient_pad;
    s.kc = (L->cfg.k_in + s.sp) / 32;
    s.main_bytes = s.sparse ? (int64_t)(L->cfg.k_in / 128) * PN_PAIR24 : (int64_t)(L->cfg.k_in / 32) * 8192;
    s.group_bytes = s.main_bytes + (int64_t)(s.sp / 32) * 8192;
    s.a_bytes = (L->n_row_tiles + 15) / 16 * 2 * s.group_bytes;    // an even number of groups: a workgroup of the product takes two
    return s;
}

// The columns of salient entries [u0, u0 + 128) of the layer (any column past the last entry); all threads of the workgroup.
__device__ inline void salient_list(const TiledPlanes& p, int u0, uint32_t* list) {
    if (threadIdx.x < 128) list[threadIdx.x] = 0;
    __syncthreads();
    for (int q = threadIdx.x; q < p.nb; q += 256) {
        int u = (int)p.sal_prefix[q] - u0;
        if (u >= 128 || (int)p.sal_prefix[q + 1] - u0 <= 0) continue;
        for (int w = 0; w < 4; w++)
            for (uint32_t bits = p.sal_bitmap[4 * q + w]; bits; bits &= bits - 1, u++)
                if (u >= 0 && u < 128) list[u] = (uint32_t)(q * 128 + 32 * w + __ffs((int)bits) - 1);
    }
    __syncthreads();
}

// Workgroups [0, n_gather): gathered columns of X, 64 tokens x 128 entries each; [.., + n_res): residual columns of A', a row
// group x 128 entries; the rest: main columns of A', a wavefront a (row tile, superblock) at a time.  Bound by the stores of A'.
template <int N8, bool SPARSE>
__global__ __launch_bounds__(256) void gemm_prepare_kernel(TiledPlanes p, const __half* __restrict__ X, int T, __half* __restrict__ xsal,
                                                           char* __restrict__ A, int64_t main_bytes, int64_t group_bytes, int sp, int n_salient,
                                                           int n_gather, int n_res) {
    __shared__ ScatterLds lut;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, i = lane & 15, g = lane >> 4;
    const int segs = sp / 128;
    int wg = blockIdx.x;
    if (wg < n_gather) {
        uint32_t* const list = reinterpret_cast<uint32_t*>(&lut);
        const int seg = wg % segs, t0 = wg / segs * 64, piece = threadIdx.x & 15;
        salient_list(p, seg * 128, list);
        uint32_t col[8];
#pragma unroll
        for (int e = 0; e < 8; e++) col[e] = list[8 * piece + e];
        const unsigned short* xs = reinterpret_cast<const unsigned short*>(X);
#pragma unroll
        for (int it = 0; it < 4; it++) {
            const int tok = t0 + 16 * it + (threadIdx.x >> 4);
            if (tok >= T) continue;
            const unsigned short* row = xs + (int64_t)tok * p.k;
            uint32_t v[4];
#pragma unroll
            for (int e = 0; e < 4; e++) v[e] = (uint32_t)row[col[2 * e]] | (uint32_t)row[col[2 * e + 1]] << 16;
            // (entries past the last meet zero weights; they are cleared here as well, so that no infinity of X reaches them)
#pragma unroll
            for (int e = 0; e < 8; e++)
                if (seg * 128 + 8 * piece + e >= n_salient) v[e >> 1] &= e & 1 ? 0x0000FFFFu : 0xFFFF0000u;
            *reinterpret_cast<uint4*>(xsal + (int64_t)tok * sp + seg * 128 + 8 * piece) = make_uint4(v[0], v[1], v[2], v[3]);
        }
        return;
    }
    wg -= n_gather;
    if (wg < n_res) {
        uint32_t* const list = reinterpret_cast<uint32_t*>(&lut);
        const int seg = wg % segs, rg = wg / segs, u0 = seg * 128 + wave * 32 + 8 * g;
        char* const out = A + rg * group_bytes + main_bytes + (seg * 4 + wave) * 8192 + lane * 16;
        salient_list(p, seg * 128, list);
        uint32_t col[8];
#pragma unroll
        for (int e = 0; e < 8; e++) col[e] = list[wave * 32 + 8 * g + e];
        for (int r8 = 0; r8 < 8 && rg * 8 + r8 < p.nrt; r8++) {
            const int rt = rg * 8 + r8;
            const uint32_t signs = p.res_sign[((int64_t)rt * p.res_words + (u0 >> 5)) * 16 + i] >> (u0 & 31);
            uint32_t v[4] = {0u, 0u, 0u, 0u};
#pragma unroll
            for (int e = 0; e < 8; e++) {
                const uint32_t q = col[e] >> 7, c = col[e] & 127u;
                const int64_t tile = (int64_t)rt * p.nsb + (q >> 2);
                const uint32_t l16 = 16u * (q & 3u) + (uint32_t)i;
                const uint32_t mb = reinterpret_cast<const uint8_t*>(p.mask)[tile * 1024 + (c >> 6) * 512 + l16 * 8 + ((c >> 3) & 7u)];
                const uint32_t ar = p.res_scale[tile * 64 + l16];
                const uint32_t h = (mb >> (c & 7u)) & 1u && u0 + e < n_salient ? ar | ((signs >> e) & 1u) << 15 : 0u;
                v[e >> 1] |= h << (16 * (e & 1));
            }
            *reinterpret_cast<uint4*>(out + r8 * 1024) = make_uint4(v[0], v[1], v[2], v[3]);
        }
        return;
    }
    wg -= n_res;
    if (!SPARSE) {
        build_luts<N8>(&lut);
        __syncthreads();
    }
    uint32_t T0 = 0x09080404u, T1 = 0x0E0E0D0Cu, K7 = 0x07070707u, K3 = 0x03030303u, K4 = 0x04000400u, KS = 0x80008000u;
    asm volatile("" : "+v"(T0), "+v"(T1), "+v"(K7), "+v"(K3), "+v"(K4), "+v"(KS));
    const int64_t items = (int64_t)p.nrt * p.nsb;
    const int64_t step = (int64_t)((int)gridDim.x - n_gather - n_res) * 4;
    for (int64_t it = (int64_t)wg * 4 + wave; it < items; it += step) {
        const int rt = (int)(it / p.nsb), sb = (int)(it % p.nsb), q = 4 * sb + g;
        HalfData<N8> hd[2];
#pragma unroll
        for (int h = 0; h < 2; h++) load_half<N8>(p, it, lane_offsets<N8>(lane, h), h, hd[h]);
        const uint32_t TL = perm(hd[0].sc.y, hd[0].sc.x, 0x06040200u), TH = perm(hd[0].sc.y, hd[0].sc.x, 0x07050301u);
        if constexpr (SPARSE) {
            char* const out = A + (rt >> 3) * group_bytes + (int64_t)q * PN_PAIR24;
            char* const own = out + (rt & 7) * 1024 + i * 16;
#pragma unroll
            for (int c = 0; c < 8; c++) {                      // columns 16 c .. of the block: stage c / 4, K slot c % 4
                uint32_t v[4];
                sparse_operand(hd[c >> 2], TL, TH, c & 3, K3, K4, KS, v);
                if (q < p.nb) *reinterpret_cast<uint4*>(own + (c >> 2) * 8192 + (c & 3) * 256) = make_uint4(v[0], v[1], v[2], v[3]);
            }
            uint32_t w[2][2];
#pragma unroll
            for (int h = 0; h < 2; h++)
#pragma unroll
                for (int u = 0; u < 2; u++) w[h][u] = index_word24(hd[h].m[u], T0, T1, K7);
            // index word of K slot c: its 16 columns of the first stage below those of the second
            char* const iw = out + 16384 + (rt & 7) * 256 + i * 4;
#pragma unroll
            for (int c = 0; c < 4; c++)
                if (q < p.nb) *reinterpret_cast<uint32_t*>(iw + c * 64) = perm(w[1][c >> 1], w[0][c >> 1], c & 1 ? 0x07060302u : 0x05040100u);
        } else {
            char* const out = A + (rt >> 3) * group_bytes + ((int64_t)(4 * q) * 8 + (rt & 7)) * 1024 + i * 16;
#pragma unroll
            for (int h = 0; h < 2; h++)
#pragma unroll
                for (int t = 0; t < 8; t++) {
                    uint32_t v[4];
                    expand_group<N8>(hd[h], TL, TH, t, lut_fetch<N8>(hd[h], t, &lut, lane & 7), v);
                    if (q < p.nb) *reinterpret_cast<uint4*>(out + (2 * h + (t >> 2)) * 8192 + (t & 3) * 256) = make_uint4(v[0], v[1], v[2], v[3]);
                }
        }
    }
}

// The A operands of one K step (32 columns) of a wavefront: four row tiles, 1 KB each, next to each other.  One asm statement
// (the wait states at its start keep it clear of scalar registers that a vector instruction wrote just before).
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
struct ASet { u32x4 v[4]; };
__device__ inline void fetch_a(ASet& a, uint32_t off, const char* base) {
    asm volatile("s_nop 4\n\t"
                 "global_load_dwordx4 %0, %4, %5\n\tglobal_load_dwordx4 %1, %4, %5 offset:1024\n\t"
                 "global_load_dwordx4 %2, %4, %5 offset:2048\n\tglobal_load_dwordx4 %3, %4, %5 offset:3072"
                 : "=&v"(a.v[0]), "=&v"(a.v[1]), "=&v"(a.v[2]), "=&v"(a.v[3]) : "v"(off), "s"(base));
}
// at most K vector-memory operations younger than this set's are still on their way
template <int K> __device__ inline void wait_a(ASet& a) {
    asm volatile("s_waitcnt vmcnt(%4)" : "+v"(a.v[0]), "+v"(a.v[1]), "+v"(a.v[2]), "+v"(a.v[3]) : "n"(K) : "memory");
}

// A workgroup is 256 rows x 128 tokens: four wavefronts of 64 rows x 128 tokens (128 accumulator registers, two wavefronts a SIMD)
// and 64 KB of X stages, two workgroups a compute unit.  Large dense launches keep the matrix pipes busy for 0.76 to 0.82 of their time (8192 x
// 8192 at T = 2048: 0.80 in 217 us, 3.5 GB through L2), as a library product of that size does; the sparse form for 0.50 (8192 x 28672:
// 610 us), bound by the operands' way through L2 (14.3 MB a us, hit rate 0.72) and LDS.  (Eight wavefronts on 256 tokens, one workgroup a compute unit, read less
// but wait for each other: 266 against 258 us on 8192 x 8192 at T = 2048, 630 against 601 on 11008 x 4096 at 8192.  Four wavefronts
// of 128 x 128 need 256 accumulator registers, which the compiler moves about unless asm statements hold them: gemm_square_kernel, for 2:4.)
constexpr int PN_TOK = 128, PN_XSZ = PN_TOK * 128, PN_LDS = PN_BUFS * PN_XSZ;

// Where a workgroup's X stages come from: 64 columns of its 128 token rows, from X (stages below sx) or the gathered columns.
struct PanelX {
    const char* xt;
    const char* xst;
    uint32_t lds0, last, xpiece, ks, ss;
    int sx, wave, lane;
    __device__ PanelX(const __half* X, int k, const __half* xsal, int sp, int T, int t0, char* lds, int wave_, int lane_)
        : xt(reinterpret_cast<const char*>(X) + (int64_t)t0 * k * 2), xst(reinterpret_cast<const char*>(xsal) + (int64_t)t0 * sp * 2 - (int64_t)(k / 64) * 128),
          lds0((uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)lds), last((uint32_t)(T - 1 - t0)),
          xpiece((uint32_t)(((lane_ & 7) ^ (lane_ >> 3)) * 16)), ks((uint32_t)k * 2u), ss((uint32_t)sp * 2u), sx(k / 64), wave(wave_), lane(lane_) {}
    // Half of the wavefront's share of stage s (the last stage, `end` - 1, again past the end): two loads of 8 token rows; lane l =
    // row l / 8, position l % 8.  An LDS row is a token's 128 bytes of a stage; its 16-byte piece p sits at p ^ (row % 8), so
    // that 8 lanes that read a piece of 8 rows meet 8 positions.
    __device__ void load(int s, int end, int half) const {
        const int sc = s < end ? s : end - 1;
        const char* const base = (sc < sx ? xt : xst) + (int64_t)sc * 128;
        const uint32_t stride = sc < sx ? ks : ss;
        const uint32_t dst = lds0 + (uint32_t)(s & (PN_BUFS - 1)) * PN_XSZ + (uint32_t)wave * 4096u;
#pragma unroll
        for (int v = 0; v < 2; v++) {
            const int u = half * 2 + v;
            const uint32_t row = (uint32_t)(8 * (4 * wave + u) + (lane >> 3));
            load_to_lds(dst + u * 1024, __umul24(row < last ? row : last, stride) + xpiece, base);
        }
    }
};

// acc += A' X' over the stages [s0, s1) (an even number), dense; the A chunk of step h (32 columns) is at abase + 8192 h.  Per step
// a wavefront issues 4 x 8 matrix instructions, the A loads of three steps later, a quarter of its share of X for the stage
// pair after next, and 8 LDS reads (each B operand is reloaded as soon as its four instructions are out).
//   X stage s + 4 overwrites stage s: its loads go out in steps 2 s + 3 (after the barrier there, which every wavefront reaches
//   only with the operands of stage s in registers) and 2 s + 4; they are read from step 2 s + 7 on, behind the wait and the
//   barrier at that step's start.
__device__ __forceinline__ void panel_dense(float4_t (&acc)[4][8], char* lds, const PanelX& px, const char* abase, int s0, int s1) {
    constexpr int RT = 4, TT = 8, YOUNGER = 2 * (2 + RT);
    const int lane = px.lane, i = lane & 15, g = lane >> 4;
    const uint32_t aoff = (uint32_t)lane * 16u;
    auto a_load = [&](ASet& a, int h) { fetch_a(a, aoff, abase + (int64_t)(h < 2 * s1 ? h : 2 * s1 - 1) * 8192); };
    // B operand of token tile tt in step (stage s, half c): row 16 tt + i, piece 4 c + g
    const uint32_t bsel[2] = {(uint32_t)(i * 128 + (g ^ (i & 7)) * 16), (uint32_t)(i * 128 + ((4 + g) ^ (i & 7)) * 16)};
    uint4 b[TT];
    auto b_read = [&](int s, int c, int tt) {
        b[tt] = *reinterpret_cast<const uint4*>(lds + (uint32_t)(s & (PN_BUFS - 1)) * PN_XSZ + bsel[c] + tt * 2048);
    };
    ASet a0, a1, a2, a3;
    px.load(s0, s1, 0);
    px.load(s0, s1, 1);
    px.load(s0 + 1, s1, 0);
    a_load(a0, 2 * s0);
    px.load(s0 + 1, s1, 1);
    a_load(a1, 2 * s0 + 1);
    px.load(s0 + 2, s1, 0);
    a_load(a2, 2 * s0 + 2);
    wait_a<YOUNGER>(a0);
    __syncthreads();
#pragma unroll
    for (int tt = 0; tt < TT; tt++) b_read(s0, 0, tt);

    // step h = (stage s, half c) on the operands `a`; `an` takes those of step h + 3
    auto step = [&](auto odd, ASet& a, ASet& an, int s) {
        constexpr int c = decltype(odd)::value;
        wait_a<YOUNGER>(a);
        if (c) __syncthreads();                  // stage s + 1 is in LDS, everyone's share of it
        if (c) px.load(s + 3, s1, 0); else px.load(s + 2, s1, 1);
        a_load(an, 2 * s + c + 3);
#pragma unroll
        for (int tt = 0; tt < TT; tt++) {
            const half8_t bv = __builtin_bit_cast(half8_t, b[tt]);
#pragma unroll
            for (int r = 0; r < RT; r++)
                acc[r][tt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(half8_t, a.v[r]), bv, acc[r][tt], 0, 0, 0);
            b_read(c ? s + 1 : s, c ^ 1, tt);
        }
    };
    for (int s = s0; s < s1; s += 2) {
        step(IntC<0>{}, a0, a3, s);
        step(IntC<1>{}, a1, a0, s);
        step(IntC<0>{}, a2, a1, s + 1);
        step(IntC<1>{}, a3, a2, s + 1);
    }
    // nothing may still be on its way to this workgroup's registers or LDS
    wait_a<0>(a0);
    wait_a<0>(a1);
    wait_a<0>(a2);
    wait_a<0>(a3);
    __syncthreads();
}

// The index words of a stage pair: four row tiles, 256 bytes each.
struct ISet { uint32_t v[4]; };
__device__ inline void fetch_i(ISet& x, uint32_t off, const char* base) {
    asm volatile("s_nop 4\n\t"
                 "global_load_dword %0, %4, %5\n\tglobal_load_dword %1, %4, %5 offset:256\n\t"
                 "global_load_dword %2, %4, %5 offset:512\n\tglobal_load_dword %3, %4, %5 offset:768"
                 : "=&v"(x.v[0]), "=&v"(x.v[1]), "=&v"(x.v[2]), "=&v"(x.v[3]) : "v"(off), "s"(base));
}
template <int K> __device__ inline void wait_i(ISet& x) {
    asm volatile("s_waitcnt vmcnt(%4)" : "+v"(x.v[0]), "+v"(x.v[1]), "+v"(x.v[2]), "+v"(x.v[3]) : "n"(K) : "memory");
}

// The same on the kept weights of a 2:4 layer (v_smfmac_f32_16x16x64_f16: a stage of 64 columns is one K step); the pair of stages
// 2 p, 2 p + 1 is at abase + PN_PAIR24 p, its index words at ibase + PN_PAIR24 p.  Per stage a wavefront issues 32 matrix instructions,
// the A loads of two stages later, its X loads of three stages later, every other stage the index words of the next pair, and 16
// LDS reads: the B operand of a token tile (pieces g and 4 + g of its rows) is reloaded, four tiles ahead, once its four
// instructions are out.
//   X stage s + 3 overwrites stage s - 1: its loads go out behind the barrier of stage s, which every wavefront reaches with the
//   products of stage s - 1 issued; it is first read in stage s + 2 (its tiles 0 .. 3, ahead), behind that stage's barrier.
__device__ __forceinline__ void panel_sparse(float4_t (&acc)[4][8], char* lds, const PanelX& px, const char* abase, const char* ibase, int s0, int s1) {
    typedef uint32_t u32x8 __attribute__((ext_vector_type(8)));
    constexpr int RT = 4, TT = 8;
    const int lane = px.lane, i = lane & 15, g = lane >> 4;
    const uint32_t aoff = (uint32_t)lane * 16u, ioff = (uint32_t)lane * 4u;
    auto a_load = [&](ASet& a, int s) {
        const int sc = s < s1 ? s : s1 - 1;
        fetch_a(a, aoff, abase + (int64_t)(sc >> 1) * PN_PAIR24 + (sc & 1) * 8192);
    };
    auto i_load = [&](ISet& x, int s) { fetch_i(x, ioff, ibase + (int64_t)((s < s1 ? s : s1 - 1) >> 1) * PN_PAIR24); };
    const uint32_t blo = (uint32_t)(i * 128 + (g ^ (i & 7)) * 16);         // (piece 4 + g: the same with bit 6 of the address flipped)
    u32x8 b[4];
    auto b_read = [&](int s, int tt) {
        const char* const base = lds + (uint32_t)(s & (PN_BUFS - 1)) * PN_XSZ + tt * 2048;
        const uint4 lo = *reinterpret_cast<const uint4*>(base + blo), hi = *reinterpret_cast<const uint4*>(base + (blo ^ 64u));
        b[tt & 3] = u32x8{lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
    };
    ASet a0, a1, a2;
    ISet i0, i1;
    px.load(s0, s1, 0);
    px.load(s0, s1, 1);
    px.load(s0 + 1, s1, 0);
    px.load(s0 + 1, s1, 1);
    a_load(a0, s0);
    i_load(i0, s0);
    px.load(s0 + 2, s1, 0);
    px.load(s0 + 2, s1, 1);
    a_load(a1, s0 + 1);
    wait_a<8>(a0);
    wait_i<8>(i0);
    __syncthreads();
#pragma unroll
    for (int tt = 0; tt < 4; tt++) b_read(s0, tt);

    // stage s on the operands `a` and index words `x`; `an` takes the A of stage s + 2, `xn` (even stages) the next pair's index words.
    // Younger than what an even stage waits for: the X and A loads of the stage before; an odd one's: also a pair's index words.
    auto step = [&](auto odd, ASet& a, ASet& an, ISet& x, ISet& xn, int s) {
        constexpr int c = decltype(odd)::value;
        if (c) wait_a<12>(a);
        else { wait_a<8>(a); wait_i<8>(x); }
        __syncthreads();                         // stage s + 1 is in LDS, everyone's share of it
        px.load(s + 3, s1, 0);
        px.load(s + 3, s1, 1);
        a_load(an, s + 2);
        if (!c) i_load(xn, s + 2);
#pragma unroll
        for (int tt = 0; tt < TT; tt++) {
            const half16_t bv = __builtin_bit_cast(half16_t, b[tt & 3]);
#pragma unroll
            for (int r = 0; r < RT; r++)
                acc[r][tt] = __builtin_amdgcn_smfmac_f32_16x16x64_f16(__builtin_bit_cast(half8_t, a.v[r]), bv, acc[r][tt], (int)x.v[r], 0, c);
            if (tt < 4) b_read(s, tt + 4);
            else b_read(s + 1, tt - 4);
        }
    };
    for (int s = s0;; s += 12) {                 // (3 sets of A, 2 of index words: 6 pairs until they meet again)
        step(IntC<0>{}, a0, a2, i0, i1, s);
        step(IntC<1>{}, a1, a0, i0, i1, s + 1);
        if (s + 2 >= s1) break;
        step(IntC<0>{}, a2, a1, i1, i0, s + 2);
        step(IntC<1>{}, a0, a2, i1, i0, s + 3);
        if (s + 4 >= s1) break;
        step(IntC<0>{}, a1, a0, i0, i1, s + 4);
        step(IntC<1>{}, a2, a1, i0, i1, s + 5);
        if (s + 6 >= s1) break;
        step(IntC<0>{}, a0, a2, i1, i0, s + 6);
        step(IntC<1>{}, a1, a0, i1, i0, s + 7);
        if (s + 8 >= s1) break;
        step(IntC<0>{}, a2, a1, i0, i1, s + 8);
        step(IntC<1>{}, a0, a2, i0, i1, s + 9);
        if (s + 10 >= s1) break;
        step(IntC<0>{}, a1, a0, i1, i0, s + 10);
        step(IntC<1>{}, a2, a1, i1, i0, s + 11);
        if (s + 12 >= s1) break;
    }
    wait_a<0>(a0);
    wait_a<0>(a1);
    wait_a<0>(a2);
    wait_i<0>(i0);
    wait_i<0>(i1);
    __syncthreads();
}

// The product over stages [2 * pairs_per * split, ..) of 64 columns.
template <bool SPARSE, bool SPLIT>
__global__ __launch_bounds__(256, 2) void gemm_panel_kernel(const char* __restrict__ A, int64_t main_bytes, int64_t group_bytes, int stages,
                                                            const __half* __restrict__ X, int k, const __half* __restrict__ xsal, int sp, int T, int n,
                                                            void* __restrict__ Y, int y_fp32, float* __restrict__ part,
                                                            int pairs_per, int tiles_t, int tiles_r, int total) {
    extern __shared__ __attribute__((aligned(16))) char lds[];
    // consecutive workgroups go to the 8 XCDs in turn: give each XCD a contiguous run of tiles, 4 token tiles x some rows,
    // so that its L2 sees few row groups and few token rows
    const int per = (total + 7) / 8, lin = (int)(blockIdx.x & 7) * per + (int)(blockIdx.x >> 3);
    if ((int)(blockIdx.x >> 3) >= per || lin >= total) return;
    const int tiles = tiles_t * tiles_r, split = __builtin_amdgcn_readfirstlane(lin / tiles), rem = lin - split * tiles;
    const int tg = __builtin_amdgcn_readfirstlane(rem / (4 * tiles_r)), width = tiles_t - 4 * tg < 4 ? tiles_t - 4 * tg : 4, idx = rem - tg * 4 * tiles_r;
    const int row_tile = __builtin_amdgcn_readfirstlane(idx / width), t0 = (4 * tg + idx - row_tile * width) * PN_TOK;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, i = lane & 15, g = lane >> 4;
    const int s0 = SPLIT ? 2 * pairs_per * split : 0, s1 = SPLIT && s0 + 2 * pairs_per < stages ? s0 + 2 * pairs_per : stages;
    float4_t acc[4][8];
#pragma unroll
    for (int r = 0; r < 4; r++)
#pragma unroll
        for (int tt = 0; tt < 8; tt++) acc[r][tt] = float4_t{0.0f, 0.0f, 0.0f, 0.0f};

    const PanelX px(X, k, xsal, sp, T, t0, lds, wave, lane);
    // two wavefronts a row group: its upper and lower four row tiles
    const char* const group = A + (row_tile * 2 + (wave >> 1)) * group_bytes;
    if constexpr (SPARSE) {
        const int sx = px.sx, e = s1 < sx ? s1 : sx, d0 = s0 > sx ? s0 : sx;
        if (s0 < e) panel_sparse(acc, lds, px, group + (wave & 1) * 4096, group + 16384 + (wave & 1) * 1024, s0, e);
        if (d0 < s1) panel_dense(acc, lds, px, group + main_bytes - (int64_t)sx * 16384 + (wave & 1) * 4096, d0, s1);
    } else panel_dense(acc, lds, px, group + (wave & 1) * 4096, s0, s1);

    // D[row][token]: lane = token i, rows 4 g + v
    float* const ep = reinterpret_cast<float*>(lds + wave * ST_AREA);
    if (SPLIT) { Y = part + (int64_t)split * T * n; y_fp32 = 1; }
#pragma unroll
    for (int tp = 0; tp < 8; tp += 2) {
#pragma unroll
        for (int h = 0; h < 2; h++)
#pragma unroll
            for (int r = 0; r < 4; r++) *reinterpret_cast<float4_t*>(ep + (16 * h + i) * ST_ES + 16 * r + 4 * g) = -acc[r][tp + h];
        store_runs(ep, t0 + 16 * tp, row_tile * 256 + wave * 64, Y, y_fp32, T, n, lane);
    }
}

// ---- 2:4 layers, tiles of 256 rows x 256 tokens ------------------------------------------------------------------------
// A K step of 64 columns costs a sparse product half the matrix instructions of a dense one and the same bytes of X: two workgroups of
// gemm_panel_kernel bring 68 KB a stage to a compute unit whose matrix instructions take 1024 cycles, and run at the rate of those
// bytes (pipes 0.50 busy).  One workgroup of 256 x 256 whose A' goes through LDS as well brings 50: four wavefronts, one a SIMD, of 128 x
// 128 each, three stages of X and A' in LDS, the loads of a stage two stages ahead.  256 accumulator registers a wavefront: the matrix
// instructions are asm statements that keep them in AGPRs (left to the compiler, the loop holds up to 484 register copies).  A lone
// wavefront issues everything in its one stream, so loads and LDS reads are dealt out one or two behind a matrix instruction.
// Same order of additions as gemm_panel_kernel: the same bits.  8192 x 28672 at T = 2048: pipes 0.58 busy, the call 661 -> 581 us; 8192 x
// 8192 at 2048 175 -> 160, 4096 x 4096 at 4096 99 -> 93.5.  The 32 x 32 x 32 form of the instruction: 583, 161 and 96.  Dense layers gain
// nothing (8192 x 8192 6:8 at 2048 250 -> 248, 8192 x 8192 4:8 at 8192 798 -> 796, 11008 x 4096 4:8 at 8192 592 -> 616).
constexpr int SQ_TOK = 256, SQ_X = SQ_TOK * 128, SQ_A = 16384, SQ_STAGE = SQ_X + SQ_A, SQ_BUFS = 3;
constexpr int SQ_I = SQ_BUFS * SQ_STAGE;                        // index words of two stage pairs, behind the stages
constexpr int SQ_LDS = SQ_I + 2 * 4096;
static_assert(2 * (SQ_X + 2 * SQ_A) <= SQ_LDS && 4 * ST_AREA <= SQ_LDS, "two stages of residual columns; the output tiles");

// at most K vector-memory operations still on their way
template <int K> __device__ inline void wait_loads() { asm volatile("s_waitcnt vmcnt(%0)" : : "n"(K) : "memory"); }

typedef uint32_t u32x8 __attribute__((ext_vector_type(8)));
typedef float4_t SquareAcc[8][8];               // 16 x 16 tiles of a wavefront: [row tile][token tile]
__device__ __forceinline__ void dense_into(float4_t& acc, u32x4 a, u32x4 b) { asm volatile("v_mfma_f32_16x16x32_f16 %0, %1, %2, %0" : "+a"(acc) : "v"(a), "v"(b)); }
template <int SECOND> __device__ __forceinline__ void sparse_into(float4_t& acc, u32x4 a, u32x8 b, uint32_t x) {
    if (SECOND) asm volatile("v_smfmac_f32_16x16x64_f16 %0, %1, %2, %3 abid:1" : "+a"(acc) : "v"(a), "v"(b), "v"(x));
    else asm volatile("v_smfmac_f32_16x16x64_f16 %0, %1, %2, %3" : "+a"(acc) : "v"(a), "v"(b), "v"(x));
}
// The compiler does not know that the statements above are matrix instructions: nothing may read their accumulators before this
// (32 wait states, more than a 16 x 16 instruction takes to write back), and nothing but LDS reads may write their operands right before
// them (index words are moved at the end of a turn of the loop: the wait states at its start).
__device__ __forceinline__ void settle(SquareAcc& acc) {
#pragma unroll
    for (int r = 0; r < 8; r++)
        asm volatile("s_nop 15\n\ts_nop 15" : "+a"(acc[r][0]), "+a"(acc[r][1]), "+a"(acc[r][2]), "+a"(acc[r][3]), "+a"(acc[r][4]), "+a"(acc[r][5]), "+a"(acc[r][6]), "+a"(acc[r][7]));
}

// load_to_lds at base + OFF in LDS
template <int OFF> __device__ __forceinline__ void load_to_lds_at(uint32_t lds_base, uint32_t voff, const void* base) {
    asm volatile("s_add_u32 m0, %0, %3\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" : : "s"(lds_base), "v"(voff), "s"(base), "n"(OFF) : "memory", "m0", "scc");
}

// What a wavefront loads of a stage: 64 of its 256 token rows of 64 columns, and its share of A'.  An LDS row is a token's 128 bytes; its
// 16-byte piece p sits at p ^ (row / 2 % 8), which spreads the rows that one cycle of a 16-byte LDS read takes over all banks.
struct SquareLoads {
    const char* xt;                             // token rows of the workgroup, from the first
    const char* group;                          // A' of its two row groups
    int64_t group_bytes;
    uint32_t lds0;
    uint32_t xoff[8], aoff[8];
    int wave, lane;
    __device__ SquareLoads(const char* rows, uint32_t stride, int T, int t0, const char* group_, int64_t group_bytes_, char* lds, int wave_, int lane_)
        : xt(rows + (int64_t)t0 * stride), group(group_), group_bytes(group_bytes_),
          lds0((uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)lds), wave(wave_), lane(lane_) {
        const uint32_t last = (uint32_t)(T - 1 - t0);
#pragma unroll
        for (int u = 0; u < 8; u++) {
            const uint32_t row = (uint32_t)(64 * wave + 8 * u + (lane >> 3));
            xoff[u] = __umul24(row < last ? row : last, stride) + ((((uint32_t)lane & 7u) ^ (row >> 1 & 7u)) * 16u);
            aoff[u] = (uint32_t)(lane * 16 + 1024 * u);
        }
    }
    // row i, piece g of the 16 rows of an operand
    __device__ uint32_t b_lane() const { return (uint32_t)(wave & 1) * 16384u + (uint32_t)((lane & 15) * 128 + ((lane >> 4) ^ (lane >> 1 & 7)) * 16); }
    __device__ uint32_t a_lane() const { return SQ_X + (uint32_t)(wave >> 1) * 8192u + (uint32_t)lane * 16u; }
};

// acc += A' X' over the stages [s0, s1) (an even number) of kept weights.  Stage s: 8 token tiles of 8 matrix instructions; the B operand of a
// tile is read four tiles ahead.  Behind tile 4 all of the stage's LDS reads are back: the wait and the barrier there say that stage s + 1 is in
// LDS and that nobody reads stage s any more, so that the loads of stage s + 3 go out in its place and the operands of s + 1 are read.
__device__ __forceinline__ void square_sparse(SquareAcc& acc, char* lds, const SquareLoads& pq, int s0, int s1) {
    // the wavefront's share of a stage: 8 loads of X, 4 of A', and (even stages) one of the pair's index words
    const char* const own = pq.group + (int64_t)(pq.wave >> 1) * pq.group_bytes + (pq.wave & 1) * 4096;
    const char* const iown = pq.group + (int64_t)(pq.wave >> 1) * pq.group_bytes + 16384 + (pq.wave & 1) * 1024;
    const uint32_t xdst = pq.lds0 + (uint32_t)pq.wave * 8192u, adst = pq.lds0 + SQ_X + (uint32_t)pq.wave * 4096u, idst = pq.lds0 + SQ_I + (uint32_t)pq.wave * 1024u;
    auto load = [&](auto which, int s, uint32_t buf) {
        constexpr int u = decltype(which)::value;
        const int sc = s < s1 ? s : s1 - 1;
        if constexpr (u < 8) load_to_lds_at<u * 1024>(xdst + buf, pq.xoff[u], pq.xt + (int64_t)sc * 128);
        else if constexpr (u < 12) load_to_lds_at<(u - 8) * 1024>(adst + buf, pq.aoff[u - 8], own + (int64_t)(sc >> 1) * PN_PAIR24 + (sc & 1) * 8192);
        else load_to_lds_at<0>(idst + (uint32_t)((s >> 1) & 1) * 4096u, pq.aoff[0], iown + (int64_t)(sc >> 1) * PN_PAIR24);
    };
    const uint32_t alane = pq.a_lane();
    const uint32_t ilane = SQ_I + (uint32_t)(pq.wave >> 1) * 2048u + (uint32_t)pq.lane * 4u;
    const uint32_t blane = pq.b_lane();
    u32x8 b[4];
    u32x4 a0[8], a1[8];
    uint32_t x0[8], x1[8];
    auto b_read = [&](uint32_t buf, int tt) {              // pieces g and 4 + g
        const char* const base = lds + tt * 2048;
        const uint4 lo = *reinterpret_cast<const uint4*>(base + (buf + blane)), hi = *reinterpret_cast<const uint4*>(base + (buf + (blane ^ 64u)));
        b[tt & 3] = u32x8{lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
    };
    auto a_read = [&](u32x4 (&a)[8], uint32_t buf, int r) { a[r] = *reinterpret_cast<const u32x4*>(lds + (buf + alane) + r * 1024); };
    auto i_read = [&](uint32_t (&x)[8], int s, int r) {
        x[r] = *reinterpret_cast<const uint32_t*>(lds + (((uint32_t)(s >> 1) & 1u) * 4096u + ilane) + r * 256);
    };
    auto all_loads = [&](auto with_index, int s, uint32_t buf) {
        load(IntC<0>{}, s, buf); load(IntC<1>{}, s, buf); load(IntC<2>{}, s, buf); load(IntC<3>{}, s, buf);
        load(IntC<4>{}, s, buf); load(IntC<5>{}, s, buf); load(IntC<6>{}, s, buf); load(IntC<7>{}, s, buf);
        load(IntC<8>{}, s, buf); load(IntC<9>{}, s, buf); load(IntC<10>{}, s, buf); load(IntC<11>{}, s, buf);
        if constexpr (decltype(with_index)::value) load(IntC<12>{}, s, buf);
    };
    constexpr uint32_t SZ = SQ_STAGE;
    all_loads(IntC<1>{}, s0, 0);
    all_loads(IntC<0>{}, s0 + 1, SZ);
    all_loads(IntC<1>{}, s0 + 2, 2 * SZ);
    wait_loads<12 + 13>();
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 8; q++) a_read(a0, 0, q);
#pragma unroll
    for (int q = 0; q < 8; q++) i_read(x0, s0, q);
#pragma unroll
    for (int tt = 0; tt < 4; tt++) b_read(0, tt);

    uint32_t cur = 0, next = SZ;
    // stage s on the operands `a` and index words `x`; `an` (and, odd stages, `xn`) takes those of the next
    auto step = [&](auto odd, u32x4 (&a)[8], u32x4 (&an)[8], uint32_t (&x)[8], uint32_t (&xn)[8], int s) {
        constexpr int c = decltype(odd)::value;
        auto one = [&](auto tile, auto row) {
            constexpr int tt = decltype(tile)::value, r = decltype(row)::value;
            sparse_into<c>(acc[r][tt], a[r], b[tt & 3], x[r]);
            if constexpr (tt < 4 && r == 7) b_read(cur, tt + 4);
            if constexpr (tt == 4 && r == 7) {
                wait_loads<c ? 12 : 13>();       // (those of stage s + 2)
                __syncthreads();
                b_read(next, 0);
            }
            if constexpr (tt > 4) {
                constexpr int slot = (tt - 5) * 4 + r / 2;
                if constexpr (r % 2 == 0) load(IntC<slot>{}, s + 3, cur);
                if constexpr (r % 2 == 1 && slot < 8) a_read(an, next, slot);
                if constexpr (r % 2 == 1 && slot >= 4 && c) i_read(xn, s + 1, slot - 4);
                if constexpr (slot == 10 && r % 2 == 1 && c) load(IntC<12>{}, s + 3, cur);
                if constexpr (r == 7) b_read(next, tt - 4);
            }
            __builtin_amdgcn_sched_barrier(0);
        };
        auto eight = [&](auto tile) {
            one(tile, IntC<0>{}); one(tile, IntC<1>{}); one(tile, IntC<2>{}); one(tile, IntC<3>{});
            one(tile, IntC<4>{}); one(tile, IntC<5>{}); one(tile, IntC<6>{}); one(tile, IntC<7>{});
        };
        eight(IntC<0>{}); eight(IntC<1>{}); eight(IntC<2>{}); eight(IntC<3>{});
        eight(IntC<4>{}); eight(IntC<5>{}); eight(IntC<6>{}); eight(IntC<7>{});
        cur = next;
        next = next == 2 * SZ ? 0 : next + SZ;
    };
    for (int s = s0; s < s1; s += 2) {
        asm volatile("s_nop 1");
        step(IntC<0>{}, a0, a1, x0, x1, s);
        step(IntC<1>{}, a1, a0, x0, x1, s + 1);
#pragma unroll
        for (int q = 0; q < 8; q++) x0[q] = x1[q];
    }
    wait_loads<0>();
    __syncthreads();
}

// The same over the stages [d0, d1) of 64 residual columns behind pq's rows (the gathered columns) and abase: two stages in LDS (X, then two chunks
// of A'), a chunk of 32 columns a step.  In a stage's second step all its LDS reads are issued: wait and barrier as above, behind the first tile.
__device__ __forceinline__ void square_dense(SquareAcc& acc, char* lds, const SquareLoads& pq, const char* abase, int d0, int d1) {
    constexpr uint32_t SZ = SQ_X + 2 * SQ_A;
    // the wavefront's share of a stage: 8 loads of X, 8 of A' (chunk wave & 1 of row group wave >> 1)
    const char* const own = abase + (int64_t)(pq.wave >> 1) * pq.group_bytes + (pq.wave & 1) * 8192;
    const uint32_t xdst = pq.lds0 + (uint32_t)pq.wave * 8192u, adst = pq.lds0 + SQ_X + (uint32_t)(pq.wave & 1) * 16384u + (uint32_t)(pq.wave >> 1) * 8192u;
    auto load = [&](auto which, int s, uint32_t buf) {
        constexpr int u = decltype(which)::value;
        const int sc = s < d1 ? s : d1 - 1;
        if constexpr (u < 8) load_to_lds_at<u * 1024>(xdst + buf, pq.xoff[u], pq.xt + (int64_t)sc * 128);
        else load_to_lds_at<(u - 8) * 1024>(adst + buf, pq.aoff[u - 8], own + (int64_t)sc * 16384);
    };
    const uint32_t alane = pq.a_lane();
    const uint32_t blane = pq.b_lane();
    u32x4 b[8], a0[8], a1[8];
    auto b_read = [&](uint32_t buf, int c, int tt) { b[tt] = *reinterpret_cast<const u32x4*>(lds + (buf + (blane ^ (uint32_t)(64 * c))) + tt * 2048); };
    auto a_read = [&](u32x4 (&a)[8], uint32_t buf, int c, int r) { a[r] = *reinterpret_cast<const u32x4*>(lds + (buf + alane) + c * 16384 + r * 1024); };
    auto all_loads = [&](int s, uint32_t buf) {
        load(IntC<0>{}, s, buf); load(IntC<1>{}, s, buf); load(IntC<2>{}, s, buf); load(IntC<3>{}, s, buf);
        load(IntC<4>{}, s, buf); load(IntC<5>{}, s, buf); load(IntC<6>{}, s, buf); load(IntC<7>{}, s, buf);
        load(IntC<8>{}, s, buf); load(IntC<9>{}, s, buf); load(IntC<10>{}, s, buf); load(IntC<11>{}, s, buf);
        load(IntC<12>{}, s, buf); load(IntC<13>{}, s, buf); load(IntC<14>{}, s, buf); load(IntC<15>{}, s, buf);
    };
    all_loads(d0, 0);
    all_loads(d0 + 1, SZ);
    wait_loads<16>();
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 8; q++) a_read(a0, 0, 0, q);
#pragma unroll
    for (int q = 0; q < 8; q++) b_read(0, 0, q);
    uint32_t cur = 0;
    auto step = [&](auto odd, u32x4 (&a)[8], u32x4 (&an)[8], int s) {
        constexpr int c = decltype(odd)::value;
        const uint32_t from = c ? SZ - cur : cur;              // where the next step's operands are
        auto one = [&](auto tile, auto row) {
            constexpr int tt = decltype(tile)::value, r = decltype(row)::value;
            dense_into(acc[r][tt], a[r], b[tt]);
            if constexpr (c && tt == 0 && r == 7) {
                wait_loads<0>();
                __syncthreads();
            }
            if constexpr (r == 7) b_read(from, c ^ 1, tt);
            if constexpr (tt > 0 && r == 0) a_read(an, from, c ^ 1, tt - 1);
            if constexpr (tt == 7 && r == 1) a_read(an, from, c ^ 1, 7);
            if constexpr (c && tt > 0 && r % 2 == 1 && r > 1) {
                constexpr int u = (tt - 1) * 3 + r / 2 - 1;
                if constexpr (u < 16) load(IntC<u>{}, s + 2, cur);
            }
            __builtin_amdgcn_sched_barrier(0);
        };
        auto eight = [&](auto tile) {
            one(tile, IntC<0>{}); one(tile, IntC<1>{}); one(tile, IntC<2>{}); one(tile, IntC<3>{});
            one(tile, IntC<4>{}); one(tile, IntC<5>{}); one(tile, IntC<6>{}); one(tile, IntC<7>{});
        };
        eight(IntC<0>{}); eight(IntC<1>{}); eight(IntC<2>{}); eight(IntC<3>{});
        eight(IntC<4>{}); eight(IntC<5>{}); eight(IntC<6>{}); eight(IntC<7>{});
        if (c) cur = SZ - cur;
    };
    for (int s = d0; s < d1; s++) {
        step(IntC<0>{}, a0, a1, s);
        step(IntC<1>{}, a1, a0, s);
    }
    wait_loads<0>();
    __syncthreads();
}

template <bool SPLIT>
__global__ __launch_bounds__(256, 1) void gemm_square_kernel(const char* __restrict__ A, int64_t main_bytes, int64_t group_bytes, int stages,
                                                             const __half* __restrict__ X, int k, const __half* __restrict__ xsal, int sp, int T, int n,
                                                             void* __restrict__ Y, int y_fp32, float* __restrict__ part,
                                                             int pairs_per, int tiles_t, int tiles_r, int total) {
    extern __shared__ __attribute__((aligned(16))) char lds[];
    const int per = (total + 7) / 8, lin = (int)(blockIdx.x & 7) * per + (int)(blockIdx.x >> 3);
    if ((int)(blockIdx.x >> 3) >= per || lin >= total) return;
    const int tiles = tiles_t * tiles_r, split = __builtin_amdgcn_readfirstlane(lin / tiles), rem = lin - split * tiles;
    const int tg = __builtin_amdgcn_readfirstlane(rem / (4 * tiles_r)), width = tiles_t - 4 * tg < 4 ? tiles_t - 4 * tg : 4, idx = rem - tg * 4 * tiles_r;
    const int row_tile = __builtin_amdgcn_readfirstlane(idx / width), t0 = (4 * tg + idx - row_tile * width) * SQ_TOK;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int s0 = SPLIT ? 2 * pairs_per * split : 0, s1 = SPLIT && s0 + 2 * pairs_per < stages ? s0 + 2 * pairs_per : stages;
    SquareAcc acc;
#pragma unroll
    for (int r = 0; r < 8; r++)
#pragma unroll
        for (int tt = 0; tt < 8; tt++) acc[r][tt] = float4_t{0.0f, 0.0f, 0.0f, 0.0f};
    const char* const group = A + (int64_t)(row_tile * 2) * group_bytes;
    const int sx = k / 64, e = s1 < sx ? s1 : sx, d0 = s0 > sx ? s0 : sx;
    if (s0 < e) {
        const SquareLoads pq(reinterpret_cast<const char*>(X), (uint32_t)k * 2u, T, t0, group, group_bytes, lds, wave, lane);
        square_sparse(acc, lds, pq, s0, e);
    }
    if (d0 < s1) {
        const SquareLoads pq(reinterpret_cast<const char*>(xsal), (uint32_t)sp * 2u, T, t0, group, group_bytes, lds, wave, lane);
        square_dense(acc, lds, pq, group + main_bytes, d0 - sx, s1 - sx);
    }
    settle(acc);
    float* const ep = reinterpret_cast<float*>(lds + wave * ST_AREA);
    if (SPLIT) { Y = part + (int64_t)split * T * n; y_fp32 = 1; }
#pragma unroll
    for (int rh = 0; rh < 2; rh++)
#pragma unroll
        for (int q = 0; q < 4; q++) {                  // 32 tokens x 64 rows at a time; D[row][token]: lane = token i, rows 4 g + v
#pragma unroll
            for (int h = 0; h < 2; h++)
#pragma unroll
                for (int r = 0; r < 4; r++)
                    *reinterpret_cast<float4_t*>(ep + (16 * h + (lane & 15)) * ST_ES + 16 * r + 4 * (lane >> 4)) = -acc[4 * rh + r][2 * q + h];
            store_runs(ep, t0 + 128 * (wave & 1) + 32 * q, row_tile * 256 + (wave >> 1) * 128 + rh * 64, Y, y_fp32, T, n, lane);
        }
}

enum { PN_DENSE, PN_SPARSE, PN_SQUARE };        // gemm_panel_kernel on either kind of layer, gemm_square_kernel
template <int KIND, bool SPLIT>
hipError_t launch_panel_as(hipStream_t st, const char* A, const PanelShape& ps, const __half* X, int k, const __half* xsal, int T, int n,
                           void* Y, int y_fp32, float* part, int groups, int pairs_per) {
    static std::atomic<bool> attr_set{false};              // a failure is not remembered: the next call tries again
    constexpr int lds = KIND == PN_SQUARE ? SQ_LDS : PN_LDS, tok = KIND == PN_SQUARE ? SQ_TOK : PN_TOK;
    const auto fn = [] {
        if constexpr (KIND == PN_SQUARE) return gemm_square_kernel<SPLIT>;
        else return gemm_panel_kernel<KIND == PN_SPARSE, SPLIT>;
    }();
    if (!attr_set.load(std::memory_order_acquire)) {
        const hipError_t attr = hipFuncSetAttribute((const void*)fn, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
        if (attr != hipSuccess) return attr;
        attr_set.store(true, std::memory_order_release);
    }
    const int tiles_t = (T + tok - 1) / tok, tiles_r = (n + 255) / 256, total = tiles_t * tiles_r * groups;
    hipLaunchKernelGGL(fn, dim3((unsigned)((total + 7) / 8 * 8)), dim3(256), lds, st, A, ps.main_bytes, ps.group_bytes, ps.kc / 2, X, k, xsal, ps.sp, T, n, Y, y_fp32, part,
                       pairs_per, tiles_t, tiles_r, total);
    return hipGetLastError();
}

struct PanelPlan {
    int groups, pairs_per;                      // K split: groups of pairs_per stage pairs (1 group: none)
    bool square;                                // tiles of 256 x 256 (gemm_square_kernel)
};

template <int N8, bool SPARSE>
hipError_t launch_prepare(hipStream_t st, const TiledPlanes& p, const stb_layout_t* L, const PanelShape& ps, const __half* X, int T, char* A, __half* xsal) {
    const int segs = ps.sp / 128, n_gather = (T + 63) / 64 * segs, n_res = (p.nrt + 7) / 8 * segs;
    const int64_t items = (int64_t)p.nrt * p.nsb;
    const int main_wgs = items / 4 < 2048 ? (int)((items + 3) / 4) : 2048;
    hipLaunchKernelGGL((gemm_prepare_kernel<N8, SPARSE>), dim3((unsigned)(n_gather + n_res + main_wgs)), dim3(256), 0, st, p, X, T, xsal, A,
                       ps.main_bytes, ps.group_bytes, ps.sp, L->cfg.n_salient, n_gather, n_res);
    return hipGetLastError();
}

}  // namespace
