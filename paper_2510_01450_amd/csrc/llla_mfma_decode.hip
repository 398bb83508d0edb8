// Matrix-core decode path of Local Linear Attention for gfx950: bf16 caches, d = 64, cache capacity
// L_max >= 256, optional per-sequence lengths.  One query per (batch, head) against a cache that already
// holds the new token: the last row of the causal forward (Section 2.3: LLA keeps a Theta(n d) KV
// cache; Section 3.2: rows are independent).
//
// The cache is streamed from HBM exactly once.  In a single pass each wave accumulates, for its
// share of the keys and relative to its own running maximum m (the online rescaling of Algorithm 1),
//     omega = sum w,  mu~ = sum w k,  Sigma~ = sum w k k^T   (Eq. (tilded_form))
//     y0v   = sum w v,  G~ = sum w k v^T                      (value moments)
// as f16 MFMA accumulators: (w (.) K)^T [K | V] with the key as the contraction index.  Eq. (lla) then
// needs no second pass over the cache:  o = sum_j w_j (y0 + k_j . y1) v_j = y0 * y0v + G~^T y1,
// where [y0; y1] solves [omega mu~^T; mu~ Sigma~ + lambda I] y = [1; q].  The four waves of a workgroup merge their
// moments in LDS; with one workgroup per head it solves and writes o itself, otherwise it leaves a record and a
// second kernel merges a head's records, solves and writes (llla_decode_tail.hpp).
#include "llla_decode_tail.hpp"

#include <algorithm>

namespace llla {
namespace {

using namespace mfma;

using S64 = Shape<64>;
constexpr int D = S64::D, NT = DEC_NT;
__host__ __device__ constexpr int tix(int I, int J) { return S64::tix(I, J); }

constexpr int STEP = 32;                       // keys per MFMA step
constexpr int NSTAGE = 2;                      // LDS stages per wave
constexpr int TILE_H = STEP * D;               // halves of one natural [32 keys][64] tile (4 KB)
constexpr int STAGE_H = 2 * TILE_H;            // K tile + V tile
constexpr int DMA_PER_STAGE = 8;
constexpr int REC_F = DecShape<D>::REC_F;      // floats per record
constexpr int KEYS_FEW = 256, KEYS_MIN = 512;  // fewest keys worth a workgroup (see make_split)
constexpr int SLOTS = 512;                     // two workgroups per compute unit are resident
constexpr int MAX_SPLIT = 16;                  // most workgroups per head
static_assert(MAX_SPLIT < MAX_RECORDS, "the flat cut can leave one piece more");
constexpr int MIN_L = 256;                     // shorter caches go to the fp32 kernels (llla_mfma_decode_f32.hip)
constexpr int PRECISE_L = 4 * D;               // sequences up to this length take the two-term weights

typedef short short4v __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) short4v *lds_short4_ptr;

// Records per head that the caller's scratch has room for: one per wave of the largest split, plus the output of a stage that
// merged groups of them (the size that was asked for when every wave left a record; what llla_decode_static accepts follows
// from it).
int record_room(int bh, int L)
{
    const int want = (SLOTS + bh - 1) / bh, most = L / (4 * 8 * STEP);
    const int nparts = 4 * std::min(std::max(std::min(want, most), 1), MAX_SPLIT);
    const int group = nparts >= 64 ? 8 : 6;
    return nparts > 16 ? nparts + (nparts + group - 1) / group : nparts;
}

// Workgroups per head.  A record costs the merge time (one workgroup reads a head's records, 27 KB each), 256 further keys cost a
// workgroup 1.2 us, and two workgroups on a compute unit slow each other down: as many as fill the GPU, with 256 keys or
// more, but 512 or more where there would be more than eight per head or more than one per compute unit; below 1024 keys one,
// which solves the head itself.  us with 256 / 512 keys: 16 heads x 4096 26.8 / 26.3 (1024 keys: 29.3), 32 x 4096 34.0 / 29.0,
// 64 x 2048 31.2 / 27.5, 128 x 1024 30.2 / 27.4; 4 x 2048 21.5 / 21.7, 16 x 1024 20.5 / 22.4; 32 x 600 21.6, one workgroup 21.7.
int make_split(int bh, int L)
{
    const int want = (SLOTS + bh - 1) / bh, room = std::min(MAX_SPLIT, record_room(bh, L));
    int n = std::min(std::min(want, L / KEYS_FEW), room);
    if (n > 8 || n * bh > SLOTS / 2 || L < 2 * KEYS_MIN) n = std::min(n, L / KEYS_MIN);
    return std::max(n, 1);
}

// two bf16 packed in a dword -> two f16 packed (exact for values in the f16 range)
__device__ inline unsigned bf16x2_to_f16x2(unsigned u)
{
    const float lo = __uint_as_float(u << 16), hi = __uint_as_float(u & 0xffff0000u);
    return __builtin_bit_cast(unsigned, __builtin_amdgcn_cvt_pkrtz(lo, hi));
}

template <int N>
__device__ inline void dma_wait_pending() { asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory"); }

// PRECISE (short sequences, chosen per sequence by the kernel): with fewer keys than features only the ridge holds
// some directions, and the 2^-11 rounding of w k is then not small against it.  Such sequences take the weights in
// fp32 and hand w and w k to the matrix cores as an f16 head plus an f16 tail.  Long ones round w to f16 once and
// use that same rounded weight in every moment.
template <bool PRECISE, bool FUSED>
__device__ __forceinline__ void decode_partial_body(unsigned char *smem, const DecPiece &pc, const bf16_t *__restrict__ Kg,
                                                    const bf16_t *__restrict__ Vg, llla_strides sk, llla_strides sv, float cscale,
                                                    const HeadOut &out, float *__restrict__ parts)
{
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64), lane = piece_lane(), g = lane / 16, nn = lane % 16;
    const int bh = pc.bh, b = pc.b, h = pc.h, L = pc.L;
    const bf16_t *qg = static_cast<const bf16_t *>(out.q);
    // the piece is divided over the four waves; rows at and beyond L are never read (a cache tail may hold anything, and
    // 0 * NaN would poison the moments)
    const int part = (int)blockIdx.x * 4 + wave;
    const int keys_per_wave = ((pc.k1 - pc.k0 + 3) / 4 + STEP - 1) / STEP * STEP;
    const int r0 = min(pc.k0 + wave * keys_per_wave, pc.k1);
    const int r1 = min(r0 + keys_per_wave, pc.k1);
    const int nsteps = __builtin_amdgcn_readfirstlane(r1 > r0 ? (r1 - r0 + STEP - 1) / STEP : 0);
    const bf16_t *Kh = Kg + b * sk.batch + h * sk.head;
    const bf16_t *Vh = Vg + b * sv.batch + h * sv.head;
    bf16_t *mystage = reinterpret_cast<bf16_t *>(smem) + wave * NSTAGE * STAGE_H;

    // query fragment, the same for every column of the B operand: lane (g, *) holds q[8g..8g+7], q[32+8g..]
    bf16x8 qf[2];
    qf[0] = *reinterpret_cast<const bf16x8 *>(qg + (size_t)bh * D + 8 * g);
    qf[1] = *reinterpret_cast<const bf16x8 *>(qg + (size_t)bh * D + 32 + 8 * g);

    // ---- per-lane constants.  A natural tile is [key][8 chunks of 8 features]; chunk c of key k is
    //      stored at chunk position c ^ ((k>>1)&7) (the DMA writes whole rows, so no padding).
    int dma_key[4], dma_col[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        const int sl = 64 * t + lane;
        dma_key[t] = sl >> 3;
        dma_col[t] = ((sl & 7) ^ ((dma_key[t] >> 1) & 7)) * 8;
    }
    // logits operand (natural rows): key 16s + nn, feature chunks g and 4+g
    const int sw_n = (nn >> 1) & 7;
    const int nat0 = nn * D + ((g ^ sw_n) * 8), nat1 = nn * D + (((4 + g) ^ sw_n) * 8);     // + s*16*D
    // transposed operand through ds_read_b64_tr_b16: inside a 16-lane group, lane j addresses 4 features
    // (16 I + 4 (j%4) ..) of key 4g + j/4; the instruction hands lane i the 4 keys 4g..4g+3 of feature 16 I + i.
    int tr_addr[4];
    {
        const int key = 4 * g + (nn >> 2);
        const int swz = (key >> 1) & 7;
#pragma unroll
        for (int I = 0; I < 4; ++I) {
            const int c = 2 * I + ((nn & 3) >> 1);
            tr_addr[I] = key * D + ((c ^ swz) * 8) + (nn & 1) * 4;                           // + half*16*D
        }
    }

    f32x4 acc[26], muacc[4], yvacc[4];             // tiles: 10 of Sigma~, 16 of G~
#pragma unroll
    for (int t = 0; t < 26; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int t = 0; t < 4; ++t) { muacc[t] = f32x4{0.f, 0.f, 0.f, 0.f}; yvacc[t] = f32x4{0.f, 0.f, 0.f, 0.f}; }
    float om = 0.f, m = -INFINITY;

    // Waves that start together on equally spaced addresses would keep hitting the same memory channels in
    // step; each wave therefore sweeps its share of the keys from a different starting step and wraps around
    // (the moments do not depend on the order of the keys).
    const int rot = nsteps > 0 ? (int)((part * 7u + bh * 13u) % (unsigned)nsteps) : 0;
    auto step_pos = [&](int step) { const int t = step + rot; return t >= nsteps ? t - nsteps : t; };
    // addresses: a scalar base per step (row j0 of the head) plus per-lane byte offsets that never change, so a
    // transfer costs no vector-ALU work; the transfers carry the non-temporal hint (the cache is read once); only a step that reaches past the sequence clamps its rows per lane
    // (to the last valid row: their weights are 0)
    unsigned koff[4], voff[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        koff[t] = 2u * (unsigned)(dma_key[t] * (int)sk.seq + dma_col[t]);
        voff[t] = 2u * (unsigned)(dma_key[t] * (int)sv.seq + dma_col[t]);
    }
    auto issue_dma = [&](int step) {
        // (LDS destinations as byte offsets: a generic pointer costs four scalar instructions per transfer to turn back)
        const unsigned dst = lds_offset(mystage) + 2u * (unsigned)((step % NSTAGE) * STAGE_H);
        const int j0 = r0 + step_pos(step) * STEP;
        if (j0 + STEP <= L) {
            const bf16_t *kb = Kh + (int64_t)j0 * sk.seq, *vb = Vh + (int64_t)j0 * sv.seq;
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                dma16_base_nt_off(kb, koff[t], dst + 2u * (512 * t));
                dma16_base_nt_off(vb, voff[t], dst + 2u * (TILE_H + 512 * t));
            }
        } else {
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const int j = min(j0 + dma_key[t], L - 1);
                dma16_nt_off(Kh + (int64_t)j * sk.seq + dma_col[t], dst + 2u * (512 * t));
                dma16_nt_off(Vh + (int64_t)j * sv.seq + dma_col[t], dst + 2u * (TILE_H + 512 * t));
            }
        }
    };

    // One stage in flight behind the one in use, and none past the last step: a wave with a few steps paid a stage's traffic for it and waited for it in
    // front of the merge (us: 128 heads of 256 to 2048 keys 34.3 -> 32.7, 256 x 700 23.3 -> 22.6, 16 x 1024 18.3 -> 17.9, 64 x 32768 100.7 -> 99.7).
    // (Four stages where a workgroup has a compute unit to itself: 16 x 4096 25.5 instead of 23.7, 256 x 700 26.3.)
    static_assert(NSTAGE == 2, "the waits count one stage");
    if (nsteps > 0) issue_dma(0);
    for (int s = 0; s < nsteps; ++s) {
        if (s + 1 < nsteps) {
            issue_dma(s + 1);
            dma_wait_pending<DMA_PER_STAGE>();
        } else {
            dma_wait_pending<0>();
        }
        const bf16_t *kt = mystage + (s % NSTAGE) * STAGE_H;
        const bf16_t *vt = kt + TILE_H;
        const int j0 = r0 + step_pos(s) * STEP;

        // logits of the 32 keys: lane (g, *) gets keys 4g..4g+3 (sub-tile 0) and 16+4g.. (sub-tile 1)
        float tl[8];
#pragma unroll
        for (int sub = 0; sub < 2; ++sub) {
            const bf16x8 k0 = *reinterpret_cast<const bf16x8 *>(kt + sub * 16 * D + nat0);
            const bf16x8 k1 = *reinterpret_cast<const bf16x8 *>(kt + sub * 16 * D + nat1);
            f32x4 z = {0.f, 0.f, 0.f, 0.f};
            z = mfma_bf16(k0, qf[0], z);
            z = mfma_bf16(k1, qf[1], z);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int j = j0 + 16 * sub + 4 * g + r;
                tl[4 * sub + r] = (j < r1) ? z[r] * cscale : -INFINITY;
            }
        }
        // running maximum over the wave's keys; the accumulators are rescaled only when it moves
        // (all 16 lanes of a row hold the same 8 logits; the maximum over the four rows goes through two row
        // broadcasts of the data-parallel primitives, without LDS round trips, and is read from the last row)
        float mx = fmaxf(fmaxf(fmaxf(tl[0], tl[1]), fmaxf(tl[2], tl[3])), fmaxf(fmaxf(tl[4], tl[5]), fmaxf(tl[6], tl[7])));
        mx = fmaxf(mx, rows_1_3_from_rows_0_2(mx));
        mx = fmaxf(mx, rows_2_3_from_row_1(mx));
        mx = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, mx), 63));
        if (mx > m) {      // both are wave-uniform
            const float alpha = (m == -INFINITY) ? 0.f : __builtin_amdgcn_exp2f(m - mx);
            m = mx;
            om *= alpha;
#pragma unroll
            for (int t = 0; t < 26; ++t) acc[t] *= alpha;
#pragma unroll
            for (int t = 0; t < 4; ++t) { muacc[t] *= alpha; yvacc[t] *= alpha; }
        }
        float wf[8];
        half8 wq, wl;
#pragma unroll
        for (int t = 0; t < 8; ++t) {
            wf[t] = __builtin_amdgcn_exp2f(tl[t] - m);                // exp2(-inf) = 0 masks the tail
            wq[t] = (_Float16)wf[t];
            if (PRECISE) {
                wl[t] = (_Float16)(wf[t] - (float)wq[t]);
                om += wf[t];
            } else {
                om += (float)wq[t];                                   // omega sums the weights as the MFMAs see them
            }
        }

        // transposed K and V fragments (bf16 -> f16, exact): slot t < 4 = key 4g+t, t >= 4 = key 16+4g+t-4
        half8 kf[4], vf[4];
#pragma unroll
        for (int I = 0; I < 4; ++I) {
            const short4v ka = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4_ptr)(kt + tr_addr[I]));
            const short4v kb = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4_ptr)(kt + 16 * D + tr_addr[I]));
            const short4v va = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4_ptr)(vt + tr_addr[I]));
            const short4v vb = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4_ptr)(vt + 16 * D + tr_addr[I]));
            const uint2 kau = __builtin_bit_cast(uint2, ka), kbu = __builtin_bit_cast(uint2, kb);
            const uint2 vau = __builtin_bit_cast(uint2, va), vbu = __builtin_bit_cast(uint2, vb);
            const uint4 kp = make_uint4(bf16x2_to_f16x2(kau.x), bf16x2_to_f16x2(kau.y), bf16x2_to_f16x2(kbu.x),
                                        bf16x2_to_f16x2(kbu.y));
            const uint4 vp = make_uint4(bf16x2_to_f16x2(vau.x), bf16x2_to_f16x2(vau.y), bf16x2_to_f16x2(vbu.x),
                                        bf16x2_to_f16x2(vbu.y));
            kf[I] = __builtin_bit_cast(half8, kp);
            vf[I] = __builtin_bit_cast(half8, vp);
        }
        auto row_mfmas = [&](int I, const half8 &af) {
#pragma unroll
            for (int J = 0; J < 4; ++J)
                if (J >= I) acc[tix(I, J)] = mfma_f16(af, kf[J], acc[tix(I, J)]);
#pragma unroll
            for (int J = 0; J < 4; ++J) acc[10 + 4 * I + J] = mfma_f16(af, vf[J], acc[10 + 4 * I + J]);
        };
        auto bcast_mfmas = [&](const half8 &wv) {
#pragma unroll
            for (int J = 0; J < 4; ++J) {
                muacc[J] = mfma_f16(wv, kf[J], muacc[J]);       // every row of the tile = mu~[16J + nn]
                yvacc[J] = mfma_f16(wv, vf[J], yvacc[J]);       // every row = (sum w v)[16J + nn]
            }
        };
        if (!PRECISE) {
#pragma unroll
            for (int I = 0; I < 4; ++I) row_mfmas(I, kf[I] * wq);
            bcast_mfmas(wq);
        } else {
            // w k in fp32 (exact up to the rounding of w), handed to the matrix cores as an f16 head plus an f16 tail
#pragma unroll
            for (int I = 0; I < 4; ++I) {
                half8 ah, al;
#pragma unroll
                for (int t = 0; t < 8; ++t) {
                    const float pr = (float)kf[I][t] * wf[t];
                    ah[t] = (_Float16)pr;
                    al[t] = (_Float16)(pr - (float)ah[t]);
                }
                row_mfmas(I, ah);
                row_mfmas(I, al);
            }
            bcast_mfmas(wq);
            bcast_mfmas(wl);
        }
    }

    om = rows_allsum(om);
    float mu[4], yv[4];
#pragma unroll
    for (int J = 0; J < 4; ++J) { mu[J] = muacc[J][0]; yv[J] = yvacc[J][0]; }
    __syncthreads();                                        // the stages of all waves are dead; the merge reuses their LDS
    finish_workgroup<D, bf16_t, false, FUSED, 2>(*reinterpret_cast<HeadLds<D, 2, 4> *>(smem), acc, mu, yv, om, m, m,
                                                 parts + (size_t)pc.rec * REC_F, out, bh, wave, lane);
}

template <bool FUSED>
__global__ __launch_bounds__(NT, 2) void decode_partial_kernel(DecSplit split, HeadOut out, const bf16_t *__restrict__ Kg,
                                                               const bf16_t *__restrict__ Vg, llla_strides sk,
                                                               llla_strides sv, float cscale, float *__restrict__ parts)
{
    static_assert(sizeof(HeadLds<D, 2, 4>) <= 4 * NSTAGE * STAGE_H * sizeof(bf16_t), "the merge reuses the stages");
    __shared__ __align__(16) unsigned char smem[4 * NSTAGE * STAGE_H * sizeof(bf16_t)];     // 4 waves x NSTAGE stages x 8 KB
    for_pieces<FUSED>(split, [&](const DecPiece &pc) {
        if (__builtin_amdgcn_readfirstlane(pc.L <= PRECISE_L ? 1 : 0))
            decode_partial_body<true, FUSED>(smem, pc, Kg, Vg, sk, sv, cscale, out, parts);
        else
            decode_partial_body<false, FUSED>(smem, pc, Kg, Vg, sk, sv, cscale, out, parts);
    });
}

}  // namespace

bool mfma_decode_supported(int d, llla_dtype in) { return (d == D || d == 128) && in == LLLA_BF16; }

size_t mfma_decode_workspace_bytes(int B, int H, int L_max, int d, llla_dtype in)
{
    if (!mfma_decode_supported(d, in) || L_max < MIN_L) return 0;
    if (d == 128) return mfma_decode128_workspace_bytes(B, H, L_max);
    return round_up((size_t)B * H * record_room(B * H, L_max) * REC_F * sizeof(float), 256);
}

size_t mfma_decode_wanted_bytes(int B, int H, int L_max, int d, llla_dtype in)
{
    const size_t need = mfma_decode_workspace_bytes(B, H, L_max, d, in);
    return need && d == 128 ? std::max(need, mfma_decode128_flat_bytes(B, H, L_max)) : need;
}

bool mfma_decode_takes(const Problem &p)
{
    // per-lane byte offsets inside one 32-key step are kept in 32 bits
    const int64_t reach = 2 * 32 * (p.sk.seq > p.sv.seq ? p.sk.seq : p.sv.seq);
    // (batch, head) is the y dimension of the grid
    return p.n >= MIN_L && reach < (int64_t(1) << 31) && (int64_t)p.B * p.H <= 65535;
}

hipError_t mfma_decode(const Problem &p)
{
    if (p.d == 128) return mfma_decode128(p);
    const DecSplit split = choose_split(p, make_split(p.B * p.H, p.n), (size_t)p.B * p.H * record_room(p.B * p.H, p.n), SLOTS, 4 * STEP,
                                        KEYS_MIN, MAX_SPLIT);
    const HeadOut out{p.Q, p.O, p.out == LLLA_BF16 ? 1 : 0, p.lambda};
    float *parts = static_cast<float *>(p.ws);
    const float cscale = p.scale * LOG2E;
    const dim3 grid = split.slots ? dim3(split.slots, p.H) : dim3(split.nsplit, p.B * p.H);
    stage_mark(p.stream, "decode_partial");
    if (split.nsplit == 1 && split.slots == 0) {
        hipLaunchKernelGGL((decode_partial_kernel<true>), grid, dim3(NT), 0, p.stream, split, out, (const bf16_t *)p.K,
                           (const bf16_t *)p.V, p.sk, p.sv, cscale, parts);
    } else {
        hipLaunchKernelGGL((decode_partial_kernel<false>), grid, dim3(NT), 0, p.stream, split, out, (const bf16_t *)p.K,
                           (const bf16_t *)p.V, p.sk, p.sv, cscale, parts);
        stage_mark(p.stream, "decode_merge");
        hipLaunchKernelGGL((decode_merge_kernel<D, bf16_t, false>), dim3(p.B * p.H), dim3(NT), 0, p.stream, split, out, (const float *)parts, dual::DualArgs{}, 0);
    }
    return hipGetLastError();
}

}  // namespace llla
