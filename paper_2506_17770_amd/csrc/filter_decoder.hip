// filter_decoder.hip -- decoder-path filter for the bilinear filter, the
// multi-layer launch and raw decoder evaluation (tile logic in
// filter_decoder.h; the bicubic instantiations are compiled in
// filter_decoder_cubic.hip).
#include "filter_decoder.h"

hipError_t ctf_internal_decoder_filter_cubic(const ctf_texture_s* t, const ctf::FilterArgs& a, hipStream_t s);
hipError_t ctf_internal_filter_layers_cubic(const ctf::dec::LayerSet& LS, int precision, const ctf::FilterArgs& a,
                                            hipStream_t s);

namespace ctf {

namespace {

using namespace dec;

// rgba[i] = decoder(xy[i]): 32 texels per pass (two MFMA tiles), persistent
// waves; the same per-row instruction sequence as the filter's decode.  The
// waves of a workgroup draw passes from an LDS counter (see TileQueue); the
// coordinates are read two passes ahead and the latents one pass ahead (an
// index past n reads texel n - 1).
template <int P>
__global__ __launch_bounds__(64 * kDecWavesMax) void k_decoder_eval(DevDecoderWeights D, const int2* __restrict__ xy,
                                                                    int64_t n, float4* __restrict__ out)
{
    const int lane = lane_id();
    const int j = lane & 15, g = lane >> 4;
    int* const queue = reinterpret_cast<int*>(dec_lds);
    queue_init(queue, 1);
    FwdWeights<P> W;
    W.load(D.w, lane);
    Biases Bz;
    Bz.load(D.bias, lane);
    const InferLane<P> K(D.grid, g >= 2);
    const int64_t last = n - 1;
    auto draw = [&]() -> int {
        int i = 0;
        if (lane == 0) i = __hip_atomic_fetch_add(queue, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        return i;
    };
    // first row of a drawn pass, and the coordinates this lane reads for it
    auto first_row = [&](int drawn) -> int64_t {
        return ((int64_t)__builtin_amdgcn_readfirstlane(drawn) * gridDim.x + blockIdx.x) * 32;
    };
    auto coord = [&](int64_t r) -> int2 {
        const int64_t f = r + (lane & 31);
        return xy[f < last ? f : last];
    };
    int64_t r0 = first_row(wave_in_block()), r1 = first_row(draw());
    int ahead = draw();
    int2 p = coord(r0);
    InferFetch F;
    infer_fetch<P>(D.grid, K, p.x, p.y, F);
    p = coord(r1);
    while (r0 < n) {
        u16x4 xa, xb;
        infer_combine<P>(F, K, xa, xb);
        infer_fetch<P>(D.grid, K, p.x, p.y, F);
        const int64_t r2 = first_row(ahead);
        ahead = draw();
        p = coord(r2);
        const f4 ya = mlp_forward_b<P>(W, Bz, xa, nullptr, nullptr);
        const f4 yb = mlp_forward_b<P>(W, Bz, xb, nullptr, nullptr);
        if (g == 0 && r0 + j < n) out[r0 + j] = make_float4(ya[0], ya[1], ya[2], ya[3]);
        if (g == 0 && r0 + 16 + j < n) out[r0 + 16 + j] = make_float4(yb[0], yb[1], yb[2], yb[3]);
        r0 = r1;
        r1 = r2;
    }
}

}  // namespace

}  // namespace ctf

using namespace ctf;
using namespace ctf::dec;

hipError_t ctf_internal_decoder_filter(const ctf_texture_s* t, const FilterArgs& a, hipStream_t s)
{
    if (a.filter != CTF_FILTER_BILINEAR) return ctf_internal_decoder_filter_cubic(t, a, s);
    const DevDecoderWeights& d = t->dec;
    return t->dec.precision == CTF_BF16 ? launch_dec_p<CTF_BF16, CTF_FILTER_BILINEAR>(a, d, s)
                                        : launch_dec_p<CTF_FP16, CTF_FILTER_BILINEAR>(a, d, s);
}

hipError_t ctf_internal_filter_layers(const ctf_texture_s* const* texs, const float* xforms, int n,
                                      const FilterArgs& a, hipStream_t s)
{
    if (n < 1 || n > kMaxLayers) return hipErrorInvalidValue;
    LayerSet LS;
    LS.n = n;
    const int prec = texs[0]->dec.precision;
    for (int l = 0; l < n; ++l) {
        if (texs[l]->dev.kind != CTF_TEX_DECODER || texs[l]->dec.precision != prec) return hipErrorInvalidValue;
        LS.dec[l] = texs[l]->dec;
        for (int k = 0; k < 4; ++k) LS.xf[l][k] = xforms[4 * l + k];
    }
    if (a.filter != CTF_FILTER_BILINEAR) return ctf_internal_filter_layers_cubic(LS, prec, a, s);
    return prec == CTF_BF16 ? launch_layers_p<CTF_BF16, CTF_FILTER_BILINEAR>(a, LS, s)
                            : launch_layers_p<CTF_FP16, CTF_FILTER_BILINEAR>(a, LS, s);
}

hipError_t ctf_internal_decoder_eval(const ctf_texture_s* t, const int32_t* xy, int64_t n, float* out,
                                     hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    const DevDecoderWeights& d = t->dec;
    // three waves per SIMD
    const int64_t cus = t->ctx->cus, passes = (n + 31) / 32;
    const int waves = dec_waves(passes, cus);
    int64_t blocks = (passes + waves - 1) / waves;
    if (blocks > cus * (kDecWavesMax / waves)) blocks = cus * (kDecWavesMax / waves);
    const dim3 block(64 * waves);
    const int2* p = reinterpret_cast<const int2*>(xy);
    float4* o = reinterpret_cast<float4*>(out);
    if (t->dec.precision == CTF_BF16)
        hipLaunchKernelGGL(k_decoder_eval<CTF_BF16>, dim3((unsigned)blocks), block, kQueueBytes, s, d, p, n, o);
    else
        hipLaunchKernelGGL(k_decoder_eval<CTF_FP16>, dim3((unsigned)blocks), block, kQueueBytes, s, d, p, n, o);
    return hipGetLastError();
}
