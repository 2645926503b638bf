// Measurement aid: the projection on a prepared layer with its tile form given instead of chosen (kv_gemm_forms.h), so that
// the choice can be compared with all of them.  Linked against the product library, whose kernels it launches.
#include "../csrc/hk_internal.h"
#include "../csrc/kv_gemm_forms.h"

extern "C" int hkprobe_tile_form_count(void) { return hk::forms::kCount; }

// The form the library takes, and the tile of form i.
extern "C" int hkprobe_tile_form_pick(int64_t M, int32_t d, int32_t cus) { return hk::forms::pick(M, d, cus); }
extern "C" int hkprobe_tile_form_tile(int32_t i, int32_t *bm, int32_t *bn)
{
    if (i < 0 || i >= hk::forms::kCount || !bm || !bn) return -2;
    *bm = hk::forms::kForms[i].bm;
    *bn = hk::forms::kForms[i].bn;
    return 0;
}

// Row statistics and projection of act [M, d] into K, V [1, n_heads, M, d / n_heads] on a layer that hk_prepare_layer
// filled; stats: scratch of M float2.  Enqueues on `stream`.  0, or -2 for sizes, -7 for a launch that failed.
extern "C" int hkprobe_tile_form_run(int32_t form, const void *act, int64_t M, int32_t d, int32_t n_heads, int32_t dtype,
                                     const void *prepared, void *stats, void *K, void *V, void *stream)
{
    if (M <= 0 || M > (1 << 24) || d < 128 || n_heads <= 0 || d % n_heads != 0 || d % 64 != 0) return -2;
    if (!act || !prepared || !stats || !K || !V) return -2;
    auto up = [](size_t n) { return (n + 255) / 256 * 256; };
    const char *p = static_cast<const char *>(prepared);
    hk::KvGemmArgs a = {};
    a.act = act;
    a.stats = static_cast<const float2 *>(stats);
    a.Wp = p;
    a.cvec = reinterpret_cast<const float *>(p + up((size_t)4 * d * d));
    a.bvec = a.cvec + up((size_t)8 * d) / 4;
    a.K_out = K;
    a.V_out = V;
    a.M = M;
    a.d = d;
    a.n_heads = n_heads;
    a.head_dim = d / n_heads;
    a.L_act = (int)M;
    a.L_cap = (int)M;
    a.dtype = dtype;
    hipStream_t s = static_cast<hipStream_t>(stream);
    if (hk::launch_ln_stats(act, static_cast<float2 *>(stats), M, d, 1e-5f, a.bvec + 2 * d, s, dtype) != hipSuccess) return -7;
    return hk::launch_kv_gemm_form(a, form, s) == hipSuccess ? 0 : -7;
}
