// Batch plans: many images of uneven sizes and radii in one launch.
//
// The batch is described the way the paper rewrites OP2's kernel for
// PENCIL (Sec. III-A): no arrays of pointers, only arenas plus per-image
// offsets. Every image's outputs are independent iterations (Sec. II-B.3),
// so all images' tiles form one flat list, a workgroup to each.
#include <string.h>

#include <algorithm>
#include <string>
#include <vector>

#include "pf_internal.h"

struct pf_batch_plan {
    int32_t n = 0;
    int64_t npix = 0, nfilt = 0;
    int32_t flags = 0;
    std::vector<int32_t> variant;  // per image
    int64_t ntasks = 0;
    int shape = 0;   // of the tiles (kBatchShapes)
    int used = 3;    // variants in use, which select the kernel
    void *dev = nullptr;  // descriptors and tile list, one allocation
    const pf::BatchImg *imgs = nullptr;
    const pf::BatchTask *tasks = nullptr;
};

namespace pf {

// Validates a batch description (sizes, radii, kinds, arena ranges, no two
// images overlapping) and builds the plan's host tables: the image
// descriptors with their variant, and the flat list of tiles.
pf_status build_plan_tables(int32_t n, const int32_t *h, const int32_t *w, const int32_t *r, const int32_t *kind,
                            const int64_t *pix_off, const int64_t *filt_off, int64_t npix, int64_t nfilt,
                            int32_t flags, PlanTables *t) {
    if (n < 1) return fail(PF_EINVAL, "batch needs at least one image");
    if (!h || !w || !r || !kind || !pix_off || !filt_off) return fail(PF_EINVAL, "null descriptor array");
    if (npix < 1 || nfilt < 1) return fail(PF_EINVAL, "arena sizes must be >= 1");
    if (flags & ~(PF_FLAG_EXACT | PF_BATCH_GRAPH | PF_BATCH_NO_TUNE)) return fail(PF_EINVAL, "unknown flags");

    std::vector<std::pair<int64_t, int64_t>> spans;
    spans.reserve(n);
    for (int i = 0; i < n; ++i) {
        const std::string at = " (image " + std::to_string(i) + ")";
        if (h[i] < 1 || w[i] < 1) return fail(PF_EINVAL, "image sizes must be >= 1" + at);
        if (r[i] < 0 || r[i] > PF_R_MAX) return fail(PF_EINVAL, "radius outside 0.." + std::to_string(PF_R_MAX) + at);
        if (r[i] > PF_BATCH_R_MAX)
            return fail(PF_EUNSUPPORTED,
                        "batches take radii 0.." + std::to_string(PF_BATCH_R_MAX) + " (larger: single-image calls)" + at);
        if (kind[i] != PF_KIND_2D && kind[i] != PF_KIND_SEP) return fail(PF_EINVAL, "unknown filter kind" + at);
        const int64_t px = (int64_t)h[i] * w[i];
        const int64_t k = 2 * r[i] + 1;
        const int64_t nf = kind[i] == PF_KIND_2D ? k * k : 2 * k;
        if (pix_off[i] < 0 || pix_off[i] > npix - px) return fail(PF_EINVAL, "image outside the pixel arena" + at);
        if (filt_off[i] < 0 || filt_off[i] > nfilt - nf) return fail(PF_EINVAL, "filter outside the filter arena" + at);
        spans.push_back({pix_off[i], px});
    }
    // Outputs of distinct images must not overlap (restrict, Sec. II-B.1).
    std::sort(spans.begin(), spans.end());
    for (int i = 1; i < n; ++i)
        if (spans[i - 1].first + spans[i - 1].second > spans[i].first)
            return fail(PF_EALIAS, "two images overlap in the pixel arena");

    t->variant.resize(n);
    t->imgs.resize(n);
    for (int i = 0; i < n; ++i) {
        const int var = kind[i] == PF_KIND_2D ? PF_VAR_DIRECT : PF_VAR_SEPARABLE;
        t->variant[i] = var;
        t->used |= 1 << var;
        BatchImg &d = t->imgs[i];
        d.in_off = pix_off[i];
        d.out_off = pix_off[i];
        d.filt_off = filt_off[i];
        d.h = h[i];
        d.w = w[i];
        d.r = r[i];
        d.var = var;
    }
    int64_t ntiles = 0;
    t->shape = batch_shape(t->imgs, &ntiles);
    if (ntiles > INT32_MAX) return fail(PF_EUNSUPPORTED, "batch has more than 2^31-1 tiles");
    t->tasks.reserve((size_t)ntiles);
    for (int i = 0; i < n; ++i) append_tiles(t->tasks, i, t->imgs[i]);
    return PF_OK;
}

// Replays, on the host, where every tile of the tables reads and writes, with
// the geometry functions the FP32 tile kernel itself calls (tile_inside,
// tile_load_col): each tile must name a valid image and lie in it; the staged
// rows and columns of a tile that loads without clamping must lie in the
// image, each 16-byte load of one at the edge inside its row; and the image
// must lie inside the pixel arena. Clamped rows, loads of single clamped
// columns and the stores, guarded per column and row, stay in bounds by
// construction. Returns the number of violations; the first is described in
// *first.
int64_t check_plan_tables(const PlanTables &t, int64_t npix, std::string *first) {
    int64_t bad = 0;
    auto report = [&](size_t k, const std::string &what) {
        if (!bad++) *first = "tile " + std::to_string(k) + ": " + what;
    };
    for (const BatchImg &d : t.imgs)
        if (d.in_off < 0 || d.in_off + (int64_t)d.h * d.w > npix || d.out_off < 0 ||
            d.out_off + (int64_t)d.h * d.w > npix)
            report(0, "image outside the arena");
    const BatchShape sh = kBatchShapes[t.shape];
    for (size_t k = 0; k < t.tasks.size(); ++k) {
        const BatchTask tk = t.tasks[k];
        if (tk.img < 0 || tk.img >= (int)t.imgs.size()) {
            report(k, "image index out of range");
            continue;
        }
        const BatchImg &d = t.imgs[tk.img];
        if (tk.tile < 0 || tk.tile >= (int64_t)d.tiles_x * d.tiles_y) {
            report(k, "tile number out of range");
            continue;
        }
        const int ty = tk.tile / d.tiles_x, tx = tk.tile - ty * d.tiles_x;
        const int x0 = tx * sh.w, y0 = ty * sh.h, pad = tile_pad(d.r);
        if (x0 < 0 || x0 >= d.w || y0 < 0 || y0 >= d.h) {
            report(k, "tile origin outside the image");
            continue;
        }
        if (tile_inside(d.r, sh.w, sh.h, x0, y0, d.h, d.w)) {
            if (x0 - pad < 0 || x0 + sh.w + pad > d.w || y0 - d.r < 0 || y0 + sh.h + d.r > d.h)
                report(k, "unclamped load outside the image");
            continue;
        }
        if (d.w < 4) continue;
        for (int c = -pad; c < sh.w + pad; c += 4) {
            const int at = x0 + tile_load_col(c, x0, d.w);
            if (at < 0 || at + 4 > d.w) report(k, "16-byte load outside the row (column " + std::to_string(x0 + c) + ")");
        }
    }
    return bad;
}

}  // namespace pf

using namespace pf;

extern "C" {

pf_status pf_batch_plan_create(int32_t n, const int32_t *__restrict h, const int32_t *__restrict w,
                               const int32_t *__restrict r, const int32_t *__restrict kind,
                               const int64_t *__restrict pix_off, const int64_t *__restrict filt_off, int64_t npix,
                               int64_t nfilt, int32_t flags, pf_batch_plan **const __restrict plan) {
    clear_error();
    if (!plan) return fail(PF_EINVAL, "null plan out-parameter");
    *plan = nullptr;
    PlanTables t;
    pf_status st = build_plan_tables(n, h, w, r, kind, pix_off, filt_off, npix, nfilt, flags, &t);
    if (st) return st;

    pf_batch_plan *p = new (std::nothrow) pf_batch_plan;
    if (!p) return fail(PF_ENOMEM, "plan allocation");
    p->n = n;
    p->npix = npix;
    p->nfilt = nfilt;
    p->flags = flags;
    p->variant = t.variant;
    p->ntasks = (int64_t)t.tasks.size();
    p->shape = t.shape;
    p->used = t.used;
    const size_t bi = (t.imgs.size() * sizeof(BatchImg) + 255) & ~(size_t)255;
    const size_t bytes = bi + t.tasks.size() * sizeof(BatchTask);
    hipError_t e = hipMalloc(&p->dev, bytes);
    if (e != hipSuccess) {
        delete p;
        return fail_hip(e, "plan descriptor allocation");
    }
    std::vector<char> host(bytes, 0);
    memcpy(host.data(), t.imgs.data(), t.imgs.size() * sizeof(BatchImg));
    memcpy(host.data() + bi, t.tasks.data(), t.tasks.size() * sizeof(BatchTask));
    p->imgs = (const BatchImg *)p->dev;
    p->tasks = (const BatchTask *)((char *)p->dev + bi);
    e = hipMemcpy(p->dev, host.data(), host.size(), hipMemcpyHostToDevice);
    if (e != hipSuccess) {
        (void)hipFree(p->dev);
        delete p;
        return fail_hip(e, "plan descriptor upload");
    }
    *plan = p;
    return PF_OK;
}

pf_status pf_batch_plan_check(int32_t n, const int32_t *__restrict h, const int32_t *__restrict w,
                              const int32_t *__restrict r, const int32_t *__restrict kind,
                              const int64_t *__restrict pix_off, const int64_t *__restrict filt_off, int64_t npix,
                              int64_t nfilt, int32_t flags, int64_t *const __restrict tiles,
                              int64_t *const __restrict violations) {
    clear_error();
    if (!tiles || !violations) return fail(PF_EINVAL, "null out-parameter");
    *tiles = *violations = 0;
    PlanTables t;
    pf_status st = build_plan_tables(n, h, w, r, kind, pix_off, filt_off, npix, nfilt, flags, &t);
    if (st) return st;
    std::string first;
    *tiles = (int64_t)t.tasks.size();
    *violations = check_plan_tables(t, npix, &first);
    if (*violations) return fail(PF_EINVAL, first);
    return PF_OK;
}

pf_status pf_batch_plan_run(pf_batch_plan *p, int64_t npix, int64_t nfilt, const float *__restrict in,
                            const float *__restrict filt, float *__restrict out, void *stream) {
    clear_error();
    if (!p) return fail(PF_EINVAL, "null plan");
    if (npix != p->npix || nfilt != p->nfilt) return fail(PF_EINVAL, "arena sizes differ from the plan's");
    if (!in || !filt || !out) return fail(PF_EINVAL, "null arena pointer");
    if (((uintptr_t)in | (uintptr_t)filt | (uintptr_t)out) % 4) return fail(PF_EINVAL, "arenas must be 4-byte aligned");
    const uintptr_t i0 = (uintptr_t)in, b = (uintptr_t)out, nb = (uintptr_t)npix * 4;
    if (i0 < b + nb && b < i0 + nb) return fail(PF_EALIAS, "input and output arenas overlap (restrict)");
    const uintptr_t f = (uintptr_t)filt, fb = (uintptr_t)nfilt * 4;
    if (f < b + nb && b < f + fb) return fail(PF_EALIAS, "filter and output arenas overlap (restrict)");
    hipError_t e = launch_batch((p->flags & PF_FLAG_EXACT) != 0, p->used, p->shape, p->imgs, p->tasks, p->ntasks, in,
                                filt, out, (hipStream_t)stream);
    if (e != hipSuccess) return fail_hip(e, "batch launch");
    return PF_OK;
}

pf_status pf_batch_plan_variants(const pf_batch_plan *p, int32_t n, int32_t *__restrict variant) {
    clear_error();
    if (!p || !variant) return fail(PF_EINVAL, "null argument");
    if (n != p->n) return fail(PF_EINVAL, "n differs from the plan's image count");
    for (int i = 0; i < n; ++i) variant[i] = p->variant[i];
    return PF_OK;
}

pf_status pf_batch_plan_info(const pf_batch_plan *p, int64_t *const __restrict tasks, int32_t *const __restrict launches,
                             int32_t *const __restrict grid) {
    clear_error();
    if (!p || !tasks || !launches || !grid) return fail(PF_EINVAL, "null argument");
    *tasks = p->ntasks;
    *launches = 1;
    const dim3 g = batch_grid(p->ntasks);
    *grid = (int32_t)(g.x * g.y);
    return PF_OK;
}

pf_status pf_batch_plan_destroy(pf_batch_plan *p) {
    clear_error();
    if (!p) return PF_OK;
    if (p->dev) (void)hipFree(p->dev);
    delete p;
    return PF_OK;
}

}  // extern "C"
