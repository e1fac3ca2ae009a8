// Configurations, the Table 1 resource model and the lite-space builder of
// the paper's device-guided space building (Sec. 5.2), on one CDNA4 CU.
// Host-only: no HIP runtime calls.
#include "space.h"

#include <algorithm>
#include <climits>
#include <cmath>
#include <cstdio>
#include <cstring>

namespace nnjit {

// The variant tables, in configuration order.
struct VariantTable {
    const Variant *v;
    int n;
};
static const VariantTable *variant_tables(int *count) {
    static const VariantTable t[] = {{kGemmF32Variants, kNumGemmF32Variants},
                                     {kGemmF32sVariants, kNumGemmF32sVariants},
                                     {kGemmF32rVariants, kNumGemmF32rVariants},
                                     {kGemmF16Variants, kNumGemmF16Variants},
                                     {kGemmF16sVariants, kNumGemmF16sVariants},
                                     {kGemmF16rVariants, kNumGemmF16rVariants},
                                     {kGemvVariants, kNumGemvVariants},
                                     {kGemvQ4Variants, kNumGemvQ4Variants}};
    *count = (int)(sizeof(t) / sizeof(t[0]));
    return t;
}

static const Variant *variant_at(int gi) {
    int n = 0;
    const VariantTable *t = variant_tables(&n);
    for (int i = 0; i < n; ++i) {
        if (gi < t[i].n) return &t[i].v[gi];
        gi -= t[i].n;
    }
    return nullptr;
}

int total_variants() {
    int n = 0, total = 0;
    const VariantTable *t = variant_tables(&n);
    for (int i = 0; i < n; ++i) total += t[i].n;
    return total;
}

int variant_index(const Variant *v) {
    int n = 0, base = 0;
    const VariantTable *t = variant_tables(&n);
    for (int i = 0; i < n; ++i) {
        if (v >= t[i].v && v < t[i].v + t[i].n) return base + (int)(v - t[i].v);
        base += t[i].n;
    }
    return -1;
}

const std::vector<int> &gemm_splits() {
    static const std::vector<int> s = {1, 2, 4, 8, 16};
    return s;
}
const std::vector<int> &gemv_splits() {
    static const std::vector<int> s = {1, 2, 4, 8, 16, 32, 64, 128};
    return s;
}

int family_dtype(int family) {
    return (family == FAM_GEMM_F16 || family == FAM_GEMV_F16 || family == FAM_GEMV_Q4) ? NNJIT_F16 : NNJIT_F32;
}
bool family_is_gemv(int family) { return family == FAM_GEMV_F32 || family == FAM_GEMV_F16; }
bool family_is_q4(int family) { return family == FAM_GEMV_Q4; }
int family_of(int kind, int dtype) {
    if (kind == NNJIT_KIND_GEMV_Q4) return FAM_GEMV_Q4;
    if (kind == NNJIT_KIND_GEMV) return dtype == NNJIT_F16 ? FAM_GEMV_F16 : FAM_GEMV_F32;
    return dtype == NNJIT_F16 ? FAM_GEMM_F16 : FAM_GEMM_F32;
}
const char *family_name(int family) {
    switch (family) {
    case FAM_GEMM_F32: return "gemm_f32";
    case FAM_GEMM_F16: return "gemm_f16";
    case FAM_GEMV_F32: return "gemv_f32";
    case FAM_GEMV_F16: return "gemv_f16";
    case FAM_GEMV_Q4: return "gemv_q4";
    default: return "?";
    }
}

const std::vector<Config> &configs() {
    static const std::vector<Config> all = [] {
        std::vector<Config> out;
        const int nv = total_variants();
        for (int gi = 0; gi < nv; ++gi) {
            const Variant *v = variant_at(gi);
            static const std::vector<int> no_split = {1};
            const std::vector<int> &splits =
                family_is_q4(v->family) ? no_split : family_is_gemv(v->family) ? gemv_splits() : gemm_splits();
            for (int s : splits) out.push_back(Config{(int)out.size(), v, s});
            if (has_stream_k(*v)) out.push_back(Config{(int)out.size(), v, kStreamK});
        }
        return out;
    }();
    return all;
}

nnjit_device_limits mi355x_limits() {
    nnjit_device_limits d;
    d.num_cus = 256;
    d.simds_per_cu = 4;
    d.vgprs_per_lane = 512;
    d.vgpr_granule = 8;
    d.max_waves_per_simd = 8;
    d.wave_size = 64;
    d.lds_per_cu = 163840;
    d.lds_per_wg = 163840;
    d.max_threads_per_wg = 1024;
    return d;
}

// Table 1 of the paper, on one compute unit ("core"):
//   Reg_thread   -> VGPR+AGPR per lane (measured from the compiled kernel, or
//                   the estimate inflated by the relaxation ratio)
//   L1_block     -> LDS bytes of the workgroup (the C tile lives in registers)
//   Thread_block -> workgroup size;  Warp_block -> waves of 64 lanes
//   Block_core   =  min(RegLimit, L1Limit, WarpLimit)
// RegLimit counts whole waves: a SIMD holds floor(512 / regs) waves (regs
// rounded up to the allocation granule), at most max_waves_per_simd.
nnjit_resources resources_of(const Variant &v, const nnjit_device_limits &d, int measured_regs) {
    nnjit_resources r{};
    const int regs = measured_regs >= 0 ? measured_regs : (int)std::ceil(v.est_regs / kRelaxation);
    r.regs_per_lane = regs;
    r.regs_measured = measured_regs >= 0 ? 1 : 0;
    r.lds_per_wg = v.lds_bytes;
    r.threads_per_wg = v.threads;
    r.waves_per_wg = (v.threads + d.wave_size - 1) / d.wave_size;
    const int gran = d.vgpr_granule > 0 ? d.vgpr_granule : 1;
    const int g = ((std::max(regs, 1) + gran - 1) / gran) * gran;
    const int wps = std::min(d.max_waves_per_simd, d.vgprs_per_lane / g);
    r.reg_limit = (d.simds_per_cu * wps) / r.waves_per_wg;
    r.lds_limit = v.lds_bytes > 0 ? (int)std::min<int64_t>(d.lds_per_cu / v.lds_bytes, 1 << 20) : (1 << 20);
    r.wave_limit = (d.simds_per_cu * d.max_waves_per_simd) / r.waves_per_wg;
    r.wg_per_cu = std::min(r.reg_limit, std::min(r.lds_limit, r.wave_limit));
    return r;
}

static int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }
static int64_t pow2ceil(int64_t x) {
    int64_t p = 1;
    while (p < x) p <<= 1;
    return p;
}

bool has_stream_k(const Variant &v) { return v.family == FAM_GEMM_F32 && v.direct_copy == 1 && v.kslices == 1; }

Geometry geometry_of(const Config &c, int64_t batch, int64_t M, int64_t N, int64_t K, int64_t sk_wgs) {
    Geometry g;
    const Variant &v = *c.v;
    g.split = c.split == kStreamK ? 1 : c.split;
    if (c.split == kStreamK && batch == 1 && K > 0 && sk_wgs > 0) {
        g.stream_k = true;
        g.tiles_m = (int)ceil_div(std::max<int64_t>(M, 1), v.mt);
        g.tiles_n = (int)ceil_div(std::max<int64_t>(N, 1), v.nt);
        g.nslab = (int)ceil_div(K, v.kt);
        g.units = (int64_t)g.tiles_m * g.tiles_n * g.nslab;
        g.kchunk = (int)(g.nslab * (int64_t)v.kt);
        g.wgs = std::max<int64_t>(1, std::min<int64_t>(sk_wgs, g.units));
        g.ws_floats = 2 * g.wgs * (int64_t)v.mt * v.nt;
        return g;
    }
    if (family_is_q4(v.family)) {
        // one workgroup per nt output rows, no split (batch carries the group size)
        g.group = std::max<int64_t>(1, batch);
        g.tiles_m = 1;
        g.tiles_n = (int)ceil_div(std::max<int64_t>(N, 1), v.nt);
        g.kchunk = (int)std::max<int64_t>(K, 1);
        g.split = 1;
        g.wgs = g.tiles_n;
        g.ws_floats = 0;
        return g;
    }
    if (!family_is_gemv(v.family)) {
        g.tiles_m = (int)ceil_div(std::max<int64_t>(M, 1), v.mt);
        g.tiles_n = (int)ceil_div(std::max<int64_t>(N, 1), v.wg_cols());
        const int64_t per = ceil_div(std::max<int64_t>(K, 1), g.split);
        g.kchunk = (int)(ceil_div(per, v.kt) * v.kt);
        const int64_t tiles = batch * g.tiles_m * (int64_t)g.tiles_n;
        g.wgs = tiles * g.split;
        g.ws_floats = g.split > 1 ? (int64_t)g.split * batch * std::max<int64_t>(M, 1) * std::max<int64_t>(N, 1) : 0;
    } else {
        g.tiles_m = 1;
        g.tiles_n = (int)ceil_div(std::max<int64_t>(N, 1), v.nt);
        g.kchunk = (int)std::max<int64_t>(1, ceil_div(std::max<int64_t>(K, 1), c.split));
        g.wgs = (int64_t)g.tiles_n * c.split;
        g.ws_floats = c.split > 1 ? (int64_t)c.split * std::max<int64_t>(N, 1) : 0;
    }
    return g;
}

const std::vector<ConsistentSetting> &consistent_settings() {
    static const std::vector<ConsistentSetting> t = {
#include "consistent.inc"
    };
    return t;
}

int primitive_value(const Variant &v, int primitive) {
    switch (primitive) {
    case PRIM_DIRECT: return v.direct_copy;
    case PRIM_LAYOUT: return v.lds_layout;
    case PRIM_UNROLL: return v.rolled;
    case PRIM_STAGES: return v.stages;
    case PRIM_PREFETCH: return v.prefetch;
    case PRIM_KT: return v.kt;
    case PRIM_MFMA: return v.mfma_m;
    case PRIM_VEC: return v.vec_bytes;
    default: return -1;
    }
}

// Do u and v differ in nothing but `primitive` (for the staging primitive:
// the same tile hierarchy, instruction shape and load width)?  The groups
// the offline microbenchmark compares.
static bool same_group(const Variant &u, const Variant &v, int primitive) {
    if (u.family != v.family || u.mfma_m != v.mfma_m || u.mfma_k != v.mfma_k || u.mt != v.mt || u.nt != v.nt ||
        u.kt != v.kt || u.wm != v.wm || u.wn != v.wn || u.vec_bytes != v.vec_bytes)
        return false;
    if (primitive == PRIM_DIRECT) return true;
    for (int q : {PRIM_DIRECT, PRIM_LAYOUT, PRIM_UNROLL, PRIM_STAGES, PRIM_PREFETCH, PRIM_KT, PRIM_MFMA, PRIM_VEC})
        if (q != primitive && primitive_value(u, q) != primitive_value(v, q)) return false;
    return u.kslices == v.kslices && u.wg_cols() == v.wg_cols();
}

// A variant is excluded when a fixed (consistent) setting differs from its
// own and the compiled set holds its twin with the fixed setting: the
// primitive is fixed where the choice exists, not for variants the
// benchmark never compared.
bool follows_consistent(const Variant &v) {
    for (const ConsistentSetting &c : consistent_settings()) {
        if (c.family != v.family) continue;
        // (the settings were measured for the first two kinds of staging only)
        if (v.direct_copy == 2 || !(v.direct_copy ? c.direct_copy : c.reg_staged)) continue;
        if (primitive_value(v, c.primitive) == c.value) continue;
        for (const Config &u : configs())
            if (u.split == 1 && primitive_value(*u.v, c.primitive) == c.value && same_group(*u.v, v, c.primitive))
                return false;
    }
    return true;
}

namespace {
struct Cand {
    int id;
    nnjit_resources r;
    double eff;      // fill of the last wave of workgroups
    int64_t area;    // macro-tile area (GEMM) or columns x rows per pass (GEMV)
    int split;
};
}  // namespace

LiteResult lite_space(const Shape &s, const nnjit_device_limits &d, const std::vector<int> *measured_regs,
                      const std::vector<int> *spills) {
    LiteResult out;
    const int fam = family_of(s.kind, s.dtype);
    const bool gemv = family_is_gemv(fam);
    const bool q4 = family_is_q4(fam);
    const int V = vec_elems(s.dtype);
    const bool vec_ok = q4 ? (s.batch % 32 == 0) : gemv ? (s.N % V == 0) : (s.K % V == 0 && s.N % V == 0);

    // size of the unpruned parameter space over the same axes
    if (q4) {
        out.n_naive = 4 /*rows per wave*/ * 3 /*threads*/ * 3 /*K-slices*/ * 2 /*blocks in flight*/;
    } else if (!gemv) {
        const int64_t kt_choices = fam == FAM_GEMM_F32 ? 2 : 1;
        out.n_naive = 2 /*mfma*/ * 5 /*Mt*/ * 5 /*Nt*/ * kt_choices * 3 /*WM*/ * 3 /*WN*/ * 2 /*stages*/ *
                      (int64_t)gemm_splits().size();
    } else {
        out.n_naive = 3 /*L*/ * 5 /*threads*/ * 4 /*U*/ * (int64_t)gemv_splits().size();
    }

    std::vector<Cand> cands, unfit;  // unfit: pass the resource heuristics, fail the shape fit (split 1 only)
    std::vector<Cand> off_cands, off_unfit;  // the same, with a setting the consistent-primitive table excludes
    for (const Config &c : configs()) {
        const Variant &v = *c.v;
        if (v.family != fam) continue;
        ++out.n_enumerated;
        // single-row kernels serve exactly the products with one row per
        // slice (M = 1), whatever their alignment; vector loads only where
        // the shape allows them
        if (!gemv && !q4 && (v.mt == 1) != (s.M == 1)) continue;
        if (!(v.mt == 1 && !gemv && !q4) && (v.vec_bytes == 16) != vec_ok) continue;
        const bool consistent = follows_consistent(v);
        const int gi = variant_index(&v);
        if (spills && gi < (int)spills->size() && (*spills)[gi]) continue;
        const int mregs = (measured_regs && gi < (int)measured_regs->size()) ? (*measured_regs)[gi] : -1;
        const nnjit_resources r = resources_of(v, d, mregs);
        if (r.threads_per_wg > d.max_threads_per_wg) continue;                // heuristic 5
        if (r.lds_per_wg > d.lds_per_wg) continue;                            // heuristic 6
        if (r.wg_per_cu < 1) continue;

        const int64_t slots = (int64_t)d.num_cus * r.wg_per_cu;
        const Geometry g = geometry_of(c, s.batch, s.M, s.N, s.K, slots);
        Cand cd;
        cd.id = c.id;
        cd.r = r;
        const int64_t waves = ceil_div(std::max<int64_t>(g.wgs, 1), slots);
        cd.eff = (double)g.wgs / (double)(waves * slots);
        cd.area = (int64_t)v.mt * v.wg_cols() * ((gemv || q4) ? v.kt : 1);
        cd.split = c.split;
        bool fit = true;
        if (q4) {
            // no workgroup wider than the (power-of-two rounded) output count;
            // K-slices and blocks in flight only where K has the blocks for them
            if (v.nt > std::max<int64_t>(8, pow2ceil(s.N))) fit = false;
            const int64_t nblk = std::max<int64_t>(1, ceil_div(s.K, v.kt));
            if (v.kslices > 1 && nblk < v.kslices) fit = false;
            if (v.unroll > 1 && ceil_div(nblk, v.kslices) < v.unroll) fit = false;
        } else if (!gemv) {
            // shape fit: no macro tile wider than the (power-of-two rounded) matrix
            if (v.mt > std::max<int64_t>(16, pow2ceil(s.M)) || v.wg_cols() > std::max<int64_t>(16, pow2ceil(s.N))) fit = false;
            const int64_t tiles = s.batch * g.tiles_m * (int64_t)g.tiles_n;
            if (c.split == kStreamK) {
                // stream-K: only where the tiles leave the last wave of
                // workgroups short, with at least four K slabs per workgroup
                if (!g.stream_k || g.units < 4 * g.wgs) continue;
                const int64_t tw = ceil_div(tiles, slots);
                if ((double)tiles / (double)(tw * slots) >= 0.95) continue;
                cd.eff = 1.0;
            }
            // K groups inside a workgroup pay off only while the chip has
            // few workgroups (fewer than two per CU)
            if (v.kslices > 1 && tiles * c.split >= 2LL * d.num_cus) continue;
            if (c.split > 1) {
                // split K only to fill the CUs: keep the smallest power of two
                // that gives every CU a workgroup, and twice that
                if (tiles >= d.num_cus) continue;
                int64_t sfill = 1;
                while (tiles * sfill < d.num_cus) sfill <<= 1;
                // a workgroup with K groups needs half the split for the same waves
                const int64_t lo = v.kslices > 1 ? std::max<int64_t>(1, sfill / 2) : sfill;
                if (c.split < lo || c.split > 2 * sfill) continue;
                // over-split: more than two waves of workgroups, unless they
                // form whole waves (at most four)
                const int64_t wgs = tiles * c.split;
                if (wgs > 2 * slots && !(wgs % slots == 0 && wgs <= 4 * slots)) continue;
                if (s.K < 2LL * c.split * v.kt) continue;    // at least two K slabs per split
            }
        } else {
            if (v.nt > std::max<int64_t>(64, pow2ceil(s.N))) fit = false;
            const int rows_per_pass = v.kt;
            if (c.split > 1) {
                if (g.kchunk < rows_per_pass) continue;  // every split gets at least one pass of rows
                int smax = 1;
                for (int sp : gemv_splits())
                    if (ceil_div(std::max<int64_t>(s.K, 1), sp) >= rows_per_pass) smax = sp;
                // split only to fill the CUs: the smallest power of two that
                // gives every CU a workgroup, and twice that (or the largest
                // split K allows)
                if (g.tiles_n >= d.num_cus) continue;
                int64_t sfill = 1;
                while (g.tiles_n * sfill < d.num_cus) sfill <<= 1;
                if ((c.split < sfill || c.split > 2 * sfill) && c.split != smax) continue;
                if (g.wgs > 4 * slots) continue;                                  // over-split
                if (g.wgs < d.num_cus / 2 && c.split != smax) continue;           // under-filled
                // Little's law: bytes in flight per CU must cover HBM latency
                const int64_t wg_here = std::min<int64_t>(r.wg_per_cu, ceil_div(g.wgs, d.num_cus));
                if (wg_here * v.threads * (int64_t)v.unroll * 16 < 8192 && c.split != smax) continue;
            }
        }
        if (fit) (consistent ? cands : off_cands).push_back(cd);
        else if (c.split == 1) (consistent ? unfit : off_unfit).push_back(cd);
    }
    // settings fixed offline (consistent primitives) prune the rest, unless
    // nothing would be left (e.g. element-load shapes when 16-byte loads are
    // the fixed setting)
    if (cands.empty() && unfit.empty()) {
        cands.swap(off_cands);
        unfit.swap(off_unfit);
    }
    // the shape fit never empties the space: tiny shapes fall back to the
    // unsplit configurations that passed the resource heuristics
    if (cands.empty()) cands = unfit;

    // heuristic 7: keep register-bound candidates (Block_core == RegLimit),
    // relaxed when too few survive.  A direct-copy variant keeps its staging
    // (the slabs in flight, a register term of Table 1 for the others) in
    // LDS, so for it the bound that plays this role is L1Limit; a variant of the
    // third kind keeps planes of halves there besides its staging registers,
    // and either bound does.
    std::vector<Cand> kept;
    for (const Cand &c : cands) {
        const int direct = configs()[c.id].v->direct_copy;
        if (direct == 2 || c.r.wg_per_cu == (direct ? c.r.lds_limit : c.r.reg_limit)) kept.push_back(c);
    }
    if ((int)kept.size() < kMinSurvivors) kept = cands;

    // evaluation order: most workgroups per CU first, then fuller last wave,
    // larger tile, smaller split, lower id -- within each staging kind
    // (registers / LDS direct copies / split products), the orders merged in
    // turn so that the cap below never drops one kind wholesale
    auto before = [](const Cand &a, const Cand &b) {
        if (a.r.wg_per_cu != b.r.wg_per_cu) return a.r.wg_per_cu > b.r.wg_per_cu;
        if (std::fabs(a.eff - b.eff) > 1e-9) return a.eff > b.eff;
        if (a.area != b.area) return a.area > b.area;
        if (a.split != b.split) return a.split < b.split;
        return a.id < b.id;
    };
    std::vector<Cand> by_kind[3];
    for (const Cand &c : kept) by_kind[configs()[c.id].v->direct_copy].push_back(c);
    for (auto &v : by_kind) std::stable_sort(v.begin(), v.end(), before);
    std::vector<Cand> order;
    for (size_t i = 0; i < std::max({by_kind[0].size(), by_kind[1].size(), by_kind[2].size()}); ++i)
        for (auto &v : by_kind)
            if (i < v.size()) order.push_back(v[i]);
    // the lite space is the head of that order: at most kMaxTimed candidates
    // are ever evaluated on the device.  (Third-kind candidates take the place of
    // up to 13 register-staged ones at the end of the order.  Over 49 shapes
    // where that happens, the fastest of those took 1.13 to 2.8 times as long
    // as the fastest of the lite space.)
    for (const Cand &c : order) {
        if ((int)out.ids.size() >= kMaxTimed) break;
        out.ids.push_back(c.id);
    }
    return out;
}

// Configuration id of a variant name and split (-1: not compiled).
static int id_of(const char *name, int split = 1) {
    for (const Config &c : configs())
        if (c.split == split && !std::strcmp(c.v->name, name)) return c.id;
    return -1;
}

// The largest compiled split of `tiles` workgroups that keeps them at most
// `most` and leaves each at least `rows` of the K rows (1: none does).
static int split_within(int64_t tiles, int64_t most, int64_t K, int64_t rows) {
    int best = 1;
    for (int s : gemm_splits())
        if (tiles * s <= most && K >= rows * s) best = s;
    return best;
}

// Single rows (M = 1).  The widest segment whose rows of one slice are all in
// flight at once (8 loads of each of 256 / L row slots), so that neighbouring
// lanes read long runs; a longer sum takes the narrowest segment, for
// workgroups, and 1024 threads once 256 would go round more than about twice.
// fp16, 32 slices: 1023 columns of 128 rows L16 4.4, L32 5.0, L8 5.5; 128
// columns of 1023 rows L4 5.2, with 1024 threads 5.6, and of 2048 rows (64
// slices) 7.3 and 7.1.  fp32: 128 columns of 1023 rows 1024 threads 5.7, 256
// threads above 7.
// fp32 has half the columns per lane and twice the bytes: where the slices and
// segments fill the chip anyway, long runs count for more than workgroups, so
// the segment is the widest of which every CU gets about four (8 slices of 11008
// columns and 1024 rows: L16 62, L8 with 1024 threads 92; 32 of 4096 and 1024:
// L32 92, 118; 256 of 1024 and 512: L64 92, 136), up to eight of the widest
// (512 of 1024 and 256: L8 90, L64 111); and 1024 threads only while there are
// at most two narrow ones per CU (2 of 11008 and 1024: 21.5, 25.1).
// Few segments and a long sum, at least two rounds of 1024 threads: the
// narrowest with 256 threads, split to about four workgroups per CU (fp32, 8
// slices of 128 columns: 4096 rows 9.1, unsplit 14.7; 16384 rows 25 and 77;
// fp16 16384 rows 12 and 31), from 16 tiles of 64 columns on: those shapes
// took scratch before there were row kernels, the smaller ones did not and can
// be captured without a run before.
static int predefined_row(const Shape &s, bool aligned, const nnjit_device_limits &d) {
    static const int f16_id[] = {id_of("gemm_f16r_L4_t256_u8"), id_of("gemm_f16r_L8_t256_u8"),
                                 id_of("gemm_f16r_L16_t256_u8"), id_of("gemm_f16r_L32_t256_u8"),
                                 id_of("gemm_f16r_L4_t1024_u8")};
    static const int f32_id[] = {id_of("gemm_f32r_L8_t256_u8"), id_of("gemm_f32r_L16_t256_u8"),
                                 id_of("gemm_f32r_L32_t256_u8"), id_of("gemm_f32r_L64_t256_u8"),
                                 id_of("gemm_f32r_L8_t1024_u8")};
    const bool f16 = s.dtype == NNJIT_F16;
    const int64_t cus = d.num_cus;
    auto segments = [&](int columns) { return s.batch * ceil_div(s.N, columns); };
    if (aligned && s.K >= (f16 ? 4096 : 2048) && segments(32) <= cus / 2 && segments(64) >= cus / 16)
        return id_of(f16 ? "gemm_f16r_L4_t256_u8" : "gemm_f32r_L8_t256_u8", split_within(segments(32), 4 * cus, s.K, 1));
    if (f16) return f16_id[s.K <= 64 ? 3 : s.K <= 128 ? 2 : s.K <= 256 ? 1 : s.K <= 1024 ? 0 : 4];
    const bool many = segments(256) >= 8 * cus;
    int wide = 0;
    while (!many && wide < 3 && 2 * segments(32 << (wide + 1)) >= 7 * cus) ++wide;
    const int by_sum = s.K <= (many ? 64 : 32) ? 2 : s.K <= 128 ? 1 : 0;
    if (s.K <= 256 || segments(32) > 2 * cus) return f32_id[std::max(wide, by_sum)];
    return f32_id[4];
}

// All lines below from device times of one MI355X (us; the first of the lite
// space, which served before, stands in brackets).
int predefined_config(const Shape &s, bool aligned, const nnjit_device_limits &d) {
    if (s.kind != NNJIT_KIND_GEMM && s.kind != NNJIT_KIND_BATCHED) return -1;
    const bool f16 = s.dtype == NNJIT_F16;
    const int64_t cus = d.num_cus;
    auto tiles = [&](int64_t t) { return s.batch * ceil_div(s.M, t) * ceil_div(s.N, t); };
    if (s.M == 1) return predefined_row(s, aligned, d);
    if (f16) {
        // The staged kernels take any alignment at the same speed.  128 x 128
        // tiles from two per CU on (64 x 1000 x 1000 x 64: 65, 64 x 64 tiles
        // 72 [170]; 32 x 333 x 333 x 128, 288 tiles: 10.9 and 10.5), else 64 x
        // 64 (32 x 336 x 128 x 336: 7.7 [12.7]; 512 x 4096 x 4096: 37 [105];
        // 16 x 80 x 80 x 64: 4.3 [5.9]).  A long sum over few tiles is better
        // off with a split, which the first of the lite space has (128 x 768 x
        // 3072: 18.7 [13.7]; 16 x 4096 x 4096: 25.6 [14.2]).
        static const int big = id_of("gemm_f16s_128x128x32_w2x4_p1_vfalse"), mid = id_of("gemm_f16s_64x64x32_w2x2_p3_vfalse");
        if (aligned && tiles(64) < cus && s.K > 1024) return -1;
        return s.M > 64 && s.N > 64 && tiles(128) >= 2 * cus ? big : mid;
    }
    // fp32: 128 x 128 split-product tiles where each CU gets one (1024 x 4096
    // x 1024: 52, 64 x 64 tiles 64 [101]), 64 x 64 ones likewise (512 x 4096 x
    // 4096: 129, 128 x 128 144 [223]; 32 x 333 x 128 x 333: 15.4 [22.4]).
    static const int big = id_of("gemm_f32s_128x128x16_w2x4_p3_vfalse"), mid = id_of("gemm_f32s_64x64x16_w2x2_p3_vfalse");
    // Up to 16 rows: 16-row tiles, which the lite space begins with, over many
    // columns (8 x 32000 x 4096: 131, 64 x 64 tiles 158; 16 x 11008 x 4096: 41,
    // 32 x 32 tiles 56; 32 x 16 x 1024 x 128: 7.8 and 9.2; not fewer: 16 x 8192 x
    // 1024 15.2 and 10.5), and for long sums that 32 x 32 tiles share over less
    // than seven eighths of the CUs (14 x 2584 x 6320, 162 workgroups: 22.8 and
    // 25.6; 8 x 6976 x 4752, 218: 30.0 and 31.4; 16 x 4096 x 4096, 256: 25.1 and 19.7).
    if (aligned && s.M <= 16) {
        const int64_t t = tiles(32);
        if (t > cus || (t > cus / 4 && s.K >= 2048 && 8 * t * split_within(t, cus, s.K, 256) < 7 * cus)) return -1;
    }
    if (s.M > 64 && s.N > 64 && tiles(128) >= cus) return big;
    if (tiles(64) >= cus) return mid;
    if (aligned) {
        // 32 x 32 tiles with a K slice per wave while they are at most two per
        // CU (64 x 768 x 768: 7.3 [10.7]; 128 x 768 x 3072: 17.9 [19.9]; 12 x
        // 200 x 64 x 200: 5.1 [10.1]), then 64 x 64 (12 x 200 x 200 x 64: 5.1,
        // 32 x 32 7.1 [7.0])
        static const int w32 = id_of("gemm_f32w_32x32x16_k4_s4"), t64 = id_of("gemm_f32t_64x64x16_w2x2_s4");
        return tiles(32) <= 2 * cus ? w32 : t64;
    }
    // any alignment: a long sum shared by four waves (12 x 197 x 64 x 197: 6.7,
    // one wave 10.1; 16 x 77 x 64 x 77: 5.7 and 6.2), a short one not (12 x 197
    // x 197 x 64: 7.7 and 6.4; 12 x 31 x 64 x 31: 5.5 and 4.6)
    static const int k4 = id_of("gemm_f32_32x32x16_w1x1_m32_s2_p2_k4_vfalse"), k1 = id_of("gemm_f32_32x32x16_w1x1_m32_s2_p1_k1_vfalse");
    return s.K > 64 ? k4 : k1;
}

// From sums of 1024 on, 256 and more to a workgroup, up to a workgroup per CU
// (us; unsplit in brackets): fp32 32 x 32 tiles, 256 x 256 x 4096 in four 12.1 [22.4],
// 8 x 16 x 128 x 4096 in eight 9.5 [21.7], 40 x 1024 x 11008 in four 21.7 [54], 33 x
// 513 x 8193 in four 26.5 [73]; fp16 64 x 64, 33 x 513 x 8193 in sixteen 13.5 [52].
int predefined_split(const Shape &s, int id, const nnjit_device_limits &d) {
    const Config &c = configs()[id];
    if (s.M == 1 || s.K < 1024) return id;
    const int64_t tiles = s.batch * ceil_div(s.M, c.v->mt) * ceil_div(s.N, c.v->wg_cols());
    const int split = split_within(tiles, d.num_cus, s.K, 256);
    if (split == 1 || c.split != 1) return id;
    for (const Config &o : configs())
        if (o.v == c.v && o.split == split) return o.id;
    return id;
}

bool takes_scratch(const Shape &s, bool aligned, const LiteResult &lite, const nnjit_device_limits &d) {
    if (aligned || s.dtype != NNJIT_F16) return !lite.ids.empty() && configs()[lite.ids[0]].split > 1;
    // (32 x 32 tiles with 64-deep slabs, the smallest split that gives every CU
    // a workgroup)
    const int64_t tiles = s.batch * ceil_div(s.M, 32) * ceil_div(s.N, 32);
    if (tiles >= d.num_cus || tiles * 16 < d.num_cus) return false;
    int64_t fill = 1;
    while (tiles * fill < d.num_cus) fill <<= 1;
    return s.K >= 2 * fill * 64;
}

}  // namespace nnjit
