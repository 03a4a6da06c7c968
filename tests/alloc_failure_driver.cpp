// Host allocations that fail, one at a time: every geometry constructor and the table
// builders with the N-th allocation failing, N = 1, 2, .. until a run needs fewer.
// A constructor returns SHT_ENOMEM and leaves nothing allocated; a table builder
// throws std::bad_alloc, or does with fewer threads, and its result is then the same.
#include <atomic>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <new>
#include <vector>

#include "../paper_1303_4945_amd/csrc/host.h"

static std::atomic<long> g_no{0}, g_fail_at{0}, g_live{0};

void *operator new(size_t n)
{
    if (++g_no == g_fail_at) throw std::bad_alloc();
    void *p = std::malloc(n ? n : 1);
    if (!p) throw std::bad_alloc();
    ++g_live;
    return p;
}
void *operator new(size_t n, const std::nothrow_t &) noexcept
{
    try {
        return operator new(n);
    } catch (const std::bad_alloc &) {
        return nullptr;
    }
}
void operator delete(void *p) noexcept
{
    if (p) --g_live;
    std::free(p);
}
void operator delete(void *p, size_t) noexcept { operator delete(p); }
void operator delete(void *p, const std::nothrow_t &) noexcept { operator delete(p); }

static int g_bad = 0;

// run() with every allocation failing in turn; returns how many failed
template <typename Run>
static int each(const char *what, Run run)
{
    int n = 1;
    for (;; ++n) {
        const long live = g_live;
        g_no = 0;
        g_fail_at = n;
        const bool ok = run();
        const bool reached = g_no >= n;
        g_fail_at = 0;
        if (g_live != live) {
            std::printf("%s: allocation %d fails: %ld left\n", what, n, (long)g_live - live);
            ++g_bad;
        }
        if (!reached) {
            if (!ok) {
                std::printf("%s: fails without a failed allocation\n", what);
                ++g_bad;
            }
            break;
        }
    }
    std::printf("%s: %d allocations\n", what, n - 1);
    std::fflush(stdout);
    return n - 1;
}

template <typename Make>
static void geometry(const char *what, Make make)
{
    // (the registry keeps its buckets: grown here, not in the counted runs)
    sht_geom *warm = nullptr;
    if (make(&warm) != SHT_OK) ++g_bad;
    sht_geom_destroy(warm);
    const int n = each(what, [&] {
        sht_geom *g = reinterpret_cast<sht_geom *>(1);
        const int rc = make(&g);
        if (rc == SHT_OK) {
            sht_geom_destroy(g);
            return true;
        }
        if (rc != SHT_ENOMEM || g != nullptr || !std::strlen(sht_last_error())) {
            std::printf("%s: status %d\n", what, rc);
            ++g_bad;
        }
        return false;
    });
    if (n < 3) ++g_bad;
}

template <typename T>
static bool same(const std::vector<T> &a, const std::vector<T> &b)
{
    return a.size() == b.size() && !std::memcmp(a.data(), b.data(), a.size() * sizeof(T));
}

int main()
{
    geometry("gauss", [](sht_geom **g) { return sht_geom_gauss(9, 16, 0.0, g); });
    geometry("ecp", [](sht_geom **g) { return sht_geom_ecp(9, 16, SHT_ECP_CC, 0.0, g); });
    geometry("reduced gauss", [](sht_geom **g) { return sht_geom_reduced_gauss(9, 16, 8, 8, 0, 0.0, g); });
    geometry("healpix", [](sht_geom **g) { return sht_geom_healpix(2, g); });
    const double th[2] = {0.3, 1.0}, p0[2] = {0.0, 0.0};
    const int64_t np[2] = {4, 4};
    geometry("given rings", [&](sht_geom **g) { return sht_geom_create(2, th, np, p0, nullptr, nullptr, 1, g); });

    // tables large enough for several threads
    sht::PlanShape ps{};
    ps.lmax = ps.mmax = 1023;
    std::vector<sht::Coef4> ref, c;
    std::vector<double> fref, f;
    std::vector<int64_t> oref, o;
    sht::build_coef2(ps, ref, oref);
    const auto drop = [&] {
        std::vector<sht::Coef4>().swap(c);
        std::vector<double>().swap(f);
        std::vector<int64_t>().swap(o);
    };
    each("two-step table", [&] {
        bool ok = true;
        try {
            sht::build_coef2(ps, c, o);
            if (!same(c, ref) || !same(o, oref)) ++g_bad;
        } catch (const std::bad_alloc &) {
            ok = false;
        }
        drop();
        return ok;
    });
    sht::build_coef(ps, ref, fref, oref);
    each("one-step table", [&] {
        bool ok = true;
        try {
            sht::build_coef(ps, c, f, o);
            if (!same(c, ref) || !same(f, fref) || !same(o, oref)) ++g_bad;
        } catch (const std::bad_alloc &) {
            ok = false;
        }
        drop();
        return ok;
    });
    std::vector<sht::StartCoef> sref, st;
    ps.spin = 2;
    sht::build_start(ps, sref);
    each("start values", [&] {
        bool ok = true;
        try {
            sht::build_start(ps, st);
            if (!same(st, sref)) ++g_bad;
        } catch (const std::bad_alloc &) {
            ok = false;
        }
        std::vector<sht::StartCoef>().swap(st);
        return ok;
    });
    std::printf(g_bad ? "FAILED\n" : "all checks passed\n");
    return g_bad ? 1 : 0;
}
