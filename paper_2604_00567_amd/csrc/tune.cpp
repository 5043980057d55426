// Autotuner: times every compiled configuration for one (N, precision) on
// synthetic data with HIP events, accepts a candidate only when its output is
// bit-identical to the first configuration that runs (the default one, unless
// it fails; all configurations compute the same butterflies, so any difference
// is a defect), and records the fastest
// in a process-wide registry that plan creation consults.  Records persist in
// a plain-text file named by DSFFT_TUNE_FILE (one record per line:
// "arch cus dtype log2n variant_a variant_b two_pass GB/s"; '#' starts a
// comment line, "# batch B" before a record says how many transforms it was
// tuned with).  Records shipped
// with the library (tuning_records.txt beside libdsfft.so, measured on the
// target device) are read first; DSFFT_TUNE_FILE records override them.
#include <dlfcn.h>
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <string>
#include <tuple>
#include <vector>

#include "batch_launch.hpp"
#include "dsfft.h"
#include "plan.hpp"
#include "tables.hpp"

namespace dsfft {

constexpr int64_t kShipped = INT64_MAX;

struct TuneRec {
    int va = 0, vb = 0, two = 0;
    double gbs = 0;
    // How many transforms a plan needs for the record to decide its kernels where the
    // rule for few transforms would choose others: those it was tuned with (1 if not
    // known; kShipped for the library's own records, which always give way to the rule).
    int64_t batch = 1;
};

static std::mutex g_tune_mu;
static std::map<std::tuple<int, int>, TuneRec> g_tuned;   // (dtype, log2 n)
static bool g_tune_loaded = false;

static std::string device_tag() {
    int dev = 0;
    hipDeviceProp_t prop;
    if (hipGetDevice(&dev) != hipSuccess || hipGetDeviceProperties(&prop, dev) != hipSuccess)
        return "unknown 0";
    std::string arch = prop.gcnArchName;
    const size_t colon = arch.find(':');
    if (colon != std::string::npos) arch = arch.substr(0, colon);
    return arch + " " + std::to_string(prop.multiProcessorCount);
}

// One record per line; blank lines, lines starting with '#' and lines that do
// not hold a well-formed record are skipped, so one bad line costs only itself.
static void read_records(const std::string& path, const std::string& tag, bool shipped) {
    FILE* f = std::fopen(path.c_str(), "r");
    if (!f) return;
    char line[512];
    long long batch = 1;                          // of a comment "# batch B" before a record
    while (std::fgets(line, sizeof line, f)) {
        const size_t len = std::strlen(line);
        if (len + 1 == sizeof line && line[len - 1] != '\n') {      // overlong: skip the rest
            int c;
            while ((c = std::fgetc(f)) != EOF && c != '\n') {
            }
            continue;
        }
        const char* q = line + std::strspn(line, " \t");
        if (*q == '#') (void)std::sscanf(q, "# batch %lld", &batch);
        if (*q == '#' || *q == '\n' || *q == '\0') continue;
        const int64_t tuned_batch = shipped ? kShipped : (batch > 0 ? batch : 1);
        batch = 1;
        char arch[64];
        int cus, dt, m, va, vb, two;
        double gbs;
        if (std::sscanf(q, "%63s %d %d %d %d %d %d %lf", arch, &cus, &dt, &m, &va, &vb, &two, &gbs) != 8) continue;
        if (dt < DT_F16 || dt > DT_F16F32 || m < 1 || m > 20 || va < 0 || vb < 0 || (two != 0 && two != 1))
            continue;
        if (tag != std::string(arch) + " " + std::to_string(cus)) continue;
        g_tuned[std::make_tuple(dt, m)] = TuneRec{va, vb, two, gbs, tuned_batch};
    }
    std::fclose(f);
}

// tuning_records.txt in the directory holding this library
static std::string shipped_records() {
    Dl_info info;
    if (!dladdr((void*)&shipped_records, &info) || !info.dli_fname) return "";
    std::string p = info.dli_fname;
    const size_t slash = p.rfind('/');
    return (slash == std::string::npos ? std::string() : p.substr(0, slash + 1)) + "tuning_records.txt";
}

static void load_records_locked() {
    if (g_tune_loaded) return;
    g_tune_loaded = true;
    const std::string tag = device_tag();
    const std::string shipped = shipped_records();
    if (!shipped.empty()) read_records(shipped, tag, true);
    if (const char* path = std::getenv("DSFFT_TUNE_FILE")) read_records(path, tag, false);
}

// The tuned choice for (dtype, log2 n), if any: variants[3] = {a, b, two_pass}.
bool tuned_choice(int dtype, int log_n, int* variants, int64_t* batch) {
    std::lock_guard<std::mutex> lock(g_tune_mu);
    load_records_locked();
    auto it = g_tuned.find(std::make_tuple(dtype, log_n));
    if (it == g_tuned.end()) return false;
    variants[0] = it->second.va;
    variants[1] = it->second.vb;
    variants[2] = it->second.two;
    if (batch) *batch = it->second.batch;
    return true;
}

static void store_record(int dtype, int log_n, const TuneRec& r) {
    std::lock_guard<std::mutex> lock(g_tune_mu);
    load_records_locked();
    g_tuned[std::make_tuple(dtype, log_n)] = r;
    const char* path = std::getenv("DSFFT_TUNE_FILE");
    if (!path) return;
    FILE* f = std::fopen(path, "a");
    if (!f) return;
    std::fprintf(f, "# batch %lld\n%s %d %d %d %d %d %.1f\n", (long long)r.batch, device_tag().c_str(), dtype,
                 log_n, r.va, r.vb, r.two, r.gbs);
    std::fclose(f);
}

// Deterministic synthetic data in [-1, 1): a 64-bit LCG, rounded to the
// storage precision (binary16 for both binary16-stored dtypes).
static void fill_synthetic(std::vector<uint8_t>& buf, int dtype, uint64_t seed) {
    uint64_t s = seed * 6364136223846793005ULL + 1442695040888963407ULL;
    if (dtype != DT_F32) {
        uint16_t* p = (uint16_t*)buf.data();
        for (size_t i = 0; i < buf.size() / 2; ++i) {
            s = s * 6364136223846793005ULL + 1442695040888963407ULL;
            const double u = (double)(s >> 11) * (1.0 / 9007199254740992.0) * 2.0 - 1.0;
            p[i] = f64_to_f16(u);
        }
    } else {
        float* p = (float*)buf.data();
        for (size_t i = 0; i < buf.size() / 4; ++i) {
            s = s * 6364136223846793005ULL + 1442695040888963407ULL;
            p[i] = (float)((double)(s >> 11) * (1.0 / 9007199254740992.0) * 2.0 - 1.0);
        }
    }
}

}  // namespace dsfft

using namespace dsfft;

extern "C" {

int fft_tune(int64_t n, int64_t batch, fft_dtype dtype, fft_table_kind kind, int reps,
             char* report, size_t cap) {
    if (n < 2 || (n & (n - 1)) || n > (int64_t(1) << 20) || batch < 1 || reps < 1)
        return set_error(FFT_EINVAL, "bad tuning request");
    int m = 0;
    while ((int64_t(1) << m) < n) ++m;
    int single = 0, cols = 0, rows = 0;
    int rc = fft_config_count(n, dtype, &single, &cols, &rows);
    if (rc != FFT_OK) return rc;
    std::vector<std::tuple<int, int, int>> cands;
    for (int v = 0; v < single; ++v) cands.emplace_back(v, 0, 0);
    for (int a = 0; a < cols; ++a)
        for (int b = 0; b < rows; ++b) cands.emplace_back(a, b, 1);
    if (cands.empty()) return set_error(FFT_EUNSUPPORTED, "no configuration for this size");

    const size_t bytes = (size_t)n * batch * elem_bytes((int)dtype);
    std::vector<uint8_t> host(bytes), ref(bytes), got(bytes);
    fill_synthetic(host, (int)dtype, (uint64_t)n * 131 + (uint64_t)batch);
    // Timed launches rotate over input/output sets larger than the 256 MB
    // memory-side cache together, so that no candidate is timed on data the
    // cache still holds from the previous launch.
    const int nsets = (int)std::max<size_t>(2, (size_t)(1.2e9 / (2.0 * bytes)) + 1);
    std::vector<void*> din(nsets, nullptr), dout(nsets, nullptr);
    hipStream_t st = nullptr;
    hipEvent_t e0 = nullptr, e1 = nullptr;
    hipError_t e = hipSuccess;
    std::string rep = "[";
    TuneRec best;
    double best_ms = 1e30;
    int accepted = 0;
    bool have_ref = false;
    auto cleanup = [&]() {
        if (st) (void)hipStreamSynchronize(st);     // nothing in flight reads the buffers
        for (void* p : din)
            if (p) (void)hipFree(p);
        for (void* p : dout)
            if (p) (void)hipFree(p);
        if (e0) (void)hipEventDestroy(e0);
        if (e1) (void)hipEventDestroy(e1);
        if (st) (void)hipStreamDestroy(st);
    };
    for (int k = 0; k < nsets && e == hipSuccess; ++k)
        if ((e = hipMalloc(&din[k], bytes)) == hipSuccess) e = hipMalloc(&dout[k], bytes);
    if (e != hipSuccess || (e = hipStreamCreateWithFlags(&st, hipStreamNonBlocking)) != hipSuccess ||
        (e = hipEventCreate(&e0)) != hipSuccess || (e = hipEventCreate(&e1)) != hipSuccess) {
        cleanup();
        return e == hipErrorOutOfMemory ? set_error(FFT_ENOMEM, "tuning buffers")
                                        : hip_error(e, "tuning setup");
    }
    for (int k = 0; k < nsets && e == hipSuccess; ++k)
        e = hipMemcpy(din[k], host.data(), bytes, hipMemcpyHostToDevice);
    if (e != hipSuccess) {
        cleanup();
        return hip_error(e, "hipMemcpy");
    }
    for (size_t c = 0; c < cands.size(); ++c) {
        const int v[3] = {std::get<0>(cands[c]), std::get<1>(cands[c]), std::get<2>(cands[c])};
        fft_plan* p = plan_create(n, batch, (int)dtype, (int)kind, v);
        if (!p) continue;
        bool ok = plan_execute(p, din[0], dout[0], st) == FFT_OK;
        ok = ok && hipStreamSynchronize(st) == hipSuccess;
        // the first candidate that runs is the reference the others must match
        ok = ok && hipMemcpy(have_ref ? got.data() : ref.data(), dout[0], bytes, hipMemcpyDeviceToHost) == hipSuccess;
        const bool same = ok && (!have_ref || std::memcmp(ref.data(), got.data(), bytes) == 0);
        if (ok) have_ref = true;
        float ms = 0;
        if (same) {
            for (int k = 1; k < nsets && ok; ++k) ok = plan_execute(p, din[k], dout[k], st) == FFT_OK;
            ok = ok && hipEventRecord(e0, st) == hipSuccess;
            for (int r = 0; r < reps && ok; ++r)
                ok = plan_execute(p, din[r % nsets], dout[r % nsets], st) == FFT_OK;
            ok = ok && hipEventRecord(e1, st) == hipSuccess && hipEventSynchronize(e1) == hipSuccess &&
                 hipEventElapsedTime(&ms, e0, e1) == hipSuccess;
            ms /= reps;
        }
        const double gbs = (ok && same && ms > 0) ? 2.0 * bytes / (ms * 1e-3) / 1e9 : 0.0;
        char buf[320];
        std::snprintf(buf, sizeof buf, "%s{\"variant\":[%d,%d,%d],\"ms\":%.5f,\"GBs\":%.1f,\"bit_exact\":%s,\"config\":\"%s\"}",
                      rep.size() > 1 ? "," : "", v[0], v[1], v[2], ms, gbs, same ? "true" : "false",
                      (describe(p, p->k1) + (p->k2 ? " | " + describe(p, p->k2) : std::string())).c_str());
        rep += buf;
        if (ok && same && ms > 0) {
            ++accepted;
            if (ms < best_ms) {
                best_ms = ms;
                best = TuneRec{v[0], v[1], v[2], gbs, batch};
            }
        }
        delete p;
    }
    cleanup();
    rep += "]";
    if (report && cap) std::snprintf(report, cap, "%s", rep.c_str());
    if (!accepted) return set_error(FFT_EHIP, "no configuration could be timed");
    store_record((int)dtype, m, best);
    return FFT_OK;
}

// The recorded choice for (n, dtype): variants and measured GB/s; FFT_EINVAL
// when nothing is recorded.
int fft_tuned_choice(int64_t n, fft_dtype dtype, int* variant_a, int* variant_b, int* two_pass) {
    int m = 0;
    while ((int64_t(1) << m) < n) ++m;
    int v[3];
    if (!tuned_choice((int)dtype, m, v)) return set_error(FFT_EINVAL, "no tuning record");
    if (variant_a) *variant_a = v[0];
    if (variant_b) *variant_b = v[1];
    if (two_pass) *two_pass = v[2];
    return FFT_OK;
}

}  // extern "C"

namespace dsfft {
fft_batch* batch_create(const int64_t* n, int64_t count, int dtype, int kind, const int* alt);
int batch_execute(fft_batch* b, const void* in, void* out, hipStream_t s);
}  // namespace dsfft

extern "C" {

// Per size class of the uneven-batch kernel with an alternative configuration
// (kAltCfg): times a batch of that class alone (2^24 elements) with each
// configuration (HIP events, `reps` graph replays), requires the outputs to be
// bit-identical, and sets alt_out[m] to 1 where the alternative is faster.
int fft_batch_tune_classes(fft_dtype dtype, fft_table_kind kind, int reps, int32_t* alt_out) {
    if (reps < 1 || !alt_out) return set_error(FFT_EINVAL, "bad tuning request");
    if ((int)dtype != DT_F16 && (int)dtype != DT_F32) return set_error(FFT_EINVAL, "dtype must be FFT_F16 or FFT_F32");
    for (int m = 0; m <= kMaxSingleLog; ++m) alt_out[m] = 0;
    for (int m = 1; m <= kMaxSingleLog; ++m) {
        if (kAltCfg[m] < 0) continue;
        const int64_t n = int64_t(1) << m, count = (int64_t(1) << 24) / n;   // 2^24 elements
        std::vector<int64_t> ns((size_t)count, n);
        const size_t bytes = (size_t)n * count * elem_bytes((int)dtype);
        std::vector<uint8_t> host(bytes), ref(bytes), got(bytes);
        fill_synthetic(host, (int)dtype, 977 + m);
        void *din = nullptr, *dout = nullptr;
        hipStream_t st = nullptr;
        hipEvent_t e0 = nullptr, e1 = nullptr;
        hipError_t e;
        if ((e = hipMalloc(&din, bytes)) != hipSuccess || (e = hipMalloc(&dout, bytes)) != hipSuccess ||
            (e = hipStreamCreateWithFlags(&st, hipStreamNonBlocking)) != hipSuccess ||
            (e = hipEventCreate(&e0)) != hipSuccess || (e = hipEventCreate(&e1)) != hipSuccess ||
            (e = hipMemcpy(din, host.data(), bytes, hipMemcpyHostToDevice)) != hipSuccess) {
            if (din) (void)hipFree(din);
            if (dout) (void)hipFree(dout);
            if (st) (void)hipStreamDestroy(st);
            if (e0) (void)hipEventDestroy(e0);
            if (e1) (void)hipEventDestroy(e1);
            return hip_error(e, "batch tuning setup");
        }
        float best = 1e30f;
        for (int alt = 0; alt < 2; ++alt) {
            int a[kMaxSingleLog + 1] = {};
            a[m] = alt;
            fft_batch* b = batch_create(ns.data(), count, (int)dtype, (int)kind, a);
            if (!b) continue;
            bool ok = batch_execute(b, din, dout, st) == FFT_OK && hipStreamSynchronize(st) == hipSuccess;
            ok = ok && hipMemcpy(alt == 0 ? ref.data() : got.data(), dout, bytes, hipMemcpyDeviceToHost) == hipSuccess;
            ok = ok && (alt == 0 || std::memcmp(ref.data(), got.data(), bytes) == 0);
            float ms = 0;
            if (ok) {
                ok = hipEventRecord(e0, st) == hipSuccess;
                for (int r = 0; r < reps && ok; ++r) ok = batch_execute(b, din, dout, st) == FFT_OK;
                ok = ok && hipEventRecord(e1, st) == hipSuccess && hipEventSynchronize(e1) == hipSuccess &&
                     hipEventElapsedTime(&ms, e0, e1) == hipSuccess;
            }
            fft_batch_destroy(b);
            if (ok && ms < best) {
                best = ms;
                alt_out[m] = alt;
            }
        }
        (void)hipFree(din);
        (void)hipFree(dout);
        (void)hipStreamDestroy(st);
        (void)hipEventDestroy(e0);
        (void)hipEventDestroy(e1);
    }
    return FFT_OK;
}

// The 2^10 and 2^12 classes' choices of fft_batch_tune_classes.
int fft_batch_tune(fft_dtype dtype, fft_table_kind kind, int reps, int* choice_1024,
                   int* choice_4096) {
    if (!choice_1024 || !choice_4096) return set_error(FFT_EINVAL, "bad tuning request");
    int32_t alt[kMaxSingleLog + 1];
    const int rc = fft_batch_tune_classes(dtype, kind, reps, alt);
    if (rc != FFT_OK) return rc;
    *choice_1024 = alt[10];
    *choice_4096 = alt[12];
    return FFT_OK;
}

}  // extern "C"
