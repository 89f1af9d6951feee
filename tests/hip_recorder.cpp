// A HIP runtime and a set of kernel launchers that compute nothing and remember everything: linked with the host side of
// the stage library (bp_stage.cpp, bp_schedule.cpp) they run its calls on the CPU and check what the GPU would not tell.
//   Order: streams and events carry vector clocks; two accesses to the same bytes, one of them a write, of which neither
//     is known to come first are an error, and so is an access outside an allocation or to freed memory.
//   Contents: every write leaves a hash of the kernel and of what it read; a gradient is the list of the products (or
//     column sums) added into it, so a contribution that is lost, doubled or made of reused memory shows.
//   Shortage: device memory has a size, and the n-th launch of a kernel can be made to fail.
#include <algorithm>
#include <cstring>
#include <map>
#include <set>
#include <string>
#include <vector>

#include "../paper_2410_19367_amd/csrc/bp_host.h"

namespace {

typedef uint64_t u64;
typedef uintptr_t addr;

u64 mix(u64 a, u64 b) {
    u64 x = a * 0x9E3779B97F4A7C15ull ^ (b + 0x632BE59BD9B4E019ull + (a << 6) + (a >> 2));
    x ^= x >> 31; x *= 0xBF58476D1CE4E5B9ull; x ^= x >> 29;
    return x;
}
u64 name_hash(const char* s) {
    u64 h = 1469598103934665603ull;
    for (; *s; ++s) h = (h ^ (unsigned char)*s) * 1099511628211ull;
    return h;
}

typedef std::vector<long> Clock;
void merge(Clock& a, const Clock& b) {
    if (a.size() < b.size()) a.resize(b.size(), 0);
    for (size_t i = 0; i < b.size(); ++i) a[i] = std::max(a[i], b[i]);
}
bool reached(const Clock& c, int stream, long seq) { return (size_t)stream < c.size() && c[stream] >= seq; }

struct Str { int id; Clock c; long seq = 0; };
struct Ev { Clock c; };
struct Access { addr lo, hi; int stream; long seq; bool write; const char* what; };
struct Alloc { size_t size; bool caller; std::vector<Access> acc; };
struct Content { addr hi; u64 hash; bool sum; std::vector<u64> terms; };     // sum: an accumulator, the terms added so far

std::vector<Str*> streams;
Clock host;
std::map<addr, Alloc> allocs;
std::map<addr, Content> contents;
std::vector<std::pair<addr, size_t>> pinned;
std::vector<std::vector<u64>> read_back(1);       // id 0: zeros
std::set<std::string> errors;
std::string error_text, fail_name;
long fail_in = -1;
const size_t total_bytes = (size_t)288 << 30;
size_t used_bytes = 0, others_bytes = 0;
size_t free_bytes() { return total_bytes - used_bytes - others_bytes; }
addr next_addr = (addr)1 << 44;
std::map<std::string, long> launches;

Str* str(hipStream_t s) {
    if (streams.empty()) streams.push_back(new Str{0});
    return s ? (Str*)s : streams[0];
}
void error(const std::string& s) { if (errors.size() < 50) errors.insert(s); }

struct Op {
    Str* s;
    const char* what;
    Op(hipStream_t st, const char* name) : s(str(st)), what(name) {
        merge(s->c, host);
        if (s->c.size() <= (size_t)s->id) s->c.resize(s->id + 1, 0);
        s->c[s->id] = ++s->seq;
        ++launches[name];
    }
    void access(const void* p, size_t bytes, bool write) {
        if (!bytes) return;
        const addr lo = (addr)p, hi = lo + bytes;
        auto it = allocs.upper_bound(lo);
        if (it == allocs.begin() || (--it, hi > it->first + it->second.size)) {
            error(std::string(what) + (write ? " writes" : " reads") + " outside any allocation");
            return;
        }
        auto& v = it->second.acc;
        for (const Access& a : v)
            if (a.lo < hi && lo < a.hi && (write || a.write) && !reached(s->c, a.stream, a.seq))
                error(std::string("unordered: ") + a.what + (a.write ? " writes" : " reads") + ", " + what +
                      (write ? " writes" : " reads"));
        v.erase(std::remove_if(v.begin(), v.end(), [&](const Access& a) {
            return a.lo >= lo && a.hi <= hi && reached(s->c, a.stream, a.seq) && (write || (!a.write && a.stream == s->id));
        }), v.end());
        v.push_back({lo, hi, s->id, s->seq, write, what});
    }
    // hash of what lies in [p, p + bytes)
    u64 peek(const void* p, size_t bytes) {
        const addr lo = (addr)p, hi = lo + bytes;
        auto it = contents.upper_bound(lo);
        if (it != contents.begin()) --it;
        u64 h = 0;
        addr at = lo;
        for (; it != contents.end() && it->first < hi; ++it) {
            if (it->second.hi <= lo) continue;
            if (it->first > at) break;
            u64 e = it->second.hash;
            if (it->first < lo || it->second.hi > hi) e = mix(e, mix(lo - std::min(lo, it->first), hi - lo));
            h = at == lo ? e : mix(h, e);
            at = it->second.hi;
        }
        if (at < hi) error(std::string(what) + " reads what nothing has written");
        return h;
    }
    u64 read(const void* p, size_t bytes) {
        if (!p) return 1;
        access(p, bytes, false);
        return peek(p, bytes);
    }
    static void clear(addr lo, addr hi) {
        auto it = contents.upper_bound(lo);
        if (it != contents.begin()) --it;
        while (it != contents.end() && it->first < hi) {
            const addr elo = it->first;
            if (it->second.hi <= lo) { ++it; continue; }
            const Content e = it->second;
            it = contents.erase(it);
            auto part = [&](addr a, addr b) {
                Content c = e;
                c.hi = b;
                if (!(e.sum && e.terms.empty())) { c.hash = mix(e.hash, mix(a - elo, b - a)); c.sum = false; }
                contents[a] = c;
            };
            if (elo < lo) part(elo, lo);
            if (e.hi > hi) part(hi, e.hi);
        }
    }
    static void set(addr lo, addr hi, u64 h) { clear(lo, hi); contents[lo] = Content{hi, h, false, {}}; }
    void write(const void* p, size_t bytes, u64 h) {
        access(p, bytes, true);
        set((addr)p, (addr)p + bytes, mix(h, name_hash(what)));
    }
    void scratch(const void* p, size_t bytes) { if (p) access(p, bytes, true); }
    void zero(const void* p, size_t bytes) {
        access(p, bytes, true);
        clear((addr)p, (addr)p + bytes);
        contents[(addr)p] = Content{(addr)p + bytes, 7, true, {}};
    }
    void add(const void* p, size_t bytes, const std::vector<u64>& t, bool overwrite) {
        access(p, bytes, true);
        const addr lo = (addr)p, hi = lo + bytes;
        std::vector<u64> all;
        if (!overwrite) {
            auto it = contents.upper_bound(lo);
            if (it == contents.begin() || (--it, it->second.hi < hi) || !it->second.sum ||
                (!it->second.terms.empty() && (it->first != lo || it->second.hi != hi)))
                error(std::string(what) + " adds to what is no sum");
            else
                all = it->second.terms;
        }
        all.insert(all.end(), t.begin(), t.end());
        clear(lo, hi);
        u64 h = 7;
        for (u64 x : all) h = mix(h, x);
        contents[lo] = Content{hi, h, true, all};
    }
    // everything in [src, src + bytes) to dst, or added to what is there
    void move(const void* dst, const void* src, size_t bytes, bool plus) {
        access(src, bytes, false);
        access(dst, bytes, true);
        const addr slo = (addr)src, shi = slo + bytes, dlo = (addr)dst;
        std::vector<std::pair<addr, Content>> parts;
        auto it = contents.upper_bound(slo);
        if (it != contents.begin()) --it;
        for (; it != contents.end() && it->first < shi; ++it)
            if (it->second.hi > slo) parts.push_back(*it);
        if (!plus) clear(dlo, dlo + bytes);
        for (auto& e : parts) {
            const bool whole = e.first >= slo && e.second.hi <= shi;
            const addr lo = std::max(e.first, slo), hi = std::min(e.second.hi, shi);
            if (!whole && !(e.second.sum && e.second.terms.empty())) {
                e.second.hash = mix(e.second.hash, mix(lo - e.first, hi - lo));
                e.second.sum = false;
            }
            e.second.hi = dlo + (hi - slo);
            if (!plus) contents[dlo + (lo - slo)] = e.second;
            else if (!e.second.sum) error(std::string(what) + " adds what is no sum");
            else if (!e.second.terms.empty()) add((const void*)(dlo + (lo - slo)), hi - lo, e.second.terms, false);
        }
    }
    // to host memory: the first word becomes the number of the list of terms
    void to_host(void* dst, const void* src, size_t bytes) {
        const u64 h = read(src, bytes);
        auto it = contents.find((addr)src);
        read_back.push_back(it != contents.end() && it->second.sum && it->second.hi == (addr)src + bytes ? it->second.terms
                                                                                                   : std::vector<u64>{h});
        const uint32_t id = (uint32_t)read_back.size() - 1;
        if (bytes >= 4) memcpy(dst, &id, 4);
    }
};

bool fails(const char* name) {
    if (fail_in < 0 || fail_name != name) return false;
    return fail_in-- == 0;
}
#define BP_MAYBE_FAIL(name) if (fails(name)) return hipErrorLaunchFailure

bool is_pinned(const void* p) {
    for (auto& r : pinned)
        if ((addr)p >= r.first && (addr)p < r.first + r.second) return true;
    return false;
}
size_t chunks(int T) { return bp::colsum_chunks(T); }

void* allocate(size_t bytes, bool caller) {
    const addr a = next_addr;
    next_addr += (bytes + ((size_t)2 << 20)) & ~(((addr)1 << 12) - 1);       // addresses are used once
    allocs[a] = Alloc{bytes, caller, {}};
    return (void*)a;
}

}  // namespace

// ---------------------------------------------------------------- the runtime

extern "C" {

hipError_t hipMalloc(void** p, size_t bytes) {
    if (bytes > free_bytes()) return hipErrorOutOfMemory;
    used_bytes += bytes;
    *p = allocate(bytes, false);
    return hipSuccess;
}
hipError_t hipFree(void* p) {
    if (!p) return hipSuccess;
    auto it = allocs.find((addr)p);
    if (it == allocs.end()) { error("hipFree of what is not allocated"); return hipErrorInvalidValue; }
    for (const Access& a : it->second.acc)
        if (!reached(host, a.stream, a.seq)) error(std::string("freed while in use by ") + a.what);
    used_bytes -= it->second.caller ? 0 : it->second.size;
    Op::clear(it->first, it->first + it->second.size);
    allocs.erase(it);
    return hipSuccess;
}
hipError_t hipMemGetInfo(size_t* f, size_t* t) { *f = free_bytes(); *t = total_bytes; return hipSuccess; }
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
const char* hipGetErrorString(hipError_t e) { return e == hipSuccess ? "ok" : "made to fail"; }
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) {
    str(nullptr);
    streams.push_back(new Str{(int)streams.size()});
    *s = (hipStream_t)streams.back();
    return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t s) { merge(host, str(s)->c); return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e) { *e = (hipEvent_t) new Ev; return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t e) { delete (Ev*)e; return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) {
    BP_MAYBE_FAIL("event");
    ((Ev*)e)->c = str(s)->c;
    merge(((Ev*)e)->c, host);
    return hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t e) { merge(host, ((Ev*)e)->c); return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) { *ms = 0.f; return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned) { merge(str(s)->c, ((Ev*)e)->c); return hipSuccess; }
hipError_t hipMemsetAsync(void* p, int, size_t bytes, hipStream_t s) { Op(s, "memset").zero(p, bytes); return hipSuccess; }
hipError_t hipMemcpyAsync(void* dst, const void* src, size_t bytes, hipMemcpyKind kind, hipStream_t s) {
    BP_MAYBE_FAIL("copy");
    Op op(s, "copy");
    if (kind == hipMemcpyDeviceToHost) op.to_host(dst, src, bytes);
    else if (kind == hipMemcpyHostToDevice) {
        u64 seed = 0;       // (the values of parameters and lengths: the first word stands for them)
        memcpy(&seed, src, std::min<size_t>(bytes, 4));
        op.write(dst, bytes, seed);
    } else op.move(dst, src, bytes, false);
    return hipSuccess;
}
hipError_t hipPointerGetAttributes(hipPointerAttribute_t* a, const void* p) {
    memset(a, 0, sizeof *a);
    if (!is_pinned(p)) return hipErrorInvalidValue;
    a->type = hipMemoryTypeHost;
    a->devicePointer = const_cast<void*>(p);
    a->hostPointer = const_cast<void*>(p);
    return hipSuccess;
}
hipError_t hipMemGetAddressRange(hipDeviceptr_t* base, size_t* size, hipDeviceptr_t p) {
    for (auto& r : pinned)
        if ((addr)p >= r.first && (addr)p < r.first + r.second) { *base = (void*)r.first; *size = r.second; return hipSuccess; }
    return hipErrorNotFound;
}

// ---------------------------------------------------------------- what the test asks for

void rec_reset() {
    allocs.clear(); contents.clear(); pinned.clear(); errors.clear(); read_back.assign(1, {});
    host.clear(); fail_in = -1; launches.clear();
    used_bytes = others_bytes = 0;
    for (Str* s : streams) { s->c.clear(); s->seq = 0; }
}
const char* rec_errors() {
    error_text.clear();
    for (auto& e : errors) error_text += e + "\n";
    return error_text.c_str();
}
void rec_others_leave(size_t bytes) {            // of the device's memory, what the object does not hold now
    others_bytes = total_bytes - used_bytes - std::min(bytes, total_bytes - used_bytes);
}
size_t rec_used() { return used_bytes; }
void rec_fail(const char* name, long in) { fail_name = name; fail_in = in; }
int rec_still_to_fail() { return fail_in >= 0; }
long rec_launches(const char* name) { return launches[name]; }
void rec_pin(const void* p, size_t bytes) { pinned.push_back({(addr)p, bytes}); }
void* rec_tensor(size_t bytes, u64 seed) {       // a tensor of the caller's (seed 0: not written yet)
    void* p = allocate(bytes, true);
    if (seed) Op::set((addr)p, (addr)p + bytes, seed);
    return p;
}
u64 rec_hash(const void* p, size_t bytes) {     // as the caller's next kernel on the default stream would read it
    return Op(nullptr, "caller").read(p, bytes);
}
int rec_terms(uint32_t id, u64* out, int cap) {
    if (id >= read_back.size()) return -1;
    const auto& t = read_back[id];
    for (int i = 0; i < (int)t.size() && i < cap; ++i) out[i] = t[i];
    return (int)t.size();
}

}  // extern "C"

// ---------------------------------------------------------------- the kernels

namespace bp {

static size_t es(int dtype) { return dtype_size(dtype); }

bool gemm_can_fuse_epilogue(int, const GemmArgs&) { return true; }

hipError_t launch_gemm(int dtype, const GemmArgs& g, hipStream_t s) {
    BP_MAYBE_FAIL(g.accumulate ? "wgrad" : "gemm");
    Op op(s, g.accumulate ? "wgrad" : "gemm");
    const size_t e = es(dtype), a = (size_t)(g.a_t ? g.K : g.M) * g.lda * e, b = (size_t)(g.b_t ? g.N : g.K) * g.ldb * e;
    std::vector<u64> t;
    for (int i = 0; i < g.nseg; ++i) {
        const u64 ha = op.read(i ? g.A_more[i - 1] : g.A, a);
        t.push_back(mix(ha, op.read(i ? g.B_more[i - 1] : g.B, b)));
    }
    op.scratch(g.split_ws, g.split_ws_elems * 4);
    if (g.accumulate) {
        op.add(g.C, (size_t)g.M * g.ldc * 4, t, g.accumulate == 2);
        return hipSuccess;
    }
    const size_t c = (size_t)g.M * g.ldc * e;
    u64 h = mix(t[0], op.read(g.bias, (size_t)g.N * 4));
    h = mix(h, op.read(g.residual, c));
    if (g.epi == EPI_GELU_BWD) h = mix(h, op.read(g.U, c));
    op.write(g.C, c, h);
    if (g.epi == EPI_GELU_FWD) op.write(g.C2, c, h + 1);
    if (g.epi == EPI_GELU_BWD) op.write(g.colpart, chunks(g.M) * g.N * 4, h + 2);
    return hipSuccess;
}
hipError_t launch_ln_fwd(int dtype, int T, int H, const void* x, const float* gamma, const float* beta, float, void* out,
                         float* mean, float* rstd, void* xcopy, hipStream_t s) {
    BP_MAYBE_FAIL("ln_fwd");
    Op op(s, "ln_fwd");
    const size_t n = (size_t)T * H * es(dtype);
    const u64 hx = op.read(x, n), h = mix(hx, mix(op.read(gamma, H * 4), op.read(beta, H * 4)));
    op.write(out, n, h);
    op.write(mean, T * 4, hx + 1);
    op.write(rstd, T * 4, hx + 2);
    if (xcopy) op.move(xcopy, x, n, false);
    return hipSuccess;
}
hipError_t launch_ln_bwd_rows(int dtype, int T, int H, const void* dout, const void* x, const float* mean, const float* rstd,
                              const float* gamma, const void* res, void* dx, hipStream_t s) {
    BP_MAYBE_FAIL("ln_bwd");
    Op op(s, "ln_bwd");
    const size_t n = (size_t)T * H * es(dtype);
    u64 h = mix(op.read(dout, n), op.read(x, n));
    h = mix(h, mix(op.read(mean, T * 4), op.read(rstd, T * 4)));
    h = mix(h, mix(op.read(gamma, H * 4), op.read(res, n)));
    op.write(dx, n, h);
    return hipSuccess;
}
hipError_t launch_colsum_batch(int dtype, int T, const ColsumBatch& b, hipStream_t s) {
    BP_MAYBE_FAIL("colsum");
    Op op(s, "colsum");
    for (int i = 0; i < b.n; ++i) {
        const ColsumJob& j = b.jobs[i];
        const size_t n = (size_t)T * j.N * es(dtype), part = chunks(T) * j.N * 4;
        if (!j.A) {
            op.add(j.out_a, (size_t)j.N * 4, {op.read(j.part, part)}, b.overwrite);
            continue;
        }
        const u64 ha = op.read(j.A, n);
        op.scratch(j.part, part * (j.out_ax ? 2 : 1));
        op.add(j.out_a, (size_t)j.N * 4, {ha}, b.overwrite);
        if (j.out_ax)
            op.add(j.out_ax, (size_t)j.N * 4, {mix(ha, mix(op.read(j.X, n), mix(op.read(j.mean, T * 4), op.read(j.rstd, T * 4))))},
                   b.overwrite);
    }
    return hipSuccess;
}
hipError_t launch_gelu_fwd(int dtype, int T, int F, const void* u, const float* bias, void* g, hipStream_t s) {
    Op op(s, "gelu_fwd");
    const size_t n = (size_t)T * F * es(dtype);
    const u64 hu = op.read(u, n);
    op.write(g, n, mix(hu, op.read(bias, (size_t)F * 4)));
    return hipSuccess;
}
hipError_t launch_gelu_bwd(int dtype, int T, int F, const void* dg, const void* u, const float* bias, void* du, float*, float* ws,
                           hipStream_t s) {
    Op op(s, "gelu_bwd");
    const size_t n = (size_t)T * F * es(dtype);
    const u64 h = mix(op.read(dg, n), mix(op.read(u, n), op.read(bias, (size_t)F * 4)));
    op.write(du, n, h);
    op.write(ws, chunks(T) * F * 4, h + 1);
    return hipSuccess;
}
hipError_t launch_attn_fwd(int dtype, const AttnArgs& a, hipStream_t s) {
    BP_MAYBE_FAIL("attn_fwd");
    Op op(s, "attn_fwd");
    const size_t n = (size_t)a.B * a.S * a.heads * a.d * es(dtype);
    const u64 h = mix(op.read(a.qkv, 3 * n), op.read(a.lens, a.B * 4));
    op.write(a.ctx, n, h);
    op.write(a.lse, (size_t)a.B * a.heads * a.S * 4, h + 1);
    return hipSuccess;
}
hipError_t launch_attn_bwd(int dtype, const AttnArgs& a, hipStream_t s) {
    BP_MAYBE_FAIL("attn_bwd");
    Op op(s, "attn_bwd");
    const size_t n = (size_t)a.B * a.S * a.heads * a.d * es(dtype), l = (size_t)a.B * a.heads * a.S * 4;
    u64 h = mix(op.read(a.qkv, 3 * n), mix(op.read(a.lens, a.B * 4), op.read(a.ctx, n)));
    h = mix(h, mix(op.read(a.lse, l), op.read(a.dctx, n)));
    op.scratch(a.delta, l);
    op.write(a.dqkv, 3 * n, h);
    return hipSuccess;
}
hipError_t launch_loss(int dtype, size_t n, const void* z, const void* target, float, void* grad, float* loss, float* ws,
                       hipStream_t s) {
    Op op(s, "loss");
    const u64 h = mix(op.read(z, n * es(dtype)), op.read(target, n * es(dtype)));
    op.scratch(ws, 1024 * 4);
    op.write(grad, n * es(dtype), h);
    op.write(loss, 4, h + 1);
    return hipSuccess;
}
hipError_t launch_read_small(const float* src, float* dst, int n, hipStream_t s) {
    Op op(s, "read_small");
    for (int i = 0; i < n; ++i)
        if (!is_pinned(dst + i)) { error("read_small writes host memory that is not pinned"); break; }
    op.to_host(dst, src, (size_t)n * 4);
    return hipSuccess;
}
hipError_t launch_fill_f32(float* p, size_t n, float v, hipStream_t s) {
    Op op(s, "fill");
    if (v == 0.f) op.zero(p, n * 4);
    else op.write(p, n * 4, 11);
    return hipSuccess;
}
hipError_t launch_add_f32(float* dst, const float* src, size_t n, hipStream_t s) {
    Op(s, "add").move(dst, src, n * 4, true);
    return hipSuccess;
}
hipError_t launch_transpose(int dtype, int rows, int cols, const void* src, void* dst, hipStream_t s) {
    Op op(s, "transpose");
    const size_t n = (size_t)rows * cols * es(dtype);
    op.write(dst, n, op.read(src, n));
    return hipSuccess;
}
hipError_t launch_cast_from_f32(int dtype, const float* src, void* dst, size_t n, hipStream_t s) {
    Op op(s, "cast");
    op.write(dst, n * es(dtype), op.read(src, n * 4));
    return hipSuccess;
}

}  // namespace bp
