// Drives the library's host code on a runtime double: the HIP calls it makes are answered here, nothing runs on a GPU.
// Kernels are not executed; an encoder launch tells the host its stream lengths as the kernel would.  What is kept is what
// each stream has been ordered behind (launches and copies per stream, carried by events), so that the order a call leaves
// behind can be checked.  Run as: host_order SCENARIO; prints "ok" or what is out of order.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <map>
#include <string>
#include <vector>
#include <hip/hip_runtime.h>
#include "neuzip_format.h"

namespace {

using Clock = std::map<hipStream_t, uint64_t>;  // work of a stream: how many pieces of it have gone before
struct Event { Clock at; };

// (the library registers its kernels before this program's own variables are initialised)
std::map<const void *, std::string> &names() { static auto *n = new std::map<const void *, std::string>; return *n; }
std::map<hipStream_t, Clock> g_seen;            // what the next piece of work on a stream is ordered behind
std::map<hipStream_t, uint64_t> g_work;         // pieces of work given to a stream
std::map<hipStream_t, std::vector<Clock>> g_behind;  // per piece of work: what it was ordered behind
Clock g_host;                                   // what the host has waited for
nz::HostRecord *g_record = nullptr;
uint64_t g_words = 1000;                        // stream length that the encoder reports for every tensor
int g_mallocs_until_failure = -1;
int g_waits = 0;
bool g_capturing = false;
uint32_t g_threads = 0;                         // of a workgroup of the last launch
std::string g_launched;                         // the last kernel
bool g_slow_kernels = false;                    // the host has to wait for the stream before it is told anything
std::vector<std::pair<uint32_t, unsigned long long>> g_to_tell;
struct { dim3 grid, block; size_t shared; hipStream_t stream; } g_call;

void join(Clock &into, const Clock &from)
{
    for (const auto &e : from)
        if (into[e.first] < e.second)
            into[e.first] = e.second;
}

void work(hipStream_t s)
{
    join(g_seen[s], g_host);
    g_behind[s].push_back(g_seen[s]);
    g_seen[s][s] = ++g_work[s];
}

void wait_for(const Clock &c) { join(g_host, c); }

[[noreturn]] void wrong(const std::string &what)
{
    std::printf("%s\n", what.c_str());
    std::fflush(stdout);
    std::_Exit(1);
}
void expect(bool ok, const std::string &what)
{
    if (!ok)
        wrong(what);
}

}  // namespace

extern "C" {
void **__hipRegisterFatBinary(const void *) { static void *handle; return &handle; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *fn, char *, const char *name, unsigned, void *, void *, void *, void *, int *)
{
    names()[fn] = name;
}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t shared, hipStream_t stream)
{
    g_call = {grid, block, shared, stream};
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *shared, hipStream_t *stream)
{
    *grid = g_call.grid, *block = g_call.block, *shared = g_call.shared, *stream = g_call.stream;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void *fn, dim3, dim3 block, void **args, size_t, hipStream_t stream)
{
    const std::string &name = names()[fn];
    g_threads = block.x;
    g_launched = name;
    work(stream);
    if (name.find("encode_kernel") != std::string::npos) {
        const nz::CompressBatch &b = *static_cast<const nz::CompressBatch *>(args[0]);
        for (uint32_t i = 0; i < b.count && g_record; ++i) {
            const unsigned long long told = nz::told_of(g_words, 0, b.seq);
            if (g_slow_kernels)
                g_to_tell.push_back({i, told});
            else
                g_record->item[i].told = told;
        }
    }
    return hipSuccess;
}
hipError_t hipMalloc(void **p, size_t n)
{
    if (g_mallocs_until_failure == 0)
        return hipErrorOutOfMemory;
    if (g_mallocs_until_failure > 0)
        --g_mallocs_until_failure;
    *p = std::calloc(1, 64);  // (an address: nothing reads or writes it)
    (void)n;
    return hipSuccess;
}
hipError_t hipFree(void *p)
{
    for (const auto &w : g_work)  // waits for the device
        g_host[w.first] = w.second;
    std::free(p);
    return hipSuccess;
}
hipError_t hipHostMalloc(void **p, size_t n, unsigned)
{
    *p = std::calloc(1, n);
    g_record = static_cast<nz::HostRecord *>(*p);
    return hipSuccess;
}
hipError_t hipHostFree(void *p)
{
    g_record = nullptr;
    std::free(p);
    return hipSuccess;
}
hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetLastError(void) { return hipSuccess; }
hipError_t hipGetSymbolAddress(void **p, const void *) { static uint64_t somewhere[4]; *p = somewhere; return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { *e = reinterpret_cast<hipEvent_t>(new Event); return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t e) { delete reinterpret_cast<Event *>(e); return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s)
{
    join(g_seen[s], g_host);
    reinterpret_cast<Event *>(e)->at = g_seen[s];
    return hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t e) { wait_for(reinterpret_cast<Event *>(e)->at); return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned)
{
    expect(!g_capturing, "an event of another stream in a stream under capture");
    ++g_waits;
    join(g_seen[s], reinterpret_cast<Event *>(e)->at);
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t s)
{
    wait_for(g_seen[s]);
    for (const auto &t : g_to_tell)
        g_record->item[t.first].told = t.second;
    g_to_tell.clear();
    return hipSuccess;
}
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus *st)
{
    *st = g_capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void *to, const void *, size_t n, hipMemcpyKind kind, hipStream_t s)
{
    if (kind == hipMemcpyDeviceToHost)
        std::memset(to, 0, n);
    work(s);
    return hipSuccess;
}
}

namespace {

const hipStream_t A = reinterpret_cast<hipStream_t>(0x1000), B = reinterpret_cast<hipStream_t>(0x2000);
void *const kSomewhere = reinterpret_cast<void *>(0x100000);
constexpr uint64_t kElems = 128 * 8000;

neuzip_blob *compressed(hipStream_t s, neuzip_blob *blob = nullptr, uint64_t n = kElems)
{
    expect(neuzip_compress(kSomewhere, n, NEUZIP_BF16, 7, s, &blob) == NEUZIP_OK, "compress");
    return blob;
}

// `call` gives work to B: every piece of it is behind all that A has been given by now.
void expect_behind(const char *what, const std::function<int()> &call)
{
    const size_t first = g_behind[B].size();
    const uint64_t before = g_work[A];
    expect(call() == NEUZIP_OK, std::string(what) + " failed");
    expect(g_behind[B].size() > first, std::string(what) + " did nothing");
    for (size_t i = first; i < g_behind[B].size(); ++i)
        expect(g_behind[B][i][A] >= before, std::string(what) + " is not ordered behind the other stream's work");
}

// A compress call into an existing blob fails on A for want of memory after its kernels have been launched; a call on B uses
// the workspace next.  (Twice, since the first failure gives the old word section back, and a free waits for the device.)
void after_a_failure()
{
    g_words = 0;
    neuzip_blob *blob = compressed(A);
    g_words = 500000;
    g_mallocs_until_failure = 0;
    for (int i = 0; i < 2; ++i)
        expect(neuzip_compress(kSomewhere, kElems, NEUZIP_BF16, 7, A, &blob) == NEUZIP_ENOMEM, "the failing call");
    g_mallocs_until_failure = -1;
    g_words = 1000;
    expect_behind("the next call", [] { compressed(B); return 0; });
}

// The calls that read blobs, on B, each with blobs that the latest compress call has filled on A.
struct Reader { const char *what; std::function<int(neuzip_blob *, hipStream_t)> call; };
std::vector<Reader> readers()
{
    auto room = [] { static uint8_t buffer[1 << 22]; return static_cast<void *>(buffer); };
    return {
        {"decompress", [](neuzip_blob *b, hipStream_t s) { return neuzip_decompress(b, kSomewhere, kElems, NEUZIP_BF16, s); }},
        {"decompress_batch", [](neuzip_blob *b, hipStream_t s) {
             void *dst = kSomewhere;
             return neuzip_decompress_batch(&b, &dst, 1, s);
         }},
        {"decompress_sequence", [](neuzip_blob *b, hipStream_t s) {
             return neuzip_decompress_sequence(&b, 1, kSomewhere, kElems, nullptr, s);
         }},
        {"linear", [](neuzip_blob *b, hipStream_t s) {
             return neuzip_linear(b, kElems / 128, 128, kSomewhere, 1, nullptr,
                                  static_cast<float *>(kSomewhere), s);
         }},
        {"update", [](neuzip_blob *b, hipStream_t s) {
             const void *grad = static_cast<uint8_t *>(kSomewhere) + 256;
             void *weight = kSomewhere;
             return neuzip_update(&b, &grad, &weight, 1, 1.0f, NEUZIP_UPDATE_FROM_BLOB, s, nullptr);
         }},
        {"recompress", [](neuzip_blob *b, hipStream_t s) {
             const void *src = kSomewhere;
             return neuzip_recompress(&src, 1, s, &b, nullptr);
         }},
        {"compress_noalloc", [](neuzip_blob *b, hipStream_t s) {
             return neuzip_compress_noalloc(kSomewhere, kElems, NEUZIP_BF16, 7, s, b);
         }},
        {"export", [room](neuzip_blob *b, hipStream_t s) {
             uint64_t written = 0;
             return neuzip_export(b, room(), 1 << 22, &written, s);
         }},
        {"check", [](neuzip_blob *b, hipStream_t s) { return neuzip_check(b, s); }},
    };
}

void expect_no_wait(const char *what, const std::function<int()> &call)
{
    const int before = g_waits;
    expect(call() == NEUZIP_OK, std::string(what) + " failed");
    expect(g_waits == before, std::string(what) + " made a stream wait for nothing");
}

void read_on_another_stream()
{
    for (const Reader &r : readers()) {
        neuzip_blob *blob = compressed(A);
        expect_behind(r.what, [&] { return r.call(blob, B); });
        neuzip_free(blob);
    }
}

// Where there is nothing to wait for, no event gets between: the same stream, a later call that has reported, a workspace that
// has been given back (which waits), a call that synchronises.
void read_without_waiting()
{
    for (const Reader &r : readers()) {
        const std::string what = r.what;
        if (what == "update" || what == "recompress")   // (they use the workspace, and wait for it)
            continue;
        neuzip_blob *blob = compressed(A);
        expect_no_wait(r.what, [&] { return r.call(blob, A); });
        blob = compressed(A, blob);
        neuzip_blob *other = compressed(A);
        expect_no_wait(r.what, [&] { return r.call(blob, B); });
        blob = compressed(A, blob);
        expect(neuzip_release_workspace() == NEUZIP_OK, "release");
        expect_no_wait(r.what, [&] { return r.call(blob, B); });
        expect(neuzip_compress_noalloc(kSomewhere, kElems, NEUZIP_BF16, 7, A, blob) == NEUZIP_OK, "noalloc");
        expect_no_wait(r.what, [&] { return r.call(blob, B); });
        neuzip_free(blob);
        neuzip_free(other);
    }
}

void read_under_capture()
{
    neuzip_blob *blob = compressed(A);
    g_capturing = true;
    expect_no_wait("decompress", [&] { return readers()[0].call(blob, B); });
    expect_no_wait("linear", [&] { return readers()[3].call(blob, B); });
}

// Stamps come around again: what a call long ago has left in the record is not taken for this call's.
void an_old_stamp()
{
    const uint64_t tiles = (kElems + 16 * nz::kChunk - 1) / (16 * nz::kChunk);
    for (bool tiled : {false, true}) {
        expect(neuzip_set_workspace_limit(tiled ? 102400 : 0) == NEUZIP_OK, "limit");
        expect(neuzip_release_workspace() == NEUZIP_OK, "release");
        neuzip_blob *blob = compressed(A);              // stamps 1, or 1 to the number of tiles
        const uint64_t bytes = neuzip_compressed_bytes(blob);
        g_record->item[0].told = nz::told_of(77, 0, tiled ? static_cast<uint32_t>(tiles) + 1 : 2u);
        g_slow_kernels = true;
        blob = compressed(A, blob);
        g_slow_kernels = false;
        expect(neuzip_compressed_bytes(blob) == bytes, "a length that another call has left");
        neuzip_free(blob);
    }
}

// A decoder's workgroup has as many chunks as their words fit the LDS window by their average and a hundredth, four at a time.
void chunks_of_a_workgroup()
{
    for (int k : {7, 3, 1, 0})
        for (uint64_t chunks : {4096, 5000})
            for (uint64_t bytes = 1000; bytes <= 6000; bytes += 20) {     // of a chunk's words
                const uint32_t lanes = nz::has_entry_points(static_cast<uint32_t>(chunks)) ? 32 : 16, most = 512 / lanes;
                const double window = 62 * 1024 - (k == 1 ? 2048 : (k == 0 ? 128 : 0));
                g_words = chunks * bytes / 2;
                neuzip_blob *blob = nullptr;
                expect(neuzip_compress(kSomewhere, chunks * nz::kChunk, NEUZIP_BF16, k, A, &blob) == NEUZIP_OK, "compress");
                expect(neuzip_decompress(blob, kSomewhere, chunks * nz::kChunk, NEUZIP_BF16, A) == NEUZIP_OK, "decompress");
                const uint32_t per = g_threads / lanes;
                const std::string what = std::to_string(per) + " chunks of " + std::to_string(bytes) + " bytes, k = " + std::to_string(k);
                expect(per % 4 == 0 && per * lanes == g_threads && per >= 4 && per <= most, what);
                expect(per * bytes * 1.005 < window, what + " do not fit");
                expect(per == most || (per + 4) * (bytes + 2) * 1.0105 > window, what + " are fewer than fit");
                neuzip_free(blob);
            }
}

// Blobs with entry points are walked without a branch in the step where every CU has one workgroup at most, but not those
// whose runs all have 256 bytes.  (The last template argument: single launches' "entry points", batches' form of the walk.)
void form_of_the_walk()
{
    for (double bits : {2.0, 7.75, 7.94, 7.96, 8.0, 8.005, 8.02, 11.0}) {
        const bool in_step = bits > 7.95 && bits < 8.01;
        for (uint64_t chunks : {3, 250, 2048}) {
            const uint64_t n = chunks * nz::kChunk;
            g_words = static_cast<uint64_t>(n * bits / 16);
            neuzip_blob *blobs[2] = {compressed(A, nullptr, n), compressed(A, nullptr, n)};
            void *dsts[2] = {kSomewhere, kSomewhere};
            const std::string what = std::to_string(bits) + " bits: ";
            expect(neuzip_decompress(blobs[0], kSomewhere, n, NEUZIP_BF16, A) == NEUZIP_OK, "decompress");
            expect(g_launched.find(in_step ? "decode_batch_kernelILi7ELb0ELi0ELi2EE" : "decode_kernelILi7ELb0ELi0ELb1EE") != std::string::npos, what + g_launched);
            expect(neuzip_decompress_batch(blobs, dsts, 2, A) == NEUZIP_OK, "decompress_batch");
            const uint64_t per = g_threads / 32, alone = !in_step && 2 * ((chunks + per - 1) / per) <= 256;
            expect(g_launched.find(alone ? "decode_batch_kernelILi7ELb0ELi0ELi4EE" : "decode_batch_kernelILi7ELb0ELi0ELi2EE") != std::string::npos, what + g_launched);
            neuzip_free(blobs[0]);
            neuzip_free(blobs[1]);
        }
    }
    g_words = 4096 * 4096 / 2;  // a batch of more workgroups than CUs
    neuzip_blob *blobs[2] = {compressed(A, nullptr, 4096 * 4096), compressed(A, nullptr, 4096 * 4096)};
    void *dsts[2] = {kSomewhere, kSomewhere};
    expect(neuzip_decompress_batch(blobs, dsts, 2, A) == NEUZIP_OK, "decompress_batch");
    expect(g_launched.find("decode_batch_kernelILi7ELb0ELi0ELi2EE") != std::string::npos, g_launched);
}

// Whole walks have their words copied straight into LDS where all workgroups run at once, two on each of 256 CUs.
void form_of_the_whole_walk()
{
    for (uint64_t bytes : {1400, 2500, 3800, 5000})        // of a chunk's words: 32, 24, 16 and 12 chunks to a workgroup
        for (uint64_t chunks : {4097, 5000, 6144, 6145, 8192, 8193, 12288, 12289, 16383, 16384}) {
            const uint64_t n = chunks * nz::kChunk;
            g_words = chunks * bytes / 2;
            neuzip_blob *blob = compressed(A, nullptr, n);
            expect(neuzip_decompress(blob, kSomewhere, n, NEUZIP_BF16, A) == NEUZIP_OK, "decompress");
            const uint64_t per = g_threads / 16, workgroups = (chunks + per - 1) / per;
            const bool direct = workgroups <= 512 && n < (64ull << 20);
            expect((g_launched.find("decode_direct_kernelILi7ELb0EE") != std::string::npos) == direct,
                   std::to_string(workgroups) + " workgroups: " + g_launched);
            neuzip_free(blob);
        }
}

// The linear layer's walk in launches of few workgroups (its last template argument): without a branch unless the runs of most
// weights are of 128 or 256 bytes.
void form_of_the_linear_walk()
{
    for (double bits : {2.0, 3.94, 3.96, 4.0, 4.02, 7.94, 7.96, 8.0, 8.02}) {
        const bool in_step = (bits > 3.95 && bits < 4.01) || (bits > 7.95 && bits < 8.01);
        const uint64_t rows[2] = {1024, 300}, n = 1024 * 1024;
        g_words = static_cast<uint64_t>(n * bits / 16);
        neuzip_blob *weights[2] = {compressed(A, nullptr, n), nullptr};
        float *const ys[2] = {static_cast<float *>(kSomewhere), static_cast<float *>(kSomewhere)};
        auto last = [](bool eager) { return std::string(eager ? "ELb0ELb1EE" : "ELb0ELb0EE"); };
        expect(neuzip_linear_batch(weights, rows, 1, 1024, kSomewhere, 1, nullptr, ys, A) == NEUZIP_OK, "linear");
        expect(g_launched.find(last(!in_step)) != std::string::npos, std::to_string(bits) + " bits: " + g_launched);
        g_words = 300 * 1024 / 8;
        weights[1] = compressed(A, nullptr, 300 * 1024);   // (of fewer elements: it does not decide)
        expect(neuzip_linear_batch(weights, rows, 2, 1024, kSomewhere, 1, nullptr, ys, A) == NEUZIP_OK, "linear_batch");
        expect(g_launched.find(last(!in_step)) != std::string::npos, std::to_string(bits) + " bits: " + g_launched);
    }
}

// More than 16 tokens on weights with entry points that put two workgroups on CUs: in halves (16 columns) where the activations
// are laid out, whole (32 columns) as they lie, up to a few tokens and but for short rows.  One workgroup per CU: in halves.
void columns_of_the_linear_walk()
{
    const struct { uint64_t rows[2], in_features; uint32_t tokens; bool laid_out, as_it_lies; } cases[] = {
        {{4096, 1024}, 4096, 17, true, true}, {{4096, 1024}, 4096, 20, true, true}, {{4096, 1024}, 4096, 21, true, false},
        {{4096, 1024}, 4096, 64, true, false}, {{5000, 5000}, 1920, 64, true, false}, {{8192, 2048}, 2048, 24, true, true},
        {{8192, 2048}, 2048, 25, true, false}, {{14336, 4096}, 1024, 32, true, true}, {{14336, 4096}, 1024, 33, true, false},
        {{30000, 30000}, 512, 64, true, true}, {{2048, 1024}, 4096, 64, true, true}, {{4096, 4096}, 14336, 64, false, false}};
    for (const auto &c : cases) {
        neuzip_blob *weights[2] = {nullptr, nullptr};
        float *const ys[2] = {static_cast<float *>(kSomewhere), static_cast<float *>(kSomewhere)};
        for (int i = 0; i < 2; ++i) {
            g_words = c.rows[i] * c.in_features / 6;
            weights[i] = compressed(A, nullptr, c.rows[i] * c.in_features);
        }
        const uint64_t size = neuzip_linear_scratch_bytes(c.rows, 2, c.in_features, c.tokens);
        for (bool room : {true, false}) {
            g_launched.clear();
            expect(neuzip_linear_batch_scratch(weights, c.rows, 2, c.in_features, kSomewhere, c.tokens, nullptr, ys,
                                               room ? kSomewhere : nullptr, size, A) == NEUZIP_OK, "linear_batch_scratch");
            const bool halves = room && size > 0 ? c.laid_out : c.as_it_lies;
            const std::string want = halves ? "linear_batch_kernelILi7ELi16E" : "linear_batch_kernelILi7ELi32E";
            // (sums of pieces are added up behind the walk)
            expect(g_launched.find(want) != std::string::npos || (room && g_launched.find("linear_sum_kernel") != std::string::npos),
                   std::to_string(c.rows[0]) + " x " + std::to_string(c.in_features) + ", " + std::to_string(c.tokens) + " tokens: " + g_launched);
        }
        neuzip_free(weights[0]);
        neuzip_free(weights[1]);
    }
}

// Blobs of a batch that other streams have filled: behind the latest of them.
void read_a_batch()
{
    neuzip_blob *blobs[3] = {compressed(B), compressed(A), compressed(A)};
    void *dsts[3] = {kSomewhere, kSomewhere, kSomewhere};
    expect_behind("decompress_batch", [&] { return neuzip_decompress_batch(blobs, dsts, 3, B); });
    blobs[0] = compressed(A, blobs[0]);
    expect_behind("decompress_batch", [&] { return neuzip_decompress_batch(blobs, dsts, 3, B); });
}

}  // namespace

int main(int argc, char **argv)
{
    const std::string s = argc > 1 ? argv[1] : "";
    if (s == "failure") {
        after_a_failure();
    } else if (s == "failure_in_a_tile") {
        expect(neuzip_set_workspace_limit(102400) == NEUZIP_OK, "limit");
        after_a_failure();
    } else if (s == "other_stream") {
        read_on_another_stream();
    } else if (s == "other_stream_in_tiles") {
        expect(neuzip_set_workspace_limit(102400) == NEUZIP_OK, "limit");
        read_on_another_stream();
    } else if (s == "nothing_to_wait_for") {
        read_without_waiting();
    } else if (s == "capture") {
        read_under_capture();
    } else if (s == "chunks_of_a_workgroup") {
        chunks_of_a_workgroup();
    } else if (s == "form_of_the_walk") {
        form_of_the_walk();
    } else if (s == "form_of_the_linear_walk") {
        form_of_the_linear_walk();
    } else if (s == "columns_of_the_linear_walk") {
        columns_of_the_linear_walk();
    } else if (s == "form_of_the_whole_walk") {
        form_of_the_whole_walk();
    } else if (s == "old_stamp") {
        an_old_stamp();
    } else if (s == "batch") {
        read_a_batch();
    } else {
        wrong("unknown scenario " + s);
    }
    std::printf("ok\n");
    return 0;
}
