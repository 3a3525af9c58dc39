// The host runtime (tp_host.cpp) on a HIP runtime of host memory, for CPU tests of
// its bookkeeping: what it allocates and gives back, what a failed call leaves
// behind, what a captured call holds.  Enqueued work runs at once, or goes into the
// graph its stream is captured into and runs at each launch of it.  The kernels are
// stood in for: the pass counts every event of a sample in class 0 (in the
// sample's first replica if it has any) and lists one event of each sample; the
// exact tier folds the replicas and counts a listed event in class 1.
//
// The runtime refuses what HIP refuses: calls that may wait or allocate while a
// stream is being captured (unless the thread's capture mode is relaxed), a wait
// for uncaptured work inside a capture, a wait for a captured stream.  Its last
// error stays until it is read.
#include "tp_host.cpp"

#include <functional>
#include <set>

typedef std::function<void()> Work;

struct ihipGraph { std::vector<Work> work; };
struct hipGraphExec { std::vector<Work> work; };
struct ihipStream_t { ihipGraph *capture = nullptr; };
struct ihipEvent_t { ihipGraph *capture = nullptr; };

namespace {

hipError_t fk_last = hipSuccess;
std::string fk_name;            // the next calls of this function: the fk_after'th fails
int fk_after = 0;
std::map<void *, size_t> fk_alloc;
size_t fk_pinned = 0;
int fk_wrong = 0;               // frees of what is not allocated
int fk_captures = 0;            // captures under way
hipStreamCaptureMode fk_mode = hipStreamCaptureModeGlobal;
std::vector<KParams> fk_launches;
std::vector<hipStream_t> fk_streams;

hipError_t ret(hipError_t e)
{
    if (e != hipSuccess) fk_last = e;
    return e;
}

// The injected error of a call of ``name``, if it is due.
bool due(const char *name) { return fk_name == name && fk_after > 0 && --fk_after == 0; }

bool unsafe() { return fk_captures > 0 && fk_mode != hipStreamCaptureModeRelaxed; }

#define FK(name)                                       \
    if (due(#name)) return ret(hipErrorUnknown)
#define FK_UNSAFE(name)                                \
    FK(name);                                          \
    if (unsafe()) return ret(hipErrorStreamCaptureUnsupported)

void enqueue(hipStream_t st, Work w)
{
    if (st && st->capture) st->capture->work.push_back(std::move(w));
    else w();
}

}  // namespace

extern "C" {

hipError_t hipGetLastError()
{
    const hipError_t e = fk_last;
    fk_last = hipSuccess;
    return e;
}
const char *hipGetErrorString(hipError_t) { return "refused"; }
hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int) { *v = 256; return hipSuccess; }
hipError_t hipDeviceSynchronize() { FK_UNSAFE(hipDeviceSynchronize); return hipSuccess; }

hipError_t hipMalloc(void **p, size_t n)
{
    FK_UNSAFE(hipMalloc);
    *p = std::malloc(n);
    std::memset(*p, 0x5a, n);       // fresh memory is not clear
    fk_alloc[*p] = n;
    return hipSuccess;
}
hipError_t hipFree(void *p)
{
    if (!p) return hipSuccess;
    FK_UNSAFE(hipFree);
    if (!fk_alloc.erase(p)) {
        ++fk_wrong;
        return ret(hipErrorInvalidValue);
    }
    std::free(p);
    return hipSuccess;
}
hipError_t hipHostMalloc(void **p, size_t n, unsigned)
{
    FK_UNSAFE(hipHostMalloc);
    *p = std::calloc(1, n);
    ++fk_pinned;
    return hipSuccess;
}
hipError_t hipHostFree(void *p)
{
    if (!p) return hipSuccess;
    FK_UNSAFE(hipHostFree);
    std::free(p);
    --fk_pinned;
    return hipSuccess;
}
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind)
{
    FK_UNSAFE(hipMemcpy);
    std::memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t st)
{
    FK(hipMemcpyAsync);
    enqueue(st, [=] { std::memcpy(d, s, n); });
    return hipSuccess;
}
hipError_t hipMemset(void *d, int v, size_t n)
{
    FK_UNSAFE(hipMemset);
    std::memset(d, v, n);
    return hipSuccess;
}
hipError_t hipMemsetAsync(void *d, int v, size_t n, hipStream_t st)
{
    FK(hipMemsetAsync);
    if (st && st->capture) return ret(hipErrorUnknown);         // not to be recorded into a graph
    std::memset(d, v, n);
    return hipSuccess;
}

hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned)
{
    FK(hipStreamCreateWithFlags);
    *s = new ihipStream_t();
    fk_streams.push_back(*s);
    return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t s)
{
    fk_streams.erase(std::find(fk_streams.begin(), fk_streams.end(), s));
    delete s;
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t s)
{
    FK(hipStreamSynchronize);
    if ((s && s->capture) || unsafe()) return ret(hipErrorStreamCaptureUnsupported);
    return hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned)
{
    FK(hipStreamWaitEvent);
    if (e->capture) s->capture = e->capture;        // joins the capture
    else if (s && s->capture) return ret(hipErrorStreamCaptureIsolation);
    return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned)
{
    FK(hipEventCreateWithFlags);
    *e = new ihipEvent_t();
    return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t *e) { return hipEventCreateWithFlags(e, 0); }
hipError_t hipEventDestroy(hipEvent_t e)
{
    delete e;
    return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s)
{
    FK(hipEventRecord);
    e->capture = s ? s->capture : nullptr;
    return hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t e)
{
    FK_UNSAFE(hipEventSynchronize);
    return e->capture ? ret(hipErrorCapturedEvent) : hipSuccess;
}
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t)
{
    *ms = 1.0f;
    return hipSuccess;
}

hipError_t hipThreadExchangeStreamCaptureMode(hipStreamCaptureMode *m)
{
    std::swap(*m, fk_mode);
    return hipSuccess;
}
hipError_t hipStreamIsCapturing(hipStream_t s, hipStreamCaptureStatus *c)
{
    *c = s && s->capture ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return hipSuccess;
}
hipError_t hipStreamBeginCapture(hipStream_t s, hipStreamCaptureMode)
{
    FK(hipStreamBeginCapture);
    s->capture = new ihipGraph();
    ++fk_captures;
    return hipSuccess;
}
hipError_t hipStreamEndCapture(hipStream_t s, hipGraph_t *g)
{
    ihipGraph *cap = s->capture;
    for (hipStream_t t : fk_streams)
        if (t->capture == cap) t->capture = nullptr;
    --fk_captures;
    *g = nullptr;
    if (due("hipStreamEndCapture")) {
        delete cap;
        return ret(hipErrorUnknown);
    }
    *g = cap;
    return hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t *x, hipGraph_t g, hipGraphNode_t *, char *, size_t)
{
    FK(hipGraphInstantiate);
    *x = new hipGraphExec{ g->work };
    return hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t x, hipStream_t)
{
    FK(hipGraphLaunch);
    for (Work &w : x->work) w();
    return hipSuccess;
}
hipError_t hipGraphDestroy(hipGraph_t g)
{
    delete g;
    return hipSuccess;
}
hipError_t hipGraphExecDestroy(hipGraphExec_t x)
{
    delete x;
    return hipSuccess;
}

// ------------------------------------------------------------------ controls
void fk_fail(const char *name, int after) { fk_name = name; fk_after = after; }
int fk_pending() { return (int)hipGetLastError(); }
int64_t fk_bytes()
{
    size_t n = 0;
    for (auto &a : fk_alloc) n += a.second;
    return (int64_t)n;
}
int fk_wrong_frees() { return fk_wrong; }
int64_t fk_blocks() { return (int64_t)(fk_alloc.size() + fk_pinned); }
// Whether a block of device memory that starts at or holds p is allocated.
int fk_live(const void *p)
{
    auto it = fk_alloc.upper_bound(const_cast<void *>(p));
    if (it == fk_alloc.begin()) return 0;
    --it;
    return static_cast<const char *>(p) < static_cast<char *>(it->first) + it->second;
}
int fk_launch_count() { return (int)fk_launches.size(); }
const void *fk_launch_list(int i) { return fk_launches[(size_t)i].xlist; }
const void *fk_launch_samples(int i) { return fk_launches[(size_t)i].samples; }
void *fk_stream() { hipStream_t s; hipStreamCreateWithFlags(&s, 0); return s; }
void fk_begin(void *s) { hipStreamBeginCapture((hipStream_t)s, hipStreamCaptureModeGlobal); }
void *fk_end(void *s)
{
    hipGraph_t g;
    hipStreamEndCapture((hipStream_t)s, &g);
    return g;
}
void fk_replay(void *g) { for (Work &w : static_cast<ihipGraph *>(g)->work) w(); }

}  // extern "C"

// ------------------------------------------------------------------ the kernels
namespace tpk {

hipError_t launch_pass(int, int, int mode, int, int, int, bool, const KParams &kp, int, int, size_t, hipStream_t st)
{
    FK(launch_pass);
    fk_launches.push_back(kp);
    enqueue(st, [=] {
        for (int s = kp.sbeg; s < kp.send; ++s) {
            const KSample &S = kp.samples[s];
            uint64_t *counts = S.counts, *stats = S.stats;
            if (S.rep_off >= 0 && kp.rep) {
                counts = kp.rep + S.rep_off;
                stats = counts + (S.nbtot + 1) * 4;
            }
            if (mode == 0) counts[0] += (uint64_t)S.n - 1;
            stats[ST_EVENTS] += (uint64_t)S.n;
            kp.xlist[(*kp.xcount)++] = (uint64_t)s << 40;
        }
    });
    return hipSuccess;
}

hipError_t launch_exact(int, int mode, const KParams &kp, int, hipStream_t st)
{
    FK(launch_exact);
    enqueue(st, [=] {
        for (int f = 0; f < kp.nfold; ++f) {
            const uint32_t item = kp.fold ? kp.fold[f] : (uint32_t)f;
            const KSample &S = kp.samples[kp.fold ? item >> 8 : 0];
            const int nrow = (S.nbtot + 1) * 4;
            for (int w = (int)(item & 255u) * FOLD; w < std::min(((int)(item & 255u) + 1) * FOLD, rep_words(S.nbtot)); ++w)
                for (int r = 0; r <= S.rep_mask; ++r) {
                    uint64_t &v = kp.rep[S.rep_off + (int64_t)r * rep_stride(S.nbtot) + w];
                    uint64_t *to = w < nrow ? (S.counts ? S.counts + w : nullptr) : S.stats + (w - nrow);
                    if (to) *to += v;
                    v = 0;
                }
        }
        for (uint32_t k = 0; k < *kp.xcount; ++k) {
            const KSample &S = kp.samples[kp.xlist[k] >> 40];
            if (mode == 0) ++S.counts[1];
        }
        *kp.xcount = 0;
        *kp.xdone = 0;
        if (kp.mail) *kp.mail = kp.samples[0].stats[ST_UNRESOLVED];
    });
    return hipSuccess;
}

hipError_t launch_probe(const KSample &, float *, float *, double *, double *, hipStream_t) { return hipSuccess; }
hipError_t noalloc_scratch(int, unsigned char **) { return ret(hipErrorUnknown); }
hipError_t launch_noalloc_setup(const KSample &, const double *, int, int64_t, unsigned char *, hipStream_t)
{
    return hipSuccess;
}

}  // namespace tpk

namespace tpe {
hipError_t launch_pairsums(const EParams &, hipStream_t) { return hipSuccess; }
hipError_t launch_coords(const CParams &, int, hipStream_t) { return hipSuccess; }
}  // namespace tpe
