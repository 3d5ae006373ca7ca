"""What the library's host code asks of the HIP runtime, watched on the CPU: a stand-in for the runtime's calls is loaded
before libenec.so in a process of its own (device pointers are made-up numbers; nothing is launched)."""
import ctypes
import json
import os
import subprocess
import sys

import pytest

from conftest import ROOT

STAND_IN = r"""
#include <pthread.h>
#include <stdint.h>
#include <stdlib.h>

typedef struct { uint32_t x, y, z; } dim3_;
static pthread_mutex_t mu = PTHREAD_MUTEX_INITIALIZER;
static pthread_cond_t moved = PTHREAD_COND_INITIALIZER;
int slots_held, slots_most, frees_unguarded, mallocs_unguarded, launches;
int counted = 100000, wrong_syncs;                   /* what a counting kernel hands over: so many elements, none in the first wrong_syncs waits */
static struct { char *at; size_t bytes; } slot[16];  /* pinned memory: counts first, the word that says they are there 64 bytes before its end */
int capturing, launch_fails, sync_fails, gather;     /* set by the test; gather: callers that meet in a wait */
static int gathered;
uint32_t grid[64], block[64], lds[64];
uint64_t fn[64];
int keep_bytes;                                      /* of the next launches' first argument, the last launch's are kept */
uint8_t kept[2048];
static _Thread_local int mode;                       /* 0 = global, 2 = relaxed */
static _Thread_local dim3_ pushed_grid, pushed_block;
static _Thread_local size_t pushed_lds;
static _Thread_local void *pushed_stream;

int hipThreadExchangeStreamCaptureMode(int *m) { int old = mode; mode = *m; *m = old; return 0; }
int hipStreamIsCapturing(void *s, int *status) { *status = capturing; return 0; }
int hipHostMalloc(void **p, size_t n, unsigned flags)
{
    pthread_mutex_lock(&mu);
    if (mode != 2) ++mallocs_unguarded;
    if (++slots_held > slots_most) slots_most = slots_held;
    *p = calloc(1, n);
    for (int i = 0; i < 16; ++i) if (!slot[i].at) { slot[i].at = *p; slot[i].bytes = n; break; }
    pthread_mutex_unlock(&mu);
    return 0;
}
int hipHostFree(void *p)
{
    pthread_mutex_lock(&mu);
    if (mode != 2) ++frees_unguarded;
    --slots_held;
    for (int i = 0; i < 16; ++i) if (slot[i].at == p) slot[i].at = 0;
    pthread_mutex_unlock(&mu);
    free(p);
    return 0;
}
int hipStreamSynchronize(void *s)
{
    pthread_mutex_lock(&mu);
    if (gather) {
        ++gathered;
        pthread_cond_broadcast(&moved);
        while (gathered < gather) pthread_cond_wait(&moved, &mu);
    }
    if (wrong_syncs > 0) --wrong_syncs;
    else for (int i = 0; i < 16; ++i) if (slot[i].at) { *(uint64_t *)slot[i].at = (uint64_t)counted; *(uint32_t *)(slot[i].at + slot[i].bytes - 64) = 1; }
    pthread_mutex_unlock(&mu);
    return capturing ? 900 : sync_fails;
}
int hipLaunchKernel(const void *f, dim3_ g, dim3_ b, void **args, size_t shared, void *s)
{
    pthread_mutex_lock(&mu);
    if (launches < 64) { grid[launches] = g.x; block[launches] = b.x; lds[launches] = (uint32_t)shared; fn[launches] = (uint64_t)f; }
    ++launches;
    for (int i = 0; i < keep_bytes; ++i) kept[i] = ((uint8_t *)args[0])[i];
    pthread_mutex_unlock(&mu);
    return launch_fails;
}
/* what a <<<>>> launch does before and inside the kernel's stub */
int __hipPushCallConfiguration(dim3_ g, dim3_ b, size_t shared, void *s) { pushed_grid = g; pushed_block = b; pushed_lds = shared; pushed_stream = s; return 0; }
int __hipPopCallConfiguration(dim3_ *g, dim3_ *b, size_t *shared, void **s) { *g = pushed_grid; *b = pushed_block; *shared = pushed_lds; *s = pushed_stream; return 0; }
int hipGetLastError(void) { return 0; }
int hipGetDevice(int *d) { *d = 0; return 0; }
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *f, int threads, size_t dynamic) { *n = 3; return 0; }
int hipDeviceGetAttribute(int *v, int what, int device) { *v = 256; return 0; }
int hipFuncSetAttribute(const void *f, int what, int value) { return 0; }
"""

PRELUDE = r"""
import ctypes as C, json, struct, sys, threading
rt = C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)         # before the library: its calls end here
L = C.CDLL(sys.argv[2])
def word(name): return C.c_int.in_dll(rt, name)
def launches(): return [(C.c_uint32 * 64).in_dll(rt, "grid")[i] for i in range(word("launches").value)], [(C.c_uint32 * 64).in_dll(rt, "block")[i] for i in range(word("launches").value)]
FAKE = 1 << 20                                       # a "device" pointer, 16-byte aligned
class P(C.Structure): _fields_ = [(f, C.c_uint8) for f in "bnmL"]
def tune(stream=64):
    prm = P()
    return L.enec_tune(C.c_void_p(FAKE), C.c_size_t(100000), 0, C.byref(prm), None, C.c_void_p(FAKE), C.c_size_t(1 << 20), C.c_void_p(stream))
def report(**kw): print(json.dumps(kw))
"""


@pytest.fixture(scope="module")
def stand_in(tmp_path_factory):
    from paper_2604_03298_amd import enec
    if not os.path.exists(enec.LIB_PATH):
        from paper_2604_03298_amd import build
        build.build()
    where = tmp_path_factory.mktemp("stand_in")
    src, so = where / "runtime.c", where / "runtime.so"
    src.write_text(STAND_IN)
    subprocess.run(["gcc", "-O1", "-shared", "-fPIC", "-pthread", "-o", str(so), str(src)], check=True)

    def run(body):
        script = where / "script.py"
        script.write_text(PRELUDE + body)
        res = subprocess.run([sys.executable, str(script), str(so), enec.LIB_PATH], capture_output=True, text=True, timeout=60, cwd=ROOT)
        assert res.returncode == 0, res.stdout + res.stderr
        return json.loads(res.stdout.splitlines()[-1])

    return run


def test_a_search_on_a_capturing_stream_is_refused_with_nothing_enqueued(stand_in):
    got = stand_in("""
word("capturing").value = 1
rcs = {tune() for _ in range(50)}
during = word("launches").value, word("slots_held").value
word("capturing").value = 0
report(rcs=list(rcs), during=during, after=tune(), held=word("slots_held").value)
""")
    assert got == dict(rcs=[8], during=[0, 0], after=0, held=1)


def test_a_search_whose_launch_fails_gives_its_slot_back(stand_in):
    got = stand_in("""
word("launch_fails").value = 719
rcs = {tune() for _ in range(50)}
report(rcs=list(rcs), held=word("slots_held").value)
""")
    assert got == dict(rcs=[8], held=1)


def test_counts_that_are_wrong_twice_are_not_used(stand_in):
    """A kernel that ends without handing over, or whose counts don't add up to the elements: cleared and counted once more, and
    refused after that.  The slot is given back either way."""
    got = stand_in("""
word("wrong_syncs").value = 1
once = tune(), word("launches").value
word("wrong_syncs").value, word("launches").value = 2, 0
twice = tune(), word("launches").value
word("counted").value = 99999
short = {tune() for _ in range(50)}
word("counted").value = 100000
report(once=once, twice=twice, short=list(short), after=tune(), held=word("slots_held").value)
""")
    assert got == dict(once=[0, 3], twice=[8, 3], short=[8], after=0, held=1)


def test_slots_beyond_those_kept_are_freed_without_ending_a_capture_elsewhere(stand_in):
    """Nine calls at once hold nine slots; five of them are freed afterwards, in the mode that spares other threads' captures."""
    got = stand_in("""
word("gather").value = 9
threads = [threading.Thread(target=tune) for _ in range(9)]
for t in threads: t.start()
for t in threads: t.join()
report(most=word("slots_most").value, held=word("slots_held").value, unguarded=[word("mallocs_unguarded").value, word("frees_unguarded").value])
""")
    assert got == dict(most=9, held=4, unguarded=[0, 0])


DECOMPRESS = """
class Item(C.Structure): _fields_ = [("src", C.c_void_p), ("in_bytes", C.c_size_t), ("header", C.c_void_p), ("out", C.c_void_p), ("n", C.c_size_t), ("status", C.c_void_p)]
def decompress(streams, dtype=0):
    '''One call for streams of (elements, block size); the workgroups and the threads of its launches.'''
    items, keep = (Item * len(streams))(), []
    for it, (n, B) in zip(items, streams):
        nb = -(-n // B)
        h = struct.pack("<4sHBBQII4BIQ", b"ENEC", 1, dtype, 16, n, B, nb, 8, 5, 3, 5 if dtype == 1 else 8, 0, 1 << 40) + bytes(24)
        keep.append(C.create_string_buffer(h, 64))
        it.src, it.in_bytes, it.header, it.out, it.n = FAKE, 1 << 40, C.addressof(keep[-1]), FAKE, n
    word("launches").value = 0
    assert L.enec_decompress_batch(items, C.c_size_t(len(streams)), C.c_void_p(64)) == 0
    return launches()
"""


@pytest.mark.parametrize("dtype", [0, 1, 2])
def test_a_decompression_launch_has_the_threads_of_a_block_it_holds(stand_in, dtype):
    """Sixteen streams to a launch: the streams of the largest block size are in it first; of a smaller size as many join as make one
    launch less for that size, and only if they have few blocks."""
    got = stand_in(DECOMPRESS + f"""
d = {dtype}
norm, matrix, wide = (4096, 4096), (4 << 20, 16384), (17 << 15, 32768)
report(before=decompress([norm] * 20 + [matrix], d), after=decompress([matrix] + [norm] * 20, d),
       sixteen=decompress([norm] * 16 + [matrix], d), few=decompress([norm, matrix, norm], d), alone=decompress([norm] * 20, d),
       many=decompress([norm] * 3 + [matrix] * 18, d), three=decompress([norm] * 15 + [matrix] * 15 + [wide] * 2, d),
       long=decompress([(17 * 2048, 2048), (16 * 2048, 2048), matrix], d), rest=decompress([(17 * 2048, 2048)] + [(2048, 2048)] * 17 + [matrix], d),
       sizes=decompress([(2048, 2048), (4096, 4096), (8192, 8192)] * 13 + [(2048, 2048)], d), empty=decompress([(0, 2048), norm, (0, 16384)], d))
""")
    joined = [256 + 4, 16]
    assert got == dict(before=[joined, [256, 64]], after=[joined, [256, 64]], sixteen=[[256, 16], [256, 64]], few=[[258], [256]], alone=[[16, 4], [64, 64]],
                       many=[[16 * 256, 2 * 256 + 3], [256, 256]],
                       three=[[2 * 17, 15 * 256, 15], [512, 256, 64]],
                       long=[[17 + 16, 256], [64, 256]], rest=[[17 + 15, 256 + 2], [64, 256]], sizes=[[13, 13, 14], [128, 64, 64]], empty=[[1], [64]])


@pytest.mark.parametrize("dtype", [0, 1, 2])
def test_a_stream_alone_has_its_own_decompression_kernel(stand_in, dtype):
    """One for a launch of one stream, whatever its blocks, one for several of one block size, one for several block sizes."""
    got = stand_in(DECOMPRESS + f"""
def kernels(streams): return [(C.c_uint64 * 64).in_dll(rt, "fn")[i] for i in range(len(decompress(streams, {dtype})[0]))]
norm, matrix, wide = (4096, 4096), (4 << 20, 16384), (17 << 15, 32768)
one = [kernels([s]) for s in (norm, matrix, wide)]
same = [kernels([s] * n) for s in (norm, matrix) for n in (2, 3, 16)]
mixed = [kernels(s) for s in ([norm, matrix], [matrix, norm, norm])]
left = kernels([matrix] * 17)
report(one=one, same=same, mixed=mixed, left=left)
""")
    one, same, mixed = got["one"][0][0], got["same"][0][0], got["mixed"][0][0]
    assert len({one, same, mixed}) == 3
    assert got["one"] == [[one]] * 3 and got["same"] == [[same]] * 6 and got["left"] == [same, one]
    assert got["mixed"] == [[mixed]] * 2


COMPRESS = """
class Item(C.Structure): _fields_ = [("src", C.c_void_p), ("n", C.c_size_t), ("B", C.c_uint32), ("params", C.POINTER(P)), ("out", C.c_void_p), ("cap", C.c_size_t), ("out_bytes", C.c_void_p)]
big, small = P(122, 6, 3, 16), P(122, 5, 3, 16)
def compress(larges, smalls, big=big):
    items = (Item * (larges + smalls))()
    for i, it in enumerate(items):
        it.src = it.out = FAKE
        it.n, it.B, it.params = (32768, 16384, C.pointer(big)) if i < larges else (4096, 4096, C.pointer(small))
        it.cap = 1 << 30
    word("launches").value = 0
    assert L.enec_compress_batch(items, C.c_size_t(larges + smalls), 0, C.c_void_p(FAKE), C.c_size_t(1 << 20), C.c_void_p(64)) == 0
    return launches()
"""


def test_tensors_of_one_block_ride_along_where_there_is_room(stand_in):
    """They come on top of the grid of the first launch of default blocks: sixteen at most, fewer where its items leave less room
    among the arguments, none where it holds sixteen or its instance has not the code; the rest are launched together at the end."""
    got = stand_in(COMPRESS + """
report(layer=compress(7, 2), few=compress(1, 19), many=compress(12, 7), full=compress(16, 3), two=compress(17, 3), none=compress(0, 3),
       tuples=[compress(2, 2, P(100, n, m, 16))[0] for n, m in ((8, 7), (2, 1), (3, 2), (5, 5), (8, 4), (8, 5))],
       lengths=compress(2, 2, P(100, 6, 3, 8))[0])
""")
    assert got == dict(layer=[[16], [256]], few=[[2 + 16, 3], [256, 512]], many=[[24 + 5, 2], [256, 512]], full=[[32, 3], [256, 512]],
                       two=[[32, 2 + 3], [256, 256]], none=[[3], [512]],
                       tuples=[[4 + 2], [4, 2], [4 + 2], [4, 2], [4, 2], [4 + 2]], lengths=[4, 2])


def test_the_benchmark_knows_what_makes_one_launch(stand_in):
    """bench.py's compression calls make one launch each, as many of them as one call for all tensors makes, and no tensor is lost."""
    import random
    import bench
    from paper_2604_03298_amd import enec
    rng, cases, want = random.Random(5), [], []
    for k in range(60):
        tensors = []
        for _ in range(rng.choice([1, 3, 9, 20, 45])):
            n = rng.choice([100, 2048, 4096, 9000, 16384, 16385, 40000, 70000])
            width, m = rng.choice([(6, 3), (6, 4), (2, 1), (2, 2), (8, 0), (8, 7), (3, 2)])
            tensors.append((n, enec.default_block_size(n), (7, width, m, rng.choice([8, 16]))))
        blocks, nblocks = [b for _, b, _ in tensors], [-(-n // b) for n, b, _ in tensors]
        calls = bench.compression_calls([p for _, _, p in tensors], blocks, nblocks)
        assert sorted(i for g in calls for i in g) == list(range(len(tensors)))
        cases.append([tensors] + [[tensors[i] for i in g] for g in calls])
        want.append([1] * len(calls))
    got = stand_in(COMPRESS + f"""
def launches_of(tensors):
    items = (Item * len(tensors))()
    for it, (n, B, p) in zip(items, tensors):
        it.src = it.out = FAKE
        it.n, it.B, it.params, it.cap = n, B, C.pointer(P(*p)), 1 << 30
    word("launches").value = 0
    assert L.enec_compress_batch(items, C.c_size_t(len(tensors)), 0, C.c_void_p(FAKE), C.c_size_t(1 << 20), C.c_void_p(64)) == 0
    return word("launches").value
report(of=[[launches_of(t) for t in case] for case in {cases!r}])
""")["of"]
    assert [c[1:] for c in got] == want
    assert [c[0] for c in got] == [len(w) for w in want]


@pytest.mark.parametrize("count, slots", [(1, 4), (3, 4), (5, 16)])
def test_a_launch_for_tensors_of_one_block_passes_nothing_but_these(stand_in, count, slots):
    """The slots behind them are zero, whatever lay on the stack (an earlier call's tensors)."""
    got = stand_in(COMPRESS + f"""
compress(0, 4), compress(0, 16)
word("keep_bytes").value = {64 * slots}
grid = compress(0, {count})[0]
args = bytes((C.c_uint8 * 2048).in_dll(rt, "kept"))
report(grid=grid, used=[args[64 * i:64 * i + 64] != bytes(64) for i in range({slots})])
""")
    assert got == dict(grid=[count], used=[True] * count + [False] * (slots - count))


@pytest.mark.parametrize("per_block", [False, True])
def test_a_launch_passes_no_items_of_earlier_ones(stand_in, per_block):
    """Between a launch's items (88 bytes each, behind 40) and the tensors of one block at the end of the same 1408 bytes lie zeros."""
    got = stand_in(COMPRESS + f"""
class Tensor(C.Structure): _fields_ = [("src", C.c_void_p), ("n", C.c_size_t), ("B", C.c_uint32), ("out", C.c_void_p), ("cap", C.c_size_t), ("out_bytes", C.c_void_p)]
compress(16, 0)
word("keep_bytes").value = 1448
if {per_block}:
    items = (Tensor * 17)()
    for it in items: it.src, it.n, it.B, it.out, it.cap = FAKE, 32768, 16384, FAKE, 1 << 30
    assert L.enec_compress_per_block_batch(items, C.c_size_t(17), 0, 16, C.c_void_p(FAKE), C.c_size_t(1 << 20), C.c_void_p(64)) == 0
else:
    compress(1, 2)
args = bytes((C.c_uint8 * 2048).in_dll(rt, "kept"))
end = 1448 - (0 if {per_block} else 2 * 64)
report(first=args[40:48] != bytes(8), between=args[128:end] == bytes(end - 128), rest=args[end:end + 8] != bytes(8))
""")
    assert got == dict(first=True, between=True, rest=not per_block)
