"""The library's kernels on the CPU, for tests: build() compiles them for it, and as a pytest plugin (-p emulated_gpu) this
module makes GPU tests run on the result: device tensors are host memory, streams and events are over at once."""
import contextlib
import ctypes as C
import os
import re
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
PACKAGE = os.path.join(os.path.dirname(os.path.dirname(HERE)), "paper_1910_10032_amd")


def _converted(sources: dict) -> dict:
    """The sources without what only the device's compiler takes.  Every rule has to find its places: a function that is
    renamed or rewritten stops this, and does not quietly go untested."""
    def put(pattern, by, places=None):
        found = 0
        for name, s in sources.items():
            sources[name], n = re.subn(pattern, by, s)
            found += n
        if found != places if places else found == 0:
            raise RuntimeError(f"{pattern}: found {found} times, expected {places or 'some'}")

    put(r'asm volatile\("s_getreg_b32 %0, hwreg\(HW_REG_XCC_ID\)" : "=s"\(xcc\)\);', "xcc = 0;", 2)
    put(r'asm volatile\("s_mov_b32 m0[^;]*;', "(void)*(const volatile uint32_t *)p;", 1)              # a load without a target
    put(r'asm volatile\((?:[^()"]|"[^"]*"|\([^()]*\))*\);', ";")                                     # waits, and what is hidden from the compiler
    put(r"__attribute__\(\((address_space|amdgpu_num_vgpr)\(\d+\)\)\)", "")
    # what the lanes that happen to be here do together (the last argument: which of these places)
    put(r"const unsigned long long m = __ballot\(1\);", "const unsigned long long m = ballot_here(1, counter);", 1)
    put(r"__builtin_amdgcn_readlane\(\(int\)base, leader\)", "readlane_here(base, leader, counter)", 1)
    put(r"m_all = __ballot\(1\), m_new = __ballot\(!dup\);", "m_all = ballot_here(1, &queue), m_new = ballot_here(!dup, &slots);", 1)
    put(r"__shfl\(base, leader, 64\)", "readlane_here(base, leader, &queue)", 1)
    for name, s in sources.items():
        for left in ("asm volatile(", "__attribute__((a", "__ballot(1)"):
            if left in s:
                raise RuntimeError(f"{name}: {left} is not converted")
    return sources


def build(folder: str) -> str:
    """Compile copies of the sources, without the machine code in them, into a library in `folder`."""
    os.makedirs(os.path.join(folder, "package", "csrc"), exist_ok=True)
    os.makedirs(os.path.join(folder, "include"), exist_ok=True)
    header = os.path.join(os.path.dirname(PACKAGE), "include", "wfst_decode.h")
    with open(header) as f, open(os.path.join(folder, "include", "wfst_decode.h"), "w") as g:
        g.write(f.read())
    sources = {}
    for name in os.listdir(os.path.join(PACKAGE, "csrc")):
        with open(os.path.join(PACKAGE, "csrc", name)) as f:
            sources[name] = f.read()
    for name, s in _converted(sources).items():
        with open(os.path.join(folder, "package", "csrc", name), "w") as g:
            g.write(s)
    out = os.path.join(folder, "libemulated.so")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-fPIC", "-shared", "-ffp-contract=off", "-fno-strict-aliasing", "-w", "-I" + HERE, "-x", "c++",
                           os.path.join(folder, "package", "csrc", "wfst_decode.hip"), os.path.join(HERE, "workgroup.cpp"), "-o", out, "-lpthread"])
    return out


def _install(path):
    import torch
    load = C.CDLL
    lib = load(path)
    lib.emulated_alloc.restype, lib.emulated_alloc.argtypes = C.c_void_p, [C.c_size_t]
    C.CDLL = lambda p, *a, **k: load(path if "_libwfst_decode" in str(p) else p, *a, **k)

    def on_device(t):
        t = t.contiguous()
        if t.numel() == 0:
            return t
        n = t.numel() * t.element_size()
        return torch.frombuffer((C.c_uint8 * n).from_address(lib.emulated_alloc(n)), dtype=t.dtype).view(t.shape).copy_(t)

    def made_on_device(make):
        def f(*a, device=None, **k):
            return on_device(make(*a, **k)) if "cuda" in str(device) else make(*a, **k)
        return f

    class Done:                                   # a stream or an event
        cuda_stream = 0

        def __init__(self, *a, **k):
            pass

        def query(self):
            return True

        def synchronize(self, *a):
            pass

        record = wait_stream = synchronize

    torch.Tensor.cuda = lambda self, *a, **k: on_device(self)
    torch.Tensor.is_cuda = property(lambda self: True)
    for name in ("empty", "zeros", "full"):
        setattr(torch, name, made_on_device(getattr(torch, name)))
    torch.cuda.is_available = lambda: True
    torch.cuda.synchronize = torch.cuda.set_device = lambda *a: None
    torch.cuda.current_stream = lambda *a: Done()
    torch.cuda.Stream = torch.cuda.Event = Done
    torch.cuda.stream = lambda s: contextlib.nullcontext()


if os.environ.get("EMULATED_LIBRARY"):
    _install(os.environ["EMULATED_LIBRARY"])
