"""Build libbmx.so (hand-written HIP for gfx950) in-tree with hipcc, and the native module of the
Python binding with the host compiler."""
import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
BUILD = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libbmx.so")
SOURCES = ["bmx_api.hip", "pack.hip", "gemm.hip", "gemm_mfma.hip", "gemm_fp4.hip", "gemm_block.hip", "gemm_i8.hip", "gemm_small.hip", "conv.hip", "conv_mfma.hip", "conv_one.hip", "conv_small.hip", "fc_small.hip", "probe.hip"]
HOST_BINDING = os.path.join(HERE, "_bmx_host.so")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
         # packed-fp32 VALU forms are kept out of generated code on the test machines
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         # host-pass errors inside kernel bodies are reported, not deferred (deferred, they leave the
         # kernel's host stub undefined without a word)
         "-fno-gpu-defer-diag",
         "-Wno-unused-command-line-argument"]


def _stale(out, deps):
    if not os.path.exists(out):
        return True
    t = os.path.getmtime(out)
    return any(os.path.getmtime(d) > t for d in deps)


def device_asm(src, folder=BUILD):
    """Path of the gfx950 assembly that -save-temps leaves next to the object of `src`."""
    return os.path.join(folder, os.path.splitext(src)[0] + "-hip-amdgcn-amd-amdhsa-gfx950.s")


def _isa_check():
    try:
        from . import isa_check
    except ImportError:  # run as a script
        sys.path.insert(0, HERE)
        import isa_check
    return isa_check


def current_asm(src):
    """device_asm(src), emitted alone if it is missing or older than the source (a fresh checkout)."""
    path, s = device_asm(src), os.path.join(CSRC, src)
    if _stale(path, [s]):
        os.makedirs(BUILD, exist_ok=True)
        subprocess.check_call([HIPCC] + FLAGS + ["-S", "--cuda-device-only", s, "-o", path],
                              stderr=subprocess.DEVNULL)
    return path


def check_scalar_loads():
    """Scan the compiled device code of every source for registers of an inline-asm scalar
    load that are touched while the load is still in flight (see isa_check.py; the kernels have
    no such load, the scan guards against one coming back)."""
    isa_check = _isa_check()
    for src in SOURCES:
        bad = isa_check.scan(current_asm(src))
        if bad:
            raise RuntimeError("in-flight scalar load hazard in %s:\n%s" % (src, isa_check.report(bad)))


def check_asm_hazards(asm=current_asm):
    """Scan the compiled device code of every source, asm(source), for wait states missing in front of or behind an
    instruction written as asm (isa_check.asm_hazards)."""
    isa_check = _isa_check()
    for src in SOURCES:
        bad = isa_check.asm_hazards(asm(src))
        if bad:
            raise RuntimeError("missing wait states in %s:\n%s" % (src, isa_check.report_hazards(bad)))


def check_codegen():
    """Properties of the generated code that a harmless-looking source change can lose without
    any test failing, only the clock: no kernel spills vector registers (the 64 x 64 tile of the
    register-operand matrix-core GEMM aside, which parks a dozen loop-invariant values); no
    kernel touches scratch memory (the same kernel and one convolution form of the popcount
    GEMM aside: a small array indexed at run time lands there, and every scratch access also
    waits for all stores issued before it, which cost the K-split GEMM 0.7 us per launch); and
    the convolution kernel with its filters in LDS reads each MFMA's filter operand with one
    ds_read_b128 (split into dword pairs, the rows meet four ways on the banks), holds one set of
    result stores for blocks inside the result and one for its edge, and spills no scalar registers
    (its instructions come from a cold cache at every launch); and the 64 x 64 per wave product kernel
    requests a segment at two places, ahead of its loop and in it, the last like any other (a place of its own for a row's
    last segment cost a launch up to 0.9 us), and undivided puts its packed words together with one
    v_writelane_b32 a half word (which the source reaches by the name of the compiler's intrinsic) and one store; no kernel calls a function."""
    import re
    isa_check = _isa_check()
    for src in SOURCES:
        for name, nbytes in isa_check.metadata(device_asm(src), "private_segment_fixed_size").items():
            known = "gemm_mfma_kernelILi2ELi2E" in name or "gemm_kernelILi16ELi32ELb0ELb0ELb1E" in name
            if nbytes and not known:
                raise RuntimeError("%s: kernel %s uses %d bytes of scratch memory per lane" % (src, name, nbytes))
        sgpr = isa_check.metadata(device_asm(src), "sgpr_spill_count")
        for name, (spills, ops) in isa_check.kernel_stats(device_asm(src)).items():
            allowed = 16 if "gemm_mfma_kernelILi2ELi2E" in name else 0
            if spills > allowed:
                raise RuntimeError("%s: kernel %s spills %d vector registers" % (src, name, spills))
            m = re.search(r"\d+gemm_fp4_kernelILi(\d+)ELb\dELi\dELb\dELb\dELb0ELb0E", name)
            if m and src == "gemm_fp4.hip" and ops["global_load_lds_dwordx4"] != 2 * 4 * (int(m.group(1)) + 1):
                raise RuntimeError("%s: kernel %s holds %d loads to LDS, expected two sets of them" % (src, name, ops["global_load_lds_dwordx4"]))
            if m and src == "gemm_fp4.hip" and "ILi1ELb1ELi2ELb0E" in name and (ops["v_writelane_b32"], ops["global_store_dwordx2"]) != (128, 1):
                raise RuntimeError("%s: kernel %s makes its packed words with %d v_writelane_b32 and %d stores, expected 128 and one" %
                                   (src, name, ops["v_writelane_b32"], ops["global_store_dwordx2"]))
            if any(op.startswith("s_swappc") for op in ops):
                raise RuntimeError("%s: kernel %s calls a function" % (src, name))
            m = re.search(r"conv_mfma_ws_kernelILi(\d+)ELi(\d+)E", name)
            if m and ops["ds_read_b128"] < int(m.group(1)) * int(m.group(2)):
                raise RuntimeError("%s: kernel %s reads its filter operands with %d ds_read_b128, "
                                   "expected %d" % (src, name, ops["ds_read_b128"],
                                                    int(m.group(1)) * int(m.group(2))))
            stores = ops["global_store_dword"]
            if m and stores > 32 * int(m.group(2)) + 8:
                raise RuntimeError("%s: kernel %s holds %d result stores, expected one set for blocks inside the "
                                   "result and one for its edge" % (src, name, stores))
            if m and m.group(2) == "1" and sgpr[name]:
                raise RuntimeError("%s: kernel %s spills %d scalar registers" % (src, name, sgpr[name]))


def build_host_binding():
    """Compile the native module of the Python calls (host code against PyTorch's C++ API; the
    library's entry points are found at import, in the libbmx.so that binding.py has loaded)."""
    import sysconfig
    import torch
    t = os.path.dirname(torch.__file__)
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-fvisibility=hidden", "-Wall", "-D__HIP_PLATFORM_AMD__=1",
           "-DUSE_ROCM=1", "-D_GLIBCXX_USE_CXX11_ABI=%d" % torch._C._GLIBCXX_USE_CXX11_ABI,
           "-isystem", os.path.join(t, "include"), "-isystem", "/opt/rocm/include",
           "-isystem", sysconfig.get_paths()["include"], os.path.join(CSRC, "host_binding.cpp"), "-o", HOST_BINDING,
           "-L" + os.path.join(t, "lib"), "-ltorch_python", "-ltorch_hip", "-ltorch_cpu", "-lc10_hip", "-lc10", "-Wl,-z,now"]
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    if r.returncode != 0:
        raise RuntimeError("g++ failed for host_binding.cpp:\n%s" % r.stdout)


def build(force=True, verbose=False):
    """Compile every translation unit, verify the hand-placed scalar loads in the generated
    code, and link the shared library.  Returns its path."""
    os.makedirs(BUILD, exist_ok=True)
    headers = [os.path.join(CSRC, f) for f in os.listdir(CSRC) if f.endswith((".h", ".hpp"))]
    headers.append(os.path.join(os.path.dirname(HERE), "include", "bmx.h"))

    def compile_one(src):
        s = os.path.join(CSRC, src)
        o = os.path.join(BUILD, src + ".o")
        if force or _stale(o, [s] + headers):
            cmd = [HIPCC] + FLAGS + ["-save-temps=obj", "-c", s, "-o", o]
            if verbose:
                print(" ".join(cmd), flush=True)
            r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
            if r.returncode != 0:
                raise RuntimeError("hipcc failed for %s:\n%s" % (src, r.stdout))
            warn = [l for l in r.stdout.splitlines() if "packed-fp32-ops" not in l and l.strip()]
            if verbose and warn:
                print("\n".join(warn))
        return o

    with ThreadPoolExecutor(max_workers=min(4, len(SOURCES))) as ex:
        objs = list(ex.map(compile_one, SOURCES))
    check_scalar_loads()
    check_asm_hazards()
    check_codegen()
    # (-z defs: an undefined symbol, e.g. a kernel stub the host pass dropped, fails the link here
    # instead of the first call)
    cmd = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-Wl,-z,defs"] + objs + ["-o", LIB]
    subprocess.check_call(cmd)
    if force or _stale(HOST_BINDING, [os.path.join(CSRC, "host_binding.cpp")] + headers):
        build_host_binding()
    return LIB


if __name__ == "__main__":
    print(build(force="--incremental" not in sys.argv, verbose=True))
