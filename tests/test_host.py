"""CPU-side checks of the boundary: the library loads and exports exactly what
include/qzo.h declares; host-only entry points behave; argument errors are
reported before anything touches a GPU."""
import ctypes as C
import os
import re
import shutil
import subprocess

import pytest

from paper_2505_13430_amd import binding as qb
from paper_2505_13430_amd import build as hip_build
from paper_2505_13430_amd import synth

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _declared():
    text = open(os.path.join(ROOT, "include", "qzo.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(qzo_[a-z0-9_]+)\s*\(", text)))


def test_library_exports_every_declared_symbol():
    lib = qb.lib()
    names = _declared()
    assert "qzo_step" in names and "qzo_dequant_gemm" in names and "qzo_forward_loss" in names
    assert "qzo_model_create" in names
    for n in names:
        assert hasattr(lib, n), n
    assert sorted(qb.EXPORTS) == names


LLVM = "/opt/rocm/llvm/bin/llvm-"


def _device_objects(tmp_path):
    """File names of the built library's code objects, extracted to tmp_path."""
    shutil.copy(hip_build.LIB, tmp_path / "lib.so")
    subprocess.run([LLVM + "objdump", "--offloading", "lib.so"], cwd=tmp_path, check=True, capture_output=True)
    bundles = [f for f in os.listdir(tmp_path) if "gfx950" in f]
    assert len(bundles) >= len(hip_build.SOURCES) - 1            # every source but the API's holds kernels
    return bundles


def _device_code(tmp_path):
    """Instructions of the built library's kernels: lists of (mnemonic, operands), a list per kernel."""
    kernels = []
    for f in _device_objects(tmp_path):
        text = subprocess.run([LLVM + "objdump", "-d", "--no-show-raw-insn", f], cwd=tmp_path, check=True, capture_output=True, text=True)
        for line in text.stdout.split("\n"):
            if re.match(r"[0-9a-f]+ <", line):
                kernels.append([])
            elif line.startswith("\t") and kernels:
                op, _, args = line.split("//")[0].strip().partition(" ")
                kernels[-1].append((op, [a.strip() for a in args.split(",")]))
    return kernels


def _scalars(args, file="s"):
    out = set()
    for a in args:
        for m in re.finditer(rf"(?<![a-z0-9_]){file}(?:(\d+)|\[(\d+):(\d+)\])", a):
            out |= set(range(int(m[2]), int(m[3]) + 1)) if m[2] else {int(m[1])}
    return out


def test_wait_states_of_direct_to_lds_loads(tmp_path):
    """The loads that write the LDS directly are asm, behind which the compiler inserts no wait states: one between a scalar
    write of M0 (the LDS address) and the load, five between a vector instruction that writes a scalar register and the load
    that reads it."""
    loads = 0
    for kernel in _device_code(tmp_path):
        for i, (op, args) in enumerate(kernel):
            if not (op.startswith("buffer_load") and args[-1].endswith(" lds")):
                continue
            loads += 1
            reads, states, j = _scalars(args), 0, i - 1
            while j >= 0 and states < 5:
                before, operands = kernel[j]
                assert not (states < 1 and operands[0] == "m0"), (i, op, args)
                assert not (before.startswith("v_") and _scalars(operands[:1]) & reads), (i, before, operands, args)
                states += int(operands[0]) + 1 if before == "s_nop" else 1
                j -= 1
    assert loads > 1000


def test_wait_states_of_accumulator_reads(tmp_path):
    """Kernels that hold accumulators in AGPRs read them with asm: twelve wait states behind a matrix instruction of eight
    passes that wrote the register (all that the library uses on AGPRs), and two between a vector instruction, asm among
    them, and the exchange between a wavefront's halves that reads its result."""
    def since(kernel, i, most, writes):
        states = 0
        for before, operands in reversed(kernel[max(0, i - most):i]):
            if writes(before, operands):
                return states
            states += int(operands[0]) + 1 if before == "s_nop" else 1
            if states >= most:
                break
        return most

    reads = swaps = 0
    for kernel in _device_code(tmp_path):
        for i, (op, args) in enumerate(kernel):
            if op.startswith("v_accvgpr_read"):
                acc, reads = _scalars(args[1:2], "a"), reads + 1
                assert since(kernel, i, 12, lambda o, a: "mfma" in o and _scalars(a[:1], "a") & acc) == 12, (i, args)
            elif op.startswith("v_permlane32_swap"):
                both, swaps = _scalars(args[:2], "v"), swaps + 1
                assert since(kernel, i, 2, lambda o, a: o.startswith("v_") and _scalars(a[:1], "v") & both) == 2, (i, args)
        assert not any("mfma" in op and "32x32x16" not in op and _scalars(args[:1], "a") for op, args in kernel)
    assert reads > 1000 and swaps > 1000


def test_kernels_with_counted_waits_do_not_spill(tmp_path):
    """Scratch memory is accessed by the counter of outstanding loads: a register spilled in a kernel whose waits leave a number of
    loads on their way empties that queue at every access."""
    seen = 0
    for f in _device_objects(tmp_path):
        notes = subprocess.run([LLVM + "readelf", "--notes", f], cwd=tmp_path, check=True, capture_output=True, text=True).stdout
        for kernel in re.split(r"^  - ", notes, flags=re.M):
            name = re.search(r"\.name: +(_Z\S+)", kernel)
            if name and re.search("few_gemm_kernel|w4_gemm_kernel|mid_gemm_kernel", name[1]):
                seen += 1
                assert re.search(r"\.vgpr_spill_count: +0$", kernel, flags=re.M), name[1]
    assert seen == 12 + 24 + 6          # tiles, passes, zero-points; tile heights, formats; widths, formats


def test_scale_count_is_table2(oracle):
    assert qb.qzo_model_scale_count(synth.SHAPES["llama-2-7b"]) == 50593792
    opt67 = dict(arch="opt", n_layers=32, d_model=4096, n_heads=32, d_ffn=16384, vocab=50272, max_seq=64)
    assert qb.qzo_model_scale_count(opt67) == 50331648
    for name in ("tiny", "tiny_opt", "opt-1.3b", "llama-2-13b"):
        assert qb.qzo_model_scale_count(synth.SHAPES[name]) == synth.n_scales(synth.SHAPES[name])


def test_config_errors_are_reported():
    bad = dict(synth.SHAPES["tiny"], d_model=200)
    with pytest.raises(qb.QzoError) as e:
        qb.qzo_model_scale_count(bad)
    assert e.value.status == qb.QZO_ERR_SHAPE and "128" in str(e.value)
    bad = dict(synth.SHAPES["tiny"], n_heads=16)      # head size 16
    with pytest.raises(qb.QzoError):
        qb.qzo_model_scale_count(bad)
    cfg = qb.make_config(synth.SHAPES["tiny"])
    cfg.struct_size = 4
    out = C.c_uint64(0)
    assert qb.lib().qzo_model_scale_count(C.byref(cfg), C.byref(out)) == qb.QZO_ERR_ARG
    # null pointers never reach a kernel
    assert qb.lib().qzo_dequant_gemm(None, None, None, 0, 1, 8, 128, 128, C.c_uint64(0),
                                     C.c_float(0), 1, None, None, None, C.c_uint64(0), None) == qb.QZO_ERR_ARG
    assert qb.lib().qzo_step(None, None, 1, 2, C.c_uint64(0), C.c_float(0), C.c_float(0),
                             C.c_float(1), None, C.c_uint64(0), None, None) == qb.QZO_ERR_ARG


@pytest.mark.parametrize("over,status", [
    (dict(x=None), qb.QZO_ERR_ARG), (dict(epi=1), qb.QZO_ERR_ARG), (dict(epi=32, rope=None), qb.QZO_ERR_ARG), (dict(y=24), qb.QZO_ERR_ALIGN),
    (dict(height=9), qb.QZO_ERR_ARG), (dict(passes=3), qb.QZO_ERR_ARG), (dict(epi=8), qb.QZO_ERR_ARG), (dict(epi=17, bias=16), qb.QZO_ERR_ARG),
    (dict(nf4=1, zp=16), qb.QZO_ERR_ARG), (dict(K=192), qb.QZO_ERR_SHAPE), (dict(N=388), qb.QZO_ERR_SHAPE), (dict(epi=16), qb.QZO_ERR_SHAPE),
    (dict(epi=32, N=256, dh=64), qb.QZO_ERR_SHAPE), (dict(epi=32, dh=128), qb.QZO_ERR_SHAPE), (dict(epi=32, dh=32), qb.QZO_ERR_SHAPE),
    (dict(epi=32, dh=64, S=0), qb.QZO_ERR_SHAPE), (dict(M=1 << 22), qb.QZO_ERR_SHAPE)])
def test_inspection_of_the_fused_linear_refuses(over, status):
    v = dict(x=16, zp=0, nf4=0, M=64, passes=1, N=384, K=128, epi=0, bias=0, rope=16, S=8, dh=128, height=0, y=16)
    v.update(over)
    p, u = (lambda k: C.c_void_p(v[k] or None)), (lambda k: C.c_uint32(v[k]))
    height = C.c_uint32(v["height"])
    assert qb.lib().qzo_debug_fused_linear(p("x"), C.c_void_p(16), C.c_void_p(16), p("zp"), C.c_int(v["nf4"]), C.c_uint32(0), u("M"),
                                           u("passes"), u("N"), u("K"), C.c_uint64(1), C.c_float(0), C.c_int(1), u("epi"), p("bias"),
                                           None, p("rope"), u("S"), u("dh"), C.byref(height), p("y"), None) == status


def test_counts_of_the_other_formats(oracle):
    tiny = synth.SHAPES["tiny"]
    n0 = qb.qzo_model_scale_count(tiny)
    # zero-points do not change the scales; NormalFloat-4 blocks of 64 double them; the codebook
    # format has one scale per quantized output row
    assert qb.qzo_model_scale_count(dict(tiny, quant=2)) == n0
    assert qb.qzo_model_scale_count(dict(tiny, quant=3, group=64)) == 2 * n0
    rows = tiny["n_layers"] * (5 * tiny["d_model"] + 2 * tiny["d_ffn"])      # qkv 3d, o d, gate+up 2F, down d
    assert qb.qzo_model_scale_count(dict(tiny, quant=1)) == rows
    with pytest.raises(qb.QzoError) as e:
        qb.qzo_model_scale_count(dict(tiny, quant=3))              # NormalFloat-4 needs group_size 64
    assert e.value.status == qb.QZO_ERR_SHAPE
    with pytest.raises(qb.QzoError):
        qb.qzo_model_scale_count(dict(tiny, quant=0, group=64))
    with pytest.raises(qb.QzoError) as e:
        qb.qzo_model_scale_count(dict(tiny, quant=4))
    assert e.value.status == qb.QZO_ERR_UNSUPPORTED
    with pytest.raises(qb.QzoError):
        qb.qzo_model_scale_count(dict(synth.SHAPES["tiny_opt"], quant=1))   # codebook: Llama family only


@pytest.mark.parametrize("name", ["tiny", "tiny_opt", "llama-2-7b"])
def test_dense_count_is_the_16_bit_part_of_the_table(oracle, name):
    sh = synth.SHAPES[name]
    d, F, V, L = sh["d_model"], sh["d_ffn"], sh["vocab"], sh["n_layers"]
    if sh["arch"] == "llama":
        want = 2 * V * d + L * 2 * d + d
    else:
        want = 2 * V * d + sh["max_seq"] * d + L * (4 * d + 3 * d + d + F + d) + 2 * d
    assert qb.qzo_model_dense_count(sh) == want
    assert qb.qzo_model_dense_count(dict(sh, quant=2)) == want
    if sh["arch"] == "llama":
        assert qb.qzo_model_dense_count(dict(sh, quant=1)) == want + L * 4 * 65536 * 8
    if name != "llama-2-7b":
        from oracle import oracle as O
        m = O.build_model(sh, synth.tensor_table(sh, 3))
        assert O.dense_master(m).size == want


class _Unbacked:
    """A tensor that host-only calls can be handed: an aligned address nothing reads, and a size in elements."""
    is_cuda = True

    def __init__(self, numel, element_size):
        self._n, self._e = numel, element_size

    def is_contiguous(self):
        return True

    def data_ptr(self):
        return 1 << 20

    def numel(self):
        return self._n

    def element_size(self):
        return self._e


def _host_model(shape):
    """A model handle without device memory (creating one is host work only): the int4 / NormalFloat-4 tables."""
    d, F, V = shape["d_model"], shape["d_ffn"], shape["vocab"]
    llama = shape["arch"] == "llama"

    def b16(n):
        return [_Unbacked(n, 2)]

    def weight(N, K):
        return [_Unbacked(N * K // 2, 1)] + ([_Unbacked(N * K // 128, 1)] if shape.get("quant") == 2 else [])

    table = b16(V * d) + ([] if llama else b16(shape["max_seq"] * d))
    for _ in range(shape["n_layers"]):
        if llama:
            table += b16(d) + weight(3 * d, d) + weight(d, d) + b16(d) + weight(2 * F, d) + weight(d, F)
        else:
            table += (b16(d) * 2 + weight(3 * d, d) + b16(3 * d) + weight(d, d) + b16(d) + b16(d) * 2 + weight(F, d) + b16(F) +
                      weight(d, F) + b16(d))
    table += b16(d) + ([] if llama else b16(d)) + b16(V * d)
    return qb.qzo_model_create(shape, table, _Unbacked(qb.qzo_model_scale_count(shape), 2))


@pytest.mark.parametrize("name,batch,seq,stacked", [
    # separate passes are the faster ones (time of the stacked step over theirs in brackets)
    ("llama-2-7b", 9, 57, False), ("llama-2-7b", 9, 128, False), ("llama-2-7b", 7, 512, False),      # 1.05, 1.06, 1.05
    ("llama-2-13b", 7, 256, False), ("opt-6.7b", 8, 65, False),                                     # 1.07, 1.16
    ("llama-2-13b", 8, 60, True),                                                                  # 0.89
    ("llama-2-7b", 6, 256, True), ("llama-2-13b", 5, 256, True),                                   # 0.93, 0.89
    ("opt-1.3b", 9, 64, True), ("opt-1.3b", 16, 256, True)])                                       # 0.73, 0.90
def test_nf4_passes_are_stacked_where_it_pays(name, batch, seq, stacked):
    """A NormalFloat-4 step beyond 512 tokens: both passes' expanded matrices lie in the workspace, or one."""
    shape = dict(synth.SHAPES["opt-1.3b"], d_model=4096, n_heads=32, d_ffn=16384) if name == "opt-6.7b" else synth.SHAPES[name]
    shape = dict(shape, n_layers=1, max_seq=512, quant=3, group=64)
    m = _host_model(shape)
    d, F, M1 = shape["d_model"], shape["d_ffn"], batch * seq
    widest = max(3 * d * d, (2 if shape["arch"] == "llama" else 1) * F * d)
    # activations of one pass; K-slice sums are at most one 256 x 256 fp32 tile per compute unit
    rows = M1 * (12 * d + 2 * F + 32 * -(-shape["vocab"] // 256)) + 4 * qb.qzo_model_scale_count(shape)
    extra = qb.qzo_workspace_bytes(m, batch, seq) - rows
    assert (extra > 4 * widest) == stacked, (extra / widest)
    if not stacked:
        assert extra < 2 * widest + 256 * 256 * 256 * 4 + (4 << 20)
    qb.qzo_model_destroy(m)


def test_nf4_workspace_holds_no_block_sums():
    """Up to 512 tokens a NormalFloat-4 workspace is activations, cross-entropy partials, the rotary table and K-slice sums,
    nothing for block sums (which only integer codes need)."""
    shape = dict(synth.SHAPES["tiny"], n_layers=1, d_model=128, n_heads=1, d_ffn=128 * 256, vocab=256, max_seq=64, quant=3, group=64)
    m = _host_model(shape)
    d, F, rows = 128, 128 * 256, 2 * 64                # both passes of 64 tokens
    # the largest sums: gate and up (2F rows, one group each: never cut)
    want = rows * (12 * d + 2 * F + 4 * 8 + 8) + 256 + 64 * 64 * 8 + 4 * rows * 2 * F
    assert qb.qzo_workspace_bytes(m, 1, 64) == want
    qb.qzo_model_destroy(m)


def test_few_token_passes_are_stacked_only_where_their_sums_fit():
    """33 to 64 int4 tokens: with millions of output rows the partial sums of both passes exceed the kernels' 32-bit
    offsets while those of one pass do not; such a step runs two forwards (its workspace holds 64 rows at 64 tokens
    as at the 32 whose passes are always stacked, not 128)."""
    for F, both in ((1 << 21, False), (1 << 16, True)):
        shape = dict(synth.SHAPES["tiny"], n_layers=1, d_model=128, n_heads=1, d_ffn=F, max_seq=64)
        m = _host_model(shape)
        ratio = qb.qzo_workspace_bytes(m, 1, 64) / qb.qzo_workspace_bytes(m, 1, 32)
        assert (ratio > 1.9) == both and (ratio < 1.1) == (not both), (F, ratio)
        qb.qzo_model_destroy(m)


def test_scratch_sizes_and_mode_switches():
    assert qb.qzo_nf4_scratch_bytes(512, 1024) >= 512 * 1024 * 2 + 512 * 16 * 4
    assert qb.qzo_int4_scratch_bytes(512, 1024) >= 512 * 1024 * 2 + 512 * 8 * 4
    assert qb.qzo_nf4_scratch_bytes(512, 1024) % 256 == 0
    with pytest.raises(qb.QzoError) as e:
        qb.qzo_model_set_int4_path(None, 1)                    # a field of a model: no model, no switch
    assert e.value.status == qb.QZO_ERR_ARG
    # scratch of a single perturbed linear: nothing for a many-tile call without the loss, one float per
    # tile with it, K-slice partial sums on the few-token path (at most 8 M N floats)
    assert qb.qzo_linear_scratch_bytes(2048, 11008, 4096, False) == 0
    assert 344 * 4 <= qb.qzo_linear_scratch_bytes(2048, 11008, 4096, True) <= 344 * 4 + 256
    few = qb.qzo_linear_scratch_bytes(16, 4096, 4096, False)
    assert 16 * 4096 * 4 <= few <= 8 * 16 * 4096 * 4 + 256 and few % 256 == 0
    assert qb.qzo_linear_scratch_bytes(0, 4096, 4096, True) == 0
    assert qb.qzo_codebook_scratch_bytes(300, 520, True) == 256 and qb.qzo_codebook_scratch_bytes(300, 520, False) == 0
    with pytest.raises(qb.QzoError):
        qb.qzo_linear_scratch_bytes(16, 4096, 100, False)
    tiny = synth.SHAPES["tiny"]
    assert qb.qzo_model_joint_table_bytes(tiny) >= (3 + 2 * tiny["n_layers"]) * 24
    with pytest.raises(qb.QzoError):
        qb.qzo_profile_stride(0)
    qb.qzo_profile_stride(1)
    # argument errors of the single-linear expand entry points are found on the host
    lib = qb.lib()
    assert lib.qzo_nf4_expand(None, None, 0, 8, 128, 64, C.c_uint64(0), C.c_float(0), 1, None, None, None) == qb.QZO_ERR_ARG
    assert lib.qzo_int4_expand(None, None, None, None, 0, 8, 128, 128, C.c_uint64(0), C.c_float(0), 1, None, None,
                               None) == qb.QZO_ERR_ARG
    assert lib.qzo_step_joint(None, None, 1, 2, C.c_uint64(0), C.c_float(0), C.c_float(0), C.c_float(0),
                              C.c_float(1), None, C.c_uint64(0), None, None) == qb.QZO_ERR_ARG
