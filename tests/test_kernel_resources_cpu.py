"""Compile-time properties of the hot kernels, checked without a GPU: the gfx950 code object
must keep the tiled and skinny GEMM kernels free of scratch spills (a spill in the K loop costs
~30 % on an MI355X) and inside the LDS and register budgets their launch configuration assumes."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"


@pytest.fixture(scope="module")
def asm(tmp_path_factory):
    if not os.path.exists(HIPCC):
        pytest.skip("hipcc not available")
    out = tmp_path_factory.mktemp("asm") / "fle_kernels.s"
    subprocess.check_call([HIPCC, "-O3", "--offload-arch=gfx950", "-std=c++17", "-I" + os.path.join(ROOT, "include"),
                           "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-S", "--cuda-device-only",
                           "-o", str(out), os.path.join(ROOT, "paper_2511_16964_amd", "csrc", "fle_kernels.hip")],
                          stderr=subprocess.DEVNULL)
    return out.read_text()


def kernel_props(asm):
    props = {}
    for m in re.finditer(r"\.amdhsa_kernel (\S+)(.*?)\.end_amdhsa_kernel", asm, flags=re.S):
        body = m.group(2)
        get = lambda key: int(re.search(r"\.amdhsa_%s (\d+)" % key, body).group(1))
        props[m.group(1)] = dict(lds=get("group_segment_fixed_size"), scratch=get("private_segment_fixed_size"),
                                 vgpr=get("next_free_vgpr"))
    return props


def test_hot_kernels_do_not_spill_and_fit_their_budgets(asm):
    props = kernel_props(asm)
    names = {k: v for k, v in props.items() if "gemm_bf16_skinny" in k or "gemm_tiled_" in k}
    assert len(names) == 17 + 20 + 24, sorted(props)   # skinny: 7 shapes x 2 dtypes and 3 K steps in fp32; tiled: 2 tiles x 4 dtypes (fp8 among them) x 2 epilogues, and the block-scaled fp8 form of each tile and epilogue; grouped: the same 4 dtypes plus the 128 tile with streamed W
    for name, p in names.items():
        assert p["scratch"] == 0, "%s spills %d bytes of scratch" % (name, p["scratch"])
        assert p["lds"] <= 160 * 1024, name
        assert p["vgpr"] <= 512, name
    for t128 in [v for k, v in names.items() if "tiled_128" in k or "grouped_128" in k]:
        assert t128["lds"] <= 80 * 1024 and t128["vgpr"] <= 256  # two workgroups per CU
    for t256 in [v for k, v in names.items() if "tiled_256" in k or "grouped_256" in k]:
        assert t256["lds"] == 160 * 1024


def test_deep_tiles_do_not_spill_and_fit_one_workgroup_per_cu(asm):
    deep = {k: v for k, v in kernel_props(asm).items() if "gemm_deep_" in k}
    assert len(deep) == 4 * 2 + 3 * 2, sorted(deep)   # bf16, fp16, fp8, block-scaled fp8 x two epilogues; grouped: without the block-scaled form
    for name, p in deep.items():
        assert p["scratch"] == 0 and p["vgpr"] <= 512 and p["lds"] <= 160 * 1024, (name, p)


def test_tiles_of_fewer_rows_do_not_spill(asm):
    rows = {k: v for k, v in kernel_props(asm).items() if "gemm_rows_256" in k}
    assert len(rows) == 2 * 2 * 3, sorted(rows)   # bf16, fp16 x two epilogues x 160, 192, 224 rows
    for name, p in rows.items():
        assert p["scratch"] == 0 and p["vgpr"] <= 512 and p["lds"] <= 160 * 1024, (name, p)


def test_no_accumulator_is_read_among_the_matrix_instructions(asm):
    """The 16x16 tiles' matrix instructions are inline assembly, whose wait states the compiler does not know: in a stretch of them no
    accumulator may be read out.  One body in a tile of fewer rows, four (64, 128, 192, 256 rows) in the grouped 256 tile."""
    for name, bodies in (("gemm_rows_256", 1), ("gemm_tiled_grouped_256", 4)):
        kernels = re.findall(r"^(_ZN3fle\d+%sILi[12]E\S*):(.*?)\.amdhsa_kernel" % name, asm, flags=re.S | re.M)
        assert len(kernels) == (12 if bodies == 1 else 4), [k for k, _ in kernels]
        for kernel, text in kernels:
            assert "scratch_" not in text, kernel
            stretches = 0
            for block in re.split(r"^\.LBB\S*:", text, flags=re.M):
                at = [m.start() for m in re.finditer(r"v_mfma_f32_16x16x32_", block)]
                if len(at) >= 16:
                    stretches += 1
                    assert "v_accvgpr_read" not in block[at[0]:at[-1]], kernel
            assert stretches >= bodies, (kernel, stretches)


def test_sums_scaled_in_place_wait_for_the_matrix_pipe(asm):
    """Attention over heads of 256 reads, scales and writes its accumulators in inline assembly.  24 states must pass in front of the first of
    these reads and behind the last write (a 32x32 product needs 19 and 2), with no matrix instruction between; outside of these stretches
    the steps move no sums out of the accumulation registers and back."""
    kernels = re.findall(r"^(_ZN3fle15flash_attentionILi[12]ELi256ELi1EEE\S*):(.*?)\.amdhsa_kernel", asm, flags=re.S | re.M)
    assert len(kernels) == 2
    for name, text in kernels:
        wait = r"\ts_nop 15\n\ts_nop 7\n"
        stretches = re.findall(wait + r"(.*?)" + wait, text, flags=re.S)
        assert len(re.findall(wait, text)) == 2 * len(stretches) and len(stretches) >= 2, name
        for s in stretches:
            assert s.count("v_accvgpr_read_b32") == 128 and s.count("v_accvgpr_write_b32") == 128 and "v_mfma" not in s, name
        left = re.sub(wait + r"(.*?)" + wait, "", text, flags=re.S)
        loops = [b for b in re.split(r"^\.LBB\S*:", left, flags=re.M) if b.count("v_mfma_f32_32x32x16") >= 48]
        assert loops, name
        for b in loops:   # (the scores of a block are read out once, for the maximum and the exponentials)
            assert b.count("v_accvgpr_write") <= 64, (name, b.count("v_accvgpr_write"))


def test_passes_that_hold_whole_rows_do_not_spill(asm):
    """LayerNorm of x in front of the product, a row in registers, and the row pass over short rows.  Waves per SIMD by registers: two and
    more up to 8 vectors a lane (fp32's converted values are the loaded ones), one with 16."""
    props = kernel_props(asm)
    rows = {k: v for k, v in props.items() if "ln_rowsI" in k}
    assert len(rows) == 3 * 2 * 7, sorted(rows)   # dtypes x whole or broken vectors x (a wave with 2, 4, 8; a workgroup with 2, 4, 8, 16)
    for name, p in rows.items():
        nv = int(re.search(r"ELi(\d+)ELb", name).group(1))
        assert p["scratch"] == 0 and p["vgpr"] <= {2: 128, 4: 168, 8: 256, 16: 512}[nv], (name, p)
    short = {k: v for k, v in props.items() if "finalize_shortI" in k}
    assert len(short) == 2 * 2 * 3 * 2, sorted(short)   # whole or broken rows x LayerNorm or softmax x dtypes x 1 or 2 vectors
    for name, p in short.items():
        assert p["scratch"] == 0 and p["vgpr"] <= 128, (name, p)


def test_counted_waits_cover_the_copies_of_a_step(asm):
    """The fp8 forms of the deep tile: loads land in the order of issue, and the wait in front of a K step's barrier leaves a fixed
    number of the youngest on their way.  The start's loads and the waits are read from the compiled kernel, the order of
    the steps is the source's; counted for 1 .. 12 steps, the copies of the next step have landed at every barrier."""
    stages = 4
    kernels = re.findall(r"^(_ZN3fle13gemm_deep_128ILi3ELb[01]ELb([01])E\S*):(.*?)\.amdhsa_kernel", asm, flags=re.S | re.M)
    assert len(kernels) == 4
    for name, scaled, body in kernels:
        copies, first = (9, 7) if scaled == "1" else (8, 6)   # of a wave and step, block scales included; those right behind the barrier
        start = body[:body.index("v_mfma")]
        loads = re.findall(r"\tbuffer_load_dword[^\n]*", start[:start.index("s_barrier")])
        assert all(" lds" in l for l in loads), (name, loads)     # nothing but copies in front of the first barrier ...
        sizes = ["x4" in l for l in loads]
        assert sizes == ([False] * (copies - 8) + [True] * 8) * (stages - 1), (name, loads)   # ... whole steps in turn
        loop = body[:body.rindex("v_mfma")]
        waits = [int(n) for n in re.findall(r"s_waitcnt vmcnt\((\d+)\) lgkmcnt\(0\)\n\ts_barrier", loop)][:5]   # loop, its last trip, then 3, 2 and 1 steps left
        first_wait = int(re.search(r"s_waitcnt vmcnt\((\d+)\)", start[start.index(" lds"):]).group(1))
        assert all(" lds" in l for l in re.findall(r"\tbuffer_load[^\n]*", loop)), name   # no load into registers stands among the copies
        for steps in range(1, 13):
            queue = [j for j in range(min(steps, stages - 1)) for _ in range(copies)]   # the step of each copy
            landed = len(queue) - (first_wait if steps >= stages - 1 else 0)
            assert 0 not in queue[landed:], (name, steps)
            queue += [stages - 1] * (first if steps >= stages else 0)
            for step in range(steps - 1):
                left = steps - 1 - step
                queue += [step + stages - 1] * (copies - first if left >= stages - 1 else 0)
                landed = max(landed, len(queue) - waits[0 if left > stages else 5 - min(left, stages)])
                assert step + 1 not in queue[landed:] and queue.count(step + 1) == copies, (name, steps, step)
                queue += [step + stages] * (first if left >= stages else 0)


def test_thin_kernels_do_not_spill(asm):
    props = kernel_props(asm)
    thin = {k: v for k, v in props.items() if "gemm_thin" in k or "gemm_gemv" in k}
    assert len(thin) == 6 + 13 + 12, sorted(thin)   # MFMA form: 3 dtypes x 2 row counts; dot-product form: 1, 2, 4 rows and the 16-wave form x 3 dtypes, 8 rows in fp32; the same again, up to 4 rows, with the LayerNorm of x folded in
    for name, p in thin.items():
        assert p["scratch"] == 0 and p["vgpr"] <= 256, (name, p)   # at least two waves per SIMD


def test_kernels_that_normalise_x_first_do_not_spill(asm):
    norm = {k: v for k, v in kernel_props(asm).items() if "norm_dot" in k}
    assert len(norm) == 9, sorted(norm)   # 3 dtypes x (16 waves; one and two rows)
    for name, p in norm.items():
        assert p["scratch"] == 0 and p["vgpr"] <= (128 if "Li1EEEv" in name else 256) and p["lds"] <= 80 * 1024, (name, p)


def test_attention_kernels_keep_two_waves_per_simd(asm):
    props = kernel_props(asm)
    att = {k: v for k, v in props.items() if "flash_attention" in k}
    assert len(att) == 8, sorted(att)   # bf16 / fp16 x head dimension 32 / 64 / 128 / 256
    for name, p in att.items():
        assert p["scratch"] == 0, (name, p)
        if "Li256ELi1E" in name:        # head dimension 256: one wave per SIMD, one workgroup per CU
            assert p["vgpr"] <= 512 and p["lds"] == 128 * 1024, (name, p)
        else:
            assert p["vgpr"] <= 256 and p["lds"] <= 64 * 1024, (name, p)
    assert "ds_read_b64_tr_b16" in asm   # V is transposed by the LDS read itself


def test_chain_kernel_leaves_room_for_all_workgroups(asm):
    """The persistent perceptron kernel waits at a grid barrier, so every workgroup must be resident: a CU holds 16 waves of
    at most 128 registers and next to no LDS, the one workgroup per CU that the launch asks for."""
    props = kernel_props(asm)
    chain = {k: v for k, v in props.items() if "mlp_chain" in k}
    assert len(chain) == 5, sorted(chain)   # three dtypes, and bf16 / fp16 weights under fp32 activations
    for name, p in chain.items():
        # (the only LDS is the few words through which a workgroup agrees on whether its barrier wait was given up)
        assert p["scratch"] == 0 and p["vgpr"] <= 128 and p["lds"] <= 1024, (name, p)
    assert "buffer_wbl2" not in asm and "buffer_inv" not in asm   # no kernel flushes or invalidates a cache


def test_perceptron_in_lds_leaves_room_for_its_workgroup(asm):
    """It waits at the same grid barrier, one workgroup of 16 waves per CU: four waves per SIMD, so 128 registers each."""
    chain = {k: v for k, v in kernel_props(asm).items() if "perceptron_lds" in k}
    assert len(chain) == 10, sorted(chain)   # the five combinations of dtypes, 8 and 16 KB ahead
    for name, p in chain.items():
        assert p["scratch"] == 0 and p["vgpr"] <= 128 and p["lds"] <= 80 * 1024, (name, p)


def test_decode_attention_keeps_its_workgroups_per_cu(asm):
    """Two workgroups per CU (four at head dimension 32) by LDS (160 KB) and by registers (512 per lane of a SIMD)."""
    props = kernel_props(asm)
    for D, waves, per_cu in ((32, 4, 4), (64, 4, 2), (128, 2, 2), (256, 1, 2)):
        found = {k: v for k, v in props.items() if "decode_attentionI" in k and "Li%dEEE" % D in k}
        assert len(found) == 2, sorted(found)   # bf16, fp16
        for name, p in found.items():
            per_simd = (waves * per_cu + 3) // 4
            assert p["scratch"] == 0 and p["lds"] * per_cu <= 160 * 1024 and (p["vgpr"] + 7) // 8 * 8 * per_simd <= 512, (name, p)
    combine = [v for k, v in props.items() if "decode_combine" in k]
    assert len(combine) == 8 and all(v["scratch"] == 0 and v["vgpr"] <= 64 for v in combine), combine


def test_split_reduction_with_a_row_reduction_does_not_spill(asm):
    red = {k: v for k, v in kernel_props(asm).items() if "reduce_rows" in k}
    assert len(red) == 9, sorted(red)   # 3 dtypes x 3 widths
    for name, p in red.items():
        assert p["scratch"] == 0 and p["vgpr"] <= 128, (name, p)   # (16 waves: four per SIMD)


def test_ragged_row_passes_do_not_spill(asm):
    """Streaming passes over memory: at least three waves per SIMD for the row pass, six for the copies."""
    props = kernel_props(asm)
    fin = {k: v for k, v in props.items() if "finalize_rowsILb0" in k}
    assert len(fin) == 6 and all(v["scratch"] == 0 and v["vgpr"] <= 168 for v in fin.values()), fin
    copies = [v for k, v in props.items() if "copy_rows" in k]
    assert len(copies) == 2 and all(v["scratch"] == 0 and v["vgpr"] <= 80 for v in copies), copies


def test_chain_kernels_tell_the_compiler_that_their_barriers_order_lds():
    """The barrier builtin counts as no memory access: a raw one lets the compiler move LDS reads and writes across it."""
    text = open(os.path.join(ROOT, "paper_2511_16964_amd", "csrc", "fle_chain.h")).read()
    raw = [m.start() for m in re.finditer(r"__builtin_amdgcn_s_barrier\(\)", text)]
    assert raw
    for at in raw:
        body = text[text.rindex("{\n", 0, at):text.index("\n}\n", at)]
        before, after = body.split("__builtin_amdgcn_s_barrier();")
        clobber = 'asm volatile("" ::: "memory");'
        assert before.count(clobber) == 1 and after.count(clobber) == 1, body


def test_streaming_finalize_keeps_its_occupancy(asm):
    """The LayerNorm finalize pass is a streaming kernel: it needs several waves per SIMD, so its register count
    must stay bounded (a shared code path once pushed it to 149 and cost 40 % of its speed; holding a whole item's
    loads as one batch takes 116, four waves per SIMD, and measured faster than 79 with the loads one by one)."""
    props = kernel_props(asm)
    ln = [v for k, v in props.items() if "finalize_rowsILb1ELb1" in k]
    assert len(ln) == 3 and all(v["vgpr"] <= 128 and v["scratch"] == 0 for v in ln), ln   # one per storage dtype


def test_main_loop_uses_the_intended_instructions(asm):
    body = asm
    assert re.search(r"buffer_load_dwordx4 .* lds", body)          # direct-to-LDS copies
    assert "v_mfma_f32_16x16x4_f32" in asm                         # fp32 path stays on fp32 MFMA
    m = re.search(r"^_ZN3fle14gemm_tiled_256ILi0ELb0ELi32ELin1ELb0EEEvNS_8GemmArgsE:(.*?)s_endpgm", asm, flags=re.S | re.M)   # fp32 operands
    assert m and "v_mfma_f32_32x32x2_f32" in m.group(1) and "_bf16" not in m.group(1) and "x16_f16" not in m.group(1) and "x32_f16" not in m.group(1)
    # 2-byte operands: the tiled loop runs on the 16x16x32 shape, whose accumulators stay where they are (no
    # accumulator moves between register files inside the K loop) and nothing spills
    for dt, mn in ((1, "v_mfma_f32_16x16x32_bf16"), (2, "v_mfma_f32_16x16x32_f16")):
        for kern in ("gemm_tiled_256", "gemm_tiled_128"):
            m = re.search(r"^_ZN3fle14%sILi%dELb0ELi16ELin1ELb0EEEvNS_8GemmArgsE:(.*?)s_endpgm" % (kern, dt), asm, flags=re.S | re.M)
            assert m, (kern, dt)
            text = m.group(1)
            first, last = text.index(mn), text.rindex(mn)
            assert text.count(mn) >= 128 and "32x32x16" not in text
            # (the only accumulator moves allowed between the matrix instructions are the one-time zero fill,
            # which the compiler places between its copies of the K step)
            assert text[first:last].count("v_accvgpr") <= 256 and "v_accvgpr_read" not in text[first:last] and "scratch_" not in text
    assert "v_mfma_f32_16x16x16_bf16" in asm and "v_mfma_f32_16x16x16_f16" in asm   # general kernel on 2-byte operands
    assert "v_pk_fma_f32" not in asm and "v_pk_mul_f32" not in asm and "v_pk_add_f32" not in asm
