"""Registers of the dense and the stream attention kernel, as the compiler reports them."""
import os
import re
import subprocess

from paper_2603_12201_amd import build


def test_dense_attention_registers_are_the_compilers_own():
    """Nothing is kept in registers the compiler does not know to be in use (it counts accumulation registers only where asm
    statements name them: this kernel's are all of one file), and nothing is spilled."""
    src = os.path.join(build.CSRC, "ic_sparse_attn.hip")
    p = subprocess.run(["hipcc"] + build.FLAGS + ["--offload-device-only", "-Rpass-analysis=kernel-resource-usage", "-S", src, "-o", os.devnull],
                       stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, check=True)
    seen = 0
    for name, body in re.findall(r"Function Name: (\S+)(.*?)(?=Function Name|\Z)", p.stdout, re.S):
        if "attn_dense_kernel" not in name:
            continue
        seen += 1
        use = {k: int(v) for k, v in re.findall(r"(AGPRs|VGPRs Spill|VGPRs|ScratchSize \[bytes/lane\]): (\d+)", body)}
        assert use["AGPRs"] == 0 and use["VGPRs Spill"] == 0 and use["ScratchSize [bytes/lane]"] == 0, (name, use)
        assert use["VGPRs"] <= 256, (name, use)
    assert seen == 2                              # contiguous and paged


def test_stream_attention_spills_no_vector_register():
    """The stream form works in the same 256 registers: a reload from scratch would wait behind the gathers in flight."""
    src = os.path.join(build.CSRC, "ic_sparse_attn.hip")
    p = subprocess.run(["hipcc"] + build.FLAGS + ["--offload-device-only", "-Rpass-analysis=kernel-resource-usage", "-S", src, "-o", os.devnull],
                       stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, check=True)
    seen = 0
    for name, body in re.findall(r"Function Name: (\S+)(.*?)(?=Function Name|\Z)", p.stdout, re.S):
        if "attn_stream_kernel" not in name:
            continue
        seen += 1
        use = {k: int(v) for k, v in re.findall(r"(AGPRs|VGPRs Spill|VGPRs|ScratchSize \[bytes/lane\]): (\d+)", body)}
        assert use["AGPRs"] == 0 and use["VGPRs Spill"] == 0 and use["ScratchSize [bytes/lane]"] == 0, (name, use)
        assert use["VGPRs"] <= 256, (name, use)
    assert seen == 6                              # one and several layers, contiguous and paged; rows left over; probabilities


def test_dense_attention_of_several_layers_spills_no_vector_register():
    src = os.path.join(build.CSRC, "ic_sparse_attn.hip")
    p = subprocess.run(["hipcc"] + build.FLAGS + ["--offload-device-only", "-Rpass-analysis=kernel-resource-usage", "-S", src, "-o", os.devnull],
                       stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, check=True)
    seen = 0
    for name, body in re.findall(r"Function Name: (\S+)(.*?)(?=Function Name|\Z)", p.stdout, re.S):
        if "attn_layers_dense_kernel" not in name:
            continue
        seen += 1
        use = {k: int(v) for k, v in re.findall(r"(AGPRs|VGPRs Spill|VGPRs|ScratchSize \[bytes/lane\]): (\d+)", body)}
        assert use["AGPRs"] == 0 and use["VGPRs Spill"] == 0 and use["ScratchSize [bytes/lane]"] == 0, (name, use)
        assert use["VGPRs"] <= 256, (name, use)
    assert seen == 2                              # contiguous and paged


def test_scalar_spills_stay_out_of_the_products(tmp_path):
    """Scalar registers that the attention kernels spill go to lanes of a vector register: between blocks and queries that costs
    nothing to speak of, in a loop with matrix products each way would take its place among them."""
    src, out = os.path.join(build.CSRC, "ic_sparse_attn.hip"), str(tmp_path / "attn.s")
    subprocess.run(["hipcc"] + build.FLAGS + ["--offload-device-only", "-S", src, "-o", out], stderr=subprocess.DEVNULL, check=True)
    seen = 0
    for name, body in re.findall(r"^(_ZN2ic\S*(?:dense|stream)_kernel[^:\n]*):[^\n]*\n(.*?)\n\.Lfunc_end", open(out).read(), re.S | re.M):
        seen += 1
        for block in re.split(r"\n(?=\.LBB|; %bb)", body):
            if block.count("v_mfma") >= 4:
                moves = len(re.findall(r"v_readlane|v_writelane", block))
                assert moves <= (2 if "dense_kernelILb1" in name else 0), (name, block.split("\n")[0], moves)
    assert seen == 10                             # dense: one layer and several, contiguous and paged; stream: six
