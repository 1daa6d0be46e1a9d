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
