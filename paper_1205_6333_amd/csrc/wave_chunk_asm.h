// wave_chunk_asm.h -- generated by gen_sym_chunk.py; do not edit.
// One chunk of the wave-symmetric kernel in gfx950 assembly (see the
// generator's docstring for what it computes and the register map).
#pragma once

// one chunk; 1321 instructions per chunk, 0 products with same-parity sources
#define SD_WAVE_CHUNK_RPY_FREE \
    "ds_read_b32 v59, v31 offset:0\n" \
    "ds_read_b32 v61, v31 offset:128\n" \
    "ds_read_b32 v63, v31 offset:256\n" \
    "ds_read_b32 v65, v31 offset:4\n" \
    "ds_read_b32 v67, v31 offset:132\n" \
    "ds_read_b32 v69, v31 offset:260\n" \
    "ds_read_b32 v76, v31 offset:384\n" \
    "ds_read_b32 v78, v31 offset:512\n" \
    "ds_read_b32 v80, v31 offset:640\n" \
    "ds_read_b32 v82, v31 offset:388\n" \
    "ds_read_b32 v84, v31 offset:516\n" \
    "ds_read_b32 v86, v31 offset:644\n" \
    "s_waitcnt lgkmcnt(9)\n" \
    "v_sub_f32 v71, v24, v59\n" \
    "v_sub_f32 v73, v26, v61\n" \
    "v_sub_f32 v75, v28, v63\n" \
    "v_sub_f32 v77, v30, v59\n" \
    "v_sub_f32 v79, v32, v61\n" \
    "v_sub_f32 v81, v34, v63\n" \
    "v_mul_f32 v95, v75, v75\n" \
    "v_fmac_f32 v95, v73, v73\n" \
    "v_fmac_f32 v95, v71, v71\n" \
    "v_mul_f32 v88, v81, v81\n" \
    "v_fmac_f32 v88, v79, v79\n" \
    "v_fmac_f32 v88, v77, v77\n" \
    "v_min_f32 v99, v95, v88\n" \
    "s_waitcnt lgkmcnt(6)\n" \
    "v_sub_f32 v83, v24, v65\n" \
    "v_sub_f32 v85, v26, v67\n" \
    "v_sub_f32 v87, v28, v69\n" \
    "v_sub_f32 v89, v30, v65\n" \
    "v_sub_f32 v91, v32, v67\n" \
    "v_sub_f32 v93, v34, v69\n" \
    "v_mul_f32 v97, v87, v87\n" \
    "v_fmac_f32 v97, v85, v85\n" \
    "v_fmac_f32 v97, v83, v83\n" \
    "v_mul_f32 v90, v93, v93\n" \
    "v_fmac_f32 v90, v91, v91\n" \
    "v_fmac_f32 v90, v89, v89\n" \
    "v_min_f32 v92, v97, v90\n" \
    "v_min_f32 v99, v99, v92\n" \
    "v_cmp_lt_f32 vcc, v99, v50\n" \
    "s_waitcnt lgkmcnt(0)\n" \
    "v_mul_f32 v111, v75, v80\n" \
    "v_fmac_f32 v111, v73, v78\n" \
    "v_fmac_f32 v111, v71, v76\n" \
    "v_mul_f32 v113, v75, v40\n" \
    "v_fmac_f32 v113, v73, v38\n" \
    "v_fmac_f32 v113, v71, v36\n" \
    "v_mul_f32 v121, v81, v80\n" \
    "v_fmac_f32 v121, v79, v78\n" \
    "v_fmac_f32 v121, v77, v76\n" \
    "v_mul_f32 v123, v81, v46\n" \
    "v_fmac_f32 v123, v79, v44\n" \
    "v_fmac_f32 v123, v77, v42\n" \
    "s_cbranch_vccz SD_SKIP0_%=\n" \
    "s_or_b64 %[nl], %[nl], vcc\n" \
    "v_cmp_lt_f32 vcc, v95, v50\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v95, v95, v27, vcc\n" \
    "v_cmp_lt_f32 vcc, v88, v25\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v88, v88, v27, vcc\n" \
    "v_cmp_lt_f32 vcc, v97, v50\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v97, v97, v27, vcc\n" \
    "v_cmp_lt_f32 vcc, v90, v25\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v90, v90, v27, vcc\n" \
    "SD_SKIP0_%=:\n" \
    "v_rsq_f32 v105, v95\n" \
    "v_rsq_f32 v115, v88\n" \
    "v_mul_f32 v94, v105, v105\n" \
    "v_mul_f32 v104, v115, v115\n" \
    "v_mul_f32 v107, v94, v105\n" \
    "v_mul_f32 v117, v104, v115\n" \
    "v_fma_f32 v109, v48, v107, v105\n" \
    "v_fma_f32 v96, v29, v94, 1.0\n" \
    "v_fma_f32 v119, v48, v117, v115\n" \
    "v_fma_f32 v106, v29, v104, 1.0\n" \
    "v_mul_f32 v98, v107, v96\n" \
    "v_mul_f32 v100, v98, v111\n" \
    "v_mul_f32 v102, v98, v113\n" \
    "v_mul_f32 v108, v117, v106\n" \
    "v_mul_f32 v110, v108, v121\n" \
    "v_mul_f32 v112, v108, v123\n" \
    "v_mul_f32 v52, v100, v71\n" \
    "v_fmac_f32 v52, v109, v76\n" \
    "v_mul_f32 v54, v100, v73\n" \
    "v_fmac_f32 v54, v109, v78\n" \
    "v_mul_f32 v56, v100, v75\n" \
    "v_fmac_f32 v56, v109, v80\n" \
    "v_mul_f32 v58, v110, v77\n" \
    "v_fmac_f32 v58, v119, v76\n" \
    "v_mul_f32 v60, v110, v79\n" \
    "v_fmac_f32 v60, v119, v78\n" \
    "v_mul_f32 v62, v110, v81\n" \
    "v_fmac_f32 v62, v119, v80\n" \
    "v_mul_f32 v53, v102, v71\n" \
    "v_fmac_f32 v53, v109, v36\n" \
    "v_mul_f32 v55, v102, v73\n" \
    "v_fmac_f32 v55, v109, v38\n" \
    "v_mul_f32 v57, v102, v75\n" \
    "v_fmac_f32 v57, v109, v40\n" \
    "v_fmac_f32 v53, v112, v77\n" \
    "v_fmac_f32 v53, v119, v42\n" \
    "v_fmac_f32 v55, v112, v79\n" \
    "v_fmac_f32 v55, v119, v44\n" \
    "v_fmac_f32 v57, v112, v81\n" \
    "v_fmac_f32 v57, v119, v46\n" \
    "v_rsq_f32 v105, v97\n" \
    "v_rsq_f32 v115, v90\n" \
    "v_mul_f32 v111, v87, v86\n" \
    "v_fmac_f32 v111, v85, v84\n" \
    "v_fmac_f32 v111, v83, v82\n" \
    "v_mul_f32 v113, v87, v40\n" \
    "v_fmac_f32 v113, v85, v38\n" \
    "v_fmac_f32 v113, v83, v36\n" \
    "v_mul_f32 v121, v93, v86\n" \
    "v_fmac_f32 v121, v91, v84\n" \
    "v_fmac_f32 v121, v89, v82\n" \
    "v_mul_f32 v123, v93, v46\n" \
    "v_fmac_f32 v123, v91, v44\n" \
    "v_fmac_f32 v123, v89, v42\n" \
    "v_mul_f32 v94, v105, v105\n" \
    "v_mul_f32 v104, v115, v115\n" \
    "v_mul_f32 v107, v94, v105\n" \
    "v_mul_f32 v117, v104, v115\n" \
    "v_fma_f32 v109, v48, v107, v105\n" \
    "v_fma_f32 v96, v29, v94, 1.0\n" \
    "v_fma_f32 v119, v48, v117, v115\n" \
    "v_fma_f32 v106, v29, v104, 1.0\n" \
    "v_mul_f32 v98, v107, v96\n" \
    "v_mul_f32 v100, v98, v111\n" \
    "v_mul_f32 v102, v98, v113\n" \
    "v_mul_f32 v108, v117, v106\n" \
    "v_mul_f32 v110, v108, v121\n" \
    "v_mul_f32 v112, v108, v123\n" \
    "v_fmac_f32 v52, v100, v83\n" \
    "v_fmac_f32 v52, v109, v82\n" \
    "v_fmac_f32 v54, v100, v85\n" \
    "v_fmac_f32 v54, v109, v84\n" \
    "v_fmac_f32 v56, v100, v87\n" \
    "v_fmac_f32 v56, v109, v86\n" \
    "v_fmac_f32 v58, v110, v89\n" \
    "v_fmac_f32 v58, v119, v82\n" \
    "v_fmac_f32 v60, v110, v91\n" \
    "v_fmac_f32 v60, v119, v84\n" \
    "v_fmac_f32 v62, v110, v93\n" \
    "v_fmac_f32 v62, v119, v86\n" \
    "v_mul_f32 v120, v102, v83\n" \
    "v_fmac_f32 v120, v109, v36\n" \
    "v_mul_f32 v122, v102, v85\n" \
    "v_fmac_f32 v122, v109, v38\n" \
    "v_mul_f32 v124, v102, v87\n" \
    "v_fmac_f32 v124, v109, v40\n" \
    "v_fmac_f32 v120, v112, v89\n" \
    "v_fmac_f32 v120, v119, v42\n" \
    "v_fmac_f32 v122, v112, v91\n" \
    "v_fmac_f32 v122, v119, v44\n" \
    "v_fmac_f32 v124, v112, v93\n" \
    "v_fmac_f32 v124, v119, v46\n" \
    "ds_read_b32 v59, v31 offset:8\n" \
    "ds_read_b32 v61, v31 offset:136\n" \
    "ds_read_b32 v63, v31 offset:264\n" \
    "ds_read_b32 v65, v31 offset:12\n" \
    "ds_read_b32 v67, v31 offset:140\n" \
    "ds_read_b32 v69, v31 offset:268\n" \
    "ds_read_b32 v76, v31 offset:392\n" \
    "ds_read_b32 v78, v31 offset:520\n" \
    "ds_read_b32 v80, v31 offset:648\n" \
    "ds_read_b32 v82, v31 offset:396\n" \
    "ds_read_b32 v84, v31 offset:524\n" \
    "ds_read_b32 v86, v31 offset:652\n" \
    "s_waitcnt lgkmcnt(9)\n" \
    "v_sub_f32 v71, v24, v59\n" \
    "v_sub_f32 v73, v26, v61\n" \
    "v_sub_f32 v75, v28, v63\n" \
    "v_sub_f32 v77, v30, v59\n" \
    "v_sub_f32 v79, v32, v61\n" \
    "v_sub_f32 v81, v34, v63\n" \
    "v_mul_f32 v95, v75, v75\n" \
    "v_fmac_f32 v95, v73, v73\n" \
    "v_fmac_f32 v95, v71, v71\n" \
    "v_mul_f32 v88, v81, v81\n" \
    "v_fmac_f32 v88, v79, v79\n" \
    "v_fmac_f32 v88, v77, v77\n" \
    "v_min_f32 v99, v95, v88\n" \
    "s_waitcnt lgkmcnt(6)\n" \
    "v_sub_f32 v83, v24, v65\n" \
    "v_sub_f32 v85, v26, v67\n" \
    "v_sub_f32 v87, v28, v69\n" \
    "v_sub_f32 v89, v30, v65\n" \
    "v_sub_f32 v91, v32, v67\n" \
    "v_sub_f32 v93, v34, v69\n" \
    "v_mul_f32 v97, v87, v87\n" \
    "v_fmac_f32 v97, v85, v85\n" \
    "v_fmac_f32 v97, v83, v83\n" \
    "v_mul_f32 v90, v93, v93\n" \
    "v_fmac_f32 v90, v91, v91\n" \
    "v_fmac_f32 v90, v89, v89\n" \
    "v_min_f32 v92, v97, v90\n" \
    "v_min_f32 v99, v99, v92\n" \
    "v_cmp_lt_f32 vcc, v99, v50\n" \
    "s_waitcnt lgkmcnt(0)\n" \
    "v_mul_f32 v111, v75, v80\n" \
    "v_fmac_f32 v111, v73, v78\n" \
    "v_fmac_f32 v111, v71, v76\n" \
    "v_add_f32_dpp v53, v120, v53 row_ror:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_add_f32_dpp v55, v122, v55 row_ror:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_add_f32_dpp v57, v124, v57 row_ror:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_mul_f32 v113, v75, v40\n" \
    "v_fmac_f32 v113, v73, v38\n" \
    "v_fmac_f32 v113, v71, v36\n" \
    "v_mul_f32 v121, v81, v80\n" \
    "v_fmac_f32 v121, v79, v78\n" \
    "v_fmac_f32 v121, v77, v76\n" \
    "v_mul_f32 v123, v81, v46\n" \
    "v_fmac_f32 v123, v79, v44\n" \
    "v_fmac_f32 v123, v77, v42\n" \
    "s_cbranch_vccz SD_SKIP1_%=\n" \
    "s_or_b64 %[nl], %[nl], vcc\n" \
    "v_cmp_lt_f32 vcc, v95, v50\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v95, v95, v27, vcc\n" \
    "v_cmp_lt_f32 vcc, v88, v25\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v88, v88, v27, vcc\n" \
    "v_cmp_lt_f32 vcc, v97, v50\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v97, v97, v27, vcc\n" \
    "v_cmp_lt_f32 vcc, v90, v25\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v90, v90, v27, vcc\n" \
    "SD_SKIP1_%=:\n" \
    "v_rsq_f32 v105, v95\n" \
    "v_rsq_f32 v115, v88\n" \
    "v_mul_f32 v94, v105, v105\n" \
    "v_mul_f32 v104, v115, v115\n" \
    "v_mul_f32 v107, v94, v105\n" \
    "v_mul_f32 v117, v104, v115\n" \
    "v_fma_f32 v109, v48, v107, v105\n" \
    "v_fma_f32 v96, v29, v94, 1.0\n" \
    "v_fma_f32 v119, v48, v117, v115\n" \
    "v_fma_f32 v106, v29, v104, 1.0\n" \
    "v_mul_f32 v98, v107, v96\n" \
    "v_mul_f32 v100, v98, v111\n" \
    "v_mul_f32 v102, v98, v113\n" \
    "v_mul_f32 v108, v117, v106\n" \
    "v_mul_f32 v110, v108, v121\n" \
    "v_mul_f32 v112, v108, v123\n" \
    "v_fmac_f32 v52, v100, v71\n" \
    "v_fmac_f32 v52, v109, v76\n" \
    "v_fmac_f32 v54, v100, v73\n" \
    "v_fmac_f32 v54, v109, v78\n" \
    "v_fmac_f32 v56, v100, v75\n" \
    "v_fmac_f32 v56, v109, v80\n" \
    "v_fmac_f32 v58, v110, v77\n" \
    "v_fmac_f32 v58, v119, v76\n" \
    "v_fmac_f32 v60, v110, v79\n" \
    "v_fmac_f32 v60, v119, v78\n" \
    "v_fmac_f32 v62, v110, v81\n" \
    "v_fmac_f32 v62, v119, v80\n" \
    "v_mul_f32 v114, v102, v71\n" \
    "v_fmac_f32 v114, v109, v36\n" \
    "v_mul_f32 v116, v102, v73\n" \
    "v_fmac_f32 v116, v109, v38\n" \
    "v_mul_f32 v118, v102, v75\n" \
    "v_fmac_f32 v118, v109, v40\n" \
    "v_fmac_f32 v114, v112, v77\n" \
    "v_fmac_f32 v114, v119, v42\n" \
    "v_fmac_f32 v116, v112, v79\n" \
    "v_fmac_f32 v116, v119, v44\n" \
    "v_fmac_f32 v118, v112, v81\n" \
    "v_fmac_f32 v118, v119, v46\n" \
    "v_rsq_f32 v105, v97\n" \
    "v_rsq_f32 v115, v90\n" \
    "v_mul_f32 v111, v87, v86\n" \
    "v_fmac_f32 v111, v85, v84\n" \
    "v_fmac_f32 v111, v83, v82\n" \
    "v_add_f32_dpp v53, v114, v53 row_ror:2 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_add_f32_dpp v55, v116, v55 row_ror:2 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_add_f32_dpp v57, v118, v57 row_ror:2 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_mul_f32 v113, v87, v40\n" \
    "v_fmac_f32 v113, v85, v38\n" \
    "v_fmac_f32 v113, v83, v36\n" \
    "v_mul_f32 v121, v93, v86\n" \
    "v_fmac_f32 v121, v91, v84\n" \
    "v_fmac_f32 v121, v89, v82\n" \
    "v_mul_f32 v123, v93, v46\n" \
    "v_fmac_f32 v123, v91, v44\n" \
    "v_fmac_f32 v123, v89, v42\n" \
    "v_mul_f32 v94, v105, v105\n" \
    "v_mul_f32 v104, v115, v115\n" \
    "v_mul_f32 v107, v94, v105\n" \
    "v_mul_f32 v117, v104, v115\n" \
    "v_fma_f32 v109, v48, v107, v105\n" \
    "v_fma_f32 v96, v29, v94, 1.0\n" \
    "v_fma_f32 v119, v48, v117, v115\n" \
    "v_fma_f32 v106, v29, v104, 1.0\n" \
    "v_mul_f32 v98, v107, v96\n" \
    "v_mul_f32 v100, v98, v111\n" \
    "v_mul_f32 v102, v98, v113\n" \
    "v_mul_f32 v108, v117, v106\n" \
    "v_mul_f32 v110, v108, v121\n" \
    "v_mul_f32 v112, v108, v123\n" \
    "v_fmac_f32 v52, v100, v83\n" \
    "v_fmac_f32 v52, v109, v82\n" \
    "v_fmac_f32 v54, v100, v85\n" \
    "v_fmac_f32 v54, v109, v84\n" \
    "v_fmac_f32 v56, v100, v87\n" \
    "v_fmac_f32 v56, v109, v86\n" \
    "v_fmac_f32 v58, v110, v89\n" \
    "v_fmac_f32 v58, v119, v82\n" \
    "v_fmac_f32 v60, v110, v91\n" \
    "v_fmac_f32 v60, v119, v84\n" \
    "v_fmac_f32 v62, v110, v93\n" \
    "v_fmac_f32 v62, v119, v86\n" \
    "v_mul_f32 v120, v102, v83\n" \
    "v_fmac_f32 v120, v109, v36\n" \
    "v_mul_f32 v122, v102, v85\n" \
    "v_fmac_f32 v122, v109, v38\n" \
    "v_mul_f32 v124, v102, v87\n" \
    "v_fmac_f32 v124, v109, v40\n" \
    "v_fmac_f32 v120, v112, v89\n" \
    "v_fmac_f32 v120, v119, v42\n" \
    "v_fmac_f32 v122, v112, v91\n" \
    "v_fmac_f32 v122, v119, v44\n" \
    "v_fmac_f32 v124, v112, v93\n" \
    "v_fmac_f32 v124, v119, v46\n" \
    "v_add_f32 v35, v35, v52\n" \
    "v_add_f32 v37, v37, v54\n" \
    "v_add_f32 v39, v39, v56\n" \
    "v_add_f32 v41, v41, v58\n" \
    "v_add_f32 v43, v43, v60\n" \
    "v_add_f32 v45, v45, v62\n" \
    "ds_read_b32 v59, v31 offset:16\n" \
    "ds_read_b32 v61, v31 offset:144\n" \
    "ds_read_b32 v63, v31 offset:272\n" \
    "ds_read_b32 v65, v31 offset:20\n" \
    "ds_read_b32 v67, v31 offset:148\n" \
    "ds_read_b32 v69, v31 offset:276\n" \
    "ds_read_b32 v76, v31 offset:400\n" \
    "ds_read_b32 v78, v31 offset:528\n" \
    "ds_read_b32 v80, v31 offset:656\n" \
    "ds_read_b32 v82, v31 offset:404\n" \
    "ds_read_b32 v84, v31 offset:532\n" \
    "ds_read_b32 v86, v31 offset:660\n" \
    "s_waitcnt lgkmcnt(9)\n" \
    "v_sub_f32 v71, v24, v59\n" \
    "v_sub_f32 v73, v26, v61\n" \
    "v_sub_f32 v75, v28, v63\n" \
    "v_sub_f32 v77, v30, v59\n" \
    "v_sub_f32 v79, v32, v61\n" \
    "v_sub_f32 v81, v34, v63\n" \
    "v_mul_f32 v95, v75, v75\n" \
    "v_fmac_f32 v95, v73, v73\n" \
    "v_fmac_f32 v95, v71, v71\n" \
    "v_mul_f32 v88, v81, v81\n" \
    "v_fmac_f32 v88, v79, v79\n" \
    "v_fmac_f32 v88, v77, v77\n" \
    "v_min_f32 v99, v95, v88\n" \
    "s_waitcnt lgkmcnt(6)\n" \
    "v_sub_f32 v83, v24, v65\n" \
    "v_sub_f32 v85, v26, v67\n" \
    "v_sub_f32 v87, v28, v69\n" \
    "v_sub_f32 v89, v30, v65\n" \
    "v_sub_f32 v91, v32, v67\n" \
    "v_sub_f32 v93, v34, v69\n" \
    "v_mul_f32 v97, v87, v87\n" \
    "v_fmac_f32 v97, v85, v85\n" \
    "v_fmac_f32 v97, v83, v83\n" \
    "v_mul_f32 v90, v93, v93\n" \
    "v_fmac_f32 v90, v91, v91\n" \
    "v_fmac_f32 v90, v89, v89\n" \
    "v_min_f32 v92, v97, v90\n" \
    "v_min_f32 v99, v99, v92\n" \
    "v_cmp_lt_f32 vcc, v99, v50\n" \
    "s_waitcnt lgkmcnt(0)\n" \
    "v_mul_f32 v111, v75, v80\n" \
    "v_fmac_f32 v111, v73, v78\n" \
    "v_fmac_f32 v111, v71, v76\n" \
    "v_add_f32_dpp v53, v120, v53 row_ror:3 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_add_f32_dpp v55, v122, v55 row_ror:3 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_add_f32_dpp v57, v124, v57 row_ror:3 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_mul_f32 v113, v75, v40\n" \
    "v_fmac_f32 v113, v73, v38\n" \
    "v_fmac_f32 v113, v71, v36\n" \
    "v_mul_f32 v121, v81, v80\n" \
    "v_fmac_f32 v121, v79, v78\n" \
    "v_fmac_f32 v121, v77, v76\n" \
    "v_mul_f32 v123, v81, v46\n" \
    "v_fmac_f32 v123, v79, v44\n" \
    "v_fmac_f32 v123, v77, v42\n" \
    "s_cbranch_vccz SD_SKIP2_%=\n" \
    "s_or_b64 %[nl], %[nl], vcc\n" \
    "v_cmp_lt_f32 vcc, v95, v50\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v95, v95, v27, vcc\n" \
    "v_cmp_lt_f32 vcc, v88, v25\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v88, v88, v27, vcc\n" \
    "v_cmp_lt_f32 vcc, v97, v50\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v97, v97, v27, vcc\n" \
    "v_cmp_lt_f32 vcc, v90, v25\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v90, v90, v27, vcc\n" \
    "SD_SKIP2_%=:\n" \
    "v_rsq_f32 v105, v95\n" \
    "v_rsq_f32 v115, v88\n" \
    "v_mul_f32 v94, v105, v105\n" \
    "v_mul_f32 v104, v115, v115\n" \
    "v_mul_f32 v107, v94, v105\n" \
    "v_mul_f32 v117, v104, v115\n" \
    "v_fma_f32 v109, v48, v107, v105\n" \
    "v_fma_f32 v96, v29, v94, 1.0\n" \
    "v_fma_f32 v119, v48, v117, v115\n" \
    "v_fma_f32 v106, v29, v104, 1.0\n" \
    "v_mul_f32 v98, v107, v96\n" \
    "v_mul_f32 v100, v98, v111\n" \
    "v_mul_f32 v102, v98, v113\n" \
    "v_mul_f32 v108, v117, v106\n" \
    "v_mul_f32 v110, v108, v121\n" \
    "v_mul_f32 v112, v108, v123\n" \
    "v_mul_f32 v52, v100, v71\n" \
    "v_fmac_f32 v52, v109, v76\n" \
    "v_mul_f32 v54, v100, v73\n" \
    "v_fmac_f32 v54, v109, v78\n" \
    "v_mul_f32 v56, v100, v75\n" \
    "v_fmac_f32 v56, v109, v80\n" \
    "v_mul_f32 v58, v110, v77\n" \
    "v_fmac_f32 v58, v119, v76\n" \
    "v_mul_f32 v60, v110, v79\n" \
    "v_fmac_f32 v60, v119, v78\n" \
    "v_mul_f32 v62, v110, v81\n" \
    "v_fmac_f32 v62, v119, v80\n" \
    "v_mul_f32 v114, v102, v71\n" \
    "v_fmac_f32 v114, v109, v36\n" \
    "v_mul_f32 v116, v102, v73\n" \
    "v_fmac_f32 v116, v109, v38\n" \
    "v_mul_f32 v118, v102, v75\n" \
    "v_fmac_f32 v118, v109, v40\n" \
    "v_fmac_f32 v114, v112, v77\n" \
    "v_fmac_f32 v114, v119, v42\n" \
    "v_fmac_f32 v116, v112, v79\n" \
    "v_fmac_f32 v116, v119, v44\n" \
    "v_fmac_f32 v118, v112, v81\n" \
    "v_fmac_f32 v118, v119, v46\n" \
    "v_rsq_f32 v105, v97\n" \
    "v_rsq_f32 v115, v90\n" \
    "v_mul_f32 v111, v87, v86\n" \
    "v_fmac_f32 v111, v85, v84\n" \
    "v_fmac_f32 v111, v83, v82\n" \
    "v_mov_b32_dpp v47, v114 row_ror:4 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_mov_b32_dpp v49, v116 row_ror:4 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_mov_b32_dpp v51, v118 row_ror:4 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_mul_f32 v113, v87, v40\n" \
    "v_fmac_f32 v113, v85, v38\n" \
    "v_fmac_f32 v113, v83, v36\n" \
    "v_mul_f32 v121, v93, v86\n" \
    "v_fmac_f32 v121, v91, v84\n" \
    "v_fmac_f32 v121, v89, v82\n" \
    "v_mul_f32 v123, v93, v46\n" \
    "v_fmac_f32 v123, v91, v44\n" \
    "v_fmac_f32 v123, v89, v42\n" \
    "v_mul_f32 v94, v105, v105\n" \
    "v_mul_f32 v104, v115, v115\n" \
    "v_mul_f32 v107, v94, v105\n" \
    "v_mul_f32 v117, v104, v115\n" \
    "v_fma_f32 v109, v48, v107, v105\n" \
    "v_fma_f32 v96, v29, v94, 1.0\n" \
    "v_fma_f32 v119, v48, v117, v115\n" \
    "v_fma_f32 v106, v29, v104, 1.0\n" \
    "v_mul_f32 v98, v107, v96\n" \
    "v_mul_f32 v100, v98, v111\n" \
    "v_mul_f32 v102, v98, v113\n" \
    "v_mul_f32 v108, v117, v106\n" \
    "v_mul_f32 v110, v108, v121\n" \
    "v_mul_f32 v112, v108, v123\n" \
    "v_fmac_f32 v52, v100, v83\n" \
    "v_fmac_f32 v52, v109, v82\n" \
    "v_fmac_f32 v54, v100, v85\n" \
    "v_fmac_f32 v54, v109, v84\n" \
    "v_fmac_f32 v56, v100, v87\n" \
    "v_fmac_f32 v56, v109, v86\n" \
    "v_fmac_f32 v58, v110, v89\n" \
    "v_fmac_f32 v58, v119, v82\n" \
    "v_fmac_f32 v60, v110, v91\n" \
    "v_fmac_f32 v60, v119, v84\n" \
    "v_fmac_f32 v62, v110, v93\n" \
    "v_fmac_f32 v62, v119, v86\n" \
    "v_mul_f32 v120, v102, v83\n" \
    "v_fmac_f32 v120, v109, v36\n" \
    "v_mul_f32 v122, v102, v85\n" \
    "v_fmac_f32 v122, v109, v38\n" \
    "v_mul_f32 v124, v102, v87\n" \
    "v_fmac_f32 v124, v109, v40\n" \
    "v_fmac_f32 v120, v112, v89\n" \
    "v_fmac_f32 v120, v119, v42\n" \
    "v_fmac_f32 v122, v112, v91\n" \
    "v_fmac_f32 v122, v119, v44\n" \
    "v_fmac_f32 v124, v112, v93\n" \
    "v_fmac_f32 v124, v119, v46\n" \
    "ds_read_b32 v59, v31 offset:24\n" \
    "ds_read_b32 v61, v31 offset:152\n" \
    "ds_read_b32 v63, v31 offset:280\n" \
    "ds_read_b32 v65, v31 offset:28\n" \
    "ds_read_b32 v67, v31 offset:156\n" \
    "ds_read_b32 v69, v31 offset:284\n" \
    "ds_read_b32 v76, v31 offset:408\n" \
    "ds_read_b32 v78, v31 offset:536\n" \
    "ds_read_b32 v80, v31 offset:664\n" \
    "ds_read_b32 v82, v31 offset:412\n" \
    "ds_read_b32 v84, v31 offset:540\n" \
    "ds_read_b32 v86, v31 offset:668\n" \
    "s_waitcnt lgkmcnt(9)\n" \
    "v_sub_f32 v71, v24, v59\n" \
    "v_sub_f32 v73, v26, v61\n" \
    "v_sub_f32 v75, v28, v63\n" \
    "v_sub_f32 v77, v30, v59\n" \
    "v_sub_f32 v79, v32, v61\n" \
    "v_sub_f32 v81, v34, v63\n" \
    "v_mul_f32 v95, v75, v75\n" \
    "v_fmac_f32 v95, v73, v73\n" \
    "v_fmac_f32 v95, v71, v71\n" \
    "v_mul_f32 v88, v81, v81\n" \
    "v_fmac_f32 v88, v79, v79\n" \
    "v_fmac_f32 v88, v77, v77\n" \
    "v_min_f32 v99, v95, v88\n" \
    "s_waitcnt lgkmcnt(6)\n" \
    "v_sub_f32 v83, v24, v65\n" \
    "v_sub_f32 v85, v26, v67\n" \
    "v_sub_f32 v87, v28, v69\n" \
    "v_sub_f32 v89, v30, v65\n" \
    "v_sub_f32 v91, v32, v67\n" \
    "v_sub_f32 v93, v34, v69\n" \
    "v_mul_f32 v97, v87, v87\n" \
    "v_fmac_f32 v97, v85, v85\n" \
    "v_fmac_f32 v97, v83, v83\n" \
    "v_mul_f32 v90, v93, v93\n" \
    "v_fmac_f32 v90, v91, v91\n" \
    "v_fmac_f32 v90, v89, v89\n" \
    "v_min_f32 v92, v97, v90\n" \
    "v_min_f32 v99, v99, v92\n" \
    "v_cmp_lt_f32 vcc, v99, v50\n" \
    "s_waitcnt lgkmcnt(0)\n" \
    "v_mul_f32 v111, v75, v80\n" \
    "v_fmac_f32 v111, v73, v78\n" \
    "v_fmac_f32 v111, v71, v76\n" \
    "v_add_f32_dpp v47, v120, v47 row_ror:5 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_add_f32_dpp v49, v122, v49 row_ror:5 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_add_f32_dpp v51, v124, v51 row_ror:5 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_mul_f32 v113, v75, v40\n" \
    "v_fmac_f32 v113, v73, v38\n" \
    "v_fmac_f32 v113, v71, v36\n" \
    "v_mul_f32 v121, v81, v80\n" \
    "v_fmac_f32 v121, v79, v78\n" \
    "v_fmac_f32 v121, v77, v76\n" \
    "v_mul_f32 v123, v81, v46\n" \
    "v_fmac_f32 v123, v79, v44\n" \
    "v_fmac_f32 v123, v77, v42\n" \
    "s_cbranch_vccz SD_SKIP3_%=\n" \
    "s_or_b64 %[nl], %[nl], vcc\n" \
    "v_cmp_lt_f32 vcc, v95, v50\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v95, v95, v27, vcc\n" \
    "v_cmp_lt_f32 vcc, v88, v25\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v88, v88, v27, vcc\n" \
    "v_cmp_lt_f32 vcc, v97, v50\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v97, v97, v27, vcc\n" \
    "v_cmp_lt_f32 vcc, v90, v25\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v90, v90, v27, vcc\n" \
    "SD_SKIP3_%=:\n" \
    "v_rsq_f32 v105, v95\n" \
    "v_rsq_f32 v115, v88\n" \
    "v_mul_f32 v94, v105, v105\n" \
    "v_mul_f32 v104, v115, v115\n" \
    "v_mul_f32 v107, v94, v105\n" \
    "v_mul_f32 v117, v104, v115\n" \
    "v_fma_f32 v109, v48, v107, v105\n" \
    "v_fma_f32 v96, v29, v94, 1.0\n" \
    "v_fma_f32 v119, v48, v117, v115\n" \
    "v_fma_f32 v106, v29, v104, 1.0\n" \
    "v_mul_f32 v98, v107, v96\n" \
    "v_mul_f32 v100, v98, v111\n" \
    "v_mul_f32 v102, v98, v113\n" \
    "v_mul_f32 v108, v117, v106\n" \
    "v_mul_f32 v110, v108, v121\n" \
    "v_mul_f32 v112, v108, v123\n" \
    "v_fmac_f32 v52, v100, v71\n" \
    "v_fmac_f32 v52, v109, v76\n" \
    "v_fmac_f32 v54, v100, v73\n" \
    "v_fmac_f32 v54, v109, v78\n" \
    "v_fmac_f32 v56, v100, v75\n" \
    "v_fmac_f32 v56, v109, v80\n" \
    "v_fmac_f32 v58, v110, v77\n" \
    "v_fmac_f32 v58, v119, v76\n" \
    "v_fmac_f32 v60, v110, v79\n" \
    "v_fmac_f32 v60, v119, v78\n" \
    "v_fmac_f32 v62, v110, v81\n" \
    "v_fmac_f32 v62, v119, v80\n" \
    "v_mul_f32 v114, v102, v71\n" \
    "v_fmac_f32 v114, v109, v36\n" \
    "v_mul_f32 v116, v102, v73\n" \
    "v_fmac_f32 v116, v109, v38\n" \
    "v_mul_f32 v118, v102, v75\n" \
    "v_fmac_f32 v118, v109, v40\n" \
    "v_fmac_f32 v114, v112, v77\n" \
    "v_fmac_f32 v114, v119, v42\n" \
    "v_fmac_f32 v116, v112, v79\n" \
    "v_fmac_f32 v116, v119, v44\n" \
    "v_fmac_f32 v118, v112, v81\n" \
    "v_fmac_f32 v118, v119, v46\n" \
    "v_rsq_f32 v105, v97\n" \
    "v_rsq_f32 v115, v90\n" \
    "v_mul_f32 v111, v87, v86\n" \
    "v_fmac_f32 v111, v85, v84\n" \
    "v_fmac_f32 v111, v83, v82\n" \
    "v_add_f32_dpp v47, v114, v47 row_ror:6 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_add_f32_dpp v49, v116, v49 row_ror:6 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_add_f32_dpp v51, v118, v51 row_ror:6 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_mul_f32 v113, v87, v40\n" \
    "v_fmac_f32 v113, v85, v38\n" \
    "v_fmac_f32 v113, v83, v36\n" \
    "v_mul_f32 v121, v93, v86\n" \
    "v_fmac_f32 v121, v91, v84\n" \
    "v_fmac_f32 v121, v89, v82\n" \
    "v_mul_f32 v123, v93, v46\n" \
    "v_fmac_f32 v123, v91, v44\n" \
    "v_fmac_f32 v123, v89, v42\n" \
    "v_mul_f32 v94, v105, v105\n" \
    "v_mul_f32 v104, v115, v115\n" \
    "v_mul_f32 v107, v94, v105\n" \
    "v_mul_f32 v117, v104, v115\n" \
    "v_fma_f32 v109, v48, v107, v105\n" \
    "v_fma_f32 v96, v29, v94, 1.0\n" \
    "v_fma_f32 v119, v48, v117, v115\n" \
    "v_fma_f32 v106, v29, v104, 1.0\n" \
    "v_mul_f32 v98, v107, v96\n" \
    "v_mul_f32 v100, v98, v111\n" \
    "v_mul_f32 v102, v98, v113\n" \
    "v_mul_f32 v108, v117, v106\n" \
    "v_mul_f32 v110, v108, v121\n" \
    "v_mul_f32 v112, v108, v123\n" \
    "v_fmac_f32 v52, v100, v83\n" \
    "v_fmac_f32 v52, v109, v82\n" \
    "v_fmac_f32 v54, v100, v85\n" \
    "v_fmac_f32 v54, v109, v84\n" \
    "v_fmac_f32 v56, v100, v87\n" \
    "v_fmac_f32 v56, v109, v86\n" \
    "v_fmac_f32 v58, v110, v89\n" \
    "v_fmac_f32 v58, v119, v82\n" \
    "v_fmac_f32 v60, v110, v91\n" \
    "v_fmac_f32 v60, v119, v84\n" \
    "v_fmac_f32 v62, v110, v93\n" \
    "v_fmac_f32 v62, v119, v86\n" \
    "v_mul_f32 v120, v102, v83\n" \
    "v_fmac_f32 v120, v109, v36\n" \
    "v_mul_f32 v122, v102, v85\n" \
    "v_fmac_f32 v122, v109, v38\n" \
    "v_mul_f32 v124, v102, v87\n" \
    "v_fmac_f32 v124, v109, v40\n" \
    "v_fmac_f32 v120, v112, v89\n" \
    "v_fmac_f32 v120, v119, v42\n" \
    "v_fmac_f32 v122, v112, v91\n" \
    "v_fmac_f32 v122, v119, v44\n" \
    "v_fmac_f32 v124, v112, v93\n" \
    "v_fmac_f32 v124, v119, v46\n" \
    "v_add_f32 v35, v35, v52\n" \
    "v_add_f32 v37, v37, v54\n" \
    "v_add_f32 v39, v39, v56\n" \
    "v_add_f32 v41, v41, v58\n" \
    "v_add_f32 v43, v43, v60\n" \
    "v_add_f32 v45, v45, v62\n" \
    "ds_read_b32 v59, v31 offset:32\n" \
    "ds_read_b32 v61, v31 offset:160\n" \
    "ds_read_b32 v63, v31 offset:288\n" \
    "ds_read_b32 v65, v31 offset:36\n" \
    "ds_read_b32 v67, v31 offset:164\n" \
    "ds_read_b32 v69, v31 offset:292\n" \
    "ds_read_b32 v76, v31 offset:416\n" \
    "ds_read_b32 v78, v31 offset:544\n" \
    "ds_read_b32 v80, v31 offset:672\n" \
    "ds_read_b32 v82, v31 offset:420\n" \
    "ds_read_b32 v84, v31 offset:548\n" \
    "ds_read_b32 v86, v31 offset:676\n" \
    "s_waitcnt lgkmcnt(9)\n" \
    "v_sub_f32 v71, v24, v59\n" \
    "v_sub_f32 v73, v26, v61\n" \
    "v_sub_f32 v75, v28, v63\n" \
    "v_sub_f32 v77, v30, v59\n" \
    "v_sub_f32 v79, v32, v61\n" \
    "v_sub_f32 v81, v34, v63\n" \
    "v_mul_f32 v95, v75, v75\n" \
    "v_fmac_f32 v95, v73, v73\n" \
    "v_fmac_f32 v95, v71, v71\n" \
    "v_mul_f32 v88, v81, v81\n" \
    "v_fmac_f32 v88, v79, v79\n" \
    "v_fmac_f32 v88, v77, v77\n" \
    "v_min_f32 v99, v95, v88\n" \
    "s_waitcnt lgkmcnt(6)\n" \
    "v_sub_f32 v83, v24, v65\n" \
    "v_sub_f32 v85, v26, v67\n" \
    "v_sub_f32 v87, v28, v69\n" \
    "v_sub_f32 v89, v30, v65\n" \
    "v_sub_f32 v91, v32, v67\n" \
    "v_sub_f32 v93, v34, v69\n" \
    "v_mul_f32 v97, v87, v87\n" \
    "v_fmac_f32 v97, v85, v85\n" \
    "v_fmac_f32 v97, v83, v83\n" \
    "v_mul_f32 v90, v93, v93\n" \
    "v_fmac_f32 v90, v91, v91\n" \
    "v_fmac_f32 v90, v89, v89\n" \
    "v_min_f32 v92, v97, v90\n" \
    "v_min_f32 v99, v99, v92\n" \
    "v_cmp_lt_f32 vcc, v99, v50\n" \
    "s_waitcnt lgkmcnt(0)\n" \
    "v_mul_f32 v111, v75, v80\n" \
    "v_fmac_f32 v111, v73, v78\n" \
    "v_fmac_f32 v111, v71, v76\n" \
    "v_add_f32_dpp v47, v120, v47 row_ror:7 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_add_f32_dpp v49, v122, v49 row_ror:7 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_add_f32_dpp v51, v124, v51 row_ror:7 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_mul_f32 v113, v75, v40\n" \
    "v_fmac_f32 v113, v73, v38\n" \
    "v_fmac_f32 v113, v71, v36\n" \
    "v_mul_f32 v121, v81, v80\n" \
    "v_fmac_f32 v121, v79, v78\n" \
    "v_fmac_f32 v121, v77, v76\n" \
    "v_mul_f32 v123, v81, v46\n" \
    "v_fmac_f32 v123, v79, v44\n" \
    "v_fmac_f32 v123, v77, v42\n" \
    "v_add_f32 v53, v53, v47\n" \
    "v_add_f32 v55, v55, v49\n" \
    "v_add_f32 v57, v57, v51\n" \
    "ds_write_b32 v33, v53 offset:0\n" \
    "ds_write_b32 v33, v55 offset:64\n" \
    "ds_write_b32 v33, v57 offset:128\n" \
    "s_cbranch_vccz SD_SKIP4_%=\n" \
    "s_or_b64 %[nl], %[nl], vcc\n" \
    "v_cmp_lt_f32 vcc, v95, v50\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v95, v95, v27, vcc\n" \
    "v_cmp_lt_f32 vcc, v88, v25\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v88, v88, v27, vcc\n" \
    "v_cmp_lt_f32 vcc, v97, v50\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v97, v97, v27, vcc\n" \
    "v_cmp_lt_f32 vcc, v90, v25\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v90, v90, v27, vcc\n" \
    "SD_SKIP4_%=:\n" \
    "v_rsq_f32 v105, v95\n" \
    "v_rsq_f32 v115, v88\n" \
    "v_mul_f32 v94, v105, v105\n" \
    "v_mul_f32 v104, v115, v115\n" \
    "v_mul_f32 v107, v94, v105\n" \
    "v_mul_f32 v117, v104, v115\n" \
    "v_fma_f32 v109, v48, v107, v105\n" \
    "v_fma_f32 v96, v29, v94, 1.0\n" \
    "v_fma_f32 v119, v48, v117, v115\n" \
    "v_fma_f32 v106, v29, v104, 1.0\n" \
    "v_mul_f32 v98, v107, v96\n" \
    "v_mul_f32 v100, v98, v111\n" \
    "v_mul_f32 v102, v98, v113\n" \
    "v_mul_f32 v108, v117, v106\n" \
    "v_mul_f32 v110, v108, v121\n" \
    "v_mul_f32 v112, v108, v123\n" \
    "v_mul_f32 v52, v100, v71\n" \
    "v_fmac_f32 v52, v109, v76\n" \
    "v_mul_f32 v54, v100, v73\n" \
    "v_fmac_f32 v54, v109, v78\n" \
    "v_mul_f32 v56, v100, v75\n" \
    "v_fmac_f32 v56, v109, v80\n" \
    "v_mul_f32 v58, v110, v77\n" \
    "v_fmac_f32 v58, v119, v76\n" \
    "v_mul_f32 v60, v110, v79\n" \
    "v_fmac_f32 v60, v119, v78\n" \
    "v_mul_f32 v62, v110, v81\n" \
    "v_fmac_f32 v62, v119, v80\n" \
    "v_mul_f32 v114, v102, v71\n" \
    "v_fmac_f32 v114, v109, v36\n" \
    "v_mul_f32 v116, v102, v73\n" \
    "v_fmac_f32 v116, v109, v38\n" \
    "v_mul_f32 v118, v102, v75\n" \
    "v_fmac_f32 v118, v109, v40\n" \
    "v_fmac_f32 v114, v112, v77\n" \
    "v_fmac_f32 v114, v119, v42\n" \
    "v_fmac_f32 v116, v112, v79\n" \
    "v_fmac_f32 v116, v119, v44\n" \
    "v_fmac_f32 v118, v112, v81\n" \
    "v_fmac_f32 v118, v119, v46\n" \
    "v_rsq_f32 v105, v97\n" \
    "v_rsq_f32 v115, v90\n" \
    "v_mul_f32 v111, v87, v86\n" \
    "v_fmac_f32 v111, v85, v84\n" \
    "v_fmac_f32 v111, v83, v82\n" \
    "v_mov_b32_dpp v53, v114 row_ror:8 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_mov_b32_dpp v55, v116 row_ror:8 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_mov_b32_dpp v57, v118 row_ror:8 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_mul_f32 v113, v87, v40\n" \
    "v_fmac_f32 v113, v85, v38\n" \
    "v_fmac_f32 v113, v83, v36\n" \
    "v_mul_f32 v121, v93, v86\n" \
    "v_fmac_f32 v121, v91, v84\n" \
    "v_fmac_f32 v121, v89, v82\n" \
    "v_mul_f32 v123, v93, v46\n" \
    "v_fmac_f32 v123, v91, v44\n" \
    "v_fmac_f32 v123, v89, v42\n" \
    "v_mul_f32 v94, v105, v105\n" \
    "v_mul_f32 v104, v115, v115\n" \
    "v_mul_f32 v107, v94, v105\n" \
    "v_mul_f32 v117, v104, v115\n" \
    "v_fma_f32 v109, v48, v107, v105\n" \
    "v_fma_f32 v96, v29, v94, 1.0\n" \
    "v_fma_f32 v119, v48, v117, v115\n" \
    "v_fma_f32 v106, v29, v104, 1.0\n" \
    "v_mul_f32 v98, v107, v96\n" \
    "v_mul_f32 v100, v98, v111\n" \
    "v_mul_f32 v102, v98, v113\n" \
    "v_mul_f32 v108, v117, v106\n" \
    "v_mul_f32 v110, v108, v121\n" \
    "v_mul_f32 v112, v108, v123\n" \
    "v_fmac_f32 v52, v100, v83\n" \
    "v_fmac_f32 v52, v109, v82\n" \
    "v_fmac_f32 v54, v100, v85\n" \
    "v_fmac_f32 v54, v109, v84\n" \
    "v_fmac_f32 v56, v100, v87\n" \
    "v_fmac_f32 v56, v109, v86\n" \
    "v_fmac_f32 v58, v110, v89\n" \
    "v_fmac_f32 v58, v119, v82\n" \
    "v_fmac_f32 v60, v110, v91\n" \
    "v_fmac_f32 v60, v119, v84\n" \
    "v_fmac_f32 v62, v110, v93\n" \
    "v_fmac_f32 v62, v119, v86\n" \
    "v_mul_f32 v120, v102, v83\n" \
    "v_fmac_f32 v120, v109, v36\n" \
    "v_mul_f32 v122, v102, v85\n" \
    "v_fmac_f32 v122, v109, v38\n" \
    "v_mul_f32 v124, v102, v87\n" \
    "v_fmac_f32 v124, v109, v40\n" \
    "v_fmac_f32 v120, v112, v89\n" \
    "v_fmac_f32 v120, v119, v42\n" \
    "v_fmac_f32 v122, v112, v91\n" \
    "v_fmac_f32 v122, v119, v44\n" \
    "v_fmac_f32 v124, v112, v93\n" \
    "v_fmac_f32 v124, v119, v46\n" \
    "ds_read_b32 v59, v31 offset:40\n" \
    "ds_read_b32 v61, v31 offset:168\n" \
    "ds_read_b32 v63, v31 offset:296\n" \
    "ds_read_b32 v65, v31 offset:44\n" \
    "ds_read_b32 v67, v31 offset:172\n" \
    "ds_read_b32 v69, v31 offset:300\n" \
    "ds_read_b32 v76, v31 offset:424\n" \
    "ds_read_b32 v78, v31 offset:552\n" \
    "ds_read_b32 v80, v31 offset:680\n" \
    "ds_read_b32 v82, v31 offset:428\n" \
    "ds_read_b32 v84, v31 offset:556\n" \
    "ds_read_b32 v86, v31 offset:684\n" \
    "s_waitcnt lgkmcnt(9)\n" \
    "v_sub_f32 v71, v24, v59\n" \
    "v_sub_f32 v73, v26, v61\n" \
    "v_sub_f32 v75, v28, v63\n" \
    "v_sub_f32 v77, v30, v59\n" \
    "v_sub_f32 v79, v32, v61\n" \
    "v_sub_f32 v81, v34, v63\n" \
    "v_mul_f32 v95, v75, v75\n" \
    "v_fmac_f32 v95, v73, v73\n" \
    "v_fmac_f32 v95, v71, v71\n" \
    "v_mul_f32 v88, v81, v81\n" \
    "v_fmac_f32 v88, v79, v79\n" \
    "v_fmac_f32 v88, v77, v77\n" \
    "v_min_f32 v99, v95, v88\n" \
    "s_waitcnt lgkmcnt(6)\n" \
    "v_sub_f32 v83, v24, v65\n" \
    "v_sub_f32 v85, v26, v67\n" \
    "v_sub_f32 v87, v28, v69\n" \
    "v_sub_f32 v89, v30, v65\n" \
    "v_sub_f32 v91, v32, v67\n" \
    "v_sub_f32 v93, v34, v69\n" \
    "v_mul_f32 v97, v87, v87\n" \
    "v_fmac_f32 v97, v85, v85\n" \
    "v_fmac_f32 v97, v83, v83\n" \
    "v_mul_f32 v90, v93, v93\n" \
    "v_fmac_f32 v90, v91, v91\n" \
    "v_fmac_f32 v90, v89, v89\n" \
    "v_min_f32 v92, v97, v90\n" \
    "v_min_f32 v99, v99, v92\n" \
    "v_cmp_lt_f32 vcc, v99, v50\n" \
    "s_waitcnt lgkmcnt(0)\n" \
    "v_mul_f32 v111, v75, v80\n" \
    "v_fmac_f32 v111, v73, v78\n" \
    "v_fmac_f32 v111, v71, v76\n" \
    "v_add_f32_dpp v53, v120, v53 row_ror:9 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_add_f32_dpp v55, v122, v55 row_ror:9 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_add_f32_dpp v57, v124, v57 row_ror:9 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_mul_f32 v113, v75, v40\n" \
    "v_fmac_f32 v113, v73, v38\n" \
    "v_fmac_f32 v113, v71, v36\n" \
    "v_mul_f32 v121, v81, v80\n" \
    "v_fmac_f32 v121, v79, v78\n" \
    "v_fmac_f32 v121, v77, v76\n" \
    "v_mul_f32 v123, v81, v46\n" \
    "v_fmac_f32 v123, v79, v44\n" \
    "v_fmac_f32 v123, v77, v42\n" \
    "s_cbranch_vccz SD_SKIP5_%=\n" \
    "s_or_b64 %[nl], %[nl], vcc\n" \
    "v_cmp_lt_f32 vcc, v95, v50\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v95, v95, v27, vcc\n" \
    "v_cmp_lt_f32 vcc, v88, v25\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v88, v88, v27, vcc\n" \
    "v_cmp_lt_f32 vcc, v97, v50\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v97, v97, v27, vcc\n" \
    "v_cmp_lt_f32 vcc, v90, v25\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v90, v90, v27, vcc\n" \
    "SD_SKIP5_%=:\n" \
    "v_rsq_f32 v105, v95\n" \
    "v_rsq_f32 v115, v88\n" \
    "v_mul_f32 v94, v105, v105\n" \
    "v_mul_f32 v104, v115, v115\n" \
    "v_mul_f32 v107, v94, v105\n" \
    "v_mul_f32 v117, v104, v115\n" \
    "v_fma_f32 v109, v48, v107, v105\n" \
    "v_fma_f32 v96, v29, v94, 1.0\n" \
    "v_fma_f32 v119, v48, v117, v115\n" \
    "v_fma_f32 v106, v29, v104, 1.0\n" \
    "v_mul_f32 v98, v107, v96\n" \
    "v_mul_f32 v100, v98, v111\n" \
    "v_mul_f32 v102, v98, v113\n" \
    "v_mul_f32 v108, v117, v106\n" \
    "v_mul_f32 v110, v108, v121\n" \
    "v_mul_f32 v112, v108, v123\n" \
    "v_fmac_f32 v52, v100, v71\n" \
    "v_fmac_f32 v52, v109, v76\n" \
    "v_fmac_f32 v54, v100, v73\n" \
    "v_fmac_f32 v54, v109, v78\n" \
    "v_fmac_f32 v56, v100, v75\n" \
    "v_fmac_f32 v56, v109, v80\n" \
    "v_fmac_f32 v58, v110, v77\n" \
    "v_fmac_f32 v58, v119, v76\n" \
    "v_fmac_f32 v60, v110, v79\n" \
    "v_fmac_f32 v60, v119, v78\n" \
    "v_fmac_f32 v62, v110, v81\n" \
    "v_fmac_f32 v62, v119, v80\n" \
    "v_mul_f32 v114, v102, v71\n" \
    "v_fmac_f32 v114, v109, v36\n" \
    "v_mul_f32 v116, v102, v73\n" \
    "v_fmac_f32 v116, v109, v38\n" \
    "v_mul_f32 v118, v102, v75\n" \
    "v_fmac_f32 v118, v109, v40\n" \
    "v_fmac_f32 v114, v112, v77\n" \
    "v_fmac_f32 v114, v119, v42\n" \
    "v_fmac_f32 v116, v112, v79\n" \
    "v_fmac_f32 v116, v119, v44\n" \
    "v_fmac_f32 v118, v112, v81\n" \
    "v_fmac_f32 v118, v119, v46\n" \
    "v_rsq_f32 v105, v97\n" \
    "v_rsq_f32 v115, v90\n" \
    "v_mul_f32 v111, v87, v86\n" \
    "v_fmac_f32 v111, v85, v84\n" \
    "v_fmac_f32 v111, v83, v82\n" \
    "v_add_f32_dpp v53, v114, v53 row_ror:10 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_add_f32_dpp v55, v116, v55 row_ror:10 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_add_f32_dpp v57, v118, v57 row_ror:10 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_mul_f32 v113, v87, v40\n" \
    "v_fmac_f32 v113, v85, v38\n" \
    "v_fmac_f32 v113, v83, v36\n" \
    "v_mul_f32 v121, v93, v86\n" \
    "v_fmac_f32 v121, v91, v84\n" \
    "v_fmac_f32 v121, v89, v82\n" \
    "v_mul_f32 v123, v93, v46\n" \
    "v_fmac_f32 v123, v91, v44\n" \
    "v_fmac_f32 v123, v89, v42\n" \
    "v_mul_f32 v94, v105, v105\n" \
    "v_mul_f32 v104, v115, v115\n" \
    "v_mul_f32 v107, v94, v105\n" \
    "v_mul_f32 v117, v104, v115\n" \
    "v_fma_f32 v109, v48, v107, v105\n" \
    "v_fma_f32 v96, v29, v94, 1.0\n" \
    "v_fma_f32 v119, v48, v117, v115\n" \
    "v_fma_f32 v106, v29, v104, 1.0\n" \
    "v_mul_f32 v98, v107, v96\n" \
    "v_mul_f32 v100, v98, v111\n" \
    "v_mul_f32 v102, v98, v113\n" \
    "v_mul_f32 v108, v117, v106\n" \
    "v_mul_f32 v110, v108, v121\n" \
    "v_mul_f32 v112, v108, v123\n" \
    "v_fmac_f32 v52, v100, v83\n" \
    "v_fmac_f32 v52, v109, v82\n" \
    "v_fmac_f32 v54, v100, v85\n" \
    "v_fmac_f32 v54, v109, v84\n" \
    "v_fmac_f32 v56, v100, v87\n" \
    "v_fmac_f32 v56, v109, v86\n" \
    "v_fmac_f32 v58, v110, v89\n" \
    "v_fmac_f32 v58, v119, v82\n" \
    "v_fmac_f32 v60, v110, v91\n" \
    "v_fmac_f32 v60, v119, v84\n" \
    "v_fmac_f32 v62, v110, v93\n" \
    "v_fmac_f32 v62, v119, v86\n" \
    "v_mul_f32 v120, v102, v83\n" \
    "v_fmac_f32 v120, v109, v36\n" \
    "v_mul_f32 v122, v102, v85\n" \
    "v_fmac_f32 v122, v109, v38\n" \
    "v_mul_f32 v124, v102, v87\n" \
    "v_fmac_f32 v124, v109, v40\n" \
    "v_fmac_f32 v120, v112, v89\n" \
    "v_fmac_f32 v120, v119, v42\n" \
    "v_fmac_f32 v122, v112, v91\n" \
    "v_fmac_f32 v122, v119, v44\n" \
    "v_fmac_f32 v124, v112, v93\n" \
    "v_fmac_f32 v124, v119, v46\n" \
    "v_add_f32 v35, v35, v52\n" \
    "v_add_f32 v37, v37, v54\n" \
    "v_add_f32 v39, v39, v56\n" \
    "v_add_f32 v41, v41, v58\n" \
    "v_add_f32 v43, v43, v60\n" \
    "v_add_f32 v45, v45, v62\n" \
    "ds_read_b32 v59, v31 offset:48\n" \
    "ds_read_b32 v61, v31 offset:176\n" \
    "ds_read_b32 v63, v31 offset:304\n" \
    "ds_read_b32 v65, v31 offset:52\n" \
    "ds_read_b32 v67, v31 offset:180\n" \
    "ds_read_b32 v69, v31 offset:308\n" \
    "ds_read_b32 v76, v31 offset:432\n" \
    "ds_read_b32 v78, v31 offset:560\n" \
    "ds_read_b32 v80, v31 offset:688\n" \
    "ds_read_b32 v82, v31 offset:436\n" \
    "ds_read_b32 v84, v31 offset:564\n" \
    "ds_read_b32 v86, v31 offset:692\n" \
    "s_waitcnt lgkmcnt(9)\n" \
    "v_sub_f32 v71, v24, v59\n" \
    "v_sub_f32 v73, v26, v61\n" \
    "v_sub_f32 v75, v28, v63\n" \
    "v_sub_f32 v77, v30, v59\n" \
    "v_sub_f32 v79, v32, v61\n" \
    "v_sub_f32 v81, v34, v63\n" \
    "v_mul_f32 v95, v75, v75\n" \
    "v_fmac_f32 v95, v73, v73\n" \
    "v_fmac_f32 v95, v71, v71\n" \
    "v_mul_f32 v88, v81, v81\n" \
    "v_fmac_f32 v88, v79, v79\n" \
    "v_fmac_f32 v88, v77, v77\n" \
    "v_min_f32 v99, v95, v88\n" \
    "s_waitcnt lgkmcnt(6)\n" \
    "v_sub_f32 v83, v24, v65\n" \
    "v_sub_f32 v85, v26, v67\n" \
    "v_sub_f32 v87, v28, v69\n" \
    "v_sub_f32 v89, v30, v65\n" \
    "v_sub_f32 v91, v32, v67\n" \
    "v_sub_f32 v93, v34, v69\n" \
    "v_mul_f32 v97, v87, v87\n" \
    "v_fmac_f32 v97, v85, v85\n" \
    "v_fmac_f32 v97, v83, v83\n" \
    "v_mul_f32 v90, v93, v93\n" \
    "v_fmac_f32 v90, v91, v91\n" \
    "v_fmac_f32 v90, v89, v89\n" \
    "v_min_f32 v92, v97, v90\n" \
    "v_min_f32 v99, v99, v92\n" \
    "v_cmp_lt_f32 vcc, v99, v50\n" \
    "s_waitcnt lgkmcnt(0)\n" \
    "v_mul_f32 v111, v75, v80\n" \
    "v_fmac_f32 v111, v73, v78\n" \
    "v_fmac_f32 v111, v71, v76\n" \
    "v_add_f32_dpp v53, v120, v53 row_ror:11 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_add_f32_dpp v55, v122, v55 row_ror:11 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_add_f32_dpp v57, v124, v57 row_ror:11 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_mul_f32 v113, v75, v40\n" \
    "v_fmac_f32 v113, v73, v38\n" \
    "v_fmac_f32 v113, v71, v36\n" \
    "v_mul_f32 v121, v81, v80\n" \
    "v_fmac_f32 v121, v79, v78\n" \
    "v_fmac_f32 v121, v77, v76\n" \
    "v_mul_f32 v123, v81, v46\n" \
    "v_fmac_f32 v123, v79, v44\n" \
    "v_fmac_f32 v123, v77, v42\n" \
    "s_cbranch_vccz SD_SKIP6_%=\n" \
    "s_or_b64 %[nl], %[nl], vcc\n" \
    "v_cmp_lt_f32 vcc, v95, v50\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v95, v95, v27, vcc\n" \
    "v_cmp_lt_f32 vcc, v88, v25\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v88, v88, v27, vcc\n" \
    "v_cmp_lt_f32 vcc, v97, v50\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v97, v97, v27, vcc\n" \
    "v_cmp_lt_f32 vcc, v90, v25\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v90, v90, v27, vcc\n" \
    "SD_SKIP6_%=:\n" \
    "v_rsq_f32 v105, v95\n" \
    "v_rsq_f32 v115, v88\n" \
    "v_mul_f32 v94, v105, v105\n" \
    "v_mul_f32 v104, v115, v115\n" \
    "v_mul_f32 v107, v94, v105\n" \
    "v_mul_f32 v117, v104, v115\n" \
    "v_fma_f32 v109, v48, v107, v105\n" \
    "v_fma_f32 v96, v29, v94, 1.0\n" \
    "v_fma_f32 v119, v48, v117, v115\n" \
    "v_fma_f32 v106, v29, v104, 1.0\n" \
    "v_mul_f32 v98, v107, v96\n" \
    "v_mul_f32 v100, v98, v111\n" \
    "v_mul_f32 v102, v98, v113\n" \
    "v_mul_f32 v108, v117, v106\n" \
    "v_mul_f32 v110, v108, v121\n" \
    "v_mul_f32 v112, v108, v123\n" \
    "v_mul_f32 v52, v100, v71\n" \
    "v_fmac_f32 v52, v109, v76\n" \
    "v_mul_f32 v54, v100, v73\n" \
    "v_fmac_f32 v54, v109, v78\n" \
    "v_mul_f32 v56, v100, v75\n" \
    "v_fmac_f32 v56, v109, v80\n" \
    "v_mul_f32 v58, v110, v77\n" \
    "v_fmac_f32 v58, v119, v76\n" \
    "v_mul_f32 v60, v110, v79\n" \
    "v_fmac_f32 v60, v119, v78\n" \
    "v_mul_f32 v62, v110, v81\n" \
    "v_fmac_f32 v62, v119, v80\n" \
    "v_mul_f32 v114, v102, v71\n" \
    "v_fmac_f32 v114, v109, v36\n" \
    "v_mul_f32 v116, v102, v73\n" \
    "v_fmac_f32 v116, v109, v38\n" \
    "v_mul_f32 v118, v102, v75\n" \
    "v_fmac_f32 v118, v109, v40\n" \
    "v_fmac_f32 v114, v112, v77\n" \
    "v_fmac_f32 v114, v119, v42\n" \
    "v_fmac_f32 v116, v112, v79\n" \
    "v_fmac_f32 v116, v119, v44\n" \
    "v_fmac_f32 v118, v112, v81\n" \
    "v_fmac_f32 v118, v119, v46\n" \
    "v_rsq_f32 v105, v97\n" \
    "v_rsq_f32 v115, v90\n" \
    "v_mul_f32 v111, v87, v86\n" \
    "v_fmac_f32 v111, v85, v84\n" \
    "v_fmac_f32 v111, v83, v82\n" \
    "v_mov_b32_dpp v47, v114 row_ror:12 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_mov_b32_dpp v49, v116 row_ror:12 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_mov_b32_dpp v51, v118 row_ror:12 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_mul_f32 v113, v87, v40\n" \
    "v_fmac_f32 v113, v85, v38\n" \
    "v_fmac_f32 v113, v83, v36\n" \
    "v_mul_f32 v121, v93, v86\n" \
    "v_fmac_f32 v121, v91, v84\n" \
    "v_fmac_f32 v121, v89, v82\n" \
    "v_mul_f32 v123, v93, v46\n" \
    "v_fmac_f32 v123, v91, v44\n" \
    "v_fmac_f32 v123, v89, v42\n" \
    "v_mul_f32 v94, v105, v105\n" \
    "v_mul_f32 v104, v115, v115\n" \
    "v_mul_f32 v107, v94, v105\n" \
    "v_mul_f32 v117, v104, v115\n" \
    "v_fma_f32 v109, v48, v107, v105\n" \
    "v_fma_f32 v96, v29, v94, 1.0\n" \
    "v_fma_f32 v119, v48, v117, v115\n" \
    "v_fma_f32 v106, v29, v104, 1.0\n" \
    "v_mul_f32 v98, v107, v96\n" \
    "v_mul_f32 v100, v98, v111\n" \
    "v_mul_f32 v102, v98, v113\n" \
    "v_mul_f32 v108, v117, v106\n" \
    "v_mul_f32 v110, v108, v121\n" \
    "v_mul_f32 v112, v108, v123\n" \
    "v_fmac_f32 v52, v100, v83\n" \
    "v_fmac_f32 v52, v109, v82\n" \
    "v_fmac_f32 v54, v100, v85\n" \
    "v_fmac_f32 v54, v109, v84\n" \
    "v_fmac_f32 v56, v100, v87\n" \
    "v_fmac_f32 v56, v109, v86\n" \
    "v_fmac_f32 v58, v110, v89\n" \
    "v_fmac_f32 v58, v119, v82\n" \
    "v_fmac_f32 v60, v110, v91\n" \
    "v_fmac_f32 v60, v119, v84\n" \
    "v_fmac_f32 v62, v110, v93\n" \
    "v_fmac_f32 v62, v119, v86\n" \
    "v_mul_f32 v120, v102, v83\n" \
    "v_fmac_f32 v120, v109, v36\n" \
    "v_mul_f32 v122, v102, v85\n" \
    "v_fmac_f32 v122, v109, v38\n" \
    "v_mul_f32 v124, v102, v87\n" \
    "v_fmac_f32 v124, v109, v40\n" \
    "v_fmac_f32 v120, v112, v89\n" \
    "v_fmac_f32 v120, v119, v42\n" \
    "v_fmac_f32 v122, v112, v91\n" \
    "v_fmac_f32 v122, v119, v44\n" \
    "v_fmac_f32 v124, v112, v93\n" \
    "v_fmac_f32 v124, v119, v46\n" \
    "ds_read_b32 v59, v31 offset:56\n" \
    "ds_read_b32 v61, v31 offset:184\n" \
    "ds_read_b32 v63, v31 offset:312\n" \
    "ds_read_b32 v65, v31 offset:60\n" \
    "ds_read_b32 v67, v31 offset:188\n" \
    "ds_read_b32 v69, v31 offset:316\n" \
    "ds_read_b32 v76, v31 offset:440\n" \
    "ds_read_b32 v78, v31 offset:568\n" \
    "ds_read_b32 v80, v31 offset:696\n" \
    "ds_read_b32 v82, v31 offset:444\n" \
    "ds_read_b32 v84, v31 offset:572\n" \
    "ds_read_b32 v86, v31 offset:700\n" \
    "s_waitcnt lgkmcnt(9)\n" \
    "v_sub_f32 v71, v24, v59\n" \
    "v_sub_f32 v73, v26, v61\n" \
    "v_sub_f32 v75, v28, v63\n" \
    "v_sub_f32 v77, v30, v59\n" \
    "v_sub_f32 v79, v32, v61\n" \
    "v_sub_f32 v81, v34, v63\n" \
    "v_mul_f32 v95, v75, v75\n" \
    "v_fmac_f32 v95, v73, v73\n" \
    "v_fmac_f32 v95, v71, v71\n" \
    "v_mul_f32 v88, v81, v81\n" \
    "v_fmac_f32 v88, v79, v79\n" \
    "v_fmac_f32 v88, v77, v77\n" \
    "v_min_f32 v99, v95, v88\n" \
    "s_waitcnt lgkmcnt(6)\n" \
    "v_sub_f32 v83, v24, v65\n" \
    "v_sub_f32 v85, v26, v67\n" \
    "v_sub_f32 v87, v28, v69\n" \
    "v_sub_f32 v89, v30, v65\n" \
    "v_sub_f32 v91, v32, v67\n" \
    "v_sub_f32 v93, v34, v69\n" \
    "v_mul_f32 v97, v87, v87\n" \
    "v_fmac_f32 v97, v85, v85\n" \
    "v_fmac_f32 v97, v83, v83\n" \
    "v_mul_f32 v90, v93, v93\n" \
    "v_fmac_f32 v90, v91, v91\n" \
    "v_fmac_f32 v90, v89, v89\n" \
    "v_min_f32 v92, v97, v90\n" \
    "v_min_f32 v99, v99, v92\n" \
    "v_cmp_lt_f32 vcc, v99, v50\n" \
    "s_waitcnt lgkmcnt(0)\n" \
    "v_mul_f32 v111, v75, v80\n" \
    "v_fmac_f32 v111, v73, v78\n" \
    "v_fmac_f32 v111, v71, v76\n" \
    "v_add_f32_dpp v47, v120, v47 row_ror:13 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_add_f32_dpp v49, v122, v49 row_ror:13 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_add_f32_dpp v51, v124, v51 row_ror:13 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_mul_f32 v113, v75, v40\n" \
    "v_fmac_f32 v113, v73, v38\n" \
    "v_fmac_f32 v113, v71, v36\n" \
    "v_mul_f32 v121, v81, v80\n" \
    "v_fmac_f32 v121, v79, v78\n" \
    "v_fmac_f32 v121, v77, v76\n" \
    "v_mul_f32 v123, v81, v46\n" \
    "v_fmac_f32 v123, v79, v44\n" \
    "v_fmac_f32 v123, v77, v42\n" \
    "s_cbranch_vccz SD_SKIP7_%=\n" \
    "s_or_b64 %[nl], %[nl], vcc\n" \
    "v_cmp_lt_f32 vcc, v95, v50\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v95, v95, v27, vcc\n" \
    "v_cmp_lt_f32 vcc, v88, v25\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v88, v88, v27, vcc\n" \
    "v_cmp_lt_f32 vcc, v97, v50\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v97, v97, v27, vcc\n" \
    "v_cmp_lt_f32 vcc, v90, v25\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v90, v90, v27, vcc\n" \
    "SD_SKIP7_%=:\n" \
    "v_rsq_f32 v105, v95\n" \
    "v_rsq_f32 v115, v88\n" \
    "v_mul_f32 v94, v105, v105\n" \
    "v_mul_f32 v104, v115, v115\n" \
    "v_mul_f32 v107, v94, v105\n" \
    "v_mul_f32 v117, v104, v115\n" \
    "v_fma_f32 v109, v48, v107, v105\n" \
    "v_fma_f32 v96, v29, v94, 1.0\n" \
    "v_fma_f32 v119, v48, v117, v115\n" \
    "v_fma_f32 v106, v29, v104, 1.0\n" \
    "v_mul_f32 v98, v107, v96\n" \
    "v_mul_f32 v100, v98, v111\n" \
    "v_mul_f32 v102, v98, v113\n" \
    "v_mul_f32 v108, v117, v106\n" \
    "v_mul_f32 v110, v108, v121\n" \
    "v_mul_f32 v112, v108, v123\n" \
    "v_fmac_f32 v52, v100, v71\n" \
    "v_fmac_f32 v52, v109, v76\n" \
    "v_fmac_f32 v54, v100, v73\n" \
    "v_fmac_f32 v54, v109, v78\n" \
    "v_fmac_f32 v56, v100, v75\n" \
    "v_fmac_f32 v56, v109, v80\n" \
    "v_fmac_f32 v58, v110, v77\n" \
    "v_fmac_f32 v58, v119, v76\n" \
    "v_fmac_f32 v60, v110, v79\n" \
    "v_fmac_f32 v60, v119, v78\n" \
    "v_fmac_f32 v62, v110, v81\n" \
    "v_fmac_f32 v62, v119, v80\n" \
    "v_mul_f32 v114, v102, v71\n" \
    "v_fmac_f32 v114, v109, v36\n" \
    "v_mul_f32 v116, v102, v73\n" \
    "v_fmac_f32 v116, v109, v38\n" \
    "v_mul_f32 v118, v102, v75\n" \
    "v_fmac_f32 v118, v109, v40\n" \
    "v_fmac_f32 v114, v112, v77\n" \
    "v_fmac_f32 v114, v119, v42\n" \
    "v_fmac_f32 v116, v112, v79\n" \
    "v_fmac_f32 v116, v119, v44\n" \
    "v_fmac_f32 v118, v112, v81\n" \
    "v_fmac_f32 v118, v119, v46\n" \
    "v_rsq_f32 v105, v97\n" \
    "v_rsq_f32 v115, v90\n" \
    "v_mul_f32 v111, v87, v86\n" \
    "v_fmac_f32 v111, v85, v84\n" \
    "v_fmac_f32 v111, v83, v82\n" \
    "v_add_f32_dpp v47, v114, v47 row_ror:14 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_add_f32_dpp v49, v116, v49 row_ror:14 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_add_f32_dpp v51, v118, v51 row_ror:14 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_mul_f32 v113, v87, v40\n" \
    "v_fmac_f32 v113, v85, v38\n" \
    "v_fmac_f32 v113, v83, v36\n" \
    "v_mul_f32 v121, v93, v86\n" \
    "v_fmac_f32 v121, v91, v84\n" \
    "v_fmac_f32 v121, v89, v82\n" \
    "v_mul_f32 v123, v93, v46\n" \
    "v_fmac_f32 v123, v91, v44\n" \
    "v_fmac_f32 v123, v89, v42\n" \
    "v_mul_f32 v94, v105, v105\n" \
    "v_mul_f32 v104, v115, v115\n" \
    "v_mul_f32 v107, v94, v105\n" \
    "v_mul_f32 v117, v104, v115\n" \
    "v_fma_f32 v109, v48, v107, v105\n" \
    "v_fma_f32 v96, v29, v94, 1.0\n" \
    "v_fma_f32 v119, v48, v117, v115\n" \
    "v_fma_f32 v106, v29, v104, 1.0\n" \
    "v_mul_f32 v98, v107, v96\n" \
    "v_mul_f32 v100, v98, v111\n" \
    "v_mul_f32 v102, v98, v113\n" \
    "v_mul_f32 v108, v117, v106\n" \
    "v_mul_f32 v110, v108, v121\n" \
    "v_mul_f32 v112, v108, v123\n" \
    "v_fmac_f32 v52, v100, v83\n" \
    "v_fmac_f32 v52, v109, v82\n" \
    "v_fmac_f32 v54, v100, v85\n" \
    "v_fmac_f32 v54, v109, v84\n" \
    "v_fmac_f32 v56, v100, v87\n" \
    "v_fmac_f32 v56, v109, v86\n" \
    "v_fmac_f32 v58, v110, v89\n" \
    "v_fmac_f32 v58, v119, v82\n" \
    "v_fmac_f32 v60, v110, v91\n" \
    "v_fmac_f32 v60, v119, v84\n" \
    "v_fmac_f32 v62, v110, v93\n" \
    "v_fmac_f32 v62, v119, v86\n" \
    "v_mul_f32 v120, v102, v83\n" \
    "v_fmac_f32 v120, v109, v36\n" \
    "v_mul_f32 v122, v102, v85\n" \
    "v_fmac_f32 v122, v109, v38\n" \
    "v_mul_f32 v124, v102, v87\n" \
    "v_fmac_f32 v124, v109, v40\n" \
    "v_fmac_f32 v120, v112, v89\n" \
    "v_fmac_f32 v120, v119, v42\n" \
    "v_fmac_f32 v122, v112, v91\n" \
    "v_fmac_f32 v122, v119, v44\n" \
    "v_fmac_f32 v124, v112, v93\n" \
    "v_fmac_f32 v124, v119, v46\n" \
    "v_add_f32 v35, v35, v52\n" \
    "v_add_f32 v37, v37, v54\n" \
    "v_add_f32 v39, v39, v56\n" \
    "v_add_f32 v41, v41, v58\n" \
    "v_add_f32 v43, v43, v60\n" \
    "v_add_f32 v45, v45, v62\n" \
    "s_nop 1\n" \
    "v_add_f32_dpp v47, v120, v47 row_ror:15 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_add_f32_dpp v49, v122, v49 row_ror:15 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_add_f32_dpp v51, v124, v51 row_ror:15 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_add_f32 v53, v53, v47\n" \
    "v_add_f32 v55, v55, v49\n" \
    "v_add_f32 v57, v57, v51\n" \
    "ds_write_b32 v33, v53 offset:768\n" \
    "ds_write_b32 v33, v55 offset:832\n" \
    "ds_write_b32 v33, v57 offset:896\n" \
    "v_add_f32 v125, v64, v35\n" \
    "v_sub_f32 v126, v125, v64\n" \
    "v_sub_f32 v35, v35, v126\n" \
    "v_mov_b32 v64, v125\n" \
    "v_add_f32 v125, v66, v37\n" \
    "v_sub_f32 v126, v125, v66\n" \
    "v_sub_f32 v37, v37, v126\n" \
    "v_mov_b32 v66, v125\n" \
    "v_add_f32 v125, v68, v39\n" \
    "v_sub_f32 v126, v125, v68\n" \
    "v_sub_f32 v39, v39, v126\n" \
    "v_mov_b32 v68, v125\n" \
    "v_add_f32 v125, v70, v41\n" \
    "v_sub_f32 v126, v125, v70\n" \
    "v_sub_f32 v41, v41, v126\n" \
    "v_mov_b32 v70, v125\n" \
    "v_add_f32 v125, v72, v43\n" \
    "v_sub_f32 v126, v125, v72\n" \
    "v_sub_f32 v43, v43, v126\n" \
    "v_mov_b32 v72, v125\n" \
    "v_add_f32 v125, v74, v45\n" \
    "v_sub_f32 v126, v125, v74\n" \
    "v_sub_f32 v45, v45, v126\n" \
    "v_mov_b32 v74, v125\n"

// one chunk; 1417 instructions per chunk, 0 products with same-parity sources
#define SD_WAVE_CHUNK_RPY_PER \
    "ds_read_b32 v59, v31 offset:0\n" \
    "ds_read_b32 v61, v31 offset:128\n" \
    "ds_read_b32 v63, v31 offset:256\n" \
    "ds_read_b32 v65, v31 offset:4\n" \
    "ds_read_b32 v67, v31 offset:132\n" \
    "ds_read_b32 v69, v31 offset:260\n" \
    "ds_read_b32 v76, v31 offset:384\n" \
    "ds_read_b32 v78, v31 offset:512\n" \
    "ds_read_b32 v80, v31 offset:640\n" \
    "ds_read_b32 v82, v31 offset:388\n" \
    "ds_read_b32 v84, v31 offset:516\n" \
    "ds_read_b32 v86, v31 offset:644\n" \
    "s_waitcnt lgkmcnt(9)\n" \
    "v_sub_u32 v101, v24, v59\n" \
    "v_cvt_f32_i32 v71, v101\n" \
    "v_sub_u32 v101, v26, v61\n" \
    "v_cvt_f32_i32 v73, v101\n" \
    "v_sub_u32 v101, v28, v63\n" \
    "v_cvt_f32_i32 v75, v101\n" \
    "v_sub_u32 v103, v30, v59\n" \
    "v_cvt_f32_i32 v77, v103\n" \
    "v_sub_u32 v103, v32, v61\n" \
    "v_cvt_f32_i32 v79, v103\n" \
    "v_sub_u32 v103, v34, v63\n" \
    "v_cvt_f32_i32 v81, v103\n" \
    "v_mul_f32 v95, v75, v75\n" \
    "v_fmac_f32 v95, v73, v73\n" \
    "v_fmac_f32 v95, v71, v71\n" \
    "v_mul_f32 v88, v81, v81\n" \
    "v_fmac_f32 v88, v79, v79\n" \
    "v_fmac_f32 v88, v77, v77\n" \
    "v_min_f32 v99, v95, v88\n" \
    "s_waitcnt lgkmcnt(6)\n" \
    "v_sub_u32 v101, v24, v65\n" \
    "v_cvt_f32_i32 v83, v101\n" \
    "v_sub_u32 v101, v26, v67\n" \
    "v_cvt_f32_i32 v85, v101\n" \
    "v_sub_u32 v101, v28, v69\n" \
    "v_cvt_f32_i32 v87, v101\n" \
    "v_sub_u32 v103, v30, v65\n" \
    "v_cvt_f32_i32 v89, v103\n" \
    "v_sub_u32 v103, v32, v67\n" \
    "v_cvt_f32_i32 v91, v103\n" \
    "v_sub_u32 v103, v34, v69\n" \
    "v_cvt_f32_i32 v93, v103\n" \
    "v_mul_f32 v97, v87, v87\n" \
    "v_fmac_f32 v97, v85, v85\n" \
    "v_fmac_f32 v97, v83, v83\n" \
    "v_mul_f32 v90, v93, v93\n" \
    "v_fmac_f32 v90, v91, v91\n" \
    "v_fmac_f32 v90, v89, v89\n" \
    "v_min_f32 v92, v97, v90\n" \
    "v_min_f32 v99, v99, v92\n" \
    "v_cmp_lt_f32 vcc, v99, v50\n" \
    "s_waitcnt lgkmcnt(0)\n" \
    "v_mul_f32 v111, v75, v80\n" \
    "v_fmac_f32 v111, v73, v78\n" \
    "v_fmac_f32 v111, v71, v76\n" \
    "v_mul_f32 v113, v75, v40\n" \
    "v_fmac_f32 v113, v73, v38\n" \
    "v_fmac_f32 v113, v71, v36\n" \
    "v_mul_f32 v121, v81, v80\n" \
    "v_fmac_f32 v121, v79, v78\n" \
    "v_fmac_f32 v121, v77, v76\n" \
    "v_mul_f32 v123, v81, v46\n" \
    "v_fmac_f32 v123, v79, v44\n" \
    "v_fmac_f32 v123, v77, v42\n" \
    "s_cbranch_vccz SD_SKIP0_%=\n" \
    "s_or_b64 %[nl], %[nl], vcc\n" \
    "v_cmp_lt_f32 vcc, v95, v50\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v95, v95, v27, vcc\n" \
    "v_cmp_lt_f32 vcc, v88, v25\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v88, v88, v27, vcc\n" \
    "v_cmp_lt_f32 vcc, v97, v50\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v97, v97, v27, vcc\n" \
    "v_cmp_lt_f32 vcc, v90, v25\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v90, v90, v27, vcc\n" \
    "SD_SKIP0_%=:\n" \
    "v_rsq_f32 v105, v95\n" \
    "v_rsq_f32 v115, v88\n" \
    "v_mul_f32 v94, v105, v105\n" \
    "v_mul_f32 v104, v115, v115\n" \
    "v_mul_f32 v107, v94, v105\n" \
    "v_mul_f32 v117, v104, v115\n" \
    "v_fma_f32 v109, v48, v107, v105\n" \
    "v_fma_f32 v96, v29, v94, 1.0\n" \
    "v_fma_f32 v119, v48, v117, v115\n" \
    "v_fma_f32 v106, v29, v104, 1.0\n" \
    "v_mul_f32 v98, v107, v96\n" \
    "v_mul_f32 v100, v98, v111\n" \
    "v_mul_f32 v102, v98, v113\n" \
    "v_mul_f32 v108, v117, v106\n" \
    "v_mul_f32 v110, v108, v121\n" \
    "v_mul_f32 v112, v108, v123\n" \
    "v_mul_f32 v52, v100, v71\n" \
    "v_fmac_f32 v52, v109, v76\n" \
    "v_mul_f32 v54, v100, v73\n" \
    "v_fmac_f32 v54, v109, v78\n" \
    "v_mul_f32 v56, v100, v75\n" \
    "v_fmac_f32 v56, v109, v80\n" \
    "v_mul_f32 v58, v110, v77\n" \
    "v_fmac_f32 v58, v119, v76\n" \
    "v_mul_f32 v60, v110, v79\n" \
    "v_fmac_f32 v60, v119, v78\n" \
    "v_mul_f32 v62, v110, v81\n" \
    "v_fmac_f32 v62, v119, v80\n" \
    "v_mul_f32 v53, v102, v71\n" \
    "v_fmac_f32 v53, v109, v36\n" \
    "v_mul_f32 v55, v102, v73\n" \
    "v_fmac_f32 v55, v109, v38\n" \
    "v_mul_f32 v57, v102, v75\n" \
    "v_fmac_f32 v57, v109, v40\n" \
    "v_fmac_f32 v53, v112, v77\n" \
    "v_fmac_f32 v53, v119, v42\n" \
    "v_fmac_f32 v55, v112, v79\n" \
    "v_fmac_f32 v55, v119, v44\n" \
    "v_fmac_f32 v57, v112, v81\n" \
    "v_fmac_f32 v57, v119, v46\n" \
    "v_rsq_f32 v105, v97\n" \
    "v_rsq_f32 v115, v90\n" \
    "v_mul_f32 v111, v87, v86\n" \
    "v_fmac_f32 v111, v85, v84\n" \
    "v_fmac_f32 v111, v83, v82\n" \
    "v_mul_f32 v113, v87, v40\n" \
    "v_fmac_f32 v113, v85, v38\n" \
    "v_fmac_f32 v113, v83, v36\n" \
    "v_mul_f32 v121, v93, v86\n" \
    "v_fmac_f32 v121, v91, v84\n" \
    "v_fmac_f32 v121, v89, v82\n" \
    "v_mul_f32 v123, v93, v46\n" \
    "v_fmac_f32 v123, v91, v44\n" \
    "v_fmac_f32 v123, v89, v42\n" \
    "v_mul_f32 v94, v105, v105\n" \
    "v_mul_f32 v104, v115, v115\n" \
    "v_mul_f32 v107, v94, v105\n" \
    "v_mul_f32 v117, v104, v115\n" \
    "v_fma_f32 v109, v48, v107, v105\n" \
    "v_fma_f32 v96, v29, v94, 1.0\n" \
    "v_fma_f32 v119, v48, v117, v115\n" \
    "v_fma_f32 v106, v29, v104, 1.0\n" \
    "v_mul_f32 v98, v107, v96\n" \
    "v_mul_f32 v100, v98, v111\n" \
    "v_mul_f32 v102, v98, v113\n" \
    "v_mul_f32 v108, v117, v106\n" \
    "v_mul_f32 v110, v108, v121\n" \
    "v_mul_f32 v112, v108, v123\n" \
    "v_fmac_f32 v52, v100, v83\n" \
    "v_fmac_f32 v52, v109, v82\n" \
    "v_fmac_f32 v54, v100, v85\n" \
    "v_fmac_f32 v54, v109, v84\n" \
    "v_fmac_f32 v56, v100, v87\n" \
    "v_fmac_f32 v56, v109, v86\n" \
    "v_fmac_f32 v58, v110, v89\n" \
    "v_fmac_f32 v58, v119, v82\n" \
    "v_fmac_f32 v60, v110, v91\n" \
    "v_fmac_f32 v60, v119, v84\n" \
    "v_fmac_f32 v62, v110, v93\n" \
    "v_fmac_f32 v62, v119, v86\n" \
    "v_mul_f32 v120, v102, v83\n" \
    "v_fmac_f32 v120, v109, v36\n" \
    "v_mul_f32 v122, v102, v85\n" \
    "v_fmac_f32 v122, v109, v38\n" \
    "v_mul_f32 v124, v102, v87\n" \
    "v_fmac_f32 v124, v109, v40\n" \
    "v_fmac_f32 v120, v112, v89\n" \
    "v_fmac_f32 v120, v119, v42\n" \
    "v_fmac_f32 v122, v112, v91\n" \
    "v_fmac_f32 v122, v119, v44\n" \
    "v_fmac_f32 v124, v112, v93\n" \
    "v_fmac_f32 v124, v119, v46\n" \
    "ds_read_b32 v59, v31 offset:8\n" \
    "ds_read_b32 v61, v31 offset:136\n" \
    "ds_read_b32 v63, v31 offset:264\n" \
    "ds_read_b32 v65, v31 offset:12\n" \
    "ds_read_b32 v67, v31 offset:140\n" \
    "ds_read_b32 v69, v31 offset:268\n" \
    "ds_read_b32 v76, v31 offset:392\n" \
    "ds_read_b32 v78, v31 offset:520\n" \
    "ds_read_b32 v80, v31 offset:648\n" \
    "ds_read_b32 v82, v31 offset:396\n" \
    "ds_read_b32 v84, v31 offset:524\n" \
    "ds_read_b32 v86, v31 offset:652\n" \
    "s_waitcnt lgkmcnt(9)\n" \
    "v_sub_u32 v101, v24, v59\n" \
    "v_cvt_f32_i32 v71, v101\n" \
    "v_sub_u32 v101, v26, v61\n" \
    "v_cvt_f32_i32 v73, v101\n" \
    "v_sub_u32 v101, v28, v63\n" \
    "v_cvt_f32_i32 v75, v101\n" \
    "v_sub_u32 v103, v30, v59\n" \
    "v_cvt_f32_i32 v77, v103\n" \
    "v_sub_u32 v103, v32, v61\n" \
    "v_cvt_f32_i32 v79, v103\n" \
    "v_sub_u32 v103, v34, v63\n" \
    "v_cvt_f32_i32 v81, v103\n" \
    "v_mul_f32 v95, v75, v75\n" \
    "v_fmac_f32 v95, v73, v73\n" \
    "v_fmac_f32 v95, v71, v71\n" \
    "v_mul_f32 v88, v81, v81\n" \
    "v_fmac_f32 v88, v79, v79\n" \
    "v_fmac_f32 v88, v77, v77\n" \
    "v_min_f32 v99, v95, v88\n" \
    "s_waitcnt lgkmcnt(6)\n" \
    "v_sub_u32 v101, v24, v65\n" \
    "v_cvt_f32_i32 v83, v101\n" \
    "v_sub_u32 v101, v26, v67\n" \
    "v_cvt_f32_i32 v85, v101\n" \
    "v_sub_u32 v101, v28, v69\n" \
    "v_cvt_f32_i32 v87, v101\n" \
    "v_sub_u32 v103, v30, v65\n" \
    "v_cvt_f32_i32 v89, v103\n" \
    "v_sub_u32 v103, v32, v67\n" \
    "v_cvt_f32_i32 v91, v103\n" \
    "v_sub_u32 v103, v34, v69\n" \
    "v_cvt_f32_i32 v93, v103\n" \
    "v_mul_f32 v97, v87, v87\n" \
    "v_fmac_f32 v97, v85, v85\n" \
    "v_fmac_f32 v97, v83, v83\n" \
    "v_mul_f32 v90, v93, v93\n" \
    "v_fmac_f32 v90, v91, v91\n" \
    "v_fmac_f32 v90, v89, v89\n" \
    "v_min_f32 v92, v97, v90\n" \
    "v_min_f32 v99, v99, v92\n" \
    "v_cmp_lt_f32 vcc, v99, v50\n" \
    "s_waitcnt lgkmcnt(0)\n" \
    "v_mul_f32 v111, v75, v80\n" \
    "v_fmac_f32 v111, v73, v78\n" \
    "v_fmac_f32 v111, v71, v76\n" \
    "v_add_f32_dpp v53, v120, v53 row_ror:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_add_f32_dpp v55, v122, v55 row_ror:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_add_f32_dpp v57, v124, v57 row_ror:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_mul_f32 v113, v75, v40\n" \
    "v_fmac_f32 v113, v73, v38\n" \
    "v_fmac_f32 v113, v71, v36\n" \
    "v_mul_f32 v121, v81, v80\n" \
    "v_fmac_f32 v121, v79, v78\n" \
    "v_fmac_f32 v121, v77, v76\n" \
    "v_mul_f32 v123, v81, v46\n" \
    "v_fmac_f32 v123, v79, v44\n" \
    "v_fmac_f32 v123, v77, v42\n" \
    "s_cbranch_vccz SD_SKIP1_%=\n" \
    "s_or_b64 %[nl], %[nl], vcc\n" \
    "v_cmp_lt_f32 vcc, v95, v50\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v95, v95, v27, vcc\n" \
    "v_cmp_lt_f32 vcc, v88, v25\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v88, v88, v27, vcc\n" \
    "v_cmp_lt_f32 vcc, v97, v50\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v97, v97, v27, vcc\n" \
    "v_cmp_lt_f32 vcc, v90, v25\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v90, v90, v27, vcc\n" \
    "SD_SKIP1_%=:\n" \
    "v_rsq_f32 v105, v95\n" \
    "v_rsq_f32 v115, v88\n" \
    "v_mul_f32 v94, v105, v105\n" \
    "v_mul_f32 v104, v115, v115\n" \
    "v_mul_f32 v107, v94, v105\n" \
    "v_mul_f32 v117, v104, v115\n" \
    "v_fma_f32 v109, v48, v107, v105\n" \
    "v_fma_f32 v96, v29, v94, 1.0\n" \
    "v_fma_f32 v119, v48, v117, v115\n" \
    "v_fma_f32 v106, v29, v104, 1.0\n" \
    "v_mul_f32 v98, v107, v96\n" \
    "v_mul_f32 v100, v98, v111\n" \
    "v_mul_f32 v102, v98, v113\n" \
    "v_mul_f32 v108, v117, v106\n" \
    "v_mul_f32 v110, v108, v121\n" \
    "v_mul_f32 v112, v108, v123\n" \
    "v_fmac_f32 v52, v100, v71\n" \
    "v_fmac_f32 v52, v109, v76\n" \
    "v_fmac_f32 v54, v100, v73\n" \
    "v_fmac_f32 v54, v109, v78\n" \
    "v_fmac_f32 v56, v100, v75\n" \
    "v_fmac_f32 v56, v109, v80\n" \
    "v_fmac_f32 v58, v110, v77\n" \
    "v_fmac_f32 v58, v119, v76\n" \
    "v_fmac_f32 v60, v110, v79\n" \
    "v_fmac_f32 v60, v119, v78\n" \
    "v_fmac_f32 v62, v110, v81\n" \
    "v_fmac_f32 v62, v119, v80\n" \
    "v_mul_f32 v114, v102, v71\n" \
    "v_fmac_f32 v114, v109, v36\n" \
    "v_mul_f32 v116, v102, v73\n" \
    "v_fmac_f32 v116, v109, v38\n" \
    "v_mul_f32 v118, v102, v75\n" \
    "v_fmac_f32 v118, v109, v40\n" \
    "v_fmac_f32 v114, v112, v77\n" \
    "v_fmac_f32 v114, v119, v42\n" \
    "v_fmac_f32 v116, v112, v79\n" \
    "v_fmac_f32 v116, v119, v44\n" \
    "v_fmac_f32 v118, v112, v81\n" \
    "v_fmac_f32 v118, v119, v46\n" \
    "v_rsq_f32 v105, v97\n" \
    "v_rsq_f32 v115, v90\n" \
    "v_mul_f32 v111, v87, v86\n" \
    "v_fmac_f32 v111, v85, v84\n" \
    "v_fmac_f32 v111, v83, v82\n" \
    "v_add_f32_dpp v53, v114, v53 row_ror:2 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_add_f32_dpp v55, v116, v55 row_ror:2 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_add_f32_dpp v57, v118, v57 row_ror:2 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_mul_f32 v113, v87, v40\n" \
    "v_fmac_f32 v113, v85, v38\n" \
    "v_fmac_f32 v113, v83, v36\n" \
    "v_mul_f32 v121, v93, v86\n" \
    "v_fmac_f32 v121, v91, v84\n" \
    "v_fmac_f32 v121, v89, v82\n" \
    "v_mul_f32 v123, v93, v46\n" \
    "v_fmac_f32 v123, v91, v44\n" \
    "v_fmac_f32 v123, v89, v42\n" \
    "v_mul_f32 v94, v105, v105\n" \
    "v_mul_f32 v104, v115, v115\n" \
    "v_mul_f32 v107, v94, v105\n" \
    "v_mul_f32 v117, v104, v115\n" \
    "v_fma_f32 v109, v48, v107, v105\n" \
    "v_fma_f32 v96, v29, v94, 1.0\n" \
    "v_fma_f32 v119, v48, v117, v115\n" \
    "v_fma_f32 v106, v29, v104, 1.0\n" \
    "v_mul_f32 v98, v107, v96\n" \
    "v_mul_f32 v100, v98, v111\n" \
    "v_mul_f32 v102, v98, v113\n" \
    "v_mul_f32 v108, v117, v106\n" \
    "v_mul_f32 v110, v108, v121\n" \
    "v_mul_f32 v112, v108, v123\n" \
    "v_fmac_f32 v52, v100, v83\n" \
    "v_fmac_f32 v52, v109, v82\n" \
    "v_fmac_f32 v54, v100, v85\n" \
    "v_fmac_f32 v54, v109, v84\n" \
    "v_fmac_f32 v56, v100, v87\n" \
    "v_fmac_f32 v56, v109, v86\n" \
    "v_fmac_f32 v58, v110, v89\n" \
    "v_fmac_f32 v58, v119, v82\n" \
    "v_fmac_f32 v60, v110, v91\n" \
    "v_fmac_f32 v60, v119, v84\n" \
    "v_fmac_f32 v62, v110, v93\n" \
    "v_fmac_f32 v62, v119, v86\n" \
    "v_mul_f32 v120, v102, v83\n" \
    "v_fmac_f32 v120, v109, v36\n" \
    "v_mul_f32 v122, v102, v85\n" \
    "v_fmac_f32 v122, v109, v38\n" \
    "v_mul_f32 v124, v102, v87\n" \
    "v_fmac_f32 v124, v109, v40\n" \
    "v_fmac_f32 v120, v112, v89\n" \
    "v_fmac_f32 v120, v119, v42\n" \
    "v_fmac_f32 v122, v112, v91\n" \
    "v_fmac_f32 v122, v119, v44\n" \
    "v_fmac_f32 v124, v112, v93\n" \
    "v_fmac_f32 v124, v119, v46\n" \
    "v_add_f32 v35, v35, v52\n" \
    "v_add_f32 v37, v37, v54\n" \
    "v_add_f32 v39, v39, v56\n" \
    "v_add_f32 v41, v41, v58\n" \
    "v_add_f32 v43, v43, v60\n" \
    "v_add_f32 v45, v45, v62\n" \
    "ds_read_b32 v59, v31 offset:16\n" \
    "ds_read_b32 v61, v31 offset:144\n" \
    "ds_read_b32 v63, v31 offset:272\n" \
    "ds_read_b32 v65, v31 offset:20\n" \
    "ds_read_b32 v67, v31 offset:148\n" \
    "ds_read_b32 v69, v31 offset:276\n" \
    "ds_read_b32 v76, v31 offset:400\n" \
    "ds_read_b32 v78, v31 offset:528\n" \
    "ds_read_b32 v80, v31 offset:656\n" \
    "ds_read_b32 v82, v31 offset:404\n" \
    "ds_read_b32 v84, v31 offset:532\n" \
    "ds_read_b32 v86, v31 offset:660\n" \
    "s_waitcnt lgkmcnt(9)\n" \
    "v_sub_u32 v101, v24, v59\n" \
    "v_cvt_f32_i32 v71, v101\n" \
    "v_sub_u32 v101, v26, v61\n" \
    "v_cvt_f32_i32 v73, v101\n" \
    "v_sub_u32 v101, v28, v63\n" \
    "v_cvt_f32_i32 v75, v101\n" \
    "v_sub_u32 v103, v30, v59\n" \
    "v_cvt_f32_i32 v77, v103\n" \
    "v_sub_u32 v103, v32, v61\n" \
    "v_cvt_f32_i32 v79, v103\n" \
    "v_sub_u32 v103, v34, v63\n" \
    "v_cvt_f32_i32 v81, v103\n" \
    "v_mul_f32 v95, v75, v75\n" \
    "v_fmac_f32 v95, v73, v73\n" \
    "v_fmac_f32 v95, v71, v71\n" \
    "v_mul_f32 v88, v81, v81\n" \
    "v_fmac_f32 v88, v79, v79\n" \
    "v_fmac_f32 v88, v77, v77\n" \
    "v_min_f32 v99, v95, v88\n" \
    "s_waitcnt lgkmcnt(6)\n" \
    "v_sub_u32 v101, v24, v65\n" \
    "v_cvt_f32_i32 v83, v101\n" \
    "v_sub_u32 v101, v26, v67\n" \
    "v_cvt_f32_i32 v85, v101\n" \
    "v_sub_u32 v101, v28, v69\n" \
    "v_cvt_f32_i32 v87, v101\n" \
    "v_sub_u32 v103, v30, v65\n" \
    "v_cvt_f32_i32 v89, v103\n" \
    "v_sub_u32 v103, v32, v67\n" \
    "v_cvt_f32_i32 v91, v103\n" \
    "v_sub_u32 v103, v34, v69\n" \
    "v_cvt_f32_i32 v93, v103\n" \
    "v_mul_f32 v97, v87, v87\n" \
    "v_fmac_f32 v97, v85, v85\n" \
    "v_fmac_f32 v97, v83, v83\n" \
    "v_mul_f32 v90, v93, v93\n" \
    "v_fmac_f32 v90, v91, v91\n" \
    "v_fmac_f32 v90, v89, v89\n" \
    "v_min_f32 v92, v97, v90\n" \
    "v_min_f32 v99, v99, v92\n" \
    "v_cmp_lt_f32 vcc, v99, v50\n" \
    "s_waitcnt lgkmcnt(0)\n" \
    "v_mul_f32 v111, v75, v80\n" \
    "v_fmac_f32 v111, v73, v78\n" \
    "v_fmac_f32 v111, v71, v76\n" \
    "v_add_f32_dpp v53, v120, v53 row_ror:3 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_add_f32_dpp v55, v122, v55 row_ror:3 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_add_f32_dpp v57, v124, v57 row_ror:3 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_mul_f32 v113, v75, v40\n" \
    "v_fmac_f32 v113, v73, v38\n" \
    "v_fmac_f32 v113, v71, v36\n" \
    "v_mul_f32 v121, v81, v80\n" \
    "v_fmac_f32 v121, v79, v78\n" \
    "v_fmac_f32 v121, v77, v76\n" \
    "v_mul_f32 v123, v81, v46\n" \
    "v_fmac_f32 v123, v79, v44\n" \
    "v_fmac_f32 v123, v77, v42\n" \
    "s_cbranch_vccz SD_SKIP2_%=\n" \
    "s_or_b64 %[nl], %[nl], vcc\n" \
    "v_cmp_lt_f32 vcc, v95, v50\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v95, v95, v27, vcc\n" \
    "v_cmp_lt_f32 vcc, v88, v25\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v88, v88, v27, vcc\n" \
    "v_cmp_lt_f32 vcc, v97, v50\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v97, v97, v27, vcc\n" \
    "v_cmp_lt_f32 vcc, v90, v25\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v90, v90, v27, vcc\n" \
    "SD_SKIP2_%=:\n" \
    "v_rsq_f32 v105, v95\n" \
    "v_rsq_f32 v115, v88\n" \
    "v_mul_f32 v94, v105, v105\n" \
    "v_mul_f32 v104, v115, v115\n" \
    "v_mul_f32 v107, v94, v105\n" \
    "v_mul_f32 v117, v104, v115\n" \
    "v_fma_f32 v109, v48, v107, v105\n" \
    "v_fma_f32 v96, v29, v94, 1.0\n" \
    "v_fma_f32 v119, v48, v117, v115\n" \
    "v_fma_f32 v106, v29, v104, 1.0\n" \
    "v_mul_f32 v98, v107, v96\n" \
    "v_mul_f32 v100, v98, v111\n" \
    "v_mul_f32 v102, v98, v113\n" \
    "v_mul_f32 v108, v117, v106\n" \
    "v_mul_f32 v110, v108, v121\n" \
    "v_mul_f32 v112, v108, v123\n" \
    "v_mul_f32 v52, v100, v71\n" \
    "v_fmac_f32 v52, v109, v76\n" \
    "v_mul_f32 v54, v100, v73\n" \
    "v_fmac_f32 v54, v109, v78\n" \
    "v_mul_f32 v56, v100, v75\n" \
    "v_fmac_f32 v56, v109, v80\n" \
    "v_mul_f32 v58, v110, v77\n" \
    "v_fmac_f32 v58, v119, v76\n" \
    "v_mul_f32 v60, v110, v79\n" \
    "v_fmac_f32 v60, v119, v78\n" \
    "v_mul_f32 v62, v110, v81\n" \
    "v_fmac_f32 v62, v119, v80\n" \
    "v_mul_f32 v114, v102, v71\n" \
    "v_fmac_f32 v114, v109, v36\n" \
    "v_mul_f32 v116, v102, v73\n" \
    "v_fmac_f32 v116, v109, v38\n" \
    "v_mul_f32 v118, v102, v75\n" \
    "v_fmac_f32 v118, v109, v40\n" \
    "v_fmac_f32 v114, v112, v77\n" \
    "v_fmac_f32 v114, v119, v42\n" \
    "v_fmac_f32 v116, v112, v79\n" \
    "v_fmac_f32 v116, v119, v44\n" \
    "v_fmac_f32 v118, v112, v81\n" \
    "v_fmac_f32 v118, v119, v46\n" \
    "v_rsq_f32 v105, v97\n" \
    "v_rsq_f32 v115, v90\n" \
    "v_mul_f32 v111, v87, v86\n" \
    "v_fmac_f32 v111, v85, v84\n" \
    "v_fmac_f32 v111, v83, v82\n" \
    "v_mov_b32_dpp v47, v114 row_ror:4 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_mov_b32_dpp v49, v116 row_ror:4 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_mov_b32_dpp v51, v118 row_ror:4 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_mul_f32 v113, v87, v40\n" \
    "v_fmac_f32 v113, v85, v38\n" \
    "v_fmac_f32 v113, v83, v36\n" \
    "v_mul_f32 v121, v93, v86\n" \
    "v_fmac_f32 v121, v91, v84\n" \
    "v_fmac_f32 v121, v89, v82\n" \
    "v_mul_f32 v123, v93, v46\n" \
    "v_fmac_f32 v123, v91, v44\n" \
    "v_fmac_f32 v123, v89, v42\n" \
    "v_mul_f32 v94, v105, v105\n" \
    "v_mul_f32 v104, v115, v115\n" \
    "v_mul_f32 v107, v94, v105\n" \
    "v_mul_f32 v117, v104, v115\n" \
    "v_fma_f32 v109, v48, v107, v105\n" \
    "v_fma_f32 v96, v29, v94, 1.0\n" \
    "v_fma_f32 v119, v48, v117, v115\n" \
    "v_fma_f32 v106, v29, v104, 1.0\n" \
    "v_mul_f32 v98, v107, v96\n" \
    "v_mul_f32 v100, v98, v111\n" \
    "v_mul_f32 v102, v98, v113\n" \
    "v_mul_f32 v108, v117, v106\n" \
    "v_mul_f32 v110, v108, v121\n" \
    "v_mul_f32 v112, v108, v123\n" \
    "v_fmac_f32 v52, v100, v83\n" \
    "v_fmac_f32 v52, v109, v82\n" \
    "v_fmac_f32 v54, v100, v85\n" \
    "v_fmac_f32 v54, v109, v84\n" \
    "v_fmac_f32 v56, v100, v87\n" \
    "v_fmac_f32 v56, v109, v86\n" \
    "v_fmac_f32 v58, v110, v89\n" \
    "v_fmac_f32 v58, v119, v82\n" \
    "v_fmac_f32 v60, v110, v91\n" \
    "v_fmac_f32 v60, v119, v84\n" \
    "v_fmac_f32 v62, v110, v93\n" \
    "v_fmac_f32 v62, v119, v86\n" \
    "v_mul_f32 v120, v102, v83\n" \
    "v_fmac_f32 v120, v109, v36\n" \
    "v_mul_f32 v122, v102, v85\n" \
    "v_fmac_f32 v122, v109, v38\n" \
    "v_mul_f32 v124, v102, v87\n" \
    "v_fmac_f32 v124, v109, v40\n" \
    "v_fmac_f32 v120, v112, v89\n" \
    "v_fmac_f32 v120, v119, v42\n" \
    "v_fmac_f32 v122, v112, v91\n" \
    "v_fmac_f32 v122, v119, v44\n" \
    "v_fmac_f32 v124, v112, v93\n" \
    "v_fmac_f32 v124, v119, v46\n" \
    "ds_read_b32 v59, v31 offset:24\n" \
    "ds_read_b32 v61, v31 offset:152\n" \
    "ds_read_b32 v63, v31 offset:280\n" \
    "ds_read_b32 v65, v31 offset:28\n" \
    "ds_read_b32 v67, v31 offset:156\n" \
    "ds_read_b32 v69, v31 offset:284\n" \
    "ds_read_b32 v76, v31 offset:408\n" \
    "ds_read_b32 v78, v31 offset:536\n" \
    "ds_read_b32 v80, v31 offset:664\n" \
    "ds_read_b32 v82, v31 offset:412\n" \
    "ds_read_b32 v84, v31 offset:540\n" \
    "ds_read_b32 v86, v31 offset:668\n" \
    "s_waitcnt lgkmcnt(9)\n" \
    "v_sub_u32 v101, v24, v59\n" \
    "v_cvt_f32_i32 v71, v101\n" \
    "v_sub_u32 v101, v26, v61\n" \
    "v_cvt_f32_i32 v73, v101\n" \
    "v_sub_u32 v101, v28, v63\n" \
    "v_cvt_f32_i32 v75, v101\n" \
    "v_sub_u32 v103, v30, v59\n" \
    "v_cvt_f32_i32 v77, v103\n" \
    "v_sub_u32 v103, v32, v61\n" \
    "v_cvt_f32_i32 v79, v103\n" \
    "v_sub_u32 v103, v34, v63\n" \
    "v_cvt_f32_i32 v81, v103\n" \
    "v_mul_f32 v95, v75, v75\n" \
    "v_fmac_f32 v95, v73, v73\n" \
    "v_fmac_f32 v95, v71, v71\n" \
    "v_mul_f32 v88, v81, v81\n" \
    "v_fmac_f32 v88, v79, v79\n" \
    "v_fmac_f32 v88, v77, v77\n" \
    "v_min_f32 v99, v95, v88\n" \
    "s_waitcnt lgkmcnt(6)\n" \
    "v_sub_u32 v101, v24, v65\n" \
    "v_cvt_f32_i32 v83, v101\n" \
    "v_sub_u32 v101, v26, v67\n" \
    "v_cvt_f32_i32 v85, v101\n" \
    "v_sub_u32 v101, v28, v69\n" \
    "v_cvt_f32_i32 v87, v101\n" \
    "v_sub_u32 v103, v30, v65\n" \
    "v_cvt_f32_i32 v89, v103\n" \
    "v_sub_u32 v103, v32, v67\n" \
    "v_cvt_f32_i32 v91, v103\n" \
    "v_sub_u32 v103, v34, v69\n" \
    "v_cvt_f32_i32 v93, v103\n" \
    "v_mul_f32 v97, v87, v87\n" \
    "v_fmac_f32 v97, v85, v85\n" \
    "v_fmac_f32 v97, v83, v83\n" \
    "v_mul_f32 v90, v93, v93\n" \
    "v_fmac_f32 v90, v91, v91\n" \
    "v_fmac_f32 v90, v89, v89\n" \
    "v_min_f32 v92, v97, v90\n" \
    "v_min_f32 v99, v99, v92\n" \
    "v_cmp_lt_f32 vcc, v99, v50\n" \
    "s_waitcnt lgkmcnt(0)\n" \
    "v_mul_f32 v111, v75, v80\n" \
    "v_fmac_f32 v111, v73, v78\n" \
    "v_fmac_f32 v111, v71, v76\n" \
    "v_add_f32_dpp v47, v120, v47 row_ror:5 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_add_f32_dpp v49, v122, v49 row_ror:5 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_add_f32_dpp v51, v124, v51 row_ror:5 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_mul_f32 v113, v75, v40\n" \
    "v_fmac_f32 v113, v73, v38\n" \
    "v_fmac_f32 v113, v71, v36\n" \
    "v_mul_f32 v121, v81, v80\n" \
    "v_fmac_f32 v121, v79, v78\n" \
    "v_fmac_f32 v121, v77, v76\n" \
    "v_mul_f32 v123, v81, v46\n" \
    "v_fmac_f32 v123, v79, v44\n" \
    "v_fmac_f32 v123, v77, v42\n" \
    "s_cbranch_vccz SD_SKIP3_%=\n" \
    "s_or_b64 %[nl], %[nl], vcc\n" \
    "v_cmp_lt_f32 vcc, v95, v50\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v95, v95, v27, vcc\n" \
    "v_cmp_lt_f32 vcc, v88, v25\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v88, v88, v27, vcc\n" \
    "v_cmp_lt_f32 vcc, v97, v50\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v97, v97, v27, vcc\n" \
    "v_cmp_lt_f32 vcc, v90, v25\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v90, v90, v27, vcc\n" \
    "SD_SKIP3_%=:\n" \
    "v_rsq_f32 v105, v95\n" \
    "v_rsq_f32 v115, v88\n" \
    "v_mul_f32 v94, v105, v105\n" \
    "v_mul_f32 v104, v115, v115\n" \
    "v_mul_f32 v107, v94, v105\n" \
    "v_mul_f32 v117, v104, v115\n" \
    "v_fma_f32 v109, v48, v107, v105\n" \
    "v_fma_f32 v96, v29, v94, 1.0\n" \
    "v_fma_f32 v119, v48, v117, v115\n" \
    "v_fma_f32 v106, v29, v104, 1.0\n" \
    "v_mul_f32 v98, v107, v96\n" \
    "v_mul_f32 v100, v98, v111\n" \
    "v_mul_f32 v102, v98, v113\n" \
    "v_mul_f32 v108, v117, v106\n" \
    "v_mul_f32 v110, v108, v121\n" \
    "v_mul_f32 v112, v108, v123\n" \
    "v_fmac_f32 v52, v100, v71\n" \
    "v_fmac_f32 v52, v109, v76\n" \
    "v_fmac_f32 v54, v100, v73\n" \
    "v_fmac_f32 v54, v109, v78\n" \
    "v_fmac_f32 v56, v100, v75\n" \
    "v_fmac_f32 v56, v109, v80\n" \
    "v_fmac_f32 v58, v110, v77\n" \
    "v_fmac_f32 v58, v119, v76\n" \
    "v_fmac_f32 v60, v110, v79\n" \
    "v_fmac_f32 v60, v119, v78\n" \
    "v_fmac_f32 v62, v110, v81\n" \
    "v_fmac_f32 v62, v119, v80\n" \
    "v_mul_f32 v114, v102, v71\n" \
    "v_fmac_f32 v114, v109, v36\n" \
    "v_mul_f32 v116, v102, v73\n" \
    "v_fmac_f32 v116, v109, v38\n" \
    "v_mul_f32 v118, v102, v75\n" \
    "v_fmac_f32 v118, v109, v40\n" \
    "v_fmac_f32 v114, v112, v77\n" \
    "v_fmac_f32 v114, v119, v42\n" \
    "v_fmac_f32 v116, v112, v79\n" \
    "v_fmac_f32 v116, v119, v44\n" \
    "v_fmac_f32 v118, v112, v81\n" \
    "v_fmac_f32 v118, v119, v46\n" \
    "v_rsq_f32 v105, v97\n" \
    "v_rsq_f32 v115, v90\n" \
    "v_mul_f32 v111, v87, v86\n" \
    "v_fmac_f32 v111, v85, v84\n" \
    "v_fmac_f32 v111, v83, v82\n" \
    "v_add_f32_dpp v47, v114, v47 row_ror:6 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_add_f32_dpp v49, v116, v49 row_ror:6 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_add_f32_dpp v51, v118, v51 row_ror:6 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_mul_f32 v113, v87, v40\n" \
    "v_fmac_f32 v113, v85, v38\n" \
    "v_fmac_f32 v113, v83, v36\n" \
    "v_mul_f32 v121, v93, v86\n" \
    "v_fmac_f32 v121, v91, v84\n" \
    "v_fmac_f32 v121, v89, v82\n" \
    "v_mul_f32 v123, v93, v46\n" \
    "v_fmac_f32 v123, v91, v44\n" \
    "v_fmac_f32 v123, v89, v42\n" \
    "v_mul_f32 v94, v105, v105\n" \
    "v_mul_f32 v104, v115, v115\n" \
    "v_mul_f32 v107, v94, v105\n" \
    "v_mul_f32 v117, v104, v115\n" \
    "v_fma_f32 v109, v48, v107, v105\n" \
    "v_fma_f32 v96, v29, v94, 1.0\n" \
    "v_fma_f32 v119, v48, v117, v115\n" \
    "v_fma_f32 v106, v29, v104, 1.0\n" \
    "v_mul_f32 v98, v107, v96\n" \
    "v_mul_f32 v100, v98, v111\n" \
    "v_mul_f32 v102, v98, v113\n" \
    "v_mul_f32 v108, v117, v106\n" \
    "v_mul_f32 v110, v108, v121\n" \
    "v_mul_f32 v112, v108, v123\n" \
    "v_fmac_f32 v52, v100, v83\n" \
    "v_fmac_f32 v52, v109, v82\n" \
    "v_fmac_f32 v54, v100, v85\n" \
    "v_fmac_f32 v54, v109, v84\n" \
    "v_fmac_f32 v56, v100, v87\n" \
    "v_fmac_f32 v56, v109, v86\n" \
    "v_fmac_f32 v58, v110, v89\n" \
    "v_fmac_f32 v58, v119, v82\n" \
    "v_fmac_f32 v60, v110, v91\n" \
    "v_fmac_f32 v60, v119, v84\n" \
    "v_fmac_f32 v62, v110, v93\n" \
    "v_fmac_f32 v62, v119, v86\n" \
    "v_mul_f32 v120, v102, v83\n" \
    "v_fmac_f32 v120, v109, v36\n" \
    "v_mul_f32 v122, v102, v85\n" \
    "v_fmac_f32 v122, v109, v38\n" \
    "v_mul_f32 v124, v102, v87\n" \
    "v_fmac_f32 v124, v109, v40\n" \
    "v_fmac_f32 v120, v112, v89\n" \
    "v_fmac_f32 v120, v119, v42\n" \
    "v_fmac_f32 v122, v112, v91\n" \
    "v_fmac_f32 v122, v119, v44\n" \
    "v_fmac_f32 v124, v112, v93\n" \
    "v_fmac_f32 v124, v119, v46\n" \
    "v_add_f32 v35, v35, v52\n" \
    "v_add_f32 v37, v37, v54\n" \
    "v_add_f32 v39, v39, v56\n" \
    "v_add_f32 v41, v41, v58\n" \
    "v_add_f32 v43, v43, v60\n" \
    "v_add_f32 v45, v45, v62\n" \
    "ds_read_b32 v59, v31 offset:32\n" \
    "ds_read_b32 v61, v31 offset:160\n" \
    "ds_read_b32 v63, v31 offset:288\n" \
    "ds_read_b32 v65, v31 offset:36\n" \
    "ds_read_b32 v67, v31 offset:164\n" \
    "ds_read_b32 v69, v31 offset:292\n" \
    "ds_read_b32 v76, v31 offset:416\n" \
    "ds_read_b32 v78, v31 offset:544\n" \
    "ds_read_b32 v80, v31 offset:672\n" \
    "ds_read_b32 v82, v31 offset:420\n" \
    "ds_read_b32 v84, v31 offset:548\n" \
    "ds_read_b32 v86, v31 offset:676\n" \
    "s_waitcnt lgkmcnt(9)\n" \
    "v_sub_u32 v101, v24, v59\n" \
    "v_cvt_f32_i32 v71, v101\n" \
    "v_sub_u32 v101, v26, v61\n" \
    "v_cvt_f32_i32 v73, v101\n" \
    "v_sub_u32 v101, v28, v63\n" \
    "v_cvt_f32_i32 v75, v101\n" \
    "v_sub_u32 v103, v30, v59\n" \
    "v_cvt_f32_i32 v77, v103\n" \
    "v_sub_u32 v103, v32, v61\n" \
    "v_cvt_f32_i32 v79, v103\n" \
    "v_sub_u32 v103, v34, v63\n" \
    "v_cvt_f32_i32 v81, v103\n" \
    "v_mul_f32 v95, v75, v75\n" \
    "v_fmac_f32 v95, v73, v73\n" \
    "v_fmac_f32 v95, v71, v71\n" \
    "v_mul_f32 v88, v81, v81\n" \
    "v_fmac_f32 v88, v79, v79\n" \
    "v_fmac_f32 v88, v77, v77\n" \
    "v_min_f32 v99, v95, v88\n" \
    "s_waitcnt lgkmcnt(6)\n" \
    "v_sub_u32 v101, v24, v65\n" \
    "v_cvt_f32_i32 v83, v101\n" \
    "v_sub_u32 v101, v26, v67\n" \
    "v_cvt_f32_i32 v85, v101\n" \
    "v_sub_u32 v101, v28, v69\n" \
    "v_cvt_f32_i32 v87, v101\n" \
    "v_sub_u32 v103, v30, v65\n" \
    "v_cvt_f32_i32 v89, v103\n" \
    "v_sub_u32 v103, v32, v67\n" \
    "v_cvt_f32_i32 v91, v103\n" \
    "v_sub_u32 v103, v34, v69\n" \
    "v_cvt_f32_i32 v93, v103\n" \
    "v_mul_f32 v97, v87, v87\n" \
    "v_fmac_f32 v97, v85, v85\n" \
    "v_fmac_f32 v97, v83, v83\n" \
    "v_mul_f32 v90, v93, v93\n" \
    "v_fmac_f32 v90, v91, v91\n" \
    "v_fmac_f32 v90, v89, v89\n" \
    "v_min_f32 v92, v97, v90\n" \
    "v_min_f32 v99, v99, v92\n" \
    "v_cmp_lt_f32 vcc, v99, v50\n" \
    "s_waitcnt lgkmcnt(0)\n" \
    "v_mul_f32 v111, v75, v80\n" \
    "v_fmac_f32 v111, v73, v78\n" \
    "v_fmac_f32 v111, v71, v76\n" \
    "v_add_f32_dpp v47, v120, v47 row_ror:7 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_add_f32_dpp v49, v122, v49 row_ror:7 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_add_f32_dpp v51, v124, v51 row_ror:7 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_mul_f32 v113, v75, v40\n" \
    "v_fmac_f32 v113, v73, v38\n" \
    "v_fmac_f32 v113, v71, v36\n" \
    "v_mul_f32 v121, v81, v80\n" \
    "v_fmac_f32 v121, v79, v78\n" \
    "v_fmac_f32 v121, v77, v76\n" \
    "v_mul_f32 v123, v81, v46\n" \
    "v_fmac_f32 v123, v79, v44\n" \
    "v_fmac_f32 v123, v77, v42\n" \
    "v_add_f32 v53, v53, v47\n" \
    "v_add_f32 v55, v55, v49\n" \
    "v_add_f32 v57, v57, v51\n" \
    "ds_write_b32 v33, v53 offset:0\n" \
    "ds_write_b32 v33, v55 offset:64\n" \
    "ds_write_b32 v33, v57 offset:128\n" \
    "s_cbranch_vccz SD_SKIP4_%=\n" \
    "s_or_b64 %[nl], %[nl], vcc\n" \
    "v_cmp_lt_f32 vcc, v95, v50\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v95, v95, v27, vcc\n" \
    "v_cmp_lt_f32 vcc, v88, v25\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v88, v88, v27, vcc\n" \
    "v_cmp_lt_f32 vcc, v97, v50\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v97, v97, v27, vcc\n" \
    "v_cmp_lt_f32 vcc, v90, v25\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v90, v90, v27, vcc\n" \
    "SD_SKIP4_%=:\n" \
    "v_rsq_f32 v105, v95\n" \
    "v_rsq_f32 v115, v88\n" \
    "v_mul_f32 v94, v105, v105\n" \
    "v_mul_f32 v104, v115, v115\n" \
    "v_mul_f32 v107, v94, v105\n" \
    "v_mul_f32 v117, v104, v115\n" \
    "v_fma_f32 v109, v48, v107, v105\n" \
    "v_fma_f32 v96, v29, v94, 1.0\n" \
    "v_fma_f32 v119, v48, v117, v115\n" \
    "v_fma_f32 v106, v29, v104, 1.0\n" \
    "v_mul_f32 v98, v107, v96\n" \
    "v_mul_f32 v100, v98, v111\n" \
    "v_mul_f32 v102, v98, v113\n" \
    "v_mul_f32 v108, v117, v106\n" \
    "v_mul_f32 v110, v108, v121\n" \
    "v_mul_f32 v112, v108, v123\n" \
    "v_mul_f32 v52, v100, v71\n" \
    "v_fmac_f32 v52, v109, v76\n" \
    "v_mul_f32 v54, v100, v73\n" \
    "v_fmac_f32 v54, v109, v78\n" \
    "v_mul_f32 v56, v100, v75\n" \
    "v_fmac_f32 v56, v109, v80\n" \
    "v_mul_f32 v58, v110, v77\n" \
    "v_fmac_f32 v58, v119, v76\n" \
    "v_mul_f32 v60, v110, v79\n" \
    "v_fmac_f32 v60, v119, v78\n" \
    "v_mul_f32 v62, v110, v81\n" \
    "v_fmac_f32 v62, v119, v80\n" \
    "v_mul_f32 v114, v102, v71\n" \
    "v_fmac_f32 v114, v109, v36\n" \
    "v_mul_f32 v116, v102, v73\n" \
    "v_fmac_f32 v116, v109, v38\n" \
    "v_mul_f32 v118, v102, v75\n" \
    "v_fmac_f32 v118, v109, v40\n" \
    "v_fmac_f32 v114, v112, v77\n" \
    "v_fmac_f32 v114, v119, v42\n" \
    "v_fmac_f32 v116, v112, v79\n" \
    "v_fmac_f32 v116, v119, v44\n" \
    "v_fmac_f32 v118, v112, v81\n" \
    "v_fmac_f32 v118, v119, v46\n" \
    "v_rsq_f32 v105, v97\n" \
    "v_rsq_f32 v115, v90\n" \
    "v_mul_f32 v111, v87, v86\n" \
    "v_fmac_f32 v111, v85, v84\n" \
    "v_fmac_f32 v111, v83, v82\n" \
    "v_mov_b32_dpp v53, v114 row_ror:8 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_mov_b32_dpp v55, v116 row_ror:8 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_mov_b32_dpp v57, v118 row_ror:8 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_mul_f32 v113, v87, v40\n" \
    "v_fmac_f32 v113, v85, v38\n" \
    "v_fmac_f32 v113, v83, v36\n" \
    "v_mul_f32 v121, v93, v86\n" \
    "v_fmac_f32 v121, v91, v84\n" \
    "v_fmac_f32 v121, v89, v82\n" \
    "v_mul_f32 v123, v93, v46\n" \
    "v_fmac_f32 v123, v91, v44\n" \
    "v_fmac_f32 v123, v89, v42\n" \
    "v_mul_f32 v94, v105, v105\n" \
    "v_mul_f32 v104, v115, v115\n" \
    "v_mul_f32 v107, v94, v105\n" \
    "v_mul_f32 v117, v104, v115\n" \
    "v_fma_f32 v109, v48, v107, v105\n" \
    "v_fma_f32 v96, v29, v94, 1.0\n" \
    "v_fma_f32 v119, v48, v117, v115\n" \
    "v_fma_f32 v106, v29, v104, 1.0\n" \
    "v_mul_f32 v98, v107, v96\n" \
    "v_mul_f32 v100, v98, v111\n" \
    "v_mul_f32 v102, v98, v113\n" \
    "v_mul_f32 v108, v117, v106\n" \
    "v_mul_f32 v110, v108, v121\n" \
    "v_mul_f32 v112, v108, v123\n" \
    "v_fmac_f32 v52, v100, v83\n" \
    "v_fmac_f32 v52, v109, v82\n" \
    "v_fmac_f32 v54, v100, v85\n" \
    "v_fmac_f32 v54, v109, v84\n" \
    "v_fmac_f32 v56, v100, v87\n" \
    "v_fmac_f32 v56, v109, v86\n" \
    "v_fmac_f32 v58, v110, v89\n" \
    "v_fmac_f32 v58, v119, v82\n" \
    "v_fmac_f32 v60, v110, v91\n" \
    "v_fmac_f32 v60, v119, v84\n" \
    "v_fmac_f32 v62, v110, v93\n" \
    "v_fmac_f32 v62, v119, v86\n" \
    "v_mul_f32 v120, v102, v83\n" \
    "v_fmac_f32 v120, v109, v36\n" \
    "v_mul_f32 v122, v102, v85\n" \
    "v_fmac_f32 v122, v109, v38\n" \
    "v_mul_f32 v124, v102, v87\n" \
    "v_fmac_f32 v124, v109, v40\n" \
    "v_fmac_f32 v120, v112, v89\n" \
    "v_fmac_f32 v120, v119, v42\n" \
    "v_fmac_f32 v122, v112, v91\n" \
    "v_fmac_f32 v122, v119, v44\n" \
    "v_fmac_f32 v124, v112, v93\n" \
    "v_fmac_f32 v124, v119, v46\n" \
    "ds_read_b32 v59, v31 offset:40\n" \
    "ds_read_b32 v61, v31 offset:168\n" \
    "ds_read_b32 v63, v31 offset:296\n" \
    "ds_read_b32 v65, v31 offset:44\n" \
    "ds_read_b32 v67, v31 offset:172\n" \
    "ds_read_b32 v69, v31 offset:300\n" \
    "ds_read_b32 v76, v31 offset:424\n" \
    "ds_read_b32 v78, v31 offset:552\n" \
    "ds_read_b32 v80, v31 offset:680\n" \
    "ds_read_b32 v82, v31 offset:428\n" \
    "ds_read_b32 v84, v31 offset:556\n" \
    "ds_read_b32 v86, v31 offset:684\n" \
    "s_waitcnt lgkmcnt(9)\n" \
    "v_sub_u32 v101, v24, v59\n" \
    "v_cvt_f32_i32 v71, v101\n" \
    "v_sub_u32 v101, v26, v61\n" \
    "v_cvt_f32_i32 v73, v101\n" \
    "v_sub_u32 v101, v28, v63\n" \
    "v_cvt_f32_i32 v75, v101\n" \
    "v_sub_u32 v103, v30, v59\n" \
    "v_cvt_f32_i32 v77, v103\n" \
    "v_sub_u32 v103, v32, v61\n" \
    "v_cvt_f32_i32 v79, v103\n" \
    "v_sub_u32 v103, v34, v63\n" \
    "v_cvt_f32_i32 v81, v103\n" \
    "v_mul_f32 v95, v75, v75\n" \
    "v_fmac_f32 v95, v73, v73\n" \
    "v_fmac_f32 v95, v71, v71\n" \
    "v_mul_f32 v88, v81, v81\n" \
    "v_fmac_f32 v88, v79, v79\n" \
    "v_fmac_f32 v88, v77, v77\n" \
    "v_min_f32 v99, v95, v88\n" \
    "s_waitcnt lgkmcnt(6)\n" \
    "v_sub_u32 v101, v24, v65\n" \
    "v_cvt_f32_i32 v83, v101\n" \
    "v_sub_u32 v101, v26, v67\n" \
    "v_cvt_f32_i32 v85, v101\n" \
    "v_sub_u32 v101, v28, v69\n" \
    "v_cvt_f32_i32 v87, v101\n" \
    "v_sub_u32 v103, v30, v65\n" \
    "v_cvt_f32_i32 v89, v103\n" \
    "v_sub_u32 v103, v32, v67\n" \
    "v_cvt_f32_i32 v91, v103\n" \
    "v_sub_u32 v103, v34, v69\n" \
    "v_cvt_f32_i32 v93, v103\n" \
    "v_mul_f32 v97, v87, v87\n" \
    "v_fmac_f32 v97, v85, v85\n" \
    "v_fmac_f32 v97, v83, v83\n" \
    "v_mul_f32 v90, v93, v93\n" \
    "v_fmac_f32 v90, v91, v91\n" \
    "v_fmac_f32 v90, v89, v89\n" \
    "v_min_f32 v92, v97, v90\n" \
    "v_min_f32 v99, v99, v92\n" \
    "v_cmp_lt_f32 vcc, v99, v50\n" \
    "s_waitcnt lgkmcnt(0)\n" \
    "v_mul_f32 v111, v75, v80\n" \
    "v_fmac_f32 v111, v73, v78\n" \
    "v_fmac_f32 v111, v71, v76\n" \
    "v_add_f32_dpp v53, v120, v53 row_ror:9 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_add_f32_dpp v55, v122, v55 row_ror:9 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_add_f32_dpp v57, v124, v57 row_ror:9 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_mul_f32 v113, v75, v40\n" \
    "v_fmac_f32 v113, v73, v38\n" \
    "v_fmac_f32 v113, v71, v36\n" \
    "v_mul_f32 v121, v81, v80\n" \
    "v_fmac_f32 v121, v79, v78\n" \
    "v_fmac_f32 v121, v77, v76\n" \
    "v_mul_f32 v123, v81, v46\n" \
    "v_fmac_f32 v123, v79, v44\n" \
    "v_fmac_f32 v123, v77, v42\n" \
    "s_cbranch_vccz SD_SKIP5_%=\n" \
    "s_or_b64 %[nl], %[nl], vcc\n" \
    "v_cmp_lt_f32 vcc, v95, v50\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v95, v95, v27, vcc\n" \
    "v_cmp_lt_f32 vcc, v88, v25\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v88, v88, v27, vcc\n" \
    "v_cmp_lt_f32 vcc, v97, v50\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v97, v97, v27, vcc\n" \
    "v_cmp_lt_f32 vcc, v90, v25\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v90, v90, v27, vcc\n" \
    "SD_SKIP5_%=:\n" \
    "v_rsq_f32 v105, v95\n" \
    "v_rsq_f32 v115, v88\n" \
    "v_mul_f32 v94, v105, v105\n" \
    "v_mul_f32 v104, v115, v115\n" \
    "v_mul_f32 v107, v94, v105\n" \
    "v_mul_f32 v117, v104, v115\n" \
    "v_fma_f32 v109, v48, v107, v105\n" \
    "v_fma_f32 v96, v29, v94, 1.0\n" \
    "v_fma_f32 v119, v48, v117, v115\n" \
    "v_fma_f32 v106, v29, v104, 1.0\n" \
    "v_mul_f32 v98, v107, v96\n" \
    "v_mul_f32 v100, v98, v111\n" \
    "v_mul_f32 v102, v98, v113\n" \
    "v_mul_f32 v108, v117, v106\n" \
    "v_mul_f32 v110, v108, v121\n" \
    "v_mul_f32 v112, v108, v123\n" \
    "v_fmac_f32 v52, v100, v71\n" \
    "v_fmac_f32 v52, v109, v76\n" \
    "v_fmac_f32 v54, v100, v73\n" \
    "v_fmac_f32 v54, v109, v78\n" \
    "v_fmac_f32 v56, v100, v75\n" \
    "v_fmac_f32 v56, v109, v80\n" \
    "v_fmac_f32 v58, v110, v77\n" \
    "v_fmac_f32 v58, v119, v76\n" \
    "v_fmac_f32 v60, v110, v79\n" \
    "v_fmac_f32 v60, v119, v78\n" \
    "v_fmac_f32 v62, v110, v81\n" \
    "v_fmac_f32 v62, v119, v80\n" \
    "v_mul_f32 v114, v102, v71\n" \
    "v_fmac_f32 v114, v109, v36\n" \
    "v_mul_f32 v116, v102, v73\n" \
    "v_fmac_f32 v116, v109, v38\n" \
    "v_mul_f32 v118, v102, v75\n" \
    "v_fmac_f32 v118, v109, v40\n" \
    "v_fmac_f32 v114, v112, v77\n" \
    "v_fmac_f32 v114, v119, v42\n" \
    "v_fmac_f32 v116, v112, v79\n" \
    "v_fmac_f32 v116, v119, v44\n" \
    "v_fmac_f32 v118, v112, v81\n" \
    "v_fmac_f32 v118, v119, v46\n" \
    "v_rsq_f32 v105, v97\n" \
    "v_rsq_f32 v115, v90\n" \
    "v_mul_f32 v111, v87, v86\n" \
    "v_fmac_f32 v111, v85, v84\n" \
    "v_fmac_f32 v111, v83, v82\n" \
    "v_add_f32_dpp v53, v114, v53 row_ror:10 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_add_f32_dpp v55, v116, v55 row_ror:10 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_add_f32_dpp v57, v118, v57 row_ror:10 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_mul_f32 v113, v87, v40\n" \
    "v_fmac_f32 v113, v85, v38\n" \
    "v_fmac_f32 v113, v83, v36\n" \
    "v_mul_f32 v121, v93, v86\n" \
    "v_fmac_f32 v121, v91, v84\n" \
    "v_fmac_f32 v121, v89, v82\n" \
    "v_mul_f32 v123, v93, v46\n" \
    "v_fmac_f32 v123, v91, v44\n" \
    "v_fmac_f32 v123, v89, v42\n" \
    "v_mul_f32 v94, v105, v105\n" \
    "v_mul_f32 v104, v115, v115\n" \
    "v_mul_f32 v107, v94, v105\n" \
    "v_mul_f32 v117, v104, v115\n" \
    "v_fma_f32 v109, v48, v107, v105\n" \
    "v_fma_f32 v96, v29, v94, 1.0\n" \
    "v_fma_f32 v119, v48, v117, v115\n" \
    "v_fma_f32 v106, v29, v104, 1.0\n" \
    "v_mul_f32 v98, v107, v96\n" \
    "v_mul_f32 v100, v98, v111\n" \
    "v_mul_f32 v102, v98, v113\n" \
    "v_mul_f32 v108, v117, v106\n" \
    "v_mul_f32 v110, v108, v121\n" \
    "v_mul_f32 v112, v108, v123\n" \
    "v_fmac_f32 v52, v100, v83\n" \
    "v_fmac_f32 v52, v109, v82\n" \
    "v_fmac_f32 v54, v100, v85\n" \
    "v_fmac_f32 v54, v109, v84\n" \
    "v_fmac_f32 v56, v100, v87\n" \
    "v_fmac_f32 v56, v109, v86\n" \
    "v_fmac_f32 v58, v110, v89\n" \
    "v_fmac_f32 v58, v119, v82\n" \
    "v_fmac_f32 v60, v110, v91\n" \
    "v_fmac_f32 v60, v119, v84\n" \
    "v_fmac_f32 v62, v110, v93\n" \
    "v_fmac_f32 v62, v119, v86\n" \
    "v_mul_f32 v120, v102, v83\n" \
    "v_fmac_f32 v120, v109, v36\n" \
    "v_mul_f32 v122, v102, v85\n" \
    "v_fmac_f32 v122, v109, v38\n" \
    "v_mul_f32 v124, v102, v87\n" \
    "v_fmac_f32 v124, v109, v40\n" \
    "v_fmac_f32 v120, v112, v89\n" \
    "v_fmac_f32 v120, v119, v42\n" \
    "v_fmac_f32 v122, v112, v91\n" \
    "v_fmac_f32 v122, v119, v44\n" \
    "v_fmac_f32 v124, v112, v93\n" \
    "v_fmac_f32 v124, v119, v46\n" \
    "v_add_f32 v35, v35, v52\n" \
    "v_add_f32 v37, v37, v54\n" \
    "v_add_f32 v39, v39, v56\n" \
    "v_add_f32 v41, v41, v58\n" \
    "v_add_f32 v43, v43, v60\n" \
    "v_add_f32 v45, v45, v62\n" \
    "ds_read_b32 v59, v31 offset:48\n" \
    "ds_read_b32 v61, v31 offset:176\n" \
    "ds_read_b32 v63, v31 offset:304\n" \
    "ds_read_b32 v65, v31 offset:52\n" \
    "ds_read_b32 v67, v31 offset:180\n" \
    "ds_read_b32 v69, v31 offset:308\n" \
    "ds_read_b32 v76, v31 offset:432\n" \
    "ds_read_b32 v78, v31 offset:560\n" \
    "ds_read_b32 v80, v31 offset:688\n" \
    "ds_read_b32 v82, v31 offset:436\n" \
    "ds_read_b32 v84, v31 offset:564\n" \
    "ds_read_b32 v86, v31 offset:692\n" \
    "s_waitcnt lgkmcnt(9)\n" \
    "v_sub_u32 v101, v24, v59\n" \
    "v_cvt_f32_i32 v71, v101\n" \
    "v_sub_u32 v101, v26, v61\n" \
    "v_cvt_f32_i32 v73, v101\n" \
    "v_sub_u32 v101, v28, v63\n" \
    "v_cvt_f32_i32 v75, v101\n" \
    "v_sub_u32 v103, v30, v59\n" \
    "v_cvt_f32_i32 v77, v103\n" \
    "v_sub_u32 v103, v32, v61\n" \
    "v_cvt_f32_i32 v79, v103\n" \
    "v_sub_u32 v103, v34, v63\n" \
    "v_cvt_f32_i32 v81, v103\n" \
    "v_mul_f32 v95, v75, v75\n" \
    "v_fmac_f32 v95, v73, v73\n" \
    "v_fmac_f32 v95, v71, v71\n" \
    "v_mul_f32 v88, v81, v81\n" \
    "v_fmac_f32 v88, v79, v79\n" \
    "v_fmac_f32 v88, v77, v77\n" \
    "v_min_f32 v99, v95, v88\n" \
    "s_waitcnt lgkmcnt(6)\n" \
    "v_sub_u32 v101, v24, v65\n" \
    "v_cvt_f32_i32 v83, v101\n" \
    "v_sub_u32 v101, v26, v67\n" \
    "v_cvt_f32_i32 v85, v101\n" \
    "v_sub_u32 v101, v28, v69\n" \
    "v_cvt_f32_i32 v87, v101\n" \
    "v_sub_u32 v103, v30, v65\n" \
    "v_cvt_f32_i32 v89, v103\n" \
    "v_sub_u32 v103, v32, v67\n" \
    "v_cvt_f32_i32 v91, v103\n" \
    "v_sub_u32 v103, v34, v69\n" \
    "v_cvt_f32_i32 v93, v103\n" \
    "v_mul_f32 v97, v87, v87\n" \
    "v_fmac_f32 v97, v85, v85\n" \
    "v_fmac_f32 v97, v83, v83\n" \
    "v_mul_f32 v90, v93, v93\n" \
    "v_fmac_f32 v90, v91, v91\n" \
    "v_fmac_f32 v90, v89, v89\n" \
    "v_min_f32 v92, v97, v90\n" \
    "v_min_f32 v99, v99, v92\n" \
    "v_cmp_lt_f32 vcc, v99, v50\n" \
    "s_waitcnt lgkmcnt(0)\n" \
    "v_mul_f32 v111, v75, v80\n" \
    "v_fmac_f32 v111, v73, v78\n" \
    "v_fmac_f32 v111, v71, v76\n" \
    "v_add_f32_dpp v53, v120, v53 row_ror:11 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_add_f32_dpp v55, v122, v55 row_ror:11 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_add_f32_dpp v57, v124, v57 row_ror:11 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_mul_f32 v113, v75, v40\n" \
    "v_fmac_f32 v113, v73, v38\n" \
    "v_fmac_f32 v113, v71, v36\n" \
    "v_mul_f32 v121, v81, v80\n" \
    "v_fmac_f32 v121, v79, v78\n" \
    "v_fmac_f32 v121, v77, v76\n" \
    "v_mul_f32 v123, v81, v46\n" \
    "v_fmac_f32 v123, v79, v44\n" \
    "v_fmac_f32 v123, v77, v42\n" \
    "s_cbranch_vccz SD_SKIP6_%=\n" \
    "s_or_b64 %[nl], %[nl], vcc\n" \
    "v_cmp_lt_f32 vcc, v95, v50\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v95, v95, v27, vcc\n" \
    "v_cmp_lt_f32 vcc, v88, v25\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v88, v88, v27, vcc\n" \
    "v_cmp_lt_f32 vcc, v97, v50\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v97, v97, v27, vcc\n" \
    "v_cmp_lt_f32 vcc, v90, v25\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v90, v90, v27, vcc\n" \
    "SD_SKIP6_%=:\n" \
    "v_rsq_f32 v105, v95\n" \
    "v_rsq_f32 v115, v88\n" \
    "v_mul_f32 v94, v105, v105\n" \
    "v_mul_f32 v104, v115, v115\n" \
    "v_mul_f32 v107, v94, v105\n" \
    "v_mul_f32 v117, v104, v115\n" \
    "v_fma_f32 v109, v48, v107, v105\n" \
    "v_fma_f32 v96, v29, v94, 1.0\n" \
    "v_fma_f32 v119, v48, v117, v115\n" \
    "v_fma_f32 v106, v29, v104, 1.0\n" \
    "v_mul_f32 v98, v107, v96\n" \
    "v_mul_f32 v100, v98, v111\n" \
    "v_mul_f32 v102, v98, v113\n" \
    "v_mul_f32 v108, v117, v106\n" \
    "v_mul_f32 v110, v108, v121\n" \
    "v_mul_f32 v112, v108, v123\n" \
    "v_mul_f32 v52, v100, v71\n" \
    "v_fmac_f32 v52, v109, v76\n" \
    "v_mul_f32 v54, v100, v73\n" \
    "v_fmac_f32 v54, v109, v78\n" \
    "v_mul_f32 v56, v100, v75\n" \
    "v_fmac_f32 v56, v109, v80\n" \
    "v_mul_f32 v58, v110, v77\n" \
    "v_fmac_f32 v58, v119, v76\n" \
    "v_mul_f32 v60, v110, v79\n" \
    "v_fmac_f32 v60, v119, v78\n" \
    "v_mul_f32 v62, v110, v81\n" \
    "v_fmac_f32 v62, v119, v80\n" \
    "v_mul_f32 v114, v102, v71\n" \
    "v_fmac_f32 v114, v109, v36\n" \
    "v_mul_f32 v116, v102, v73\n" \
    "v_fmac_f32 v116, v109, v38\n" \
    "v_mul_f32 v118, v102, v75\n" \
    "v_fmac_f32 v118, v109, v40\n" \
    "v_fmac_f32 v114, v112, v77\n" \
    "v_fmac_f32 v114, v119, v42\n" \
    "v_fmac_f32 v116, v112, v79\n" \
    "v_fmac_f32 v116, v119, v44\n" \
    "v_fmac_f32 v118, v112, v81\n" \
    "v_fmac_f32 v118, v119, v46\n" \
    "v_rsq_f32 v105, v97\n" \
    "v_rsq_f32 v115, v90\n" \
    "v_mul_f32 v111, v87, v86\n" \
    "v_fmac_f32 v111, v85, v84\n" \
    "v_fmac_f32 v111, v83, v82\n" \
    "v_mov_b32_dpp v47, v114 row_ror:12 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_mov_b32_dpp v49, v116 row_ror:12 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_mov_b32_dpp v51, v118 row_ror:12 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_mul_f32 v113, v87, v40\n" \
    "v_fmac_f32 v113, v85, v38\n" \
    "v_fmac_f32 v113, v83, v36\n" \
    "v_mul_f32 v121, v93, v86\n" \
    "v_fmac_f32 v121, v91, v84\n" \
    "v_fmac_f32 v121, v89, v82\n" \
    "v_mul_f32 v123, v93, v46\n" \
    "v_fmac_f32 v123, v91, v44\n" \
    "v_fmac_f32 v123, v89, v42\n" \
    "v_mul_f32 v94, v105, v105\n" \
    "v_mul_f32 v104, v115, v115\n" \
    "v_mul_f32 v107, v94, v105\n" \
    "v_mul_f32 v117, v104, v115\n" \
    "v_fma_f32 v109, v48, v107, v105\n" \
    "v_fma_f32 v96, v29, v94, 1.0\n" \
    "v_fma_f32 v119, v48, v117, v115\n" \
    "v_fma_f32 v106, v29, v104, 1.0\n" \
    "v_mul_f32 v98, v107, v96\n" \
    "v_mul_f32 v100, v98, v111\n" \
    "v_mul_f32 v102, v98, v113\n" \
    "v_mul_f32 v108, v117, v106\n" \
    "v_mul_f32 v110, v108, v121\n" \
    "v_mul_f32 v112, v108, v123\n" \
    "v_fmac_f32 v52, v100, v83\n" \
    "v_fmac_f32 v52, v109, v82\n" \
    "v_fmac_f32 v54, v100, v85\n" \
    "v_fmac_f32 v54, v109, v84\n" \
    "v_fmac_f32 v56, v100, v87\n" \
    "v_fmac_f32 v56, v109, v86\n" \
    "v_fmac_f32 v58, v110, v89\n" \
    "v_fmac_f32 v58, v119, v82\n" \
    "v_fmac_f32 v60, v110, v91\n" \
    "v_fmac_f32 v60, v119, v84\n" \
    "v_fmac_f32 v62, v110, v93\n" \
    "v_fmac_f32 v62, v119, v86\n" \
    "v_mul_f32 v120, v102, v83\n" \
    "v_fmac_f32 v120, v109, v36\n" \
    "v_mul_f32 v122, v102, v85\n" \
    "v_fmac_f32 v122, v109, v38\n" \
    "v_mul_f32 v124, v102, v87\n" \
    "v_fmac_f32 v124, v109, v40\n" \
    "v_fmac_f32 v120, v112, v89\n" \
    "v_fmac_f32 v120, v119, v42\n" \
    "v_fmac_f32 v122, v112, v91\n" \
    "v_fmac_f32 v122, v119, v44\n" \
    "v_fmac_f32 v124, v112, v93\n" \
    "v_fmac_f32 v124, v119, v46\n" \
    "ds_read_b32 v59, v31 offset:56\n" \
    "ds_read_b32 v61, v31 offset:184\n" \
    "ds_read_b32 v63, v31 offset:312\n" \
    "ds_read_b32 v65, v31 offset:60\n" \
    "ds_read_b32 v67, v31 offset:188\n" \
    "ds_read_b32 v69, v31 offset:316\n" \
    "ds_read_b32 v76, v31 offset:440\n" \
    "ds_read_b32 v78, v31 offset:568\n" \
    "ds_read_b32 v80, v31 offset:696\n" \
    "ds_read_b32 v82, v31 offset:444\n" \
    "ds_read_b32 v84, v31 offset:572\n" \
    "ds_read_b32 v86, v31 offset:700\n" \
    "s_waitcnt lgkmcnt(9)\n" \
    "v_sub_u32 v101, v24, v59\n" \
    "v_cvt_f32_i32 v71, v101\n" \
    "v_sub_u32 v101, v26, v61\n" \
    "v_cvt_f32_i32 v73, v101\n" \
    "v_sub_u32 v101, v28, v63\n" \
    "v_cvt_f32_i32 v75, v101\n" \
    "v_sub_u32 v103, v30, v59\n" \
    "v_cvt_f32_i32 v77, v103\n" \
    "v_sub_u32 v103, v32, v61\n" \
    "v_cvt_f32_i32 v79, v103\n" \
    "v_sub_u32 v103, v34, v63\n" \
    "v_cvt_f32_i32 v81, v103\n" \
    "v_mul_f32 v95, v75, v75\n" \
    "v_fmac_f32 v95, v73, v73\n" \
    "v_fmac_f32 v95, v71, v71\n" \
    "v_mul_f32 v88, v81, v81\n" \
    "v_fmac_f32 v88, v79, v79\n" \
    "v_fmac_f32 v88, v77, v77\n" \
    "v_min_f32 v99, v95, v88\n" \
    "s_waitcnt lgkmcnt(6)\n" \
    "v_sub_u32 v101, v24, v65\n" \
    "v_cvt_f32_i32 v83, v101\n" \
    "v_sub_u32 v101, v26, v67\n" \
    "v_cvt_f32_i32 v85, v101\n" \
    "v_sub_u32 v101, v28, v69\n" \
    "v_cvt_f32_i32 v87, v101\n" \
    "v_sub_u32 v103, v30, v65\n" \
    "v_cvt_f32_i32 v89, v103\n" \
    "v_sub_u32 v103, v32, v67\n" \
    "v_cvt_f32_i32 v91, v103\n" \
    "v_sub_u32 v103, v34, v69\n" \
    "v_cvt_f32_i32 v93, v103\n" \
    "v_mul_f32 v97, v87, v87\n" \
    "v_fmac_f32 v97, v85, v85\n" \
    "v_fmac_f32 v97, v83, v83\n" \
    "v_mul_f32 v90, v93, v93\n" \
    "v_fmac_f32 v90, v91, v91\n" \
    "v_fmac_f32 v90, v89, v89\n" \
    "v_min_f32 v92, v97, v90\n" \
    "v_min_f32 v99, v99, v92\n" \
    "v_cmp_lt_f32 vcc, v99, v50\n" \
    "s_waitcnt lgkmcnt(0)\n" \
    "v_mul_f32 v111, v75, v80\n" \
    "v_fmac_f32 v111, v73, v78\n" \
    "v_fmac_f32 v111, v71, v76\n" \
    "v_add_f32_dpp v47, v120, v47 row_ror:13 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_add_f32_dpp v49, v122, v49 row_ror:13 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_add_f32_dpp v51, v124, v51 row_ror:13 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_mul_f32 v113, v75, v40\n" \
    "v_fmac_f32 v113, v73, v38\n" \
    "v_fmac_f32 v113, v71, v36\n" \
    "v_mul_f32 v121, v81, v80\n" \
    "v_fmac_f32 v121, v79, v78\n" \
    "v_fmac_f32 v121, v77, v76\n" \
    "v_mul_f32 v123, v81, v46\n" \
    "v_fmac_f32 v123, v79, v44\n" \
    "v_fmac_f32 v123, v77, v42\n" \
    "s_cbranch_vccz SD_SKIP7_%=\n" \
    "s_or_b64 %[nl], %[nl], vcc\n" \
    "v_cmp_lt_f32 vcc, v95, v50\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v95, v95, v27, vcc\n" \
    "v_cmp_lt_f32 vcc, v88, v25\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v88, v88, v27, vcc\n" \
    "v_cmp_lt_f32 vcc, v97, v50\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v97, v97, v27, vcc\n" \
    "v_cmp_lt_f32 vcc, v90, v25\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v90, v90, v27, vcc\n" \
    "SD_SKIP7_%=:\n" \
    "v_rsq_f32 v105, v95\n" \
    "v_rsq_f32 v115, v88\n" \
    "v_mul_f32 v94, v105, v105\n" \
    "v_mul_f32 v104, v115, v115\n" \
    "v_mul_f32 v107, v94, v105\n" \
    "v_mul_f32 v117, v104, v115\n" \
    "v_fma_f32 v109, v48, v107, v105\n" \
    "v_fma_f32 v96, v29, v94, 1.0\n" \
    "v_fma_f32 v119, v48, v117, v115\n" \
    "v_fma_f32 v106, v29, v104, 1.0\n" \
    "v_mul_f32 v98, v107, v96\n" \
    "v_mul_f32 v100, v98, v111\n" \
    "v_mul_f32 v102, v98, v113\n" \
    "v_mul_f32 v108, v117, v106\n" \
    "v_mul_f32 v110, v108, v121\n" \
    "v_mul_f32 v112, v108, v123\n" \
    "v_fmac_f32 v52, v100, v71\n" \
    "v_fmac_f32 v52, v109, v76\n" \
    "v_fmac_f32 v54, v100, v73\n" \
    "v_fmac_f32 v54, v109, v78\n" \
    "v_fmac_f32 v56, v100, v75\n" \
    "v_fmac_f32 v56, v109, v80\n" \
    "v_fmac_f32 v58, v110, v77\n" \
    "v_fmac_f32 v58, v119, v76\n" \
    "v_fmac_f32 v60, v110, v79\n" \
    "v_fmac_f32 v60, v119, v78\n" \
    "v_fmac_f32 v62, v110, v81\n" \
    "v_fmac_f32 v62, v119, v80\n" \
    "v_mul_f32 v114, v102, v71\n" \
    "v_fmac_f32 v114, v109, v36\n" \
    "v_mul_f32 v116, v102, v73\n" \
    "v_fmac_f32 v116, v109, v38\n" \
    "v_mul_f32 v118, v102, v75\n" \
    "v_fmac_f32 v118, v109, v40\n" \
    "v_fmac_f32 v114, v112, v77\n" \
    "v_fmac_f32 v114, v119, v42\n" \
    "v_fmac_f32 v116, v112, v79\n" \
    "v_fmac_f32 v116, v119, v44\n" \
    "v_fmac_f32 v118, v112, v81\n" \
    "v_fmac_f32 v118, v119, v46\n" \
    "v_rsq_f32 v105, v97\n" \
    "v_rsq_f32 v115, v90\n" \
    "v_mul_f32 v111, v87, v86\n" \
    "v_fmac_f32 v111, v85, v84\n" \
    "v_fmac_f32 v111, v83, v82\n" \
    "v_add_f32_dpp v47, v114, v47 row_ror:14 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_add_f32_dpp v49, v116, v49 row_ror:14 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_add_f32_dpp v51, v118, v51 row_ror:14 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_mul_f32 v113, v87, v40\n" \
    "v_fmac_f32 v113, v85, v38\n" \
    "v_fmac_f32 v113, v83, v36\n" \
    "v_mul_f32 v121, v93, v86\n" \
    "v_fmac_f32 v121, v91, v84\n" \
    "v_fmac_f32 v121, v89, v82\n" \
    "v_mul_f32 v123, v93, v46\n" \
    "v_fmac_f32 v123, v91, v44\n" \
    "v_fmac_f32 v123, v89, v42\n" \
    "v_mul_f32 v94, v105, v105\n" \
    "v_mul_f32 v104, v115, v115\n" \
    "v_mul_f32 v107, v94, v105\n" \
    "v_mul_f32 v117, v104, v115\n" \
    "v_fma_f32 v109, v48, v107, v105\n" \
    "v_fma_f32 v96, v29, v94, 1.0\n" \
    "v_fma_f32 v119, v48, v117, v115\n" \
    "v_fma_f32 v106, v29, v104, 1.0\n" \
    "v_mul_f32 v98, v107, v96\n" \
    "v_mul_f32 v100, v98, v111\n" \
    "v_mul_f32 v102, v98, v113\n" \
    "v_mul_f32 v108, v117, v106\n" \
    "v_mul_f32 v110, v108, v121\n" \
    "v_mul_f32 v112, v108, v123\n" \
    "v_fmac_f32 v52, v100, v83\n" \
    "v_fmac_f32 v52, v109, v82\n" \
    "v_fmac_f32 v54, v100, v85\n" \
    "v_fmac_f32 v54, v109, v84\n" \
    "v_fmac_f32 v56, v100, v87\n" \
    "v_fmac_f32 v56, v109, v86\n" \
    "v_fmac_f32 v58, v110, v89\n" \
    "v_fmac_f32 v58, v119, v82\n" \
    "v_fmac_f32 v60, v110, v91\n" \
    "v_fmac_f32 v60, v119, v84\n" \
    "v_fmac_f32 v62, v110, v93\n" \
    "v_fmac_f32 v62, v119, v86\n" \
    "v_mul_f32 v120, v102, v83\n" \
    "v_fmac_f32 v120, v109, v36\n" \
    "v_mul_f32 v122, v102, v85\n" \
    "v_fmac_f32 v122, v109, v38\n" \
    "v_mul_f32 v124, v102, v87\n" \
    "v_fmac_f32 v124, v109, v40\n" \
    "v_fmac_f32 v120, v112, v89\n" \
    "v_fmac_f32 v120, v119, v42\n" \
    "v_fmac_f32 v122, v112, v91\n" \
    "v_fmac_f32 v122, v119, v44\n" \
    "v_fmac_f32 v124, v112, v93\n" \
    "v_fmac_f32 v124, v119, v46\n" \
    "v_add_f32 v35, v35, v52\n" \
    "v_add_f32 v37, v37, v54\n" \
    "v_add_f32 v39, v39, v56\n" \
    "v_add_f32 v41, v41, v58\n" \
    "v_add_f32 v43, v43, v60\n" \
    "v_add_f32 v45, v45, v62\n" \
    "s_nop 1\n" \
    "v_add_f32_dpp v47, v120, v47 row_ror:15 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_add_f32_dpp v49, v122, v49 row_ror:15 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_add_f32_dpp v51, v124, v51 row_ror:15 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_add_f32 v53, v53, v47\n" \
    "v_add_f32 v55, v55, v49\n" \
    "v_add_f32 v57, v57, v51\n" \
    "ds_write_b32 v33, v53 offset:768\n" \
    "ds_write_b32 v33, v55 offset:832\n" \
    "ds_write_b32 v33, v57 offset:896\n" \
    "v_add_f32 v125, v64, v35\n" \
    "v_sub_f32 v126, v125, v64\n" \
    "v_sub_f32 v35, v35, v126\n" \
    "v_mov_b32 v64, v125\n" \
    "v_add_f32 v125, v66, v37\n" \
    "v_sub_f32 v126, v125, v66\n" \
    "v_sub_f32 v37, v37, v126\n" \
    "v_mov_b32 v66, v125\n" \
    "v_add_f32 v125, v68, v39\n" \
    "v_sub_f32 v126, v125, v68\n" \
    "v_sub_f32 v39, v39, v126\n" \
    "v_mov_b32 v68, v125\n" \
    "v_add_f32 v125, v70, v41\n" \
    "v_sub_f32 v126, v125, v70\n" \
    "v_sub_f32 v41, v41, v126\n" \
    "v_mov_b32 v70, v125\n" \
    "v_add_f32 v125, v72, v43\n" \
    "v_sub_f32 v126, v125, v72\n" \
    "v_sub_f32 v43, v43, v126\n" \
    "v_mov_b32 v72, v125\n" \
    "v_add_f32 v125, v74, v45\n" \
    "v_sub_f32 v126, v125, v74\n" \
    "v_sub_f32 v45, v45, v126\n" \
    "v_mov_b32 v74, v125\n"

// one chunk; 1289 instructions per chunk, 0 products with same-parity sources
#define SD_WAVE_CHUNK_OSEEN_FREE \
    "ds_read_b32 v59, v31 offset:0\n" \
    "ds_read_b32 v61, v31 offset:128\n" \
    "ds_read_b32 v63, v31 offset:256\n" \
    "ds_read_b32 v65, v31 offset:4\n" \
    "ds_read_b32 v67, v31 offset:132\n" \
    "ds_read_b32 v69, v31 offset:260\n" \
    "ds_read_b32 v76, v31 offset:384\n" \
    "ds_read_b32 v78, v31 offset:512\n" \
    "ds_read_b32 v80, v31 offset:640\n" \
    "ds_read_b32 v82, v31 offset:388\n" \
    "ds_read_b32 v84, v31 offset:516\n" \
    "ds_read_b32 v86, v31 offset:644\n" \
    "s_waitcnt lgkmcnt(9)\n" \
    "v_sub_f32 v71, v24, v59\n" \
    "v_sub_f32 v73, v26, v61\n" \
    "v_sub_f32 v75, v28, v63\n" \
    "v_sub_f32 v77, v30, v59\n" \
    "v_sub_f32 v79, v32, v61\n" \
    "v_sub_f32 v81, v34, v63\n" \
    "v_mul_f32 v95, v75, v75\n" \
    "v_fmac_f32 v95, v73, v73\n" \
    "v_fmac_f32 v95, v71, v71\n" \
    "v_mul_f32 v88, v81, v81\n" \
    "v_fmac_f32 v88, v79, v79\n" \
    "v_fmac_f32 v88, v77, v77\n" \
    "v_min_f32 v99, v95, v88\n" \
    "s_waitcnt lgkmcnt(6)\n" \
    "v_sub_f32 v83, v24, v65\n" \
    "v_sub_f32 v85, v26, v67\n" \
    "v_sub_f32 v87, v28, v69\n" \
    "v_sub_f32 v89, v30, v65\n" \
    "v_sub_f32 v91, v32, v67\n" \
    "v_sub_f32 v93, v34, v69\n" \
    "v_mul_f32 v97, v87, v87\n" \
    "v_fmac_f32 v97, v85, v85\n" \
    "v_fmac_f32 v97, v83, v83\n" \
    "v_mul_f32 v90, v93, v93\n" \
    "v_fmac_f32 v90, v91, v91\n" \
    "v_fmac_f32 v90, v89, v89\n" \
    "v_min_f32 v92, v97, v90\n" \
    "v_min_f32 v99, v99, v92\n" \
    "v_cmp_lt_f32 vcc, v99, v50\n" \
    "s_waitcnt lgkmcnt(0)\n" \
    "v_mul_f32 v111, v75, v80\n" \
    "v_fmac_f32 v111, v73, v78\n" \
    "v_fmac_f32 v111, v71, v76\n" \
    "v_mul_f32 v113, v75, v40\n" \
    "v_fmac_f32 v113, v73, v38\n" \
    "v_fmac_f32 v113, v71, v36\n" \
    "v_mul_f32 v121, v81, v80\n" \
    "v_fmac_f32 v121, v79, v78\n" \
    "v_fmac_f32 v121, v77, v76\n" \
    "v_mul_f32 v123, v81, v46\n" \
    "v_fmac_f32 v123, v79, v44\n" \
    "v_fmac_f32 v123, v77, v42\n" \
    "s_cbranch_vccz SD_SKIP0_%=\n" \
    "s_or_b64 %[nl], %[nl], vcc\n" \
    "v_cmp_lt_f32 vcc, v95, v50\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v95, v95, v27, vcc\n" \
    "v_cmp_lt_f32 vcc, v88, v25\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v88, v88, v27, vcc\n" \
    "v_cmp_lt_f32 vcc, v97, v50\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v97, v97, v27, vcc\n" \
    "v_cmp_lt_f32 vcc, v90, v25\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v90, v90, v27, vcc\n" \
    "SD_SKIP0_%=:\n" \
    "v_rsq_f32 v105, v95\n" \
    "v_rsq_f32 v115, v88\n" \
    "v_mul_f32 v94, v105, v105\n" \
    "v_mul_f32 v104, v115, v115\n" \
    "v_mul_f32 v107, v94, v105\n" \
    "v_mul_f32 v117, v104, v115\n" \
    "v_mul_f32 v100, v94, v111\n" \
    "v_mul_f32 v100, v100, v105\n" \
    "v_mul_f32 v102, v94, v113\n" \
    "v_mul_f32 v102, v102, v105\n" \
    "v_mul_f32 v110, v104, v121\n" \
    "v_mul_f32 v110, v110, v115\n" \
    "v_mul_f32 v112, v104, v123\n" \
    "v_mul_f32 v112, v112, v115\n" \
    "v_mul_f32 v52, v100, v71\n" \
    "v_fmac_f32 v52, v105, v76\n" \
    "v_mul_f32 v54, v100, v73\n" \
    "v_fmac_f32 v54, v105, v78\n" \
    "v_mul_f32 v56, v100, v75\n" \
    "v_fmac_f32 v56, v105, v80\n" \
    "v_mul_f32 v58, v110, v77\n" \
    "v_fmac_f32 v58, v115, v76\n" \
    "v_mul_f32 v60, v110, v79\n" \
    "v_fmac_f32 v60, v115, v78\n" \
    "v_mul_f32 v62, v110, v81\n" \
    "v_fmac_f32 v62, v115, v80\n" \
    "v_mul_f32 v53, v102, v71\n" \
    "v_fmac_f32 v53, v105, v36\n" \
    "v_mul_f32 v55, v102, v73\n" \
    "v_fmac_f32 v55, v105, v38\n" \
    "v_mul_f32 v57, v102, v75\n" \
    "v_fmac_f32 v57, v105, v40\n" \
    "v_fmac_f32 v53, v112, v77\n" \
    "v_fmac_f32 v53, v115, v42\n" \
    "v_fmac_f32 v55, v112, v79\n" \
    "v_fmac_f32 v55, v115, v44\n" \
    "v_fmac_f32 v57, v112, v81\n" \
    "v_fmac_f32 v57, v115, v46\n" \
    "v_rsq_f32 v105, v97\n" \
    "v_rsq_f32 v115, v90\n" \
    "v_mul_f32 v111, v87, v86\n" \
    "v_fmac_f32 v111, v85, v84\n" \
    "v_fmac_f32 v111, v83, v82\n" \
    "v_mul_f32 v113, v87, v40\n" \
    "v_fmac_f32 v113, v85, v38\n" \
    "v_fmac_f32 v113, v83, v36\n" \
    "v_mul_f32 v121, v93, v86\n" \
    "v_fmac_f32 v121, v91, v84\n" \
    "v_fmac_f32 v121, v89, v82\n" \
    "v_mul_f32 v123, v93, v46\n" \
    "v_fmac_f32 v123, v91, v44\n" \
    "v_fmac_f32 v123, v89, v42\n" \
    "v_mul_f32 v94, v105, v105\n" \
    "v_mul_f32 v104, v115, v115\n" \
    "v_mul_f32 v107, v94, v105\n" \
    "v_mul_f32 v117, v104, v115\n" \
    "v_mul_f32 v100, v94, v111\n" \
    "v_mul_f32 v100, v100, v105\n" \
    "v_mul_f32 v102, v94, v113\n" \
    "v_mul_f32 v102, v102, v105\n" \
    "v_mul_f32 v110, v104, v121\n" \
    "v_mul_f32 v110, v110, v115\n" \
    "v_mul_f32 v112, v104, v123\n" \
    "v_mul_f32 v112, v112, v115\n" \
    "v_fmac_f32 v52, v100, v83\n" \
    "v_fmac_f32 v52, v105, v82\n" \
    "v_fmac_f32 v54, v100, v85\n" \
    "v_fmac_f32 v54, v105, v84\n" \
    "v_fmac_f32 v56, v100, v87\n" \
    "v_fmac_f32 v56, v105, v86\n" \
    "v_fmac_f32 v58, v110, v89\n" \
    "v_fmac_f32 v58, v115, v82\n" \
    "v_fmac_f32 v60, v110, v91\n" \
    "v_fmac_f32 v60, v115, v84\n" \
    "v_fmac_f32 v62, v110, v93\n" \
    "v_fmac_f32 v62, v115, v86\n" \
    "v_mul_f32 v120, v102, v83\n" \
    "v_fmac_f32 v120, v105, v36\n" \
    "v_mul_f32 v122, v102, v85\n" \
    "v_fmac_f32 v122, v105, v38\n" \
    "v_mul_f32 v124, v102, v87\n" \
    "v_fmac_f32 v124, v105, v40\n" \
    "v_fmac_f32 v120, v112, v89\n" \
    "v_fmac_f32 v120, v115, v42\n" \
    "v_fmac_f32 v122, v112, v91\n" \
    "v_fmac_f32 v122, v115, v44\n" \
    "v_fmac_f32 v124, v112, v93\n" \
    "v_fmac_f32 v124, v115, v46\n" \
    "ds_read_b32 v59, v31 offset:8\n" \
    "ds_read_b32 v61, v31 offset:136\n" \
    "ds_read_b32 v63, v31 offset:264\n" \
    "ds_read_b32 v65, v31 offset:12\n" \
    "ds_read_b32 v67, v31 offset:140\n" \
    "ds_read_b32 v69, v31 offset:268\n" \
    "ds_read_b32 v76, v31 offset:392\n" \
    "ds_read_b32 v78, v31 offset:520\n" \
    "ds_read_b32 v80, v31 offset:648\n" \
    "ds_read_b32 v82, v31 offset:396\n" \
    "ds_read_b32 v84, v31 offset:524\n" \
    "ds_read_b32 v86, v31 offset:652\n" \
    "s_waitcnt lgkmcnt(9)\n" \
    "v_sub_f32 v71, v24, v59\n" \
    "v_sub_f32 v73, v26, v61\n" \
    "v_sub_f32 v75, v28, v63\n" \
    "v_sub_f32 v77, v30, v59\n" \
    "v_sub_f32 v79, v32, v61\n" \
    "v_sub_f32 v81, v34, v63\n" \
    "v_mul_f32 v95, v75, v75\n" \
    "v_fmac_f32 v95, v73, v73\n" \
    "v_fmac_f32 v95, v71, v71\n" \
    "v_mul_f32 v88, v81, v81\n" \
    "v_fmac_f32 v88, v79, v79\n" \
    "v_fmac_f32 v88, v77, v77\n" \
    "v_min_f32 v99, v95, v88\n" \
    "s_waitcnt lgkmcnt(6)\n" \
    "v_sub_f32 v83, v24, v65\n" \
    "v_sub_f32 v85, v26, v67\n" \
    "v_sub_f32 v87, v28, v69\n" \
    "v_sub_f32 v89, v30, v65\n" \
    "v_sub_f32 v91, v32, v67\n" \
    "v_sub_f32 v93, v34, v69\n" \
    "v_mul_f32 v97, v87, v87\n" \
    "v_fmac_f32 v97, v85, v85\n" \
    "v_fmac_f32 v97, v83, v83\n" \
    "v_mul_f32 v90, v93, v93\n" \
    "v_fmac_f32 v90, v91, v91\n" \
    "v_fmac_f32 v90, v89, v89\n" \
    "v_min_f32 v92, v97, v90\n" \
    "v_min_f32 v99, v99, v92\n" \
    "v_cmp_lt_f32 vcc, v99, v50\n" \
    "s_waitcnt lgkmcnt(0)\n" \
    "v_mul_f32 v111, v75, v80\n" \
    "v_fmac_f32 v111, v73, v78\n" \
    "v_fmac_f32 v111, v71, v76\n" \
    "v_add_f32_dpp v53, v120, v53 row_ror:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_add_f32_dpp v55, v122, v55 row_ror:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_add_f32_dpp v57, v124, v57 row_ror:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_mul_f32 v113, v75, v40\n" \
    "v_fmac_f32 v113, v73, v38\n" \
    "v_fmac_f32 v113, v71, v36\n" \
    "v_mul_f32 v121, v81, v80\n" \
    "v_fmac_f32 v121, v79, v78\n" \
    "v_fmac_f32 v121, v77, v76\n" \
    "v_mul_f32 v123, v81, v46\n" \
    "v_fmac_f32 v123, v79, v44\n" \
    "v_fmac_f32 v123, v77, v42\n" \
    "s_cbranch_vccz SD_SKIP1_%=\n" \
    "s_or_b64 %[nl], %[nl], vcc\n" \
    "v_cmp_lt_f32 vcc, v95, v50\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v95, v95, v27, vcc\n" \
    "v_cmp_lt_f32 vcc, v88, v25\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v88, v88, v27, vcc\n" \
    "v_cmp_lt_f32 vcc, v97, v50\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v97, v97, v27, vcc\n" \
    "v_cmp_lt_f32 vcc, v90, v25\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v90, v90, v27, vcc\n" \
    "SD_SKIP1_%=:\n" \
    "v_rsq_f32 v105, v95\n" \
    "v_rsq_f32 v115, v88\n" \
    "v_mul_f32 v94, v105, v105\n" \
    "v_mul_f32 v104, v115, v115\n" \
    "v_mul_f32 v107, v94, v105\n" \
    "v_mul_f32 v117, v104, v115\n" \
    "v_mul_f32 v100, v94, v111\n" \
    "v_mul_f32 v100, v100, v105\n" \
    "v_mul_f32 v102, v94, v113\n" \
    "v_mul_f32 v102, v102, v105\n" \
    "v_mul_f32 v110, v104, v121\n" \
    "v_mul_f32 v110, v110, v115\n" \
    "v_mul_f32 v112, v104, v123\n" \
    "v_mul_f32 v112, v112, v115\n" \
    "v_fmac_f32 v52, v100, v71\n" \
    "v_fmac_f32 v52, v105, v76\n" \
    "v_fmac_f32 v54, v100, v73\n" \
    "v_fmac_f32 v54, v105, v78\n" \
    "v_fmac_f32 v56, v100, v75\n" \
    "v_fmac_f32 v56, v105, v80\n" \
    "v_fmac_f32 v58, v110, v77\n" \
    "v_fmac_f32 v58, v115, v76\n" \
    "v_fmac_f32 v60, v110, v79\n" \
    "v_fmac_f32 v60, v115, v78\n" \
    "v_fmac_f32 v62, v110, v81\n" \
    "v_fmac_f32 v62, v115, v80\n" \
    "v_mul_f32 v114, v102, v71\n" \
    "v_fmac_f32 v114, v105, v36\n" \
    "v_mul_f32 v116, v102, v73\n" \
    "v_fmac_f32 v116, v105, v38\n" \
    "v_mul_f32 v118, v102, v75\n" \
    "v_fmac_f32 v118, v105, v40\n" \
    "v_fmac_f32 v114, v112, v77\n" \
    "v_fmac_f32 v114, v115, v42\n" \
    "v_fmac_f32 v116, v112, v79\n" \
    "v_fmac_f32 v116, v115, v44\n" \
    "v_fmac_f32 v118, v112, v81\n" \
    "v_fmac_f32 v118, v115, v46\n" \
    "v_rsq_f32 v105, v97\n" \
    "v_rsq_f32 v115, v90\n" \
    "v_mul_f32 v111, v87, v86\n" \
    "v_fmac_f32 v111, v85, v84\n" \
    "v_fmac_f32 v111, v83, v82\n" \
    "v_add_f32_dpp v53, v114, v53 row_ror:2 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_add_f32_dpp v55, v116, v55 row_ror:2 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_add_f32_dpp v57, v118, v57 row_ror:2 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_mul_f32 v113, v87, v40\n" \
    "v_fmac_f32 v113, v85, v38\n" \
    "v_fmac_f32 v113, v83, v36\n" \
    "v_mul_f32 v121, v93, v86\n" \
    "v_fmac_f32 v121, v91, v84\n" \
    "v_fmac_f32 v121, v89, v82\n" \
    "v_mul_f32 v123, v93, v46\n" \
    "v_fmac_f32 v123, v91, v44\n" \
    "v_fmac_f32 v123, v89, v42\n" \
    "v_mul_f32 v94, v105, v105\n" \
    "v_mul_f32 v104, v115, v115\n" \
    "v_mul_f32 v107, v94, v105\n" \
    "v_mul_f32 v117, v104, v115\n" \
    "v_mul_f32 v100, v94, v111\n" \
    "v_mul_f32 v100, v100, v105\n" \
    "v_mul_f32 v102, v94, v113\n" \
    "v_mul_f32 v102, v102, v105\n" \
    "v_mul_f32 v110, v104, v121\n" \
    "v_mul_f32 v110, v110, v115\n" \
    "v_mul_f32 v112, v104, v123\n" \
    "v_mul_f32 v112, v112, v115\n" \
    "v_fmac_f32 v52, v100, v83\n" \
    "v_fmac_f32 v52, v105, v82\n" \
    "v_fmac_f32 v54, v100, v85\n" \
    "v_fmac_f32 v54, v105, v84\n" \
    "v_fmac_f32 v56, v100, v87\n" \
    "v_fmac_f32 v56, v105, v86\n" \
    "v_fmac_f32 v58, v110, v89\n" \
    "v_fmac_f32 v58, v115, v82\n" \
    "v_fmac_f32 v60, v110, v91\n" \
    "v_fmac_f32 v60, v115, v84\n" \
    "v_fmac_f32 v62, v110, v93\n" \
    "v_fmac_f32 v62, v115, v86\n" \
    "v_mul_f32 v120, v102, v83\n" \
    "v_fmac_f32 v120, v105, v36\n" \
    "v_mul_f32 v122, v102, v85\n" \
    "v_fmac_f32 v122, v105, v38\n" \
    "v_mul_f32 v124, v102, v87\n" \
    "v_fmac_f32 v124, v105, v40\n" \
    "v_fmac_f32 v120, v112, v89\n" \
    "v_fmac_f32 v120, v115, v42\n" \
    "v_fmac_f32 v122, v112, v91\n" \
    "v_fmac_f32 v122, v115, v44\n" \
    "v_fmac_f32 v124, v112, v93\n" \
    "v_fmac_f32 v124, v115, v46\n" \
    "v_add_f32 v35, v35, v52\n" \
    "v_add_f32 v37, v37, v54\n" \
    "v_add_f32 v39, v39, v56\n" \
    "v_add_f32 v41, v41, v58\n" \
    "v_add_f32 v43, v43, v60\n" \
    "v_add_f32 v45, v45, v62\n" \
    "ds_read_b32 v59, v31 offset:16\n" \
    "ds_read_b32 v61, v31 offset:144\n" \
    "ds_read_b32 v63, v31 offset:272\n" \
    "ds_read_b32 v65, v31 offset:20\n" \
    "ds_read_b32 v67, v31 offset:148\n" \
    "ds_read_b32 v69, v31 offset:276\n" \
    "ds_read_b32 v76, v31 offset:400\n" \
    "ds_read_b32 v78, v31 offset:528\n" \
    "ds_read_b32 v80, v31 offset:656\n" \
    "ds_read_b32 v82, v31 offset:404\n" \
    "ds_read_b32 v84, v31 offset:532\n" \
    "ds_read_b32 v86, v31 offset:660\n" \
    "s_waitcnt lgkmcnt(9)\n" \
    "v_sub_f32 v71, v24, v59\n" \
    "v_sub_f32 v73, v26, v61\n" \
    "v_sub_f32 v75, v28, v63\n" \
    "v_sub_f32 v77, v30, v59\n" \
    "v_sub_f32 v79, v32, v61\n" \
    "v_sub_f32 v81, v34, v63\n" \
    "v_mul_f32 v95, v75, v75\n" \
    "v_fmac_f32 v95, v73, v73\n" \
    "v_fmac_f32 v95, v71, v71\n" \
    "v_mul_f32 v88, v81, v81\n" \
    "v_fmac_f32 v88, v79, v79\n" \
    "v_fmac_f32 v88, v77, v77\n" \
    "v_min_f32 v99, v95, v88\n" \
    "s_waitcnt lgkmcnt(6)\n" \
    "v_sub_f32 v83, v24, v65\n" \
    "v_sub_f32 v85, v26, v67\n" \
    "v_sub_f32 v87, v28, v69\n" \
    "v_sub_f32 v89, v30, v65\n" \
    "v_sub_f32 v91, v32, v67\n" \
    "v_sub_f32 v93, v34, v69\n" \
    "v_mul_f32 v97, v87, v87\n" \
    "v_fmac_f32 v97, v85, v85\n" \
    "v_fmac_f32 v97, v83, v83\n" \
    "v_mul_f32 v90, v93, v93\n" \
    "v_fmac_f32 v90, v91, v91\n" \
    "v_fmac_f32 v90, v89, v89\n" \
    "v_min_f32 v92, v97, v90\n" \
    "v_min_f32 v99, v99, v92\n" \
    "v_cmp_lt_f32 vcc, v99, v50\n" \
    "s_waitcnt lgkmcnt(0)\n" \
    "v_mul_f32 v111, v75, v80\n" \
    "v_fmac_f32 v111, v73, v78\n" \
    "v_fmac_f32 v111, v71, v76\n" \
    "v_add_f32_dpp v53, v120, v53 row_ror:3 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_add_f32_dpp v55, v122, v55 row_ror:3 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_add_f32_dpp v57, v124, v57 row_ror:3 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_mul_f32 v113, v75, v40\n" \
    "v_fmac_f32 v113, v73, v38\n" \
    "v_fmac_f32 v113, v71, v36\n" \
    "v_mul_f32 v121, v81, v80\n" \
    "v_fmac_f32 v121, v79, v78\n" \
    "v_fmac_f32 v121, v77, v76\n" \
    "v_mul_f32 v123, v81, v46\n" \
    "v_fmac_f32 v123, v79, v44\n" \
    "v_fmac_f32 v123, v77, v42\n" \
    "s_cbranch_vccz SD_SKIP2_%=\n" \
    "s_or_b64 %[nl], %[nl], vcc\n" \
    "v_cmp_lt_f32 vcc, v95, v50\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v95, v95, v27, vcc\n" \
    "v_cmp_lt_f32 vcc, v88, v25\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v88, v88, v27, vcc\n" \
    "v_cmp_lt_f32 vcc, v97, v50\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v97, v97, v27, vcc\n" \
    "v_cmp_lt_f32 vcc, v90, v25\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v90, v90, v27, vcc\n" \
    "SD_SKIP2_%=:\n" \
    "v_rsq_f32 v105, v95\n" \
    "v_rsq_f32 v115, v88\n" \
    "v_mul_f32 v94, v105, v105\n" \
    "v_mul_f32 v104, v115, v115\n" \
    "v_mul_f32 v107, v94, v105\n" \
    "v_mul_f32 v117, v104, v115\n" \
    "v_mul_f32 v100, v94, v111\n" \
    "v_mul_f32 v100, v100, v105\n" \
    "v_mul_f32 v102, v94, v113\n" \
    "v_mul_f32 v102, v102, v105\n" \
    "v_mul_f32 v110, v104, v121\n" \
    "v_mul_f32 v110, v110, v115\n" \
    "v_mul_f32 v112, v104, v123\n" \
    "v_mul_f32 v112, v112, v115\n" \
    "v_mul_f32 v52, v100, v71\n" \
    "v_fmac_f32 v52, v105, v76\n" \
    "v_mul_f32 v54, v100, v73\n" \
    "v_fmac_f32 v54, v105, v78\n" \
    "v_mul_f32 v56, v100, v75\n" \
    "v_fmac_f32 v56, v105, v80\n" \
    "v_mul_f32 v58, v110, v77\n" \
    "v_fmac_f32 v58, v115, v76\n" \
    "v_mul_f32 v60, v110, v79\n" \
    "v_fmac_f32 v60, v115, v78\n" \
    "v_mul_f32 v62, v110, v81\n" \
    "v_fmac_f32 v62, v115, v80\n" \
    "v_mul_f32 v114, v102, v71\n" \
    "v_fmac_f32 v114, v105, v36\n" \
    "v_mul_f32 v116, v102, v73\n" \
    "v_fmac_f32 v116, v105, v38\n" \
    "v_mul_f32 v118, v102, v75\n" \
    "v_fmac_f32 v118, v105, v40\n" \
    "v_fmac_f32 v114, v112, v77\n" \
    "v_fmac_f32 v114, v115, v42\n" \
    "v_fmac_f32 v116, v112, v79\n" \
    "v_fmac_f32 v116, v115, v44\n" \
    "v_fmac_f32 v118, v112, v81\n" \
    "v_fmac_f32 v118, v115, v46\n" \
    "v_rsq_f32 v105, v97\n" \
    "v_rsq_f32 v115, v90\n" \
    "v_mul_f32 v111, v87, v86\n" \
    "v_fmac_f32 v111, v85, v84\n" \
    "v_fmac_f32 v111, v83, v82\n" \
    "v_mov_b32_dpp v47, v114 row_ror:4 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_mov_b32_dpp v49, v116 row_ror:4 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_mov_b32_dpp v51, v118 row_ror:4 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_mul_f32 v113, v87, v40\n" \
    "v_fmac_f32 v113, v85, v38\n" \
    "v_fmac_f32 v113, v83, v36\n" \
    "v_mul_f32 v121, v93, v86\n" \
    "v_fmac_f32 v121, v91, v84\n" \
    "v_fmac_f32 v121, v89, v82\n" \
    "v_mul_f32 v123, v93, v46\n" \
    "v_fmac_f32 v123, v91, v44\n" \
    "v_fmac_f32 v123, v89, v42\n" \
    "v_mul_f32 v94, v105, v105\n" \
    "v_mul_f32 v104, v115, v115\n" \
    "v_mul_f32 v107, v94, v105\n" \
    "v_mul_f32 v117, v104, v115\n" \
    "v_mul_f32 v100, v94, v111\n" \
    "v_mul_f32 v100, v100, v105\n" \
    "v_mul_f32 v102, v94, v113\n" \
    "v_mul_f32 v102, v102, v105\n" \
    "v_mul_f32 v110, v104, v121\n" \
    "v_mul_f32 v110, v110, v115\n" \
    "v_mul_f32 v112, v104, v123\n" \
    "v_mul_f32 v112, v112, v115\n" \
    "v_fmac_f32 v52, v100, v83\n" \
    "v_fmac_f32 v52, v105, v82\n" \
    "v_fmac_f32 v54, v100, v85\n" \
    "v_fmac_f32 v54, v105, v84\n" \
    "v_fmac_f32 v56, v100, v87\n" \
    "v_fmac_f32 v56, v105, v86\n" \
    "v_fmac_f32 v58, v110, v89\n" \
    "v_fmac_f32 v58, v115, v82\n" \
    "v_fmac_f32 v60, v110, v91\n" \
    "v_fmac_f32 v60, v115, v84\n" \
    "v_fmac_f32 v62, v110, v93\n" \
    "v_fmac_f32 v62, v115, v86\n" \
    "v_mul_f32 v120, v102, v83\n" \
    "v_fmac_f32 v120, v105, v36\n" \
    "v_mul_f32 v122, v102, v85\n" \
    "v_fmac_f32 v122, v105, v38\n" \
    "v_mul_f32 v124, v102, v87\n" \
    "v_fmac_f32 v124, v105, v40\n" \
    "v_fmac_f32 v120, v112, v89\n" \
    "v_fmac_f32 v120, v115, v42\n" \
    "v_fmac_f32 v122, v112, v91\n" \
    "v_fmac_f32 v122, v115, v44\n" \
    "v_fmac_f32 v124, v112, v93\n" \
    "v_fmac_f32 v124, v115, v46\n" \
    "ds_read_b32 v59, v31 offset:24\n" \
    "ds_read_b32 v61, v31 offset:152\n" \
    "ds_read_b32 v63, v31 offset:280\n" \
    "ds_read_b32 v65, v31 offset:28\n" \
    "ds_read_b32 v67, v31 offset:156\n" \
    "ds_read_b32 v69, v31 offset:284\n" \
    "ds_read_b32 v76, v31 offset:408\n" \
    "ds_read_b32 v78, v31 offset:536\n" \
    "ds_read_b32 v80, v31 offset:664\n" \
    "ds_read_b32 v82, v31 offset:412\n" \
    "ds_read_b32 v84, v31 offset:540\n" \
    "ds_read_b32 v86, v31 offset:668\n" \
    "s_waitcnt lgkmcnt(9)\n" \
    "v_sub_f32 v71, v24, v59\n" \
    "v_sub_f32 v73, v26, v61\n" \
    "v_sub_f32 v75, v28, v63\n" \
    "v_sub_f32 v77, v30, v59\n" \
    "v_sub_f32 v79, v32, v61\n" \
    "v_sub_f32 v81, v34, v63\n" \
    "v_mul_f32 v95, v75, v75\n" \
    "v_fmac_f32 v95, v73, v73\n" \
    "v_fmac_f32 v95, v71, v71\n" \
    "v_mul_f32 v88, v81, v81\n" \
    "v_fmac_f32 v88, v79, v79\n" \
    "v_fmac_f32 v88, v77, v77\n" \
    "v_min_f32 v99, v95, v88\n" \
    "s_waitcnt lgkmcnt(6)\n" \
    "v_sub_f32 v83, v24, v65\n" \
    "v_sub_f32 v85, v26, v67\n" \
    "v_sub_f32 v87, v28, v69\n" \
    "v_sub_f32 v89, v30, v65\n" \
    "v_sub_f32 v91, v32, v67\n" \
    "v_sub_f32 v93, v34, v69\n" \
    "v_mul_f32 v97, v87, v87\n" \
    "v_fmac_f32 v97, v85, v85\n" \
    "v_fmac_f32 v97, v83, v83\n" \
    "v_mul_f32 v90, v93, v93\n" \
    "v_fmac_f32 v90, v91, v91\n" \
    "v_fmac_f32 v90, v89, v89\n" \
    "v_min_f32 v92, v97, v90\n" \
    "v_min_f32 v99, v99, v92\n" \
    "v_cmp_lt_f32 vcc, v99, v50\n" \
    "s_waitcnt lgkmcnt(0)\n" \
    "v_mul_f32 v111, v75, v80\n" \
    "v_fmac_f32 v111, v73, v78\n" \
    "v_fmac_f32 v111, v71, v76\n" \
    "v_add_f32_dpp v47, v120, v47 row_ror:5 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_add_f32_dpp v49, v122, v49 row_ror:5 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_add_f32_dpp v51, v124, v51 row_ror:5 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_mul_f32 v113, v75, v40\n" \
    "v_fmac_f32 v113, v73, v38\n" \
    "v_fmac_f32 v113, v71, v36\n" \
    "v_mul_f32 v121, v81, v80\n" \
    "v_fmac_f32 v121, v79, v78\n" \
    "v_fmac_f32 v121, v77, v76\n" \
    "v_mul_f32 v123, v81, v46\n" \
    "v_fmac_f32 v123, v79, v44\n" \
    "v_fmac_f32 v123, v77, v42\n" \
    "s_cbranch_vccz SD_SKIP3_%=\n" \
    "s_or_b64 %[nl], %[nl], vcc\n" \
    "v_cmp_lt_f32 vcc, v95, v50\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v95, v95, v27, vcc\n" \
    "v_cmp_lt_f32 vcc, v88, v25\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v88, v88, v27, vcc\n" \
    "v_cmp_lt_f32 vcc, v97, v50\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v97, v97, v27, vcc\n" \
    "v_cmp_lt_f32 vcc, v90, v25\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v90, v90, v27, vcc\n" \
    "SD_SKIP3_%=:\n" \
    "v_rsq_f32 v105, v95\n" \
    "v_rsq_f32 v115, v88\n" \
    "v_mul_f32 v94, v105, v105\n" \
    "v_mul_f32 v104, v115, v115\n" \
    "v_mul_f32 v107, v94, v105\n" \
    "v_mul_f32 v117, v104, v115\n" \
    "v_mul_f32 v100, v94, v111\n" \
    "v_mul_f32 v100, v100, v105\n" \
    "v_mul_f32 v102, v94, v113\n" \
    "v_mul_f32 v102, v102, v105\n" \
    "v_mul_f32 v110, v104, v121\n" \
    "v_mul_f32 v110, v110, v115\n" \
    "v_mul_f32 v112, v104, v123\n" \
    "v_mul_f32 v112, v112, v115\n" \
    "v_fmac_f32 v52, v100, v71\n" \
    "v_fmac_f32 v52, v105, v76\n" \
    "v_fmac_f32 v54, v100, v73\n" \
    "v_fmac_f32 v54, v105, v78\n" \
    "v_fmac_f32 v56, v100, v75\n" \
    "v_fmac_f32 v56, v105, v80\n" \
    "v_fmac_f32 v58, v110, v77\n" \
    "v_fmac_f32 v58, v115, v76\n" \
    "v_fmac_f32 v60, v110, v79\n" \
    "v_fmac_f32 v60, v115, v78\n" \
    "v_fmac_f32 v62, v110, v81\n" \
    "v_fmac_f32 v62, v115, v80\n" \
    "v_mul_f32 v114, v102, v71\n" \
    "v_fmac_f32 v114, v105, v36\n" \
    "v_mul_f32 v116, v102, v73\n" \
    "v_fmac_f32 v116, v105, v38\n" \
    "v_mul_f32 v118, v102, v75\n" \
    "v_fmac_f32 v118, v105, v40\n" \
    "v_fmac_f32 v114, v112, v77\n" \
    "v_fmac_f32 v114, v115, v42\n" \
    "v_fmac_f32 v116, v112, v79\n" \
    "v_fmac_f32 v116, v115, v44\n" \
    "v_fmac_f32 v118, v112, v81\n" \
    "v_fmac_f32 v118, v115, v46\n" \
    "v_rsq_f32 v105, v97\n" \
    "v_rsq_f32 v115, v90\n" \
    "v_mul_f32 v111, v87, v86\n" \
    "v_fmac_f32 v111, v85, v84\n" \
    "v_fmac_f32 v111, v83, v82\n" \
    "v_add_f32_dpp v47, v114, v47 row_ror:6 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_add_f32_dpp v49, v116, v49 row_ror:6 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_add_f32_dpp v51, v118, v51 row_ror:6 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_mul_f32 v113, v87, v40\n" \
    "v_fmac_f32 v113, v85, v38\n" \
    "v_fmac_f32 v113, v83, v36\n" \
    "v_mul_f32 v121, v93, v86\n" \
    "v_fmac_f32 v121, v91, v84\n" \
    "v_fmac_f32 v121, v89, v82\n" \
    "v_mul_f32 v123, v93, v46\n" \
    "v_fmac_f32 v123, v91, v44\n" \
    "v_fmac_f32 v123, v89, v42\n" \
    "v_mul_f32 v94, v105, v105\n" \
    "v_mul_f32 v104, v115, v115\n" \
    "v_mul_f32 v107, v94, v105\n" \
    "v_mul_f32 v117, v104, v115\n" \
    "v_mul_f32 v100, v94, v111\n" \
    "v_mul_f32 v100, v100, v105\n" \
    "v_mul_f32 v102, v94, v113\n" \
    "v_mul_f32 v102, v102, v105\n" \
    "v_mul_f32 v110, v104, v121\n" \
    "v_mul_f32 v110, v110, v115\n" \
    "v_mul_f32 v112, v104, v123\n" \
    "v_mul_f32 v112, v112, v115\n" \
    "v_fmac_f32 v52, v100, v83\n" \
    "v_fmac_f32 v52, v105, v82\n" \
    "v_fmac_f32 v54, v100, v85\n" \
    "v_fmac_f32 v54, v105, v84\n" \
    "v_fmac_f32 v56, v100, v87\n" \
    "v_fmac_f32 v56, v105, v86\n" \
    "v_fmac_f32 v58, v110, v89\n" \
    "v_fmac_f32 v58, v115, v82\n" \
    "v_fmac_f32 v60, v110, v91\n" \
    "v_fmac_f32 v60, v115, v84\n" \
    "v_fmac_f32 v62, v110, v93\n" \
    "v_fmac_f32 v62, v115, v86\n" \
    "v_mul_f32 v120, v102, v83\n" \
    "v_fmac_f32 v120, v105, v36\n" \
    "v_mul_f32 v122, v102, v85\n" \
    "v_fmac_f32 v122, v105, v38\n" \
    "v_mul_f32 v124, v102, v87\n" \
    "v_fmac_f32 v124, v105, v40\n" \
    "v_fmac_f32 v120, v112, v89\n" \
    "v_fmac_f32 v120, v115, v42\n" \
    "v_fmac_f32 v122, v112, v91\n" \
    "v_fmac_f32 v122, v115, v44\n" \
    "v_fmac_f32 v124, v112, v93\n" \
    "v_fmac_f32 v124, v115, v46\n" \
    "v_add_f32 v35, v35, v52\n" \
    "v_add_f32 v37, v37, v54\n" \
    "v_add_f32 v39, v39, v56\n" \
    "v_add_f32 v41, v41, v58\n" \
    "v_add_f32 v43, v43, v60\n" \
    "v_add_f32 v45, v45, v62\n" \
    "ds_read_b32 v59, v31 offset:32\n" \
    "ds_read_b32 v61, v31 offset:160\n" \
    "ds_read_b32 v63, v31 offset:288\n" \
    "ds_read_b32 v65, v31 offset:36\n" \
    "ds_read_b32 v67, v31 offset:164\n" \
    "ds_read_b32 v69, v31 offset:292\n" \
    "ds_read_b32 v76, v31 offset:416\n" \
    "ds_read_b32 v78, v31 offset:544\n" \
    "ds_read_b32 v80, v31 offset:672\n" \
    "ds_read_b32 v82, v31 offset:420\n" \
    "ds_read_b32 v84, v31 offset:548\n" \
    "ds_read_b32 v86, v31 offset:676\n" \
    "s_waitcnt lgkmcnt(9)\n" \
    "v_sub_f32 v71, v24, v59\n" \
    "v_sub_f32 v73, v26, v61\n" \
    "v_sub_f32 v75, v28, v63\n" \
    "v_sub_f32 v77, v30, v59\n" \
    "v_sub_f32 v79, v32, v61\n" \
    "v_sub_f32 v81, v34, v63\n" \
    "v_mul_f32 v95, v75, v75\n" \
    "v_fmac_f32 v95, v73, v73\n" \
    "v_fmac_f32 v95, v71, v71\n" \
    "v_mul_f32 v88, v81, v81\n" \
    "v_fmac_f32 v88, v79, v79\n" \
    "v_fmac_f32 v88, v77, v77\n" \
    "v_min_f32 v99, v95, v88\n" \
    "s_waitcnt lgkmcnt(6)\n" \
    "v_sub_f32 v83, v24, v65\n" \
    "v_sub_f32 v85, v26, v67\n" \
    "v_sub_f32 v87, v28, v69\n" \
    "v_sub_f32 v89, v30, v65\n" \
    "v_sub_f32 v91, v32, v67\n" \
    "v_sub_f32 v93, v34, v69\n" \
    "v_mul_f32 v97, v87, v87\n" \
    "v_fmac_f32 v97, v85, v85\n" \
    "v_fmac_f32 v97, v83, v83\n" \
    "v_mul_f32 v90, v93, v93\n" \
    "v_fmac_f32 v90, v91, v91\n" \
    "v_fmac_f32 v90, v89, v89\n" \
    "v_min_f32 v92, v97, v90\n" \
    "v_min_f32 v99, v99, v92\n" \
    "v_cmp_lt_f32 vcc, v99, v50\n" \
    "s_waitcnt lgkmcnt(0)\n" \
    "v_mul_f32 v111, v75, v80\n" \
    "v_fmac_f32 v111, v73, v78\n" \
    "v_fmac_f32 v111, v71, v76\n" \
    "v_add_f32_dpp v47, v120, v47 row_ror:7 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_add_f32_dpp v49, v122, v49 row_ror:7 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_add_f32_dpp v51, v124, v51 row_ror:7 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_mul_f32 v113, v75, v40\n" \
    "v_fmac_f32 v113, v73, v38\n" \
    "v_fmac_f32 v113, v71, v36\n" \
    "v_mul_f32 v121, v81, v80\n" \
    "v_fmac_f32 v121, v79, v78\n" \
    "v_fmac_f32 v121, v77, v76\n" \
    "v_mul_f32 v123, v81, v46\n" \
    "v_fmac_f32 v123, v79, v44\n" \
    "v_fmac_f32 v123, v77, v42\n" \
    "v_add_f32 v53, v53, v47\n" \
    "v_add_f32 v55, v55, v49\n" \
    "v_add_f32 v57, v57, v51\n" \
    "ds_write_b32 v33, v53 offset:0\n" \
    "ds_write_b32 v33, v55 offset:64\n" \
    "ds_write_b32 v33, v57 offset:128\n" \
    "s_cbranch_vccz SD_SKIP4_%=\n" \
    "s_or_b64 %[nl], %[nl], vcc\n" \
    "v_cmp_lt_f32 vcc, v95, v50\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v95, v95, v27, vcc\n" \
    "v_cmp_lt_f32 vcc, v88, v25\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v88, v88, v27, vcc\n" \
    "v_cmp_lt_f32 vcc, v97, v50\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v97, v97, v27, vcc\n" \
    "v_cmp_lt_f32 vcc, v90, v25\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v90, v90, v27, vcc\n" \
    "SD_SKIP4_%=:\n" \
    "v_rsq_f32 v105, v95\n" \
    "v_rsq_f32 v115, v88\n" \
    "v_mul_f32 v94, v105, v105\n" \
    "v_mul_f32 v104, v115, v115\n" \
    "v_mul_f32 v107, v94, v105\n" \
    "v_mul_f32 v117, v104, v115\n" \
    "v_mul_f32 v100, v94, v111\n" \
    "v_mul_f32 v100, v100, v105\n" \
    "v_mul_f32 v102, v94, v113\n" \
    "v_mul_f32 v102, v102, v105\n" \
    "v_mul_f32 v110, v104, v121\n" \
    "v_mul_f32 v110, v110, v115\n" \
    "v_mul_f32 v112, v104, v123\n" \
    "v_mul_f32 v112, v112, v115\n" \
    "v_mul_f32 v52, v100, v71\n" \
    "v_fmac_f32 v52, v105, v76\n" \
    "v_mul_f32 v54, v100, v73\n" \
    "v_fmac_f32 v54, v105, v78\n" \
    "v_mul_f32 v56, v100, v75\n" \
    "v_fmac_f32 v56, v105, v80\n" \
    "v_mul_f32 v58, v110, v77\n" \
    "v_fmac_f32 v58, v115, v76\n" \
    "v_mul_f32 v60, v110, v79\n" \
    "v_fmac_f32 v60, v115, v78\n" \
    "v_mul_f32 v62, v110, v81\n" \
    "v_fmac_f32 v62, v115, v80\n" \
    "v_mul_f32 v114, v102, v71\n" \
    "v_fmac_f32 v114, v105, v36\n" \
    "v_mul_f32 v116, v102, v73\n" \
    "v_fmac_f32 v116, v105, v38\n" \
    "v_mul_f32 v118, v102, v75\n" \
    "v_fmac_f32 v118, v105, v40\n" \
    "v_fmac_f32 v114, v112, v77\n" \
    "v_fmac_f32 v114, v115, v42\n" \
    "v_fmac_f32 v116, v112, v79\n" \
    "v_fmac_f32 v116, v115, v44\n" \
    "v_fmac_f32 v118, v112, v81\n" \
    "v_fmac_f32 v118, v115, v46\n" \
    "v_rsq_f32 v105, v97\n" \
    "v_rsq_f32 v115, v90\n" \
    "v_mul_f32 v111, v87, v86\n" \
    "v_fmac_f32 v111, v85, v84\n" \
    "v_fmac_f32 v111, v83, v82\n" \
    "v_mov_b32_dpp v53, v114 row_ror:8 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_mov_b32_dpp v55, v116 row_ror:8 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_mov_b32_dpp v57, v118 row_ror:8 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_mul_f32 v113, v87, v40\n" \
    "v_fmac_f32 v113, v85, v38\n" \
    "v_fmac_f32 v113, v83, v36\n" \
    "v_mul_f32 v121, v93, v86\n" \
    "v_fmac_f32 v121, v91, v84\n" \
    "v_fmac_f32 v121, v89, v82\n" \
    "v_mul_f32 v123, v93, v46\n" \
    "v_fmac_f32 v123, v91, v44\n" \
    "v_fmac_f32 v123, v89, v42\n" \
    "v_mul_f32 v94, v105, v105\n" \
    "v_mul_f32 v104, v115, v115\n" \
    "v_mul_f32 v107, v94, v105\n" \
    "v_mul_f32 v117, v104, v115\n" \
    "v_mul_f32 v100, v94, v111\n" \
    "v_mul_f32 v100, v100, v105\n" \
    "v_mul_f32 v102, v94, v113\n" \
    "v_mul_f32 v102, v102, v105\n" \
    "v_mul_f32 v110, v104, v121\n" \
    "v_mul_f32 v110, v110, v115\n" \
    "v_mul_f32 v112, v104, v123\n" \
    "v_mul_f32 v112, v112, v115\n" \
    "v_fmac_f32 v52, v100, v83\n" \
    "v_fmac_f32 v52, v105, v82\n" \
    "v_fmac_f32 v54, v100, v85\n" \
    "v_fmac_f32 v54, v105, v84\n" \
    "v_fmac_f32 v56, v100, v87\n" \
    "v_fmac_f32 v56, v105, v86\n" \
    "v_fmac_f32 v58, v110, v89\n" \
    "v_fmac_f32 v58, v115, v82\n" \
    "v_fmac_f32 v60, v110, v91\n" \
    "v_fmac_f32 v60, v115, v84\n" \
    "v_fmac_f32 v62, v110, v93\n" \
    "v_fmac_f32 v62, v115, v86\n" \
    "v_mul_f32 v120, v102, v83\n" \
    "v_fmac_f32 v120, v105, v36\n" \
    "v_mul_f32 v122, v102, v85\n" \
    "v_fmac_f32 v122, v105, v38\n" \
    "v_mul_f32 v124, v102, v87\n" \
    "v_fmac_f32 v124, v105, v40\n" \
    "v_fmac_f32 v120, v112, v89\n" \
    "v_fmac_f32 v120, v115, v42\n" \
    "v_fmac_f32 v122, v112, v91\n" \
    "v_fmac_f32 v122, v115, v44\n" \
    "v_fmac_f32 v124, v112, v93\n" \
    "v_fmac_f32 v124, v115, v46\n" \
    "ds_read_b32 v59, v31 offset:40\n" \
    "ds_read_b32 v61, v31 offset:168\n" \
    "ds_read_b32 v63, v31 offset:296\n" \
    "ds_read_b32 v65, v31 offset:44\n" \
    "ds_read_b32 v67, v31 offset:172\n" \
    "ds_read_b32 v69, v31 offset:300\n" \
    "ds_read_b32 v76, v31 offset:424\n" \
    "ds_read_b32 v78, v31 offset:552\n" \
    "ds_read_b32 v80, v31 offset:680\n" \
    "ds_read_b32 v82, v31 offset:428\n" \
    "ds_read_b32 v84, v31 offset:556\n" \
    "ds_read_b32 v86, v31 offset:684\n" \
    "s_waitcnt lgkmcnt(9)\n" \
    "v_sub_f32 v71, v24, v59\n" \
    "v_sub_f32 v73, v26, v61\n" \
    "v_sub_f32 v75, v28, v63\n" \
    "v_sub_f32 v77, v30, v59\n" \
    "v_sub_f32 v79, v32, v61\n" \
    "v_sub_f32 v81, v34, v63\n" \
    "v_mul_f32 v95, v75, v75\n" \
    "v_fmac_f32 v95, v73, v73\n" \
    "v_fmac_f32 v95, v71, v71\n" \
    "v_mul_f32 v88, v81, v81\n" \
    "v_fmac_f32 v88, v79, v79\n" \
    "v_fmac_f32 v88, v77, v77\n" \
    "v_min_f32 v99, v95, v88\n" \
    "s_waitcnt lgkmcnt(6)\n" \
    "v_sub_f32 v83, v24, v65\n" \
    "v_sub_f32 v85, v26, v67\n" \
    "v_sub_f32 v87, v28, v69\n" \
    "v_sub_f32 v89, v30, v65\n" \
    "v_sub_f32 v91, v32, v67\n" \
    "v_sub_f32 v93, v34, v69\n" \
    "v_mul_f32 v97, v87, v87\n" \
    "v_fmac_f32 v97, v85, v85\n" \
    "v_fmac_f32 v97, v83, v83\n" \
    "v_mul_f32 v90, v93, v93\n" \
    "v_fmac_f32 v90, v91, v91\n" \
    "v_fmac_f32 v90, v89, v89\n" \
    "v_min_f32 v92, v97, v90\n" \
    "v_min_f32 v99, v99, v92\n" \
    "v_cmp_lt_f32 vcc, v99, v50\n" \
    "s_waitcnt lgkmcnt(0)\n" \
    "v_mul_f32 v111, v75, v80\n" \
    "v_fmac_f32 v111, v73, v78\n" \
    "v_fmac_f32 v111, v71, v76\n" \
    "v_add_f32_dpp v53, v120, v53 row_ror:9 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_add_f32_dpp v55, v122, v55 row_ror:9 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_add_f32_dpp v57, v124, v57 row_ror:9 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_mul_f32 v113, v75, v40\n" \
    "v_fmac_f32 v113, v73, v38\n" \
    "v_fmac_f32 v113, v71, v36\n" \
    "v_mul_f32 v121, v81, v80\n" \
    "v_fmac_f32 v121, v79, v78\n" \
    "v_fmac_f32 v121, v77, v76\n" \
    "v_mul_f32 v123, v81, v46\n" \
    "v_fmac_f32 v123, v79, v44\n" \
    "v_fmac_f32 v123, v77, v42\n" \
    "s_cbranch_vccz SD_SKIP5_%=\n" \
    "s_or_b64 %[nl], %[nl], vcc\n" \
    "v_cmp_lt_f32 vcc, v95, v50\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v95, v95, v27, vcc\n" \
    "v_cmp_lt_f32 vcc, v88, v25\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v88, v88, v27, vcc\n" \
    "v_cmp_lt_f32 vcc, v97, v50\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v97, v97, v27, vcc\n" \
    "v_cmp_lt_f32 vcc, v90, v25\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v90, v90, v27, vcc\n" \
    "SD_SKIP5_%=:\n" \
    "v_rsq_f32 v105, v95\n" \
    "v_rsq_f32 v115, v88\n" \
    "v_mul_f32 v94, v105, v105\n" \
    "v_mul_f32 v104, v115, v115\n" \
    "v_mul_f32 v107, v94, v105\n" \
    "v_mul_f32 v117, v104, v115\n" \
    "v_mul_f32 v100, v94, v111\n" \
    "v_mul_f32 v100, v100, v105\n" \
    "v_mul_f32 v102, v94, v113\n" \
    "v_mul_f32 v102, v102, v105\n" \
    "v_mul_f32 v110, v104, v121\n" \
    "v_mul_f32 v110, v110, v115\n" \
    "v_mul_f32 v112, v104, v123\n" \
    "v_mul_f32 v112, v112, v115\n" \
    "v_fmac_f32 v52, v100, v71\n" \
    "v_fmac_f32 v52, v105, v76\n" \
    "v_fmac_f32 v54, v100, v73\n" \
    "v_fmac_f32 v54, v105, v78\n" \
    "v_fmac_f32 v56, v100, v75\n" \
    "v_fmac_f32 v56, v105, v80\n" \
    "v_fmac_f32 v58, v110, v77\n" \
    "v_fmac_f32 v58, v115, v76\n" \
    "v_fmac_f32 v60, v110, v79\n" \
    "v_fmac_f32 v60, v115, v78\n" \
    "v_fmac_f32 v62, v110, v81\n" \
    "v_fmac_f32 v62, v115, v80\n" \
    "v_mul_f32 v114, v102, v71\n" \
    "v_fmac_f32 v114, v105, v36\n" \
    "v_mul_f32 v116, v102, v73\n" \
    "v_fmac_f32 v116, v105, v38\n" \
    "v_mul_f32 v118, v102, v75\n" \
    "v_fmac_f32 v118, v105, v40\n" \
    "v_fmac_f32 v114, v112, v77\n" \
    "v_fmac_f32 v114, v115, v42\n" \
    "v_fmac_f32 v116, v112, v79\n" \
    "v_fmac_f32 v116, v115, v44\n" \
    "v_fmac_f32 v118, v112, v81\n" \
    "v_fmac_f32 v118, v115, v46\n" \
    "v_rsq_f32 v105, v97\n" \
    "v_rsq_f32 v115, v90\n" \
    "v_mul_f32 v111, v87, v86\n" \
    "v_fmac_f32 v111, v85, v84\n" \
    "v_fmac_f32 v111, v83, v82\n" \
    "v_add_f32_dpp v53, v114, v53 row_ror:10 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_add_f32_dpp v55, v116, v55 row_ror:10 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_add_f32_dpp v57, v118, v57 row_ror:10 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_mul_f32 v113, v87, v40\n" \
    "v_fmac_f32 v113, v85, v38\n" \
    "v_fmac_f32 v113, v83, v36\n" \
    "v_mul_f32 v121, v93, v86\n" \
    "v_fmac_f32 v121, v91, v84\n" \
    "v_fmac_f32 v121, v89, v82\n" \
    "v_mul_f32 v123, v93, v46\n" \
    "v_fmac_f32 v123, v91, v44\n" \
    "v_fmac_f32 v123, v89, v42\n" \
    "v_mul_f32 v94, v105, v105\n" \
    "v_mul_f32 v104, v115, v115\n" \
    "v_mul_f32 v107, v94, v105\n" \
    "v_mul_f32 v117, v104, v115\n" \
    "v_mul_f32 v100, v94, v111\n" \
    "v_mul_f32 v100, v100, v105\n" \
    "v_mul_f32 v102, v94, v113\n" \
    "v_mul_f32 v102, v102, v105\n" \
    "v_mul_f32 v110, v104, v121\n" \
    "v_mul_f32 v110, v110, v115\n" \
    "v_mul_f32 v112, v104, v123\n" \
    "v_mul_f32 v112, v112, v115\n" \
    "v_fmac_f32 v52, v100, v83\n" \
    "v_fmac_f32 v52, v105, v82\n" \
    "v_fmac_f32 v54, v100, v85\n" \
    "v_fmac_f32 v54, v105, v84\n" \
    "v_fmac_f32 v56, v100, v87\n" \
    "v_fmac_f32 v56, v105, v86\n" \
    "v_fmac_f32 v58, v110, v89\n" \
    "v_fmac_f32 v58, v115, v82\n" \
    "v_fmac_f32 v60, v110, v91\n" \
    "v_fmac_f32 v60, v115, v84\n" \
    "v_fmac_f32 v62, v110, v93\n" \
    "v_fmac_f32 v62, v115, v86\n" \
    "v_mul_f32 v120, v102, v83\n" \
    "v_fmac_f32 v120, v105, v36\n" \
    "v_mul_f32 v122, v102, v85\n" \
    "v_fmac_f32 v122, v105, v38\n" \
    "v_mul_f32 v124, v102, v87\n" \
    "v_fmac_f32 v124, v105, v40\n" \
    "v_fmac_f32 v120, v112, v89\n" \
    "v_fmac_f32 v120, v115, v42\n" \
    "v_fmac_f32 v122, v112, v91\n" \
    "v_fmac_f32 v122, v115, v44\n" \
    "v_fmac_f32 v124, v112, v93\n" \
    "v_fmac_f32 v124, v115, v46\n" \
    "v_add_f32 v35, v35, v52\n" \
    "v_add_f32 v37, v37, v54\n" \
    "v_add_f32 v39, v39, v56\n" \
    "v_add_f32 v41, v41, v58\n" \
    "v_add_f32 v43, v43, v60\n" \
    "v_add_f32 v45, v45, v62\n" \
    "ds_read_b32 v59, v31 offset:48\n" \
    "ds_read_b32 v61, v31 offset:176\n" \
    "ds_read_b32 v63, v31 offset:304\n" \
    "ds_read_b32 v65, v31 offset:52\n" \
    "ds_read_b32 v67, v31 offset:180\n" \
    "ds_read_b32 v69, v31 offset:308\n" \
    "ds_read_b32 v76, v31 offset:432\n" \
    "ds_read_b32 v78, v31 offset:560\n" \
    "ds_read_b32 v80, v31 offset:688\n" \
    "ds_read_b32 v82, v31 offset:436\n" \
    "ds_read_b32 v84, v31 offset:564\n" \
    "ds_read_b32 v86, v31 offset:692\n" \
    "s_waitcnt lgkmcnt(9)\n" \
    "v_sub_f32 v71, v24, v59\n" \
    "v_sub_f32 v73, v26, v61\n" \
    "v_sub_f32 v75, v28, v63\n" \
    "v_sub_f32 v77, v30, v59\n" \
    "v_sub_f32 v79, v32, v61\n" \
    "v_sub_f32 v81, v34, v63\n" \
    "v_mul_f32 v95, v75, v75\n" \
    "v_fmac_f32 v95, v73, v73\n" \
    "v_fmac_f32 v95, v71, v71\n" \
    "v_mul_f32 v88, v81, v81\n" \
    "v_fmac_f32 v88, v79, v79\n" \
    "v_fmac_f32 v88, v77, v77\n" \
    "v_min_f32 v99, v95, v88\n" \
    "s_waitcnt lgkmcnt(6)\n" \
    "v_sub_f32 v83, v24, v65\n" \
    "v_sub_f32 v85, v26, v67\n" \
    "v_sub_f32 v87, v28, v69\n" \
    "v_sub_f32 v89, v30, v65\n" \
    "v_sub_f32 v91, v32, v67\n" \
    "v_sub_f32 v93, v34, v69\n" \
    "v_mul_f32 v97, v87, v87\n" \
    "v_fmac_f32 v97, v85, v85\n" \
    "v_fmac_f32 v97, v83, v83\n" \
    "v_mul_f32 v90, v93, v93\n" \
    "v_fmac_f32 v90, v91, v91\n" \
    "v_fmac_f32 v90, v89, v89\n" \
    "v_min_f32 v92, v97, v90\n" \
    "v_min_f32 v99, v99, v92\n" \
    "v_cmp_lt_f32 vcc, v99, v50\n" \
    "s_waitcnt lgkmcnt(0)\n" \
    "v_mul_f32 v111, v75, v80\n" \
    "v_fmac_f32 v111, v73, v78\n" \
    "v_fmac_f32 v111, v71, v76\n" \
    "v_add_f32_dpp v53, v120, v53 row_ror:11 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_add_f32_dpp v55, v122, v55 row_ror:11 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_add_f32_dpp v57, v124, v57 row_ror:11 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_mul_f32 v113, v75, v40\n" \
    "v_fmac_f32 v113, v73, v38\n" \
    "v_fmac_f32 v113, v71, v36\n" \
    "v_mul_f32 v121, v81, v80\n" \
    "v_fmac_f32 v121, v79, v78\n" \
    "v_fmac_f32 v121, v77, v76\n" \
    "v_mul_f32 v123, v81, v46\n" \
    "v_fmac_f32 v123, v79, v44\n" \
    "v_fmac_f32 v123, v77, v42\n" \
    "s_cbranch_vccz SD_SKIP6_%=\n" \
    "s_or_b64 %[nl], %[nl], vcc\n" \
    "v_cmp_lt_f32 vcc, v95, v50\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v95, v95, v27, vcc\n" \
    "v_cmp_lt_f32 vcc, v88, v25\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v88, v88, v27, vcc\n" \
    "v_cmp_lt_f32 vcc, v97, v50\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v97, v97, v27, vcc\n" \
    "v_cmp_lt_f32 vcc, v90, v25\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v90, v90, v27, vcc\n" \
    "SD_SKIP6_%=:\n" \
    "v_rsq_f32 v105, v95\n" \
    "v_rsq_f32 v115, v88\n" \
    "v_mul_f32 v94, v105, v105\n" \
    "v_mul_f32 v104, v115, v115\n" \
    "v_mul_f32 v107, v94, v105\n" \
    "v_mul_f32 v117, v104, v115\n" \
    "v_mul_f32 v100, v94, v111\n" \
    "v_mul_f32 v100, v100, v105\n" \
    "v_mul_f32 v102, v94, v113\n" \
    "v_mul_f32 v102, v102, v105\n" \
    "v_mul_f32 v110, v104, v121\n" \
    "v_mul_f32 v110, v110, v115\n" \
    "v_mul_f32 v112, v104, v123\n" \
    "v_mul_f32 v112, v112, v115\n" \
    "v_mul_f32 v52, v100, v71\n" \
    "v_fmac_f32 v52, v105, v76\n" \
    "v_mul_f32 v54, v100, v73\n" \
    "v_fmac_f32 v54, v105, v78\n" \
    "v_mul_f32 v56, v100, v75\n" \
    "v_fmac_f32 v56, v105, v80\n" \
    "v_mul_f32 v58, v110, v77\n" \
    "v_fmac_f32 v58, v115, v76\n" \
    "v_mul_f32 v60, v110, v79\n" \
    "v_fmac_f32 v60, v115, v78\n" \
    "v_mul_f32 v62, v110, v81\n" \
    "v_fmac_f32 v62, v115, v80\n" \
    "v_mul_f32 v114, v102, v71\n" \
    "v_fmac_f32 v114, v105, v36\n" \
    "v_mul_f32 v116, v102, v73\n" \
    "v_fmac_f32 v116, v105, v38\n" \
    "v_mul_f32 v118, v102, v75\n" \
    "v_fmac_f32 v118, v105, v40\n" \
    "v_fmac_f32 v114, v112, v77\n" \
    "v_fmac_f32 v114, v115, v42\n" \
    "v_fmac_f32 v116, v112, v79\n" \
    "v_fmac_f32 v116, v115, v44\n" \
    "v_fmac_f32 v118, v112, v81\n" \
    "v_fmac_f32 v118, v115, v46\n" \
    "v_rsq_f32 v105, v97\n" \
    "v_rsq_f32 v115, v90\n" \
    "v_mul_f32 v111, v87, v86\n" \
    "v_fmac_f32 v111, v85, v84\n" \
    "v_fmac_f32 v111, v83, v82\n" \
    "v_mov_b32_dpp v47, v114 row_ror:12 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_mov_b32_dpp v49, v116 row_ror:12 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_mov_b32_dpp v51, v118 row_ror:12 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_mul_f32 v113, v87, v40\n" \
    "v_fmac_f32 v113, v85, v38\n" \
    "v_fmac_f32 v113, v83, v36\n" \
    "v_mul_f32 v121, v93, v86\n" \
    "v_fmac_f32 v121, v91, v84\n" \
    "v_fmac_f32 v121, v89, v82\n" \
    "v_mul_f32 v123, v93, v46\n" \
    "v_fmac_f32 v123, v91, v44\n" \
    "v_fmac_f32 v123, v89, v42\n" \
    "v_mul_f32 v94, v105, v105\n" \
    "v_mul_f32 v104, v115, v115\n" \
    "v_mul_f32 v107, v94, v105\n" \
    "v_mul_f32 v117, v104, v115\n" \
    "v_mul_f32 v100, v94, v111\n" \
    "v_mul_f32 v100, v100, v105\n" \
    "v_mul_f32 v102, v94, v113\n" \
    "v_mul_f32 v102, v102, v105\n" \
    "v_mul_f32 v110, v104, v121\n" \
    "v_mul_f32 v110, v110, v115\n" \
    "v_mul_f32 v112, v104, v123\n" \
    "v_mul_f32 v112, v112, v115\n" \
    "v_fmac_f32 v52, v100, v83\n" \
    "v_fmac_f32 v52, v105, v82\n" \
    "v_fmac_f32 v54, v100, v85\n" \
    "v_fmac_f32 v54, v105, v84\n" \
    "v_fmac_f32 v56, v100, v87\n" \
    "v_fmac_f32 v56, v105, v86\n" \
    "v_fmac_f32 v58, v110, v89\n" \
    "v_fmac_f32 v58, v115, v82\n" \
    "v_fmac_f32 v60, v110, v91\n" \
    "v_fmac_f32 v60, v115, v84\n" \
    "v_fmac_f32 v62, v110, v93\n" \
    "v_fmac_f32 v62, v115, v86\n" \
    "v_mul_f32 v120, v102, v83\n" \
    "v_fmac_f32 v120, v105, v36\n" \
    "v_mul_f32 v122, v102, v85\n" \
    "v_fmac_f32 v122, v105, v38\n" \
    "v_mul_f32 v124, v102, v87\n" \
    "v_fmac_f32 v124, v105, v40\n" \
    "v_fmac_f32 v120, v112, v89\n" \
    "v_fmac_f32 v120, v115, v42\n" \
    "v_fmac_f32 v122, v112, v91\n" \
    "v_fmac_f32 v122, v115, v44\n" \
    "v_fmac_f32 v124, v112, v93\n" \
    "v_fmac_f32 v124, v115, v46\n" \
    "ds_read_b32 v59, v31 offset:56\n" \
    "ds_read_b32 v61, v31 offset:184\n" \
    "ds_read_b32 v63, v31 offset:312\n" \
    "ds_read_b32 v65, v31 offset:60\n" \
    "ds_read_b32 v67, v31 offset:188\n" \
    "ds_read_b32 v69, v31 offset:316\n" \
    "ds_read_b32 v76, v31 offset:440\n" \
    "ds_read_b32 v78, v31 offset:568\n" \
    "ds_read_b32 v80, v31 offset:696\n" \
    "ds_read_b32 v82, v31 offset:444\n" \
    "ds_read_b32 v84, v31 offset:572\n" \
    "ds_read_b32 v86, v31 offset:700\n" \
    "s_waitcnt lgkmcnt(9)\n" \
    "v_sub_f32 v71, v24, v59\n" \
    "v_sub_f32 v73, v26, v61\n" \
    "v_sub_f32 v75, v28, v63\n" \
    "v_sub_f32 v77, v30, v59\n" \
    "v_sub_f32 v79, v32, v61\n" \
    "v_sub_f32 v81, v34, v63\n" \
    "v_mul_f32 v95, v75, v75\n" \
    "v_fmac_f32 v95, v73, v73\n" \
    "v_fmac_f32 v95, v71, v71\n" \
    "v_mul_f32 v88, v81, v81\n" \
    "v_fmac_f32 v88, v79, v79\n" \
    "v_fmac_f32 v88, v77, v77\n" \
    "v_min_f32 v99, v95, v88\n" \
    "s_waitcnt lgkmcnt(6)\n" \
    "v_sub_f32 v83, v24, v65\n" \
    "v_sub_f32 v85, v26, v67\n" \
    "v_sub_f32 v87, v28, v69\n" \
    "v_sub_f32 v89, v30, v65\n" \
    "v_sub_f32 v91, v32, v67\n" \
    "v_sub_f32 v93, v34, v69\n" \
    "v_mul_f32 v97, v87, v87\n" \
    "v_fmac_f32 v97, v85, v85\n" \
    "v_fmac_f32 v97, v83, v83\n" \
    "v_mul_f32 v90, v93, v93\n" \
    "v_fmac_f32 v90, v91, v91\n" \
    "v_fmac_f32 v90, v89, v89\n" \
    "v_min_f32 v92, v97, v90\n" \
    "v_min_f32 v99, v99, v92\n" \
    "v_cmp_lt_f32 vcc, v99, v50\n" \
    "s_waitcnt lgkmcnt(0)\n" \
    "v_mul_f32 v111, v75, v80\n" \
    "v_fmac_f32 v111, v73, v78\n" \
    "v_fmac_f32 v111, v71, v76\n" \
    "v_add_f32_dpp v47, v120, v47 row_ror:13 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_add_f32_dpp v49, v122, v49 row_ror:13 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_add_f32_dpp v51, v124, v51 row_ror:13 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_mul_f32 v113, v75, v40\n" \
    "v_fmac_f32 v113, v73, v38\n" \
    "v_fmac_f32 v113, v71, v36\n" \
    "v_mul_f32 v121, v81, v80\n" \
    "v_fmac_f32 v121, v79, v78\n" \
    "v_fmac_f32 v121, v77, v76\n" \
    "v_mul_f32 v123, v81, v46\n" \
    "v_fmac_f32 v123, v79, v44\n" \
    "v_fmac_f32 v123, v77, v42\n" \
    "s_cbranch_vccz SD_SKIP7_%=\n" \
    "s_or_b64 %[nl], %[nl], vcc\n" \
    "v_cmp_lt_f32 vcc, v95, v50\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v95, v95, v27, vcc\n" \
    "v_cmp_lt_f32 vcc, v88, v25\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v88, v88, v27, vcc\n" \
    "v_cmp_lt_f32 vcc, v97, v50\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v97, v97, v27, vcc\n" \
    "v_cmp_lt_f32 vcc, v90, v25\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v90, v90, v27, vcc\n" \
    "SD_SKIP7_%=:\n" \
    "v_rsq_f32 v105, v95\n" \
    "v_rsq_f32 v115, v88\n" \
    "v_mul_f32 v94, v105, v105\n" \
    "v_mul_f32 v104, v115, v115\n" \
    "v_mul_f32 v107, v94, v105\n" \
    "v_mul_f32 v117, v104, v115\n" \
    "v_mul_f32 v100, v94, v111\n" \
    "v_mul_f32 v100, v100, v105\n" \
    "v_mul_f32 v102, v94, v113\n" \
    "v_mul_f32 v102, v102, v105\n" \
    "v_mul_f32 v110, v104, v121\n" \
    "v_mul_f32 v110, v110, v115\n" \
    "v_mul_f32 v112, v104, v123\n" \
    "v_mul_f32 v112, v112, v115\n" \
    "v_fmac_f32 v52, v100, v71\n" \
    "v_fmac_f32 v52, v105, v76\n" \
    "v_fmac_f32 v54, v100, v73\n" \
    "v_fmac_f32 v54, v105, v78\n" \
    "v_fmac_f32 v56, v100, v75\n" \
    "v_fmac_f32 v56, v105, v80\n" \
    "v_fmac_f32 v58, v110, v77\n" \
    "v_fmac_f32 v58, v115, v76\n" \
    "v_fmac_f32 v60, v110, v79\n" \
    "v_fmac_f32 v60, v115, v78\n" \
    "v_fmac_f32 v62, v110, v81\n" \
    "v_fmac_f32 v62, v115, v80\n" \
    "v_mul_f32 v114, v102, v71\n" \
    "v_fmac_f32 v114, v105, v36\n" \
    "v_mul_f32 v116, v102, v73\n" \
    "v_fmac_f32 v116, v105, v38\n" \
    "v_mul_f32 v118, v102, v75\n" \
    "v_fmac_f32 v118, v105, v40\n" \
    "v_fmac_f32 v114, v112, v77\n" \
    "v_fmac_f32 v114, v115, v42\n" \
    "v_fmac_f32 v116, v112, v79\n" \
    "v_fmac_f32 v116, v115, v44\n" \
    "v_fmac_f32 v118, v112, v81\n" \
    "v_fmac_f32 v118, v115, v46\n" \
    "v_rsq_f32 v105, v97\n" \
    "v_rsq_f32 v115, v90\n" \
    "v_mul_f32 v111, v87, v86\n" \
    "v_fmac_f32 v111, v85, v84\n" \
    "v_fmac_f32 v111, v83, v82\n" \
    "v_add_f32_dpp v47, v114, v47 row_ror:14 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_add_f32_dpp v49, v116, v49 row_ror:14 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_add_f32_dpp v51, v118, v51 row_ror:14 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_mul_f32 v113, v87, v40\n" \
    "v_fmac_f32 v113, v85, v38\n" \
    "v_fmac_f32 v113, v83, v36\n" \
    "v_mul_f32 v121, v93, v86\n" \
    "v_fmac_f32 v121, v91, v84\n" \
    "v_fmac_f32 v121, v89, v82\n" \
    "v_mul_f32 v123, v93, v46\n" \
    "v_fmac_f32 v123, v91, v44\n" \
    "v_fmac_f32 v123, v89, v42\n" \
    "v_mul_f32 v94, v105, v105\n" \
    "v_mul_f32 v104, v115, v115\n" \
    "v_mul_f32 v107, v94, v105\n" \
    "v_mul_f32 v117, v104, v115\n" \
    "v_mul_f32 v100, v94, v111\n" \
    "v_mul_f32 v100, v100, v105\n" \
    "v_mul_f32 v102, v94, v113\n" \
    "v_mul_f32 v102, v102, v105\n" \
    "v_mul_f32 v110, v104, v121\n" \
    "v_mul_f32 v110, v110, v115\n" \
    "v_mul_f32 v112, v104, v123\n" \
    "v_mul_f32 v112, v112, v115\n" \
    "v_fmac_f32 v52, v100, v83\n" \
    "v_fmac_f32 v52, v105, v82\n" \
    "v_fmac_f32 v54, v100, v85\n" \
    "v_fmac_f32 v54, v105, v84\n" \
    "v_fmac_f32 v56, v100, v87\n" \
    "v_fmac_f32 v56, v105, v86\n" \
    "v_fmac_f32 v58, v110, v89\n" \
    "v_fmac_f32 v58, v115, v82\n" \
    "v_fmac_f32 v60, v110, v91\n" \
    "v_fmac_f32 v60, v115, v84\n" \
    "v_fmac_f32 v62, v110, v93\n" \
    "v_fmac_f32 v62, v115, v86\n" \
    "v_mul_f32 v120, v102, v83\n" \
    "v_fmac_f32 v120, v105, v36\n" \
    "v_mul_f32 v122, v102, v85\n" \
    "v_fmac_f32 v122, v105, v38\n" \
    "v_mul_f32 v124, v102, v87\n" \
    "v_fmac_f32 v124, v105, v40\n" \
    "v_fmac_f32 v120, v112, v89\n" \
    "v_fmac_f32 v120, v115, v42\n" \
    "v_fmac_f32 v122, v112, v91\n" \
    "v_fmac_f32 v122, v115, v44\n" \
    "v_fmac_f32 v124, v112, v93\n" \
    "v_fmac_f32 v124, v115, v46\n" \
    "v_add_f32 v35, v35, v52\n" \
    "v_add_f32 v37, v37, v54\n" \
    "v_add_f32 v39, v39, v56\n" \
    "v_add_f32 v41, v41, v58\n" \
    "v_add_f32 v43, v43, v60\n" \
    "v_add_f32 v45, v45, v62\n" \
    "s_nop 1\n" \
    "v_add_f32_dpp v47, v120, v47 row_ror:15 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_add_f32_dpp v49, v122, v49 row_ror:15 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_add_f32_dpp v51, v124, v51 row_ror:15 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_add_f32 v53, v53, v47\n" \
    "v_add_f32 v55, v55, v49\n" \
    "v_add_f32 v57, v57, v51\n" \
    "ds_write_b32 v33, v53 offset:768\n" \
    "ds_write_b32 v33, v55 offset:832\n" \
    "ds_write_b32 v33, v57 offset:896\n" \
    "v_add_f32 v125, v64, v35\n" \
    "v_sub_f32 v126, v125, v64\n" \
    "v_sub_f32 v35, v35, v126\n" \
    "v_mov_b32 v64, v125\n" \
    "v_add_f32 v125, v66, v37\n" \
    "v_sub_f32 v126, v125, v66\n" \
    "v_sub_f32 v37, v37, v126\n" \
    "v_mov_b32 v66, v125\n" \
    "v_add_f32 v125, v68, v39\n" \
    "v_sub_f32 v126, v125, v68\n" \
    "v_sub_f32 v39, v39, v126\n" \
    "v_mov_b32 v68, v125\n" \
    "v_add_f32 v125, v70, v41\n" \
    "v_sub_f32 v126, v125, v70\n" \
    "v_sub_f32 v41, v41, v126\n" \
    "v_mov_b32 v70, v125\n" \
    "v_add_f32 v125, v72, v43\n" \
    "v_sub_f32 v126, v125, v72\n" \
    "v_sub_f32 v43, v43, v126\n" \
    "v_mov_b32 v72, v125\n" \
    "v_add_f32 v125, v74, v45\n" \
    "v_sub_f32 v126, v125, v74\n" \
    "v_sub_f32 v45, v45, v126\n" \
    "v_mov_b32 v74, v125\n"

// one chunk; 1385 instructions per chunk, 0 products with same-parity sources
#define SD_WAVE_CHUNK_OSEEN_PER \
    "ds_read_b32 v59, v31 offset:0\n" \
    "ds_read_b32 v61, v31 offset:128\n" \
    "ds_read_b32 v63, v31 offset:256\n" \
    "ds_read_b32 v65, v31 offset:4\n" \
    "ds_read_b32 v67, v31 offset:132\n" \
    "ds_read_b32 v69, v31 offset:260\n" \
    "ds_read_b32 v76, v31 offset:384\n" \
    "ds_read_b32 v78, v31 offset:512\n" \
    "ds_read_b32 v80, v31 offset:640\n" \
    "ds_read_b32 v82, v31 offset:388\n" \
    "ds_read_b32 v84, v31 offset:516\n" \
    "ds_read_b32 v86, v31 offset:644\n" \
    "s_waitcnt lgkmcnt(9)\n" \
    "v_sub_u32 v101, v24, v59\n" \
    "v_cvt_f32_i32 v71, v101\n" \
    "v_sub_u32 v101, v26, v61\n" \
    "v_cvt_f32_i32 v73, v101\n" \
    "v_sub_u32 v101, v28, v63\n" \
    "v_cvt_f32_i32 v75, v101\n" \
    "v_sub_u32 v103, v30, v59\n" \
    "v_cvt_f32_i32 v77, v103\n" \
    "v_sub_u32 v103, v32, v61\n" \
    "v_cvt_f32_i32 v79, v103\n" \
    "v_sub_u32 v103, v34, v63\n" \
    "v_cvt_f32_i32 v81, v103\n" \
    "v_mul_f32 v95, v75, v75\n" \
    "v_fmac_f32 v95, v73, v73\n" \
    "v_fmac_f32 v95, v71, v71\n" \
    "v_mul_f32 v88, v81, v81\n" \
    "v_fmac_f32 v88, v79, v79\n" \
    "v_fmac_f32 v88, v77, v77\n" \
    "v_min_f32 v99, v95, v88\n" \
    "s_waitcnt lgkmcnt(6)\n" \
    "v_sub_u32 v101, v24, v65\n" \
    "v_cvt_f32_i32 v83, v101\n" \
    "v_sub_u32 v101, v26, v67\n" \
    "v_cvt_f32_i32 v85, v101\n" \
    "v_sub_u32 v101, v28, v69\n" \
    "v_cvt_f32_i32 v87, v101\n" \
    "v_sub_u32 v103, v30, v65\n" \
    "v_cvt_f32_i32 v89, v103\n" \
    "v_sub_u32 v103, v32, v67\n" \
    "v_cvt_f32_i32 v91, v103\n" \
    "v_sub_u32 v103, v34, v69\n" \
    "v_cvt_f32_i32 v93, v103\n" \
    "v_mul_f32 v97, v87, v87\n" \
    "v_fmac_f32 v97, v85, v85\n" \
    "v_fmac_f32 v97, v83, v83\n" \
    "v_mul_f32 v90, v93, v93\n" \
    "v_fmac_f32 v90, v91, v91\n" \
    "v_fmac_f32 v90, v89, v89\n" \
    "v_min_f32 v92, v97, v90\n" \
    "v_min_f32 v99, v99, v92\n" \
    "v_cmp_lt_f32 vcc, v99, v50\n" \
    "s_waitcnt lgkmcnt(0)\n" \
    "v_mul_f32 v111, v75, v80\n" \
    "v_fmac_f32 v111, v73, v78\n" \
    "v_fmac_f32 v111, v71, v76\n" \
    "v_mul_f32 v113, v75, v40\n" \
    "v_fmac_f32 v113, v73, v38\n" \
    "v_fmac_f32 v113, v71, v36\n" \
    "v_mul_f32 v121, v81, v80\n" \
    "v_fmac_f32 v121, v79, v78\n" \
    "v_fmac_f32 v121, v77, v76\n" \
    "v_mul_f32 v123, v81, v46\n" \
    "v_fmac_f32 v123, v79, v44\n" \
    "v_fmac_f32 v123, v77, v42\n" \
    "s_cbranch_vccz SD_SKIP0_%=\n" \
    "s_or_b64 %[nl], %[nl], vcc\n" \
    "v_cmp_lt_f32 vcc, v95, v50\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v95, v95, v27, vcc\n" \
    "v_cmp_lt_f32 vcc, v88, v25\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v88, v88, v27, vcc\n" \
    "v_cmp_lt_f32 vcc, v97, v50\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v97, v97, v27, vcc\n" \
    "v_cmp_lt_f32 vcc, v90, v25\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v90, v90, v27, vcc\n" \
    "SD_SKIP0_%=:\n" \
    "v_rsq_f32 v105, v95\n" \
    "v_rsq_f32 v115, v88\n" \
    "v_mul_f32 v94, v105, v105\n" \
    "v_mul_f32 v104, v115, v115\n" \
    "v_mul_f32 v107, v94, v105\n" \
    "v_mul_f32 v117, v104, v115\n" \
    "v_mul_f32 v100, v94, v111\n" \
    "v_mul_f32 v100, v100, v105\n" \
    "v_mul_f32 v102, v94, v113\n" \
    "v_mul_f32 v102, v102, v105\n" \
    "v_mul_f32 v110, v104, v121\n" \
    "v_mul_f32 v110, v110, v115\n" \
    "v_mul_f32 v112, v104, v123\n" \
    "v_mul_f32 v112, v112, v115\n" \
    "v_mul_f32 v52, v100, v71\n" \
    "v_fmac_f32 v52, v105, v76\n" \
    "v_mul_f32 v54, v100, v73\n" \
    "v_fmac_f32 v54, v105, v78\n" \
    "v_mul_f32 v56, v100, v75\n" \
    "v_fmac_f32 v56, v105, v80\n" \
    "v_mul_f32 v58, v110, v77\n" \
    "v_fmac_f32 v58, v115, v76\n" \
    "v_mul_f32 v60, v110, v79\n" \
    "v_fmac_f32 v60, v115, v78\n" \
    "v_mul_f32 v62, v110, v81\n" \
    "v_fmac_f32 v62, v115, v80\n" \
    "v_mul_f32 v53, v102, v71\n" \
    "v_fmac_f32 v53, v105, v36\n" \
    "v_mul_f32 v55, v102, v73\n" \
    "v_fmac_f32 v55, v105, v38\n" \
    "v_mul_f32 v57, v102, v75\n" \
    "v_fmac_f32 v57, v105, v40\n" \
    "v_fmac_f32 v53, v112, v77\n" \
    "v_fmac_f32 v53, v115, v42\n" \
    "v_fmac_f32 v55, v112, v79\n" \
    "v_fmac_f32 v55, v115, v44\n" \
    "v_fmac_f32 v57, v112, v81\n" \
    "v_fmac_f32 v57, v115, v46\n" \
    "v_rsq_f32 v105, v97\n" \
    "v_rsq_f32 v115, v90\n" \
    "v_mul_f32 v111, v87, v86\n" \
    "v_fmac_f32 v111, v85, v84\n" \
    "v_fmac_f32 v111, v83, v82\n" \
    "v_mul_f32 v113, v87, v40\n" \
    "v_fmac_f32 v113, v85, v38\n" \
    "v_fmac_f32 v113, v83, v36\n" \
    "v_mul_f32 v121, v93, v86\n" \
    "v_fmac_f32 v121, v91, v84\n" \
    "v_fmac_f32 v121, v89, v82\n" \
    "v_mul_f32 v123, v93, v46\n" \
    "v_fmac_f32 v123, v91, v44\n" \
    "v_fmac_f32 v123, v89, v42\n" \
    "v_mul_f32 v94, v105, v105\n" \
    "v_mul_f32 v104, v115, v115\n" \
    "v_mul_f32 v107, v94, v105\n" \
    "v_mul_f32 v117, v104, v115\n" \
    "v_mul_f32 v100, v94, v111\n" \
    "v_mul_f32 v100, v100, v105\n" \
    "v_mul_f32 v102, v94, v113\n" \
    "v_mul_f32 v102, v102, v105\n" \
    "v_mul_f32 v110, v104, v121\n" \
    "v_mul_f32 v110, v110, v115\n" \
    "v_mul_f32 v112, v104, v123\n" \
    "v_mul_f32 v112, v112, v115\n" \
    "v_fmac_f32 v52, v100, v83\n" \
    "v_fmac_f32 v52, v105, v82\n" \
    "v_fmac_f32 v54, v100, v85\n" \
    "v_fmac_f32 v54, v105, v84\n" \
    "v_fmac_f32 v56, v100, v87\n" \
    "v_fmac_f32 v56, v105, v86\n" \
    "v_fmac_f32 v58, v110, v89\n" \
    "v_fmac_f32 v58, v115, v82\n" \
    "v_fmac_f32 v60, v110, v91\n" \
    "v_fmac_f32 v60, v115, v84\n" \
    "v_fmac_f32 v62, v110, v93\n" \
    "v_fmac_f32 v62, v115, v86\n" \
    "v_mul_f32 v120, v102, v83\n" \
    "v_fmac_f32 v120, v105, v36\n" \
    "v_mul_f32 v122, v102, v85\n" \
    "v_fmac_f32 v122, v105, v38\n" \
    "v_mul_f32 v124, v102, v87\n" \
    "v_fmac_f32 v124, v105, v40\n" \
    "v_fmac_f32 v120, v112, v89\n" \
    "v_fmac_f32 v120, v115, v42\n" \
    "v_fmac_f32 v122, v112, v91\n" \
    "v_fmac_f32 v122, v115, v44\n" \
    "v_fmac_f32 v124, v112, v93\n" \
    "v_fmac_f32 v124, v115, v46\n" \
    "ds_read_b32 v59, v31 offset:8\n" \
    "ds_read_b32 v61, v31 offset:136\n" \
    "ds_read_b32 v63, v31 offset:264\n" \
    "ds_read_b32 v65, v31 offset:12\n" \
    "ds_read_b32 v67, v31 offset:140\n" \
    "ds_read_b32 v69, v31 offset:268\n" \
    "ds_read_b32 v76, v31 offset:392\n" \
    "ds_read_b32 v78, v31 offset:520\n" \
    "ds_read_b32 v80, v31 offset:648\n" \
    "ds_read_b32 v82, v31 offset:396\n" \
    "ds_read_b32 v84, v31 offset:524\n" \
    "ds_read_b32 v86, v31 offset:652\n" \
    "s_waitcnt lgkmcnt(9)\n" \
    "v_sub_u32 v101, v24, v59\n" \
    "v_cvt_f32_i32 v71, v101\n" \
    "v_sub_u32 v101, v26, v61\n" \
    "v_cvt_f32_i32 v73, v101\n" \
    "v_sub_u32 v101, v28, v63\n" \
    "v_cvt_f32_i32 v75, v101\n" \
    "v_sub_u32 v103, v30, v59\n" \
    "v_cvt_f32_i32 v77, v103\n" \
    "v_sub_u32 v103, v32, v61\n" \
    "v_cvt_f32_i32 v79, v103\n" \
    "v_sub_u32 v103, v34, v63\n" \
    "v_cvt_f32_i32 v81, v103\n" \
    "v_mul_f32 v95, v75, v75\n" \
    "v_fmac_f32 v95, v73, v73\n" \
    "v_fmac_f32 v95, v71, v71\n" \
    "v_mul_f32 v88, v81, v81\n" \
    "v_fmac_f32 v88, v79, v79\n" \
    "v_fmac_f32 v88, v77, v77\n" \
    "v_min_f32 v99, v95, v88\n" \
    "s_waitcnt lgkmcnt(6)\n" \
    "v_sub_u32 v101, v24, v65\n" \
    "v_cvt_f32_i32 v83, v101\n" \
    "v_sub_u32 v101, v26, v67\n" \
    "v_cvt_f32_i32 v85, v101\n" \
    "v_sub_u32 v101, v28, v69\n" \
    "v_cvt_f32_i32 v87, v101\n" \
    "v_sub_u32 v103, v30, v65\n" \
    "v_cvt_f32_i32 v89, v103\n" \
    "v_sub_u32 v103, v32, v67\n" \
    "v_cvt_f32_i32 v91, v103\n" \
    "v_sub_u32 v103, v34, v69\n" \
    "v_cvt_f32_i32 v93, v103\n" \
    "v_mul_f32 v97, v87, v87\n" \
    "v_fmac_f32 v97, v85, v85\n" \
    "v_fmac_f32 v97, v83, v83\n" \
    "v_mul_f32 v90, v93, v93\n" \
    "v_fmac_f32 v90, v91, v91\n" \
    "v_fmac_f32 v90, v89, v89\n" \
    "v_min_f32 v92, v97, v90\n" \
    "v_min_f32 v99, v99, v92\n" \
    "v_cmp_lt_f32 vcc, v99, v50\n" \
    "s_waitcnt lgkmcnt(0)\n" \
    "v_mul_f32 v111, v75, v80\n" \
    "v_fmac_f32 v111, v73, v78\n" \
    "v_fmac_f32 v111, v71, v76\n" \
    "v_add_f32_dpp v53, v120, v53 row_ror:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_add_f32_dpp v55, v122, v55 row_ror:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_add_f32_dpp v57, v124, v57 row_ror:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_mul_f32 v113, v75, v40\n" \
    "v_fmac_f32 v113, v73, v38\n" \
    "v_fmac_f32 v113, v71, v36\n" \
    "v_mul_f32 v121, v81, v80\n" \
    "v_fmac_f32 v121, v79, v78\n" \
    "v_fmac_f32 v121, v77, v76\n" \
    "v_mul_f32 v123, v81, v46\n" \
    "v_fmac_f32 v123, v79, v44\n" \
    "v_fmac_f32 v123, v77, v42\n" \
    "s_cbranch_vccz SD_SKIP1_%=\n" \
    "s_or_b64 %[nl], %[nl], vcc\n" \
    "v_cmp_lt_f32 vcc, v95, v50\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v95, v95, v27, vcc\n" \
    "v_cmp_lt_f32 vcc, v88, v25\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v88, v88, v27, vcc\n" \
    "v_cmp_lt_f32 vcc, v97, v50\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v97, v97, v27, vcc\n" \
    "v_cmp_lt_f32 vcc, v90, v25\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v90, v90, v27, vcc\n" \
    "SD_SKIP1_%=:\n" \
    "v_rsq_f32 v105, v95\n" \
    "v_rsq_f32 v115, v88\n" \
    "v_mul_f32 v94, v105, v105\n" \
    "v_mul_f32 v104, v115, v115\n" \
    "v_mul_f32 v107, v94, v105\n" \
    "v_mul_f32 v117, v104, v115\n" \
    "v_mul_f32 v100, v94, v111\n" \
    "v_mul_f32 v100, v100, v105\n" \
    "v_mul_f32 v102, v94, v113\n" \
    "v_mul_f32 v102, v102, v105\n" \
    "v_mul_f32 v110, v104, v121\n" \
    "v_mul_f32 v110, v110, v115\n" \
    "v_mul_f32 v112, v104, v123\n" \
    "v_mul_f32 v112, v112, v115\n" \
    "v_fmac_f32 v52, v100, v71\n" \
    "v_fmac_f32 v52, v105, v76\n" \
    "v_fmac_f32 v54, v100, v73\n" \
    "v_fmac_f32 v54, v105, v78\n" \
    "v_fmac_f32 v56, v100, v75\n" \
    "v_fmac_f32 v56, v105, v80\n" \
    "v_fmac_f32 v58, v110, v77\n" \
    "v_fmac_f32 v58, v115, v76\n" \
    "v_fmac_f32 v60, v110, v79\n" \
    "v_fmac_f32 v60, v115, v78\n" \
    "v_fmac_f32 v62, v110, v81\n" \
    "v_fmac_f32 v62, v115, v80\n" \
    "v_mul_f32 v114, v102, v71\n" \
    "v_fmac_f32 v114, v105, v36\n" \
    "v_mul_f32 v116, v102, v73\n" \
    "v_fmac_f32 v116, v105, v38\n" \
    "v_mul_f32 v118, v102, v75\n" \
    "v_fmac_f32 v118, v105, v40\n" \
    "v_fmac_f32 v114, v112, v77\n" \
    "v_fmac_f32 v114, v115, v42\n" \
    "v_fmac_f32 v116, v112, v79\n" \
    "v_fmac_f32 v116, v115, v44\n" \
    "v_fmac_f32 v118, v112, v81\n" \
    "v_fmac_f32 v118, v115, v46\n" \
    "v_rsq_f32 v105, v97\n" \
    "v_rsq_f32 v115, v90\n" \
    "v_mul_f32 v111, v87, v86\n" \
    "v_fmac_f32 v111, v85, v84\n" \
    "v_fmac_f32 v111, v83, v82\n" \
    "v_add_f32_dpp v53, v114, v53 row_ror:2 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_add_f32_dpp v55, v116, v55 row_ror:2 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_add_f32_dpp v57, v118, v57 row_ror:2 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_mul_f32 v113, v87, v40\n" \
    "v_fmac_f32 v113, v85, v38\n" \
    "v_fmac_f32 v113, v83, v36\n" \
    "v_mul_f32 v121, v93, v86\n" \
    "v_fmac_f32 v121, v91, v84\n" \
    "v_fmac_f32 v121, v89, v82\n" \
    "v_mul_f32 v123, v93, v46\n" \
    "v_fmac_f32 v123, v91, v44\n" \
    "v_fmac_f32 v123, v89, v42\n" \
    "v_mul_f32 v94, v105, v105\n" \
    "v_mul_f32 v104, v115, v115\n" \
    "v_mul_f32 v107, v94, v105\n" \
    "v_mul_f32 v117, v104, v115\n" \
    "v_mul_f32 v100, v94, v111\n" \
    "v_mul_f32 v100, v100, v105\n" \
    "v_mul_f32 v102, v94, v113\n" \
    "v_mul_f32 v102, v102, v105\n" \
    "v_mul_f32 v110, v104, v121\n" \
    "v_mul_f32 v110, v110, v115\n" \
    "v_mul_f32 v112, v104, v123\n" \
    "v_mul_f32 v112, v112, v115\n" \
    "v_fmac_f32 v52, v100, v83\n" \
    "v_fmac_f32 v52, v105, v82\n" \
    "v_fmac_f32 v54, v100, v85\n" \
    "v_fmac_f32 v54, v105, v84\n" \
    "v_fmac_f32 v56, v100, v87\n" \
    "v_fmac_f32 v56, v105, v86\n" \
    "v_fmac_f32 v58, v110, v89\n" \
    "v_fmac_f32 v58, v115, v82\n" \
    "v_fmac_f32 v60, v110, v91\n" \
    "v_fmac_f32 v60, v115, v84\n" \
    "v_fmac_f32 v62, v110, v93\n" \
    "v_fmac_f32 v62, v115, v86\n" \
    "v_mul_f32 v120, v102, v83\n" \
    "v_fmac_f32 v120, v105, v36\n" \
    "v_mul_f32 v122, v102, v85\n" \
    "v_fmac_f32 v122, v105, v38\n" \
    "v_mul_f32 v124, v102, v87\n" \
    "v_fmac_f32 v124, v105, v40\n" \
    "v_fmac_f32 v120, v112, v89\n" \
    "v_fmac_f32 v120, v115, v42\n" \
    "v_fmac_f32 v122, v112, v91\n" \
    "v_fmac_f32 v122, v115, v44\n" \
    "v_fmac_f32 v124, v112, v93\n" \
    "v_fmac_f32 v124, v115, v46\n" \
    "v_add_f32 v35, v35, v52\n" \
    "v_add_f32 v37, v37, v54\n" \
    "v_add_f32 v39, v39, v56\n" \
    "v_add_f32 v41, v41, v58\n" \
    "v_add_f32 v43, v43, v60\n" \
    "v_add_f32 v45, v45, v62\n" \
    "ds_read_b32 v59, v31 offset:16\n" \
    "ds_read_b32 v61, v31 offset:144\n" \
    "ds_read_b32 v63, v31 offset:272\n" \
    "ds_read_b32 v65, v31 offset:20\n" \
    "ds_read_b32 v67, v31 offset:148\n" \
    "ds_read_b32 v69, v31 offset:276\n" \
    "ds_read_b32 v76, v31 offset:400\n" \
    "ds_read_b32 v78, v31 offset:528\n" \
    "ds_read_b32 v80, v31 offset:656\n" \
    "ds_read_b32 v82, v31 offset:404\n" \
    "ds_read_b32 v84, v31 offset:532\n" \
    "ds_read_b32 v86, v31 offset:660\n" \
    "s_waitcnt lgkmcnt(9)\n" \
    "v_sub_u32 v101, v24, v59\n" \
    "v_cvt_f32_i32 v71, v101\n" \
    "v_sub_u32 v101, v26, v61\n" \
    "v_cvt_f32_i32 v73, v101\n" \
    "v_sub_u32 v101, v28, v63\n" \
    "v_cvt_f32_i32 v75, v101\n" \
    "v_sub_u32 v103, v30, v59\n" \
    "v_cvt_f32_i32 v77, v103\n" \
    "v_sub_u32 v103, v32, v61\n" \
    "v_cvt_f32_i32 v79, v103\n" \
    "v_sub_u32 v103, v34, v63\n" \
    "v_cvt_f32_i32 v81, v103\n" \
    "v_mul_f32 v95, v75, v75\n" \
    "v_fmac_f32 v95, v73, v73\n" \
    "v_fmac_f32 v95, v71, v71\n" \
    "v_mul_f32 v88, v81, v81\n" \
    "v_fmac_f32 v88, v79, v79\n" \
    "v_fmac_f32 v88, v77, v77\n" \
    "v_min_f32 v99, v95, v88\n" \
    "s_waitcnt lgkmcnt(6)\n" \
    "v_sub_u32 v101, v24, v65\n" \
    "v_cvt_f32_i32 v83, v101\n" \
    "v_sub_u32 v101, v26, v67\n" \
    "v_cvt_f32_i32 v85, v101\n" \
    "v_sub_u32 v101, v28, v69\n" \
    "v_cvt_f32_i32 v87, v101\n" \
    "v_sub_u32 v103, v30, v65\n" \
    "v_cvt_f32_i32 v89, v103\n" \
    "v_sub_u32 v103, v32, v67\n" \
    "v_cvt_f32_i32 v91, v103\n" \
    "v_sub_u32 v103, v34, v69\n" \
    "v_cvt_f32_i32 v93, v103\n" \
    "v_mul_f32 v97, v87, v87\n" \
    "v_fmac_f32 v97, v85, v85\n" \
    "v_fmac_f32 v97, v83, v83\n" \
    "v_mul_f32 v90, v93, v93\n" \
    "v_fmac_f32 v90, v91, v91\n" \
    "v_fmac_f32 v90, v89, v89\n" \
    "v_min_f32 v92, v97, v90\n" \
    "v_min_f32 v99, v99, v92\n" \
    "v_cmp_lt_f32 vcc, v99, v50\n" \
    "s_waitcnt lgkmcnt(0)\n" \
    "v_mul_f32 v111, v75, v80\n" \
    "v_fmac_f32 v111, v73, v78\n" \
    "v_fmac_f32 v111, v71, v76\n" \
    "v_add_f32_dpp v53, v120, v53 row_ror:3 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_add_f32_dpp v55, v122, v55 row_ror:3 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_add_f32_dpp v57, v124, v57 row_ror:3 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_mul_f32 v113, v75, v40\n" \
    "v_fmac_f32 v113, v73, v38\n" \
    "v_fmac_f32 v113, v71, v36\n" \
    "v_mul_f32 v121, v81, v80\n" \
    "v_fmac_f32 v121, v79, v78\n" \
    "v_fmac_f32 v121, v77, v76\n" \
    "v_mul_f32 v123, v81, v46\n" \
    "v_fmac_f32 v123, v79, v44\n" \
    "v_fmac_f32 v123, v77, v42\n" \
    "s_cbranch_vccz SD_SKIP2_%=\n" \
    "s_or_b64 %[nl], %[nl], vcc\n" \
    "v_cmp_lt_f32 vcc, v95, v50\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v95, v95, v27, vcc\n" \
    "v_cmp_lt_f32 vcc, v88, v25\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v88, v88, v27, vcc\n" \
    "v_cmp_lt_f32 vcc, v97, v50\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v97, v97, v27, vcc\n" \
    "v_cmp_lt_f32 vcc, v90, v25\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v90, v90, v27, vcc\n" \
    "SD_SKIP2_%=:\n" \
    "v_rsq_f32 v105, v95\n" \
    "v_rsq_f32 v115, v88\n" \
    "v_mul_f32 v94, v105, v105\n" \
    "v_mul_f32 v104, v115, v115\n" \
    "v_mul_f32 v107, v94, v105\n" \
    "v_mul_f32 v117, v104, v115\n" \
    "v_mul_f32 v100, v94, v111\n" \
    "v_mul_f32 v100, v100, v105\n" \
    "v_mul_f32 v102, v94, v113\n" \
    "v_mul_f32 v102, v102, v105\n" \
    "v_mul_f32 v110, v104, v121\n" \
    "v_mul_f32 v110, v110, v115\n" \
    "v_mul_f32 v112, v104, v123\n" \
    "v_mul_f32 v112, v112, v115\n" \
    "v_mul_f32 v52, v100, v71\n" \
    "v_fmac_f32 v52, v105, v76\n" \
    "v_mul_f32 v54, v100, v73\n" \
    "v_fmac_f32 v54, v105, v78\n" \
    "v_mul_f32 v56, v100, v75\n" \
    "v_fmac_f32 v56, v105, v80\n" \
    "v_mul_f32 v58, v110, v77\n" \
    "v_fmac_f32 v58, v115, v76\n" \
    "v_mul_f32 v60, v110, v79\n" \
    "v_fmac_f32 v60, v115, v78\n" \
    "v_mul_f32 v62, v110, v81\n" \
    "v_fmac_f32 v62, v115, v80\n" \
    "v_mul_f32 v114, v102, v71\n" \
    "v_fmac_f32 v114, v105, v36\n" \
    "v_mul_f32 v116, v102, v73\n" \
    "v_fmac_f32 v116, v105, v38\n" \
    "v_mul_f32 v118, v102, v75\n" \
    "v_fmac_f32 v118, v105, v40\n" \
    "v_fmac_f32 v114, v112, v77\n" \
    "v_fmac_f32 v114, v115, v42\n" \
    "v_fmac_f32 v116, v112, v79\n" \
    "v_fmac_f32 v116, v115, v44\n" \
    "v_fmac_f32 v118, v112, v81\n" \
    "v_fmac_f32 v118, v115, v46\n" \
    "v_rsq_f32 v105, v97\n" \
    "v_rsq_f32 v115, v90\n" \
    "v_mul_f32 v111, v87, v86\n" \
    "v_fmac_f32 v111, v85, v84\n" \
    "v_fmac_f32 v111, v83, v82\n" \
    "v_mov_b32_dpp v47, v114 row_ror:4 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_mov_b32_dpp v49, v116 row_ror:4 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_mov_b32_dpp v51, v118 row_ror:4 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_mul_f32 v113, v87, v40\n" \
    "v_fmac_f32 v113, v85, v38\n" \
    "v_fmac_f32 v113, v83, v36\n" \
    "v_mul_f32 v121, v93, v86\n" \
    "v_fmac_f32 v121, v91, v84\n" \
    "v_fmac_f32 v121, v89, v82\n" \
    "v_mul_f32 v123, v93, v46\n" \
    "v_fmac_f32 v123, v91, v44\n" \
    "v_fmac_f32 v123, v89, v42\n" \
    "v_mul_f32 v94, v105, v105\n" \
    "v_mul_f32 v104, v115, v115\n" \
    "v_mul_f32 v107, v94, v105\n" \
    "v_mul_f32 v117, v104, v115\n" \
    "v_mul_f32 v100, v94, v111\n" \
    "v_mul_f32 v100, v100, v105\n" \
    "v_mul_f32 v102, v94, v113\n" \
    "v_mul_f32 v102, v102, v105\n" \
    "v_mul_f32 v110, v104, v121\n" \
    "v_mul_f32 v110, v110, v115\n" \
    "v_mul_f32 v112, v104, v123\n" \
    "v_mul_f32 v112, v112, v115\n" \
    "v_fmac_f32 v52, v100, v83\n" \
    "v_fmac_f32 v52, v105, v82\n" \
    "v_fmac_f32 v54, v100, v85\n" \
    "v_fmac_f32 v54, v105, v84\n" \
    "v_fmac_f32 v56, v100, v87\n" \
    "v_fmac_f32 v56, v105, v86\n" \
    "v_fmac_f32 v58, v110, v89\n" \
    "v_fmac_f32 v58, v115, v82\n" \
    "v_fmac_f32 v60, v110, v91\n" \
    "v_fmac_f32 v60, v115, v84\n" \
    "v_fmac_f32 v62, v110, v93\n" \
    "v_fmac_f32 v62, v115, v86\n" \
    "v_mul_f32 v120, v102, v83\n" \
    "v_fmac_f32 v120, v105, v36\n" \
    "v_mul_f32 v122, v102, v85\n" \
    "v_fmac_f32 v122, v105, v38\n" \
    "v_mul_f32 v124, v102, v87\n" \
    "v_fmac_f32 v124, v105, v40\n" \
    "v_fmac_f32 v120, v112, v89\n" \
    "v_fmac_f32 v120, v115, v42\n" \
    "v_fmac_f32 v122, v112, v91\n" \
    "v_fmac_f32 v122, v115, v44\n" \
    "v_fmac_f32 v124, v112, v93\n" \
    "v_fmac_f32 v124, v115, v46\n" \
    "ds_read_b32 v59, v31 offset:24\n" \
    "ds_read_b32 v61, v31 offset:152\n" \
    "ds_read_b32 v63, v31 offset:280\n" \
    "ds_read_b32 v65, v31 offset:28\n" \
    "ds_read_b32 v67, v31 offset:156\n" \
    "ds_read_b32 v69, v31 offset:284\n" \
    "ds_read_b32 v76, v31 offset:408\n" \
    "ds_read_b32 v78, v31 offset:536\n" \
    "ds_read_b32 v80, v31 offset:664\n" \
    "ds_read_b32 v82, v31 offset:412\n" \
    "ds_read_b32 v84, v31 offset:540\n" \
    "ds_read_b32 v86, v31 offset:668\n" \
    "s_waitcnt lgkmcnt(9)\n" \
    "v_sub_u32 v101, v24, v59\n" \
    "v_cvt_f32_i32 v71, v101\n" \
    "v_sub_u32 v101, v26, v61\n" \
    "v_cvt_f32_i32 v73, v101\n" \
    "v_sub_u32 v101, v28, v63\n" \
    "v_cvt_f32_i32 v75, v101\n" \
    "v_sub_u32 v103, v30, v59\n" \
    "v_cvt_f32_i32 v77, v103\n" \
    "v_sub_u32 v103, v32, v61\n" \
    "v_cvt_f32_i32 v79, v103\n" \
    "v_sub_u32 v103, v34, v63\n" \
    "v_cvt_f32_i32 v81, v103\n" \
    "v_mul_f32 v95, v75, v75\n" \
    "v_fmac_f32 v95, v73, v73\n" \
    "v_fmac_f32 v95, v71, v71\n" \
    "v_mul_f32 v88, v81, v81\n" \
    "v_fmac_f32 v88, v79, v79\n" \
    "v_fmac_f32 v88, v77, v77\n" \
    "v_min_f32 v99, v95, v88\n" \
    "s_waitcnt lgkmcnt(6)\n" \
    "v_sub_u32 v101, v24, v65\n" \
    "v_cvt_f32_i32 v83, v101\n" \
    "v_sub_u32 v101, v26, v67\n" \
    "v_cvt_f32_i32 v85, v101\n" \
    "v_sub_u32 v101, v28, v69\n" \
    "v_cvt_f32_i32 v87, v101\n" \
    "v_sub_u32 v103, v30, v65\n" \
    "v_cvt_f32_i32 v89, v103\n" \
    "v_sub_u32 v103, v32, v67\n" \
    "v_cvt_f32_i32 v91, v103\n" \
    "v_sub_u32 v103, v34, v69\n" \
    "v_cvt_f32_i32 v93, v103\n" \
    "v_mul_f32 v97, v87, v87\n" \
    "v_fmac_f32 v97, v85, v85\n" \
    "v_fmac_f32 v97, v83, v83\n" \
    "v_mul_f32 v90, v93, v93\n" \
    "v_fmac_f32 v90, v91, v91\n" \
    "v_fmac_f32 v90, v89, v89\n" \
    "v_min_f32 v92, v97, v90\n" \
    "v_min_f32 v99, v99, v92\n" \
    "v_cmp_lt_f32 vcc, v99, v50\n" \
    "s_waitcnt lgkmcnt(0)\n" \
    "v_mul_f32 v111, v75, v80\n" \
    "v_fmac_f32 v111, v73, v78\n" \
    "v_fmac_f32 v111, v71, v76\n" \
    "v_add_f32_dpp v47, v120, v47 row_ror:5 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_add_f32_dpp v49, v122, v49 row_ror:5 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_add_f32_dpp v51, v124, v51 row_ror:5 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_mul_f32 v113, v75, v40\n" \
    "v_fmac_f32 v113, v73, v38\n" \
    "v_fmac_f32 v113, v71, v36\n" \
    "v_mul_f32 v121, v81, v80\n" \
    "v_fmac_f32 v121, v79, v78\n" \
    "v_fmac_f32 v121, v77, v76\n" \
    "v_mul_f32 v123, v81, v46\n" \
    "v_fmac_f32 v123, v79, v44\n" \
    "v_fmac_f32 v123, v77, v42\n" \
    "s_cbranch_vccz SD_SKIP3_%=\n" \
    "s_or_b64 %[nl], %[nl], vcc\n" \
    "v_cmp_lt_f32 vcc, v95, v50\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v95, v95, v27, vcc\n" \
    "v_cmp_lt_f32 vcc, v88, v25\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v88, v88, v27, vcc\n" \
    "v_cmp_lt_f32 vcc, v97, v50\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v97, v97, v27, vcc\n" \
    "v_cmp_lt_f32 vcc, v90, v25\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v90, v90, v27, vcc\n" \
    "SD_SKIP3_%=:\n" \
    "v_rsq_f32 v105, v95\n" \
    "v_rsq_f32 v115, v88\n" \
    "v_mul_f32 v94, v105, v105\n" \
    "v_mul_f32 v104, v115, v115\n" \
    "v_mul_f32 v107, v94, v105\n" \
    "v_mul_f32 v117, v104, v115\n" \
    "v_mul_f32 v100, v94, v111\n" \
    "v_mul_f32 v100, v100, v105\n" \
    "v_mul_f32 v102, v94, v113\n" \
    "v_mul_f32 v102, v102, v105\n" \
    "v_mul_f32 v110, v104, v121\n" \
    "v_mul_f32 v110, v110, v115\n" \
    "v_mul_f32 v112, v104, v123\n" \
    "v_mul_f32 v112, v112, v115\n" \
    "v_fmac_f32 v52, v100, v71\n" \
    "v_fmac_f32 v52, v105, v76\n" \
    "v_fmac_f32 v54, v100, v73\n" \
    "v_fmac_f32 v54, v105, v78\n" \
    "v_fmac_f32 v56, v100, v75\n" \
    "v_fmac_f32 v56, v105, v80\n" \
    "v_fmac_f32 v58, v110, v77\n" \
    "v_fmac_f32 v58, v115, v76\n" \
    "v_fmac_f32 v60, v110, v79\n" \
    "v_fmac_f32 v60, v115, v78\n" \
    "v_fmac_f32 v62, v110, v81\n" \
    "v_fmac_f32 v62, v115, v80\n" \
    "v_mul_f32 v114, v102, v71\n" \
    "v_fmac_f32 v114, v105, v36\n" \
    "v_mul_f32 v116, v102, v73\n" \
    "v_fmac_f32 v116, v105, v38\n" \
    "v_mul_f32 v118, v102, v75\n" \
    "v_fmac_f32 v118, v105, v40\n" \
    "v_fmac_f32 v114, v112, v77\n" \
    "v_fmac_f32 v114, v115, v42\n" \
    "v_fmac_f32 v116, v112, v79\n" \
    "v_fmac_f32 v116, v115, v44\n" \
    "v_fmac_f32 v118, v112, v81\n" \
    "v_fmac_f32 v118, v115, v46\n" \
    "v_rsq_f32 v105, v97\n" \
    "v_rsq_f32 v115, v90\n" \
    "v_mul_f32 v111, v87, v86\n" \
    "v_fmac_f32 v111, v85, v84\n" \
    "v_fmac_f32 v111, v83, v82\n" \
    "v_add_f32_dpp v47, v114, v47 row_ror:6 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_add_f32_dpp v49, v116, v49 row_ror:6 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_add_f32_dpp v51, v118, v51 row_ror:6 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_mul_f32 v113, v87, v40\n" \
    "v_fmac_f32 v113, v85, v38\n" \
    "v_fmac_f32 v113, v83, v36\n" \
    "v_mul_f32 v121, v93, v86\n" \
    "v_fmac_f32 v121, v91, v84\n" \
    "v_fmac_f32 v121, v89, v82\n" \
    "v_mul_f32 v123, v93, v46\n" \
    "v_fmac_f32 v123, v91, v44\n" \
    "v_fmac_f32 v123, v89, v42\n" \
    "v_mul_f32 v94, v105, v105\n" \
    "v_mul_f32 v104, v115, v115\n" \
    "v_mul_f32 v107, v94, v105\n" \
    "v_mul_f32 v117, v104, v115\n" \
    "v_mul_f32 v100, v94, v111\n" \
    "v_mul_f32 v100, v100, v105\n" \
    "v_mul_f32 v102, v94, v113\n" \
    "v_mul_f32 v102, v102, v105\n" \
    "v_mul_f32 v110, v104, v121\n" \
    "v_mul_f32 v110, v110, v115\n" \
    "v_mul_f32 v112, v104, v123\n" \
    "v_mul_f32 v112, v112, v115\n" \
    "v_fmac_f32 v52, v100, v83\n" \
    "v_fmac_f32 v52, v105, v82\n" \
    "v_fmac_f32 v54, v100, v85\n" \
    "v_fmac_f32 v54, v105, v84\n" \
    "v_fmac_f32 v56, v100, v87\n" \
    "v_fmac_f32 v56, v105, v86\n" \
    "v_fmac_f32 v58, v110, v89\n" \
    "v_fmac_f32 v58, v115, v82\n" \
    "v_fmac_f32 v60, v110, v91\n" \
    "v_fmac_f32 v60, v115, v84\n" \
    "v_fmac_f32 v62, v110, v93\n" \
    "v_fmac_f32 v62, v115, v86\n" \
    "v_mul_f32 v120, v102, v83\n" \
    "v_fmac_f32 v120, v105, v36\n" \
    "v_mul_f32 v122, v102, v85\n" \
    "v_fmac_f32 v122, v105, v38\n" \
    "v_mul_f32 v124, v102, v87\n" \
    "v_fmac_f32 v124, v105, v40\n" \
    "v_fmac_f32 v120, v112, v89\n" \
    "v_fmac_f32 v120, v115, v42\n" \
    "v_fmac_f32 v122, v112, v91\n" \
    "v_fmac_f32 v122, v115, v44\n" \
    "v_fmac_f32 v124, v112, v93\n" \
    "v_fmac_f32 v124, v115, v46\n" \
    "v_add_f32 v35, v35, v52\n" \
    "v_add_f32 v37, v37, v54\n" \
    "v_add_f32 v39, v39, v56\n" \
    "v_add_f32 v41, v41, v58\n" \
    "v_add_f32 v43, v43, v60\n" \
    "v_add_f32 v45, v45, v62\n" \
    "ds_read_b32 v59, v31 offset:32\n" \
    "ds_read_b32 v61, v31 offset:160\n" \
    "ds_read_b32 v63, v31 offset:288\n" \
    "ds_read_b32 v65, v31 offset:36\n" \
    "ds_read_b32 v67, v31 offset:164\n" \
    "ds_read_b32 v69, v31 offset:292\n" \
    "ds_read_b32 v76, v31 offset:416\n" \
    "ds_read_b32 v78, v31 offset:544\n" \
    "ds_read_b32 v80, v31 offset:672\n" \
    "ds_read_b32 v82, v31 offset:420\n" \
    "ds_read_b32 v84, v31 offset:548\n" \
    "ds_read_b32 v86, v31 offset:676\n" \
    "s_waitcnt lgkmcnt(9)\n" \
    "v_sub_u32 v101, v24, v59\n" \
    "v_cvt_f32_i32 v71, v101\n" \
    "v_sub_u32 v101, v26, v61\n" \
    "v_cvt_f32_i32 v73, v101\n" \
    "v_sub_u32 v101, v28, v63\n" \
    "v_cvt_f32_i32 v75, v101\n" \
    "v_sub_u32 v103, v30, v59\n" \
    "v_cvt_f32_i32 v77, v103\n" \
    "v_sub_u32 v103, v32, v61\n" \
    "v_cvt_f32_i32 v79, v103\n" \
    "v_sub_u32 v103, v34, v63\n" \
    "v_cvt_f32_i32 v81, v103\n" \
    "v_mul_f32 v95, v75, v75\n" \
    "v_fmac_f32 v95, v73, v73\n" \
    "v_fmac_f32 v95, v71, v71\n" \
    "v_mul_f32 v88, v81, v81\n" \
    "v_fmac_f32 v88, v79, v79\n" \
    "v_fmac_f32 v88, v77, v77\n" \
    "v_min_f32 v99, v95, v88\n" \
    "s_waitcnt lgkmcnt(6)\n" \
    "v_sub_u32 v101, v24, v65\n" \
    "v_cvt_f32_i32 v83, v101\n" \
    "v_sub_u32 v101, v26, v67\n" \
    "v_cvt_f32_i32 v85, v101\n" \
    "v_sub_u32 v101, v28, v69\n" \
    "v_cvt_f32_i32 v87, v101\n" \
    "v_sub_u32 v103, v30, v65\n" \
    "v_cvt_f32_i32 v89, v103\n" \
    "v_sub_u32 v103, v32, v67\n" \
    "v_cvt_f32_i32 v91, v103\n" \
    "v_sub_u32 v103, v34, v69\n" \
    "v_cvt_f32_i32 v93, v103\n" \
    "v_mul_f32 v97, v87, v87\n" \
    "v_fmac_f32 v97, v85, v85\n" \
    "v_fmac_f32 v97, v83, v83\n" \
    "v_mul_f32 v90, v93, v93\n" \
    "v_fmac_f32 v90, v91, v91\n" \
    "v_fmac_f32 v90, v89, v89\n" \
    "v_min_f32 v92, v97, v90\n" \
    "v_min_f32 v99, v99, v92\n" \
    "v_cmp_lt_f32 vcc, v99, v50\n" \
    "s_waitcnt lgkmcnt(0)\n" \
    "v_mul_f32 v111, v75, v80\n" \
    "v_fmac_f32 v111, v73, v78\n" \
    "v_fmac_f32 v111, v71, v76\n" \
    "v_add_f32_dpp v47, v120, v47 row_ror:7 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_add_f32_dpp v49, v122, v49 row_ror:7 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_add_f32_dpp v51, v124, v51 row_ror:7 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_mul_f32 v113, v75, v40\n" \
    "v_fmac_f32 v113, v73, v38\n" \
    "v_fmac_f32 v113, v71, v36\n" \
    "v_mul_f32 v121, v81, v80\n" \
    "v_fmac_f32 v121, v79, v78\n" \
    "v_fmac_f32 v121, v77, v76\n" \
    "v_mul_f32 v123, v81, v46\n" \
    "v_fmac_f32 v123, v79, v44\n" \
    "v_fmac_f32 v123, v77, v42\n" \
    "v_add_f32 v53, v53, v47\n" \
    "v_add_f32 v55, v55, v49\n" \
    "v_add_f32 v57, v57, v51\n" \
    "ds_write_b32 v33, v53 offset:0\n" \
    "ds_write_b32 v33, v55 offset:64\n" \
    "ds_write_b32 v33, v57 offset:128\n" \
    "s_cbranch_vccz SD_SKIP4_%=\n" \
    "s_or_b64 %[nl], %[nl], vcc\n" \
    "v_cmp_lt_f32 vcc, v95, v50\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v95, v95, v27, vcc\n" \
    "v_cmp_lt_f32 vcc, v88, v25\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v88, v88, v27, vcc\n" \
    "v_cmp_lt_f32 vcc, v97, v50\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v97, v97, v27, vcc\n" \
    "v_cmp_lt_f32 vcc, v90, v25\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v90, v90, v27, vcc\n" \
    "SD_SKIP4_%=:\n" \
    "v_rsq_f32 v105, v95\n" \
    "v_rsq_f32 v115, v88\n" \
    "v_mul_f32 v94, v105, v105\n" \
    "v_mul_f32 v104, v115, v115\n" \
    "v_mul_f32 v107, v94, v105\n" \
    "v_mul_f32 v117, v104, v115\n" \
    "v_mul_f32 v100, v94, v111\n" \
    "v_mul_f32 v100, v100, v105\n" \
    "v_mul_f32 v102, v94, v113\n" \
    "v_mul_f32 v102, v102, v105\n" \
    "v_mul_f32 v110, v104, v121\n" \
    "v_mul_f32 v110, v110, v115\n" \
    "v_mul_f32 v112, v104, v123\n" \
    "v_mul_f32 v112, v112, v115\n" \
    "v_mul_f32 v52, v100, v71\n" \
    "v_fmac_f32 v52, v105, v76\n" \
    "v_mul_f32 v54, v100, v73\n" \
    "v_fmac_f32 v54, v105, v78\n" \
    "v_mul_f32 v56, v100, v75\n" \
    "v_fmac_f32 v56, v105, v80\n" \
    "v_mul_f32 v58, v110, v77\n" \
    "v_fmac_f32 v58, v115, v76\n" \
    "v_mul_f32 v60, v110, v79\n" \
    "v_fmac_f32 v60, v115, v78\n" \
    "v_mul_f32 v62, v110, v81\n" \
    "v_fmac_f32 v62, v115, v80\n" \
    "v_mul_f32 v114, v102, v71\n" \
    "v_fmac_f32 v114, v105, v36\n" \
    "v_mul_f32 v116, v102, v73\n" \
    "v_fmac_f32 v116, v105, v38\n" \
    "v_mul_f32 v118, v102, v75\n" \
    "v_fmac_f32 v118, v105, v40\n" \
    "v_fmac_f32 v114, v112, v77\n" \
    "v_fmac_f32 v114, v115, v42\n" \
    "v_fmac_f32 v116, v112, v79\n" \
    "v_fmac_f32 v116, v115, v44\n" \
    "v_fmac_f32 v118, v112, v81\n" \
    "v_fmac_f32 v118, v115, v46\n" \
    "v_rsq_f32 v105, v97\n" \
    "v_rsq_f32 v115, v90\n" \
    "v_mul_f32 v111, v87, v86\n" \
    "v_fmac_f32 v111, v85, v84\n" \
    "v_fmac_f32 v111, v83, v82\n" \
    "v_mov_b32_dpp v53, v114 row_ror:8 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_mov_b32_dpp v55, v116 row_ror:8 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_mov_b32_dpp v57, v118 row_ror:8 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_mul_f32 v113, v87, v40\n" \
    "v_fmac_f32 v113, v85, v38\n" \
    "v_fmac_f32 v113, v83, v36\n" \
    "v_mul_f32 v121, v93, v86\n" \
    "v_fmac_f32 v121, v91, v84\n" \
    "v_fmac_f32 v121, v89, v82\n" \
    "v_mul_f32 v123, v93, v46\n" \
    "v_fmac_f32 v123, v91, v44\n" \
    "v_fmac_f32 v123, v89, v42\n" \
    "v_mul_f32 v94, v105, v105\n" \
    "v_mul_f32 v104, v115, v115\n" \
    "v_mul_f32 v107, v94, v105\n" \
    "v_mul_f32 v117, v104, v115\n" \
    "v_mul_f32 v100, v94, v111\n" \
    "v_mul_f32 v100, v100, v105\n" \
    "v_mul_f32 v102, v94, v113\n" \
    "v_mul_f32 v102, v102, v105\n" \
    "v_mul_f32 v110, v104, v121\n" \
    "v_mul_f32 v110, v110, v115\n" \
    "v_mul_f32 v112, v104, v123\n" \
    "v_mul_f32 v112, v112, v115\n" \
    "v_fmac_f32 v52, v100, v83\n" \
    "v_fmac_f32 v52, v105, v82\n" \
    "v_fmac_f32 v54, v100, v85\n" \
    "v_fmac_f32 v54, v105, v84\n" \
    "v_fmac_f32 v56, v100, v87\n" \
    "v_fmac_f32 v56, v105, v86\n" \
    "v_fmac_f32 v58, v110, v89\n" \
    "v_fmac_f32 v58, v115, v82\n" \
    "v_fmac_f32 v60, v110, v91\n" \
    "v_fmac_f32 v60, v115, v84\n" \
    "v_fmac_f32 v62, v110, v93\n" \
    "v_fmac_f32 v62, v115, v86\n" \
    "v_mul_f32 v120, v102, v83\n" \
    "v_fmac_f32 v120, v105, v36\n" \
    "v_mul_f32 v122, v102, v85\n" \
    "v_fmac_f32 v122, v105, v38\n" \
    "v_mul_f32 v124, v102, v87\n" \
    "v_fmac_f32 v124, v105, v40\n" \
    "v_fmac_f32 v120, v112, v89\n" \
    "v_fmac_f32 v120, v115, v42\n" \
    "v_fmac_f32 v122, v112, v91\n" \
    "v_fmac_f32 v122, v115, v44\n" \
    "v_fmac_f32 v124, v112, v93\n" \
    "v_fmac_f32 v124, v115, v46\n" \
    "ds_read_b32 v59, v31 offset:40\n" \
    "ds_read_b32 v61, v31 offset:168\n" \
    "ds_read_b32 v63, v31 offset:296\n" \
    "ds_read_b32 v65, v31 offset:44\n" \
    "ds_read_b32 v67, v31 offset:172\n" \
    "ds_read_b32 v69, v31 offset:300\n" \
    "ds_read_b32 v76, v31 offset:424\n" \
    "ds_read_b32 v78, v31 offset:552\n" \
    "ds_read_b32 v80, v31 offset:680\n" \
    "ds_read_b32 v82, v31 offset:428\n" \
    "ds_read_b32 v84, v31 offset:556\n" \
    "ds_read_b32 v86, v31 offset:684\n" \
    "s_waitcnt lgkmcnt(9)\n" \
    "v_sub_u32 v101, v24, v59\n" \
    "v_cvt_f32_i32 v71, v101\n" \
    "v_sub_u32 v101, v26, v61\n" \
    "v_cvt_f32_i32 v73, v101\n" \
    "v_sub_u32 v101, v28, v63\n" \
    "v_cvt_f32_i32 v75, v101\n" \
    "v_sub_u32 v103, v30, v59\n" \
    "v_cvt_f32_i32 v77, v103\n" \
    "v_sub_u32 v103, v32, v61\n" \
    "v_cvt_f32_i32 v79, v103\n" \
    "v_sub_u32 v103, v34, v63\n" \
    "v_cvt_f32_i32 v81, v103\n" \
    "v_mul_f32 v95, v75, v75\n" \
    "v_fmac_f32 v95, v73, v73\n" \
    "v_fmac_f32 v95, v71, v71\n" \
    "v_mul_f32 v88, v81, v81\n" \
    "v_fmac_f32 v88, v79, v79\n" \
    "v_fmac_f32 v88, v77, v77\n" \
    "v_min_f32 v99, v95, v88\n" \
    "s_waitcnt lgkmcnt(6)\n" \
    "v_sub_u32 v101, v24, v65\n" \
    "v_cvt_f32_i32 v83, v101\n" \
    "v_sub_u32 v101, v26, v67\n" \
    "v_cvt_f32_i32 v85, v101\n" \
    "v_sub_u32 v101, v28, v69\n" \
    "v_cvt_f32_i32 v87, v101\n" \
    "v_sub_u32 v103, v30, v65\n" \
    "v_cvt_f32_i32 v89, v103\n" \
    "v_sub_u32 v103, v32, v67\n" \
    "v_cvt_f32_i32 v91, v103\n" \
    "v_sub_u32 v103, v34, v69\n" \
    "v_cvt_f32_i32 v93, v103\n" \
    "v_mul_f32 v97, v87, v87\n" \
    "v_fmac_f32 v97, v85, v85\n" \
    "v_fmac_f32 v97, v83, v83\n" \
    "v_mul_f32 v90, v93, v93\n" \
    "v_fmac_f32 v90, v91, v91\n" \
    "v_fmac_f32 v90, v89, v89\n" \
    "v_min_f32 v92, v97, v90\n" \
    "v_min_f32 v99, v99, v92\n" \
    "v_cmp_lt_f32 vcc, v99, v50\n" \
    "s_waitcnt lgkmcnt(0)\n" \
    "v_mul_f32 v111, v75, v80\n" \
    "v_fmac_f32 v111, v73, v78\n" \
    "v_fmac_f32 v111, v71, v76\n" \
    "v_add_f32_dpp v53, v120, v53 row_ror:9 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_add_f32_dpp v55, v122, v55 row_ror:9 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_add_f32_dpp v57, v124, v57 row_ror:9 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_mul_f32 v113, v75, v40\n" \
    "v_fmac_f32 v113, v73, v38\n" \
    "v_fmac_f32 v113, v71, v36\n" \
    "v_mul_f32 v121, v81, v80\n" \
    "v_fmac_f32 v121, v79, v78\n" \
    "v_fmac_f32 v121, v77, v76\n" \
    "v_mul_f32 v123, v81, v46\n" \
    "v_fmac_f32 v123, v79, v44\n" \
    "v_fmac_f32 v123, v77, v42\n" \
    "s_cbranch_vccz SD_SKIP5_%=\n" \
    "s_or_b64 %[nl], %[nl], vcc\n" \
    "v_cmp_lt_f32 vcc, v95, v50\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v95, v95, v27, vcc\n" \
    "v_cmp_lt_f32 vcc, v88, v25\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v88, v88, v27, vcc\n" \
    "v_cmp_lt_f32 vcc, v97, v50\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v97, v97, v27, vcc\n" \
    "v_cmp_lt_f32 vcc, v90, v25\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v90, v90, v27, vcc\n" \
    "SD_SKIP5_%=:\n" \
    "v_rsq_f32 v105, v95\n" \
    "v_rsq_f32 v115, v88\n" \
    "v_mul_f32 v94, v105, v105\n" \
    "v_mul_f32 v104, v115, v115\n" \
    "v_mul_f32 v107, v94, v105\n" \
    "v_mul_f32 v117, v104, v115\n" \
    "v_mul_f32 v100, v94, v111\n" \
    "v_mul_f32 v100, v100, v105\n" \
    "v_mul_f32 v102, v94, v113\n" \
    "v_mul_f32 v102, v102, v105\n" \
    "v_mul_f32 v110, v104, v121\n" \
    "v_mul_f32 v110, v110, v115\n" \
    "v_mul_f32 v112, v104, v123\n" \
    "v_mul_f32 v112, v112, v115\n" \
    "v_fmac_f32 v52, v100, v71\n" \
    "v_fmac_f32 v52, v105, v76\n" \
    "v_fmac_f32 v54, v100, v73\n" \
    "v_fmac_f32 v54, v105, v78\n" \
    "v_fmac_f32 v56, v100, v75\n" \
    "v_fmac_f32 v56, v105, v80\n" \
    "v_fmac_f32 v58, v110, v77\n" \
    "v_fmac_f32 v58, v115, v76\n" \
    "v_fmac_f32 v60, v110, v79\n" \
    "v_fmac_f32 v60, v115, v78\n" \
    "v_fmac_f32 v62, v110, v81\n" \
    "v_fmac_f32 v62, v115, v80\n" \
    "v_mul_f32 v114, v102, v71\n" \
    "v_fmac_f32 v114, v105, v36\n" \
    "v_mul_f32 v116, v102, v73\n" \
    "v_fmac_f32 v116, v105, v38\n" \
    "v_mul_f32 v118, v102, v75\n" \
    "v_fmac_f32 v118, v105, v40\n" \
    "v_fmac_f32 v114, v112, v77\n" \
    "v_fmac_f32 v114, v115, v42\n" \
    "v_fmac_f32 v116, v112, v79\n" \
    "v_fmac_f32 v116, v115, v44\n" \
    "v_fmac_f32 v118, v112, v81\n" \
    "v_fmac_f32 v118, v115, v46\n" \
    "v_rsq_f32 v105, v97\n" \
    "v_rsq_f32 v115, v90\n" \
    "v_mul_f32 v111, v87, v86\n" \
    "v_fmac_f32 v111, v85, v84\n" \
    "v_fmac_f32 v111, v83, v82\n" \
    "v_add_f32_dpp v53, v114, v53 row_ror:10 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_add_f32_dpp v55, v116, v55 row_ror:10 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_add_f32_dpp v57, v118, v57 row_ror:10 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_mul_f32 v113, v87, v40\n" \
    "v_fmac_f32 v113, v85, v38\n" \
    "v_fmac_f32 v113, v83, v36\n" \
    "v_mul_f32 v121, v93, v86\n" \
    "v_fmac_f32 v121, v91, v84\n" \
    "v_fmac_f32 v121, v89, v82\n" \
    "v_mul_f32 v123, v93, v46\n" \
    "v_fmac_f32 v123, v91, v44\n" \
    "v_fmac_f32 v123, v89, v42\n" \
    "v_mul_f32 v94, v105, v105\n" \
    "v_mul_f32 v104, v115, v115\n" \
    "v_mul_f32 v107, v94, v105\n" \
    "v_mul_f32 v117, v104, v115\n" \
    "v_mul_f32 v100, v94, v111\n" \
    "v_mul_f32 v100, v100, v105\n" \
    "v_mul_f32 v102, v94, v113\n" \
    "v_mul_f32 v102, v102, v105\n" \
    "v_mul_f32 v110, v104, v121\n" \
    "v_mul_f32 v110, v110, v115\n" \
    "v_mul_f32 v112, v104, v123\n" \
    "v_mul_f32 v112, v112, v115\n" \
    "v_fmac_f32 v52, v100, v83\n" \
    "v_fmac_f32 v52, v105, v82\n" \
    "v_fmac_f32 v54, v100, v85\n" \
    "v_fmac_f32 v54, v105, v84\n" \
    "v_fmac_f32 v56, v100, v87\n" \
    "v_fmac_f32 v56, v105, v86\n" \
    "v_fmac_f32 v58, v110, v89\n" \
    "v_fmac_f32 v58, v115, v82\n" \
    "v_fmac_f32 v60, v110, v91\n" \
    "v_fmac_f32 v60, v115, v84\n" \
    "v_fmac_f32 v62, v110, v93\n" \
    "v_fmac_f32 v62, v115, v86\n" \
    "v_mul_f32 v120, v102, v83\n" \
    "v_fmac_f32 v120, v105, v36\n" \
    "v_mul_f32 v122, v102, v85\n" \
    "v_fmac_f32 v122, v105, v38\n" \
    "v_mul_f32 v124, v102, v87\n" \
    "v_fmac_f32 v124, v105, v40\n" \
    "v_fmac_f32 v120, v112, v89\n" \
    "v_fmac_f32 v120, v115, v42\n" \
    "v_fmac_f32 v122, v112, v91\n" \
    "v_fmac_f32 v122, v115, v44\n" \
    "v_fmac_f32 v124, v112, v93\n" \
    "v_fmac_f32 v124, v115, v46\n" \
    "v_add_f32 v35, v35, v52\n" \
    "v_add_f32 v37, v37, v54\n" \
    "v_add_f32 v39, v39, v56\n" \
    "v_add_f32 v41, v41, v58\n" \
    "v_add_f32 v43, v43, v60\n" \
    "v_add_f32 v45, v45, v62\n" \
    "ds_read_b32 v59, v31 offset:48\n" \
    "ds_read_b32 v61, v31 offset:176\n" \
    "ds_read_b32 v63, v31 offset:304\n" \
    "ds_read_b32 v65, v31 offset:52\n" \
    "ds_read_b32 v67, v31 offset:180\n" \
    "ds_read_b32 v69, v31 offset:308\n" \
    "ds_read_b32 v76, v31 offset:432\n" \
    "ds_read_b32 v78, v31 offset:560\n" \
    "ds_read_b32 v80, v31 offset:688\n" \
    "ds_read_b32 v82, v31 offset:436\n" \
    "ds_read_b32 v84, v31 offset:564\n" \
    "ds_read_b32 v86, v31 offset:692\n" \
    "s_waitcnt lgkmcnt(9)\n" \
    "v_sub_u32 v101, v24, v59\n" \
    "v_cvt_f32_i32 v71, v101\n" \
    "v_sub_u32 v101, v26, v61\n" \
    "v_cvt_f32_i32 v73, v101\n" \
    "v_sub_u32 v101, v28, v63\n" \
    "v_cvt_f32_i32 v75, v101\n" \
    "v_sub_u32 v103, v30, v59\n" \
    "v_cvt_f32_i32 v77, v103\n" \
    "v_sub_u32 v103, v32, v61\n" \
    "v_cvt_f32_i32 v79, v103\n" \
    "v_sub_u32 v103, v34, v63\n" \
    "v_cvt_f32_i32 v81, v103\n" \
    "v_mul_f32 v95, v75, v75\n" \
    "v_fmac_f32 v95, v73, v73\n" \
    "v_fmac_f32 v95, v71, v71\n" \
    "v_mul_f32 v88, v81, v81\n" \
    "v_fmac_f32 v88, v79, v79\n" \
    "v_fmac_f32 v88, v77, v77\n" \
    "v_min_f32 v99, v95, v88\n" \
    "s_waitcnt lgkmcnt(6)\n" \
    "v_sub_u32 v101, v24, v65\n" \
    "v_cvt_f32_i32 v83, v101\n" \
    "v_sub_u32 v101, v26, v67\n" \
    "v_cvt_f32_i32 v85, v101\n" \
    "v_sub_u32 v101, v28, v69\n" \
    "v_cvt_f32_i32 v87, v101\n" \
    "v_sub_u32 v103, v30, v65\n" \
    "v_cvt_f32_i32 v89, v103\n" \
    "v_sub_u32 v103, v32, v67\n" \
    "v_cvt_f32_i32 v91, v103\n" \
    "v_sub_u32 v103, v34, v69\n" \
    "v_cvt_f32_i32 v93, v103\n" \
    "v_mul_f32 v97, v87, v87\n" \
    "v_fmac_f32 v97, v85, v85\n" \
    "v_fmac_f32 v97, v83, v83\n" \
    "v_mul_f32 v90, v93, v93\n" \
    "v_fmac_f32 v90, v91, v91\n" \
    "v_fmac_f32 v90, v89, v89\n" \
    "v_min_f32 v92, v97, v90\n" \
    "v_min_f32 v99, v99, v92\n" \
    "v_cmp_lt_f32 vcc, v99, v50\n" \
    "s_waitcnt lgkmcnt(0)\n" \
    "v_mul_f32 v111, v75, v80\n" \
    "v_fmac_f32 v111, v73, v78\n" \
    "v_fmac_f32 v111, v71, v76\n" \
    "v_add_f32_dpp v53, v120, v53 row_ror:11 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_add_f32_dpp v55, v122, v55 row_ror:11 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_add_f32_dpp v57, v124, v57 row_ror:11 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_mul_f32 v113, v75, v40\n" \
    "v_fmac_f32 v113, v73, v38\n" \
    "v_fmac_f32 v113, v71, v36\n" \
    "v_mul_f32 v121, v81, v80\n" \
    "v_fmac_f32 v121, v79, v78\n" \
    "v_fmac_f32 v121, v77, v76\n" \
    "v_mul_f32 v123, v81, v46\n" \
    "v_fmac_f32 v123, v79, v44\n" \
    "v_fmac_f32 v123, v77, v42\n" \
    "s_cbranch_vccz SD_SKIP6_%=\n" \
    "s_or_b64 %[nl], %[nl], vcc\n" \
    "v_cmp_lt_f32 vcc, v95, v50\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v95, v95, v27, vcc\n" \
    "v_cmp_lt_f32 vcc, v88, v25\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v88, v88, v27, vcc\n" \
    "v_cmp_lt_f32 vcc, v97, v50\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v97, v97, v27, vcc\n" \
    "v_cmp_lt_f32 vcc, v90, v25\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v90, v90, v27, vcc\n" \
    "SD_SKIP6_%=:\n" \
    "v_rsq_f32 v105, v95\n" \
    "v_rsq_f32 v115, v88\n" \
    "v_mul_f32 v94, v105, v105\n" \
    "v_mul_f32 v104, v115, v115\n" \
    "v_mul_f32 v107, v94, v105\n" \
    "v_mul_f32 v117, v104, v115\n" \
    "v_mul_f32 v100, v94, v111\n" \
    "v_mul_f32 v100, v100, v105\n" \
    "v_mul_f32 v102, v94, v113\n" \
    "v_mul_f32 v102, v102, v105\n" \
    "v_mul_f32 v110, v104, v121\n" \
    "v_mul_f32 v110, v110, v115\n" \
    "v_mul_f32 v112, v104, v123\n" \
    "v_mul_f32 v112, v112, v115\n" \
    "v_mul_f32 v52, v100, v71\n" \
    "v_fmac_f32 v52, v105, v76\n" \
    "v_mul_f32 v54, v100, v73\n" \
    "v_fmac_f32 v54, v105, v78\n" \
    "v_mul_f32 v56, v100, v75\n" \
    "v_fmac_f32 v56, v105, v80\n" \
    "v_mul_f32 v58, v110, v77\n" \
    "v_fmac_f32 v58, v115, v76\n" \
    "v_mul_f32 v60, v110, v79\n" \
    "v_fmac_f32 v60, v115, v78\n" \
    "v_mul_f32 v62, v110, v81\n" \
    "v_fmac_f32 v62, v115, v80\n" \
    "v_mul_f32 v114, v102, v71\n" \
    "v_fmac_f32 v114, v105, v36\n" \
    "v_mul_f32 v116, v102, v73\n" \
    "v_fmac_f32 v116, v105, v38\n" \
    "v_mul_f32 v118, v102, v75\n" \
    "v_fmac_f32 v118, v105, v40\n" \
    "v_fmac_f32 v114, v112, v77\n" \
    "v_fmac_f32 v114, v115, v42\n" \
    "v_fmac_f32 v116, v112, v79\n" \
    "v_fmac_f32 v116, v115, v44\n" \
    "v_fmac_f32 v118, v112, v81\n" \
    "v_fmac_f32 v118, v115, v46\n" \
    "v_rsq_f32 v105, v97\n" \
    "v_rsq_f32 v115, v90\n" \
    "v_mul_f32 v111, v87, v86\n" \
    "v_fmac_f32 v111, v85, v84\n" \
    "v_fmac_f32 v111, v83, v82\n" \
    "v_mov_b32_dpp v47, v114 row_ror:12 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_mov_b32_dpp v49, v116 row_ror:12 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_mov_b32_dpp v51, v118 row_ror:12 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_mul_f32 v113, v87, v40\n" \
    "v_fmac_f32 v113, v85, v38\n" \
    "v_fmac_f32 v113, v83, v36\n" \
    "v_mul_f32 v121, v93, v86\n" \
    "v_fmac_f32 v121, v91, v84\n" \
    "v_fmac_f32 v121, v89, v82\n" \
    "v_mul_f32 v123, v93, v46\n" \
    "v_fmac_f32 v123, v91, v44\n" \
    "v_fmac_f32 v123, v89, v42\n" \
    "v_mul_f32 v94, v105, v105\n" \
    "v_mul_f32 v104, v115, v115\n" \
    "v_mul_f32 v107, v94, v105\n" \
    "v_mul_f32 v117, v104, v115\n" \
    "v_mul_f32 v100, v94, v111\n" \
    "v_mul_f32 v100, v100, v105\n" \
    "v_mul_f32 v102, v94, v113\n" \
    "v_mul_f32 v102, v102, v105\n" \
    "v_mul_f32 v110, v104, v121\n" \
    "v_mul_f32 v110, v110, v115\n" \
    "v_mul_f32 v112, v104, v123\n" \
    "v_mul_f32 v112, v112, v115\n" \
    "v_fmac_f32 v52, v100, v83\n" \
    "v_fmac_f32 v52, v105, v82\n" \
    "v_fmac_f32 v54, v100, v85\n" \
    "v_fmac_f32 v54, v105, v84\n" \
    "v_fmac_f32 v56, v100, v87\n" \
    "v_fmac_f32 v56, v105, v86\n" \
    "v_fmac_f32 v58, v110, v89\n" \
    "v_fmac_f32 v58, v115, v82\n" \
    "v_fmac_f32 v60, v110, v91\n" \
    "v_fmac_f32 v60, v115, v84\n" \
    "v_fmac_f32 v62, v110, v93\n" \
    "v_fmac_f32 v62, v115, v86\n" \
    "v_mul_f32 v120, v102, v83\n" \
    "v_fmac_f32 v120, v105, v36\n" \
    "v_mul_f32 v122, v102, v85\n" \
    "v_fmac_f32 v122, v105, v38\n" \
    "v_mul_f32 v124, v102, v87\n" \
    "v_fmac_f32 v124, v105, v40\n" \
    "v_fmac_f32 v120, v112, v89\n" \
    "v_fmac_f32 v120, v115, v42\n" \
    "v_fmac_f32 v122, v112, v91\n" \
    "v_fmac_f32 v122, v115, v44\n" \
    "v_fmac_f32 v124, v112, v93\n" \
    "v_fmac_f32 v124, v115, v46\n" \
    "ds_read_b32 v59, v31 offset:56\n" \
    "ds_read_b32 v61, v31 offset:184\n" \
    "ds_read_b32 v63, v31 offset:312\n" \
    "ds_read_b32 v65, v31 offset:60\n" \
    "ds_read_b32 v67, v31 offset:188\n" \
    "ds_read_b32 v69, v31 offset:316\n" \
    "ds_read_b32 v76, v31 offset:440\n" \
    "ds_read_b32 v78, v31 offset:568\n" \
    "ds_read_b32 v80, v31 offset:696\n" \
    "ds_read_b32 v82, v31 offset:444\n" \
    "ds_read_b32 v84, v31 offset:572\n" \
    "ds_read_b32 v86, v31 offset:700\n" \
    "s_waitcnt lgkmcnt(9)\n" \
    "v_sub_u32 v101, v24, v59\n" \
    "v_cvt_f32_i32 v71, v101\n" \
    "v_sub_u32 v101, v26, v61\n" \
    "v_cvt_f32_i32 v73, v101\n" \
    "v_sub_u32 v101, v28, v63\n" \
    "v_cvt_f32_i32 v75, v101\n" \
    "v_sub_u32 v103, v30, v59\n" \
    "v_cvt_f32_i32 v77, v103\n" \
    "v_sub_u32 v103, v32, v61\n" \
    "v_cvt_f32_i32 v79, v103\n" \
    "v_sub_u32 v103, v34, v63\n" \
    "v_cvt_f32_i32 v81, v103\n" \
    "v_mul_f32 v95, v75, v75\n" \
    "v_fmac_f32 v95, v73, v73\n" \
    "v_fmac_f32 v95, v71, v71\n" \
    "v_mul_f32 v88, v81, v81\n" \
    "v_fmac_f32 v88, v79, v79\n" \
    "v_fmac_f32 v88, v77, v77\n" \
    "v_min_f32 v99, v95, v88\n" \
    "s_waitcnt lgkmcnt(6)\n" \
    "v_sub_u32 v101, v24, v65\n" \
    "v_cvt_f32_i32 v83, v101\n" \
    "v_sub_u32 v101, v26, v67\n" \
    "v_cvt_f32_i32 v85, v101\n" \
    "v_sub_u32 v101, v28, v69\n" \
    "v_cvt_f32_i32 v87, v101\n" \
    "v_sub_u32 v103, v30, v65\n" \
    "v_cvt_f32_i32 v89, v103\n" \
    "v_sub_u32 v103, v32, v67\n" \
    "v_cvt_f32_i32 v91, v103\n" \
    "v_sub_u32 v103, v34, v69\n" \
    "v_cvt_f32_i32 v93, v103\n" \
    "v_mul_f32 v97, v87, v87\n" \
    "v_fmac_f32 v97, v85, v85\n" \
    "v_fmac_f32 v97, v83, v83\n" \
    "v_mul_f32 v90, v93, v93\n" \
    "v_fmac_f32 v90, v91, v91\n" \
    "v_fmac_f32 v90, v89, v89\n" \
    "v_min_f32 v92, v97, v90\n" \
    "v_min_f32 v99, v99, v92\n" \
    "v_cmp_lt_f32 vcc, v99, v50\n" \
    "s_waitcnt lgkmcnt(0)\n" \
    "v_mul_f32 v111, v75, v80\n" \
    "v_fmac_f32 v111, v73, v78\n" \
    "v_fmac_f32 v111, v71, v76\n" \
    "v_add_f32_dpp v47, v120, v47 row_ror:13 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_add_f32_dpp v49, v122, v49 row_ror:13 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_add_f32_dpp v51, v124, v51 row_ror:13 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_mul_f32 v113, v75, v40\n" \
    "v_fmac_f32 v113, v73, v38\n" \
    "v_fmac_f32 v113, v71, v36\n" \
    "v_mul_f32 v121, v81, v80\n" \
    "v_fmac_f32 v121, v79, v78\n" \
    "v_fmac_f32 v121, v77, v76\n" \
    "v_mul_f32 v123, v81, v46\n" \
    "v_fmac_f32 v123, v79, v44\n" \
    "v_fmac_f32 v123, v77, v42\n" \
    "s_cbranch_vccz SD_SKIP7_%=\n" \
    "s_or_b64 %[nl], %[nl], vcc\n" \
    "v_cmp_lt_f32 vcc, v95, v50\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v95, v95, v27, vcc\n" \
    "v_cmp_lt_f32 vcc, v88, v25\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v88, v88, v27, vcc\n" \
    "v_cmp_lt_f32 vcc, v97, v50\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v97, v97, v27, vcc\n" \
    "v_cmp_lt_f32 vcc, v90, v25\n" \
    "s_nop 1\n" \
    "v_cndmask_b32 v90, v90, v27, vcc\n" \
    "SD_SKIP7_%=:\n" \
    "v_rsq_f32 v105, v95\n" \
    "v_rsq_f32 v115, v88\n" \
    "v_mul_f32 v94, v105, v105\n" \
    "v_mul_f32 v104, v115, v115\n" \
    "v_mul_f32 v107, v94, v105\n" \
    "v_mul_f32 v117, v104, v115\n" \
    "v_mul_f32 v100, v94, v111\n" \
    "v_mul_f32 v100, v100, v105\n" \
    "v_mul_f32 v102, v94, v113\n" \
    "v_mul_f32 v102, v102, v105\n" \
    "v_mul_f32 v110, v104, v121\n" \
    "v_mul_f32 v110, v110, v115\n" \
    "v_mul_f32 v112, v104, v123\n" \
    "v_mul_f32 v112, v112, v115\n" \
    "v_fmac_f32 v52, v100, v71\n" \
    "v_fmac_f32 v52, v105, v76\n" \
    "v_fmac_f32 v54, v100, v73\n" \
    "v_fmac_f32 v54, v105, v78\n" \
    "v_fmac_f32 v56, v100, v75\n" \
    "v_fmac_f32 v56, v105, v80\n" \
    "v_fmac_f32 v58, v110, v77\n" \
    "v_fmac_f32 v58, v115, v76\n" \
    "v_fmac_f32 v60, v110, v79\n" \
    "v_fmac_f32 v60, v115, v78\n" \
    "v_fmac_f32 v62, v110, v81\n" \
    "v_fmac_f32 v62, v115, v80\n" \
    "v_mul_f32 v114, v102, v71\n" \
    "v_fmac_f32 v114, v105, v36\n" \
    "v_mul_f32 v116, v102, v73\n" \
    "v_fmac_f32 v116, v105, v38\n" \
    "v_mul_f32 v118, v102, v75\n" \
    "v_fmac_f32 v118, v105, v40\n" \
    "v_fmac_f32 v114, v112, v77\n" \
    "v_fmac_f32 v114, v115, v42\n" \
    "v_fmac_f32 v116, v112, v79\n" \
    "v_fmac_f32 v116, v115, v44\n" \
    "v_fmac_f32 v118, v112, v81\n" \
    "v_fmac_f32 v118, v115, v46\n" \
    "v_rsq_f32 v105, v97\n" \
    "v_rsq_f32 v115, v90\n" \
    "v_mul_f32 v111, v87, v86\n" \
    "v_fmac_f32 v111, v85, v84\n" \
    "v_fmac_f32 v111, v83, v82\n" \
    "v_add_f32_dpp v47, v114, v47 row_ror:14 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_add_f32_dpp v49, v116, v49 row_ror:14 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_add_f32_dpp v51, v118, v51 row_ror:14 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_mul_f32 v113, v87, v40\n" \
    "v_fmac_f32 v113, v85, v38\n" \
    "v_fmac_f32 v113, v83, v36\n" \
    "v_mul_f32 v121, v93, v86\n" \
    "v_fmac_f32 v121, v91, v84\n" \
    "v_fmac_f32 v121, v89, v82\n" \
    "v_mul_f32 v123, v93, v46\n" \
    "v_fmac_f32 v123, v91, v44\n" \
    "v_fmac_f32 v123, v89, v42\n" \
    "v_mul_f32 v94, v105, v105\n" \
    "v_mul_f32 v104, v115, v115\n" \
    "v_mul_f32 v107, v94, v105\n" \
    "v_mul_f32 v117, v104, v115\n" \
    "v_mul_f32 v100, v94, v111\n" \
    "v_mul_f32 v100, v100, v105\n" \
    "v_mul_f32 v102, v94, v113\n" \
    "v_mul_f32 v102, v102, v105\n" \
    "v_mul_f32 v110, v104, v121\n" \
    "v_mul_f32 v110, v110, v115\n" \
    "v_mul_f32 v112, v104, v123\n" \
    "v_mul_f32 v112, v112, v115\n" \
    "v_fmac_f32 v52, v100, v83\n" \
    "v_fmac_f32 v52, v105, v82\n" \
    "v_fmac_f32 v54, v100, v85\n" \
    "v_fmac_f32 v54, v105, v84\n" \
    "v_fmac_f32 v56, v100, v87\n" \
    "v_fmac_f32 v56, v105, v86\n" \
    "v_fmac_f32 v58, v110, v89\n" \
    "v_fmac_f32 v58, v115, v82\n" \
    "v_fmac_f32 v60, v110, v91\n" \
    "v_fmac_f32 v60, v115, v84\n" \
    "v_fmac_f32 v62, v110, v93\n" \
    "v_fmac_f32 v62, v115, v86\n" \
    "v_mul_f32 v120, v102, v83\n" \
    "v_fmac_f32 v120, v105, v36\n" \
    "v_mul_f32 v122, v102, v85\n" \
    "v_fmac_f32 v122, v105, v38\n" \
    "v_mul_f32 v124, v102, v87\n" \
    "v_fmac_f32 v124, v105, v40\n" \
    "v_fmac_f32 v120, v112, v89\n" \
    "v_fmac_f32 v120, v115, v42\n" \
    "v_fmac_f32 v122, v112, v91\n" \
    "v_fmac_f32 v122, v115, v44\n" \
    "v_fmac_f32 v124, v112, v93\n" \
    "v_fmac_f32 v124, v115, v46\n" \
    "v_add_f32 v35, v35, v52\n" \
    "v_add_f32 v37, v37, v54\n" \
    "v_add_f32 v39, v39, v56\n" \
    "v_add_f32 v41, v41, v58\n" \
    "v_add_f32 v43, v43, v60\n" \
    "v_add_f32 v45, v45, v62\n" \
    "s_nop 1\n" \
    "v_add_f32_dpp v47, v120, v47 row_ror:15 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_add_f32_dpp v49, v122, v49 row_ror:15 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_add_f32_dpp v51, v124, v51 row_ror:15 row_mask:0xf bank_mask:0xf bound_ctrl:1\n" \
    "v_add_f32 v53, v53, v47\n" \
    "v_add_f32 v55, v55, v49\n" \
    "v_add_f32 v57, v57, v51\n" \
    "ds_write_b32 v33, v53 offset:768\n" \
    "ds_write_b32 v33, v55 offset:832\n" \
    "ds_write_b32 v33, v57 offset:896\n" \
    "v_add_f32 v125, v64, v35\n" \
    "v_sub_f32 v126, v125, v64\n" \
    "v_sub_f32 v35, v35, v126\n" \
    "v_mov_b32 v64, v125\n" \
    "v_add_f32 v125, v66, v37\n" \
    "v_sub_f32 v126, v125, v66\n" \
    "v_sub_f32 v37, v37, v126\n" \
    "v_mov_b32 v66, v125\n" \
    "v_add_f32 v125, v68, v39\n" \
    "v_sub_f32 v126, v125, v68\n" \
    "v_sub_f32 v39, v39, v126\n" \
    "v_mov_b32 v68, v125\n" \
    "v_add_f32 v125, v70, v41\n" \
    "v_sub_f32 v126, v125, v70\n" \
    "v_sub_f32 v41, v41, v126\n" \
    "v_mov_b32 v70, v125\n" \
    "v_add_f32 v125, v72, v43\n" \
    "v_sub_f32 v126, v125, v72\n" \
    "v_sub_f32 v43, v43, v126\n" \
    "v_mov_b32 v72, v125\n" \
    "v_add_f32 v125, v74, v45\n" \
    "v_sub_f32 v126, v125, v74\n" \
    "v_sub_f32 v45, v45, v126\n" \
    "v_mov_b32 v74, v125\n"

// pinned operand registers
#define SD_WAVE_R_X0x "{v24}"
#define SD_WAVE_R_FI0x "{v36}"
#define SD_WAVE_R_S0x "{v64}"
#define SD_WAVE_R_Y0x "{v35}"
#define SD_WAVE_R_X0y "{v26}"
#define SD_WAVE_R_FI0y "{v38}"
#define SD_WAVE_R_S0y "{v66}"
#define SD_WAVE_R_Y0y "{v37}"
#define SD_WAVE_R_X0z "{v28}"
#define SD_WAVE_R_FI0z "{v40}"
#define SD_WAVE_R_S0z "{v68}"
#define SD_WAVE_R_Y0z "{v39}"
#define SD_WAVE_R_X1x "{v30}"
#define SD_WAVE_R_FI1x "{v42}"
#define SD_WAVE_R_S1x "{v70}"
#define SD_WAVE_R_Y1x "{v41}"
#define SD_WAVE_R_X1y "{v32}"
#define SD_WAVE_R_FI1y "{v44}"
#define SD_WAVE_R_S1y "{v72}"
#define SD_WAVE_R_Y1y "{v43}"
#define SD_WAVE_R_X1z "{v34}"
#define SD_WAVE_R_FI1z "{v46}"
#define SD_WAVE_R_S1z "{v74}"
#define SD_WAVE_R_Y1z "{v45}"
#define SD_WAVE_R_GAMMA "{v48}"
#define SD_WAVE_R_THR2 "{v50}"
#define SD_WAVE_R_THR2O "{v25}"
#define SD_WAVE_R_INF "{v27}"
#define SD_WAVE_R_M3G "{v29}"
#define SD_WAVE_R_ADDR "{v31}"
#define SD_WAVE_R_JADDR "{v33}"
// clobbered temporaries
#define SD_WAVE_CLOBBERS "v47", "v49", "v51", "v52", "v53", "v54", "v55", "v56", "v57", "v58", "v59", "v60", "v61", "v62", "v63", "v65", "v67", "v69", "v71", "v73", "v75", "v76", "v77", "v78", "v79", "v80", "v81", "v82", "v83", "v84", "v85", "v86", "v87", "v88", "v89", "v90", "v91", "v92", "v93", "v94", "v95", "v96", "v97", "v98", "v99", "v100", "v101", "v102", "v103", "v104", "v105", "v106", "v107", "v108", "v109", "v110", "v111", "v112", "v113", "v114", "v115", "v116", "v117", "v118", "v119", "v120", "v121", "v122", "v123", "v124", "v125", "v126"
// highest register used by the chunk: v126
