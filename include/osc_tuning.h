/*
 * libosc -- kernel-choice overrides for tests and tuning.  Not part of the product interface:
 * the settings change which kernel serves a call, never its result (the parity tests force
 * every kernel through these knobs to show exactly that).  Process-wide; -1 restores the
 * library's own choice.  No entry point of osc.h reads the environment.
 */
#ifndef OSC_TUNING_H
#define OSC_TUNING_H

#ifdef __cplusplus
extern "C" {
#endif

enum {
    OSC_TUNE_GEMM_TILE = 0,        /* tile rows / 64 of the GEMM kernels: 1, 2 or 4; with kernel 7 its tile: 0 128 x 256, 1 128 x 192,
                                      2 128 x 128, 3 64 x 128 */
    OSC_TUNE_GEMM_KERNEL = 1,      /* 0 staged, 1 DMA, 2 persistent, 3 skinny, 4 and 5 ring, 6 streaming, 7 flowing (ignored
                                      where a kernel cannot serve the shape) */
    OSC_TUNE_GROUPED_ONE_TILE = 2, /* accepted, no effect */
    OSC_TUNE_SWIGLU_TABLE = 3,     /* accepted, no effect: the SwiGLU fusions have one kernel each */
    OSC_TUNE_GEMM_KSPLIT = 4       /* accepted, no effect: no kernel splits the K loop of a small tile any more */
};

/* Errors: OSC_ERR_UNSUPPORTED for an unknown knob.  Any negative value means "automatic". */
int osc_tuning_set(int knob, int value);
/* The current setting (-1 = automatic, also for an unknown knob). */
int osc_tuning_get(int knob);
/*
 * What served the calling thread's last GEMM call that launched anything (-1 before the first): kernel id | detail << 8.
 * Ids as above, and 8 the 16-row kernel and 9 the wide kernel of the formats with a scale per 16 channels.  Detail: tile
 * rows / 64 of kernels 0, 1 and 2; wavefronts of a workgroup of kernels 3, 6 and 9; the tile of kernel 7; channels / 16 of a
 * workgroup of kernel 8.  For tests: a forced kernel gives way silently where it cannot serve a shape.
 */
int osc_tuning_last_gemm(void);

#ifdef __cplusplus
}
#endif
#endif /* OSC_TUNING_H */
