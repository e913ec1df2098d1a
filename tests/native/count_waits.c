/* Stands in front of hipStreamSynchronize and counts its calls. */
typedef int (*sync_fn)(void *);
static sync_fn real;
static int calls;

void count_waits_real(void *fn) { real = (sync_fn)fn; }
int count_waits(void) { return calls; }

int hipStreamSynchronize(void *stream)
{
    ++calls;
    return real(stream);
}
